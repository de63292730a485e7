// Host-side view of the library's layouts, for tests without a GPU: the job
// queue, the descriptors and the memory a batch would be given.
#include <cstring>

#include "../paper_2605_28400_amd/csrc/common.h"

using namespace trioseq;

// The layout of a plan (default options, the packed panel jobs allowed: 0 none, 1
// pairs, 2 any). info:
// [0] status, [1] modes, [2] packed, [3] halves, [4] longest sweep, [5] panels
// reported, [6] jobs, [7] descriptors, [8] face pool ints, [9] plane ints,
// [10] single-wave workgroups, [11] engine reported. desc (7 per descriptor,
// up to cap: lens, out, start of the sweep, direction, longest sweep's
// sequence) may be null.
extern "C" void probe_layout(const uint32_t* lens, size_t n, const trioseq_scoring* sc, int panels, int64_t* info,
                             int64_t* desc, size_t cap) {
  const trioseq_plan_options o{-1, 0, 0, 0, 0, 0};
  Layout L;
  info[0] = build_layout(lens, nullptr, n, *sc, o, 256 * kWavesPerCuHint, &L, false, (PackedPanels)panels);
  info[1] = L.modes;
  info[2] = L.packed;
  info[3] = L.halves;
  info[4] = L.lds_n0;
  info[5] = L.panels;
  info[6] = (int64_t)L.jobs.size();
  info[7] = (int64_t)L.desc.size();
  info[8] = (int64_t)L.pool_ints;
  info[9] = (int64_t)L.plane_ints;
  info[10] = L.pk_self;
  info[11] = L.engine;
  if (!desc) return;
  for (size_t d = 0; d < L.desc.size() && d < cap; ++d) {
    const TripletDesc& t = L.desc[d];
    const int64_t row[7] = {t.len[0], t.len[1], t.len[2], t.out, t.start[0], t.rev, 0};
    std::memcpy(desc + 7 * d, row, sizeof row);
  }
}

// Which packed forms a lone triplet of these lengths may take: bit 0 semi-global
// halves, bit 1 a pair with itself (of that kind).
extern "C" int probe_lone(const uint32_t* lens, int kind) {
  return (semi_global_halves(lens) ? 1 : 0) | (self_pair(kind, lens) ? 2 : 0);
}

// What a traceback workspace counts against the bytes that are kept: pinned
// staging of `stage` bytes and `out` split-point ints beside `device` bytes.
extern "C" uint64_t probe_workspace_bytes(uint64_t device, uint64_t stage, uint64_t out) {
  PlaneWorkspace ws;
  ws.tables.bytes = device;
  ws.h_stage_bytes = stage;
  ws.h_out_ints = out;
  return ws_bytes(ws);
}
