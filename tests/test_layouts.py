"""CPU checks of the layouts plans are given: which form of the kernels a batch
takes, and the limits of each."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2605_28400_amd as ts

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ["status", "modes", "packed", "halves", "sweep", "panels", "jobs", "descs", "pool", "planes", "single_wave",
          "engine"]
WHOLE, PK_PANEL = 1, 4  # Layout::modes of whole-triplet jobs and of packed panel jobs
MAX_SWEEP = 16384
KINDS = [ts.GLOBAL, ts.SEMI_GLOBAL, ts.LOCAL]
KIND_IDS = ["global", "semi-global", "local"]


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("probe") / "layout_probe.so")
    lib = os.path.join(os.path.dirname(HERE), "paper_2605_28400_amd", "libtrioseq.so")
    ts.lib()
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "layout_probe.cpp"), lib, "-o", out], check=True)
    return ctypes.CDLL(out)


def layout(probe, lens, sc=None, panels=2):
    lens = np.ascontiguousarray(np.asarray(lens, dtype=np.uint32).reshape(-1))
    info = np.zeros(len(FIELDS), dtype=np.int64)
    probe.probe_layout(lens.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(lens.size // 3),
                       ctypes.byref(sc or ts.scoring()), ctypes.c_int(panels), info.ctypes.data_as(ctypes.c_void_p),
                       None, ctypes.c_size_t(0))
    return dict(zip(FIELDS, info.tolist()))


@pytest.mark.parametrize("inner", [40, 300])
def test_no_sweep_beyond_the_longest_the_kernels_hold(probe, inner):
    # Every term 0 (sub = 2 * gap): values never grow, so only the sweep's
    # length bounds the packed forms.
    sc = ts.scoring(-2, -2, -1)
    for longest in (2 * MAX_SWEEP, 2 * MAX_SWEEP + 2, 100000):
        got = layout(probe, [(longest, inner, inner)] * 2, sc)
        assert got["status"] == 0 and got["sweep"] <= MAX_SWEEP, (longest, got)


# Small and thin triplets: what the default options take (measured times beside
# the rule). "pairs" and "halves" are panel jobs.
@pytest.mark.parametrize("n,lens,form", [
    (2, (20, 20, 20), "whole"), (20000, (20, 20, 20), "whole"), (2048, (128, 20, 20), "whole"),
    (512, (128, 31, 31), "whole"), (64, (128, 31, 31), "halves"), (1024, (500, 31, 31), "halves"),
    (1300, (500, 31, 31), "whole"), (2000, (32, 32, 32), "whole"), (2300, (32, 32, 32), "pairs"),
    (30000, (32, 32, 32), "whole"), (600, (63, 63, 63), "pairs"), (8192, (128, 128, 128), "pairs")])
@pytest.mark.parametrize("kind", KINDS, ids=KIND_IDS)
def test_which_form_a_batch_takes(probe, kind, n, lens, form):
    got = layout(probe, [lens] * n, ts.scoring(kind=kind))
    assert got["status"] == 0 and got["packed"] == 1
    assert got["modes"] == (WHOLE if form == "whole" else PK_PANEL), got
    assert got["halves"] == (form == "halves"), got
    if lens[1] < 32 and form == "halves":  # no faces to move: one wave a workgroup
        assert got["single_wave"] == 1


def test_unlike_lengths_stay_panel_jobs(probe):
    rng = np.random.default_rng(3)
    anc = rng.uniform(100, 400, 8192)
    assert layout(probe, np.rint(anc[:, None] * rng.uniform(0.97, 1.03, (8192, 3))))["modes"] == PK_PANEL
    assert layout(probe, rng.integers(5, 61, (4096, 3)))["modes"] == PK_PANEL
    assert layout(probe, rng.integers(5, 61, (8192, 3)))["modes"] == WHOLE


@pytest.mark.parametrize("lens,halves,pair", [
    ((723, 651, 698), 1, 1), ((130, 64, 64), 1, 1), ((127, 40, 40), 0, 1), ((128, 40, 40), 0, 0), ((2047, 40, 40), 0, 0),
    ((128, 63, 95), 0, 0), ((16384, 64, 64), 1, 1), ((16385, 64, 64), 0, 1), ((64, 30000, 64), 0, 1),
    ((24000, 20, 20), 0, 1)])
def test_which_form_a_lone_semi_global_triplet_may_take(probe, lens, halves, pair):
    got = probe.probe_lone((ctypes.c_uint32 * 3)(*lens), ts.SEMI_GLOBAL)
    assert (got & 1, got >> 1) == (halves, pair)


def test_only_short_lone_triplets_of_the_other_kinds_pair_with_themselves(probe):
    for kind in (ts.GLOBAL, ts.LOCAL):
        for lens, pair in (((127, 120, 126), 1), ((128, 120, 126), 0), ((20000, 20, 20), 0), ((1000, 900, 950), 0)):
            assert probe.probe_lone((ctypes.c_uint32 * 3)(*lens), kind) >> 1 == pair


def descriptors(probe, lens, sc=None):
    lens = np.ascontiguousarray(np.asarray(lens, dtype=np.uint32).reshape(-1))
    info = np.zeros(len(FIELDS), dtype=np.int64)
    desc = np.zeros((2 * lens.size, 7), dtype=np.int64)
    probe.probe_layout(lens.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(lens.size // 3),
                       ctypes.byref(sc or ts.scoring()), ctypes.c_int(2), info.ctypes.data_as(ctypes.c_void_p),
                       desc.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(len(desc)))
    got = dict(zip(FIELDS, info.tolist()))
    return got, desc[:got["descs"]]


@pytest.mark.parametrize("n", [255, 256, 257, 1001, 4096])  # sorted by comparison, or byte by byte
def test_panel_pairs_are_neighbours_by_panels_then_slices(probe, n):
    rng = np.random.default_rng(n)
    lens = rng.integers(150, 250, (n, 3))
    got, desc = descriptors(probe, lens)
    assert got["modes"] == PK_PANEL and not got["halves"] and got["descs"] == n + n % 2
    pj, pk = desc[:, 1] // 32 + 1, desc[:, 2] // 32 + 1
    keys = list(zip((pj * pk).tolist(), pj.tolist(), desc[:, 0].tolist()))
    assert keys == sorted(keys, reverse=True)
    assert sorted(desc[:n, 3].tolist()) == list(range(n)) and desc[-1, 3] == desc[n - 1, 3]
    assert (np.sort(desc[:n, :3], axis=1) == np.sort(lens[desc[:n, 3]], axis=1)).all()


@pytest.mark.parametrize("lens,columns,rows", [((90, 31, 31), 0, 0), ((200, 40, 31), 0, 1), ((200, 31, 40), 1, 0),
                                               ((200, 40, 40), 1, 1), ((200, 64, 40), 1, 2), ((200, 95, 95), 2, 2)])
def test_a_pair_has_only_the_face_buffers_its_panels_write(probe, lens, columns, rows):
    # Halves of a lone pair of equal triplets: two pairs in one group. columns:
    # bottom-face buffers a panel column has, rows: right-face buffers a panel row.
    got, desc = descriptors(probe, [lens] * 2)
    assert got["modes"] == PK_PANEL and got["halves"]
    want = 0
    for n0, n1, n2 in desc[::2, :3].tolist():
        n0 = max(n0, lens[0] - n0)
        face_rows = (n0 + 1 + 14 + 16 + 7) // 8 * 8
        pj, pk = n1 // 32 + 1, n2 // 32 + 1
        assert (min(pj - 1, 2), min(pk - 1, 2)) in ((columns, rows), (rows, columns))
        want += face_rows * (min(pj - 1, 2) * pk * 64 + min(pk - 1, 2) * pj * 66)
    assert got["pool"] == want


def test_halves_keep_to_a_quarter_of_the_device(probe):
    # Independent lengths, which halves suit: their planes (two of rows x columns
    # for every triplet, all at once) grow with the batch, the pairs' faces do not.
    rng = np.random.default_rng(5)
    lens = rng.integers(200, 2401, (12000, 3))
    few = layout(probe, lens[:600])
    assert few["halves"] == 1 and few["planes"] * 4 > 4e9
    many = layout(probe, lens)
    assert many["modes"] == PK_PANEL and many["halves"] == 0 and many["planes"] == 0
    assert many["pool"] * 4 < 64e9
    # What a plan or a served round falls back to where even the few do not fit.
    pairs = layout(probe, lens[:600], panels=1)
    assert pairs["modes"] == PK_PANEL and pairs["halves"] == 0 and pairs["planes"] == 0
    assert layout(probe, lens[:600], panels=0)["modes"] != PK_PANEL


def test_a_kept_workspace_counts_its_pinned_memory(probe):
    probe.probe_workspace_bytes.restype = ctypes.c_uint64
    probe.probe_workspace_bytes.argtypes = [ctypes.c_uint64] * 3
    assert probe.probe_workspace_bytes(5000, 3000, 100) == 5000 + 3000 + 400
