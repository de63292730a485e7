"""GPU parity of the layouts that a batch takes by its size and shape: pairs on
unlike grids, many halves, limited memory. Scores are integers, so the bar is
equality with the oracle."""
import numpy as np
import pytest

import oracle
import paper_2605_28400_amd as ts
from paper_2605_28400_amd import synth

pytestmark = pytest.mark.gpu
KINDS = [ts.GLOBAL, ts.SEMI_GLOBAL, ts.LOCAL]
KIND_IDS = ["global", "semi-global", "local"]
OKIND = {ts.GLOBAL: oracle.GLOBAL, ts.SEMI_GLOBAL: oracle.SEMI_GLOBAL, ts.LOCAL: oracle.LOCAL}


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def run_words(torch, lens, off, d_words, sc, reps=2, **opts):
    plan = ts.Plan(lens, off, sc=sc, **opts)
    outs = []
    for _ in range(reps):
        d_scores = torch.full((len(lens) // 3,), -7, dtype=torch.int32, device="cuda")
        plan.run(d_words, d_scores)
        torch.cuda.synchronize()
        outs.append(d_scores.cpu().numpy().copy())
    info = plan.info()
    plan.close()
    return outs, info


def test_halves_that_do_not_fit_run_in_pairs(torch_cuda):
    torch = torch_cuda
    # 4000 triplets of independent lengths up to 1200: halves, whose planes and
    # faces take 16 GB; the pairs' faces take 9.
    rng = np.random.default_rng(91)
    lens = rng.integers(200, 1201, (4000, 3)).astype(np.uint32).reshape(-1)
    nw = (lens.astype(np.int64) + 15) // 16
    off = np.concatenate([[0], np.cumsum(nw)[:-1]]).astype(np.uint64)
    words = rng.integers(0, 2**32, int(nw.sum()), dtype=np.uint32)
    d_words = torch.from_numpy(words.view(np.int32)).cuda()
    sc = ts.scoring()
    print("halves with room", flush=True)
    free_run, roomy = run_words(torch, lens, off, d_words, sc, reps=1)
    free, _ = torch.cuda.mem_get_info()
    need = roomy["workspace_bytes"]
    assert need > 14 << 30
    hold = torch.empty(free - need + (2 << 30), dtype=torch.uint8, device="cuda")
    try:
        print("pairs without", flush=True)
        outs, info = run_words(torch, lens, off, d_words, sc, reps=2)
    finally:
        del hold
        torch.cuda.empty_cache()
    assert info["packed"] == 1 and info["panels"] > 0 and info["workspace_bytes"] < need - (2 << 30)
    assert all((o == free_run[0]).all() for o in outs)
    # (A few against the oracle: the shortest.)
    few = np.argsort(lens.reshape(-1, 3).astype(np.int64).prod(axis=1))[:40]
    codes = ((words[:, None] >> (2 * np.arange(16, dtype=np.uint32))) & 3).astype(np.uint8)
    trips = [tuple(codes[int(off[3 * t + s]):int(off[3 * t + s]) + int(nw[3 * t + s])].reshape(-1)[:lens[3 * t + s]]
                   for s in range(3)) for t in few]
    assert free_run[0][few].tolist() == oracle.score_batch(trips).tolist()


def run(torch, trips, sc, reps=2, **opts):
    lens, off, words = ts.pack_batch(trips)
    return run_words(torch, lens, off, torch.from_numpy(words.view(np.int32)).cuda(), sc, reps, **opts)


def want_scores(trips, scheme, kind):
    sub = [[scheme[0] if x == y else scheme[1] for y in range(4)] for x in range(4)]
    return np.asarray(oracle.score_batch(trips, sub, scheme[2], kind=OKIND[kind]), dtype=np.int64)


def halves_panels(trips):
    # Panels of both halves of every triplet: the longest sequence is cut.
    grid = [sorted(len(s) for s in t)[:2] for t in trips]
    return 2 * sum((a // 32 + 1) * (b // 32 + 1) for a, b in grid)


# Odd counts of unlike shapes, so that neighbours in the order of pairs have
# other grids than their partners: empty axes, one row or column, panel edges.
SHAPES = [((300, 5, 70), 151), ((0, 90, 120), 151), ((64, 64, 64), 151), ((1, 1, 200), 151), ((33, 200, 2), 151),
          ((0, 0, 0), 151), ((96, 0, 33), 151), ((140, 100, 20), 151), ((140, 40, 90), 151), ((70, 66, 65), 151),
          ((70, 95, 5), 151), ((100, 97, 103), 151), ((130, 31, 32), 151), ((32, 31, 33), 151), ((220, 210, 215), 7)]


@pytest.mark.parametrize("scheme", [(1, -1, -2), (5, -4, -6)])
@pytest.mark.parametrize("kind", KINDS, ids=KIND_IDS)
def test_pairs_of_unlike_shapes(torch_cuda, kind, scheme):
    rng = np.random.default_rng(92)
    trips = [tuple(synth.uniform_seq(rng, m) for m in n) for n, count in SHAPES for _ in range(count)]
    trips += [synth.mutated_triplet(rng, int(n), 0.1) for n in rng.integers(20, 150, 100)]
    assert len(trips) % 2 == 1  # the last one pairs with itself
    want = want_scores(trips, scheme, kind)
    for graph in (False, True):
        print(f"unlike pairs kind={kind} scheme={scheme} graph={graph}", flush=True)
        outs, info = run(torch_cuda, trips, ts.scoring(*scheme, kind=kind), reps=3, use_graph=graph)
        assert info["packed"] == 1 and 0 < info["panels"] != halves_panels(trips)
        for got in outs:
            bad = np.flatnonzero(got != want)
            assert bad.size == 0, [(int(q), int(got[q]), int(want[q]), [len(s) for s in trips[q]]) for q in bad[:5]]


def many_halves(rng):
    # Long thin triplets, each axis the long one in turn: by halves 8 panels a
    # triplet, in three groups.
    trips = []
    for q in range(3200):
        n = [int(m) for m in rng.integers(33, 63, 3)]
        n[q % 3] = int(rng.integers(300, 600))
        trips.append(tuple(synth.uniform_seq(rng, m) for m in n) if q % 2 else
                     synth.mutated_triplet(rng, max(n), 0.1, lens=tuple(n)))
    return trips


@pytest.mark.parametrize("kind", KINDS, ids=KIND_IDS)
def test_many_halves_share_face_buffers(torch_cuda, kind):
    trips = many_halves(np.random.default_rng(93))
    want = want_scores(trips, (1, -1, -2), kind)
    for graph in (False, True):
        print(f"many halves kind={kind} graph={graph}", flush=True)
        outs, info = run(torch_cuda, trips, ts.scoring(kind=kind), reps=3, use_graph=graph)
        assert info["packed"] == 1 and info["panels"] == halves_panels(trips) == 8 * len(trips)
        assert all(np.array_equal(got, want) for got in outs)


@pytest.mark.parametrize("form", ["pairs", "halves"])
def test_waits_that_give_up_while_buffers_are_shared(torch_cuda, form):
    # A wait bound of one clock tick: panels whose neighbour, or whose buffers'
    # earlier group, is not ready give up; every kernel ends, no score is wrong,
    # and the next run is whole again.
    rng = np.random.default_rng(94)
    trips = many_halves(rng) if form == "halves" else [synth.mutated_triplet(rng, int(n), 0.1)
                                                       for n in rng.integers(40, 75, 9000)]
    want = want_scores(trips, (1, -1, -2), ts.GLOBAL)
    lens, off, words = ts.pack_batch(trips)
    torch = torch_cuda
    d_words = torch.from_numpy(words.view(np.int32)).cuda()
    plan = ts.Plan(lens, off)
    assert plan.info()["packed"] == 1 and (plan.info()["panels"] == halves_panels(trips)) == (form == "halves")

    def once():
        d_scores = torch.full((len(trips),), -7, dtype=torch.int32, device="cuda")
        plan.run(d_words, d_scores)
        torch.cuda.synchronize()
        return d_scores.cpu().numpy()

    print(f"waits give up: {form}", flush=True)
    try:
        ts.set_wait_limit(10)
        got = once()
    finally:
        ts.set_wait_limit(0)
    assert ((got == want) | (got == -2**31)).all() and (got == -2**31).any()
    assert np.array_equal(once(), want) and np.array_equal(once(), want)
    plan.close()


# (kind, match, mismatch, gap, the longest cube that 16 bits admit, its score):
# what binds is M' itself (20 per residue of a half, below 2^16); a score's
# distance from the floors (20 per residue pair of a half, up to 30000); and the
# offset of semi-global candidates (20 per index of the padded half, below 2^16).
LIMITS = [(ts.LOCAL, 4, -4, -8, 1310, 12 * 1310), (ts.LOCAL, 20, 0, 0, 750, 60 * 750),
          (ts.SEMI_GLOBAL, 20, 0, 0, 750, 60 * 750), (ts.SEMI_GLOBAL, 0, -5, -10, 1304, 0)]


@pytest.mark.parametrize("kind,match,mismatch,gap,n,score", LIMITS)
def test_values_up_to_their_limits(torch_cuda, kind, match, mismatch, gap, n, score):
    # All-equal residues, so that values grow as fast as they can; the score of
    # a cube is then three matches a column (0 where a match is worth nothing).
    sc = ts.scoring(match, mismatch, gap, kind=kind)
    for m, packed in ((n, 1), (n + 2, 0)):
        x = np.full(m, 3, np.uint8)
        print(f"limit kind={kind} match={match} gap={gap} n={m}", flush=True)
        outs, info = run(torch_cuda, [(x, x, x)], sc)
        assert info["packed"] == packed, (m, info)
        assert [int(o[0]) for o in outs] == [3 * match * m] * 2
    assert 3 * match * n == score
    # Unlike residues at the limit, thin enough for the oracle.
    rng = np.random.default_rng(95)
    t = synth.mutated_triplet(rng, n, 0.2, lens=(n, 64, 95))
    outs, info = run(torch_cuda, [t], sc)
    assert info["packed"] == 1 and (outs[0] == want_scores([t], (match, mismatch, gap), kind)).all()


def test_tags_start_over_before_they_leave_31_bits(torch_cuda):
    torch = torch_cuda
    import ctypes
    prepare = getattr(ts.lib(), "_ZN7trioseq14launch_prepareEPiS0_S0_jS0_miP12ihipStream_t")
    prepare.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_uint32, ctypes.c_void_p, ctypes.c_uint64, ctypes.c_int,
                                                ctypes.c_void_p]
    prepare.restype = ctypes.c_int
    always, step, ints = 0x7FFFFFFF, 1000, 70001
    for last, wraps in ((0, False), (5000, False), (always - 2 * step - 1, False), (always - 2 * step, True),
                        (always - 1, True)):
        ctl = torch.tensor([7, 1, 0, last] + [9] * 60, dtype=torch.int32, device="cuda")
        counter = torch.full((96,), 5, dtype=torch.int32, device="cuda")
        red = torch.full((20,), 3, dtype=torch.int32, device="cuda")
        pool = torch.full((ints + 64,), last, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        print(f"tags last={last}", flush=True)
        st = prepare(ctl.data_ptr(), counter.data_ptr(), red.data_ptr(), 10, pool.data_ptr(), ints, step,
                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert st == 0
        first = 1 if wraps else last + 1
        assert ctl[:4].tolist() == [first, 0, 0, first + step - 1] and first + step - 1 < always
        assert counter[0] == 0 and counter[32] == 0 and counter[64] == 0
        assert (pool[:ints] == (0 if wraps else last)).all() and (pool[ints:] == last).all()


@pytest.mark.parametrize("kind", KINDS, ids=KIND_IDS)
def test_autotuner_holds_packed_lanes_against_int32(torch_cuda, monkeypatch, capfd, kind):
    # A lone triplet runs packed by default: its reference is the int32 form, the
    # defaults a candidate.
    torch = torch_cuda
    rng = np.random.default_rng(96)
    t = synth.mutated_triplet(rng, 600, 0.1, lens=(600, 66, 70))
    lens, off, words = ts.pack_batch([t])
    d_words = torch.from_numpy(words.view(np.int32)).cuda()
    monkeypatch.setenv("TRIOSEQ_TUNE_LOG", "1")
    print(f"autotune lone kind={kind}", flush=True)
    capfd.readouterr()
    res = ts.autotune(lens, off, d_words, sc=ts.scoring(kind=kind), reps=2)
    log = [line.split() for line in capfd.readouterr().err.splitlines() if line.startswith("autotune:")]
    packed = [line[line.index("packed") + 1] for line in log]
    assert packed[:2] == ["0", "1"] and len(log) == res["tried"] and res["rejected"] == 0
    default_ms = float(log[1][-2])
    assert abs(res["reference_ms"] - default_ms) < 1e-4 and res["best_ms"] <= res["reference_ms"] + 1e-9
    outs, _ = run(torch, [t], ts.scoring(kind=kind))  # (with what was remembered)
    assert (outs[0] == want_scores([t], (1, -1, -2), kind)).all()
