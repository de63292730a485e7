"""GPU parity of packed panel jobs: two triplets (or the halves of one) swept
panel by panel, two 16-bit values per register, every panel's values relative
to its own base. Scores are integers, so the bar is equality with the oracle.
"""
import numpy as np
import pytest

import oracle
import paper_2605_28400_amd as ts
from paper_2605_28400_amd import synth

pytestmark = pytest.mark.gpu
OKIND = {ts.GLOBAL: oracle.GLOBAL, ts.SEMI_GLOBAL: oracle.SEMI_GLOBAL, ts.LOCAL: oracle.LOCAL}
SCHEMES = [(1, -1, -2), (5, -4, -6), (2, 0, -1)]  # match, mismatch, gap


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def run(torch, trips, sc, reps=2, **opts):
    lens, off, words = ts.pack_batch(trips)
    plan = ts.Plan(lens, off, sc=sc, **opts)
    d_words = torch.from_numpy(words.view(np.int32)).cuda()
    outs = []
    for _ in range(reps):
        d_scores = torch.full((len(trips),), -7, dtype=torch.int32, device="cuda")
        plan.run(d_words, d_scores)
        torch.cuda.synchronize()
        outs.append(d_scores.cpu().numpy().copy())
    info = plan.info()
    plan.close()
    return outs, info


def want_scores(trips, scheme, kind):
    sub = [[scheme[0] if x == y else scheme[1] for y in range(4)] for x in range(4)]
    return np.asarray(oracle.score_batch(trips, sub, scheme[2], kind=OKIND[kind]), dtype=np.int64)


# Panel edges (31, 32, 33 and multiples), a lone row or column, empty axes,
# halves of equal and unequal length.
LONE = [(128, 31, 32), (129, 33, 63), (200, 64, 1), (257, 0, 40), (300, 0, 0), (190, 191, 188), (420, 95, 130)]


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("kind", [ts.GLOBAL, ts.LOCAL], ids=["global", "local"])
def test_lone_halves_equal_oracle(torch_cuda, kind, scheme):
    rng = np.random.default_rng(81)
    sc = ts.scoring(*scheme, kind=kind)
    for q, n in enumerate(LONE):
        t = synth.mutated_triplet(rng, max(n), 0.1, lens=n) if q % 2 else tuple(synth.uniform_seq(rng, m) for m in n)
        want = want_scores([t], scheme, kind)
        print(f"lone halves kind={kind} scheme={scheme} lens={n}", flush=True)
        for graph in (False, True):
            outs, info = run(torch_cuda, [t], sc, reps=3, use_graph=graph)
            assert info["packed"] == 1 and info["engine"] == 1
            assert all((o == want).all() for o in outs), (n, outs, want)
        outs, info = run(torch_cuda, [t], sc, packed=1)
        assert info["packed"] == 0 and (outs[0] == want).all()


@pytest.mark.parametrize("na,packed", [(1588, 1), (1594, 0)])
@pytest.mark.parametrize("kind", [ts.GLOBAL, ts.LOCAL], ids=["global", "local"])
def test_window_limit(torch_cuda, kind, na, packed):
    # Terms of up to 17 per residue pair: a panel's window of a half of 794
    # residues just fits 16 bits, one of 797 does not (int32 lanes). All-equal
    # residues make the values grow as fast as they can.
    sc = ts.scoring(5, -4, -6, kind=kind)
    t = tuple(np.full(n, 1, np.uint8) for n in (na, 70, 65))
    print(f"window kind={kind} na={na}", flush=True)
    outs, info = run(torch_cuda, [t], sc)
    assert info["packed"] == packed
    assert (outs[0] == want_scores([t], (5, -4, -6), kind)).all()


@pytest.mark.parametrize("lens,packed", [((1588, 70, 65), 1), ((1594, 70, 65), 0), ((640, 600, 610), 1)])
def test_semi_global_window(torch_cuda, lens, packed):
    # As above; the third puts the faces' values far below the panels' windows.
    t = tuple(np.full(n, 1, np.uint8) for n in lens)
    print(f"semi-global window lens={lens}", flush=True)
    outs, info = run(torch_cuda, [t], ts.scoring(5, -4, -6, kind=ts.SEMI_GLOBAL))
    assert info["packed"] == packed
    assert (outs[0] == want_scores([t], (5, -4, -6), ts.SEMI_GLOBAL)).all()


def test_largest_values(torch_cuda):
    # 17 per residue pair and all-equal residues: a half's values reach 17 *
    # (645 + 645 + 1290) of the 65535 that 16 bits recover.
    for n in (1270, 1290):
        x = np.full(n, 2, np.uint8)
        print(f"values n={n}", flush=True)
        outs, info = run(torch_cuda, [(x, x, x)], ts.scoring(5, -4, -6))
        assert info["packed"] == 1 and int(outs[0][0]) == 15 * n  # 3 pairs of 5 per column


def batches(rng):
    def mut(n):
        return synth.mutated_triplet(rng, int(n), 0.1)

    def uni(*n):
        return tuple(synth.uniform_seq(rng, m) for m in n)

    return {"two": [mut(100), mut(60)],
            "odd count": [mut(100), mut(130), mut(20)],
            "one large": [mut(220)] + [mut(n) for n in rng.integers(5, 60, 40)],
            "shapes": [uni(300, 5, 70), uni(0, 90, 120), uni(64, 64, 64), uni(1, 1, 200), uni(33, 200, 2),
                       uni(0, 0, 0), uni(96, 0, 33)],
            "halves": [mut(n) for n in (420, 400, 380)],
            # Partners whose common grid is larger than either.
            "crossed": [uni(140, 100, 20), uni(140, 40, 90), uni(70, 66, 65), uni(70, 95, 5)],
            # More panels a diagonal than a group of pairs takes: three groups
            # or more, whose faces share two sets of buffers.
            "groups": [mut(n) for n in rng.integers(40, 75, 9000)]}


@pytest.mark.parametrize("name", ["two", "odd count", "one large", "shapes", "halves", "crossed", "groups"])
@pytest.mark.parametrize("kind", [ts.GLOBAL, ts.SEMI_GLOBAL, ts.LOCAL], ids=["global", "semi-global", "local"])
def test_batches_equal_oracle(torch_cuda, kind, name):
    trips = batches(np.random.default_rng(82))[name]
    for scheme in SCHEMES[:1] if name == "groups" else SCHEMES:
        want = want_scores(trips, scheme, kind)
        for graph in (False, True):
            print(f"batch kind={kind} {name} scheme={scheme} graph={graph}", flush=True)
            outs, info = run(torch_cuda, trips, ts.scoring(*scheme, kind=kind), reps=3, use_graph=graph)
            assert info["packed"] == 1 and info["panels"] > 0
            for got in outs:
                bad = np.flatnonzero(got != want)
                assert bad.size == 0, [(int(q), int(got[q]), int(want[q])) for q in bad[:5]]


# (With inner axes 40 x 33 the axis of 33 is swept, with 63 x 63 the longest.)
@pytest.mark.parametrize("longest,inner,grid", [(512, (40, 33), 3072), (513, (40, 33), 3072),
                                                (512, (63, 63), 3072), (513, (63, 63), 2048)])
def test_many_short_panels(torch_cuda, longest, inner, grid):
    """Three waves a SIMD from 32768 panel jobs on, for sweeps up to 512."""
    rng = np.random.default_rng(85)
    some = [tuple(synth.uniform_seq(rng, int(m)) for m in rng.integers(32, 64, 3)) for _ in range(62)]
    some += [tuple(synth.uniform_seq(rng, m) for m in n) for n in ((longest, *inner), (63, 32, 63))]
    want = want_scores(some, (1, -1, -2), ts.GLOBAL)
    outs, info = run(torch_cuda, [some[q % 64] for q in range(16640)], ts.scoring(), use_graph=True)
    cus = torch_cuda.cuda.get_device_properties(0).multi_processor_count
    assert info["packed"] == 1 and info["grid"] == grid * cus // 256
    for got in outs:
        assert np.array_equal(got, np.tile(want, 260))


def test_lone_semi_global(torch_cuda):
    rng = np.random.default_rng(83)
    for n in LONE:
        t = synth.mutated_triplet(rng, max(n), 0.1, lens=n)
        print(f"lone semi-global lens={n}", flush=True)
        for scheme in SCHEMES:
            outs, _ = run(torch_cuda, [t], ts.scoring(*scheme, kind=ts.SEMI_GLOBAL))
            assert all((o == want_scores([t], scheme, ts.SEMI_GLOBAL)).all() for o in outs)


@pytest.mark.parametrize("where", ["first half", "second half", "across", "nowhere", "other axes"])
def test_lone_semi_global_halves(torch_cuda, where):
    """Alignments that start and end in either half, on every axis and face."""
    rng = np.random.default_rng(86)
    seq = lambda m: synth.uniform_seq(rng, m)
    for scheme in ((1, -1, -2), (5, -4, -6), (1, -3, 0)):
        for q, m in enumerate((20, 60, 97, 70, 130)):
            core = synth.mutated_triplet(rng, m, 0.05, lens=(m, m, m))
            pre, post = {"first half": (0, 170 - m), "second half": (170 - m, 0), "across": (85 - m // 2, 60),
                         "nowhere": (90, 90), "other axes": (0, 170)}[where]
            if where == "other axes":  # a ends in the core that b and c start late
                a = np.concatenate([core[0], seq(post)])
                b, c = np.concatenate([seq(33 * q), core[1]]), np.concatenate([seq(31), core[2]])
            else:
                a = np.concatenate([seq(pre), core[0], seq(post)])
                b, c = (seq(m), seq(m)) if where == "nowhere" else (core[1], core[2])
            for t in ((a, b, c), (b, c, a)):
                print(f"semi-global halves {where} scheme={scheme} lens={[len(z) for z in t]}", flush=True)
                want = want_scores([t], scheme, ts.SEMI_GLOBAL)
                outs, info = run(torch_cuda, [t], ts.scoring(*scheme, kind=ts.SEMI_GLOBAL))
                assert all((o == want).all() for o in outs)
                # (A negative term, mismatch - 2 gap, keeps int32 lanes; thin ones are one sweep.)
                lo, mid, _ = sorted(len(z) for z in t)
                if scheme[1] - 2 * scheme[2] >= 0 and (lo // 32 + 1) * (mid // 32 + 1) >= 9:
                    assert info["packed"] == 1 and info["panels"] == 2 * (lo // 32 + 1) * (mid // 32 + 1)


def test_bounded_wait_gives_int32_min(torch_cuda):
    # A wait bound of one clock tick: a panel whose neighbour is not there yet
    # gives up at once, every kernel ends, and no score but INT32_MIN comes
    # back; the plan works again afterwards.
    rng = np.random.default_rng(84)
    t = synth.mutated_triplet(rng, 400, 0.05, lens=(400, 380, 390))
    want = int(want_scores([t], SCHEMES[0], ts.GLOBAL)[0])
    try:
        ts.set_wait_limit(10)
        outs, info = run(torch_cuda, [t], ts.scoring())
    finally:
        ts.set_wait_limit(0)
    assert info["packed"] == 1 and all(int(o[0]) in (-2**31, want) for o in outs)
    assert any(int(o[0]) == -2**31 for o in outs)
    outs, _ = run(torch_cuda, [t], ts.scoring())
    assert all(int(o[0]) == want for o in outs)
