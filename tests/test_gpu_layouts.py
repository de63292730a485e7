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
