"""Performance cases of the triplet aligner: what a user's program runs.

Each case goes through a public entry point of the Python binding (score,
score_batch, Plan.run, align, align_batch, Server) on sequences that the seed
determines. A case fixes the lengths and the entry point; the seed fixes the
residues. Sequences are descendants of one random ancestor (substitutions and
short insertions and deletions), as aligned sequences are in practice, cut or
extended to the lengths of the case.

    listed()             the cases, each with a name
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs on the GPU (or host text, where the entry point
                         takes host text) and the plan or server that is kept
    run(state)           one pass
    work(case)           bytes and operations a pass cannot do without
    exact(case, seed)    the outputs by a plain 64-bit dynamic program
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2605_28400_amd as ts

KINDS = {"global": ts.GLOBAL, "semi-global": ts.SEMI_GLOBAL, "local": ts.LOCAL}
LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)

# (match, mismatch, gap): the library's default first; two schemes with larger
# terms; one whose mismatch costs more than two gaps.
SCHEMES = [(1, -1, -2), (2, -1, -2), (5, -4, -6), (1, -3, -1)]


def _case(name, entry, lens=(), count=1, lo=0, hi=0, log_uniform=False, kind="global",
          graph=False, scheme=0, lens_seed=0):
    return {"name": name, "entry": entry, "a": lens[0] if lens else 0, "b": lens[1] if lens else 0,
            "c": lens[2] if lens else 0, "count": count, "lo": lo, "hi": hi,
            "log_uniform": log_uniform, "kind": kind, "graph": graph, "scheme": scheme,
            "lens_seed": lens_seed}


def listed():
    return [
        # One short triplet from text to score: an interactive or scripted
        # call, bound by launches and copies.
        _case("score_48", "score", (48, 45, 51)),
        # The smallest triplet of the benchmark, scored again and again from
        # device memory by a kept plan with graph replay.
        _case("plan_128", "plan", (128, 128, 128), graph=True),
        # The benchmark's gene-length triplet, one at a time, global.
        _case("plan_1k", "plan", (1024, 1000, 1048)),
        # The same search for a shared region: local scoring.
        _case("plan_1k_local", "plan", (1024, 1000, 1048), kind="local"),
        # Overlapping reads of odd lengths: semi-global scoring.
        _case("plan_700_semi", "plan", (723, 651, 698), kind="semi-global"),
        # The largest lone triplet of the benchmark.
        _case("plan_4k", "plan", (4096, 4000, 4150)),
        # The benchmark's batch: 8192 triplets resident in device memory.
        _case("batch_8192", "plan", count=8192, lo=100, hi=400, lens_seed=3),
        # A mid-sized batch under local scoring, an odd count.
        _case("batch_1999_local", "plan", count=1999, lo=100, hi=400, kind="local", lens_seed=4),
        # A library call on host text: a few hundred short reads.
        _case("score_batch_500", "score_batch", count=500, lo=30, hi=150, lens_seed=5),
        # The alignment itself (traceback) of the gene-length triplet.
        _case("align_1k", "align", (1024, 1000, 1048)),
        # Alignments of many short triplets in one call.
        _case("align_batch_1000", "align_batch", count=1000, lo=8, hi=64, lens_seed=6),
        # A service under load: requests of mixed lengths submitted to the
        # server, every result waited for.
        _case("served_500", "served", count=500, lo=64, hi=2048, log_uniform=True, lens_seed=7),
    ]


def draw(rng):
    """One more case: entry points as listed, lengths log-uniform over the
    listed ranges, kinds, schemes and odd sizes mixed."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    entry = rng.choice(["score", "plan", "plan", "plan", "batch", "batch", "score_batch", "align",
                        "align_batch", "served"])
    kind = rng.choice(["global", "global", "global", "semi-global", "local"])
    scheme = rng.choice([0, 0, 0, 0, 1, 2, 3])
    seed = rng.randrange(1 << 30)
    if entry == "batch":
        hi = log_int(60, 500)
        lo = max(1, int(hi * rng.uniform(0.2, 0.9)))
        count = min(log_int(64, 8192), max(64, int(1.7e11 / hi ** 3)))
        c = _case("", "plan", count=count, lo=lo, hi=hi, kind=kind, scheme=scheme, lens_seed=seed,
                  graph=rng.random() < 0.5)
    elif entry == "score_batch":
        hi = log_int(30, 300)
        c = _case("", entry, count=log_int(16, 2000), lo=max(1, hi // 5), hi=hi, kind=kind, scheme=scheme,
                  lens_seed=seed)
    elif entry == "align_batch":
        hi = log_int(10, 100)
        c = _case("", entry, count=log_int(64, 1000), lo=max(1, hi // 8), hi=hi, scheme=scheme, lens_seed=seed)
    elif entry == "served":
        c = _case("", entry, count=log_int(64, 500), lo=64, hi=log_int(200, 2048), log_uniform=True, kind=kind,
                  lens_seed=seed)
    else:
        n = log_int(30, 400) if entry == "score" else log_int(100, 1600 if entry == "align" else 4000)
        lens = tuple(max(1, int(n * rng.uniform(0.85, 1.03))) for _ in range(3))
        if entry == "align":
            kind = "global"
        c = _case("", entry, lens, kind=kind, scheme=scheme, graph=entry == "plan" and rng.random() < 0.5)
    del c["name"]
    return c


def _lengths(case):
    """The triplets' lengths, an array of (count, 3): the case alone."""
    if case["count"] == 1:
        return np.array([[case["a"], case["b"], case["c"]]], dtype=np.int64)
    rng = np.random.default_rng(case["lens_seed"])
    n = case["count"]
    if case["log_uniform"]:
        anc = np.exp(rng.uniform(np.log(case["lo"]), np.log(case["hi"]), size=n))
    else:
        anc = rng.uniform(case["lo"], case["hi"], size=n)
    lens = np.rint(anc[:, None] * rng.uniform(0.97, 1.03, size=(n, 3))).astype(np.int64)
    top = case["hi"]
    return np.clip(lens, 1, top)


def _descendant(rng, anc, n, rate):
    """A mutated copy of anc of exactly n residues: substitutions at the given
    rate, 1 % insertion and 1 % deletion starts of geometric length."""
    m = anc.size
    sub = rng.random(m) < rate
    seq = np.where(sub, (anc + rng.integers(1, 4, size=m)) % 4, anc)
    copies = np.ones(m, dtype=np.int64)
    gone = np.flatnonzero(rng.random(m) < 0.01)
    for p, run in zip(gone, rng.geometric(0.5, size=gone.size)):
        copies[p:p + run] = 0
    ins = rng.random(m) < 0.01
    copies[ins] += rng.geometric(0.5, size=int(ins.sum()))
    seq = np.repeat(seq, copies)
    # What an insertion repeats is replaced by random residues.
    first = np.ones(seq.size, dtype=bool)
    first[1:] = np.repeat(np.arange(m), copies)[1:] != np.repeat(np.arange(m), copies)[:-1]
    seq = np.where(first, seq, rng.integers(0, 4, size=seq.size))
    if seq.size < n:
        seq = np.concatenate([seq, rng.integers(0, 4, size=n - seq.size)])
    return seq[:n].astype(np.uint8)


def _triplets(case, seed):
    rng = np.random.default_rng([seed, 20260528])
    out = []
    for lens in _lengths(case):
        anc = rng.integers(0, 4, size=int(lens.max())).astype(np.uint8)
        rate = rng.uniform(0.02, 0.15)
        out.append(tuple(_descendant(rng, anc, int(n), rate) for n in lens))
    return out


def _text(trips):
    return [tuple(LETTERS[s].tobytes() for s in t) for t in trips]


def _pack(trips):
    """2-bit words of all sequences, 16 residues a word, each sequence on a
    fresh word; lengths and word offsets beside them."""
    seqs = [s for t in trips for s in t]
    lens = np.array([s.size for s in seqs], dtype=np.uint32)
    nwords = (lens.astype(np.int64) + 15) // 16
    off = np.concatenate([[0], np.cumsum(nwords)[:-1]])
    flat = np.zeros(int(nwords.sum()) * 16, dtype=np.uint32)
    for s, o in zip(seqs, off):
        flat[16 * o:16 * o + s.size] = s
    words = (flat.reshape(-1, 16) << (2 * np.arange(16, dtype=np.uint32))).sum(axis=1, dtype=np.uint64)
    return lens, off.astype(np.uint64), words.astype(np.uint32)


def prepare(case, seed):
    trips = _triplets(case, seed)
    match, mismatch, gap = SCHEMES[case["scheme"]]
    sc = ts.scoring(match, mismatch, gap, kind=KINDS[case["kind"]])
    st = {"entry": case["entry"], "sc": sc}
    if case["entry"] == "plan":
        lens, off, words = _pack(trips)
        st["plan"] = ts.Plan(lens, off, sc=sc, use_graph=case["graph"])
        st["words"] = torch.from_numpy(words.view(np.int32)).cuda()
        st["scores"] = torch.zeros(len(trips), dtype=torch.int32, device="cuda")
    else:
        st["text"] = _text(trips)
        st["cap"] = max(sum(s.size for s in t) for t in trips)
    if case["entry"] == "served":
        st["server"] = ts.Server(max_len=2048, sc=sc, max_device_bytes=40 << 30)
    return st


def _rows(results, cap):
    """Alignment rows as one array, each row filled up with NULs to cap."""
    text = "".join(r.ljust(cap, "\0") for rows, _ in results for r in rows)
    return np.frombuffer(text.encode(), dtype=np.uint8).reshape(len(results), 3, cap)


def run(st):
    entry = st["entry"]
    if entry == "plan":
        st["plan"].run(st["words"], st["scores"])
        return st["scores"]
    if entry == "score":
        return ts.score(st["text"][0], st["sc"])
    if entry == "score_batch":
        return ts.score_batch(st["text"], st["sc"])
    if entry == "align":
        res = ts.align(st["text"][0], st["sc"])
        return {"rows": _rows([res], st["cap"]), "score": res[1]}
    if entry == "align_batch":
        res = ts.align_batch(st["text"], st["sc"])
        return {"rows": _rows(res, st["cap"]), "scores": np.array([s for _, s in res], dtype=np.int64)}
    srv = st["server"]
    ids = [srv.submit(t) for t in st["text"]]
    results = [srv.wait(i) for i in ids]
    return np.array([[r["score"], r["status"]] for r in results], dtype=np.int64)


def work(case):
    """Inputs once, scores (and alignment rows) once; per cell of the a*b*c
    tensor the recurrence's six maxima and five additions, local scoring its
    floor and running best besides."""
    lens = _lengths(case).astype(np.float64)
    cells = float(lens.prod(axis=1).sum())
    residues = float(lens.sum())
    if case["entry"] == "plan":
        nbytes = residues / 4 + 4 * len(lens)
    else:
        nbytes = residues + 4 * len(lens)
        if case["entry"].startswith("align"):
            nbytes += 3 * float(lens.max(axis=1).sum())
    return {"bytes": nbytes, "flops": cells * (13 if case["kind"] == "local" else 11)}


# ---- the plain dynamic program, 64-bit, over planes i + j + k = d ----------

_EXACT_CELLS = 1.2e10  # beyond this the plain program takes too long


def _shift(x, dj, dk, none):
    """y[:, j, k] = x[:, j - dj, k - dk], none where that is outside."""
    y = torch.full_like(x, none)
    y[:, dj:, dk:] = x[:, :x.shape[1] - dj, :x.shape[2] - dk]
    return y


def _group_scores(trips, scheme, kind):
    match, mismatch, gap = scheme
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    none = -(1 << 40)
    lens = torch.tensor([[s.size for s in t] for t in trips], device=dev)
    n = [int(lens[:, a].max()) for a in range(3)]
    # Residue q of a sequence at index q + 1; 4 + axis outside (no match).
    res = []
    for a in range(3):
        r = np.full((len(trips), n[a] + 1), 4 + a, dtype=np.int64)
        for q, t in enumerate(trips):
            r[q, 1:1 + t[a].size] = t[a]
        res.append(torch.from_numpy(r).to(dev))
    x1, x2 = n[1] + 1, n[2] + 1
    j = torch.arange(x1, device=dev)[None, :, None]
    k = torch.arange(x2, device=dev)[None, None, :]
    l0, l1, l2 = (lens[:, a][:, None, None] for a in range(3))
    inside = (j <= l1) & (k <= l2)
    last = (j == l1) | (k == l2)
    rb, rc = res[1][:, :, None].expand(-1, x1, x2), res[2][:, None, :].expand(-1, x1, x2)

    def s(x, y):
        return torch.where(x == y, match, mismatch)

    s_bc = s(rb, rc)
    shape = (len(trips), x1, x2)
    prev = [torch.full(shape, none, dtype=torch.int64, device=dev) for _ in range(3)]
    score = torch.full((len(trips),), 0 if kind == "local" else none, dtype=torch.int64, device=dev)
    rows = torch.arange(len(trips), device=dev)
    for d in range(n[0] + n[1] + n[2] + 1):
        i = d - j - k
        ok = inside & (i >= 0) & (i <= l0)
        ra = torch.gather(res[0], 1, i.clamp(0, n[0]).expand(len(trips), x1, x2).reshape(len(trips), -1)).reshape(shape)
        s_ab, s_ac = s(ra, rb), s(ra, rc)
        p1, p2, p3 = prev
        # i = d - j - k >= 1 is needed by the moves that consume S0's residue;
        # a plane holds `none` where i - 1 or i is outside the tensor.
        m = torch.maximum(p1, torch.maximum(_shift(p1, 1, 0, none), _shift(p1, 0, 1, none))) + 2 * gap
        m = torch.maximum(m, _shift(p2, 1, 0, none) + s_ab + 2 * gap)
        m = torch.maximum(m, _shift(p2, 0, 1, none) + s_ac + 2 * gap)
        m = torch.maximum(m, _shift(p2, 1, 1, none) + s_bc + 2 * gap)
        m = torch.maximum(m, _shift(p3, 1, 1, none) + s_ab + s_ac + s_bc)
        if d == 0:
            m[:, 0, 0] = 0
        if kind != "global":
            axis = ((j == 0) & (k == 0)) | ((j == 0) & (i == 0)) | ((k == 0) & (i == 0))
            m = torch.where(axis, 0, m)
        if kind == "local":
            m = m.clamp(min=0)
        m = torch.where(ok, m, none)
        if kind == "local":
            score = torch.maximum(score, m.amax(dim=(1, 2)))
        elif kind == "semi-global":
            score = torch.maximum(score, torch.where(last | (i == l0), m, none).amax(dim=(1, 2)))
        else:
            done = lens.sum(dim=1) == d
            score = torch.where(done, m[rows, lens[:, 1], lens[:, 2]], score)
        prev = [m, p1, p2]
    return score.cpu().numpy()


def _scores(case, seed):
    lens = _lengths(case)
    if float(lens.astype(np.float64).prod(axis=1).sum()) > _EXACT_CELLS:
        return None
    trips = _triplets(case, seed)
    order = sorted(range(len(trips)), key=lambda q: int(lens[q].max()))
    out = np.zeros(len(trips), dtype=np.int64)
    at = 0
    while at < len(order):
        # Groups of similar lengths, up to about four million plane cells.
        top = at + 1
        while top < len(order) and (top + 1 - at) * int(lens[order[top]].max() + 1) ** 2 <= (1 << 22):
            top += 1
        group = order[at:top]
        out[group] = _group_scores([trips[q] for q in group], SCHEMES[case["scheme"]], case["kind"])
        at = top
    return out


def exact(case, seed):
    s = _scores(case, seed)
    if s is None:
        return None
    entry = case["entry"]
    if entry in ("plan", "score_batch"):
        return s
    if entry == "score":
        return int(s[0])
    if entry == "align":
        return {"rows": None, "score": int(s[0])}
    if entry == "align_batch":
        return {"rows": None, "scores": s}
    return np.stack([s, np.zeros_like(s)], axis=1)
