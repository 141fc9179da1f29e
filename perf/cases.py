"""Performance cases: what a user of this library has it do, through its public entry points.

Three kinds of work, in the sizes this repository's tests, benchmark and
generators use: one fold of a device-resident sequence (score and table), a
host call that wants a structure, and many folds at once (a prepared batch, a
served stream).  Lengths run from the shortest sequences of
the batch workload (50) to the longest single fold it reports on (16000).
``exact`` evaluates Eq. 1 with 64-bit torch, without this package's code.
"""

import math

import numpy as np
import torch

from paper_1307_7820_amd import gen, nf

SERVE_BUDGET = 2 << 30  # the serving workload's device budget


def listed():
    return [
        # the shortest RNAs of the batch workload, alone: launches and latency
        {"name": "fold_60", "kind": "fold", "n": 60, "q": 0, "stems": False},
        # the small single fold (500 bases), the one every q is checked on
        {"name": "fold_500", "kind": "fold", "n": 500, "q": 0, "stems": False},
        # a ragged length at the narrower group width a caller may ask for
        {"name": "fold_1283_q4", "kind": "fold", "n": 1283, "q": 4, "stems": False},
        # a group width that does not divide 64 (tiles of 60 posts)
        {"name": "fold_3001_q5", "kind": "fold", "n": 3001, "q": 5, "stems": False},
        # the headline fold
        {"name": "fold_6000", "kind": "fold", "n": 6000, "q": 0, "stems": False},
        # the long fold: GC-rich with planted stems, as structured RNA is
        {"name": "fold_16000", "kind": "fold", "n": 16000, "q": 0, "stems": True},
        # the entry point for callers that cannot allocate, near its limit
        {"name": "noalloc_3300", "kind": "noalloc", "n": 3300, "q": 0, "stems": False},
        # a host program that wants one structure
        {"name": "structure_2000", "kind": "structure", "n": 2000, "q": 0, "stems": True},
        # a prepared batch of short folds, with all structures
        {"name": "batch_256", "kind": "batch", "count": 256, "lo": 50, "hi": 700, "q": 0, "structures": True},
        # the batch workload
        {"name": "batch_4096", "kind": "batch", "count": 4096, "lo": 50, "hi": 2000, "q": 0, "structures": False},
        # a burst of requests at the serving engine, 80 % of 100-500 bases
        # and 20 % of 2000-8000
        {"name": "serve_200", "kind": "serve", "count": 200, "hi": 8000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fold", "fold", "fold", "noalloc", "structure", "batch", "batch", "serve"])
    if kind == "fold":
        return {"kind": kind, "n": _log(rng, 50, 16000), "q": rng.choice([0, 0, 0, 8, 4, 5]),
                "stems": rng.random() < 0.5}
    if kind == "noalloc":
        return {"kind": kind, "n": _log(rng, 50, 3400), "q": rng.choice([0, 8]), "stems": rng.random() < 0.5}
    if kind == "structure":
        return {"kind": kind, "n": _log(rng, 100, 8000), "q": 0, "stems": rng.random() < 0.5}
    if kind == "batch":
        return {"kind": kind, "count": _log(rng, 8, 4000), "lo": 50, "hi": rng.randint(200, 1900), "q": 0,
                "structures": rng.random() < 0.5}
    return {"kind": "serve", "count": _log(rng, 16, 190), "hi": rng.randint(2100, 7900)}


def _lengths(case):
    """The lengths of a case: log-uniform for a batch, the serving mix for a stream."""
    if "n" in case:
        return [case["n"]]
    order = np.random.default_rng(case["count"])
    m = case["count"]
    if case["kind"] == "serve":
        u = (order.permutation(m) + 0.5) / m
        return [int(100 + 500 * x) if x < 0.8 else int(2000 + (case["hi"] - 2000) * (x - 0.8) / 0.2) for x in u]
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return [int(round(math.exp(lo + (k + 0.5) / m * (hi - lo)))) for k in order.permutation(m)]


def _sequences(case, seed):
    if case.get("stems"):
        return [gen.stem_sequence(case["n"], [seed, 1])]
    return [gen.iid_sequence(n, [seed, k]) for k, n in enumerate(_lengths(case))]


def prepare(case, seed):
    kind = case["kind"]
    seqs = _sequences(case, seed)
    state = {"case": case}
    if kind in ("fold", "noalloc"):
        n = case["n"]
        state["codes"] = torch.from_numpy(nf.encode(seqs[0]).copy()).cuda()
        state["score"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        state["table"] = torch.zeros((n, n), dtype=torch.int16, device="cuda")
    elif kind == "structure":
        state["seq"] = seqs[0]
    elif kind == "batch":
        state["batch"] = nf.Batch(seqs, case["q"])
    else:
        state["seqs"] = seqs
        if kind == "serve":
            try:
                nf.nf_serve_config(hbm_budget_bytes=SERVE_BUDGET)
            except nf.NFError as e:  # the engine of an earlier state serves this one too
                if e.code != nf.NF_E_BUSY:
                    raise
    return state


def _db(text):
    return np.frombuffer(text.encode("ascii"), dtype=np.uint8)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("fold", "noalloc"):
        call = nf.nf_fold_dev if kind == "fold" else nf.nf_fold_dev_noalloc
        call(state["codes"], case["n"], case["q"], state["score"], state["table"],
             torch.cuda.current_stream())
        return [state["score"], state["table"]]
    if kind == "structure":
        score, db = nf.nf_fold_structure(state["seq"], case["q"])
        return [score, _db(db)]
    if kind == "batch":
        b = state["batch"]
        b.run(torch.cuda.current_stream())
        out = [b.scores()]
        if case["structures"]:
            out.append(_db("".join(b.structures())))
        return out
    tickets = [nf.nf_submit(s) for s in state["seqs"]]
    return [np.array([nf.nf_wait(t) for t in tickets], dtype=np.int32)]


def work(case):
    """Codes read once; scores, tables and structures written once.  One add
    and one comparison for each of the n(n+1)/2 cells of a table: no fill does
    with less, whatever it does about the splits."""
    ns = _lengths(case)
    out = 4 * len(ns)
    if case["kind"] in ("fold", "noalloc"):
        out += 2 * case["n"] ** 2
    elif case["kind"] == "structure" or case.get("structures"):
        out += sum(ns)
    return {"bytes": sum(ns) + out, "flops": sum(n * (n + 1) for n in ns)}


# ---- Eq. 1 in 64 bits

def _table(seq, device):
    """F of Eq. 1 by fence posts, F[a, b] = D(a+1, b), filled by diagonals."""
    n = len(seq)
    codes = torch.tensor(["ACGU".index(c) for c in seq], device=device)
    ld = n + 1
    F = torch.zeros((ld, ld), dtype=torch.int64, device=device)
    G = torch.zeros((ld, ld), dtype=torch.int64, device=device)  # G[b, a] = F[a, b]
    step = max(1, (1 << 27) // max(1, n))
    for t in range(2, n + 1):
        m = n + 1 - t  # cells (a, a+t), a = 0 .. m-1
        best = torch.empty(m, dtype=torch.int64, device=device)
        for a0 in range(0, m, step):
            a1 = min(m, a0 + step)
            left = F.as_strided((a1 - a0, t - 1), (ld + 1, 1), a0 * (ld + 1) + 1)
            down = G.as_strided((a1 - a0, t - 1), (ld + 1, 1), (a0 + t) * ld + a0 + 1)
            best[a0:a1] = (left + down).amax(1)
        pair = (codes[:m] + codes[t - 1:t - 1 + m] == 3).to(torch.int64)
        inner = F.as_strided((m,), (ld + 1,), ld + 1 + t - 2)
        best = torch.maximum(best, pair + inner)
        F.as_strided((m,), (ld + 1,), t).copy_(best)
        G.as_strided((m,), (ld + 1,), t * ld).copy_(best)
    return F


def _traceback(seq, F):
    """The first maximising term of Eq. 1: the pairing, then the splits in order."""
    db = ["."] * len(seq)
    code = {"A": 0, "C": 1, "G": 2, "U": 3}
    todo = [(0, len(seq))]
    while todo:
        a, b = todo.pop()
        while b - a >= 2:
            pair = code[seq[a]] + code[seq[b - 1]] == 3
            if F[a, b] == int(pair) + F[a + 1, b - 1]:
                if pair:
                    db[a], db[b - 1] = "(", ")"
                a, b = a + 1, b - 1
                continue
            m = a + 1 + int(np.argmax(F[a, a + 1:b] + F[a + 1:b, b] == F[a, b]))
            todo.append((m, b))
            b = m
    return "".join(db)


def exact(case, seed):
    seqs = _sequences(case, seed)
    cells = sum(len(s) ** 3 for s in seqs)
    if cells > 3e11 or sum(len(s) for s in seqs) > 30000:
        return None
    device = "cuda" if torch.cuda.is_available() else "cpu"
    scores, text, table = [], [], None
    for s in seqs:
        n = len(s)
        F = _table(s, device)
        scores.append(int(F[0, n]))
        if case["kind"] in ("fold", "noalloc"):
            table = F[:n, 1:].triu()
        elif case["kind"] == "structure" or case.get("structures"):
            text.append(_traceback(s, F.cpu().numpy()))
    scores = np.array(scores, dtype=np.int64)
    if table is not None:
        return [scores, table.cpu().numpy()]
    if case["kind"] == "structure":
        return [int(scores[0]), _db(text[0])]
    return [scores, _db("".join(text))] if text else [scores]
