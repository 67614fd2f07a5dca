"""Performance cases of the permanent and boson-sampling library.

Each case is one call (or one burst of requests) that a boson-sampling program
makes through the public binding: permanents of output amplitudes, batches of
them, the Laplace minors of a sampling step, whole sampling calls and a burst of
jobs on the sampling server.  Sizes follow the repository's benchmark and tests:
60-mode Haar interferometers, up to 31 photons per single permanent, uneven
batches of 8 to 24 photons, sampling jobs of 20 to 30 photons.
"""
import math
import weakref

import numpy as np
import torch

from paper_2309_07027_amd import binding as B

MODES = 60
DEV = "cuda"


def listed():
    return [
        # one amplitude of a small experiment: launches and latency
        {"name": "perm_n8", "kind": "perm", "n": 8, "rows": "random", "formula": "bbfg"},
        # a mid-size collision-free amplitude (20 photons)
        {"name": "perm_n20", "kind": "perm", "n": 20, "rows": "distinct", "formula": "bbfg"},
        # the headline permanent: 30 distinct output modes
        {"name": "perm_n30", "kind": "perm", "n": 30, "rows": "distinct", "formula": "bbfg"},
        # an amplitude of a sampled output (repeated modes), odd photon number
        {"name": "perm_n31_random", "kind": "perm", "n": 31, "rows": "random", "formula": "bbfg"},
        # two photons in every occupied input mode: the column-multiplicity form
        {"name": "cols_14x2", "kind": "cols", "cols": 14, "power": 2, "rows": "distinct"},
        # output probabilities of many samples of one interferometer, uneven sizes
        {"name": "batch_4096", "kind": "batch", "count": 4096, "n_lo": 8, "n_hi": 24, "precision": "fp64"},
        # the same, FP32 column sums (screening, where accuracy matters less)
        {"name": "batch_4096_fp32", "kind": "batch", "count": 4096, "n_lo": 8, "n_hi": 24, "precision": "fp32"},
        # all Laplace minors of the last step of a 30-photon sample, collision-free prefix
        {"name": "minors_k30", "kind": "minors", "k": 30, "rows": "distinct"},
        # the same beyond 30 photons, with the repeated modes a real prefix has
        {"name": "minors_k35_random", "kind": "minors", "k": 35, "rows": "random"},
        # an interactive sampling call
        {"name": "sample_n20", "kind": "sample", "n": 20, "samples": 16, "loss": 0.0, "mode": "ideal"},
        # a lossy experiment through the doubled modes
        {"name": "sample_n24_lossy", "kind": "sample", "n": 24, "samples": 24, "loss": 0.3, "mode": "dilation"},
        # a burst of jobs on the sampling server
        {"name": "serve_24", "kind": "serve", "jobs": 24, "samples": 16, "n_lo": 20, "n_hi": 30},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["perm", "perm", "perm", "cols", "batch", "batch", "minors", "minors", "sample", "sample", "serve"])
    if kind == "perm":
        formula = rng.choice(["bbfg", "bbfg", "bbfg", "ryser"])
        rows = rng.choice(["distinct", "random", "random", "bunched"])
        return {"kind": kind, "n": rng.randint(6, 31 if formula == "bbfg" else 26), "rows": rows, "formula": formula}
    if kind == "cols":
        power = rng.choice([0, 2, 2, 3])  # 0: mixed multiplicities 1..3
        return {"kind": kind, "cols": rng.randint(5, {0: 14, 2: 15, 3: 9}[power]), "power": power,
                "rows": rng.choice(["distinct", "random"])}
    if kind == "batch":
        lo = rng.randint(4, 20)
        return {"kind": kind, "count": _log_int(rng, 16, 4096), "n_lo": lo, "n_hi": rng.randint(lo, 24),
                "precision": rng.choice(["fp64", "fp64", "fp32"])}
    if kind == "minors":
        rows = rng.choice(["distinct", "random", "random"])
        return {"kind": kind, "k": rng.randint(8, 30 if rows == "distinct" else 35), "rows": rows}
    if kind == "sample":
        n = rng.randint(6, 30)
        mode = rng.choice(["ideal", "ideal", "dilation", "input"])
        return {"kind": kind, "n": n, "samples": _log_int(rng, 1, 64 if n <= 24 else 16),
                "loss": 0.0 if mode == "ideal" else rng.choice([0.1, 0.3, 0.5]), "mode": mode}
    lo = rng.randint(12, 24)
    return {"kind": kind, "jobs": rng.randint(4, 24), "samples": rng.choice([4, 8, 16]), "n_lo": lo,
            "n_hi": rng.randint(lo, 30)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _haar(rng, m=MODES):
    z = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    q, r = np.linalg.qr(z)
    d = np.diag(r)
    return np.ascontiguousarray(q * (d / np.abs(d))[None, :])


def _placed(rng, n, rows):
    """Occupied output modes and their photon counts: n photons on distinct
    modes, at random on all modes, or bunched on max(2, n // 2) of them."""
    if rows == "distinct":
        modes = rng.choice(MODES, size=n, replace=False)
    elif rows == "random":
        modes = rng.integers(0, MODES, n)
    else:
        modes = rng.integers(0, max(2, n // 2), n)
    cnt = np.bincount(modes, minlength=MODES)
    kept = np.nonzero(cnt)[0]
    return kept, cnt[kept].astype(np.int32)


def _col_mult(case, rng):
    if case["power"]:
        return np.full(case["cols"], case["power"], dtype=np.int32)
    return rng.integers(1, 4, case["cols"]).astype(np.int32)


def _matrix(case, seed):
    """(A, M, N) of a perm, minors or cols case on the host (N: column multiplicities)."""
    rng = np.random.default_rng(seed)
    u = _haar(rng)
    if case["kind"] == "perm":
        rows, mult = _placed(rng, case["n"], case["rows"])
        return np.ascontiguousarray(u[rows, :case["n"]]), mult, None
    if case["kind"] == "minors":
        rows, mult = _placed(rng, case["k"] - 1, case["rows"])
        return np.ascontiguousarray(u[rows, :case["k"]]), mult, None
    cm = _col_mult(case, rng)
    rows, mult = _placed(rng, int(cm.sum()), case["rows"])
    return np.ascontiguousarray(u[rows, :case["cols"]]), mult, cm


def _batch_items(case, seed):
    rng = np.random.default_rng(seed)
    u = _haar(rng)
    items = []
    for _ in range(case["count"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        rows, mult = _placed(rng, n, "random")
        items.append((u[rows, :n], mult))
    return items


def _occupation(n):
    occ = np.zeros(MODES, dtype=np.int32)
    occ[:n] = 1
    return occ


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("perm", "minors", "cols"):
        A, M, N = _matrix(case, seed)
        return {"case": case, "A": torch.from_numpy(A).to(DEV), "M": M, "N": N}
    if kind == "batch":
        A, a_off, n_rows, M, m_off, n_cols = B.pack_batch(_batch_items(case, seed))
        return {"case": case, "A": torch.from_numpy(A).to(DEV), "shapes": (a_off, n_rows, M, m_off, n_cols)}
    rng = np.random.default_rng(seed)
    if kind == "sample":
        return {"case": case, "U": torch.from_numpy(_haar(rng)).to(DEV), "occ": _occupation(case["n"]), "seed": seed}
    # serve: requests arrive as host matrices; the server is the program's own
    jobs = []
    for j in range(case["jobs"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        jobs.append((_haar(rng), _occupation(n), seed * 1000 + j))
    server = B.Server()
    state = {"case": case, "jobs": jobs, "server": server}
    weakref.finalize(server, B.lib().bs_server_destroy, server._h)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "perm":
        f = B.perm_ryser if case["formula"] == "ryser" else B.perm_bbfg
        value, info = f(state["A"], state["M"], with_info=True)
        return {"value": np.array([value]), "kappa": info["kappa"]}
    if kind == "cols":
        return {"value": np.array([B.perm_bbfg_cols(state["A"], state["M"], state["N"])])}
    if kind == "batch":
        a_off, n_rows, M, m_off, n_cols = state["shapes"]
        precision = B.BBFG_FP32 if case["precision"] == "fp32" else B.BBFG_FP64
        return {"values": B.perm_batch_packed(state["A"], a_off, n_rows, M, m_off, n_cols, precision=precision)}
    if kind == "minors":
        return {"minors": B.perm_minors(state["A"], state["M"])}
    if kind == "sample":
        if case["mode"] == "input":
            return {"samples": B.bs_sample_extracted(state["U"], state["occ"], case["samples"], case["loss"], state["seed"])}
        return {"samples": B.bs_sample(state["U"], state["occ"], case["samples"], case["loss"], state["seed"])}
    server = state["server"]
    ids = [server.submit(U, occ, case["samples"], 0.0, seed) for U, occ, seed in state["jobs"]]
    server.drain()
    return {"samples": np.concatenate([server.poll(i)[0] for i in ids])}


# ---------------------------------------------------------------------------
# the work of a pass: addends times the flops of one (an FMA is two)
# ---------------------------------------------------------------------------
def _addends(M, ryser=False):
    M = [int(x) for x in M]
    if not ryser:
        p = min(range(len(M)), key=lambda i: M[i])
        M[p] -= 1
    return math.prod(x + 1 for x in M)


def _minors_flops(k, M):
    return _addends(M) * (22.0 * k - 36.0)


def _sample_flops(rng, n, survive=1.0):
    """One sample's steps on uniformly placed photons."""
    steps = max(1, int(round(n * survive)))
    modes = rng.integers(0, MODES, steps)
    total = 0.0
    for k in range(2, steps + 1):
        cnt = np.bincount(modes[:k - 1])
        total += _minors_flops(k, cnt[cnt > 0])
    return total


def work(case):
    kind = case["kind"]
    if kind in ("perm", "minors", "cols"):
        A, M, _ = _matrix(case, 0)
        if kind == "minors":
            flops, out = _minors_flops(case["k"], M), case["k"]
        else:
            flops = _addends(M, case.get("formula") == "ryser") * (8.0 * A.shape[1] - 4.0)
            out = 1
        return {"bytes": 16 * (A.size + out), "flops": flops}
    if kind == "batch":
        items = _batch_items(case, 0)
        return {"bytes": 16 * (sum(A.size for A, _ in items) + len(items)),
                "flops": sum(_addends(M) * (8.0 * A.shape[1] - 4.0) for A, M in items)}
    rng = np.random.default_rng(0)
    if kind == "sample":
        survive = 1.0 - case["loss"] if case["mode"] == "input" else 1.0
        flops = sum(_sample_flops(rng, case["n"], survive) for _ in range(case["samples"]))
        return {"bytes": 16 * MODES * MODES + 4 * MODES * case["samples"], "flops": flops}
    flops = 0.0
    for _ in range(case["jobs"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        flops += sum(_sample_flops(rng, n) for _ in range(case["samples"]))
    return {"bytes": case["jobs"] * (16 * MODES * MODES + 4 * MODES * case["samples"]), "flops": flops}


# ---------------------------------------------------------------------------
# the same values in plain torch, 64 bits
# ---------------------------------------------------------------------------
MOST_ADDENDS = 2.2e9


def _column_sums(A, M, ryser, chunk):
    """Yields (sums, weights) over all sign counts: chunks of column sums
    sum_k (M_k - 2 D_k) a_k (Glynn, one copy of the first rarest row held at +1)
    or sum_k D_k a_k (Ryser), and the weights prod_k (-1)^D_k C(M_k, D_k)."""
    M = [int(x) for x in M]
    free = list(M)
    if not ryser:
        free[min(range(len(M)), key=lambda i: M[i])] -= 1
    total = math.prod(f + 1 for f in free)
    a = torch.from_numpy(np.ascontiguousarray(A)).to(DEV)
    a = torch.cat([a.real, a.imag], dim=1).contiguous()
    pascal = [torch.tensor([float((-1) ** d * math.comb(f, d)) for d in range(f + 1)], dtype=torch.float64, device=DEV)
              for f in free]
    n = A.shape[1]
    for first in range(0, total, chunk):
        idx = torch.arange(first, min(total, first + chunk), device=DEV)
        coef = torch.empty((len(M), idx.numel()), dtype=torch.float64, device=DEV)
        w = torch.ones(idx.numel(), dtype=torch.float64, device=DEV)
        for k, f in enumerate(free):
            d = idx % (f + 1)
            idx = idx // (f + 1)
            coef[k] = d if ryser else M[k] - 2 * d
            if f:
                w *= pascal[k][d]
        s = coef.t() @ a
        yield torch.complex(s[:, :n].t().contiguous(), s[:, n:].t().contiguous()), w


def _exact_perm(A, M, ryser=False, chunk=1 << 20):
    total = torch.zeros((), dtype=torch.complex128, device=DEV)
    mags = torch.zeros((), dtype=torch.float64, device=DEV)
    for c, w in _column_sums(A, M, ryser, chunk):
        p = c[0]
        for j in range(1, c.shape[0]):
            p = p * c[j]
        p = p * w
        total += p.sum()
        mags += p.real.abs().sum() + p.imag.abs().sum()
    n = A.shape[1]
    value = total * (((-1.0) ** n if ryser else 2.0 ** (1 - n)))
    # the conditioning sum |addend| / |sum|, the modulus of an addend as |re| + |im|
    return complex(value.cpu()), float((mags / total.abs()).cpu())


def _exact_minors(A, M, chunk=1 << 18):
    k = A.shape[1]
    acc = torch.zeros(k, dtype=torch.complex128, device=DEV)
    for c, w in _column_sums(A, M, False, chunk):
        pre = torch.empty_like(c)
        pre[0] = w.to(torch.complex128)
        for j in range(1, k):
            torch.mul(pre[j - 1], c[j - 1], out=pre[j])
        suf = torch.ones_like(c[0])
        for j in range(k - 1, -1, -1):
            acc[j] += (pre[j] * suf).sum()
            suf = suf * c[j]
    return (acc * 2.0 ** (1 - (k - 1))).cpu().numpy()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("sample", "serve"):
        return None  # whole numbers
    if kind == "batch":
        items = _batch_items(case, seed)
        return {"values": np.array([_exact_perm(A, M)[0] for A, M in items])}
    A, M, N = _matrix(case, seed)
    if _addends(M, case.get("formula") == "ryser") > MOST_ADDENDS:
        return None
    if kind == "minors":
        return {"minors": _exact_minors(A, M)}
    if kind == "cols":
        return {"value": np.array([_exact_perm(np.repeat(A, N, axis=1), M)[0]])}
    value, kappa = _exact_perm(A, M, case["formula"] == "ryser")
    return {"value": np.array([value]), "kappa": kappa}
