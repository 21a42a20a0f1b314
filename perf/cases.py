"""The workloads whose speed is measured: dot products, SpMVs, solves, a batch
and a served mix, each through the entry points of ``rpk.py``.

A case is a dict of plain values; ``prepare`` makes what a program holds before
the call (matrix handles, right-hand sides, a server), ``run`` is one pass,
``work`` the bytes and operations the pass cannot do without and ``exact`` the
64-bit answer.  Inputs are generated on the GPU from the seed, with the stencils
and distributions of ``inputs.py``: matrix entries by their formulas, vectors
U(-1, 1); right-hand sides are b = A x* with x* ~ U(-1, 1), so the answer of a
solve is x* up to its tolerance.
"""
import math
import random

import torch

from paper_2302_04180_amd import rpk

VARIANT = {"std": rpk.STD, "pipelined": rpk.PIPELINED, "pcg": rpk.PCG}
DOTS = {"exact": rpk.EXACT, "plain": rpk.PLAIN}
TOL = 1e-8
MAXIT = 5000


def listed():
    return [
        # dot products: a vector of a tiny system (the call's latency), one solver
        # vector of the 128^3 grid, and a long one of odd length
        dict(name="dot_1000", op="dot", n=1000, mode="exact"),
        dict(name="dot_2m", op="dot", n=2097152, mode="exact"),
        dict(name="dot_40m_odd", op="dot", n=40000003, mode="exact"),
        # one exact matrix-vector product: the 27-point e-type grid (bandwidth)
        # and the unstructured banded matrix (irregular gathers)
        dict(name="spmv_etype_159", op="spmv", kind="etype", edge=159, mode="exact"),
        dict(name="spmv_banded_500k", op="spmv", kind="banded", n=500000, mode="exact"),
        # whole solves: the small grid where launches and latency count, the
        # 128^3 grid, a symmetric system of odd size whose diagonal varies, the
        # convection-diffusion grid and the unstructured matrix
        dict(name="solve_std_poisson_16", op="solve", kind="poisson", edge=16, variant="std"),
        dict(name="solve_std_poisson_128", op="solve", kind="poisson", edge=128, variant="std"),
        dict(name="solve_pcg_vardiag_101", op="solve", kind="vardiag", edge=101, variant="pcg"),
        dict(name="solve_pipe_convdiff_96", op="solve", kind="convdiff", edge=96, variant="pipelined"),
        dict(name="solve_pipe_banded_500k", op="solve", kind="banded", n=500000, variant="pipelined"),
        # many independent systems in one call: edges 8..48, alternately Poisson
        # and convection-diffusion
        dict(name="batch_std_256", op="batch", systems=256, lo=8, hi=48, mix=1000, variant="std"),
        # requests of mixed sizes sent to the server together
        dict(name="serve_pipe_16", op="serve", systems=16, lo=16, hi=128, mix=2024, variant="pipelined"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _grid(rng, pcg=False, hi7=128, hi27=96):
    kind = rng.choice(["poisson", "vardiag", "sym27"] if pcg else ["poisson", "convdiff", "vardiag", "etype"])
    return dict(kind=kind, edge=_log_int(rng, 8, hi27 if kind in ("etype", "sym27") else hi7))


def draw(rng):
    op = rng.choice(["dot", "dot", "spmv", "spmv", "solve", "solve", "solve", "batch", "serve"])
    if op == "dot":
        return dict(op=op, n=_log_int(rng, 1, 40000000), mode=rng.choice(["exact", "exact", "plain", "light"]))
    if op == "spmv":
        case = dict(op=op, mode=rng.choice(["exact", "exact", "plain"]))
        if rng.random() < 0.3:
            return dict(case, kind="banded", n=_log_int(rng, 11000, 500000))
        return dict(case, **_grid(rng, hi27=159))
    if op == "solve":
        variant = rng.choice(["std", "pipelined", "pcg"])
        if variant != "pcg" and rng.random() < 0.25:
            return dict(op=op, kind="banded", n=_log_int(rng, 11000, 500000), variant=variant)
        return dict(op=op, variant=variant, **_grid(rng, variant == "pcg"))
    variant = rng.choice(["std", "pipelined"])
    if op == "batch":
        return dict(op=op, systems=_log_int(rng, 2, 200), lo=8, hi=rng.randint(12, 48), mix=rng.randrange(1 << 20),
                    variant=variant)
    return dict(op=op, systems=rng.randint(2, 12), lo=16, hi=rng.randint(24, 112), mix=rng.randrange(1 << 20),
                variant=variant)


# ---------------------------------------------------------------------------
# matrices, row by row: columns and values [n, k] with a mask of the entries
# ---------------------------------------------------------------------------
def _uniform(n, seed, stream=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + int(stream))
    return torch.rand(n, generator=g, dtype=torch.float64, device="cuda") * 2.0 - 1.0


def _stencil(edge, coef):
    """coef: (dz, dy, dx) -> value, in ascending order of the offset."""
    n = edge ** 3
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    z = idx // (edge * edge)
    y = (idx // edge) % edge
    x = idx % edge
    cols = torch.empty((n, len(coef)), dtype=torch.int32, device="cuda")
    mask = torch.empty((n, len(coef)), dtype=torch.bool, device="cuda")
    vals = torch.empty((n, len(coef)), dtype=torch.float64, device="cuda")
    for k, ((dz, dy, dx), v) in enumerate(coef.items()):
        inside = torch.ones(n, dtype=torch.bool, device="cuda")
        for at, d in ((z, dz), (y, dy), (x, dx)):
            inside &= (at + d >= 0) & (at + d < edge)
        cols[:, k] = idx + (dz * edge * edge + dy * edge + dx)
        mask[:, k] = inside
        vals[:, k] = v
    return cols, vals, mask


def _seven(px, py, pz):
    return {(-1, 0, 0): -(1.0 + 2.0 * pz), (0, -1, 0): -(1.0 + 2.0 * py), (0, 0, -1): -(1.0 + 2.0 * px),
            (0, 0, 0): 6.0 + 2.0 * (px + py + pz), (0, 0, 1): -1.0, (0, 1, 0): -1.0, (1, 0, 0): -1.0}


def _twenty_seven(lower):
    at = [(dz, dy, dx) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
    return {o: 26.0 if o == (0, 0, 0) else (lower if o < (0, 0, 0) else -1.0) for o in at}


def _banded(n, seed, k=19, band=5000):
    """k off-diagonal columns per row inside the band and the diagonal."""
    i = torch.arange(n, dtype=torch.int64, device="cuda")
    lo = (i - band).clamp(min=0)
    width = (i + band).clamp(max=n - 1) - lo + 1
    # one column from each of k equal parts of the band (the part that holds the
    # diagonal may give it: such an entry is moved one column on)
    u = (_uniform(n * k, seed, 1).view(n, k) + 1.0) * 0.5
    part = (torch.arange(k, device="cuda")[None, :] + u * 0.96) / k
    off = lo[:, None] + (part * (width[:, None] - 1)).long()
    off = torch.where(off == i[:, None], torch.where(off + 1 < n, off + 1, off - 1), off)
    v = _uniform(n * k, seed, 2).view(n, k)
    diag = torch.zeros(n, dtype=torch.float64, device="cuda")
    for j in range(k):
        diag += v[:, j].abs()
    cols = torch.cat([off, i[:, None]], 1)
    vals = torch.cat([v, (1.1 * diag)[:, None]], 1)
    cols, order = cols.sort(dim=1)
    return cols.int(), vals.gather(1, order), torch.ones_like(cols, dtype=torch.bool)


def _entries(case, seed):
    kind = case["kind"]
    if kind == "banded":
        return _banded(case["n"], seed)
    if kind == "etype":
        return _stencil(case["edge"], _twenty_seven(-(1.0 - 0.0001)))
    if kind == "sym27":
        return _stencil(case["edge"], _twenty_seven(-1.0))
    p = float(case.get("peclet", 0.5)) if kind == "convdiff" else 0.0
    cols, vals, mask = _stencil(case["edge"], _seven(p, p / 2, p / 4))
    if kind == "vardiag":
        n = vals.shape[0]
        vals[:, 3] = 6.0 + 0.25 * (torch.arange(n, device="cuda") % 4).double()
    return cols, vals, mask


def _times(entries, x):
    """A x, the entries of a row added in column order."""
    cols, vals, mask = entries
    y = torch.zeros_like(x)
    for k in range(cols.shape[1]):
        c = torch.where(mask[:, k], cols[:, k], 0).long()
        y += torch.where(mask[:, k], vals[:, k] * x[c], 0.0)
    return y


def _matrix(entries):
    cols, vals, mask = entries
    rp = torch.zeros(cols.shape[0] + 1, dtype=torch.int32, device="cuda")
    rp[1:] = mask.sum(1, dtype=torch.int32).cumsum(0, dtype=torch.int32)
    return rpk.Matrix.from_tensors(rp, cols[mask], vals[mask])


def _mix(case):
    """The systems of a batch or of the served requests: batches draw the edge
    uniformly, requests the number of rows log-uniformly."""
    rng = random.Random(case["mix"])
    out = []
    for i in range(case["systems"]):
        if case["op"] == "batch":
            edge = rng.randint(case["lo"], case["hi"])
        else:
            edge = _log_int(rng, case["lo"], case["hi"])
        out.append(dict(kind="convdiff" if i % 2 else "poisson", edge=edge, peclet=rng.uniform(0.1, 2.0)))
    return out


def _rows(case):
    return case["edge"] ** 3 if "edge" in case else case["n"]


# ---------------------------------------------------------------------------
# the measured pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    op = case["op"]
    if op == "dot":
        return dict(case=case, x=_uniform(case["n"], seed, 1), y=_uniform(case["n"], seed, 2))
    if op == "spmv":
        A = _matrix(_entries(case, seed))
        return dict(case=case, A=A, x=_uniform(A.n, seed, 3))
    if op == "solve":
        entries = _entries(case, seed)
        return dict(case=case, A=_matrix(entries), b=_times(entries, _uniform(_rows(case), seed, 3)))
    As, bs = [], []
    for k, one in enumerate(_mix(case)):
        entries = _entries(one, seed)
        As.append(_matrix(entries))
        bs.append(_times(entries, _uniform(_rows(one), seed, 10 + k)))
    state = dict(case=case, As=As, bs=bs)
    if op == "serve":
        state["server"] = rpk.Server(hbm_budget=2 << 30, max_slots=64, chunk=4, tol=TOL, maxit=MAXIT,
                                     variant=VARIANT[case["variant"]])
    return state


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "dot":
        if case["mode"] == "light":
            return rpk.fpedot(state["x"], state["y"])
        return rpk.exdot(state["x"], state["y"], dots=DOTS[case["mode"]])
    if op == "spmv":
        return rpk.exspmv(state["A"], state["x"], dots=DOTS[case["mode"]])
    if op == "solve":
        x, info = rpk.solve(state["A"], state["b"], tol=TOL, maxit=MAXIT, variant=VARIANT[case["variant"]])
        return [x, info["iters"], info["tau"], info["true_res"]]
    if op == "batch":
        xs, infos = rpk.solve_batched(state["As"], state["bs"], tol=TOL, maxit=MAXIT,
                                      variant=VARIANT[case["variant"]])
    else:
        server = state["server"]
        xs = [torch.zeros_like(b) for b in state["bs"]]
        tickets = [server.submit(A, b, x) for A, b, x in zip(state["As"], state["bs"], xs)]
        infos = [server.wait(t) for t in tickets]
    return [torch.cat(xs), torch.tensor([i["iters"] for i in infos]),
            torch.tensor([i["true_res"] for i in infos], dtype=torch.float64)]


def _iterations(case):
    """About how many iterations a solve to the tolerance takes."""
    if case["kind"] == "banded":
        return 8
    per_edge = {"poisson": 1.5, "vardiag": 0.25, "convdiff": 1.5, "etype": 1.0, "sym27": 1.0}[case["kind"]]
    if case["variant"] == "pcg":
        per_edge *= 1.5
    return max(8, int(per_edge * case["edge"]))


def _solve_work(case):
    n = _rows(case)
    nnz = n * {"banded": 20, "etype": 27, "sym27": 27}.get(case["kind"], 7)
    spmvs = 1 if case["variant"] == "pcg" else 2
    vectors = {"std": 25, "pipelined": 42, "pcg": 13}[case["variant"]]
    it = _iterations(case)
    return (it * (spmvs * (12 * nnz + 4 * (n + 1)) + vectors * 8 * n),
            it * (spmvs * 2 * nnz + vectors * 2 * n))


def work(case):
    op = case["op"]
    if op == "dot":
        return {"bytes": 16 * case["n"] + 8, "flops": 2 * case["n"]}
    if op == "spmv":
        n = _rows(case)
        nnz = n * {"banded": 20, "etype": 27, "sym27": 27}.get(case["kind"], 7)
        return {"bytes": 12 * nnz + 4 * (n + 1) + 16 * n, "flops": 2 * nnz}
    if op == "solve":
        b, f = _solve_work(case)
        return {"bytes": b, "flops": f}
    total = [_solve_work(dict(one, variant=case["variant"])) for one in _mix(case)]
    return {"bytes": sum(b for b, _ in total), "flops": sum(f for _, f in total)}


def exact(case, seed):
    op = case["op"]
    if op == "dot":
        value = (_uniform(case["n"], seed, 1) * _uniform(case["n"], seed, 2)).sum()
        return (value, None) if case["mode"] == "light" else value
    if op == "spmv":
        return _times(_entries(case, seed), _uniform(_rows(case), seed, 3))
    if op == "solve":
        return [_uniform(_rows(case), seed, 3), None, None, None]
    return [torch.cat([_uniform(_rows(one), seed, 10 + k) for k, one in enumerate(_mix(case))]), None, None]
