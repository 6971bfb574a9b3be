"""The framework's work as timed cases: each case is one call (or one whole job)
through the public entry points of paper_2307_03276_amd.cpapr, on seeded
synthetic count tensors made on the GPU.

A case holds what a program chooses: the operation, the tensor's sizes and
distribution, the rank, the mode, the precision and the loop limits.
"""
import math

import numpy as np
import torch

from paper_2307_03276_amd import cpapr

EPS = 1e-10
KAPPA, KAPPA_TOL = 0.01, 1e-10
CHUNK = 1 << 21  # nonzeros per step of the 64-bit reference


def listed():
    """Every operation at a size it is used at, from one small tensor to 100M nonzeros."""
    return [
        # one Phi of the small parity tensor: a call whose launches weigh more than its work
        _case("phi-3way-10k-r10", "phi", "100x80x60", 10_000, 10, mu=2.0),
        # a whole small job, plan and 10 x 10 fixed schedule: what many short factorisations cost
        _case("job-3way-10k-r10", "job", "100x80x60", 10_000, 10, mu=2.0, kmax=10, lmax=10),
        # one mode's inner loop of a request in the service: odd sizes, FP32-stored factors, KKT stop
        _case("inner-4way-600k-r10-mixed", "inner", "31417x5003x70001x1201", 600_011, 10, mode=2, zipf=1.1,
              precision="mixed", tol=1e-4, lmax=10),
        # one Phi of a 5-way tensor of weights (values not exact in FP32) at a ragged rank
        _case("phi-5way-1.5M-r17-weights", "phi", "4001x777x10007x53x601", 1_500_001, 17, mode=1, zipf=1.1,
              values="weights"),
        # Phi once from coordinates, without a plan: validation, one mode's sort, Phi
        _case("coo-3way-3M-r16", "coo", "60000x45000x8000", 3_000_017, 16, mode=1, zipf=1.1),
        # the likelihood of a model, as evaluated after a solve
        _case("loglik-3way-5M-r16", "loglik", "90000x70000x12000", 5_000_003, 16, zipf=1.1, mu=3.0),
        # MTTKRP of CP-ALS on a tensor with uniform coordinates
        _case("mttkrp-3way-8M-r32", "mttkrp", "30011x20011x5003", 8_000_009, 32, mode=0),
        # the benchmark's default job: plan, 5 x 10 fixed schedule over three modes, likelihood
        _case("job-3way-20M-r16", "job", "200000x150000x20000", 20_000_000, 16, zipf=1.1, mu=3.0, kmax=5, lmax=10),
        # the largest tensor: one mode's inner loop, 4-way 100M nonzeros
        _case("inner-4way-100M-r32", "inner", "1000000x200000x10000x500", 100_000_000, 32, zipf=1.2, nzipf=2, mu=1.0,
              lmax=10),
        # many tensors of very different sizes in one batch, inner loops with KKT stops
        _case("batch-64x3way", "batch", "", 64, 0, tol=1e-4, lmax=10),
        # row solves of one mode: projected quasi-Newton on the benchmark tensor
        _case("pqnr-3way-20M-r16", "pqnr", "200000x150000x20000", 20_000_000, 16, zipf=1.1, mu=3.0, lmax=4),
        # row solves of one mode: projected damped Newton, 4-way, R = 32
        _case("pdnr-4way-5M-r32", "pdnr", "100000x40000x5000x400", 5_000_011, 32, mode=1, zipf=1.1, mu=1.0, lmax=4),
    ]


def draw(rng):
    """One more case: any operation at sizes between the listed ones."""
    op = rng.choice(["phi", "phi", "inner", "inner", "mttkrp", "loglik", "coo", "job", "batch", "pqnr", "pdnr"])
    if op == "batch":
        return _case(None, op, "", rng.randint(8, 64), 0, tol=rng.choice([0.0, 1e-4]), lmax=rng.randint(2, 10),
                     precision=rng.choice(["fp64", "mixed"]), graph=rng.random() < 0.5)
    top = {"phi": 5e7, "inner": 3e7, "mttkrp": 3e7, "loglik": 3e7, "coo": 1e7, "job": 2e6, "pqnr": 4e6, "pdnr": 4e6}[op]
    nnz = int(math.exp(rng.uniform(math.log(3e3), math.log(top))))
    n = rng.choice([2, 3, 3, 3, 4, 4, 5] if op in ("phi", "coo", "mttkrp") else [3, 3, 4])
    # dims grow with the tensor: at least a few nonzeros per row on average
    hi = min(1e6, max(60.0, nnz / 4.0))
    dims = "x".join(str(int(math.exp(rng.uniform(math.log(30), math.log(hi))))) for _ in range(n))
    ranks = [5, 8, 10, 16, 16, 17, 24, 32, 32, 40, 64] if op in ("phi", "coo", "mttkrp", "inner") else [8, 10, 16, 24, 32]
    kw = dict(mode=rng.randrange(n), zipf=rng.choice([0.0, 1.1, 1.1, 1.2]), mu=rng.choice([1.0, 2.0, 3.0]))
    if op in ("phi", "inner"):
        kw["precision"] = rng.choice(["fp64", "fp64", "mixed"])
    if op in ("phi", "mttkrp", "inner", "coo"):
        kw["values"] = rng.choice(["counts", "counts", "counts", "weights"])
    if op == "inner":
        kw.update(tol=rng.choice([0.0, 1e-4]), lmax=rng.randint(2, 10))
    if op == "job":
        kw.update(kmax=rng.randint(2, 5), lmax=rng.randint(2, 10), mode=0)
    if op in ("pqnr", "pdnr"):
        kw["lmax"] = rng.randint(2, 4)
    return _case(None, op, dims, nnz, rng.choice(ranks), **kw)


def _case(name, op, dims, nnz, rank, mode=0, zipf=0.0, nzipf=8, mu=2.0, precision="fp64", values="counts", tol=0.0,
          kmax=1, lmax=1, graph=False):
    """nnz counts tensors for a batch; zipf: exponent of the first nzipf modes' coordinates (0: uniform)."""
    c = dict(op=op, dims=dims, nnz=nnz, rank=rank, mode=mode, zipf=zipf, nzipf=nzipf, mu=mu, precision=precision,
             values=values, tol=tol, kmax=kmax, lmax=lmax, graph=graph)
    return c if name is None else dict(c, name=name)


# ---- inputs -----------------------------------------------------------------

def _dims(case):
    return [int(d) for d in case["dims"].split("x")]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _coords(g, dim, s, nnz):
    """Uniform, or bounded Zipf(s) with the rows in random order (duplicates kept)."""
    if s <= 0.0:
        return torch.randint(0, dim, (nnz,), generator=g, device="cuda", dtype=torch.int32)
    cdf = torch.cumsum(torch.arange(1, dim + 1, device="cuda", dtype=torch.float64) ** -s, 0)
    label = torch.randperm(dim, generator=g, device="cuda").to(torch.int32)
    out = torch.empty(nnz, device="cuda", dtype=torch.int32)
    for lo in range(0, nnz, 1 << 24):
        u = torch.rand(min(1 << 24, nnz - lo), generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
        out[lo:lo + u.numel()] = label[torch.searchsorted(cdf, u).clamp_(max=dim - 1)]
    return out


def _tensor(g, dims, nnz, zipf, nzipf, mu, values):
    idx = torch.empty((len(dims), nnz), device="cuda", dtype=torch.int32)
    for m, d in enumerate(dims):
        idx[m] = _coords(g, d, zipf if m < nzipf else 0.0, nnz)
    vals = 1.0 + torch.poisson(torch.full((nnz,), mu, device="cuda", dtype=torch.float32), generator=g).double()
    if values == "weights":
        vals *= 0.5 + torch.rand(nnz, generator=g, device="cuda", dtype=torch.float64)
    return idx, vals


def _model(g, dims, rank):
    """U(0,1) factors with columns scaled to sum to one, the sums' products in lambda."""
    lam, facs = torch.ones(rank, device="cuda", dtype=torch.float64), []
    for d in dims:
        a = torch.rand((d, rank), generator=g, device="cuda", dtype=torch.float64)
        s = a.sum(0)
        lam, facs = lam * s, facs + [a / s]
    return lam, facs


def _batch_sizes(case):
    """Sizes of a batch's tensors: a plan of the case, the same for every seed."""
    r = np.random.default_rng(case["nnz"])
    return [([int(d) for d in r.integers(50, 5001, 3)], int(round(math.exp(r.uniform(math.log(1e3), math.log(1e6))))),
             int(r.choice([8, 16, 32]))) for _ in range(case["nnz"])]


def _inputs(case, seed):
    g = _gen(seed)
    dims = _dims(case)
    idx, vals = _tensor(g, dims, case["nnz"], case["zipf"], case["nzipf"], case["mu"], case["values"])
    lam, A = _model(g, dims, case["rank"])
    return dims, idx, vals, lam, A


def _batch_inputs(case, seed):
    g = _gen(seed)
    for dims, nnz, rank in _batch_sizes(case):
        idx, vals = _tensor(g, dims, nnz, 0.0, 0, 2.0, "counts")
        yield dims, nnz, rank, idx, vals, _model(g, dims, rank)


METHOD = {"pqnr": cpapr.CPAPR_METHOD_PQNR, "pdnr": cpapr.CPAPR_METHOD_PDNR}


def _params(case):
    return dict(precision=cpapr.CPAPR_MIXED if case["precision"] == "mixed" else cpapr.CPAPR_FP64, tol=case["tol"],
                kmax=case["kmax"], lmax=case["lmax"], method=METHOD.get(case["op"], cpapr.CPAPR_METHOD_MU))


def prepare(case, seed):
    if case["op"] == "batch":
        return _prepare_batch(case, seed)
    dims, idx, vals, lam, A = _inputs(case, seed)
    n, R = case["mode"], case["rank"]
    st = dict(op=case["op"], mode=n, rank=R, dims=dims, lam0=lam, A0=A, params=_params(case))
    if case["op"] in ("coo", "job"):  # these start from the coordinates
        st.update(idx=idx, vals=vals, lam=lam.clone(), A=[a.clone() for a in A])
    else:
        st.update(plan=cpapr.Plan(dims, idx, vals, R, **st["params"]), lam=lam, A=A)
    st["B0"] = (A[n] * lam).contiguous()
    st["B"] = st["B0"].clone()
    st["out"] = torch.zeros_like(st["B0"])
    return st


def _prepare_batch(case, seed):
    items, stream = [], torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        for dims, nnz, R, idx, vals, (lam, A) in _batch_inputs(case, seed):
            items.append((cpapr.Plan(dims, idx, vals, R, stream=stream, **_params(case)), A, A[0] * lam))
        # all slots' B and Phi in one buffer each, so that they are reset and read at once
        starts = np.cumsum([0] + [(b.numel() + 31) // 32 * 32 for _, _, b in items])
        B0 = torch.zeros(int(starts[-1]), device="cuda", dtype=torch.float64)
        for (_, _, b), s in zip(items, starts):
            B0[s:s + b.numel()] = b.reshape(-1)
        B, Phi = B0.clone(), torch.zeros_like(B0)
        batch = cpapr.Batch(len(items), sum(p.tiles() for p, _, _ in items) + 1)
        for i, ((p, A, b), s) in enumerate(zip(items, starts)):
            batch.set(i, p, 0, B[s:s + b.numel()].view(b.shape), A, Phi[s:s + b.numel()].view(b.shape))
        batch.commit(stream)
    stream.synchronize()
    return dict(op="batch", batch=batch, stream=stream, B0=B0, B=B, Phi=Phi, lmax=case["lmax"], graph=case["graph"])


def run(st):
    op = st["op"]
    if op == "batch":
        with torch.cuda.stream(st["stream"]):
            st["B"].copy_(st["B0"])
        st["batch"].inner(st["lmax"], use_graph=st["graph"], stream=st["stream"])
        viol, updates, done = st["batch"].status(st["stream"])
        return dict(B=st["B"], Phi=st["Phi"], viol=np.array(viol), updates=np.array(updates), done=np.array(done))
    if op == "phi":
        return st["plan"].phi(st["mode"], st["B"], st["A"], out=st["out"])
    if op == "mttkrp":
        return st["plan"].mttkrp(st["mode"], st["A"], out=st["out"])
    if op == "loglik":
        return st["plan"].loglik(st["lam"], st["A"])
    if op == "coo":
        return cpapr.phi_coo(st["dims"], st["idx"], st["vals"], st["mode"], st["rank"], st["B"], st["A"], out=st["out"])
    if op == "job":
        st["lam"].copy_(st["lam0"])
        for a, a0 in zip(st["A"], st["A0"]):
            a.copy_(a0)
        plan = cpapr.Plan(st["dims"], st["idx"], st["vals"], st["rank"], **st["params"])
        stats = plan.solve(st["lam"], st["A"])
        plan.close()
        return dict(lam=st["lam"], A=st["A"], stats=stats)
    st["B"].copy_(st["B0"])  # the mode's starting point
    if op == "inner":
        phi, stats = st["plan"].mu_inner(st["mode"], st["B"], st["A"], phi_last=st["out"])
        return dict(B=st["B"], Phi=phi, stats=_inner_stats(stats))
    stats = st["plan"].pqnr_inner(st["mode"], st["B"], st["A"]) if op == "pqnr" else \
        st["plan"].pdnr_inner(st["mode"], st["B"], st["A"])
    return dict(B=st["B"], viol=stats["kkt_violation"])


def _inner_stats(s):
    return {k: s[k] for k in ("converged", "inner_iters", "kkt_violation", "phi_evals")}


# ---- work -------------------------------------------------------------------

def _pass_work(dims, nnz, R, mode, word, passes=1, reads_b=True):
    """Passes over a mode's nonzeros: coordinates of the other modes and the value
    once, the factors, B and the result once per pass."""
    n = len(dims)
    rows = [min(d, nnz) for d in dims]
    by = nnz * (4 * (n - 1) + 8) + rows[mode] * 8 + dims[mode] * R * 8 * (2 if reads_b else 1)
    by += sum(rows[m] for m in range(n) if m != mode) * R * word
    return by * passes, nnz * R * ((n - 2) + 4) * passes


def work(case):
    word = 4 if case["precision"] == "mixed" else 8
    if case["op"] == "batch":
        w = [_pass_work(d, z, r, 0, word, case["lmax"]) for d, z, r in _batch_sizes(case)]
        return {"bytes": sum(x for x, _ in w), "flops": sum(y for _, y in w)}
    dims, nnz, R, op = _dims(case), case["nnz"], case["rank"], case["op"]
    if op == "job":  # the coordinates in, every mode's passes, the likelihood
        w = [_pass_work(dims, nnz, R, m, word, case["kmax"] * case["lmax"]) for m in range(len(dims))]
        w += [_pass_work(dims, nnz, R, 0, 8)]
        return {"bytes": sum(x for x, _ in w) + nnz * (4 * len(dims) + 8) * (1 + len(dims)), "flops": sum(y for _, y in w)}
    passes = case["lmax"] if op in ("inner", "pqnr", "pdnr") else 1
    by, fl = _pass_work(dims, nnz, R, case["mode"], word, passes * (2 if op in ("pqnr", "pdnr") else 1), op != "mttkrp")
    if op == "pqnr":  # per step: m and four trial steps' changes beside Phi
        fl += passes * nnz * R * 2 * 4
    if op == "pdnr":  # per step: the Hessian of every row, and as above
        fl += passes * nnz * R * (R + 2 * 4)
    if op == "coo":
        by += nnz * (4 * len(dims) + 8)
    return {"bytes": by, "flops": fl}


# ---- the same results in plain torch, 64 bits -------------------------------

def _pi(idx, A, n, lo, hi):
    p = None
    for m in range(len(A)):
        if m != n:
            q = A[m][idx[m, lo:hi].long()]
            p = q if p is None else p * q
    return p


def _by_row(idx, vals, n):
    """The nonzeros in mode n's order, so that a row's terms are neighbours."""
    order = torch.sort(idx[n], stable=True).indices
    return idx[:, order], vals[order]


def _ref_phi(idx, vals, A, n, B, scale=True):
    """Phi (scale=False: MTTKRP) of nonzeros in mode n's order. Runs of up to 64
    neighbours of one row are summed, then 64 such sums, then the rest of each row."""
    out = torch.zeros_like(A[n])
    for lo in range(0, vals.numel(), CHUNK):
        hi = min(lo + CHUNK, vals.numel())
        x, i, s = _pi(idx, A, n, lo, hi), idx[n, lo:hi].long(), vals[lo:hi]
        if scale:
            s = s / (B[i] * x).sum(1).clamp_(min=EPS)
        x = x * s[:, None]
        for most in (64, 64, CHUNK):
            first = torch.arange(i.numel(), device=i.device) % most == 0
            first[1:] |= i[1:] != i[:-1]
            starts = torch.nonzero(first).reshape(-1)
            lengths = torch.diff(starts, append=starts.new_tensor([i.numel()]))
            x, i = torch.segment_reduce(x, "sum", lengths=lengths, axis=0, unsafe=True), i[starts]
        out[i] += x
    return out


def _ref_inner(idx, vals, A, n, B, lmax, tol):
    """MU inner loop: (B, last Phi, violation, updates, Phi evaluations, stopped)."""
    idx, vals = _by_row(idx, vals, n)
    for l in range(lmax):
        phi = _ref_phi(idx, vals, A, n, B)
        viol = float(torch.minimum(B, 1.0 - phi).abs().max())
        if tol > 0.0 and viol < tol:
            return B, phi, viol, l, l + 1, 1
        B = B * phi
    return B, phi, viol, lmax, lmax, 0


def _ref_loglik(idx, vals, lam, A):
    total, B = 0.0, A[0] * lam
    for lo in range(0, vals.numel(), CHUNK):
        hi = min(lo + CHUNK, vals.numel())
        m = (B[idx[0, lo:hi].long()] * _pi(idx, A, 0, lo, hi)).sum(1)
        total += float((vals[lo:hi] * m.clamp_(min=EPS).log()).sum())
    mass = lam.clone()
    for a in A:
        mass = mass * a.sum(0)
    return total - float(mass.sum())


def _ref_job(case, idx, vals, lam, A):
    N, last, inner, evals, viol = len(A), [None] * len(A), 0, 0, [0.0] * len(A)
    for k in range(case["kmax"]):
        for n in range(N):
            if k > 0:
                A[n] = torch.where((A[n] < KAPPA_TOL) & (last[n] > 1.0), A[n] + KAPPA, A[n])
            B, last[n], viol[n], up, ev, _ = _ref_inner(idx, vals, A, n, A[n] * lam, case["lmax"], case["tol"])
            inner, evals, lam = inner + up, evals + ev, B.sum(0)
            A[n] = torch.where(lam > 0, B / lam, torch.zeros_like(B))
    stats = dict(outer_iters=None, converged=None, inner_iters=None, phi_evals=None, row_steps=None, trial_evals=None,
                 kkt_violation=max(viol), loglik=_ref_loglik(idx, vals, lam, A))
    return dict(lam=lam, A=A, stats=stats)


def exact(case, seed):
    op = case["op"]
    if op in ("pqnr", "pdnr"):
        return None  # the row solvers' steps have no short statement here
    if op == "batch":
        B, Phi, viol = [], [], []
        for dims, nnz, R, idx, vals, (lam, A) in _batch_inputs(case, seed):
            b, p, v = _ref_inner(idx, vals, A, 0, A[0] * lam, case["lmax"], case["tol"])[:3]
            pad = torch.zeros(-b.numel() % 32, device="cuda", dtype=torch.float64)
            B, Phi, viol = B + [b.reshape(-1), pad], Phi + [p.reshape(-1), pad], viol + [v]
        return dict(B=torch.cat(B), Phi=torch.cat(Phi), viol=np.array(viol), updates=None, done=None)
    dims, idx, vals, lam, A = _inputs(case, seed)
    n = case["mode"]
    if op in ("phi", "coo"):
        return _ref_phi(*_by_row(idx, vals, n), A, n, A[n] * lam)
    if op == "mttkrp":
        return _ref_phi(*_by_row(idx, vals, n), A, n, None, scale=False)
    if op == "loglik":
        return _ref_loglik(idx, vals, lam, A)
    if op == "job":
        return _ref_job(case, idx, vals, lam, list(A))
    B, phi, viol, _, _, _ = _ref_inner(idx, vals, A, n, A[n] * lam, case["lmax"], case["tol"])
    return dict(B=B, Phi=phi, stats=dict(converged=None, inner_iters=None, kkt_violation=viol, phi_evals=None))
