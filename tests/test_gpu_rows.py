"""The row-by-row MU inner loop against the oracle, at row lengths around every
class of row (lane groups, waves, workgroups, teams of workgroups, heavy rows),
every launch shape by rank, both precisions, fixed schedules and KKT stops."""
import numpy as np
import pytest

import oracle
from paper_2307_03276_amd import cpapr, synth
from tests.gpu_util import assert_parity, dev, host

pytestmark = pytest.mark.gpu
# FP64: rows of up to 2e5 summed terms (error growth about sqrt(n) u) over a few
# multiplicative steps stay far below the library's parity gate; mixed: the
# factors' FP32 storage (6e-8 relative) enters every product N - 1 times and
# every step once
TOL64, TOL32 = 1e-12, 1e-5


def _tensor(lengths, others, seed, skew=0.0):
    """Mode 0 has rows of the given lengths; the other coordinates are random
    (skew > 0: Zipf, so rows have long fibers and hot coordinates)."""
    rng = np.random.default_rng(seed)
    lengths = np.asarray(lengths)
    nnz = int(lengths.sum())
    idx = np.empty((1 + len(others), nnz), np.int32)
    idx[0] = np.repeat(np.arange(lengths.size), lengths)
    for m, d in enumerate(others):
        if skew > 0:
            p = np.arange(1, d + 1) ** -skew
            idx[1 + m] = rng.permutation(d)[rng.choice(d, nnz, p=p / p.sum())]
        else:
            idx[1 + m] = rng.integers(0, d, nnz)
    o = rng.permutation(nnz)
    vals = 1.0 + rng.poisson(2.0, nnz)
    return synth.SparseTensor((lengths.size, *others), np.ascontiguousarray(idx[:, o]), vals.astype(np.float64))


def _check(X, R, lmax, tol=0.0, precision=cpapr.CPAPR_FP64, wait=None, seed=3, mode=0):
    M = synth.random_model(seed, X.dims, R)
    Bh = M.factors[mode] * M.lam
    P = cpapr.Plan.from_tensor(X, R, lmax=lmax, tol=tol, precision=precision)
    if wait is not None:
        cpapr.cpapr_plan_set_team_wait(P.handle, wait)
    B = dev(Bh)
    phi, st = P.mu_inner(mode, B, [dev(a) for a in M.factors])
    Bo, Po, hist, nup = oracle.mu_inner(X, mode, Bh, M.factors, lmax=lmax, tau=tol)
    t = TOL64 if precision == cpapr.CPAPR_FP64 else TOL32
    assert_parity(host(B), Bo, t, f"B R={R}", elementwise=precision == cpapr.CPAPR_FP64)
    assert_parity(host(phi), Po, t, f"Phi R={R}", elementwise=precision == cpapr.CPAPR_FP64)
    assert st["inner_iters"] == nup and st["phi_evals"] == nup + st["converged"]
    assert P.segments(mode) == np.unique(X.idx[mode]).size
    P.close()
    return hist


EDGES = [0, 1, 3, 4, 5, 19, 20, 21, 24, 25, 32, 33, 40, 41, 63, 64, 65, 80, 81, 160, 161, 319, 320, 321, 384, 385,
         639, 640, 641, 1279, 1280, 1281, 1536, 1537, 2048, 2049, 3000, 0, 0]


@pytest.mark.parametrize("R", [1, 2, 3, 4, 5, 8, 9, 10, 12, 13, 16, 17, 24, 25, 32, 33, 40, 48, 49, 63, 64])
def test_row_lengths_at_every_rank(R):
    _check(_tensor(EDGES, (37, 29), 10 + R), R, 3)


@pytest.mark.parametrize("others", [(50,), (41, 31, 17), (23, 17, 13, 11), (11, 9, 8, 7, 6, 5, 4)])
@pytest.mark.parametrize("precision", [cpapr.CPAPR_FP64, cpapr.CPAPR_MIXED])
def test_mode_counts(others, precision):
    _check(_tensor(EDGES, others, 40 + len(others)), 10, 3, precision=precision)
    _check(_tensor(EDGES, others, 50 + len(others)), 32, 2, precision=precision)


@pytest.mark.parametrize("R,longest", [(16, 170_000), (40, 45_000)])
@pytest.mark.parametrize("wait", [None, 0])
def test_teams_and_heavy_rows(R, longest, wait):
    """Rows of several workgroups, one longer than the largest team; with no wait
    for a team to start, its rows are left to one workgroup."""
    X = _tensor([longest, 5_000, 1_300, 20_000, 7, 0, 700], (200, 150), 7)
    _check(X, R, 4, wait=wait)


@pytest.mark.parametrize("wait", [None, 0])
@pytest.mark.parametrize("big", [False, True])
def test_stop_at_every_iteration(big, wait):
    """KKT stops before, inside and after the first chunk of iterations, with
    light rows, team rows and (big) heavy rows restored from their history."""
    X = _tensor(EDGES + [6_000] + ([200_000] if big else []), (60, 45), 9)
    hist = _check(X, 16, 20, seed=5, wait=wait)
    low = np.minimum.accumulate(hist)
    for l in (0, 1, 7, 15, 16, 18):
        _check(X, 16, 20, tol=float(low[l]) * (1 + 1e-9), seed=5, wait=wait)


@pytest.mark.parametrize("R,others,precision,frac", [
    (16, (900, 700), cpapr.CPAPR_FP64, False), (10, (3000, 2500), cpapr.CPAPR_MIXED, False),
    (32, (800, 60, 30), cpapr.CPAPR_FP64, True), (64, (500, 400), cpapr.CPAPR_FP64, True),
    (24, (3000, 300, 200), cpapr.CPAPR_MIXED, False), (5, (40000, 30000), cpapr.CPAPR_FP64, True)])
def test_heavy_rows_split_by_hot_coordinates(R, others, precision, frac):
    """Over 2^20 nonzeros, most in rows longer than a workgroup's registers:
    their nonzeros run by hot and cold parts, values exact in FP32 or not."""
    rng = np.random.default_rng(1)
    lengths = np.concatenate([[420_000, 160_000], rng.integers(1_500, 12_000, 90), EDGES])
    X = _tensor(lengths, others, 20 + R, skew=1.1)
    if frac:
        X = synth.SparseTensor(X.dims, X.idx, X.vals + 0.1)
    hist = _check(X, R, 3, precision=precision)
    _check(X, R, 3, tol=float(min(hist[:2])) * (1 + 1e-5), precision=precision)


@pytest.mark.parametrize("R,others,precision", [(6, (700, 60, 30), cpapr.CPAPR_FP64), (24, (500, 90, 40), cpapr.CPAPR_MIXED),
                                                (32, (800, 60, 30), cpapr.CPAPR_FP64), (48, (600, 50, 30), cpapr.CPAPR_MIXED)])
def test_four_modes_split_by_hot_coordinates(R, others, precision):
    """The same with four modes and a quarter of the nonzeros in light rows, beside
    which the heavy rows run by hot and cold parts (alone, the Phi launches)."""
    rng = np.random.default_rng(3)
    lengths = np.concatenate([[420_000, 160_000], rng.integers(1_500, 12_000, 40), [300] * 1_000, EDGES])
    X = _tensor(lengths, others, 220 + R, skew=1.1)
    hist = _check(X, R, 3, precision=precision)
    _check(X, R, 3, tol=float(min(hist[:2])) * (1 + 1e-5), precision=precision)


def test_hot_rows_at_rank_one():
    """Rank 1 with FP32-stored factors: more rows of the second factor would fit
    the LDS (35,840) than a plan has places for (17,920)."""
    X = _tensor([21_500] * 50, (30_000, 25_000), 33)
    _check(X, 1, 2, precision=cpapr.CPAPR_MIXED)


def test_empty_tensor_and_repeat():
    X = synth.SparseTensor((7, 5, 4), np.zeros((3, 0), np.int32), np.zeros(0))
    P = cpapr.Plan.from_tensor(X, 6, lmax=3, tol=0.0)
    M = synth.random_model(2, X.dims, 6)
    B = dev(M.factors[0])
    phi, st = P.mu_inner(0, B, [dev(a) for a in M.factors])
    assert not host(B).any() and not host(phi).any() and P.segments(0) == 0
    P.close()
    X = _tensor(EDGES + [30_000], (60, 45), 9)  # no atomics: every run gives the same bits
    M = synth.random_model(4, X.dims, 16)
    P = cpapr.Plan.from_tensor(X, 16, lmax=5, tol=0.0)
    out = []
    for _ in range(3):
        B = dev(M.factors[0] * M.lam)
        P.mu_inner(0, B, [dev(a) for a in M.factors])
        out.append(host(B))
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    P.close()


@pytest.mark.parametrize("use_graph", [False, True])
def test_batch_slots_row_by_row(use_graph):
    """A batch whose slots all run row by row: every launch shape and precision,
    light and team rows, a fixed schedule and stops in and after the first chunk,
    slots held, run again after a commit with other slots."""
    import torch
    stream = torch.cuda.Stream()
    rng = np.random.default_rng(4)
    with torch.cuda.stream(stream):
        items = []
        for i, R in enumerate([2, 6, 10, 16, 20, 32, 40, 64, 16, 10]):
            X = _tensor(EDGES + ([9_000] if i % 2 else []), (60, 45) if i % 3 else (30, 20, 10), 60 + i)
            M = synth.random_model(60 + i, X.dims, R)
            Bh = M.factors[0] * M.lam
            hist = oracle.mu_inner(X, 0, Bh, M.factors, lmax=20)[2]
            at = [0, 3, 14, 17, None][i % 5]
            tol = 0.0 if at is None else float(np.minimum.accumulate(hist)[at]) * (1 + 1e-5)
            prec = cpapr.CPAPR_MIXED if i >= 8 else cpapr.CPAPR_FP64
            P = cpapr.Plan.from_tensor(X, R, lmax=20, tol=tol, precision=prec)
            items.append((X, M, P, Bh, tol, prec, [dev(a) for a in M.factors], dev(Bh), dev(np.zeros_like(Bh))))
        b = cpapr.Batch(len(items), sum(it[2].tiles() for it in items) + 1)
        for i, (X, M, P, Bh, tol, prec, A, B, Phi) in enumerate(items):
            b.set(i, P, 0, B, A, Phi)
        b.commit()
        for turn in range(4):
            held = set()
            if turn == 2:
                held = {1, 4}
                b.hold([i in held for i in range(len(items))])
            if turn == 3:
                b.hold([0] * len(items))
                b.clear(0)
                b.commit()
            for it in items:
                it[7].copy_(dev(it[3]))
            b.inner(20, use_graph=use_graph)
            viol, upd, done = b.status()
            for i, (X, M, P, Bh, tol, prec, A, B, Phi) in enumerate(items):
                if i in held or (turn == 3 and i == 0):
                    assert np.array_equal(host(B), Bh)
                    continue
                Bo, Po, hist, nup = oracle.mu_inner(X, 0, Bh, M.factors, lmax=20, tau=tol)
                t, el = (TOL64, True) if prec == cpapr.CPAPR_FP64 else (TOL32, False)
                assert upd[i] == nup and done[i] == (1 if nup < 20 else 0)
                assert_parity(host(B), Bo, t, f"B slot {i}", elementwise=el)
                assert_parity(host(Phi), Po, t, f"Phi slot {i}", elementwise=el)
        b.close()


@pytest.mark.parametrize("R,others", [(4, (37, 29)), (8, (37, 29)), (10, (41, 31, 17)), (16, (60, 45)),
                                      (24, (23, 17, 13, 11)), (32, (41, 31, 17)), (48, (37, 29)), (64, (50,))])
def test_line_search_by_rows(R, others, lmax=2):
    """Row solves (line-search sums row by row) at every launch shape, with rows
    of every class, a long one cut into chunks, empty rows, and values not exact
    in FP32: iterates in lockstep with the oracle's. Two steps: from the third on
    PQNR divides by curvature s.y, differences of gradients that cancel on
    these nearly solved rows (the general line-search pass, taken by a plan with
    an explicit shape, is off by 4e-12 there too)."""
    X = _tensor(EDGES + [30_000], others, 80 + R)
    X = synth.SparseTensor(X.dims, X.idx, X.vals + 0.25)
    M = synth.random_model(81, X.dims, R)
    Bh = M.factors[0] * M.lam
    for method, run, ref in ((cpapr.CPAPR_METHOD_PQNR, "pqnr_inner", oracle.pqnr_inner),
                             (cpapr.CPAPR_METHOD_PDNR, "pdnr_inner", oracle.pdnr_inner)):
        P = cpapr.Plan.from_tensor(X, R, lmax=lmax, tol=0.0, method=method)
        B = dev(Bh)
        st = getattr(P, run)(0, B, [dev(a) for a in M.factors])
        Bo, info = ref(X, 0, Bh, M.factors, lmax=lmax)[:2]
        # the damped solve's condition bound (see the PDNR tests), never below the parity gate
        tol = TOL64 if method == cpapr.CPAPR_METHOD_PQNR else max(TOL64, 1.2e-16 * (1 + R * 4.0 ** (lmax - 1) / 1e-3))
        assert_parity(host(B), Bo, tol, f"{run} R={R}", elementwise=False)
        P.set_shape(*P.shape())
        B2 = dev(Bh)
        st2 = getattr(P, run)(0, B2, [dev(a) for a in M.factors])
        assert st["row_steps"] == st2["row_steps"] and st["trial_evals"] == st2["trial_evals"]
        assert_parity(host(B2), host(B), tol, f"{run} R={R} against the general pass", elementwise=False)
        P.close()


def test_plan_in_two_batches_and_a_single_loop():
    """One plan listed by two batches that run on streams of their own, and run by
    a single inner loop meanwhile; the batches then end before and after the plan."""
    import torch
    X = _tensor(EDGES + [9_000], (60, 45), 91)
    M = synth.random_model(91, X.dims, 10)
    Bh = M.factors[0] * M.lam
    Bo, Po, _, nup = oracle.mu_inner(X, 0, Bh, M.factors, lmax=20)
    P = cpapr.Plan.from_tensor(X, 10, lmax=20)
    A = [dev(a) for a in M.factors]
    runs = []
    for _ in range(2):
        s = torch.cuda.Stream()
        b = cpapr.Batch(1, P.tiles() + 1)
        B, Phi = dev(Bh), dev(np.zeros_like(Bh))
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            b.set(0, P, 0, B, A, Phi)
            b.commit()
        runs.append((s, b, B, Phi))
    for s, b, B, Phi in runs:
        with torch.cuda.stream(s):
            b.inner(20)
    single = dev(Bh)
    phi, st = P.mu_inner(0, single, A)
    torch.cuda.synchronize()
    for B, Phi in [(single, phi)] + [r[2:] for r in runs]:
        assert_parity(host(B), Bo, TOL64, "B")
        assert_parity(host(Phi), Po, TOL64, "Phi")
    assert st["inner_iters"] == nup
    runs[0][1].close()
    single = dev(Bh)
    P.mu_inner(0, single, A)
    assert_parity(host(single), Bo, TOL64, "B")
    P.close()
    runs[1][1].close()


def test_row_buffers_come_back_when_the_device_is_done():
    """A batch that ends (or commits) with its inner loop still queued keeps the
    plan's row buffers until the loop is done; a batch that only ran Phi never
    takes them, so a single loop takes its usual path (bit for bit)."""
    import torch
    X = _tensor(EDGES + [9_000, 30_000], (60, 45), 92)
    M = synth.random_model(92, X.dims, 10)
    Bh = M.factors[0] * M.lam
    P = cpapr.Plan.from_tensor(X, 10, lmax=20, tol=0.0)
    A = [dev(a) for a in M.factors]
    alone = dev(Bh)
    P.mu_inner(0, alone, A)
    assert_parity(host(alone), oracle.mu_inner(X, 0, Bh, M.factors, lmax=20, tau=0.0)[0], TOL64, "B")
    s = torch.cuda.Stream()
    b = cpapr.Batch(1, P.tiles() + 1)
    B, Phi = dev(Bh), dev(np.zeros_like(Bh))
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        b.set(0, P, 0, B, A, Phi)
        b.commit()
        b.run()
    single = dev(Bh)
    P.mu_inner(0, single, A)
    torch.cuda.synchronize()
    assert torch.equal(single, alone)
    for end in ("commit", "close"):
        with torch.cuda.stream(s):
            B.copy_(dev(Bh))
            torch.cuda._sleep(50_000_000)  # some 20 ms: the loop is still queued when the batch ends
            b.inner(20)
        getattr(b, end)()
        single = dev(Bh)
        P.mu_inner(0, single, A)
        torch.cuda.synchronize()
        assert torch.equal(single, alone)
        assert_parity(host(B), host(alone), TOL64, "B of the batch")
    P.close()


def test_deterministic_plans_repeat_bit_for_bit():
    """deterministic = 1: the same bits whether or not teams of workgroups could
    meet, and whether or not a batch runs inner loops of the plan."""
    import torch
    X = _tensor(EDGES + [9_000, 30_000], (60, 45), 93)
    M = synth.random_model(93, X.dims, 10)
    Bh = M.factors[0] * M.lam
    Bo = oracle.mu_inner(X, 0, Bh, M.factors, lmax=6, tau=0.0)[0]
    A = [dev(a) for a in M.factors]
    P = cpapr.Plan.from_tensor(X, 10, lmax=6, tol=0.0, deterministic=1)

    def loop():
        B = dev(Bh)
        P.mu_inner(0, B, A)
        lam, F = dev(M.lam), [dev(a) for a in M.factors]
        P.solve(lam, F)
        return [B, lam, *F]

    first = loop()
    assert_parity(host(first[0]), Bo, TOL64, "B")
    cpapr.cpapr_plan_set_team_wait(P.handle, 0)
    for again in (loop(), loop()):
        assert all(torch.equal(x, y) for x, y in zip(first, again))
    b = cpapr.Batch(1, P.tiles() + 1)
    B, Phi = dev(Bh), dev(np.zeros_like(Bh))
    b.set(0, P, 0, B, A, Phi)
    b.commit()
    b.inner(6)
    assert all(torch.equal(x, y) for x, y in zip(first, loop()))
    b.close()
    P.close()


@pytest.mark.parametrize("R,others,precision", [(16, (900, 700), cpapr.CPAPR_FP64), (24, (40, 30, 20, 10), cpapr.CPAPR_MIXED),
                                                (10, (700, 500, 90), cpapr.CPAPR_FP64)])
def test_stops_of_large_tensors(R, others, precision, lmax=5):
    """From 2^20 nonzeros on the first chunk is as long as the mode's last loop,
    and heavy rows halt at the stop: stops before, at and after the end of a
    chunk, for a new plan and for one whose last loop stopped elsewhere."""
    rng = np.random.default_rng(2)
    lengths = np.concatenate([[420_000, 160_000], rng.integers(1_500, 12_000, 90), [500] * 600, EDGES])
    X = _tensor(lengths, others, 120 + R, skew=1.1)
    M = synth.random_model(7, X.dims, R)
    Bh, A = M.factors[0] * M.lam, [dev(a) for a in M.factors]
    steps = [Bh]
    for l in range(1, lmax + 1):
        steps.append(oracle.mu_inner(X, 0, Bh, M.factors, lmax=l, tau=0.0)[0])
    hist = oracle.mu_inner(X, 0, Bh, M.factors, lmax=lmax, tau=0.0)[2]
    low = np.minimum.accumulate(hist)
    t, el = (TOL64, True) if precision == cpapr.CPAPR_FP64 else (TOL32, False)
    for l in range(lmax + 1):
        tol = float(low[l]) * (1 + 1e-4) if l < lmax else float(low[-1]) * 0.5
        stop = next((k for k in range(lmax) if hist[k] < tol), lmax)
        P = cpapr.Plan.from_tensor(X, R, lmax=lmax, tol=tol, precision=precision)
        for turn in range(3):
            if turn == 2 and stop > 0:  # the last loop ended earlier: one that starts near its end
                B = dev(steps[stop])
                P.mu_inner(0, B, A)
            B = dev(Bh)
            phi, st = P.mu_inner(0, B, A)
            assert st["inner_iters"] == stop and st["phi_evals"] == min(stop + 1, lmax)
            assert_parity(host(B), steps[stop], t, f"B, stop at {stop}, turn {turn}", elementwise=el)
        P.close()


def test_batch_of_rows_just_longer_than_a_workgroups_registers():
    """Such rows' history bounds the iterations of a batch's chunks (R = 64: 6 of
    the 16); a stop in each chunk, and one slot with a fixed schedule."""
    X = _tensor([330] * 300, (37, 29), 17)
    M = synth.random_model(17, X.dims, 64)
    Bh, A = M.factors[0] * M.lam, [dev(a) for a in M.factors]
    hist = oracle.mu_inner(X, 0, Bh, M.factors, lmax=20, tau=0.0)[2]
    low = np.minimum.accumulate(hist)
    slots = []
    for l in (0, 3, 5, 6, 9, 15, 19, None):
        tol = 0.0 if l is None else float(low[l]) * (1 + 1e-6)
        slots.append((cpapr.Plan.from_tensor(X, 64, lmax=20, tol=tol), tol, dev(Bh), dev(np.zeros_like(Bh))))
    b = cpapr.Batch(len(slots), sum(P.tiles() for P, *_ in slots) + 1)
    for i, (P, _, B, Phi) in enumerate(slots):
        b.set(i, P, 0, B, A, Phi)
    b.commit()
    b.inner(20)
    _, upd, _ = b.status()
    for i, (P, tol, B, Phi) in enumerate(slots):
        Bo, Po, _, nup = oracle.mu_inner(X, 0, Bh, M.factors, lmax=20, tau=tol)
        assert upd[i] == nup
        assert_parity(host(B), Bo, TOL64, f"B slot {i}")
        assert_parity(host(Phi), Po, TOL64, f"Phi slot {i}")
    b.close()


def test_explicit_segmented_variant_runs_the_tile_kernel():
    """CPAPR_VARIANT_SEGMENTED: the inner loop by Phi launches, bit for bit those of a
    plan with an explicit shape (rows of at most 24 of a tile's 32 nonzeros, whose
    two atomic sums commute)."""
    X = _tensor(EDGES[:10] * 12, (60, 45), 94)
    M = synth.random_model(94, X.dims, 10)
    Bh, A = M.factors[0] * M.lam, [dev(a) for a in M.factors]
    out = []
    for variant, shaped in ((cpapr.CPAPR_VARIANT_SEGMENTED, False), (cpapr.CPAPR_VARIANT_AUTO, True),
                            (cpapr.CPAPR_VARIANT_AUTO, False)):
        P = cpapr.Plan.from_tensor(X, 10, lmax=6, tol=0.0, variant=variant)
        if shaped:
            P.set_shape(*P.shape())
        B = dev(Bh)
        P.mu_inner(0, B, A)
        out.append(host(B))
        P.close()
    assert np.array_equal(out[0], out[1]) and not np.array_equal(out[0], out[2])
    assert_parity(out[0], oracle.mu_inner(X, 0, Bh, M.factors, lmax=6, tau=0.0)[0], TOL64, "B")


@pytest.mark.parametrize("use_graph", [False, True])
def test_batch_whose_slots_mostly_stop_at_once(use_graph, lmax=12):
    """After a round in which most slots stopped at their first iteration the batch
    takes that one by the Phi / update launches: the same results in the round
    that shows it and in the next ones, for slots that stop there, later or not at
    all."""
    import torch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        slots = []
        for i, at in enumerate([0, 0, 3, None, 0, 0]):
            X = _tensor(EDGES + ([9_000] if i % 2 else []), (60, 45), 160 + i)
            M = synth.random_model(160 + i, X.dims, 10)
            Bh = M.factors[0] * M.lam
            low = np.minimum.accumulate(oracle.mu_inner(X, 0, Bh, M.factors, lmax=lmax, tau=0.0)[2])
            tol = 0.0 if at is None else float(low[at]) * (1 + 1e-6)
            prec = cpapr.CPAPR_MIXED if i == 4 else cpapr.CPAPR_FP64
            if prec == cpapr.CPAPR_MIXED:
                tol = float(low[0]) * 1.01
            ref = oracle.mu_inner(X, 0, Bh, M.factors, lmax=lmax, tau=tol)
            P = cpapr.Plan.from_tensor(X, 10, lmax=lmax, tol=tol, precision=prec)
            slots.append((P, Bh, ref, prec, [dev(a) for a in M.factors], dev(Bh), dev(np.zeros_like(Bh))))
        b = cpapr.Batch(len(slots), sum(it[0].tiles() for it in slots) + 1)
        for i, (P, Bh, ref, prec, A, B, Phi) in enumerate(slots):
            b.set(i, P, 0, B, A, Phi)
        b.commit()
        for turn in range(4):
            for it in slots:
                it[5].copy_(dev(it[1]))
            b.inner(lmax, use_graph=use_graph)
            viol, upd, done = b.status()
            for i, (P, Bh, (Bo, Po, hist, nup), prec, A, B, Phi) in enumerate(slots):
                t, el = (TOL64, True) if prec == cpapr.CPAPR_FP64 else (TOL32, False)
                assert upd[i] == nup and done[i] == (1 if nup < lmax else 0), (turn, i)
                assert_parity(host(B), Bo, t, f"B slot {i} turn {turn}", elementwise=el)
                assert_parity(host(Phi), Po, t, f"Phi slot {i} turn {turn}", elementwise=el)
        b.close()


@pytest.mark.parametrize("use_graph", [False, True])
def test_batch_with_a_slot_that_cannot_run_row_by_row(use_graph):
    """A slot with a row longer than the largest team: the whole batch takes the
    general launches; without that slot, after a commit, the rows again."""
    import torch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        slots = []
        for i, extra in enumerate([[], [170_000], [9_000]]):
            X = _tensor(EDGES + extra, (60, 45), 170 + i)
            M = synth.random_model(170 + i, X.dims, 16)
            Bh = M.factors[0] * M.lam
            ref = oracle.mu_inner(X, 0, Bh, M.factors, lmax=4, tau=0.0)
            P = cpapr.Plan.from_tensor(X, 16, lmax=4, tol=0.0)
            slots.append((P, Bh, ref, [dev(a) for a in M.factors], dev(Bh), dev(np.zeros_like(Bh))))
        b = cpapr.Batch(len(slots), sum(it[0].tiles() for it in slots) + 1)
        for i, (P, Bh, ref, A, B, Phi) in enumerate(slots):
            b.set(i, P, 0, B, A, Phi)
        b.commit()
        for turn in range(3):
            if turn == 2:
                b.clear(1)
                b.commit()
            for it in slots:
                it[4].copy_(dev(it[1]))
            b.inner(4, use_graph=use_graph)
            for i, (P, Bh, (Bo, Po, _, _), A, B, Phi) in enumerate(slots):
                if turn == 2 and i == 1:
                    continue
                assert_parity(host(B), Bo, TOL64, f"B slot {i} turn {turn}")
                assert_parity(host(Phi), Po, TOL64, f"Phi slot {i} turn {turn}")
        b.close()
