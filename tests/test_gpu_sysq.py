"""The system queue at the edges of its ranges, bit for bit against one launch
per level (the same summation order): levels of one row to more than two pieces,
values read beyond the LDS ring, and columns in and out of whole groups."""
import numpy as np
import pytest

from synth import CSR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1606_00541_amd as H  # noqa: E402

# rows of a level, levels, levels back to the oldest value read.  FP64 rings of
# four columns hold 5119 rows, and half of that where values are read beyond
# them: the third to last systems read beyond theirs.
SYSTEMS = [(1, 1, 1), (1, 9, 3), (30, 110, 100), (100, 70, 45), (600, 30, 20), (1100, 12, 9)]


def banded(systems, symmetric):
    """Independent systems whose levels hold m rows each: a row reads the row
    above it, its neighbour, and two rows `back` levels away."""
    rows, base = [], 0
    for m, nlev, back in systems:
        for i in range(m * nlev):
            c = {i - m, i - m - 1, i - m * back, i - m * back - 2} if i >= m else set()
            c = {j for j in c if 0 <= j and j // m < i // m}
            if symmetric:
                up = {i + m, i + m + 1, i + m * back, i + m * back + 2}
                c |= {j for j in up if j < m * nlev}
            rows.append(sorted(base + j for j in c | {i}))
        base += m * nlev
    rp = np.cumsum([0] + [len(r) for r in rows]).astype(np.int32)
    ci = np.concatenate([np.asarray(r) for r in rows]).astype(np.int32)
    rng = np.random.default_rng(base)
    v = rng.uniform(-0.2, 0.2, ci.size)
    v[ci == np.repeat(np.arange(base), np.diff(rp))] = rng.uniform(1.5, 2.5, base)
    return CSR(base, rp, ci, v)


QUEUE = dict(schedule="level_persistent", kernel_variant=7)


@pytest.mark.parametrize("vec", ["f64", "f32"])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("system", SYSTEMS)
def test_one_system(system, dt, vec):
    L = banded([system], False)
    rng = np.random.default_rng(3)
    vt = torch.float64 if vec == "f64" else torch.float32
    for nrhs in (1, 4, 6, 8):
        b = torch.from_numpy(rng.standard_normal((L.n, nrhs))).to(vt).cuda()
        out = []
        for t in (dict(schedule="level_launch"), dict(QUEUE, max_nrhs=nrhs)):
            p = H.tri_analyze(L, "lower", dtype=dt, tune=H.tune_default(**t))
            x = torch.empty_like(b)
            for _ in range(2):
                x.fill_(float("nan"))
                H.tri_solve_lower(p, b, x)
            torch.cuda.synchronize()
            H.tri_plan_check(p)
            out.append(x)
        assert H.tri_plan_stats(p)["sysq"] == 1
        assert torch.equal(out[0], out[1]), nrhs


@pytest.mark.parametrize("nrhs,most", [(4, 4), (16, 16), (8, 16), (5, 8), (16, 8)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_batched_factors(dt, nrhs, most):
    # both triangles through the workspace between them; more systems than one
    # so that items of different widths follow each other in a workgroup
    systems = SYSTEMS + SYSTEMS[:4]
    A = banded(systems, True)
    ptr = np.cumsum([0] + [m * nlev for m, nlev, _ in systems]).astype(np.int32)
    r = torch.from_numpy(np.random.default_rng(5).standard_normal((A.n, nrhs))).cuda()
    out = []
    for t in (dict(schedule="level_launch"), dict(QUEUE, max_nrhs=most)):
        f = H.batch_setup(A, ptr, "ilu0", factor_dtype=dt, tune=H.tune_default(**t))
        z = torch.full_like(r, float("nan"))
        if nrhs > most and "max_nrhs" in t:  # the rings that max_nrhs columns fill do not take twice as many
            with pytest.raises(H.HecError, match="LDS ring exceeds"):
                H.ilu_apply(f, r, z)
            return
        for _ in range(2):
            H.ilu_apply(f, r, z)
        torch.cuda.synchronize()
        out.append(z)
    assert torch.equal(out[0], out[1])


def test_automatic_choice_by_columns():
    # too few systems for half the compute units, enough with their columns;
    # any number of right-hand sides is accepted
    import scipy.sparse as sp
    import synth

    P = synth.poisson3d(32)
    m = sp.block_diag([P.to_scipy()] * 16).tocsr()
    m.sort_indices()
    A = CSR(m.shape[0], m.indptr.astype(np.int32), m.indices.astype(np.int32), m.data.copy())
    ptr = (np.arange(17) * P.n).astype(np.int32)
    fs = [H.batch_setup(A, ptr, "ilu0", tune=H.tune_default(**t)) for t in (dict(schedule="level_launch"), dict(max_nrhs=16))]
    assert H.tri_plan_stats(H.ilu_plans(fs[1])[0])["sysq"] == 1
    for nrhs in (1, 5, 16, 48):
        r = torch.from_numpy(np.random.default_rng(nrhs).standard_normal((A.n, nrhs))).cuda()
        z = [torch.full_like(r, float("nan")) for _ in fs]
        for f, x in zip(fs, z):
            H.ilu_apply(f, r, x)
        torch.cuda.synchronize()
        assert torch.equal(z[0], z[1]), nrhs


# even systems, enough for items of many columns: levels of one row, of rows
# that do not fill a wavefront's share, of one and of several pieces
EVEN = [((1, 5, 1), 400), ((30, 12, 2), 300), ((129, 5, 1), 290), ((600, 3, 2), 270), ((1100, 2, 1), 260)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("system,count", EVEN)
def test_several_threads_to_a_row(system, count, dt):
    # 2, 6: two threads of one column; 8, 24: two of four; 16: four of four
    A = banded([system] * count, True)
    ptr = (np.arange(count + 1) * system[0] * system[1]).astype(np.int32)
    f = [H.batch_setup(A, ptr, "ilu0", factor_dtype=dt, tune=H.tune_default(**t))
         for t in (dict(schedule="level_launch"), dict(QUEUE, max_nrhs=24))]
    assert H.tri_plan_stats(H.ilu_plans(f[1])[0])["sysq"] == 1
    for nrhs in (1, 2, 4, 6, 7, 8, 16, 24):
        for vt in (torch.float64, torch.float32):
            r = torch.from_numpy(np.random.default_rng(nrhs).standard_normal((A.n, nrhs))).to(vt).cuda()
            out = []
            for h in f:
                z = torch.full_like(r, float("nan"))
                for _ in range(2):
                    H.ilu_apply(h, r, z)
                H.tri_solve_lower(H.ilu_plans(h)[0], r, r2 := torch.empty_like(r))
                out.append((z, r2))
            torch.cuda.synchronize()
            assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), nrhs


def test_finished_problems_of_an_item():
    # BiCGSTAB with zero right-hand sides, finished from the start, in some of
    # the columns that an item of eight solves together
    import synth

    A = synth.poisson3d(48, 40, 36)
    owner = synth.grid_bisection(48, 40, 36, 300)
    b = torch.from_numpy(np.random.default_rng(2).standard_normal((A.n, 16))).cuda()
    b[:, [1, 8, 9, 10, 11, 12, 13, 14, 15]] = 0.0
    M = H.hec_from_csr(A)
    out = []
    for t in (dict(schedule="level_launch"), QUEUE):
        s = H.ras_setup(A, 300, owner, overlap=1, factor_dtype="f32", tune=H.tune_default(max_nrhs=16, **t))
        x = torch.zeros_like(b)
        st, info = H.krylov_solve(M, s, b, x, method="bicgstab", rtol=1e-8)
        assert st == 0
        out.append((x, [q.iters for q in info]))
    assert out[0][1] == out[1][1] and torch.equal(out[0][0], out[1][0])


def test_many_even_systems_share_their_rows_between_columns():
    # 512 subdomains: sixteen columns together, not one or four at a time
    import synth

    A = synth.poisson3d(96)
    s = H.ras_setup(A, 512, synth.grid_bisection(96, 96, 96, 512), overlap=0, factor_dtype="f32",
                    tune=H.tune_default(max_nrhs=16, **QUEUE))
    times = {}
    for k in (1, 4, 16):
        r = torch.zeros(A.n, k, dtype=torch.float64, device="cuda")
        z = torch.empty_like(r)
        laps = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                H.ras_apply(s, r, z)
            b.record()
            b.synchronize()
            laps.append(a.elapsed_time(b))
        times[k] = min(laps)
    assert times[4] < 2.2 * times[1] and times[16] < 4.5 * times[1], times


def uneven_slabs(nx, parts, nrhs, **tune):
    """RAS in FP64 on contiguous subdomains of 1/4 to some 3 times the average size."""
    import synth

    A = synth.poisson3d(nx)
    lo = A.n // (4 * parts)
    size = lo + np.floor(np.random.default_rng(parts).dirichlet(np.full(parts, 2.0)) * (A.n - parts * lo)).astype(int)
    size[-1] += A.n - size.sum()
    owner = np.repeat(np.arange(parts, dtype=np.int32), size)
    return A, H.ras_setup(A, parts, owner, overlap=1, tune=H.tune_default(max_nrhs=nrhs, **tune))


def test_few_columns_of_a_few_uneven_systems():
    # a plan made for 16 right-hand sides that the queue's columns chose; calls
    # with few of them run on the barrier-free kernel, in a graph on the queue
    A, ref = uneven_slabs(100, 32, 16, schedule="level_launch")
    _, s = uneven_slabs(100, 32, 16)
    for step in range(2):
        for nrhs in (1, 2, 3, 4, 8, 16, 20):
            r = torch.from_numpy(np.random.default_rng(nrhs).standard_normal((A.n, nrhs))).cuda()
            want = torch.empty_like(r)
            H.ras_apply(ref, r, want)
            for _ in range(2):
                z = torch.full_like(r, float("nan"))
                H.ras_apply(s, r, z)
                assert torch.equal(z, want), (step, nrhs)
            if nrhs in (1, 16):
                g = H.hec_graph_capture(s, r, z)
                for _ in range(3):
                    z.fill_(float("nan"))
                    H.hec_graph_launch(g)
                    H.ras_apply(s, r, torch.empty_like(r))
                    torch.cuda.synchronize()
                    assert torch.equal(z, want), (step, nrhs)
        val = A.val * np.where(A.col == np.repeat(np.arange(A.n), np.diff(A.rowptr)), 1.25, 1.0)
        B = CSR(A.n, A.rowptr, A.col, val)
        for h in (ref, s):
            H.ras_refactor(h, B)


def test_few_columns_cost_what_the_barrier_free_kernel_takes():
    times = []
    for tune in (dict(schedule="level_launch", kernel_variant=5), {}):
        A, s = uneven_slabs(100, 32, 16, **tune)
        r = torch.zeros(A.n, 1, dtype=torch.float64, device="cuda")
        z = torch.empty_like(r)
        laps = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                H.ras_apply(s, r, z)
            b.record()
            b.synchronize()
            laps.append(a.elapsed_time(b))
        times.append(min(laps))
    assert times[1] < 1.1 * times[0], times


@pytest.mark.parametrize("nrhs", [1, 4, 5, 16])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_rows_that_read_more_than_two_values_beyond_the_ring(dt, nrhs):
    # ILU(1) of thin slabs: up to four such values a row
    import synth

    A = synth.poisson3d(40, 40, 80)
    owner = ((np.arange(A.n) * 130) // A.n).astype(np.int32)
    r = torch.from_numpy(np.random.default_rng(nrhs).standard_normal((A.n, nrhs))).cuda()
    out = []
    for t in (dict(schedule="level_launch"), dict(QUEUE, max_nrhs=max(4, nrhs))):
        s = H.ras_setup_ilu(A, 130, owner, overlap=1, kind="iluk", k=1, factor_dtype=dt, tune=H.tune_default(**t))
        z = torch.full_like(r, float("nan"))
        for _ in range(2):
            H.ras_apply(s, r, z)
        torch.cuda.synchronize()
        out.append(z)
    assert torch.equal(out[0], out[1])


def far_systems(m, nlev, backs):
    """Systems of levels of m rows that read the row above and one row from each
    of `backs` levels away."""
    rows = []
    for i in range(m * nlev):
        c = {i - m} | {i - m * b for b in backs}
        rows.append(sorted(j for j in c if j >= 0) + [i])
    rp = np.cumsum([0] + [len(q) for q in rows]).astype(np.int32)
    ci = np.concatenate([np.asarray(q) for q in rows]).astype(np.int32)
    v = np.random.default_rng(m).uniform(-0.2, 0.2, ci.size)
    v[rp[1:] - 1] = 1.5
    return CSR(m * nlev, rp, ci, v)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("backs", [(90,), (88, 90), (80, 88, 90), (70, 80, 88, 90), (60, 70, 80, 88, 90)])
def test_one_to_five_values_beyond_the_ring(backs, dt):
    # levels of 300 rows: FP64 rings of four columns hold 17 levels, FP32 34
    L = far_systems(300, 120, backs)
    for nrhs in (1, 4, 8):
        b = torch.from_numpy(np.random.default_rng(nrhs).standard_normal((L.n, nrhs))).cuda()
        out = []
        for t in (dict(schedule="level_launch"), dict(QUEUE, max_nrhs=nrhs)):
            p = H.tri_analyze(L, "lower", dtype=dt, tune=H.tune_default(**t))
            x = torch.full_like(b, float("nan"))
            for _ in range(2):
                H.tri_solve_lower(p, b, x)
            torch.cuda.synchronize()
            out.append(x)
        assert torch.equal(out[0], out[1]), nrhs


def test_four_values_beyond_the_ring_stay_on_the_pipelined_kernel():
    # the plain kernel takes about eight times as long as this one
    times = []
    for backs in ((88, 90), (70, 80, 88, 90)):
        L = far_systems(300, 120, backs)
        p = H.tri_analyze(L, "lower", dtype="f32", tune=H.tune_default(**dict(QUEUE, max_nrhs=4)))
        b = torch.zeros(L.n, 4, dtype=torch.float64, device="cuda")
        x = torch.empty_like(b)
        laps = []
        for _ in range(6):
            e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e[0].record()
            for _ in range(5):
                H.tri_solve_lower(p, b, x)
            e[1].record()
            e[1].synchronize()
            laps.append(e[0].elapsed_time(e[1]))
        times.append(min(laps))
    assert times[1] < 2.5 * times[0], times
