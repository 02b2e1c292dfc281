"""Dataflow plans called with more right-hand sides than their parts hold at
once: as many are taken as one part per compute unit would take, with the bits
of one launch per level."""
import numpy as np
import pytest

import synth
from synth import CSR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1606_00541_amd as H  # noqa: E402


def tridiagonal(systems, rows):
    """Independent tridiagonal systems as one matrix, and their bounds."""
    n = systems * rows
    i = np.arange(n)
    first, last = i % rows == 0, i % rows == rows - 1
    col = np.stack([i - 1, i, i + 1], axis=1)
    keep = np.stack([~first, np.ones(n, bool), ~last], axis=1)
    val = np.stack([-np.ones(n), np.full(n, 2.5), -np.ones(n)], axis=1)
    rp = np.concatenate([[0], np.cumsum(keep.sum(axis=1))]).astype(np.int32)
    return CSR(n, rp, col[keep].astype(np.int32), val[keep]), (np.arange(systems + 1) * rows).astype(np.int32)


def test_parts_that_end_with_the_systems_take_what_even_parts_take():
    A, ptr = tridiagonal(220, 2300)
    r = torch.from_numpy(np.random.default_rng(1).standard_normal((A.n, 9))).cuda()
    out = []
    for t in (dict(schedule="level_launch"), {}):
        f = H.batch_setup(A, ptr, "ilu0", factor_dtype="f32", tune=H.tune_default(**t))
        z = torch.empty_like(r)
        H.ilu_apply(f, r, z)
        torch.cuda.synchronize()
        out.append(z)
    assert H.tri_plan_stats(H.ilu_plans(f)[0])["dataflow"] == 1
    assert torch.equal(out[0], out[1])


def share_parts(pl, pu):
    """Whether both triangles run in one launch: parts of the same rows, one ELL
    width, no CSR tail."""
    st, own = [], []
    for p in (pl, pu):
        st.append(H.tri_plan_stats(p))
        x, o = H.tri_plan_layout(p)
        own.append(np.empty_like(o))
        own[-1][x] = o
    return (all(s["dataflow"] and s["nnz_tail"] == 0 for s in st) and np.array_equal(*own)
            and st[0]["ell_width"] == st[1]["ell_width"] and st[0]["num_groups"] == st[1]["num_groups"])


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("shape,counts", [((32, 32, 32), (2, 3, 5, 16)), ((64, 64, 1), (4, 5, 7, 31)), ((200, 200, 1), (3, 6)),
                                          ((64, 64, 64), (2, 4)), ((700, 700, 1), (2, 5))])
def test_groups_side_by_side(shape, counts, dt):
    # default plans (made for one right-hand side) of several parts, in place
    # as well: one group, uneven groups, more groups than one launch runs
    A = synth.poisson3d(*shape)
    ref = H.ilu_setup(A, "ilu0", factor_dtype=dt, tune=H.tune_default(schedule="level_launch"))
    f = H.ilu_setup(A, "ilu0", factor_dtype=dt)
    pl, pu = H.ilu_plans(f)
    st = H.tri_plan_stats(pl)
    assert st["dataflow"] and st["num_groups"] > 1 and st["nexport"] > 0 and share_parts(pl, pu)
    for nrhs in counts + (1,):
        r = torch.from_numpy(np.random.default_rng(nrhs).standard_normal((A.n, nrhs))).cuda()
        want = torch.empty_like(r)
        H.ilu_apply(ref, r, want)
        for _ in range(3):  # both mailbox halves
            z = torch.empty_like(r)
            H.ilu_apply(f, r, z)
            assert torch.equal(z, want), nrhs
        z = r.clone()
        H.ilu_apply(f, z, z)
        assert torch.equal(z, want), nrhs
        H.tri_solve_lower(pl, r, z)
        H.tri_solve_upper(pu, z, z)
        assert torch.equal(z, want), nrhs
        for p in (pl, pu):
            H.tri_plan_check(p)


@pytest.mark.parametrize("shape,nrhs", [((32, 32, 32), 16), ((64, 64, 1), 16), ((300, 300, 1), 8)])
def test_more_columns_than_planned_cost_less_than_a_solve_each(shape, nrhs):
    # a quarter of it is the line: side by side they take little more than one
    A = synth.poisson3d(*shape)
    f = H.ilu_setup(A, "ilu0")
    times = []
    for k in (1, nrhs):
        r = torch.zeros(A.n, k, dtype=torch.float64, device="cuda")
        z = torch.empty_like(r)
        H.ilu_apply(f, r, z)
        laps = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                H.ilu_apply(f, r, z)
            b.record()
            b.synchronize()
            laps.append(a.elapsed_time(b))
        times.append(min(laps))
    assert times[1] < times[0] * nrhs / 4, times
