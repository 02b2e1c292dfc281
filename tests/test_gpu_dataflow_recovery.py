"""The call after an aborted dataflow launch (bounded waits that the host
shortens on purpose; every kernel exits normally) reads nothing that an
earlier launch left in the mailboxes."""
import numpy as np
import pytest

import synth
from synth import CSR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1606_00541_amd as H  # noqa: E402


def chain(n):
    # unit lower bidiagonal: one level per row
    rp = np.concatenate([[0], np.arange(1, 2 * n, 2)]).astype(np.int32)
    col = np.empty(2 * n - 1, np.int32)
    val = np.empty(2 * n - 1)
    col[0], val[0] = 0, 1.0
    col[1::2], val[1::2] = np.arange(0, n - 1), -0.5
    col[2::2], val[2::2] = np.arange(1, n), 1.0
    return CSR(n, rp, col, val)


def rhs(n, seed):
    return torch.from_numpy(np.random.default_rng(seed).standard_normal((n, 1))).cuda()


@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_ilu_application_after_a_timeout(dt, which):
    A = synth.poisson3d(32)
    ref = H.ilu_setup(A, "ilu0", factor_dtype=dt, tune=H.tune_default(schedule="level_launch"))
    f = H.ilu_setup(A, "ilu0", factor_dtype=dt)
    plans = H.ilu_plans(f)
    assert all(H.tri_plan_stats(p)["dataflow"] and H.tri_plan_stats(p)["num_groups"] > 1 for p in plans)
    z, want = rhs(A.n, 0), rhs(A.n, 0)
    for seed in (1, 2):  # both mailbox halves have held values
        H.ilu_apply(f, rhs(A.n, seed), z)
    H.tri_plan_set_wait_limit(plans[which], 2)
    H.ilu_apply(f, rhs(A.n, 3), z)
    torch.cuda.synchronize()
    with pytest.raises(H.HecError) as e:
        H.ilu_apply(f, rhs(A.n, 3), z)
    assert e.value.name == "TIMEOUT"
    H.tri_plan_set_wait_limit(plans[which], 0)
    for seed in (4, 5, 6):
        r = rhs(A.n, seed)
        H.ilu_apply(f, r, z)
        H.ilu_apply(ref, r, want)
        torch.cuda.synchronize()
        for p in plans:
            H.tri_plan_check(p)
        assert torch.equal(z, want), seed


def test_queued_parts_after_a_timeout():
    # more parts than workgroups: those still in the queue when the waits give
    # up are never taken by that launch
    n = 1 << 15
    L = chain(n)
    f = H.tri_analyze(L, "lower", unit_diag=True,
                      tune=H.tune_default(schedule="owner_persistent", kernel_variant=6, part_rows=32))
    st = H.tri_plan_stats(f)
    assert st["queue"] and st["num_groups"] > 512
    ref = H.tri_analyze(L, "lower", unit_diag=True, tune=H.tune_default(schedule="level_launch"))
    x, want = rhs(n, 0), rhs(n, 0)
    for seed in (1, 2):
        H.tri_solve_lower(f, rhs(n, seed), x)
    H.tri_plan_set_wait_limit(f, 2)
    H.tri_solve_lower(f, rhs(n, 3), x)
    torch.cuda.synchronize()
    with pytest.raises(H.HecError) as e:
        H.tri_plan_check(f)
    assert e.value.name == "TIMEOUT"
    H.tri_plan_set_wait_limit(f, 0)
    for seed in (4, 5):
        b = rhs(n, seed)
        H.tri_solve_lower(f, b, x)
        H.tri_solve_lower(ref, b, want)
        torch.cuda.synchronize()
        H.tri_plan_check(f)
        assert torch.equal(x, want), seed
