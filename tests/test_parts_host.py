"""Host-only checks of the parts the automatic schedule gives the dataflow
kernel (no GPU is touched)."""
import time

import numpy as np
import pytest

import synth
from synth import CSR

import paper_1606_00541_amd as H


def plans(A, **tune):
    f = H.ilu_setup(A, "ilu0", tune=H.tune_default(host_only=1, **tune))
    return f, [H.tri_plan_stats(p) for p in H.ilu_plans(f)]


@pytest.mark.parametrize("tune", [dict(num_groups=64), dict(num_groups=256), dict(part_rows=512), dict(partition=3),
                                  dict(partition=1), dict(partition=2), dict()])
def test_u_of_an_ilu_is_cut_like_a_triangle_of_its_own(tune):
    A = synth.poisson3d(32)
    f, (_, u) = plans(A, **tune)
    rp, ci, v = H.ilu_factor(f, 1)
    alone = H.tri_plan_stats(H.tri_analyze(CSR(A.n, rp, ci, v), "upper", tune=H.tune_default(host_only=1, **tune)))
    assert u["dataflow"] == alone["dataflow"] == 1
    for key in ("num_groups", "nexport", "nremote", "crit_hops"):
        assert u[key] == alone[key], key


def test_parts_with_many_imports_fall_back_to_the_full_set():
    # 16 entries a row anywhere before it: a part of few large ones reads most
    # of the solution, which the LDS holds only beside small parts
    n, w = 81920, 16
    rng = np.random.default_rng(1)
    i = np.arange(n)[:, None]
    j = np.sort(np.floor(rng.uniform(0.0, 1.0, (n, w)) * i).astype(np.int64), axis=1)
    ok = j < i
    ok[:, 1:] &= j[:, 1:] != j[:, :-1]
    keep = np.concatenate([ok, np.ones((n, 1), bool)], axis=1)
    rp = np.concatenate([[0], np.cumsum(keep.sum(axis=1))]).astype(np.int32)
    col = np.concatenate([j, i], axis=1)[keep].astype(np.int32)
    st = H.tri_plan_stats(H.tri_analyze(CSR(n, rp, col, np.ones(col.size)), "lower", tune=H.tune_default(host_only=1)))
    assert st["dataflow"] == 1 and st["num_groups"] == 256


def test_choosing_the_parts_costs_less_than_half_of_the_rest_of_the_setup():
    A = synth.poisson3d(64)
    best = [1e9, 1e9]
    for _ in range(5):
        for k, tune in enumerate((dict(num_groups=256), dict())):
            t = time.perf_counter()
            plans(A, **tune)
            best[k] = min(best[k], time.perf_counter() - t)
    assert best[1] < 1.5 * best[0], best
