"""Host-only checks of the parts the automatic schedule gives the dataflow
kernel (no GPU is touched)."""
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
