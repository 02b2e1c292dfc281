"""The dataflow kernel's packed rows and step rotation at the edges of its
ranges, bit for bit against one launch per level (the same summation order)."""
import numpy as np
import pytest

import synth
from synth import CSR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1606_00541_amd as H  # noqa: E402


def banded(n, w, seed):
    """Lower triangle: up to w off-diagonals a row, half of them next to the
    diagonal (long chains), the others anywhere before it."""
    rng = np.random.default_rng(seed)
    rows = []
    for i in range(n):
        near = [i - 1 - k for k in range((w + 1) // 2) if i - 1 - k >= 0]
        far = rng.integers(0, i, size=w // 2).tolist() if i else []
        rows.append(sorted(set(near + far)) + [i])
    rp = np.cumsum([0] + [len(r) for r in rows]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    v = rng.uniform(-1.0, 1.0, ci.size) / w
    v[rp[1:] - 1] = rng.uniform(1.0, 2.0, n)
    return CSR(n, rp, ci, v)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("nrhs", [1, 3])
@pytest.mark.parametrize("w", [1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16])
def test_every_width_and_short_pieces(w, nrhs, dt):
    # 1 row to a few hundred: wavefronts with no step, fewer steps than the
    # rotation holds, and several rotations with a remainder
    npdt = np.float64 if dt == "f64" else np.float32
    for n, groups in ((1, 1), (5, 3), (67, 2), (401, 1), (401, 5)):
        L = banded(n, w, 10 * w + n)
        b = synth.rhs(n, nrhs, n).astype(npdt)
        out = []
        for t in (H.tune_default(schedule="level_launch"),
                  H.tune_default(schedule="owner_persistent", kernel_variant=4, num_groups=groups, max_nrhs=nrhs)):
            p = H.tri_analyze(L, "lower", dtype=dt, tune=t)
            bt = torch.from_numpy(b).cuda()
            xt = torch.empty_like(bt)
            for _ in range(3):  # both mailbox halves
                H.tri_solve_lower(p, bt, xt)
            torch.cuda.synchronize()
            H.tri_plan_check(p)
            out.append(xt.cpu().numpy())
        assert H.tri_plan_stats(p)["dataflow"] == 1
        assert np.array_equal(out[0], out[1]), (n, groups)
