"""Both triangles of an ILU application in one launch, and right-hand sides
beyond max_nrhs taken in groups of columns, bit for bit against one launch per
level."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1606_00541_amd as H  # noqa: E402


@pytest.mark.parametrize("nrhs,most", [(1, 1), (3, 4), (7, 4), (16, 1)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (13, 1, 1), (31, 17, 1), (23, 19, 7)])
def test_ilu_application(shape, dt, nrhs, most):
    A = synth.poisson3d(*shape)
    r = torch.from_numpy(np.random.default_rng(9).standard_normal((A.n, nrhs))).cuda()
    # an explicit part count takes no more than max_nrhs where steps fill a wavefront
    for groups in (0, 1, 3) if nrhs <= most else (0,):
        out = []
        for t in (dict(schedule="level_launch"), dict(max_nrhs=most, num_groups=groups)):
            f = H.ilu_setup(A, "iluk", k=1, factor_dtype=dt, tune=H.tune_default(**t))
            z = torch.full_like(r, float("nan"))
            for _ in range(3):  # both mailbox halves
                H.ilu_apply(f, r, z)
            torch.cuda.synchronize()
            out.append(z)
        assert torch.equal(out[0], out[1]), groups
