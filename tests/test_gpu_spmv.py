"""Products with right-hand sides in groups of four: bit for bit the columns that
single right-hand sides give (the same summation order per column)."""
import numpy as np
import pytest

from synth import CSR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1606_00541_amd as H  # noqa: E402


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("w", [1, 2, 5, 8, 9])
@pytest.mark.parametrize("n", [1, 63, 257, 1000])
def test_groups_of_columns(n, w, dt):
    rng = np.random.default_rng(n + w)
    # rows of one to w + 2 entries: padding, full rows and a CSR tail
    rows = [sorted({i} | set(rng.integers(0, n, size=rng.integers(0, w + 2)).tolist())) for i in range(n)]
    rp = np.cumsum([0] + [len(r) for r in rows]).astype(np.int32)
    A = CSR(n, rp, np.concatenate([np.asarray(r) for r in rows]).astype(np.int32), rng.standard_normal(int(rp[-1])))
    m = H.hec_from_csr(A, dtype=dt, ell_width=w)
    for nrhs in (4, 12, 16):
        x = torch.from_numpy(rng.standard_normal((n, nrhs)))
        x[n - 1, 0], x[n // 2, 1] = float("nan"), float("inf")  # padding must not read them into other rows
        x = x.cuda()
        y = torch.full_like(x, 7.0)
        H.hec_spmv(m, x, y)
        for k in range(nrhs):
            one = torch.full((n, 1), 7.0, dtype=torch.float64, device="cuda")
            H.hec_spmv(m, x[:, k:k + 1].contiguous(), one)
            assert torch.equal(y[:, k].isnan(), one[:, 0].isnan())
            assert torch.equal(y[:, k].nan_to_num(nan=0.0), one[:, 0].nan_to_num(nan=0.0)), (nrhs, k)
