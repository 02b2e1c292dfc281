"""Batched BiCGSTAB where the vectors' lengths lie around the elements that a
wavefront of the vector combinations takes, with systems finished from the
start among the others."""
import numpy as np
import pytest

import oracle
import synth
from synth import CSR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1606_00541_amd as H  # noqa: E402


@pytest.mark.parametrize("nrhs", [1, 3, 4])
@pytest.mark.parametrize("sides", [[(1, 1)], [(7, 9), (1, 1)], [(8, 8), (16, 12)], [(16, 16), (1, 1), (17, 15)],
                                   [(32, 32), (5, 5), (31, 33), (1, 2)]])
def test_lengths_and_finished_systems(sides, nrhs):
    import scipy.sparse as sp

    mats = [synth.poisson2d(a, b) for a, b in sides]
    m = sp.block_diag([q.to_scipy() for q in mats]).tocsr()
    m.sort_indices()
    A = CSR(m.shape[0], m.indptr.astype(np.int32), m.indices.astype(np.int32), m.data.copy())
    ptr = np.cumsum([0] + [q.n for q in mats]).astype(np.int32)
    f = H.batch_setup(A, ptr, "ilu0", tune=H.tune_default(max_nrhs=nrhs))
    M = H.hec_from_csr(A)
    for idle in range(-1, len(mats)):
        b = synth.rhs(A.n, nrhs, 5 + idle)
        x0 = np.zeros_like(b)
        if idle >= 0:
            b[ptr[idle]:ptr[idle + 1]] = 0.0  # its solution is zero, whatever the others do
        x = torch.from_numpy(x0).cuda()
        st, info = H.krylov_solve_batch(M, f, ptr, torch.from_numpy(b).cuda(), x, method="bicgstab", rtol=1e-10)
        assert st == 0
        x = x.cpu().numpy()
        for s, q in enumerate(mats):
            seg = slice(int(ptr[s]), int(ptr[s + 1]))
            for k in range(nrhs):
                if s == idle:
                    assert np.all(x[seg, k] == 0.0)
                    continue
                r = b[seg, k] - oracle.spmv(q, x[seg, k])
                assert np.linalg.norm(r) <= 1e-9 * np.linalg.norm(b[seg, k])
