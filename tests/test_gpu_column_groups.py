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
