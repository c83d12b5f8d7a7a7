"""GPU: results must not depend on how a launch spreads its work (the branches of the launch rules)."""
import numpy as np
import pytest

import cm_workloads as W

torch = pytest.importorskip("torch")
cm = pytest.importorskip("paper_2607_28435_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [cm.CM_C64, cm.CM_C128])
@pytest.mark.parametrize("batch,nk,stride", [(1, 4096, 1), (1, 5000, 7), (3, 513, 1), (160, 1100, 3), (2, 1, 1)])
def test_readout_rows_per_workgroup(dtype, batch, nk, stride):
    """Small read-outs give a workgroup one or four rows of 256 strikes of a block instead of all
    sixteen; every price equals, bit for bit, the one of a batch of 600 that takes whole blocks."""
    n = 18
    probs = W.heston_batch(4, seed=5, n=n)
    big = cm.SfftPricer([probs[i % 4] for i in range(600)], dtype, tol=1e-8, cap=32)
    u = (2 ** (n - 1) - stride * (nk // 2) + stride * np.arange(nk, dtype=np.int64))
    ref = big.run(torch.from_numpy(np.tile(u, (600, 1))).cuda()).cpu().numpy()
    small = cm.SfftPricer([probs[i % 4] for i in range(batch)], dtype, tol=1e-8, cap=32)
    got = small.run(torch.from_numpy(np.tile(u, (batch, 1))).cuda()).cpu().numpy()
    assert np.isfinite(ref).all()
    np.testing.assert_array_equal(got, ref[:batch])
