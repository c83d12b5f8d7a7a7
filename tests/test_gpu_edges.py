"""GPU: calls at the edges of what the entry points accept."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
cm = pytest.importorskip("paper_2607_28435_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [4, 12, 16, 32])
def test_sampler_train_of_no_cores(cap):
    """A train of n = 0 in a ragged batch is the scalar 1: squared norm 1, outcome 0 for every shot,
    status as given; its neighbours draw what they draw without it."""
    from test_gpu_observable import _bit_major, _random_trains, _uniforms
    tt, _ = _random_trains([7, 3, 5], min(cap, 6), cm.CM_C128, cap, seed=9)
    R = 300
    U = torch.from_numpy(_bit_major(_uniforms(3, R, 7, seed=2))).cuda()
    got = {}
    for n1 in (3, 0):
        tt.n.copy_(torch.tensor([7, n1, 5], dtype=torch.int32))
        out = torch.full((3, R), -77, dtype=torch.int64, device="cuda")
        norm2 = torch.full((3,), -1.0, dtype=torch.float64, device="cuda")
        st = torch.zeros(3, dtype=torch.int32, device="cuda")
        cm.cm_sample_outcomes(tt, U, R, out, norm2, st, cm.Workspace())
        got[n1] = out.cpu().numpy(), norm2.cpu().numpy(), st.cpu().numpy()
    out, norm2, st = got[0]
    assert np.all(st == cm.CM_OK) and norm2[1] == 1.0
    np.testing.assert_array_equal(out[1], 0)
    for b in (0, 2):
        np.testing.assert_array_equal(out[b], got[3][0][b])
        assert norm2[b] == got[3][1][b]
