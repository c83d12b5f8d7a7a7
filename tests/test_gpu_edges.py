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


# ------------------------------------------------------------------ zip-up: large batches

LARGE = 1792   # the smallest batch whose left sites run one wave per instance (from n = 14 on)


def _zip_case(model, n, dtype, batch, seed=3, cap=32, tol=1e-8):
    import cm_workloads as W
    make = {"heston": lambda: W.heston_batch(8, seed=seed, n=n), "bs": lambda: W.bs_batch(8, n=n),
            "vg": lambda: W.vg_batch(8, n=n)}[model]
    probs = make()
    pr = cm.SfftPricer([probs[i % 8] for i in range(batch)], dtype, tol=tol, cap=cap)
    pr.build()
    return pr


def _first8(pr):
    """A pricer of the first eight instances with pr's own input trains."""
    few = cm.SfftPricer([pr.problems[i] for i in range(8)], pr.dtype, tol=pr.tol, cap=pr.cap, mpo=pr.mpo)
    few.x.cores.copy_(pr.x.cores[:len(few.x.cores)])
    few.x.ranks.copy_(pr.x.ranks[:8])
    few.x.struct.flags = pr.x.struct.flags
    return few


def _table(like, core_off, cores):
    """A TTBatch of like's trains with a table of offsets and cores of its own."""
    t = cm.TTBatch(like.ns, 2, 1, like.cap_rank, like.dtype)
    t.core_off, t.cores = core_off, cores
    s = t._s
    t._s = cm.CmTTBatch(s.batch, 2, 1, s.cap_rank, s.n_max, s.dtype, 0, 0, t.n.data_ptr(), t.ranks.data_ptr(),
                        core_off.data_ptr(), cores.data_ptr())
    return t


@pytest.mark.parametrize("dtype", [cm.CM_C64, cm.CM_C128])
@pytest.mark.parametrize("n", [3, 14, 24])
def test_zip_keeps_to_tight_tables(dtype, n):
    """Output cores packed to the ranks they end with, thirty elements between neighbours: the apply
    writes the cores that a small batch writes into the capacity layout (the same kernel takes both),
    and nothing else."""
    pr = _zip_case("heston", n, dtype, LARGE)
    few = _first8(pr)
    few.apply()
    ranks = few.y.ranks.long()
    gap, reps = 30, LARGE // 8
    size = (ranks[:, :n] * 2 * ranks[:, 1:n + 1] + gap).repeat(reps, 1)
    start = (torch.cumsum(size.reshape(-1), 0) - size.reshape(-1) + gap).reshape(LARGE, n)
    off = torch.zeros((LARGE, cm.CM_MAX_N), dtype=torch.int64, device="cuda")
    off[:, :n] = start
    cores = torch.full((int(size.sum()) + 4096,), 1234.5, dtype=few.y.cores.dtype, device="cuda")
    pr.y = _table(pr.y, off, cores)
    pr.apply()
    assert int(pr.st_apply.abs().sum()) == 0
    assert torch.equal(pr.y.ranks[:, :n + 1], few.y.ranks[:, :n + 1].repeat(reps, 1))
    count = (size - gap).reshape(-1)
    within = torch.arange(int(count.sum()), device="cuda") - torch.repeat_interleave(torch.cumsum(count, 0) - count, count)
    at = torch.repeat_interleave(start.reshape(-1), count) + within
    ref = few.y.cores[torch.repeat_interleave(few.y.core_off[:, :n].repeat(reps, 1).reshape(-1), count) + within]
    assert torch.equal(torch.view_as_real(cores[at]), torch.view_as_real(ref))
    rest = torch.ones(len(cores), dtype=torch.bool, device="cuda")
    rest[at] = False
    assert bool((cores[rest] == 1234.5).all())


@pytest.mark.parametrize("dtype", [cm.CM_C64, cm.CM_C128])
@pytest.mark.parametrize("n", [14, 24])
def test_zip_into_its_input(dtype, n):
    """The output cores may be the input's buffer under the same offsets, in any batch: the cores are
    those of a small batch, bit for bit (the same kernel takes both)."""
    pr = _zip_case("heston", n, dtype, LARGE)
    ref = _first8(pr)
    ref.apply()
    pr.y = _table(pr.y, pr.x.core_off, pr.x.cores)
    pr.apply()
    assert int(pr.st_apply.abs().sum()) == 0
    assert torch.equal(pr.y.ranks[:, :n + 1], ref.y.ranks[:, :n + 1].repeat(LARGE // 8, 1))
    rk = ref.y.ranks.cpu().numpy()
    for b in (0, 3, 7, LARGE - 2):
        for l in range(n):
            k = int(rk[b % 8, l] * 2 * rk[b % 8, l + 1])
            o, p = int(pr.y.core_off[b, l]), int(ref.y.core_off[b % 8, l])
            assert torch.equal(torch.view_as_real(pr.y.cores[o:o + k]), torch.view_as_real(ref.y.cores[p:p + k])), (b, l)


@pytest.mark.parametrize("model,n", [("heston", 14), ("heston", 24), ("vg", 18), ("bs", 20)])
def test_zip_left_part_fp64(model, n):
    """Complex128 trains of a large batch, whose left sites run one wave per instance, against a small
    batch's: the same ranks, and at tolerance 1e-10 prices in the window 0.5 <= K/S0 <= 1.5 that lie
    within a few times 1e-10 S0 of the grid's own on either side, so within 1e-9 S0 of each other."""
    import cm_workloads as W
    many = _zip_case(model, n, cm.CM_C128, LARGE, tol=1e-10)
    few = _first8(many)
    few.apply()
    many.apply()
    assert int(many.st_apply.abs().sum()) == 0
    assert torch.equal(many.y.ranks[:, :n + 1], few.y.ranks[:, :n + 1].repeat(LARGE // 8, 1))
    u = [W.window_strided(p, 64) for p in few.problems]
    nk = min(len(v) for v in u)
    s = torch.from_numpy(np.stack([v[:nk] for v in u])).cuda()
    a = few.run(s).cpu().numpy()
    b = many.run(s.repeat(LARGE // 8, 1)).cpu().numpy()
    assert np.array_equal(b[:8], b[-8:])
    assert np.abs(a - b[:8]).max() <= 1e-9 * few.problems[0].S0


@pytest.mark.parametrize("n", [13, 14])
@pytest.mark.parametrize("batch", [LARGE - 1, LARGE])
def test_zip_left_rule(batch, n):
    """Either side of the rule for the left part, complex64: the ranks, statuses and prices of a small
    batch with the same inputs (the cores may differ by the last bit of FP64 sums before they are
    rounded; prices by 1e-6 S0 at most, the accuracy of a complex64 chain at tolerance 1e-8)."""
    import cm_workloads as W
    many = _zip_case("heston", n, cm.CM_C64, batch)
    few = _first8(many)
    few.apply()
    many.apply()
    k = torch.arange(batch, device="cuda") % 8
    assert int(many.st_apply.abs().sum()) == 0
    assert torch.equal(many.y.ranks[:, :n + 1], few.y.ranks[k, :n + 1])
    s = torch.from_numpy(np.stack([W.near_money(p, 64) for p in few.problems])).cuda()
    a, b = few.run(s), many.run(s[k])
    assert float((a[k] - b).abs().max()) <= 1e-6 * few.problems[0].S0


# ------------------------------------------------------------------ surrogate

@pytest.mark.parametrize("B", [1, 33, 300])
def test_training_keeps_the_accurate_silu(B):
    """Fourth-layer neurons far on the flat side (z near -80), one of them read by the output: the
    prediction is W5 silu(z) alone, and the gradients of W5 and b4 sums of silu(z) and silu'(z). From
    the pre-activations the call has kept, FP64 gives them; the call's roundings are the exponential's
    (2 units of 2^-24 relative), the sum's, the quotient's and the products' (one each), 8 in all, and
    one per term for the sum over the batch. An exponential whose argument is rounded would be off by
    up to 80 of them."""
    from test_gpu_launch_shapes import _mlp_case
    net, x, _ = _mlp_case(B, 21)
    p = net.params
    p[199168:199424] = -80.0
    p[199424:199680] = 0.0
    p[199424 + 5] = 1.0
    p[199680] = 0.0
    cm.cm_mlp_sync_bf16(net.struct)
    nb = cm.cm_mlp_act_bytes(B)
    acts = torch.empty(nb // 4, dtype=torch.float32, device="cuda")
    ws = torch.empty(nb // 2, dtype=torch.uint8, device="cuda")
    y = torch.empty(B, dtype=torch.float32, device="cuda")
    grad = torch.empty(cm.CM_MLP_NPARAMS, dtype=torch.float32, device="cuda")
    dy = torch.ones(B, dtype=torch.float32, device="cuda")
    cm.cm_mlp_forward(net.struct, x, B, y, acts, nb)
    cm.cm_mlp_backward(net.struct, x, acts, dy, B, grad, ws, nb // 2)
    z = acts[3 * B * 256:].reshape(B, 256).double()
    assert float(z.max()) < -60.0 and float(z.min()) > -87.0
    s = torch.sigmoid(z)
    silu, slope = z * s, s * (1.0 + z * (1.0 - s))
    eps = 2.0 ** -24
    rel = lambda a, b: float(((a.double() - b) / b).abs().max()) / eps
    assert rel(y, silu[:, 5]) <= 8
    assert rel(grad[199424:199680], silu.sum(0)) <= 8 + B
    assert rel(grad[199168 + 5:199168 + 6], slope[:, 5].sum(0, keepdim=True)) <= 8 + B


@pytest.mark.parametrize("B", [1, 31, 32, 33, 777, 8200, 24576])
def test_queries_do_not_depend_on_their_batch(B):
    """A query's output is the same bits in a small batch (tiles of 32 rows) and in a large one (two
    tiles of 64 in flight), at the large batch's start and at its ragged end."""
    from test_gpu_launch_shapes import _mlp_case
    net, x, _ = _mlp_case(24577 + 70, 13)
    every = net.forward(x)
    assert torch.equal(net.forward(x[:B].contiguous()), every[:B])
    assert torch.equal(net.forward(x[-B:].contiguous()), every[-B:])


@pytest.mark.parametrize("B", [24577, 32832, 49153])
def test_large_batches_against_the_training_forward(B):
    """Sizes that end in a ragged tile of 64, or leave its two halves unequal numbers of tiles: the
    inference kernel's outputs against the training forward's, whose sums run in another order. The
    hidden operands keep 2^-16, three layers deep; 1e-4 of the largest output covers both."""
    from test_gpu_launch_shapes import _mlp_case
    net, x, _ = _mlp_case(B, 14)
    nb = cm.cm_mlp_act_bytes(B)
    acts = torch.empty(nb, dtype=torch.uint8, device="cuda")
    y = torch.empty(B, dtype=torch.float32, device="cuda")
    cm.cm_mlp_forward(net.struct, x, B, y, acts, nb)
    z = net.forward(x)
    assert not torch.equal(y, z)
    assert float((y - z).abs().max()) <= 1e-4 * float(z.abs().max())


# ------------------------------------------------------------------ rounding sweeps on four waves

@pytest.mark.parametrize("n", [19, 20, 23])
@pytest.mark.parametrize("tol", [2e-8, 1e-8, 1e-10])
def test_sweeps_either_side_of_the_four_wave_rule(n, tol):
    """Complex128 batches of 256 from n = 20 on and tolerance 1e-8 down take the sweeps on four waves
    per train, of 257, shorter or looser ones on one: the same trains to the order of the FP64 sums.
    In the window 0.5 <= K/S0 <= 1.5 each side's prices are within a few times the tolerance of the
    grid's own (the undamping there is below 3^1.5), so the two lie within ten times it."""
    import cm_workloads as W
    probs = W.vg_batch(4, n=n) + W.heston_batch(4, seed=5, n=n)
    u = [W.window_strided(p, 48) for p in probs]
    k = min(len(v) for v in u)
    got = []
    for batch in (256, 257):
        pr = cm.SfftPricer([probs[i % 8] for i in range(batch)], cm.CM_C128, tol=tol, cap=32)
        s = torch.from_numpy(np.stack([u[i % 8][:k] for i in range(batch)])).cuda()
        got.append(pr.run(s).cpu().numpy())
        assert not any(v.any() for v in pr.statuses().values())
        assert np.array_equal(got[-1][:8], got[-1][8:16])
    assert np.abs(got[0] - got[1][:256]).max() <= 10 * tol * probs[0].S0


# ------------------------------------------------------------------ dense path

@pytest.mark.parametrize("dtype,n", [(cm.CM_C64, 15), (cm.CM_C128, 14)])
@pytest.mark.parametrize("model", ["heston", "vg"])
def test_dense_largest_single_pass_either_side(dtype, n, model):
    """The largest grid of one pass takes two while there are fewer than 256 grids. Near the money
    (0.5 <= K/S0 <= 1.5, undamping below 3^1.5) the two differ by the rounding of two transforms: at most
    4 units in the last place per level of each, of sums no larger than a few times the largest price."""
    import cm_workloads as W
    probs = W.heston_batch(3, seed=2, n=n) if model == "heston" else W.vg_batch(3, n=n)
    u = [W.window_strided(p, 200) for p in probs]
    k = min(len(v) for v in u)
    got = []
    for batch in (255, 256):
        s = torch.from_numpy(np.stack([u[i % 3][:k] for i in range(batch)])).cuda()
        p, st = cm.dense_prices([probs[i % 3] for i in range(batch)], dtype, s)
        assert int(st.abs().sum()) == 0
        got.append(p.double())
        assert torch.equal(p[:3], p[3:6])
    eps = 2.0 ** (-24 if dtype == cm.CM_C64 else -53)
    assert float((got[0][:3] - got[1][:3]).abs().max()) <= 8 * n * 3 ** 1.5 * 3 * eps * float(got[0].abs().max())


@pytest.mark.parametrize("dtype", [cm.CM_C64, cm.CM_C128])
@pytest.mark.parametrize("n,few,many", [(9, 512, 513), (10, 512, 513), (11, 512, 513), (10, 1, 513), (9, 2999, 3000)])
def test_dense_small_grids_either_side(dtype, n, few, many):
    """Up to 512 grids of n = 9 to 11 have a thread per value of the integrand, from 3000 problems on one
    wave finds a support: the same values and transforms, to
    the rounding that the test above allows (the compiler may fuse the products differently)."""
    import cm_workloads as W
    probs = [W.heston_batch(1, seed=2, n=n)[0], W.vg_batch(1, n=n)[0], W.bs_batch(1, n=n)[0]]
    every = [cm.dense_prices([probs[i % 3] for i in range(max(b, 3))], dtype) for b in (few, many)]
    a, b = every[0][0][:3].double(), every[1][0][:3].double()
    assert int(every[0][1].abs().sum()) == 0 and int(every[1][1].abs().sum()) == 0
    for i, p in enumerate(probs):
        u = torch.from_numpy(W.window_strided(p, 100)).cuda()
        eps = 2.0 ** (-24 if dtype == cm.CM_C64 else -53)
        assert float((a[i][u] - b[i][u]).abs().max()) <= 8 * n * 3 ** 1.5 * 3 * eps * float(a[i][u].abs().max())
