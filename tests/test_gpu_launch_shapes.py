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
    sixteen; every price equals, bit for bit, the one of a batch of 300 that takes whole blocks."""
    n = 18
    probs = W.heston_batch(4, seed=5, n=n)
    big = cm.SfftPricer([probs[i % 4] for i in range(300)], dtype, tol=1e-8, cap=32)
    u = (2 ** (n - 1) - stride * (nk // 2) + stride * np.arange(nk, dtype=np.int64))
    ref = big.run(torch.from_numpy(np.tile(u, (300, 1))).cuda()).cpu().numpy()
    small = cm.SfftPricer([probs[i % 4] for i in range(batch)], dtype, tol=1e-8, cap=32)
    got = small.run(torch.from_numpy(np.tile(u, (batch, 1))).cuda()).cpu().numpy()
    assert np.isfinite(ref).all()
    np.testing.assert_array_equal(got, ref[:batch])


def _mlp_case(B, seed):
    from paper_2607_28435_amd.surrogate import MlpNet
    lo, hi = W.surrogate_box()
    net = MlpNet(lo, hi, seed=seed)
    x = torch.from_numpy(W.surrogate_queries(B, seed).astype(np.float32)).cuda()
    t = torch.from_numpy(np.random.default_rng(seed).normal(-2.0, 1.0, B).astype(np.float32)).cuda()
    return net, x, t


def _forward64(net, x):
    """The network in FP64, hidden weights as their BF16 copies."""
    shift = torch.tensor(list(net.struct.shift), dtype=torch.float64, device="cuda")
    scale = torch.tensor(list(net.struct.scale), dtype=torch.float64, device="cuda")
    a, o = (x.double() - shift) * scale, 0
    for out, inp in ((256, 7), (256, 256), (256, 256), (256, 256), (1, 256)):
        w = net.params[o:o + out * inp].reshape(out, inp)
        a = a @ (w.bfloat16() if out == inp else w).double().T + net.params[o + out * inp:o + out * inp + out].double()
        o += out * inp + out
        a = a * torch.sigmoid(a) if out > 1 else a
    return a[:, 0]


@pytest.mark.parametrize("B", [1, 31, 32, 33, 127, 129, 4096, 4097, 8200])
def test_training_tiles_and_spans(B):
    """Rows at the edges of the 32-row tiles and of the row spans of the weight gradients: with dy
    zero but for one row, the batch's gradient is that row's own, bit for bit (every other term is
    an exact zero and each row's arithmetic does not depend on its place)."""
    net, x, _ = _mlp_case(B, 11)
    ref = None
    for row in sorted({0, B // 2, B - 1}):
        xb = x.clone()
        xb[row] = x[0]
        dy = torch.zeros(B, dtype=torch.float32, device="cuda")
        dy[row] = 0.75
        nb = cm.cm_mlp_act_bytes(B)
        acts = torch.empty(nb, dtype=torch.uint8, device="cuda")
        ws = torch.empty(nb // 2, dtype=torch.uint8, device="cuda")
        y = torch.empty(B, dtype=torch.float32, device="cuda")
        grad = torch.full((cm.CM_MLP_NPARAMS,), 7.0, dtype=torch.float32, device="cuda")
        cm.cm_mlp_forward(net.struct, xb, B, y, acts, nb)
        cm.cm_mlp_backward(net.struct, xb, acts, dy, B, grad, ws, nb // 2)
        if ref is None:
            ref = torch.full((cm.CM_MLP_NPARAMS,), 7.0, dtype=torch.float32, device="cuda")
            one = torch.full((1,), 0.75, dtype=torch.float32, device="cuda")
            cm.cm_mlp_forward(net.struct, x[:1].contiguous(), 1, y, acts, cm.cm_mlp_act_bytes(1))
            cm.cm_mlp_backward(net.struct, x[:1].contiguous(), acts, one, 1, ref, ws, cm.cm_mlp_act_bytes(1) // 2)
            assert bool(torch.isfinite(ref).all()) and float(ref.abs().max()) > 0
        assert torch.equal(grad, ref), (B, row)


@pytest.mark.parametrize("B", [1, 32, 33, 24576, 24577, 24640])
def test_inference_tile_sizes(B):
    """Both sides of the rule between tiles of 32 rows and tiles of 64, against FP64: the hidden
    operands keep 2^-16, three layers deep."""
    net, x, _ = _mlp_case(B, 12)
    y = _forward64(net, x)
    got = net.forward(x).double()
    assert float((got - y).abs().max()) <= 1e-4 * float(y.abs().max())


@pytest.mark.parametrize("dtype", [cm.CM_C64, cm.CM_C128])
@pytest.mark.parametrize("quad", ["simpson1", "rect2"])
@pytest.mark.parametrize("n", [1, 2, 3, 6, 11, 14, 15, 16, 19, 20, 21, 24])
def test_dense_chosen_strikes_and_groups(dtype, quad, n):
    """Chosen strikes are priced from the stored transform and every strike in the last pass: the
    same transform, so they agree to the rounding of the scale 2^z (two units in the last place
    each), at both ends of the grid and about the middle, over the pass plans (one pass up to
    n = 15 or 14, two, and the reverse order of the chosen strikes in a second instance). The plan
    does not depend on the batch: instances of a group agree bit for bit."""
    p = W.bs_simpson_n12().replace(n=n, quad=quad, eta=0.25 if n < 16 else 0.05, alpha=1.5)
    M = 2 ** n
    u = np.unique(np.clip(np.concatenate([np.arange(5), M // 2 + np.arange(-5, 5), M - 1 - np.arange(5)]), 0, M - 1))
    every, st = cm.dense_prices([p, p], dtype)
    chosen, st2 = cm.dense_prices([p, p], dtype, torch.from_numpy(np.stack([u, u[::-1].copy()])).cuda())
    assert int(st.abs().sum()) == 0 and int(st2.abs().sum()) == 0
    assert torch.equal(torch.nan_to_num(every[0]), torch.nan_to_num(every[1]))
    chosen = chosen.cpu().numpy()
    every = every[0].cpu().numpy()
    np.testing.assert_array_equal(chosen[1], chosen[0][::-1])
    np.testing.assert_allclose(chosen[0], every[u], rtol=4 * np.finfo(every.dtype).eps, atol=np.finfo(every.dtype).tiny)


@pytest.mark.parametrize("n", [1, 2, 5, 14, 20])
def test_wide_and_one_wave_sweeps(n):
    """Complex128 batches of 512 take the rounding sweeps on four waves per train, of 513 on one: the
    same trains to the order of the FP64 sums. At tolerance 1e-10 each side's prices in the window
    0.5 <= K/S0 <= 1.5 are within a few times 1e-10 S0 of the grid's own (the undamping there
    is below 3^1.5), so the two lie within 1e-9 S0 of each other."""
    probs = W.vg_batch(6, n=n) if n > 5 else W.bs_batch(6, n=n)
    got, codes = [], []
    for batch in (512, 513):
        pr = cm.SfftPricer([probs[i % 6] for i in range(batch)], cm.CM_C128, tol=1e-10, cap=32)
        u = [W.window_strided(p, 32) for p in probs]
        k = min(len(v) for v in u)
        s = np.stack([u[i % 6][:k] for i in range(batch)])
        got.append(pr.run(torch.from_numpy(s).cuda()).cpu().numpy())
        codes.append(np.stack([v[:512] for v in pr.statuses().values()]))
        assert np.array_equal(got[-1][:6], got[-1][6:12], equal_nan=True)
    np.testing.assert_array_equal(codes[0], codes[1])   # a five-point grid has instances the build refuses
    ok = ~codes[0].any(axis=0)
    assert ok.any() and np.abs(got[0] - got[1][:512])[ok].max() <= 1e-9 * probs[0].S0


@pytest.mark.parametrize("model,n,cap", [("heston", 16, 32), ("heston", 24, 32), ("heston", 13, 16), ("heston", 20, 64),
                                         ("bs", 1, 32), ("bs", 2, 32), ("bs", 3, 16), ("vg", 18, 24)])
def test_zip_left_part(model, n, cap):
    """Batches of 1024 run the left sites of the zip-up on one wave per instance, smaller ones on
    four: the same arithmetic per column, so complex64 trains agree bit for bit, their ranks and
    statuses too (a capacity of 16 also makes the wave hand over early)."""
    probs = {"heston": lambda: W.heston_batch(8, seed=3, n=n), "bs": lambda: W.bs_batch(8, n=n),
             "vg": lambda: W.vg_batch(8, n=n)}[model]()
    u = np.stack([W.near_money(p, 64) for p in probs])
    out = []
    for batch in (8, 1024):
        pr = cm.SfftPricer([probs[i % 8] for i in range(batch)], cm.CM_C64, tol=1e-8, cap=cap)
        pr.build()
        pr.apply()
        ranks = pr.y.ranks[:, :n + 1].clone()
        prices = pr.run(torch.from_numpy(np.tile(u, (batch // 8, 1))).cuda())
        out.append((ranks, prices, pr.statuses()["apply"]))
    (r0, p0, s0), (r1, p1, s1) = out
    assert torch.equal(r0.repeat(128, 1), r1) and bool((r1[:, n] == 1).all())
    assert torch.equal(torch.nan_to_num(p0.repeat(128, 1)), torch.nan_to_num(p1))
    assert np.array_equal(np.tile(s0, 128), s1)


# ------------------------------------------------------------------ sampler: padding and sizes

@pytest.mark.parametrize("rmax,cap", [(1, 1), (2, 8), (3, 5), (6, 8), (7, 7), (9, 9), (10, 12), (11, 32), (13, 16),
                                      (14, 32), (15, 15), (17, 20), (18, 32)])
def test_sampler_bond_paddings(rmax, cap):
    """Bonds on both sides of every padding and of every size the sampler has code of its own
    for, in trains whose ends run through the smaller bonds: the outcomes are the oracle's for
    the same uniforms. A decision may differ only where the oracle's own margin is below 1e-10:
    the masses carry some n r^2 = 12 * 18^2 roundings of 1.1e-16, 4.4e-13."""
    from test_gpu_observable import _check_samples, _probs_of_output_train, _random_trains, _sample, _uniforms
    ns = [11, 12, 2, 7]
    tt, host = _random_trains(ns, rmax, cm.CM_C128, cap, seed=500 + rmax)
    R = 1100
    U = _uniforms(len(ns), R, max(ns), seed=rmax)
    got, norm2, st = _sample(tt, U)
    assert np.all(st == cm.CM_OK), st
    for b, n in enumerate(ns):
        prob, nrm = _probs_of_output_train(host[b])
        assert abs(norm2[b] - nrm) <= 1e-11 * nrm
        _check_samples(prob, U[b, :, :n], got[b], margin_tol=1e-10, max_frac=0.0)
