"""The training products at the sizes where their kernels change or have
edges: batches whose contractions end in a short k-step, 64- and 128-wide
tiles, split and unsplit K, and a save buffer that is not 16-byte aligned (the
general kernels).

The reference is the backward pass in float64 on the GPU's own saved
activations and loss gradient (so no ReLU sits on another side), with the
BF16 form's roundings where that form rounds.  Bars: FP32 a normwise relative
error of max(5e-5, 4 u sqrt(52 B)) per tensor (u = 6e-8, the square root of
the longest sum, a depth margin); BF16 2^-8 (a value whose FP32 sum falls on
the other side of a rounding boundary moves by one unit)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

D, L = 50, 111


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def sn():
    import paper_2105_05821_amd as m
    m.lib()
    return m


def reference(torch, ws, x, acts, dz, prec):
    """Parameter and window gradients in float64; acts = a1, a2, a3, h."""
    def rnd(t):
        return t.float().to(torch.bfloat16).double() if prec == 1 else t

    B = x.shape[0]
    W = [rnd(torch.from_numpy(np.ascontiguousarray(w)).cuda().double()) for w in ws]
    a1, a2, a3, h = acts
    dzr = rnd(dz)
    g = [None] * 5
    g[4] = (dzr.t() @ h, dz.sum(0))
    dh = rnd((dzr @ W[4]) * (h > 0))
    g[3] = (dh.t() @ a3.transpose(1, 2).reshape(B, -1), dh.sum(0))
    dy = rnd((dh @ W[3]).view(B, 256, 13).transpose(1, 2) * (a3 > 0)).reshape(B * 13, 256)
    xin = rnd(x[:, :104].double()).reshape(B * 52, 100)
    for l, (rows, n) in {2: (a2, 256), 1: (a1, 128), 0: (xin, 100)}.items():
        rows = rows.reshape(-1, n)
        w = W[l].permute(0, 2, 1).reshape(W[l].shape[0], n)  # columns t * c_in + c
        gw = dy.t() @ rows
        g[l] = (gw.view(-1, 2, n // 2).permute(0, 2, 1).reshape(gw.shape), dy.sum(0))
        dy = dy @ w
        if l:
            dy = rnd(dy * (rows > 0)).reshape(-1, n // 2)
    dx = torch.zeros((B, L, D), dtype=torch.float64, device="cuda")
    dx[:, :104] = dy.view(B, 104, 50)
    return g, dx


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("B,shift", [(1, 0), (5, 0), (33, 0), (64, 0), (257, 0), (1030, 0),
                                     (37, 8)])
def test_training_products(torch, sn, prec, B, shift):
    products(torch, sn, prec, B, shift)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("B,x_off,dz_off,dp_off", [
    (45, 1, 0, 0), (45, 0, 1, 0), (45, 0, 0, 1), (45, 1, 1, 3), (2, 0, 0, 0), (556, 0, 0, 0),
    (600, 0, 0, 0), (2050, 0, 0, 2)])
def test_weight_gradients_together(torch, sn, prec, B, x_off, dz_off, dp_off):
    """Weight gradients in one launch: either side of the batch where their
    tiles change, many k-splits, and windows, loss gradients or parameter
    gradients that start off a 16- or 8-byte boundary (offsets in floats: a
    product on its own, a copy and sums on their own, single stores)."""
    products(torch, sn, prec, B, 0, x_off, dz_off, dp_off)


def moved_by(torch, t, off):
    out = torch.empty(t.numel() + off, dtype=t.dtype, device=t.device)[off:].view(t.shape)
    return out.copy_(t)


def products(torch, sn, prec, B, shift, x_off=0, dz_off=0, dp_off=0):
    layers = synth.net_c3_hybrid()
    ws, bs = synth.init_weights(3, layers, out_bias=None, out_gain=1.0)
    pred = sn.Predictor(layers, prec)
    pred.load_weights(layers, sn.flat_params(ws, bs))
    gen = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn((B, L, D), generator=gen, device="cuda")
    y = torch.randint(0, 420, (B, 2), generator=gen, device="cuda").int()
    z, save = pred.forward(x)
    _, dz = pred.loss(z, y)
    x, dz = moved_by(torch, x, x_off), moved_by(torch, dz, dz_off)
    n = pred.save_bytes(B)
    moved = torch.empty(n + shift, dtype=torch.uint8, device="cuda")[shift:]
    moved.copy_(save[:n])
    dp = torch.empty(2_204_642 + dp_off, device="cuda")[dp_off:]
    dx = pred.backward(x, moved, dz, dp, want_dx=True)
    v = save[:n].view(torch.float32 if prec == 0 else torch.bfloat16).double()
    sizes = (52 * 64, 26 * 128, 13 * 256, 512)
    at = np.cumsum([0] + [B * s for s in sizes])
    a1, a2, a3, h = (v[at[i]:at[i + 1]].view(B, s) for i, s in enumerate(sizes))
    want, want_dx = reference(torch, ws, x, (a1, a2, a3.reshape(B, 13, 256), h), dz.double(), prec)
    bar = max(5e-5, 4 * 6e-8 * np.sqrt(52.0 * B)) if prec == 0 else 2.0 ** -8

    def check(name, got, ref):
        err = float((got.double() - ref).norm() / ref.norm().clamp_min(1e-300))
        assert err <= bar, (name, err)

    off = 0
    for l, (gw, gb) in enumerate(want):
        check(f"layer {l} weights", dp[off:off + gw.numel()].view(gw.shape), gw)
        off += gw.numel()
        check(f"layer {l} biases", dp[off:off + gb.numel()], gb)
        off += gb.numel()
    check("dx", dx, want_dx)
    # accumulated onto what is there
    dp2 = torch.ones_like(dp)
    pred.backward(x, moved, dz, dp2, accumulate=True)
    assert torch.allclose(dp2 - 1, dp, rtol=0, atol=3e-7 * max(1.0, float(dp.abs().max())))
    pred.close()


@pytest.mark.parametrize("B", [1024, 4096])
def test_fp32_weight_gradient_sums_in_short_runs(torch, sn, B):
    """The head's weight gradient dZ^T H against float64 on the same dZ and H:
    its error is that of sums over runs of 128 products, however many windows a
    workgroup takes.  Bar: an operation rounds by at most u / sqrt(3) rms
    (u = 2^-24), the n partial sums of a chain grow as sqrt(n), so a chain errs
    by sqrt(n / 2) of that: runs of 128, the B / 128 runs (in one or more
    splits), and the product's own rounding."""
    layers = synth.net_c3_hybrid()
    ws, bs = synth.init_weights(3, layers, out_bias=None, out_gain=1.0)
    pred = sn.Predictor(layers, sn.SIM_FP32)
    pred.load_weights(layers, sn.flat_params(ws, bs))
    gen = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn((B, L, D), generator=gen, device="cuda")
    z, save = pred.forward(x)
    dz = torch.randn(z.shape, generator=gen, device="cuda")
    dp = torch.empty(2_204_642, device="cuda")
    pred.backward(x, save, dz, dp)
    h = save[:pred.save_bytes(B)].view(torch.float32)[-B * 512:].view(B, 512).double()
    want = dz.double().t() @ h
    got = dp[-802 - 802 * 512:-802].view(802, 512).double()
    # (against the size of the summed products: H is not negative, dZ of both signs)
    size = torch.sqrt(dz.double().square().t() @ h.square())
    err = float((got - want).norm() / size.norm())
    bar = 2.0 ** -24 / np.sqrt(3.0) * np.sqrt(128 / 2 + B / 128 / 2 + 1)
    assert err <= bar, (err, bar)
    pred.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shift", [4, 8])
def test_save_buffer_off_its_boundary(torch, sn, prec, shift):
    """A save buffer 4 or 8 bytes off a 16-byte boundary: copied in eager
    calls (first use, a larger batch, a smaller one again), read where it is by
    the general kernels in a call captured before any copy exists."""
    layers = synth.net_c3_hybrid()
    ws, bs = synth.init_weights(3, layers, out_bias=None, out_gain=1.0)
    side = torch.cuda.Stream()
    bar = 5e-6 if prec == 0 else 2.0 ** -8
    with torch.cuda.stream(side):
        pred = sn.Predictor(layers, prec)
        pred.load_weights(layers, sn.flat_params(ws, bs))
        gen = torch.Generator(device="cuda").manual_seed(9)

        def inputs(B):
            x = torch.randn((B, L, D), generator=gen, device="cuda")
            y = torch.randint(0, 420, (B, 2), generator=gen, device="cuda").int()
            z, save = pred.forward(x)
            n = pred.save_bytes(B)
            off = torch.empty(n + shift, dtype=torch.uint8, device="cuda")[shift:]
            off.copy_(save[:n])
            dz = pred.loss(z, y)[1]
            want = torch.empty(2_204_642, device="cuda")
            return x, off, dz, want, pred.backward(x, save, dz, want, want_dx=True)

        def check(got, dx, want, want_dx):
            side.synchronize()
            for a, b in ((got, want), (dx, want_dx)):
                assert float((a - b).norm() / b.norm()) <= bar

        x, off, dz, want, want_dx = inputs(150)
        got = torch.zeros_like(want)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            dx = pred.backward(x, off, dz, got, want_dx=True)
        for _ in range(3):
            got.zero_()
            graph.replay()
            check(got, dx, want, want_dx)
        for B in (150, 40):  # the copied save: the same bits as the aligned one
            x, off, dz, want, want_dx = inputs(B)
            dx = pred.backward(x, off, dz, got, want_dx=True)
            assert torch.equal(got, want) and torch.equal(dx, want_dx)
        x, off, dz, want, want_dx = inputs(260)
        dx = pred.backward(x, off, dz, got, want_dx=True)
        assert torch.equal(got, want) and torch.equal(dx, want_dx)
        pred.close()
