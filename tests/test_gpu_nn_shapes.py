"""Surrogate kernels at the sizes where their tiling can go wrong: rows of odd
length and rows longer than a segment, one pixel, dilations with a shared input
window (even, up to 32) and with one window per tap, tensors that start at any
element, and sums over few and many partials.

Bars: products of bf16 values are exact in fp32, so an fp32 result of K terms is
within K 2^-24 sum |terms| of the oracle's, taken on the oracle's terms."""
import sys

import numpy as np
import pytest

from oracle import conv_oracle as C

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2206_00366_amd import rmrt
    return rmrt


def dev(a, dtype, offset=0):
    """a on the GPU, starting `offset` elements into its allocation."""
    a = torch.tensor(np.asarray(a, dtype=np.float32), device="cuda").to(dtype)
    buf = torch.empty(a.numel() + offset, dtype=dtype, device="cuda")
    buf[offset:].copy_(a.reshape(-1))
    return buf[offset:].view(a.shape)


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


CASES = [  # B, H, W, Cin, Cout, dilation, start offset
    (1, 1, 1, 16, 16, 1, 0), (2, 3, 5, 16, 32, 3, 1), (1, 4, 127, 32, 16, 4, 2), (1, 3, 129, 32, 32, 1, 0),
    (2, 5, 131, 32, 32, 32, 1), (1, 2, 300, 16, 32, 34, 0), (3, 37, 40, 32, 32, 6, 3), (1, 600, 3, 16, 16, 2, 0),
]


@pytest.mark.parametrize("B,H,W,cin,cout,dil,off", CASES)
def test_conv_and_gradients(R, B, H, W, cin, cout, dil, off):
    print(f"[nn shapes] {B}x{H}x{W} {cin}->{cout} dil={dil} off={off}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(B + H + W + dil)
    x = C.to_bf16(rng.standard_normal((B, H, W, cin)))
    w = C.to_bf16(rng.standard_normal((cout, 3, 3, cin)) / np.sqrt(9 * cin))
    b = rng.standard_normal(cout).astype(np.float32).astype(np.float64)
    dy = C.to_bf16(rng.standard_normal((B, H, W, cout)))
    y = dev(np.zeros((B, H, W, cout)), torch.float32, off)
    a = dev(np.zeros((B, H, W, cout)), torch.bfloat16, off)
    xd, wd, dyd = dev(x, torch.bfloat16, off), dev(w, torch.bfloat16, off), dev(dy, torch.bfloat16, off)
    R.nn_conv_forward(xd, wd, dev(b, torch.float32, off), y, a, None, dil, R.NN_EPI_SILU)
    ref = C.conv_forward(x, w, b, dil)
    bar = (9 * cin + 1) * 2.0**-24 * C.conv_forward(np.abs(x), np.abs(w), np.abs(b), dil)
    assert (np.abs(host(y) - ref) <= bar).all()
    silu = C.silu(ref)
    assert (np.abs(host(a) - silu) <= 2.0**-8 * np.abs(silu) + 2 * bar + 1e-6).all()
    dw = dev(np.full(w.shape, np.nan), torch.float32, off)
    db = dev(np.full(cout, np.nan), torch.float32, off)
    scr = torch.full((R.nn_wgrad_scratch_floats(B, H, W, cin, cout),), float("nan"), device="cuda")
    R.nn_conv_backward_weight(xd, dyd, dil, dw, db, scr)
    dw_or, db_or = C.conv_backward_weight(x, dy, dil)
    dw_abs, db_abs = C.conv_backward_weight(np.abs(x), np.abs(dy), dil)
    assert (np.abs(host(dw) - dw_or) <= B * H * W * 2.0**-24 * dw_abs).all()
    assert (np.abs(host(db) - db_or) <= B * H * W * 2.0**-24 * db_abs).all()
    # without db, and the same sums again: a fixed order
    again = torch.empty_like(dw)
    R.nn_conv_backward_weight(xd, dyd, dil, again, None, scr)
    assert torch.equal(again, dw)


def test_weight_gradient_beyond_the_row_end_ignores_the_input(R):
    """A row's padding multiplies no input: an infinity there stays out of the taps that do not reach it."""
    B, H, W, c = 1, 2, 33, 16
    rng = np.random.default_rng(1)
    x = C.to_bf16(rng.standard_normal((B, H, W, c)))
    dy = C.to_bf16(rng.standard_normal((B, H, W, c)))
    dy[0, :, 32] = 0.0
    xi = x.copy()
    dw = torch.empty((c, 3, 3, c), device="cuda")
    scr = torch.empty(R.nn_wgrad_scratch_floats(B, H, W, c, c), device="cuda")
    xi[0, 1, 32, 5] = np.inf     # reached from pixel 31 by kx = 2 and from pixel 32 (dy = 0) by kx = 1
    R.nn_conv_backward_weight(dev(xi, torch.bfloat16), dev(dy, torch.bfloat16), 1, dw, None, scr)
    got = host(dw)
    assert np.isfinite(got[..., [k for k in range(c) if k != 5]]).all()
    assert np.isfinite(got[:, :, 0]).all()       # kx = 0 reads columns -1 .. 31 of the input


@pytest.mark.parametrize("P,Cs,Cu", [(1, 16, 3), (257, 16, 16), (1000, 24, 9), (140000, 16, 3), (515, 5, 3)])
def test_masked_mse(R, P, Cs, Cu):
    print(f"[nn mse] P={P} Cs={Cs} C={Cu}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(P)
    out, tgt = rng.standard_normal((P, Cs)), rng.standard_normal((P, Cu))
    wgt = rng.uniform(0.1, 1, P)
    out, tgt, wgt = (v.astype(np.float32).astype(np.float64) for v in (out, tgt, wgt))
    dout = torch.full((P, Cs), 7.0, dtype=torch.bfloat16, device="cuda")
    scr = torch.empty(1024, dtype=torch.float64, device="cuda")
    inv = torch.empty(1, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    R.nn_masked_mse(dev(out, torch.float32), dev(tgt, torch.float32), dev(wgt, torch.float32), dout, scr, inv, loss)
    d = out[:, :Cu] - tgt
    ref = (wgt[:, None] * d * d).sum() / wgt.sum()
    assert abs(loss.item() - ref) <= 2.0**-22 * ref          # differences and 1 / sum rounded to fp32
    g = 2 * wgt[:, None] * d / wgt.sum()
    scale = 2 * wgt[:, None] * (np.abs(out[:, :Cu]) + np.abs(tgt)) / wgt.sum()
    assert (np.abs(host(dout)[:, :Cu] - g) <= 2.0**-8 * np.abs(g) + 2.0**-21 * scale).all()
    assert (host(dout)[:, Cu:] == 0).all()


@pytest.mark.parametrize("B,nx,ny", [(1, 4, 4), (3, 68, 20), (2, 260, 36), (5, 64, 132)])
def test_solid_fractions(R, B, nx, ny):
    rng = np.random.default_rng(nx)
    solid = (rng.random((B, ny, nx)) < 0.3).astype(np.uint8)
    x0 = torch.empty((B, ny // 4, nx // 4, 16), dtype=torch.bfloat16, device="cuda")
    R.nn_features(torch.tensor(solid, device="cuda"), dev(np.full(B, 50.0), torch.float32), B, nx, ny, 4, 0.5, 100.0, x0)
    f = host(x0)
    col = solid.mean(axis=1).reshape(B, nx // 4, 4).mean(axis=2)
    assert (np.abs(f[..., 3] - col[:, None, :]) <= 2.0**-8 * col[:, None, :] + 1e-7).all()
    frac = solid.mean(axis=(1, 2))[:, None, None]
    assert (np.abs(f[..., 4] - frac) <= 2.0**-8 * frac + 1e-7).all()
