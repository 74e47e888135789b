"""Weight gradients of narrow images: segments of pixels that run over rows and
images (up to 32 columns), at the edges of the rule, against the oracle; scratch of
a larger image; and the time against a wide image of as many pixels.

Bar: products of bf16 values are exact in fp32, so an fp32 sum of K terms is within
K 2^-24 sum |terms| of the oracle's."""
import sys
import time

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


def dev(a, offset=0):
    a = torch.tensor(np.asarray(a, dtype=np.float32), device="cuda").to(torch.bfloat16)
    buf = torch.empty(a.numel() + offset, dtype=torch.bfloat16, device="cuda")
    buf[offset:].copy_(a.reshape(-1))
    return buf[offset:].view(a.shape)


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


# one column; less, just and more than a segment; segments over several images; the
# widest narrow row and the next; taps that leave the image on every side
CASES = [  # B, H, W, Cin, Cout, dilation, start offset
    (1, 1, 1, 16, 16, 1, 0), (1, 127, 1, 32, 16, 2, 1), (3, 64, 2, 16, 32, 1, 0), (40, 1, 7, 32, 32, 3, 0),
    (5, 9, 13, 16, 16, 8, 3), (2, 50, 31, 32, 32, 4, 0), (2, 33, 32, 32, 16, 33, 1), (2, 33, 33, 16, 32, 2, 0),
    (1, 700, 3, 32, 32, 600, 0),
]


@pytest.mark.parametrize("B,H,W,cin,cout,dil,off", CASES)
def test_weight_gradients_of_narrow_images(R, B, H, W, cin, cout, dil, off):
    print(f"[nn narrow] {B}x{H}x{W} {cin}->{cout} dil={dil} off={off}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(B + H + W + dil)
    x = C.to_bf16(rng.standard_normal((B, H, W, cin)))
    dy = C.to_bf16(rng.standard_normal((B, H, W, cout)))
    dw = torch.full((cout, 3, 3, cin), float("nan"), device="cuda")
    db = torch.full((cout,), float("nan"), device="cuda")
    # scratch of an image of more rows
    scr = torch.full((R.nn_wgrad_scratch_floats(B, H + 700, W, cin, cout),), float("nan"), device="cuda")
    R.nn_conv_backward_weight(dev(x, off), dev(dy, off), dil, dw, db, scr)
    dw_or, db_or = C.conv_backward_weight(x, dy, dil)
    dw_abs, db_abs = C.conv_backward_weight(np.abs(x), np.abs(dy), dil)
    assert (np.abs(host(dw) - dw_or) <= B * H * W * 2.0**-24 * dw_abs).all()
    assert (np.abs(host(db) - db_or) <= B * H * W * 2.0**-24 * db_abs).all()


def seconds(fn):
    for _ in range(3):
        fn()
    best = 1e30
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(20):
            fn()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return best


@pytest.mark.parametrize("W", [1, 4, 16])
def test_narrow_images_take_about_the_time_of_wide_ones(R, W):
    times = []
    for w in (W, 128):
        x, dy = (torch.randn(16, 8192 // w, w, 32, device="cuda").bfloat16() for _ in range(2))
        dw, db = torch.empty(32, 3, 3, 32, device="cuda"), torch.empty(32, device="cuda")
        scr = torch.empty(R.nn_wgrad_scratch_floats(16, 8192 // w, w, 32, 32), device="cuda")
        times.append(seconds(lambda: R.nn_conv_backward_weight(x, dy, 1, dw, db, scr)))
    assert times[0] < 2.0 * times[1], times


def test_scratch_of_exactly_a_launch_s_need_is_enough(R):
    """513 row segments take 257 workgroups; what the report asks for also serves smaller images."""
    x, dy = (torch.randn(1, 513, 128, 32, device="cuda").bfloat16() for _ in range(2))
    want, got = (torch.empty(32, 3, 3, 32, device="cuda") for _ in range(2))
    R.nn_conv_backward_weight(x, dy, 1, want, None, torch.empty(R.nn_wgrad_scratch_floats(1, 513, 128, 32, 32), device="cuda"))
    R.nn_conv_backward_weight(x, dy, 1, got, None, torch.empty(257 * (9 * 32 * 32 + 32), device="cuda"))
    assert torch.equal(want, got)
