"""rmrt_nn_wgrad_scratch_floats (host arithmetic, no GPU): scratch sized for the
largest images of a program serves all smaller ones."""
import pytest

rmrt = pytest.importorskip("paper_2206_00366_amd.rmrt", reason="librmrt.so not built")


@pytest.mark.parametrize("channels", [(16, 16), (16, 32), (32, 16), (32, 32)])
def test_smaller_images_need_no_more_scratch(channels):
    need = rmrt.nn_wgrad_scratch_floats
    for W in (1, 7, 40, 128, 129, 300):
        last = 0
        for H in range(1, 1400):
            n = need(1, H, W, *channels)
            assert n >= last > -1, (H, W)
            last = n
    assert need(1, 512, 128, *channels) <= need(1, 513, 128, *channels)
    for B, H, W in ((16, 64, 128), (3, 171, 100), (9, 57, 260)):
        top = need(B, H, W, *channels)
        assert all(need(b, h, w, *channels) <= top for b in (1, B) for h in (1, H // 2, H) for w in (1, W // 3, W))


def test_scratch_is_refused_below_what_a_launch_needs():
    """513 row segments are shared by 257 workgroups: their slots are enough, a float less
    is refused before anything is launched (no GPU: the pointers are never used)."""
    import ctypes as C
    p = C.c_void_p(16)
    slots = 257 * (9 * 32 * 32 + 32)
    code = rmrt.lib().rmrt_nn_conv_backward_weight(p, p, 1, 513, 128, 32, 32, 1, p, None, p, slots - 1, None)
    assert code == rmrt.EINVAL and b"scratch" in rmrt.lib().rmrt_last_error()
    assert rmrt.nn_wgrad_scratch_floats(1, 513, 128, 32, 32) == 512 * (9 * 32 * 32 + 32)
