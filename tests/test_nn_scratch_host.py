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
