"""The surrogate's geometry tensors (host side): the masks of a batch in one uint8
tensor, whatever their type, order and layout, and what is refused."""
import numpy as np
import pytest
import torch

from paper_2206_00366_amd import surrogate as S


@pytest.mark.parametrize("dtype", [np.bool_, np.uint8, np.int32, np.float64])
def test_masks_are_stacked_in_order(dtype):
    rng = np.random.default_rng(5)
    nx, ny = 7, 3
    masks = [(rng.random(nx * ny) < 0.4).astype(dtype) for _ in range(4)]
    masks[1] = masks[1].reshape(ny, nx)                       # any shape of nx ny values
    masks[2] = np.repeat(masks[2], 2)[::2]                    # a stride of two
    masks[3] = np.asfortranarray(masks[3].reshape(ny, nx))    # column order
    geoms = [dict(n=(nx, ny), solid=m, Re=10.5 + k) for k, m in enumerate(masks)]
    solid, re = S.geometry_tensors(geoms, device="cpu")
    want = np.stack([m.reshape(ny, nx) for m in masks]).astype(np.uint8)
    assert solid.dtype == torch.uint8 and solid.is_contiguous() and np.array_equal(solid.numpy(), want)
    assert re.dtype == torch.float32 and re.tolist() == [10.5, 11.5, 12.5, 13.5]


def test_masks_of_different_shapes_are_refused():
    a = dict(n=(7, 3), solid=np.zeros(21, bool), Re=1.0)
    for n in ((7, 1), (1, 3), (3, 7)):
        b = dict(n=n, solid=np.zeros(n[0] * n[1], bool), Re=1.0)
        with pytest.raises(ValueError):
            S.geometry_tensors([a, b], device="cpu")
    with pytest.raises(ValueError):
        S.geometry_tensors([], device="cpu")
