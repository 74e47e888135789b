"""The devices and values that the surrogate's geometry tensors take (host side)."""
import numpy as np
import torch

from paper_2206_00366_amd import surrogate as S


def geoms():
    rng = np.random.default_rng(3)
    return [dict(n=(7, 3), solid=rng.random(21) < 0.4, Re=10.5 + k) for k in range(3)]


def test_no_device_is_the_default_device():
    solid, re = S.geometry_tensors(geoms(), device=None)
    want_solid, want_re = S.geometry_tensors(geoms(), device="cpu")
    assert solid.device.type == re.device.type == "cpu"
    assert torch.equal(solid, want_solid) and torch.equal(re, want_re)


def test_a_default_device_elsewhere_changes_nothing():
    want_solid, want_re = S.geometry_tensors(geoms(), device="cpu")
    with torch.device("meta"):
        solid, re = S.geometry_tensors(geoms(), device="cpu")
    assert solid.device.type == re.device.type == "cpu"
    assert torch.equal(solid, want_solid) and torch.equal(re, want_re)


def test_reynolds_numbers_of_any_shape():
    made = geoms()
    for g in made:
        g["Re"] = np.array([g["Re"]])     # one value in an array, as a computed field gives it
    _, re = S.geometry_tensors(made, device="cpu")
    assert re.shape == (3, 1) and re.flatten().tolist() == [10.5, 11.5, 12.5]
