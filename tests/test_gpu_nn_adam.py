"""The surrogate's Adam update: one launch over the flat tensors gives the bits of one
call per tensor, and tensors that a caller puts into the lists are still updated."""
import copy

import pytest
import torch

from paper_2206_00366_amd import rmrt as R
from paper_2206_00366_amd import surrogate as S

pytestmark = pytest.mark.gpu


def _net(seed):
    net = S.Surrogate(seed=seed, B=1, H=4, W=4)
    g = torch.Generator(device="cuda").manual_seed(seed)
    for t in net.gw + net.gb:
        t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    return net


def _lists(net):
    return [net.w32, net.b32, net.wbf, net.mw, net.mb, net.vw, net.vb]


@pytest.mark.parametrize("form", ["flat", "copied", "own_tensor", "own_gradient"])
def test_flat_update_equals_one_call_per_tensor(form):
    net = _net(3)
    ref = [[t.clone() for t in lst] for lst in _lists(net)]
    gw, gb = [t.clone() for t in net.gw], [t.clone() for t in net.gb]
    if form == "copied":
        net = copy.deepcopy(net)
    if form == "own_tensor":
        net.w32[2] = net.w32[2].clone()
    if form == "own_gradient":
        net.gb[3] = net.gb[3].clone()
    assert net._shares_flat() == (form in ("flat", "copied"))
    w, b, wbf, mw, mb, vw, vb = ref
    for t in (1, 2, 3):
        net.adam(1e-2)
        for l in range(4):
            R.nn_adam(w[l], wbf[l], gw[l], mw[l], vw[l], 1e-2, t)
            R.nn_adam(b[l], None, gb[l], mb[l], vb[l], 1e-2, t)
    for got, want in zip(_lists(net), ref):
        for x, y in zip(got, want):
            assert torch.equal(x, y)
