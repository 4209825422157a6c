"""One-sided forward sweeps (spin s != 0, whose runs n = -s and n = +s feed one side each;
real signals, orders m >= 0): iterations of four orders whose sums are stored one iteration
later, the last ones of a piece after its end.  Band-limits of every remainder by four,
blocks whole and cut into pieces, and cut pieces that a workgroup runs as one: 60 maps of
2 groups of degrees in 4 pieces each are 480 or 960 slots for 256 compute units, so a
workgroup takes several consecutive ones.  Bit for bit the same; against the oracle in the
other parity tests' tolerance."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp64_err
from paper_2311_14670_amd.synth import map_gaussian

pytestmark = pytest.mark.gpu

B = 60


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("L", [96, 97, 98, 99])
@pytest.mark.parametrize("spin", [0, 2, -1])
def test_whole_cut_and_joined_pieces(monkeypatch, L, spin):
    from paper_2311_14670_amd import binding
    plans = {}
    for tiles in ("1", "4", None):                       # whole, cut in 4, the plan's own cuts
        if tiles:
            monkeypatch.setenv("S2MI_ORDER_TILES", tiles)
        else:
            monkeypatch.delenv("S2MI_ORDER_TILES")
        plans[tiles] = binding.Plan(L, spin=spin, max_batch=B)
    assert [plans[t].info["order_tiles"] for t in ("1", "4")] == [1, 4]
    g = map_gaussian((B,) + plans["1"].map_shape, seed=100 + L)
    if spin == 0:
        call, x = "forward_real", dev(g.real)
        ref = oracle.s2_forward_real(np.ascontiguousarray(g[7].real), L)
    else:
        call, x = "forward", dev(g)
        ref = oracle.s2_forward(g[7], L, spin)
    whole = getattr(plans["1"], call)(x)                 # 60 maps in one launch
    assert fp64_err(whole[7].cpu().numpy(), ref) < 1e-13
    for p in plans.values():
        assert torch.equal(getattr(p, call)(x), whole)
        alone = x[7].clone()                             # (a real map of odd size: aligned)
        assert torch.equal(getattr(p, call)(alone), whole[7])        # one slot per workgroup
