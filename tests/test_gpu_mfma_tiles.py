"""The matrix-core products at the edges of their tiling: more than 32 maps (two row tiles
and, for split BF16, four column tiles per wave), ring and degree counts whose padding ends
inside the last tile of 128, odd ones (records are written by lane pairs), K of few and of
an odd number of steps, and the generator's last, partly filled chunk of 8 degrees.
Against the oracle at the bounds of the formats: 2e-5 (FP32), 2e-4 (split BF16); a map's
result does not depend on its batch (each output sums the same products in the same order
whatever the tile), so there the bits are compared."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_14670_amd.synth import flm_gaussian, map_gaussian

pytestmark = pytest.mark.gpu

TOL = {"fp32": 2e-5, "split_bf16": 2e-4}


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("prec", ["fp32", "split_bf16"])
@pytest.mark.parametrize("L,spin,B", [(9, 0, 33), (33, 0, 40), (65, 0, 36), (129, 0, 33), (130, 1, 34), (193, 0, 33)])
def test_tiles(prec, L, spin, B):
    from paper_2311_14670_amd import binding
    plan = binding.Plan(L, spin=spin, sampling="mw", precision=prec, max_batch=B)
    flm = flm_gaussian(L, spin, seed=90, batch=B, scale="inv1pl")
    f = plan.inverse(torch.from_numpy(flm).cuda())
    g = map_gaussian((B,) + plan.map_shape, seed=91)
    a = plan.forward(torch.from_numpy(g).cuda())
    for b in (0, B - 1):
        assert rel_l2(f[b].cpu().numpy(), oracle.s2_inverse(flm[b], L, spin, oracle.MW)) < TOL[prec]
        assert rel_l2(a[b].cpu().numpy(), oracle.s2_forward(g[b], L, spin, oracle.MW)) < TOL[prec]
        assert torch.equal(f[b], plan.inverse(torch.from_numpy(flm[b]).cuda()))
        assert torch.equal(a[b], plan.forward(torch.from_numpy(g[b]).cuda()))
    alone = binding.Plan(L, spin=spin, sampling="mw", precision=prec, max_batch=1)   # one row tile
    assert torch.equal(f[1], alone.inverse(torch.from_numpy(flm[1]).cuda()))
    assert torch.equal(a[1], alone.forward(torch.from_numpy(g[1]).cuda()))
