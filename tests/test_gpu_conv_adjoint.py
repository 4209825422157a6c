"""The adjoint of the forward over the register convolution engine: the smallest engines,
whose workgroups have fewer threads than a wave (M = 64: 16, M = 128: 32; the filter sums
over them).  <F g, G> = <g, F^H G> with the oracle's F; tolerance 1e-12 of the norms (as
the other parity tests)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_14670_amd.synth import flm_gaussian, map_gaussian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sampling,L,spin", [("mw", 9, 0), ("mw", 9, -1), ("mw", 16, 2), ("mw", 19, 1),
                                             ("mwss", 17, 1), ("mwss", 19, 0), ("mwss", 34, -2), ("mwss", 74, 0)])
def test_small_engines(sampling, L, spin):
    from paper_2311_14670_amd import binding
    samp = {"mw": oracle.MW, "mwss": oracle.MWSS}[sampling]
    plan = binding.Plan(L, spin=spin, sampling=sampling, max_batch=2)
    G = flm_gaussian(L, spin, seed=80, batch=2)
    h = plan.forward_adjoint(torch.from_numpy(G).cuda()).cpu().numpy()
    g = map_gaussian(plan.map_shape, seed=81)
    a = oracle.s2_forward(g, L, spin, samp)
    for b in range(2):
        assert abs(np.vdot(G[b], a) - np.vdot(h[b], g)) <= 1e-12 * np.linalg.norm(G[b]) * np.linalg.norm(a)
    if spin == 0:
        hr = plan.forward_real_adjoint(torch.from_numpy(G).cuda()).cpu().numpy()
        gr = np.ascontiguousarray(g.real)
        ar = oracle.s2_forward_real(gr, L, samp)
        for b in range(2):
            assert (abs(np.vdot(G[b], ar).real - np.vdot(hr[b], gr))
                    <= 1e-12 * np.linalg.norm(G[b]) * np.linalg.norm(ar))
