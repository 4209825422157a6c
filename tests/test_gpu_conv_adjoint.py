"""The adjoint of the forward over the register convolution engine: the smallest engines,
whose workgroups have fewer threads than a wave (M = 64: 16, M = 128: 32), and the MWSS
filter's own form (its Nyquist component is a sum over the workgroup; four DFTs per
filter) up to the transform in two halves (2 L > 4096 with a prime factor above 13).
<F g, G> = <g, F^H G> with the oracle's F at small L and the library's at large L, where
the forward is checked by its round trip; tolerance 1e-12 of the norms (as the other
parity and large-size tests: DFTs round like log2(n) eps, the sweeps to some 1e-13)."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp64_err
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


@pytest.mark.parametrize("L,spin", [(523, 0), (1031, 1), (2053, 0), (2053, 2)])              # M = 4096 .. 16384
def test_mwss_large(L, spin):
    from paper_2311_14670_amd import binding
    plan = binding.Plan(L, spin=spin, sampling="mwss")
    flm = flm_gaussian(L, spin, seed=82, scale="inv1pl")
    back = plan.forward(plan.inverse(torch.from_numpy(flm).cuda())).cpu().numpy()
    assert fp64_err(back, flm) < 1e-12
    G = flm_gaussian(L, spin, seed=83, scale="inv1pl")
    g = map_gaussian(plan.map_shape, seed=84)                # not band-limited: the filter's Nyquist component
    a = plan.forward(torch.from_numpy(g).cuda()).cpu().numpy()
    h = plan.forward_adjoint(torch.from_numpy(G).cuda()).cpu().numpy()
    assert abs(np.vdot(G, a) - np.vdot(h, g)) <= 1e-12 * np.linalg.norm(G) * np.linalg.norm(a)
