"""The theta filter takes two consecutive orders at a time.  Maps that live on the pole
rings alone (whose samples at odd m + s have no place on the theta-torus and reach the
rings through the odd part of the weight), the last order of an odd band-limit (alone in
its pair), one-sided (real) calls and the adjoint.  Against the oracle's exact theta
integral; tolerance 1e-12 of the result as the other parity tests."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp64_err
from paper_2311_14670_amd.synth import flm_gaussian, map_gaussian

pytestmark = pytest.mark.gpu

_SAMP = {"mw": oracle.MW, "mwss": oracle.MWSS}


@pytest.mark.parametrize("sampling", ["mw", "mwss"])
@pytest.mark.parametrize("L,spin", [(2, 0), (3, 1), (16, 0), (17, 0), (33, -2), (24, 3)])
def test_pole_only_maps_and_adjoint(sampling, L, spin):
    from paper_2311_14670_amd import binding
    plan = binding.Plan(L, spin=spin, sampling=sampling, max_batch=2)
    g = np.zeros((2,) + plan.map_shape, dtype=np.complex128)
    g[0, -1] = map_gaussian(plan.map_shape[1], seed=60)                 # south pole ring
    g[1, 0 if sampling == "mwss" else -1] = map_gaussian(plan.map_shape[1], seed=61)
    a = plan.forward(torch.from_numpy(g).cuda()).cpu().numpy()
    for b in range(2):
        assert fp64_err(a[b], oracle.s2_forward(g[b], L, spin, _SAMP[sampling])) < 1e-12
    # adjoint: <F g, G> = <g, F^H G> on the same maps
    G = flm_gaussian(L, spin, seed=62)
    h = plan.forward_adjoint(torch.from_numpy(G).cuda()).cpu().numpy()
    for b in range(2):
        lhs, rhs = np.vdot(G, a[b]), np.vdot(h, g[b])
        assert abs(lhs - rhs) <= 1e-12 * np.linalg.norm(G) * np.linalg.norm(a[b])
    if spin == 0:
        ar = plan.forward_real(torch.from_numpy(np.ascontiguousarray(g.real)).cuda()).cpu().numpy()
        for b in range(2):
            assert fp64_err(ar[b], oracle.s2_forward_real(g[b].real.copy(), L, _SAMP[sampling])) < 1e-12
