"""Ring DFTs and the theta filter over the LDS engine: ring lengths of one stage (3, 9, 11,
13) and of several whose first or last stage is each of the radices (the filter joins two
transforms there; 11 and 13 take two passes), with and without mixed LDS places (multiples of
8 and 16).  Against the oracle, tolerance 1e-12 as the other parity tests."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp64_err
from paper_2311_14670_amd.synth import flm_gaussian, map_gaussian

pytestmark = pytest.mark.gpu

_SAMP = {"mw": oracle.MW, "mwss": oracle.MWSS, "healpix": oracle.HEALPIX}


@pytest.mark.parametrize("sampling,L,spin", [
    ("mw", 2, 0), ("mw", 5, 1), ("mw", 6, 0), ("mw", 7, 2),                  # 3, 9, 11, 13
    ("mw", 23, 0), ("mw", 50, -1), ("mw", 61, 0), ("mw", 72, 1), ("mw", 85, 0),   # 45, 99, 121, 143, 169
    ("mw", 88, 0), ("mw", 193, 2),                                           # 175, 385
    ("mwss", 2, 0), ("mwss", 7, 1), ("mwss", 12, 0), ("mwss", 13, 0), ("mwss", 32, 1),   # 4, 14, 24, 26, 64
    ("mwss", 88, 0), ("mwss", 128, 2),                                       # 176, 256
    ("healpix", 40, 0)])
def test_against_the_oracle(sampling, L, spin):
    from paper_2311_14670_amd import binding
    nside = 20 if sampling == "healpix" else 0
    plan = binding.Plan(L, spin=spin, sampling=sampling, nside=nside, max_batch=2)
    samp = _SAMP[sampling]
    flm = flm_gaussian(L, spin, seed=80, scale="inv1pl")
    f = plan.inverse(torch.from_numpy(flm).cuda()).cpu().numpy()
    assert fp64_err(f, oracle.s2_inverse(flm, L, spin, samp, nside)) < 1e-12
    g = map_gaussian((2,) + plan.map_shape, seed=81)
    a = plan.forward(torch.from_numpy(g).cuda()).cpu().numpy()
    assert fp64_err(a[1], oracle.s2_forward(g[1], L, spin, samp, nside)) < 1e-12
    G = flm_gaussian(L, spin, seed=82)                       # the adjoint: <F g, G> = <g, F^H G>
    h = plan.forward_adjoint(torch.from_numpy(G).cuda()).cpu().numpy()
    lhs, rhs = np.vdot(G, a[0]), np.vdot(h, g[0])
    assert abs(lhs - rhs) <= 1e-12 * np.linalg.norm(G) * np.linalg.norm(a[0])
    if spin == 0:
        fr = plan.inverse_real(torch.from_numpy(flm).cuda()).cpu().numpy()
        assert fp64_err(fr, oracle.s2_inverse_real(flm, L, samp, nside)) < 1e-12
        ar = plan.forward_real(torch.from_numpy(np.ascontiguousarray(g.real)).cuda()).cpu().numpy()
        assert fp64_err(ar[0], oracle.s2_forward_real(g[0].real.copy(), L, samp, nside)) < 1e-12
