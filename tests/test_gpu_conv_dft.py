"""Ring DFTs and the theta filter over the register convolution engine: one size per
convolution length M = 64 .. 16384 (the ring length n has a prime factor above 13 and
M / 4 < n <= (M + 1) / 2; 16384: two transforms of half the length).  Small sizes against
the oracle, tolerance 1e-12 as the other parity tests.  Large ones: a map of a single
order m is its first column times e^{i m phi}, and forward(inverse) is the identity;
tolerance 1e-12 of the largest value (a DFT of n points rounds like log2(n) eps, the
sweeps to some 1e-13 at these L)."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp64_err
from paper_2311_14670_amd.synth import flm_gaussian, map_gaussian

pytestmark = pytest.mark.gpu

_SAMP = {"mw": oracle.MW, "dh": oracle.DH, "gl": oracle.GL, "mwss": oracle.MWSS}


@pytest.mark.parametrize("sampling,L,spin", [
    ("mw", 9, 1), ("mw", 24, 0), ("mw", 64, -2), ("mw", 96, 0), ("mw", 252, 2),             # M = 64 .. 1024
    ("mwss", 17, 0), ("mwss", 37, 1), ("gl", 19, 0), ("dh", 97, 0)])
def test_against_the_oracle(sampling, L, spin):
    from paper_2311_14670_amd import binding
    plan = binding.Plan(L, spin=spin, sampling=sampling, max_batch=2)
    flm = flm_gaussian(L, spin, seed=70, scale="inv1pl")
    f = plan.inverse(torch.from_numpy(flm).cuda()).cpu().numpy()
    assert fp64_err(f, oracle.s2_inverse(flm, L, spin, _SAMP[sampling])) < 1e-12
    g = map_gaussian((2,) + plan.map_shape, seed=71)
    a = plan.forward(torch.from_numpy(g).cuda()).cpu().numpy()
    assert fp64_err(a[1], oracle.s2_forward(g[1], L, spin, _SAMP[sampling])) < 1e-12
    if spin == 0:
        fr = plan.inverse_real(torch.from_numpy(flm).cuda()).cpu().numpy()
        assert fp64_err(fr, oracle.s2_inverse_real(flm, L, _SAMP[sampling])) < 1e-12
        ar = plan.forward_real(torch.from_numpy(np.ascontiguousarray(g.real)).cuda()).cpu().numpy()
        assert fp64_err(ar[0], oracle.s2_forward_real(g[0].real.copy(), L, _SAMP[sampling])) < 1e-12


@pytest.mark.parametrize("sampling,L,spin", [("mw", 512, 0), ("mw", 1024, 2), ("mwss", 1031, 0), ("mw", 1030, 0),
                                             ("mw", 2050, 0)])                              # M = 2048 .. 16384
def test_single_orders_and_round_trip(sampling, L, spin):
    from paper_2311_14670_amd import binding
    plan = binding.Plan(L, spin=spin, sampling=sampling)
    flm = flm_gaussian(L, spin, seed=72, scale="inv1pl")
    nphi = plan.map_shape[1]
    k = np.arange(nphi)
    for m in (0, 1, -(L // 3), L - 1):
        one = np.zeros_like(flm)
        one[:, L - 1 + m] = flm[:, L - 1 + m]
        f = plan.inverse(torch.from_numpy(one).cuda()).cpu().numpy()
        want = f[:, :1] * np.exp(2j * np.pi * ((m * k) % nphi) / nphi)
        assert np.abs(f - want).max() <= 1e-12 * np.abs(f).max()
    back = plan.forward(plan.inverse(torch.from_numpy(flm).cuda())).cpu().numpy()
    assert fp64_err(back, flm) < 1e-12
    if spin == 0:
        x = plan.inverse_real(torch.from_numpy(flm).cuda())
        full = flm.copy()                                      # Hermitian completion of the orders m >= 0
        m = np.arange(1, L)
        full[:, L - 1] = full[:, L - 1].real
        full[:, L - 1 - m] = (1 - 2 * (m % 2)) * np.conj(full[:, L - 1 + m])
        assert fp64_err(plan.forward_real(x).cpu().numpy(), full) < 1e-12
