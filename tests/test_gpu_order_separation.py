"""The orders of a forward-type sweep are separate sums: ring spectra that are infinite (or
NaN) at one order reach that order's coefficients and no others.  The samples are A e^{i m
phi} with n A above the largest double, n = 63 = 9 x 7 points a ring, so that the DFT
overflows in bin m alone (the stage before holds 9 A at most).  The adjoint of the inverse
takes them through no theta filter and, on MW, with the pole ring among the slots past
the last swept ring."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

L, N = 32, 63


@pytest.mark.parametrize("m", [0, 1, 5, -12, 31])
@pytest.mark.parametrize("sampling,spin,pairing", [("mw", 0, "0"), ("mw", 2, "0"), ("mw", -5, "0"), ("gl", 0, "0"),
                                                   ("gl", 0, "1"), ("dh", 3, "0")])
def test_overflow_stays_in_its_order(monkeypatch, sampling, spin, pairing, m):
    from paper_2311_14670_amd import binding
    monkeypatch.setenv("S2MI_RING_PAIRING", pairing)
    plan = binding.Plan(L, spin=spin, sampling=sampling)
    assert plan.map_shape[1] == N
    wave = np.exp(2j * np.pi * ((m * np.arange(N)) % N) / N)
    x = np.tile(1.5 * (np.finfo(np.float64).max / N) * wave, (plan.map_shape[0], 1))
    a = plan.inverse_adjoint(torch.from_numpy(x).cuda()).cpu().numpy()
    lmin = max(abs(m), abs(spin))
    assert np.isfinite(np.delete(a, L - 1 + m, axis=1)).all()
    assert not np.isfinite(a[lmin:, L - 1 + m]).any()
    assert np.all(a[:lmin, L - 1 + m] == 0)
