"""The sweeps' forms for small sizes and the general ones, on both sides of the lines between
them: at most 64 degrees (one chunk of 8 per wave) in the inverse, at most 64 swept
rings (two steps of 32) in the forward, which a grid can cross apart (HEALPix, DH, mirror
rings, SO(3)).  Two- and one-sided runs, whole and cut, against the oracle in the other
parity tests' tolerance."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp64_err
from paper_2311_14670_amd.synth import flm_gaussian, flmn_gaussian, map_gaussian

pytestmark = pytest.mark.gpu

_SAMP = {"mw": oracle.MW, "healpix": oracle.HEALPIX, "dh": oracle.DH, "gl": oracle.GL, "mwss": oracle.MWSS}


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("tiles", ["1", "4", None])
@pytest.mark.parametrize("sampling,L,spin,nside,pairing", [
    ("mw", 2, 0, 0, "0"), ("mw", 5, 2, 0, "0"), ("mw", 57, 0, 0, "0"), ("mw", 64, -3, 0, "0"), ("mw", 65, 0, 0, "0"),
    ("mw", 65, 1, 0, "0"), ("mw", 66, 0, 0, "0"), ("dh", 32, 1, 0, "0"), ("dh", 33, 0, 0, "0"), ("dh", 64, 0, 0, "1"),
    ("dh", 65, 0, 0, "1"), ("gl", 64, 0, 0, "1"), ("healpix", 72, 0, 16, "0"), ("healpix", 72, 2, 16, "0"),
    ("healpix", 20, 0, 40, "1"), ("mwss", 66, -1, 0, "0")])
def test_forms(monkeypatch, sampling, L, spin, nside, pairing, tiles):
    from paper_2311_14670_amd import binding
    monkeypatch.setenv("S2MI_RING_PAIRING", pairing)
    if tiles:
        monkeypatch.setenv("S2MI_ORDER_TILES", tiles)
    plan = binding.Plan(L, spin=spin, sampling=sampling, nside=nside, max_batch=2)
    samp = _SAMP[sampling]
    flm = flm_gaussian(L, spin, seed=110, batch=2)
    f = plan.inverse(dev(flm)).cpu().numpy()
    assert fp64_err(f[1].ravel(), oracle.s2_inverse(flm[1], L, spin, samp, nside).ravel()) < 1e-12
    g = map_gaussian((2,) + plan.map_shape, seed=111)
    a = plan.forward(dev(g)).cpu().numpy()
    assert fp64_err(a[1], oracle.s2_forward(g[1], L, spin, samp, nside)) < 1e-12
    if spin == 0:
        fr = plan.inverse_real(dev(flm)).cpu().numpy()
        assert fp64_err(fr[0].ravel(), oracle.s2_inverse_real(flm[0], L, samp, nside).ravel()) < 1e-12
        ar = plan.forward_real(dev(g.real)).cpu().numpy()
        assert fp64_err(ar[0], oracle.s2_forward_real(np.ascontiguousarray(g[0].real), L, samp, nside)) < 1e-12


@pytest.mark.parametrize("L,N", [(9, 8), (64, 3), (65, 2), (66, 3)])
def test_forms_so3(L, N):
    from paper_2311_14670_amd import binding
    plan = binding.Plan(L, N=N)
    flmn = flmn_gaussian(L, N, seed=112)
    assert fp64_err(plan.so3_inverse(dev(flmn)).cpu().numpy(), oracle.so3_inverse(flmn, L, N)) < 1e-12
    g = map_gaussian((2 * N - 1, L, 2 * L - 1), seed=113)
    assert fp64_err(plan.so3_forward(dev(g)).cpu().numpy(), oracle.so3_forward(g, L, N)) < 1e-12
