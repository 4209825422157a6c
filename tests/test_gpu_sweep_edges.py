"""The FP64 sweeps at the edges of their tiling: degree chunks of 8, blocks of up to 256
degrees, groups of 64, iterations of four orders, 64-ring tiles and ring blocks of up to
256 rings, with and without mirror rings, one- and two-sided runs, maps of a batch in
one launch.  Against the oracle; tolerance 1e-12 as the other full-size parity tests
(rounding of the FP64 recursion and sums, see test_gpu_sizes.py)."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp64_err
from paper_2311_14670_amd.synth import flm_gaussian, flmn_gaussian, map_gaussian

pytestmark = pytest.mark.gpu

_SAMP = {"mw": oracle.MW, "healpix": oracle.HEALPIX, "dh": oracle.DH, "gl": oracle.GL, "mwss": oracle.MWSS}


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def host(x):
    torch.cuda.synchronize()
    return x.cpu().numpy()


@pytest.fixture(scope="module")
def binding():
    from paper_2311_14670_amd import binding as b
    b.load_library()
    return b


# L around one chunk, one group, one block and two blocks; rings around one tile and one block
EDGES = [("mw", 4, 1, 0), ("mw", 7, 0, 0), ("mw", 8, 0, 0), ("mw", 9, -2, 0), ("gl", 63, 0, 0), ("gl", 64, 2, 0),
         ("gl", 65, 0, 0), ("dh", 32, 0, 0), ("dh", 33, -4, 0), ("healpix", 20, 0, 16), ("healpix", 20, 2, 17),
         ("healpix", 6, 0, 65), ("mwss", 128, 0, 0), ("mwss", 129, 1, 0), ("mw", 255, 2, 0), ("mw", 256, 0, 0),
         ("gl", 257, 0, 0), ("gl", 259, -7, 0)]


@pytest.mark.parametrize("pairing", ["0", "1"])
@pytest.mark.parametrize("sampling,L,spin,nside", EDGES)
def test_tile_edges(binding, monkeypatch, sampling, L, spin, nside, pairing):
    if pairing == "1" and (sampling == "mw" or spin != 0):
        pytest.skip("mirror rings need a symmetric sampling at spin 0")
    monkeypatch.setenv("S2MI_RING_PAIRING", pairing)
    plan = binding.Plan(L, spin=spin, sampling=sampling, nside=nside, max_batch=3)
    samp = _SAMP[sampling]
    flm = flm_gaussian(L, spin, seed=50, batch=3, scale="inv1pl")
    f = host(plan.inverse(dev(flm)))                     # three maps in one launch
    for b in (0, 2):
        assert fp64_err(f[b].ravel(), oracle.s2_inverse(flm[b], L, spin, samp, nside).ravel()) < 1e-12
    assert np.array_equal(f[1], host(plan.inverse(dev(flm[1]))))     # and alone
    g = map_gaussian((3,) + plan.map_shape, seed=51)
    a = host(plan.forward(dev(g)))
    assert fp64_err(a[2], oracle.s2_forward(g[2], L, spin, samp, nside)) < 1e-12
    assert np.array_equal(a[0], host(plan.forward(dev(g[0]))))
    if spin == 0:
        fr = host(plan.inverse_real(dev(flm)))
        assert fp64_err(fr[1].ravel(), oracle.s2_inverse_real(flm[1], L, samp, nside).ravel()) < 1e-12
        gr = np.random.default_rng(52).standard_normal((3,) + plan.map_shape)
        assert fp64_err(host(plan.forward_real(dev(gr)))[1], oracle.s2_forward_real(gr[1], L, samp, nside)) < 1e-12


@pytest.mark.parametrize("L,N", [(17, 2), (65, 3)])
def test_so3_runs_and_maps_in_one_launch(binding, L, N):
    plan = binding.Plan(L, N=N, max_batch=2)
    flmn = flmn_gaussian(L, N, seed=53, batch=2)
    f = host(plan.so3_inverse(dev(flmn)))
    assert fp64_err(f[1], oracle.so3_inverse(flmn[1], L, N)) < 1e-12
    assert np.array_equal(f[0], host(plan.so3_inverse(dev(flmn[0]))))
    g = map_gaussian((2, 2 * N - 1, L, 2 * L - 1), seed=54)
    a = host(plan.so3_forward(dev(g)))
    assert fp64_err(a[0], oracle.so3_forward(g[0], L, N)) < 1e-12
    assert np.array_equal(a[1], host(plan.so3_forward(dev(g[1]))))


def test_non_finite_coefficients_stay_in_their_order(binding):
    """A NaN (an infinity) at one (l, m) reaches the ring samples through order m alone:
    the Fourier line of the map has it there and nowhere else."""
    L, m = 40, 7
    plan = binding.Plan(L, max_batch=1)
    flm = flm_gaussian(L, 0, seed=55)
    ref = host(plan.inverse(dev(flm)))
    # order m's line from the real-linear response of the other orders: the sums of each
    # order are separate, so the transform of a finite change in order m leaves them equal
    flm2 = flm.copy()
    flm2[20, L - 1 + m] += 3.0
    d = np.fft.fft(host(plan.inverse(dev(flm2))) - ref, axis=1)[: L - 1]
    off = np.delete(np.abs(d), m, axis=1)
    assert off.max() < 1e-11 * np.abs(d[:, m]).max()
    for bad in (np.nan, np.inf):
        x = flm.copy()
        x[20, L - 1 + m] = bad
        f = host(plan.inverse(dev(x)))
        assert not np.isfinite(f[: L - 1]).any()         # every sample sums every order
        y = flm.copy()
        y[5, L - 1 + m] = bad                             # below the degree range of order 7: ignored on input
        assert np.array_equal(host(plan.inverse(dev(y))), ref)
