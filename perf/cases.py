"""Timed workloads of the spin SHT and Wigner transforms on one GPU.

Each case is one pass through the package's public entry points (binding.Plan,
autograd) as a user's program calls them:

  op "pair"          inverse, then forward of its map (the paper's round trip)
  op "real_pair"     the same for a real signal (inverse_real / forward_real)
  op "so3_pair"      inverse and forward Wigner transform, azimuthal band N
  op "grad_inverse"  one optimisation step's gradient through the inverse
  op "grad_forward"  one optimisation step's gradient through the forward

`listed` names the cases that are tracked, `draw` takes further ones from the same
ranges, `prepare` / `run` make the inputs and do one pass, `work` counts what a pass
cannot do without, and `exact` computes a pass's results in 64 bits with plain torch
(d^l_{m,n} by the upward three-term recursion in l, sums as matrix products or
elementwise accumulation, ring DFTs by torch.fft).
"""
import math

import numpy as np
import torch

# Coefficients are Gaussian with the spectrum 1/(1+l) (a smooth field), maps are what
# the inverse makes of them, or white noise where a forward is called by itself.
LMIN, LMAX = 64, 4096            # band-limits of the serving mix


def _case(name, op, sampling, L, spin=0, N=1, batch=1, nside=0, precision="fp64"):
    return dict(name=name, op=op, sampling=sampling, L=L, spin=spin, N=N, batch=batch, nside=nside,
                precision=precision)


def listed():
    return [
        # smallest serving request: polarised (spin 2) map at the mix's lowest band-limit; latency
        _case("mw_L64_s2", "pair", "mw", 64, spin=2),
        # small HEALPix maps served as one batch of 8, the serving loop's batch limit
        _case("hpx_L128_b8", "pair", "healpix", 128, batch=8, nside=64),
        # Wigner transform of a directional (steerable) analysis: 7 azimuthal orders
        _case("so3_L96_N4", "so3_pair", "mw", 96, N=4),
        # odd sizes: gradient through the forward, spin 2 Gauss-Legendre maps, a small batch
        _case("gl_L301_s2_b4_grad", "grad_forward", "gl", 301, spin=2, batch=4),
        # training step: gradient of a map loss through the inverse, 16 maps at L = 512
        _case("mw_L512_b16_grad", "grad_inverse", "mw", 512, batch=16),
        # ordinary polarised map (spin 2), one at a time
        _case("mw_L1024_s2", "pair", "mw", 1024, spin=2),
        # ordinary real signal on the equiangular 2L-ring grid, ragged band-limit
        _case("dh_L700_real", "real_pair", "dh", 700),
        # the headline round trip
        _case("mw_L2048", "pair", "mw", 2048),
        # full-resolution real sky map: HEALPix nside 1024
        _case("hpx_L2048_real", "real_pair", "healpix", 2048, nside=1024),
        # large batches with the contraction on the matrix cores: fp32 and split bf16
        _case("mw_L1024_b32_fp32", "pair", "mw", 1024, batch=32, precision="fp32"),
        _case("mw_L2048_b64_bf16", "pair", "mw", 2048, batch=64, precision="split_bf16"),
        # the largest band-limit
        _case("mw_L4096", "pair", "mw", 4096),
    ]


def draw(rng):
    """One more case of the listed ranges (sizes log-uniform, odd ones among them)."""
    def logint(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["pair", "pair", "pair", "real_pair", "so3_pair", "grad_inverse", "grad_forward", "mixed"])
    if kind == "mixed":
        L = logint(256, 1280)
        return _drawn(op="pair", sampling="mw", L=L, spin=rng.choice([0, 2]), batch=rng.randint(8, 48),
                      precision=rng.choice(["fp32", "split_bf16"]))
    if kind == "so3_pair":
        return _drawn(op=kind, sampling="mw", L=logint(64, 320), N=rng.randint(2, 8), batch=rng.choice([1, 1, 2]))
    sampling = rng.choice(["mw", "mw", "healpix", "healpix", "gl", "dh", "mwss"])
    spin = 0 if kind == "real_pair" else rng.choice([0, 0, 2, 2, -1])
    if kind in ("grad_inverse", "grad_forward"):
        if kind == "grad_forward":
            sampling = rng.choice(["gl", "dh", "healpix"])
        return _drawn(op=kind, sampling=sampling, L=logint(64, 700), spin=spin, batch=rng.randint(1, 16))
    L = logint(64, 2600)
    batch = rng.randint(2, 8) if L < 600 and rng.random() < 0.5 else 1
    return _drawn(op=kind, sampling=sampling, L=L, spin=spin, batch=batch)


def _drawn(op, sampling, L, spin=0, N=1, batch=1, precision="fp64"):
    nside = (L + 1) // 2 if sampling == "healpix" else 0
    c = _case("", op, sampling, L, spin, N, batch, nside, precision)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs and one pass
def _gaussian(shape, seed, device, dtype=torch.complex128):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    if dtype == torch.float64:
        return torch.randn(shape, generator=g, dtype=torch.float64, device=device)
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=g, dtype=torch.float64, device=device))


def _coefficients(case, seed, device):
    """[batch?][2N-1?][L][2L-1], zero where l < max(|m|, |n|)."""
    L, N, B = case["L"], case["N"], case["batch"]
    so3 = case["op"] == "so3_pair"
    shape = (B,) * (B > 1) + ((2 * N - 1,) if so3 else ()) + (L, 2 * L - 1)
    x = _gaussian(shape, seed, device)
    ell = torch.arange(L, device=device)[:, None]
    m = torch.arange(-(L - 1), L, device=device)[None, :]
    ok = ell >= m.abs()
    if so3:
        n = torch.arange(-(N - 1), N, device=device)[:, None, None]
        ok = ok & (ell >= n.abs())
    else:
        ok = ok & (ell >= abs(case["spin"]))
    return x.mul_(ok.to(torch.float64) / (1.0 + ell))


def _map_shape(case):
    L = case["L"]
    return {"mw": (L, 2 * L - 1), "gl": (L, 2 * L - 1), "dh": (2 * L, 2 * L - 1), "mwss": (L + 1, 2 * L),
            "healpix": (12 * case["nside"] ** 2,)}[case["sampling"]]


def _inputs(case, seed, device):
    if case["op"] in ("pair", "real_pair", "so3_pair"):
        return (_coefficients(case, seed, device),)
    B = case["batch"]
    f = _gaussian((B,) * (B > 1) + _map_shape(case), seed + 7919, device)
    x = _coefficients(case, seed, device)
    return (x, f) if case["op"] == "grad_inverse" else (f, x)


def prepare(case, seed):
    from paper_2311_14670_amd import binding
    dev = torch.device("cuda")
    plan = binding.Plan(case["L"], spin=case["spin"], N=case["N"], sampling=case["sampling"], nside=case["nside"],
                        max_batch=case["batch"], precision=case["precision"])
    _ = plan.workspace
    xs = _inputs(case, seed, dev)
    if case["op"] in ("grad_inverse", "grad_forward"):
        xs[0].requires_grad_(True)
    return {"op": case["op"], "plan": plan, "x": xs}


def run(state):
    op, plan, xs = state["op"], state["plan"], state["x"]
    if op == "pair":
        f = plan.inverse(xs[0])
        return {"map": f, "flm": plan.forward(f)}
    if op == "real_pair":
        f = plan.inverse_real(xs[0])
        return {"map": f, "flm": plan.forward_real(f)}
    if op == "so3_pair":
        f = plan.so3_inverse(xs[0])
        return {"map": f, "flm": plan.so3_forward(f)}
    from paper_2311_14670_amd import autograd
    x, target = xs
    y = autograd.inverse(x, plan) if op == "grad_inverse" else autograd.forward(x, plan)
    r = torch.view_as_real(y - target)
    loss = (r * r).sum()
    return {"loss": loss.detach(), "grad": torch.autograd.grad(loss, x)[0]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes: each input read once, each output written once.  Flops: per direction and
    map 4 per (ring, l, m) triple (half of them for a real signal), and once per
    direction 4 for every Wigner-d value, needed for m >= 0 at spin 0 and at every m
    otherwise."""
    L, s, N, B = case["L"], abs(case["spin"]), case["N"], case["batch"]
    rings = {"mw": L, "gl": L, "dh": 2 * L, "mwss": L + 1, "healpix": 4 * case["nside"] - 1}[case["sampling"]]
    ncoef = L * (2 * L - 1)
    nsamp = int(np.prod(_map_shape(case)))
    T = rings * (L * L - s * s)
    slices = 2 * N - 1
    if case["op"] == "so3_pair":
        one = 4 * T * slices * B + 2 * T * slices
        return {"bytes": 2 * 16 * B * slices * (ncoef + nsamp), "flops": 2 * one}
    if case["op"] == "real_pair":
        return {"bytes": 2 * B * (16 * ncoef + 8 * nsamp), "flops": 2 * (2 * T * B + 2 * T)}
    one = 4 * T * B + (2 * T if s == 0 else 4 * T)
    if case["op"] == "pair":
        return {"bytes": 2 * 16 * B * (ncoef + nsamp), "flops": 2 * one}
    n_in, n_out = (ncoef, nsamp) if case["op"] == "grad_inverse" else (nsamp, ncoef)
    return {"bytes": 16 * B * (2 * n_in + n_out), "flops": 2 * one}    # input, target, gradient


# ------------------------------------------------------------------ 64-bit results in plain torch
def _rings(case):
    """theta [rings], samples per ring, first sample, half-pixel shift."""
    L, sampling, nside = case["L"], case["sampling"], case["nside"]
    if sampling == "healpix":
        th, nphi, shift = [], [], []
        for i in range(1, 4 * nside):
            j = min(i, 4 * nside - i)
            if j < nside:
                th1 = 2.0 * math.asin(j / (math.sqrt(6.0) * nside))     # 1 - cos = j^2 / (3 nside^2)
                th.append(th1 if i < 2 * nside else math.pi - th1)
                nphi.append(4 * j)
                shift.append(1)
            else:
                th.append(math.acos(4.0 / 3.0 - 2.0 * i / (3.0 * nside)))
                nphi.append(4 * nside)
                shift.append(1 if (i - nside) % 2 == 0 else 0)
        start = np.concatenate([[0], np.cumsum(nphi)[:-1]])
        return np.array(th), nphi, start, shift
    if sampling == "mw":
        th, n = (2 * np.arange(L) + 1) * np.pi / (2 * L - 1), 2 * L - 1
    elif sampling == "mwss":
        th, n = np.arange(L + 1) * np.pi / L, 2 * L
    elif sampling == "dh":
        th, n = (2 * np.arange(2 * L) + 1) * np.pi / (4 * L), 2 * L - 1
    else:
        x, _ = np.polynomial.legendre.leggauss(L)
        th, n = np.arccos(-np.sort(-x) if x[0] > x[-1] else x[::-1]), 2 * L - 1
    return th, [n] * len(th), np.arange(len(th)) * n, [0] * len(th)


def _ring_weights(case):
    """Quadrature weight of each ring of the forward (phi rule included)."""
    L, sampling = case["L"], case["sampling"]
    if sampling == "gl":
        x, w = np.polynomial.legendre.leggauss(L)
        return w[np.argsort(-x)] * 2 * np.pi / (2 * L - 1)
    if sampling == "dh":
        th = (2 * np.arange(2 * L) + 1) * np.pi / (4 * L)
        k = 2 * np.arange(L) + 1
        return 4 * np.pi / (L * (2 * L - 1)) * np.sin(th) * (np.sin(np.outer(th, k)) / k).sum(1)
    return np.full(4 * case["nside"] - 1, 4 * np.pi / (12 * case["nside"] ** 2))


class _Wigner:
    """d^l_{m,n}(theta) for m = m0 .. m1-1 (m >= 0) and all rings, l = 0, 1, ...: the
    upward recursion in l from l = max(m, |n|), each value kept as x 2^E with E <= 0 a
    multiple of 400 (a value with E < 0 is below 2^-400 and counts as zero)."""

    def __init__(self, theta, n, m0, m1, device):
        self.n, self.m0, self.m1 = n, m0, m1
        self.m = torch.arange(m0, m1, dtype=torch.float64, device=device)[:, None]
        self.cos = torch.tensor(np.cos(theta), device=device)[None, :]
        an, ld = abs(n), np.longdouble
        m = np.arange(m0, m1)
        l0 = np.maximum(m, an)
        fact = np.concatenate([[ld(0)], np.cumsum(np.log2(np.arange(1, 2 * int(l0.max()) + 2, dtype=ld)))])
        with np.errstate(divide="ignore"):
            lc = np.log2(np.abs(np.cos(np.asarray(theta, ld) / 2)))
            ls = np.log2(np.abs(np.sin(np.asarray(theta, ld) / 2)))
        # d^l_{l,n} = (-1)^{l-n} C c^{l+n} s^{l-n};  d^l_{m,l} = C c^{l+m} s^{l-m};
        # d^l_{m,-l} = (-1)^{m+l} C c^{l-m} s^{l+m},  C = sqrt(binomial)
        other = np.where(m >= an, n, m if n >= 0 else -m)
        sign = np.where(m >= an, np.where((m - n) % 2, -1.0, 1.0),
                        np.where((n < 0) & ((m + an) % 2 == 1), -1.0, 1.0))
        lb = (fact[2 * l0] - fact[l0 - other] - fact[l0 + other]) / 2
        p, q = (l0 + other)[:, None].astype(ld), (l0 - other)[:, None].astype(ld)
        with np.errstate(invalid="ignore"):
            x = lb[:, None] + np.where(p > 0, p * lc[None, :], 0) + np.where(q > 0, q * ls[None, :], 0)
        x = np.maximum(x, ld(-4e8))
        E = np.minimum(np.ceil(x / 400), 0) * 400
        self.start = torch.tensor((np.exp2(x - E) * sign[:, None]).astype(np.float64), device=device)
        self.startE = torch.tensor(E.astype(np.float64), device=device)
        self.l0 = l0
        self.cur = torch.zeros_like(self.start)
        self.prev = torch.zeros_like(self.start)
        self.E = torch.zeros_like(self.start)
        self.l = int(l0.min()) - 1
        self.live = 0                                   # orders started so far (m0 .. m0 + live - 1)

    def step(self):
        """Advance to the next l; returns (l, live orders, d over them with the not yet
        representable values set to zero)."""
        l, k = self.l, self.live
        if k:
            m, n = self.m[:k], float(self.n)
            if l == 0:
                a, b = self.cos.expand(k, -1), torch.zeros_like(m)
            else:
                l1 = float(l + 1)
                den = l * torch.sqrt((l1 * l1 - m * m) * (l1 * l1 - n * n))
                b = l1 * torch.sqrt((float(l) * l - m * m) * (float(l) * l - n * n)) / den
                a = (2 * l + 1) * (l * l1 * self.cos - m * n) / den
            new = torch.addcmul(b * self.prev[:k] * -1.0, a, self.cur[:k])
            self.prev[:k] = self.cur[:k]
            self.cur[:k] = new
            if l % 4 == 0:
                big = ((self.cur[:k].abs() > 1.0) & (self.E[:k] < 0)).double()
                f = 1.0 - big * (1.0 - 2.0 ** -50)      # 2^-50 or 1, eight times: 2^-400 or 1
                for v in (self.cur[:k], self.prev[:k]):
                    v *= f ** 8
                self.E[:k] += 400.0 * big
        self.l = l = l + 1
        new_live = int(np.searchsorted(self.l0, l, side="right"))
        if new_live > k:
            self.cur[k:new_live] = self.start[k:new_live]
            self.E[k:new_live] = self.startE[k:new_live]
            self.live = new_live
        k = self.live
        # between the checks a value may pass 1 with E < 0: bounded, and still below 2^-300
        return l, k, torch.where(self.E[:k] < 0, 0.0, self.cur[:k])


def _runs(spin):
    """(n of the run, side, sign rule): side +1 serves m >= 0 with d_{m,-spin}, side -1
    serves m = -mu < 0 with d_{-mu,-spin} = (-1)^{mu+spin} d_{mu,spin}."""
    return [(0, (+1, -1))] if spin == 0 else [(-spin, (+1,)), (spin, (-1,))]


def _synth(flm, theta, spin, w, real=False):
    """F[b][m + L - 1][ring] = sum_l w_l flm[b][l][m] d^l_{m,-spin}(theta)."""
    B, L, M = flm.shape
    dev, R = flm.device, len(theta)
    F = torch.zeros((B, M, R), dtype=torch.complex128, device=dev)
    a = flm * w[None, :, None]
    for n, sides in _runs(spin):
        for m0, m1 in _chunks(L, R, B):
            W = _Wigner(theta, n, m0, m1, dev)
            mu = torch.arange(m0, m1, device=dev)
            cs = []
            for sd in sides:
                if sd < 0 and real:
                    continue
                c = a[:, :, L - 1 + mu] if sd > 0 else a[:, :, L - 1 - mu] * (1.0 - 2.0 * ((mu + spin) % 2))
                cs.append((sd, c))
            if B > 1:
                D = torch.zeros((m1 - m0, L, R), dtype=torch.float64, device=dev)
                while W.l < L - 1:
                    l, k, d = W.step()
                    D[:k, l] = d
                for sd, c in cs:
                    A = torch.view_as_real(c).permute(2, 0, 3, 1).reshape(m1 - m0, 2 * B, L).contiguous()
                    V = torch.matmul(A, D).reshape(m1 - m0, B, 2, R).permute(1, 0, 3, 2).contiguous()
                    _put(F, sd, mu, L, torch.view_as_complex(V))
                del D
            else:
                acc = [torch.zeros((m1 - m0, R, 2), dtype=torch.float64, device=dev) for _ in cs]
                while W.l < L - 1:
                    l, k, d = W.step()
                    for (sd, c), o in zip(cs, acc):
                        v = torch.view_as_real(c[0, l, :k])
                        o[:k, :, 0].addcmul_(d, v[:, :1])
                        o[:k, :, 1].addcmul_(d, v[:, 1:])
                for (sd, c), o in zip(cs, acc):
                    _put(F, sd, mu, L, torch.view_as_complex(o)[None])
    return F


def _put(F, sd, mu, L, v):
    if sd > 0:
        F[:, L - 1 + mu] = v
    else:
        keep = mu > 0
        F[:, (L - 1 - mu)[keep]] = v[:, keep]


def _analyse(F, theta, spin, w, real=False):
    """flm[b][l][m] = w_l sum_ring F[b][m][ring] d^l_{m,-spin}(theta) (zero for l < |spin|)."""
    B, M, R = F.shape
    L, dev = (M + 1) // 2, F.device
    out = torch.zeros((B, L, M), dtype=torch.complex128, device=dev)
    for n, sides in _runs(spin):
        for m0, m1 in _chunks(L, R, B):
            W = _Wigner(theta, n, m0, m1, dev)
            mu = torch.arange(m0, m1, device=dev)
            for_sides = [sd for sd in sides if sd > 0 or not real]
            src = {sd: F[:, L - 1 + sd * mu] for sd in for_sides}
            sgn = {sd: 1.0 if sd > 0 else (1.0 - 2.0 * ((mu + spin) % 2)).to(torch.float64) for sd in for_sides}
            if B > 1:
                D = torch.zeros((m1 - m0, L, R), dtype=torch.float64, device=dev)
                while W.l < L - 1:
                    l, k, d = W.step()
                    D[:k, l] = d
                for sd in for_sides:
                    H = torch.view_as_real(src[sd]).permute(1, 2, 0, 3).reshape(m1 - m0, R, 2 * B).contiguous()
                    V = torch.matmul(D, H).reshape(m1 - m0, L, B, 2).permute(2, 1, 0, 3).contiguous()
                    out[:, :, L - 1 + sd * mu] = torch.view_as_complex(V) * sgn[sd]
                del D
            else:
                H = {sd: torch.view_as_real(src[sd][0]) for sd in for_sides}
                while W.l < L - 1:
                    l, k, d = W.step()
                    for sd in for_sides:
                        v = torch.stack([(d * H[sd][:k, :, 0]).sum(1), (d * H[sd][:k, :, 1]).sum(1)], -1)
                        s = sgn[sd] if sd > 0 else sgn[sd][:k]
                        out[0, l, L - 1 + sd * mu[:k]] = torch.view_as_complex(v) * s
    return out * w[None, :, None]


def _chunks(L, R, B):
    """Order ranges: all at once for one map, else so that the d values fit 8 GB."""
    step = L if B == 1 else max(1, min(L, int(8e9 / (8.0 * L * R))))
    return [(a, min(L, a + step)) for a in range(0, L, step)]


def _phi_inverse(F, case):
    """Order lines F[b][m][ring] -> samples [b][...]: f(phi_p) = sum_m F_m e^{i m phi_p}."""
    B, M, R = F.shape
    L = (M + 1) // 2
    _, nphi, start, shift = _rings(case)
    m = torch.arange(-(L - 1), L, device=F.device)
    if case["sampling"] != "healpix":
        X = torch.zeros((B, R, nphi[0]), dtype=torch.complex128, device=F.device)
        X[:, :, m % nphi[0]] = F.transpose(1, 2)
        return torch.fft.ifft(X, norm="forward")
    out = np.empty((B, 12 * case["nside"] ** 2), dtype=np.complex128)    # ring lengths differ: host FFTs
    Fh, mh = F.transpose(1, 2).contiguous().cpu().numpy(), np.arange(-(L - 1), L)
    for r in range(R):
        n = nphi[r]
        v = Fh[:, r]
        if shift[r]:
            v = v * np.exp(1j * np.pi / n * (mh % (2 * n)))
        head = (-(L - 1)) % n                           # bin of the lowest order
        tail = -(head + M) % n
        X = np.pad(v, ((0, 0), (head, tail))).reshape(B, -1, n).sum(1)
        out[:, start[r]:start[r] + n] = np.fft.ifft(X, norm="forward")
    return torch.from_numpy(out).to(F.device)


def _phi_forward(f, case):
    """Samples [b][...] -> F[b][m][ring] = sum_p f(phi_p) e^{-i m phi_p}."""
    L = case["L"]
    _, nphi, start, shift = _rings(case)
    B, R = f.shape[0], len(nphi)
    m = torch.arange(-(L - 1), L, device=f.device)
    if case["sampling"] != "healpix":
        return torch.fft.fft(f.reshape(B, R, nphi[0]))[:, :, m % nphi[0]].transpose(1, 2).contiguous()
    Fh, fh, mh = np.empty((B, R, 2 * L - 1), dtype=np.complex128), f.cpu().numpy(), np.arange(-(L - 1), L)
    for r in range(R):
        n = nphi[r]
        v = np.fft.fft(fh[:, start[r]:start[r] + n])[:, mh % n]
        Fh[:, r] = v * np.exp(-1j * np.pi / n * (mh % (2 * n))) if shift[r] else v
    return torch.from_numpy(Fh).to(f.device).transpose(1, 2).contiguous()


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    L, spin, B, op = case["L"], case["spin"], case["batch"], case["op"]
    xs = _inputs(case, seed, dev)
    theta = _rings(case)[0]
    ell = torch.arange(L, dtype=torch.float64, device=dev)
    w = torch.sqrt((2 * ell + 1) / (4 * math.pi)) * (-1.0) ** spin

    def shaped(v, like_batch=True):
        return v if B > 1 or not like_batch else v[0]

    if op == "so3_pair":
        x = xs[0].reshape((B,) + xs[0].shape[-3:])
        N = case["N"]
        wn = (2 * ell + 1) / (8 * math.pi ** 2)
        n = torch.arange(-(N - 1), N, device=dev)
        fn = torch.stack([_phi_inverse(_synth(x[:, k], theta, -int(n[k]), wn), case) for k in range(2 * N - 1)], 1)
        ph = torch.outer(n, torch.arange(2 * N - 1, device=dev)) % (2 * N - 1)
        e = torch.polar(torch.ones_like(ph, dtype=torch.float64), ph.double() * (2 * math.pi / (2 * N - 1)))
        f = (fn[:, :, None] * e[None, :, :, None, None]).sum(1)
        return {"map": shaped(f), "flm": xs[0]}         # exact round trip (sampling theorem)
    if op in ("pair", "real_pair"):
        real = op == "real_pair"
        x = xs[0].reshape((B,) + xs[0].shape[-2:]).clone()
        if real:                                        # Hermitian completion of the orders m >= 0
            mu = torch.arange(1, L, device=dev)
            x[:, :, L - 1] = x[:, :, L - 1].real.to(torch.complex128)
            x[:, :, L - 1 - mu] = x[:, :, L - 1 + mu].conj() * (1.0 - 2.0 * (mu % 2))
        F = _synth(x, theta, spin, w, real)
        if real:
            F[:, :L - 1] = F[:, L:].flip(1).conj()
        f = _phi_inverse(F, case)
        if case["sampling"] == "healpix":               # plain quadrature, no sampling theorem
            q = torch.tensor(_ring_weights(case), device=dev)
            y = _analyse(_phi_forward(f.real.to(torch.complex128) if real else f, case) * q, theta, spin, w, real)
            if real:
                y[:, :, L - 1 - mu] = y[:, :, L - 1 + mu].conj() * (1.0 - 2.0 * (mu % 2))
        else:
            y = x                                       # exact round trip
        return {"map": shaped((f.real if real else f).reshape((B,) + _map_shape(case))), "flm": shaped(y)}
    x, target = (v.reshape((B,) + v.shape[-(1 if case["sampling"] == "healpix" and v.shape[-1] == 12 * case["nside"] ** 2
                                            else 2):]) for v in xs)
    if op == "grad_inverse":
        r = _phi_inverse(_synth(x, theta, spin, w), case).reshape(target.shape) - target
        g = _analyse(_phi_forward(2 * r, case), theta, spin, w)
    else:
        q = torch.tensor(_ring_weights(case), device=dev)
        r = _analyse(_phi_forward(x, case) * q, theta, spin, w) - target
        g = _phi_inverse(_synth(2 * r, theta, spin, w) * q, case).reshape(x.shape)
    rr = torch.view_as_real(r.contiguous())
    return {"loss": (rr * rr).sum(), "grad": shaped(g)}
