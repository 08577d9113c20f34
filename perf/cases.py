"""The work that programs have this library do, as measurable cases.

listed() names the cases, draw() gives more of the same ranges, prepare() makes what a program has
in hand before the call (inputs on the GPU, the plan it keeps), run() is one pass through the public
entry points, work() the bytes and operations a pass cannot do without, exact() the same results in
64 bits from their definitions: the fitted taps and a plain (FFT) convolution, without the library.

Windows are given as multiples of sigma near the error-optimal ones, so that exact() needs no
window search.
"""
import math

import numpy as np
import torch

import paper_2110_11866_amd as M

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
# window half width over sigma near the smallest kernel error, by number of terms
MORLET_C = {3: 1.7, 4: 2.1, 5: 2.6, 6: 3.0, 7: 3.4, 8: 3.7}
GAUSS_C = {3: 2.7, 4: 3.3, 5: 3.7, 6: 4.1, 7: 4.4, 8: 4.7}


def listed():
    return [
        # one short signal, as a caller filters window by window: latency and launches are all
        {"name": "signal_1024", "kind": "morlet", "N": 1024, "sigma": 16.0, "K": 4, "L": 64, "mode": "sft", "dtype": "f32", "edge": False},
        # the method's headline point: one signal with a very wide wavelet, N = 102400, sigma = 8192
        {"name": "wide_102400", "kind": "morlet", "N": 102400, "sigma": 8192.0, "K": 6, "L": 32768, "mode": "asft", "dtype": "f32", "edge": False},
        # a long recording kept in bfloat16, plain SFT (float64 sums): the precision workload's size
        {"name": "bf16_4m", "kind": "morlet", "N": 1 << 22, "sigma": 1024.0, "K": 6, "L": 4096, "mode": "sft", "dtype": "bf16", "edge": False},
        # first differential of Gaussian smoothing of one very long signal
        {"name": "deriv_64m", "kind": "deriv", "N": 1 << 26, "sigma": 64.0, "K": 6, "L": 262, "mode": "asft", "dtype": "f32"},
        # one clip at many scales, half precision input: a scalogram asked for by itself
        {"name": "clip_scalogram", "kind": "scalogram", "B": 1, "S": 32, "lo": 30011, "hi": 30011, "s0": 4.0, "s1": 1024.0, "K": 5, "mode": "sft", "dtype": "f16"},
        # the benchmark's batch: 256 ragged signals, 32 scales (the largest forward)
        {"name": "ragged_scalogram", "kind": "scalogram", "B": 256, "S": 32, "lo": 4096, "hi": 262144, "s0": 4.0, "s1": 4096.0, "K": 5, "mode": "asft", "dtype": "f32"},
        # training step of the scalogram layer: forward, then gradients for the signals, widths and carriers
        {"name": "scalogram_train", "kind": "train", "B": 64, "S": 16, "lo": 32768, "hi": 32768, "s0": 8.0, "s1": 2048.0, "K": 5, "mode": "asft", "dtype": "f32"},
        # the one-signal layer with learnable width and carrier, forward and backward, an odd length
        {"name": "layer_train", "kind": "layer", "N": 131071, "sigma": 256.0, "K": 5, "L": 666, "mode": "sft", "dtype": "f32"},
        # separable Gaussian smoothing of a large image
        {"name": "image_4096", "kind": "gauss2d", "H": 4096, "W": 4096, "sigma_y": 8.0, "sigma_x": 8.0, "K": 4, "mode": "asft", "dtype": "f32", "backward": False},
        # Gabor features of a video frame with the gradient for the image
        {"name": "gabor_train_1080p", "kind": "gabor2d", "H": 1080, "W": 1920, "sigma_y": 8.0, "sigma_x": 8.0, "K": 5, "K_y": 4, "mode": "asft", "dtype": "f32", "backward": True},
        # the multiplication method on one long signal
        {"name": "multiply_4m", "kind": "multiply", "N": (1 << 22) + 3, "sigma": 64.0, "K": 3, "L": 173, "mode": "asft", "dtype": "f32", "backward": False},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every kind of call, over the sizes, widths, types and modes of the listed ones."""
    kind = rng.choice(["morlet", "morlet", "gauss", "deriv", "scalogram", "scalogram", "train", "layer", "gauss2d", "gabor2d", "multiply"])
    mode = rng.choice(["sft", "asft"])
    dtype = rng.choice(["f32", "f32", "f16", "bf16"])
    if kind in ("morlet", "gauss", "deriv", "multiply", "layer"):
        N = _logint(rng, 1024, {"morlet": 1 << 24, "gauss": 1 << 25, "deriv": 1 << 26, "multiply": 1 << 22, "layer": 1 << 20}[kind])
        sigma = round(math.exp(rng.uniform(math.log(8.0), math.log(max(16.0, min(8192.0, N / 12))))), 2)
        K = rng.choice([3, 4, 5, 6, 7, 8])
        L = int(math.ceil((GAUSS_C if kind in ("gauss", "deriv", "multiply") else MORLET_C)[K] * sigma))
        c = {"kind": kind, "N": N, "sigma": sigma, "K": K, "L": L, "mode": mode, "dtype": dtype}
        if kind in ("morlet", "gauss"):
            c["edge"] = rng.random() < 0.25
        if kind == "multiply":
            c["backward"] = rng.random() < 0.5
        return c
    if kind in ("scalogram", "train"):
        B, S = _logint(rng, 1, 128), rng.choice([8, 12, 16, 24, 32])
        lo = _logint(rng, 1024, 16384)
        hi = min(lo * rng.choice([1, 2, 8, 16]), 262144)
        if kind == "train":
            hi = min(hi, 32768)
        s0 = round(rng.uniform(3.0, 10.0), 3)
        s1 = round(s0 * math.exp(rng.uniform(math.log(8.0), math.log(max(16.0, hi / 64 / s0 * 4)))), 3)
        return {"kind": kind, "B": B if kind == "scalogram" else min(B, 64), "S": min(S, 16) if kind == "train" else S, "lo": lo, "hi": hi, "s0": s0, "s1": s1,
                "K": rng.choice([4, 5, 5, 6]), "mode": mode, "dtype": dtype}
    c = {"kind": kind, "H": _logint(rng, 128, 3072), "W": _logint(rng, 128, 3072), "sigma_y": round(rng.uniform(2.0, 24.0), 2), "sigma_x": round(rng.uniform(2.0, 24.0), 2),
         "K": rng.choice([3, 4, 5, 6]), "mode": mode, "dtype": dtype, "backward": rng.random() < 0.5}
    if kind == "gabor2d":
        c["K_y"] = rng.choice([3, 4, 5])
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _pow2(n):
    return 1 << max(1, (int(n) - 1).bit_length())


def _pink(gen, n):
    """n samples of 1/f noise of unit variance (shaped at a power-of-two length, then cropped)."""
    m = _pow2(max(n, 64))
    F = torch.fft.rfft(torch.randn(m, generator=gen, device=DEV))
    f = torch.arange(F.numel(), device=DEV, dtype=torch.float32)
    f[0] = 1.0
    F = F / f.sqrt()
    F[0] = 0
    x = torch.fft.irfft(F, m)[:n]
    return x / x.std().clamp_min(1e-6)


def _lengths(case):
    """The batch's signal lengths: log-uniform in [lo, hi], the same for every seed."""
    r = np.random.default_rng(3 + case["B"])
    return [int(v) for v in np.floor(np.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]), case["B"])) + 1e-9)] if case["hi"] > case["lo"] else [case["lo"]] * case["B"]


def _sigmas(case):
    S = case["S"]
    return [case["s0"] * (case["s1"] / case["s0"]) ** (s / max(S - 1, 1)) for s in range(S)]


def _input(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind in ("scalogram", "train"):
        x = torch.cat([_pink(gen, n) for n in _lengths(case)])
    elif kind in ("gauss2d", "gabor2d"):
        # an image: smooth shading, texture and sensor noise
        H, W = case["H"], case["W"]
        coarse = torch.randn(1, 1, H // 32 + 2, W // 32 + 2, generator=gen, device=DEV)
        x = torch.nn.functional.interpolate(coarse, size=(H, W), mode="bilinear", align_corners=False)[0, 0]
        x = x + 0.3 * torch.randn(H, W, generator=gen, device=DEV)
    elif case["dtype"] == "bf16" or kind == "layer":
        # a drifting baseline under noise (bounded, so that 16 bits hold it)
        x = torch.randn(case["N"], generator=gen, device=DEV)
        x = x + 0.5 * torch.cumsum(torch.randn(case["N"], generator=gen, device=DEV, dtype=torch.float64), 0).float() / math.sqrt(case["N"]) * 20.0
    else:
        # three tones under noise
        n = torch.arange(case["N"], device=DEV, dtype=torch.float64)
        f = torch.rand(3, generator=gen, device=DEV, dtype=torch.float64) * 0.199 + 0.001
        ph = torch.rand(3, generator=gen, device=DEV, dtype=torch.float64) * (2 * math.pi)
        x = sum(torch.sin(2 * math.pi * f[i] * n + ph[i]) for i in range(3)).float()
        x = x + 0.1 * torch.randn(case["N"], generator=gen, device=DEV)
    return x.to(DTYPES[case["dtype"]]).contiguous()


def _cotangent(case, seed):
    gen = _gen(seed + 7919)
    kind = case["kind"]
    n = sum(_lengths(case)) * case["S"] if kind == "train" else case["H"] * case["W"] if kind in ("gauss2d", "gabor2d") else case["N"]
    shape = (case["H"], case["W"]) if kind in ("gauss2d", "gabor2d") else (n,)
    dt = torch.float32 if kind == "gauss2d" else torch.complex64
    return torch.randn(shape, generator=gen, device=DEV, dtype=dt)


def _image_L(case):
    cy = GAUSS_C[case["K_y"] if case["kind"] == "gabor2d" else case["K"]]
    cx = (MORLET_C if case["kind"] == "gabor2d" else GAUSS_C)[case["K"]]
    ky = case["K_y"] if case["kind"] == "gabor2d" else case["K"]
    return max(ky, int(math.ceil(cy * case["sigma_y"]))), max(case["K"], int(math.ceil(cx * case["sigma_x"])))


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "x": _input(case, seed)}
    if kind in ("morlet", "layer"):
        cls = M.MorletPlan if kind == "morlet" else M.MorletTransform
        s["plan"] = cls(case["N"], case["sigma"], 6.0 / case["sigma"], case["K"], case["L"], mode=case["mode"])
    elif kind == "gauss":
        s["plan"] = M.GaussPlan(case["N"], case["sigma"], case["K"], case["L"], mode=case["mode"])
    elif kind == "deriv":
        s["plan"] = M.GaussDerivPlan(case["N"], case["sigma"], case["K"], case["L"], order=1, mode=case["mode"])
    elif kind == "multiply":
        s["plan"] = M.MultiplyPlan(case["N"], case["sigma"], 6.0 / case["sigma"], case["K"] - 1, case["L"], mode=case["mode"])
    elif kind in ("scalogram", "train"):
        sig = _sigmas(case)
        s["plan"] = M.ScalogramPlan(_lengths(case), sig, [6.0 / v for v in sig], case["K"], MORLET_C[case["K"]], mode=case["mode"])
    elif kind == "gauss2d":
        Ly, Lx = _image_L(case)
        s["plan"] = M.Gauss2DPlan(case["H"], case["W"], case["sigma_y"], case["sigma_x"], case["K"], Ly, Lx, mode=case["mode"])
    else:
        Ly, Lx = _image_L(case)
        s["plan"] = M.Gabor2DPlan(case["H"], case["W"], case["sigma_x"], 6.0 / case["sigma_x"], case["K"], case["sigma_y"], case["K_y"], Lx, Ly, mode=case["mode"])
    if case.get("edge"):
        s["plan"].set_boundary("edge")
    if kind in ("train", "layer") or case.get("backward"):
        s["g"] = _cotangent(case, seed)
    if kind == "layer":
        s["x"].requires_grad_(True)
    return s


def run(s):
    kind, plan, x = s["kind"], s["plan"], s["x"]
    if kind == "layer":
        # a training step's forward and backward through autograd, fresh gradients
        x.grad = None
        plan.zero_grad(set_to_none=True)
        W = plan(x)
        W.backward(s["g"])
        return {"W": W.detach(), "gx": x.grad, "gsigma": plan.sigma.grad, "gxi": plan.xi.grad}
    W = plan.forward(x)
    if "g" not in s:
        return {"W": W}
    if kind == "train":
        gx, gp = plan.backward(x, s["g"])
        return {"W": W, "gx": gx, "gp": gp}
    if kind == "multiply":
        return {"W": W, "gx": plan.backward(x, s["g"])[0]}
    return {"W": W, "gx": plan.backward(s["g"])}


def work(case):
    kind = case["kind"]
    e = 4 if case["dtype"] == "f32" else 2
    K = case["K"]
    if kind in ("scalogram", "train"):
        n = sum(_lengths(case))
        o = n * case["S"]
    else:
        n = case["H"] * case["W"] if kind in ("gauss2d", "gabor2d") else case["N"]
        o = n
    cplx = kind in ("morlet", "layer", "multiply", "scalogram", "train", "gabor2d")
    b = n * e + o * (8 if cplx else 4)
    # per output and term: one complex recurrence step (4 multiply-adds) and its weight in the result
    per = 8 * K + (4 if cplx else 2) * K
    f = o * per * (3 if kind == "multiply" else 2 if kind in ("gauss2d", "gabor2d") else 1)
    if kind in ("train", "layer"):
        b += o * 8 + n * e + n * 4          # the cotangent and the signal read once, dLoss/dx written
        f *= 4
    elif case.get("backward"):
        b += o * (4 if kind == "gauss2d" else 8) + n * 4
        f *= 2
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ results in 64 bits
def _round_half_up(v):
    return int(math.floor(v + 0.5))


def _n0(case_mode, sigma, L):
    return min(max(1, _round_half_up(sigma / 8.0)), L) if case_mode == "asft" else 0


def _basis(L, orders):
    k = np.arange(-L, L + 1)
    pk = np.mod(np.outer(k, np.asarray(orders, dtype=np.int64)), 2 * L).astype(np.float64)
    ang = math.pi * pk / L
    return np.cos(ang), np.sin(ang)


def _pinv(B):
    """Least-squares solver of the fits; columns that vanish on the grid get coefficient 0."""
    P = np.zeros((B.shape[1], B.shape[0]))
    keep = np.linalg.norm(B, axis=0) > 1e-9 * math.sqrt(B.shape[0])
    if keep.any():
        Bk = B[:, keep]
        P[keep] = np.linalg.solve(Bk.T @ Bk, Bk.T)
    return P


def _morlet(sigma, xi, k):
    """The dilated Morlet wavelet (real and imaginary part) of torch scalars sigma, xi."""
    x0 = xi * sigma
    C = (1 + torch.exp(-x0 * x0) - 2 * torch.exp(-0.75 * x0 * x0)) ** -0.5
    env = C / (math.pi ** 0.25 * torch.sqrt(sigma)) * torch.exp(-k * k / (2 * sigma * sigma))
    return env * (torch.cos(xi * k) - torch.exp(-0.5 * x0 * x0)), env * torch.sin(xi * k)


def _t(v):
    return torch.tensor(float(v), dtype=torch.float64)


def _lowest_order(sigma, xi, K, L):
    """The lowest Fourier order with the smallest fit error, ties to the smallest order."""
    k = torch.arange(-L, L + 1, dtype=torch.float64)
    re, im = (v.numpy() for v in _morlet(_t(sigma), _t(xi), k))
    hi = max(min(L - K + 1, int(math.ceil(xi * L / math.pi)) + K), 0)
    Bc, Bs = _basis(L, range(hi + K))
    best, at = math.inf, 0
    for ps in range(hi + 1):
        c, s = Bc[:, ps:ps + K], Bs[:, ps:ps + K]
        e = math.hypot(np.linalg.norm(c @ (_pinv(c) @ re) - re), np.linalg.norm(s @ (_pinv(s) @ im) - im))
        if e < best * (1 - 1e-12):
            best, at = e, ps
    return at


def _morlet_taps_fn(sigma0, xi0, K, L, mode):
    """taps(sigma, xi) -> (real, imaginary) of h[k], k = -L..L, with window, lowest order and shift frozen; and the shift."""
    ps = _lowest_order(sigma0, xi0, K, L)
    Bc, Bs = _basis(L, range(ps, ps + K))
    Pc, Ps, Bc, Bs = (torch.from_numpy(v) for v in (_pinv(Bc), _pinv(Bs), Bc, Bs))
    k = torch.arange(-L, L + 1, dtype=torch.float64)
    n0 = _n0(mode, sigma0, L)

    def taps(sigma, xi):
        re, im = _morlet(sigma, xi, k)
        re, im = Bc @ (Pc @ re), Bs @ (Ps @ im)
        if mode == "asft":
            a = torch.exp(-n0 ** 2 / (2 * sigma ** 2)) * torch.exp(-n0 / sigma ** 2 * k)
            c, s = torch.cos(xi * n0), torch.sin(xi * n0)
            re, im = a * (c * re - s * im), a * (s * re + c * im)
        return re, im

    return taps, n0


def _morlet_taps(sigma, xi, K, L, mode, params=False):
    """h (complex128 [2L+1]), [dh/dsigma, dh/dxi] if asked, the shift n0."""
    fn, n0 = _morlet_taps_fn(sigma, xi, K, L, mode)
    h = torch.complex(*fn(_t(sigma), _t(xi)))
    d = None
    if params:
        d = []
        for tan in ((1.0, 0.0), (0.0, 1.0)):
            _, dv = torch.func.jvp(fn, (_t(sigma), _t(xi)), (_t(tan[0]), _t(tan[1])))
            d.append(torch.complex(*dv).to(DEV))
    return h.to(DEV), d, n0


def _gauss_taps(sigma, K, L, mode, deriv=False):
    """Fitted Gaussian (or its first differential) as taps, and the shift n0."""
    k = np.arange(-L, L + 1, dtype=np.float64)
    g = 1.0 / (2 * sigma * sigma)
    G = math.sqrt(g / math.pi) * np.exp(-g * k * k)
    n0 = _n0(mode, sigma, L)
    alpha = n0 / sigma ** 2
    Bc, _ = _basis(L, range(K))
    fit = Bc @ (_pinv(Bc) @ G)
    if deriv:
        _, Bs = _basis(L, range(1, K + 1) if mode == "sft" else range(1, K))
        fit = Bs @ (_pinv(Bs) @ (-2 * g * k * G)) - alpha * fit * (mode == "asft")
    h = math.exp(-n0 ** 2 / (2 * sigma ** 2)) * np.exp(-alpha * k) * fit
    return torch.from_numpy(h).to(torch.complex128).to(DEV), n0


def _spectrum(h, L, n):
    nf = _pow2(n + 2 * h.shape[-1])
    return torch.fft.fft(h, nf), nf


def _conv(x, h, L, n0):
    """sum_k h[k] x[n - n0 - k] along the last axis, zero outside."""
    n = x.shape[-1]
    H, nf = _spectrum(h, L, n)
    y = torch.fft.ifft(torch.fft.fft(x.to(torch.complex128), nf) * H)
    return y[..., L - n0:L - n0 + n]


def _adj(g, h, L, n0):
    """sum_k conj(h[k]) g[j + n0 + k] along the last axis."""
    n = g.shape[-1]
    H, nf = _spectrum(h, L, n)
    y = torch.fft.ifft(torch.fft.fft(g.to(torch.complex128), nf) * H.conj())
    return torch.roll(y, L - n0, dims=-1)[..., :n]


def exact(case, seed):
    kind, mode, K = case["kind"], case["mode"], case["K"]
    x = _input(case, seed).double()
    if kind in ("scalogram", "train"):
        sig, lens, train = _sigmas(case), _lengths(case), kind == "train"
        Ls = [max(K, int(math.ceil(MORLET_C[K] * v))) for v in sig]
        T = [_morlet_taps(v, 6.0 / v, K, L, mode, train) for v, L in zip(sig, Ls)]
        W = torch.empty(sum(lens) * len(sig), dtype=torch.complex128, device=DEV)
        g = _cotangent(case, seed) if train else None
        gx, gp = torch.zeros_like(x), torch.zeros(len(sig), 2, dtype=torch.float64, device=DEV)
        spec, off = {}, 0
        for n in lens:
            nf = _pow2(n + 4 * max(Ls))
            if nf not in spec:
                spec[nf] = torch.stack([torch.fft.fft(torch.roll(torch.nn.functional.pad(h, (0, nf - h.numel())), n0 - L)) for (h, _, n0), L in zip(T, Ls)])
            X = torch.fft.fft(x[off:off + n].to(torch.complex128), nf)
            o = len(sig) * off
            W[o:o + len(sig) * n] = torch.fft.ifft(X * spec[nf])[:, :n].reshape(-1)
            if train:
                gb = g[o:o + len(sig) * n].view(len(sig), n).to(torch.complex128)
                gx[off:off + n] = torch.fft.ifft(torch.fft.fft(gb, nf) * spec[nf].conj())[:, :n].real.sum(0)
                for p in range(2):
                    if (nf, p) not in spec:
                        spec[nf, p] = torch.stack([torch.fft.fft(torch.roll(torch.nn.functional.pad(d[p], (0, nf - d[p].numel())), n0 - L)) for (_, d, n0), L in zip(T, Ls)])
                    dW = torch.fft.ifft(X * spec[nf, p])[:, :n]
                    gp[:, p] += (gb.conj() * dW).real.sum(1)
            off += n
        return {"W": W, "gx": gx, "gp": gp} if train else {"W": W}
    if kind in ("gauss2d", "gabor2d"):
        Ly, Lx = _image_L(case)
        hy, ny = _gauss_taps(case["sigma_y"], case["K_y"] if kind == "gabor2d" else K, Ly, mode)
        if kind == "gabor2d":
            hx, _, nx = _morlet_taps(case["sigma_x"], 6.0 / case["sigma_x"], K, Lx, mode)
        else:
            hx, nx = _gauss_taps(case["sigma_x"], K, Lx, mode)
        y = _conv(_conv(x, hx, Lx, nx).T.contiguous(), hy, Ly, ny).T
        out = {"W": y.contiguous() if kind == "gabor2d" else y.real.contiguous()}
        if case["backward"]:
            g = _cotangent(case, seed)
            g1 = _adj(g.T.contiguous(), hy, Ly, ny).T.contiguous()
            out["gx"] = _adj(g1, hx, Lx, nx).real.contiguous()
        return out
    L, sigma, N = case["L"], case["sigma"], case["N"]
    d = None
    if kind in ("morlet", "layer"):
        h, d, n0 = _morlet_taps(sigma, 6.0 / sigma, K, L, mode, kind == "layer")
    elif kind == "multiply":
        xi = 6.0 / sigma
        h, n0 = _gauss_taps(sigma, K, L, mode)
        k = torch.arange(-L, L + 1, dtype=torch.float64, device=DEV)
        x0 = xi * sigma
        C = (1 + math.exp(-x0 * x0) - 2 * math.exp(-0.75 * x0 * x0)) ** -0.5
        ce = C / (math.pi ** 0.25 * math.sqrt(sigma)) * math.sqrt(2 * math.pi) * sigma
        h = ce * (torch.exp(1j * xi * (k + n0)) - math.exp(-0.5 * x0 * x0)) * h
    else:
        h, n0 = _gauss_taps(sigma, K, L, mode, kind == "deriv")
    if case.get("edge"):
        xe = torch.cat([x[:1].expand(2 * L), x, x[-1:].expand(2 * L)])
        W = _conv(xe, h, L, n0)[2 * L:2 * L + N]
    else:
        W = _conv(x, h, L, n0)
    out = {"W": (W if kind in ("morlet", "layer", "multiply") else W.real).contiguous()}
    if kind == "layer" or case.get("backward"):
        g = _cotangent(case, seed).to(torch.complex128)
        out["gx"] = _adj(g, h, L, n0).real.contiguous()
        if kind == "layer":
            gp = [float((g.conj() * _conv(x, v, L, n0)).real.sum()) for v in d]
            out["gsigma"], out["gxi"] = (torch.tensor(v, dtype=torch.float64) for v in gp)
    return out
