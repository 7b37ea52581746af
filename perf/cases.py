"""Timed cases: the calls a restoration program makes of this library.

A program cuts its frames into patches (prepare_data), predicts starting
coefficients with the warm-start network, evaluates the loss and its gradient
many times, alone, inside the solver's rounds or for a group of uneven
fields, and restores the objects at the end; the network is trained on bursts
made by the library's forward model.  Each case is one such call, at sizes
from one patch to one GPU's share of the largest field.

Inputs come from the seed alone and from plain torch: random-phase objects of
a k^-3 spectrum with 10% contrast, turbulent wavefronts, 1% noise, binary
disc pupils of 0.45 N pixels and Zernike modes.
"""

import functools
import math

import numpy as np
import torch

from paper_2505_10639_amd import (Plan, Solver, WarmStartNet, _lib, filter_spec, momfbd_loss,
                                  momfbd_power_spectrum)
from paper_2505_10639_amd.batch import Field, FieldGroup

DEV = "cuda:0"
GAMMA = 1e-3
NOISE = 0.01
F64 = torch.float64

# Channel layouts: per channel its object, its defocus diversity in waves peak
# to valley, and lambda_0 / lambda.
CHANNELS = {
    "one": ((0, 0.0, 1.0),),                                     # one wideband channel
    "diversity": ((0, 0.0, 1.0), (0, 1.0, 1.0)),                 # phase-diversity pair, one object
    "two": ((0, 0.0, 1.0), (1, 1.0, 1.0)),                       # two objects, the second defocused
    "three": ((0, 0.0, 1.0), (0, 1.0, 1.0), (1, 0.0, 1.0 / 1.05)),
    "four": ((0, 0.0, 1.0), (1, 0.0, 1.0 / 0.95), (2, 0.0, 1.0 / 1.05), (3, 0.0, 1.0 / 1.1)),
}


def listed():
    return [
        # The smallest call: an interactive look at one patch (8 frames, 44 modes); launches and
        # latency count.
        dict(name="eval_one_patch_64", kind="eval", N=64, P=1, J=8, M=44, channels="one",
             option="plain"),
        # The headline: every 64 x 64 patch of a 1024 x 1024 field at stride 32.
        dict(name="eval_field_64", kind="eval", N=64, P=961, J=12, M=66, channels="two",
             option="plain"),
        # A 512 x 512 field at N = 96 through the autograd wrapper, with frame weights and a
        # per-frequency Wiener constant; odd numbers of frames and modes.
        dict(name="backward_ragged_96", kind="eval", N=96, P=81, J=13, M=55, channels="three",
             option="autograd"),
        # One GPU's share (of eight) of a 2048 x 2048 field in four wavelengths, 150 modes, with
        # the smoothness prior's table.
        dict(name="eval_share_128", kind="eval", N=128, P=128, J=24, M=150, channels="four",
             option="table"),
        # The solver on a 512 x 512 field: start, then four rounds (one line-search trial each).
        dict(name="solve_field_64", kind="solve", N=64, P=225, J=12, M=44, channels="one",
             rounds=4),
        # An observing run's uneven fields in one launch per stage.
        dict(name="eval_group_64", kind="group", N=64, fields=6, P=225, J=24, M=88),
        # The end of a restoration: filtered objects, mosaic, power spectrum of the field.
        dict(name="restore_field_64", kind="restore", N=64, side=31, J=12, M=66, channels="two"),
        # Restored objects of a 512 x 512 field at N = 128, a few odd frames.
        dict(name="estimate_field_128", kind="estimate", N=128, P=49, J=9, M=77, channels="three"),
        # Cutting, apodizing and transforming the frames of the headline's field.
        dict(name="prepare_field_64", kind="prepare", N=64, side=31, J=12, channels="two"),
        # Starting coefficients of a whole field from the warm-start network.
        dict(name="predict_field_64", kind="predict", N=64, B=961, J=12, M=44),
        # Loss and parameter gradients of one training batch of the network.
        dict(name="train_batch_64", kind="train", N=64, B=256, J=12, M=44),
        # One training batch of bursts through the forward model, with its noise.
        dict(name="bursts_64", kind="bursts", N=64, B=256, J=12, M=44),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the listed ranges; its pixels never exceed the largest listed case's."""
    kind = rng.choice(["eval", "eval", "eval", "solve", "group", "restore", "estimate", "prepare",
                       "predict", "train", "bursts"])
    N = rng.choice([64, 64, 96, 128])
    J, M = rng.randint(1, 24), rng.randint(9, 150)
    channels = rng.choice(sorted(CHANNELS))
    C = len(CHANNELS[channels])
    most = max(1, 150_000_000 // (C * J * N * N))       # patches
    if kind == "eval":
        return dict(kind=kind, N=N, P=_log_int(rng, 1, min(961, most)), J=J, M=M,
                    channels=channels, option=rng.choice(["plain", "plain", "autograd", "table"]))
    if kind == "solve":
        return dict(kind=kind, N=N, P=_log_int(rng, 1, min(225, max(1, most // 8))), J=J,
                    M=min(M, 88), channels=channels, rounds=rng.randint(1, 4))
    if kind == "group":
        return dict(kind=kind, N=N, fields=rng.randint(2, 6), P=_log_int(rng, 4, 225 * 4096 // (N * N)),
                    J=rng.randint(6, 24), M=rng.randint(44, 88))
    if kind == "restore":
        return dict(kind=kind, N=N, side=rng.choice([3, 7, 15]) if N < 128 else rng.choice([3, 7]),
                    J=min(J, 12), M=min(M, 88), channels=channels)
    if kind == "estimate":
        return dict(kind=kind, N=N, P=_log_int(rng, 1, min(225, most)), J=J, M=M, channels=channels)
    if kind == "prepare":
        return dict(kind=kind, N=N, side=rng.randint(1, max(1, min(31, int(math.sqrt(most))))), J=J,
                    channels=channels)
    B = _log_int(rng, 1, {64: 961, 96: 256, 128: 128}[N] if kind == "predict"
                 else {64: 256, 96: 96, 128: 64}[N])
    return dict(kind=kind, N=N, B=B, J=min(J, 16), M=min(max(M, 9), 66))


# ---- inputs -------------------------------------------------------------------------------------


def _noll(j):
    n = 0
    while (n + 1) * (n + 2) // 2 < j:
        n += 1
    r = j - n * (n + 1) // 2 - 1
    m = n % 2 + 2 * ((r + (n + 1) % 2) // 2)
    return n, m if j % 2 == 0 else -m


@functools.lru_cache(maxsize=64)
def _optics(N, M, lam):
    """Pupil [N][N] and Zernike modes [M][N][N] (radians, Noll 2..M+1) of a channel, float32."""
    radius = 0.5 * 0.45 * lam * N
    v = (np.arange(N) - N // 2) / radius
    y, x = np.meshgrid(v, v, indexing="ij")
    rho, theta = np.hypot(x, y), np.arctan2(y, x)
    inside = rho <= 1.0
    r = rho[inside]
    modes = np.zeros((M, N, N), np.float32)
    for i in range(M):
        n, m = _noll(i + 2)
        k = abs(m)
        radial = sum((-1) ** s * math.factorial(n - s) / (math.factorial(s) * math.factorial((n + k) // 2 - s)
                     * math.factorial((n - k) // 2 - s)) * r ** (n - 2 * s) for s in range((n - k) // 2 + 1))
        az = 1.0 if m == 0 else math.sqrt(2) * (np.cos(k * theta[inside]) if m > 0 else np.sin(k * theta[inside]))
        modes[i][inside] = lam * math.sqrt(n + 1) * radial * az
    return inside.astype(np.float32), modes


def _defocus(N, waves, lam):
    v = (np.arange(N) - N // 2) / (0.5 * 0.45 * lam * N)
    rho2 = v[:, None] ** 2 + v[None, :] ** 2
    return np.where(rho2 <= 1.0, lam * waves * math.pi * (2.0 * rho2 - 1.0), 0.0).astype(np.float32)


def _system(N, M, channels):
    """channel_object, pupil [C][N][N], basis [C][M][N][N], diversity [C][N][N]."""
    spec = CHANNELS[channels]
    pairs = [_optics(N, M, lam) for _, _, lam in spec]
    return ([k for k, _, _ in spec], np.stack([p for p, _ in pairs]), np.stack([b for _, b in pairs]),
            np.stack([_defocus(N, w, lam) for _, w, lam in spec]))


def _window(N, border):
    e = np.minimum(np.arange(N), N - 1 - np.arange(N))
    w = np.where(e < border, 0.5 * (1.0 - np.cos(np.pi * (e + 0.5) / border)), 1.0)
    return torch.from_numpy((w[:, None] * w[None, :]).astype(np.float32)).to(DEV)


def _mode_std(M):
    """Standard deviation of each mode at D/r0 = 1 (Noll's residuals), modes 2..10 corrected."""
    j = np.arange(1, M + 2, dtype=np.float64)
    res = 0.2944 * j ** (-math.sqrt(3) / 2)
    res[:3] = [1.0299, 0.582, 0.134]
    res = res[:M + 1]
    std = np.sqrt(np.maximum(res[:-1] - res[1:], 1e-6))
    std[:9] *= 0.3
    return std.astype(np.float32)


def _alpha(gen, P, J, M):
    """Turbulent coefficients [P][J][M], D/r0 from 5 to 20 over the patches."""
    r0 = torch.linspace(5.0, 20.0, P, device=DEV) ** (5.0 / 6.0)
    std = torch.from_numpy(_mode_std(M)).to(DEV)
    return (torch.randn((P, J, M), generator=gen, device=DEV) * std * r0[:, None, None]).contiguous()


def _scenes(gen, n, H):
    """n scenes [H][H] of a k^-3 power spectrum, mean 1, 10% contrast."""
    f = torch.fft.fftfreq(H, device=DEV)
    k = torch.hypot(f[:, None], f[None, :])
    amp = torch.where(k > 0, k.clamp_min(1e-9) ** -1.5, torch.zeros_like(k))
    x = torch.fft.ifft2(torch.fft.fft2(torch.randn((n, H, H), generator=gen, device=DEV)) * amp).real
    x = x - x.mean(dim=(1, 2), keepdim=True)
    return (1.0 + 0.1 * x / x.std(dim=(1, 2), keepdim=True)).clamp_min(0.0)


def _otf(alpha, pupil, basis, diversity):
    """PSF spectra (half) [P][J][N][N/2+1] of one channel, in alpha's precision."""
    N = pupil.shape[-1]
    phi = (alpha.reshape(-1, alpha.shape[-1]) @ basis.reshape(basis.shape[0], -1)).reshape(alpha.shape[:2] + (N, N))
    phi = phi + diversity
    p = torch.fft.ifft2(torch.complex(pupil * torch.cos(phi), pupil * torch.sin(phi)), norm="forward")
    s = (p.real ** 2 + p.imag ** 2) / (N * N * (pupil * pupil).sum())
    return torch.fft.rfft2(s), s


def _on_gpu(system, dtype=torch.float32):
    return [torch.from_numpy(a).to(DEV, dtype) for a in system[1:]]


def _spectra(gen, system, alpha, objects):
    """Data spectra D [P][C][J][N][N/2+1] of the objects [P][K][N][N] seen through alpha."""
    pupil, basis, div = _on_gpu(system)
    P, J, _ = alpha.shape
    C, N = pupil.shape[0], pupil.shape[-1]
    D = torch.empty((P, C, J, N, N // 2 + 1), dtype=torch.complex64, device=DEV)
    O = torch.fft.rfft2(objects)
    step = max(1, 40_000_000 // (J * N * N))
    for c, k in enumerate(system[0]):
        for a in range(0, P, step):
            S, _ = _otf(alpha[a:a + step], pupil[c], basis[c], div[c])
            n = torch.randn(S.shape[:2] + (N, N), generator=gen, device=DEV)
            D[a:a + step, c] = O[a:a + step, k, None] * S + torch.fft.rfft2(NOISE * n)
    return D


def _patches(scenes, side, stride, N):
    """[side^2][K][N][N] cut from scenes [K][H][H]."""
    x = scenes.unfold(1, N, stride).unfold(2, N, stride)[:, :side, :side]
    return x.permute(1, 2, 0, 3, 4).reshape(side * side, -1, N, N)


def _apodized(x, window):
    m = x.mean(dim=(-2, -1), keepdim=True)
    return window * (x - m) + m


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _problem(case, seed):
    """Host optics, and on the GPU the point alpha, spectra D, gamma and weights of an evaluation."""
    N, J, M = case["N"], case["J"], case["M"]
    gen = _gen(seed)
    system = _system(N, M, case["channels"])
    K = max(system[0]) + 1
    if "side" in case:
        stride = N // 2
        scenes = _scenes(gen, K, _mosaic_side(case))
        objects = _patches(scenes, case["side"], stride, N)
    else:
        objects = _scenes(gen, case["P"] * K, N).reshape(case["P"], K, N, N)
    objects = _apodized(objects, _window(N, 6 * N // 64))
    P = objects.shape[0]
    true = _alpha(gen, P, J, M)
    D = _spectra(gen, system, true, objects)
    alpha = (true + 0.1 * torch.randn(true.shape, generator=gen, device=DEV)).contiguous()
    gamma, weights = GAMMA, None
    if case.get("option") in ("autograd", "table"):
        u = torch.arange(N, device=DEV, dtype=F64)
        lap = 4.0 * torch.sin(math.pi * u / N) ** 2
        table = GAMMA + 0.01 * (lap[:, None] + lap[None, :N // 2 + 1])
        gamma = table.to(torch.float32).expand(K, N, N // 2 + 1).contiguous()
    if case.get("option") == "autograd":
        weights = (0.5 + torch.rand((len(system[0]), J), generator=gen, device=DEV)).contiguous()
    return system, alpha, D, gamma, weights


def _group_fields(case):
    """Sizes of the fields of a group: frames, modes and objects differ from field to field."""
    out = []
    for i in range(case["fields"]):
        out.append(dict(N=case["N"], P=max(1, case["P"] // (1 + i % 3)), J=max(1, case["J"] * (2 + i % 3) // 4 - i % 2),
                        M=max(9, case["M"] - 11 * (i % 4)), channels=("one", "two", "three")[i % 3]))
    return out


def _cnn_params(gen, N, J, M):
    """He-normal weights, small biases: layer by layer [out][...in], then the biases."""
    side = N // 16
    layers = [(J, 32, 9), (32, 64, 9), (64, 128, 9), (128, 128, 9), (128 * side * side, 512, 1), (512, J * M, 1)]
    parts = []
    for i, (a, b, taps) in enumerate(layers):
        gain = 0.1 if i == 5 else 1.0
        parts.append(gain * math.sqrt(2.0 / (a * taps)) * torch.randn(a * b * taps, generator=gen, device=DEV))
        parts.append(0.01 * torch.randn(b, generator=gen, device=DEV))
    return torch.cat(parts), layers


def _bursts(gen, N, B, J, M):
    """Spectra D [B][1][J][N][N/2+1] and coefficients of simulated bursts."""
    system = _system(N, M, "one")
    objects = _apodized(_scenes(gen, B, N), _window(N, 6 * N // 64)).reshape(B, 1, N, N)
    alpha = _alpha(gen, B, J, M)
    return system, _spectra(gen, system, alpha, objects), alpha


def _mosaic_side(case):
    return (case["side"] - 1) * (case["N"] // 2) + case["N"]


def _spectrum_side(case):
    return 1 << (_mosaic_side(case).bit_length() - 1)       # the largest power of two that fits


def _noise_seed(seed):
    return (int(seed) * 2654435761 + 12345) & 0xFFFFFFFF


def prepare(case, seed):
    kind, N = case["kind"], case["N"]
    if kind in ("eval", "solve", "estimate", "restore"):
        system, alpha, D, gamma, weights = _problem(case, seed)
        plan = Plan(N, alpha.shape[0], case["J"], *system, DEV)
        s = dict(case=case, plan=plan, alpha=alpha, D=D, gamma=gamma, weights=weights)
        if kind == "restore":
            K, eta = max(system[0]) + 1, NOISE ** 2 * N * N
            s["filters"] = [filter_spec("scharmer", noise_power=eta)]
            s["filters"] += [filter_spec("tophat", 0.55, 0.7, 0.45 * N)] * (K - 1)
            L = _spectrum_side(case)
            s["window"] = _window(L, L // 16)
        if kind == "solve":
            s["accepted"] = torch.empty_like(alpha)
        return s
    if kind == "group":
        fields = []
        for i, f in enumerate(_group_fields(case)):
            system, alpha, D, gamma, _ = _problem(f, seed * 16 + i)
            fields.append(Field(N, f["P"], f["J"], *system, D, gamma, alpha0=alpha, device=DEV))
        return dict(case=case, fields=fields, group=FieldGroup(fields))
    if kind == "prepare":
        gen = _gen(seed)
        H, J = _mosaic_side(case), case["J"]
        C = len(CHANNELS[case["channels"]])
        scenes = _scenes(gen, C, H)
        frames = scenes[:, None] + NOISE * torch.randn((C, J, H, H), generator=gen, device=DEV)
        plan = Plan(N, case["side"] ** 2, J, *_system(N, 1, case["channels"]), DEV)
        return dict(case=case, plan=plan, frames=frames.contiguous(), window=_window(N, 6 * N // 64))
    J, M, B = case["J"], case["M"], case["B"]
    gen = _gen(seed)
    if kind == "bursts":
        system = _system(N, M, "one")
        objects = _scenes(gen, B, N)
        return dict(case=case, plan=Plan(N, B, J, *system, DEV), seed=_noise_seed(seed),
                    alpha=_alpha(gen, B, J, M), O=torch.fft.rfft2(objects).reshape(B, 1, N, N // 2 + 1).contiguous(),
                    sigma=(1.0 / (50.0 + 150.0 * torch.rand(B, generator=gen, device=DEV))).contiguous(),
                    window=_window(N, 6 * N // 64), noise=torch.empty((B, 1, J, N, N), device=DEV))
    params, _ = _cnn_params(gen, N, J, M)
    _, D, alpha = _bursts(gen, N, B, J, M)
    net = WarmStartNet(J, M, _mode_std(M) * 10.0, batch_max=min(B, 256), device=DEV, N=N)
    net.load(params)
    return dict(case=case, net=net, D=D, target=alpha)


# ---- the passes ---------------------------------------------------------------------------------


def run(state):
    kind = state["case"]["kind"]
    if kind == "eval":
        plan, D, gamma, weights = state["plan"], state["D"], state["gamma"], state["weights"]
        if state["case"]["option"] == "autograd":
            alpha = state["alpha"].detach().requires_grad_(True)
            loss = momfbd_loss(alpha, plan, D, gamma, weights)
            loss.backward()
            return {"loss": loss.detach(), "grad": alpha.grad}
        loss, grad = plan.loss_grad(state["alpha"], D, gamma, weights)
        return {"loss": loss, "grad": grad}
    if kind == "solve":
        # each solve starts from the same point; its result is the accepted coefficients
        solver = Solver(state["plan"], state["alpha"].clone(), state["D"], state["gamma"])
        _, status = solver.rounds(state["case"]["rounds"], state["accepted"])
        return {"alpha": state["accepted"], "status": status}
    if kind == "group":
        state["group"].loss_grad()
        return [(f.loss_eval, f.grad_eval) for f in state["fields"]]
    if kind == "restore":
        case, plan = state["case"], state["plan"]
        obj = plan.object_filtered(state["alpha"], state["D"], state["filters"], state["gamma"])
        side, L = case["side"], _spectrum_side(case)
        mosaic = plan.mosaic(obj, side, side, case["N"] // 2, case["N"] // 8)
        power, sector, counts = momfbd_power_spectrum(mosaic[0, :L, :L].contiguous(), state["window"])
        return {"objects": obj, "mosaic": mosaic, "power": power, "sector": sector, "counts": counts}
    if kind == "estimate":
        return state["plan"].object_estimate(state["alpha"], state["D"], state["gamma"])
    if kind == "prepare":
        return state["plan"].prepare_data(state["frames"], state["case"]["N"] // 2, state["window"])
    if kind == "predict":
        return state["net"].predict(state["D"])
    if kind == "train":
        loss, grad = state["net"].loss_grad(state["D"], state["target"])
        return {"loss": loss, "grad": grad}
    _lib.momfbd_random_normal(state["seed"], 0x2050, 0, state["noise"])
    frames, D = state["plan"].synthesize(state["alpha"], state["O"], state["noise"], state["sigma"],
                                         state["window"])
    return {"noise": state["noise"], "frames": frames, "D": D}


# ---- what a pass cannot do without --------------------------------------------------------------


def _eval_work(P, C, K, J, M, N, grad):
    """Bytes and operations of an evaluation: D and alpha read, loss and gradient (or objects)
    written; the two complex and two real 2-D transforms of a unit (one and one for the objects)
    and the two modal products on the pupil's pixels."""
    units, fft = P * C * J, 5 * N * N * math.log2(N * N)
    modal = 2 * M * 0.159 * N * N
    bytes_ = units * N * (N // 2 + 1) * 8 + P * J * M * 4 * (2 if grad else 1)
    return {"bytes": bytes_ + (8 * P if grad else 4 * P * K * N * N),
            "flops": units * ((3.0 * fft + 2 * modal) if grad else (1.5 * fft + modal))}


def _cnn_flops(N, J, M):
    h, total = N, 0
    for a, b in ((J, 32), (32, 64), (64, 128), (128, 128)):
        h //= 2
        total += h * h * a * b * 9
    return 2.0 * (total + 128 * h * h * 512 + 512 * J * M)


def work(case):
    kind, N = case["kind"], case["N"]
    fft = 5 * N * N * math.log2(N * N)
    if kind == "group":
        parts = [work(dict(f, kind="eval")) for f in _group_fields(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    J = case["J"]
    spectrum = N * (N // 2 + 1) * 8
    if kind in ("eval", "solve", "estimate", "restore", "prepare"):
        C = len(CHANNELS[case["channels"]])
        K = max(c[0] for c in CHANNELS[case["channels"]]) + 1
        P = case["side"] ** 2 if "side" in case else case["P"]
        if kind == "prepare":
            return {"bytes": C * J * _mosaic_side(case) ** 2 * 4 + P * C * J * spectrum,
                    "flops": P * C * J * 0.5 * fft}
        w = _eval_work(P, C, K, J, case["M"], N, kind in ("eval", "solve"))
        if kind == "solve":         # the start and each round evaluate every patch
            return {k: v * (1 + case["rounds"]) for k, v in w.items()}
        if kind == "restore":       # the mosaic, and the spectrum of the first object's field
            L, H = _spectrum_side(case), _mosaic_side(case)
            return {"bytes": w["bytes"] + 4 * K * H * H + 4 * L * L,
                    "flops": w["flops"] + 2.5 * L * L * math.log2(L * L)}
        return w
    M, B = case["M"], case["B"]
    if kind == "bursts":
        return {"bytes": B * (J * M * 4 + spectrum + J * (2 * N * N * 4 + spectrum)),
                "flops": B * J * (2.5 * fft + 2 * M * 0.159 * N * N + 40 * N * N)}
    params = _cnn_params_count(N, J, M) * 4
    times = 3 if kind == "train" else 1
    return {"bytes": B * J * (spectrum + 4 * M) + params * (2 if kind == "train" else 1),
            "flops": B * (_cnn_flops(N, J, M) * times + J * 0.5 * fft)}


def _cnn_params_count(N, J, M):
    side = N // 16
    layers = [(J * 9, 32), (32 * 9, 64), (64 * 9, 128), (128 * 9, 128), (128 * side * side, 512), (512, J * M)]
    return sum(a * b + b for a, b in layers)


# ---- the same in 64 bits ------------------------------------------------------------------------


def _column_weight(N):
    w = torch.full((N // 2 + 1,), 2.0, dtype=F64, device=DEV)
    w[0] = w[-1] = 1.0
    return w


def _sums64(alpha, D, tables, chan_object, gamma, weights, K):
    """Per object N_k, Q_k (with gamma), E_k = sum w|D|^2 and sum w|S|^2, of a few patches."""
    pupil, basis, div = tables
    num, den, pow_ = [0.0] * K, [0.0] * K, [0.0] * K
    for c, k in enumerate(chan_object):
        S, _ = _otf(alpha, pupil[c], basis[c], div[c])
        d = D[:, c].to(torch.complex128)
        w = torch.ones(D.shape[2], dtype=F64, device=DEV) if weights is None else weights[c].to(F64)
        w = w[None, :, None, None]
        num[k] = num[k] + (w * d * S.conj()).sum(1)
        den[k] = den[k] + (w * (S.real ** 2 + S.imag ** 2)).sum(1)
        pow_[k] = pow_[k] + (w * (d.real ** 2 + d.imag ** 2)).sum(1)
    g = [gamma if isinstance(gamma, float) else gamma[k].to(F64) for k in range(K)]
    return num, [den[k] + g[k] for k in range(K)], pow_, den


def _chunks(P, C, J, N):
    step = max(1, 24_000_000 // (C * J * N * N))
    return [(a, min(P, a + step)) for a in range(0, P, step)]


def _eval64(system, alpha, D, gamma, weights):
    tables, chan_object = _on_gpu(system, F64), system[0]
    K, N = max(chan_object) + 1, D.shape[-2]
    losses, grads = [], []
    for a, b in _chunks(*D.shape[:3], N):
        x = alpha[a:b].to(F64).requires_grad_(True)
        num, den, pow_, _ = _sums64(x, D[a:b], tables, chan_object, gamma, weights, K)
        terms = sum(pow_[k] - (num[k].real ** 2 + num[k].imag ** 2) / den[k] for k in range(K))
        loss = (terms * _column_weight(N)).sum(dim=(1, 2))
        loss.sum().backward()
        losses.append(loss.detach())
        grads.append(x.grad)
    return torch.cat(losses), torch.cat(grads)


def _lowpass(H):
    """Clipping, 3 x 3 median and the island of the zero frequency, on the full grids H [P][N][N]."""
    H = torch.where(H < 0.2, torch.zeros_like(H), H.clamp_max(1.0))
    H = torch.stack([torch.roll(H, (dy, dx), (1, 2)) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]).median(0).values
    keep = torch.zeros_like(H, dtype=torch.bool)
    keep[:, 0, 0] = H[:, 0, 0] > 0
    while True:
        grown = keep.clone()
        for s, d in ((1, 1), (-1, 1), (1, 2), (-1, 2)):
            grown |= torch.roll(keep, s, d)
        grown &= H > 0
        if bool((grown == keep).all()):
            return torch.where(keep, H, torch.zeros_like(H))
        keep = grown


def _objects64(system, alpha, D, gamma, filtered):
    tables, chan_object = _on_gpu(system, F64), system[0]
    K, N = max(chan_object) + 1, D.shape[-2]
    u = torch.fft.fftfreq(N, 1.0 / N, device=DEV, dtype=F64)
    f = torch.hypot(u[:, None], u[None, :]) / (0.45 * N)
    tophat = (0.5 * (1.0 + torch.cos(math.pi * ((f - 0.55) / 0.15).clamp(0.0, 1.0))))[:, :N // 2 + 1]
    mirror = (-torch.arange(N, device=DEV)) % N
    out = []
    for a, b in _chunks(*D.shape[:3], N):
        num, den, _, pow_s = _sums64(alpha[a:b].to(F64), D[a:b], tables, chan_object, gamma, None, K)
        objs = []
        for k in range(K):
            O = num[k] / den[k]
            if filtered and k == 0:
                mag = num[k].real ** 2 + num[k].imag ** 2
                H = torch.where(mag > 0, 1.0 - NOISE ** 2 * N * N * pow_s[k] / mag.clamp_min(1e-300),
                                torch.zeros_like(mag))
                full = torch.cat([H, H[:, mirror][:, :, 1:N // 2].flip(2)], dim=2)
                O = O * _lowpass(full)[:, :, :N // 2 + 1]
            elif filtered:
                O = O * tophat
            objs.append(torch.fft.irfft2(O, s=(N, N)))
        out.append(torch.stack(objs, 1))
    return torch.cat(out)


def _mosaic64(obj, side, stride, border):
    N, H = obj.shape[-1], (side - 1) * stride + obj.shape[-1]
    e = torch.minimum(torch.arange(N), N - 1 - torch.arange(N)).to(DEV, F64)
    w = torch.where(e < border, 0.5 * (1.0 - torch.cos(math.pi * (e + 0.5) / border)), torch.ones_like(e))
    w = w[:, None] * w[None, :]
    acc, tot = torch.zeros((obj.shape[1], H, H), dtype=F64, device=DEV), torch.zeros((H, H), dtype=F64, device=DEV)
    for i in range(side):
        for k in range(side):
            y, x = i * stride, k * stride
            acc[:, y:y + N, x:x + N] += w * obj[i * side + k]
            tot[y:y + N, x:x + N] += w
    return acc / tot


def _spectrum64(image, window):
    L = image.shape[0]
    X = torch.fft.fft2(window.to(F64) * (image - image.mean()))
    power = X.real ** 2 + X.imag ** 2
    u = torch.fft.fftfreq(L, 1.0 / L, device=DEV, dtype=F64).round()
    u = torch.where(u == -(L // 2), -u, u)
    uy, ux = u[:, None].expand(L, L), u[None, :].expand(L, L)
    r = torch.floor(torch.sqrt(ux ** 2 + uy ** 2) + 0.5).long()
    sector = (ux != 0) & (uy != 0) & (ux ** 2 <= 3 * uy ** 2) & (uy ** 2 <= 3 * ux ** 2) & (r <= L // 2)
    counts = torch.bincount(r[sector], minlength=L // 2 + 1)
    sums = torch.bincount(r[sector], weights=power[sector], minlength=L // 2 + 1)
    return power, sums / counts.clamp_min(1)


def _cnn64(D, params, layers, N, J, M):
    frames = torch.fft.irfft2(D[:, 0].to(torch.complex128), s=(N, N))
    h = 10.0 * (frames / frames.mean(dim=(2, 3), keepdim=True) - 1.0)
    o, side = 0, N
    for i, (a, b, taps) in enumerate(layers):
        w = params[o:o + a * b * taps]
        bias = params[o + a * b * taps:o + a * b * taps + b]
        o += a * b * taps + b
        if taps == 9:
            cols = torch.nn.functional.unfold(h, 3, padding=1, stride=2)        # [B][a*9][pixels]
            wt = w.reshape(b, 3, 3, a).permute(0, 3, 1, 2).reshape(b, a * 9)
            side //= 2
            h = (wt @ cols + bias[:, None]).reshape(D.shape[0], b, side, side)
        else:
            if i == 4:
                h = h.permute(0, 2, 3, 1).reshape(D.shape[0], a)                # (y, x, channel)
            h = h @ w.reshape(b, a).T + bias
        if i < 5:
            h = torch.relu(h)
    return h.reshape(D.shape[0], J, M)


def _burst_loss64(z, target, scale):
    """Tilt means removed, the better of the two signs of the even modes, variance weights."""
    M = z.shape[-1]
    weight = scale ** 2 / (scale ** 2).mean()
    sign = torch.tensor([-1.0 if _noll(i + 2)[0] % 2 == 0 else 1.0 for i in range(M)], dtype=F64, device=DEV)
    tilt = torch.zeros(M, dtype=F64, device=DEV)
    tilt[:2] = 1.0
    p = z - tilt * z.mean(dim=1, keepdim=True)
    q = target.to(F64) / scale
    q = q - tilt * q.mean(dim=1, keepdim=True)
    return torch.minimum((weight * (p - q) ** 2).sum(2), (weight * (p - sign * q) ** 2).sum(2)).mean()


def _normals64(seed, stream, n):
    """Philox4x32-10 counters 0.. with key `seed`, and Box-Muller pairs."""
    lo = np.uint64(0xFFFFFFFF)
    b = np.arange((n + 3) // 4, dtype=np.uint64)
    c = [b & lo, b >> np.uint64(32), np.full_like(b, stream & 0xFFFFFFFF), np.full_like(b, stream >> 32)]
    k = [seed & 0xFFFFFFFF, seed >> 32]
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k[0]), p1 & lo, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k[1]), p0 & lo]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    u = [((w >> np.uint64(8)).astype(np.float64) + 0.5) * 2.0 ** -24 for w in c]
    z = np.empty((b.size, 4))
    for i in (0, 2):
        r = np.sqrt(-2.0 * np.log(u[i]))
        z[:, i], z[:, i + 1] = r * np.cos(2 * math.pi * u[i + 1]), r * np.sin(2 * math.pi * u[i + 1])
    return torch.from_numpy(z.reshape(-1)[:n])


def exact(case, seed):
    kind, N = case["kind"], case["N"]
    if kind == "solve":
        return None
    if kind == "group":
        return [_eval64(*_problem(f, seed * 16 + i)) for i, f in enumerate(_group_fields(case))]
    if kind == "eval":
        loss, grad = _eval64(*_problem(case, seed))
        return {"loss": loss.sum() if case["option"] == "autograd" else loss, "grad": grad}
    if kind in ("estimate", "restore"):
        system, alpha, D, gamma, _ = _problem(case, seed)
        obj = _objects64(system, alpha, D, gamma, kind == "restore")
        if kind == "estimate":
            return obj
        mosaic, L = _mosaic64(obj, case["side"], N // 2, N // 8), _spectrum_side(case)
        power, sector = _spectrum64(mosaic[0, :L, :L], _window(L, L // 16))
        return {"objects": obj, "mosaic": mosaic, "power": power, "sector": sector, "counts": None}
    if kind == "prepare":
        s = prepare(case, seed)
        C, J, side = s["frames"].shape[0], case["J"], case["side"]
        window, out = s["window"].to(F64), []
        for c in range(C):
            x = s["frames"][c].unfold(1, N, N // 2).unfold(2, N, N // 2)[:, :side, :side]
            x = x.permute(1, 2, 0, 3, 4).reshape(side * side, J, N, N)
            out.append(torch.cat([torch.fft.rfft2(_apodized(v.to(F64), window)) for v in x.split(64)]))
        return torch.stack(out, 1)
    J, M, B = case["J"], case["M"], case["B"]
    if kind == "bursts":
        s = prepare(case, seed)
        noise = _normals64(s["seed"], 0x2050, B * J * N * N).to(DEV).reshape(B, 1, J, N, N)
        tables = [t[0] for t in _on_gpu(_system(N, M, "one"), F64)]
        S, _ = _otf(s["alpha"].to(F64), *tables)
        x = torch.fft.irfft2(s["O"].to(torch.complex128) * S, s=(N, N)) + s["sigma"].to(F64)[:, None, None, None] * noise[:, 0]
        D = torch.fft.rfft2(_apodized(x, s["window"].to(F64)))
        return {"noise": noise, "frames": x.permute(1, 0, 2, 3).reshape(1, J, B * N, N), "D": D[:, None]}
    gen = _gen(seed)
    params, layers = _cnn_params(gen, N, J, M)
    _, D, alpha = _bursts(gen, N, B, J, M)
    scale = torch.from_numpy(_mode_std(M) * 10.0).to(DEV, F64)
    if kind == "predict":
        with torch.no_grad():
            return torch.cat([_cnn64(d, params.to(F64), layers, N, J, M) for d in D.split(64)]) * scale
    w = params.to(F64).requires_grad_(True)
    loss = 0.0
    for d, a in zip(D.split(64), alpha.split(64)):
        part = _burst_loss64(_cnn64(d, w, layers, N, J, M), a, scale) * (d.shape[0] / B)
        part.backward()
        loss = loss + part.detach()
    return {"loss": loss.reshape(1), "grad": w.grad}
