"""Performance cases: the calls a user of this library makes, over the sizes it is used at.

A case is a dict of plain values; its "call" names the entry point:

  as_tax     pam_as_tax on a batch of frames of one record length (float32 RF in HBM, outputs and
             workspace kept by the program): the latency and the throughput form of the method
  grouped    pam_as_tax_grouped: frames of several record lengths of one plan in one call
  fd_tea     pam_fd_tea_tax, the comparison beamformer on the same plan
  surrogate  SurrogatePipeline: one full-aperture propagation, the network's mask, the calibrated fallback
  conv       one 3x3 convolution layer of the network, forward and backward
  train      the network's forward pass, loss and gradients on one batch

listed() holds the set-ups of this repository's configurations, tests and benchmark; draw() spreads
the same calls over their ranges.  exact() evaluates the same outputs with torch in 64 bits.
"""
import math
import os

import numpy as np
import torch

from paper_2412_02413_amd import nn, pam, surrogate, synth

MM = 1e-3
MHZ = 1e6
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(surrogate.__file__)), "weights",
                       "surrogate_l4_b32_coh.safetensors")
CHANNELS = (32, 64, 128, 256)          # of the network's levels


def _array(call, name, elements, n_samples, n_x, n_z, frames, **kw):
    """A case on the 0.3 mm, 20 MHz, 1-5 MHz array unless told otherwise."""
    c = dict(name=name, call=call, elements=elements, pitch_mm=0.3, fs_mhz=20.0, c_mps=1540.0, n_samples=n_samples,
             lo_mhz=1.0, hi_mhz=5.0, n_x=n_x, lateral="pad", n_z=n_z, z0_mm=15.0, dz_mm=0.1, n_sub=3,
             precision="fp32", frames=frames)
    c.update(kw)
    return c


_BENCH = dict(fs_mhz=40.0, lo_mhz=0.5, hi_mhz=8.0)          # the 128-element benchmark array


def listed():
    return [
        # one frame of the small array as it arrives: the smallest call, where latency counts
        _array("as_tax", "small_frame", 64, 1024, 128, 151, 1, z0_mm=20.0, dz_mm=0.2),
        # one frame of the benchmark array: the latency of real-time imaging
        _array("as_tax", "bench_frame", 128, 4096, 256, 512, 1, **_BENCH),
        # recorded data of the benchmark array in full launches: the headline throughput
        _array("as_tax", "bench_batch", 128, 4096, 256, 512, 64, **_BENCH),
        # the serving mix's largest request: 256 elements, the longest record, 512 columns
        _array("as_tax", "large_frame", 256, 16384, 512, 1024, 1, pitch_mm=0.2, fs_mhz=40.0, lo_mhz=0.5, hi_mhz=8.0,
               dz_mm=0.05),
        # a 96-element probe zero-stuffed to 192 columns on an odd number of depths, the paper's rate and band
        _array("as_tax", "ragged_columns", 96, 2048, 192, 301, 4, pitch_mm=0.178, fs_mhz=35.6, c_mps=1500.0,
               lo_mhz=3.0, hi_mhz=15.0, lateral="stuff", z0_mm=10.0, dz_mm=0.2),
        # the benchmark array in the split-precision form
        _array("as_tax", "bench_split_bf16", 128, 4096, 256, 512, 16, precision="split_bf16", **_BENCH),
        # a queue of mixed record lengths of the small array, one call
        _array("grouped", "mixed_lengths", 64, 8192, 128, 151, 0, z0_mm=20.0, dz_mm=0.2, frames_full=9,
               frames_half=7, frames_quarter=5),
        # the comparison beamformer on the benchmark array
        _array("fd_tea", "fd_tea_frame", 128, 4096, 256, 512, 1, **_BENCH),
        # surrogate imaging of the benchmark array with the shipped weights and calibration
        _array("surrogate", "surrogate_batch", 128, 4096, 256, 512, 16, **_BENCH),
        # the network's first level (most pixels, fewest channels), forward and backward
        dict(name="conv_top", call="conv", batch=8, h=512, w=256, c_in=32, c_out=32),
        # its deepest level (fewest pixels, most channels)
        dict(name="conv_deep", call="conv", batch=8, h=64, w=32, c_in=256, c_out=256),
        # one training batch of the network: forward, loss, every gradient
        dict(name="train_batch", call="train", batch=8, h=512, w=256, levels=4),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _field_work(c, frames=None, n_samples=None):
    """Pixels times bins of a reconstruction."""
    n_t = c["n_samples"] if n_samples is None else n_samples
    bins = (c["hi_mhz"] - c["lo_mhz"]) / c["fs_mhz"] * n_t
    return bins * c["n_z"] * c["n_x"] * (c["frames"] if frames is None else frames)


_MOST = 64 * 768 * 512 * 256       # bins x pixels of the largest listed reconstruction


def _draw_array(rng, call):
    """An array and grid of the ranges the configurations span: 32-256 elements, 64-512 columns in
    steps of 32 (padded, or zero-stuffed where a multiple of the elements), odd depth counts."""
    elements = rng.choice([32, 48, 64, 64, 80, 96, 128, 128, 160, 192, 256])
    lateral = rng.choice(["pad", "pad", "stuff"])
    if lateral == "stuff":
        n_x = elements * rng.choice([2, 2, 4])
        if n_x > 512 or n_x % 32:
            lateral = "pad"
    if lateral == "pad":
        n_x = rng.choice([n for n in range(64, 513, 32) if elements <= n <= 4 * elements])
        n_x = rng.choice([n_x, min(512, 2 * elements // 32 * 32 or 64)])
        n_x = max(n_x, (elements + 31) // 32 * 32)
    fs, lo, hi = rng.choice([(20.0, 1.0, 5.0), (40.0, 0.5, 8.0), (35.6, 3.0, 15.0)])
    n_z = int(_log(rng, 45, 1024)) | 1
    return _array(call, "", elements, 2 ** rng.randint(10, 13), n_x, n_z, 1, fs_mhz=fs, lo_mhz=lo, hi_mhz=hi,
                  lateral=lateral, pitch_mm=rng.choice([0.178, 0.2, 0.3]), dz_mm=round(52.0 / n_z, 4))


def draw(rng):
    call = rng.choice(["as_tax"] * 6 + ["grouped", "fd_tea", "surrogate", "conv", "conv", "train"])
    if call == "conv":
        level = rng.randint(0, 3)
        c = dict(call=call, batch=rng.randint(1, 8), h=(rng.randint(96, 512) >> level) | 1,
                 w=32 * rng.randint(1, 8 >> level if level < 3 else 1), c_in=CHANNELS[level],
                 c_out=CHANNELS[level])
        if level < 3 and rng.random() < 0.4:
            c["c_in"] = CHANNELS[level] + CHANNELS[level + 1]      # the decoder's first convolution
        return c
    if call == "train":
        return dict(call=call, batch=rng.randint(1, 8), h=8 * rng.randint(8, 64), w=256, levels=rng.choice([3, 4]))
    if call == "surrogate":
        small = rng.random() < 0.5             # the two calibrated geometries
        c = _array(call, "", 64 if small else 128, 1024 if small else 4096, 256, 512, rng.randint(1, 24))
        if not small:
            c.update(_BENCH)
        del c["name"]
        return c
    c = _draw_array(rng, call)
    del c["name"]
    if call == "as_tax":
        c["n_sub"] = rng.choice([1, 2, 3, 3, 3, 3])
        c["precision"] = rng.choice(["fp32"] * 4 + ["split_bf16", "split_fp16"])
        cap = _MOST / 4 / _field_work(c)
        c["frames"] = max(1, min(48, int(_log(rng, 1, max(1.01, cap)))))
    elif call == "grouped":
        c["n_samples"] = max(c["n_samples"], 4096)
        cap = max(1, min(16, int(_MOST / 8 / _field_work(c))))
        c["frames"] = 0
        c.update(frames_full=rng.randint(1, cap), frames_half=rng.randint(1, cap), frames_quarter=rng.randint(0, cap))
    else:
        c["n_z"] = min(c["n_z"], 513)
        c["n_samples"] = min(c["n_samples"], 4096)
        c["frames"] = max(1, min(4, int(768 * 512 * 256 / _field_work(c))))
    return c


# -- inputs ------------------------------------------------------------------------------------

def _geometry(c, **kw):
    g = synth.Geometry(n_elements=c["elements"], pitch_m=c["pitch_mm"] * MM, fs_hz=c["fs_mhz"] * MHZ,
                       c_mps=c["c_mps"], n_samples=c["n_samples"],
                       bands_hz=[(c["lo_mhz"] * MHZ, c["hi_mhz"] * MHZ)],
                       depths_m=(c["z0_mm"] + c["dz_mm"] * np.arange(c["n_z"], dtype=np.float64)) * MM,
                       n_x=c["n_x"], lateral=c["lateral"], n_sub=c["n_sub"])
    return g.replace(**kw) if kw else g


def _rf(c, frames, n_t, seed):
    """Frames of band-limited emitters (three harmonic, two noise-like) seen with exact delays, plus
    white channel noise at 20 dB: float32 [frames][elements][n_t] on the GPU."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def uni(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)

    fs = c["fs_mhz"] * MHZ
    f = torch.arange(n_t // 2 + 1, device="cuda", dtype=torch.float64) * (fs / n_t)
    lo, hi = c["lo_mhz"] * MHZ, c["hi_mhz"] * MHZ
    band = ((f >= lo) & (f <= hi)).double()
    el = (torch.arange(c["elements"], device="cuda", dtype=torch.float64) - (c["elements"] - 1) / 2) * (c["pitch_mm"] * MM)
    half = 0.4 * c["elements"] * c["pitch_mm"] * MM
    z_lo, z_hi = c["z0_mm"] * MM, (c["z0_mm"] + c["dz_mm"] * (c["n_z"] - 1)) * MM
    out = torch.empty((frames, c["elements"], n_t), dtype=torch.float32, device="cuda")
    for k in range(frames):
        spec = torch.zeros((c["elements"], n_t // 2 + 1), dtype=torch.complex128, device="cuda")
        for e in range(5):
            noise = torch.randn((2, n_t // 2 + 1), generator=gen, device="cuda", dtype=torch.float64)
            s = torch.complex(noise[0], noise[1]) * band
            if e < 3:                                   # lines at multiples of 1.5 MHz, a few bins wide
                off = (f / (1.5 * MHZ) - torch.round(f / (1.5 * MHZ))).abs() * (1.5 * MHZ)
                s = s * torch.exp(-(off / (2.0 * fs / n_t)) ** 2)
            s = s / s.abs().square().sum().sqrt().clamp_min(1e-30)
            x, z = uni(-half, half, 1), uni(z_lo + 0.1 * (z_hi - z_lo), z_hi, 1)
            tau = ((el - x) ** 2 + z ** 2).sqrt() / c["c_mps"]
            ph = torch.outer(tau, f) * (-2.0 * math.pi)
            spec += s * torch.polar(torch.ones_like(ph), ph)
        sig = torch.fft.irfft(spec, n=n_t, dim=-1)
        sig = sig / sig.square().mean().sqrt()
        sig += 0.1 * torch.randn(sig.shape, generator=gen, device="cuda", dtype=torch.float64)
        out[k] = sig.float()
    return out


class _Plan:
    """A plan the program keeps; released with the state that holds it."""

    def __init__(self, geom, precision):
        self.plan = pam.pam_plan(geom, 0, precision)

    def __del__(self):
        pam.pam_destroy(self.plan)


class _Pipe:
    def __init__(self, geom, frames):
        self.net, calibration = surrogate.UNet.from_weights(WEIGHTS)
        self.tau = calibration[surrogate.geometry_key(geom)]["tau"]
        self.pipe = surrogate.SurrogatePipeline(geom, self.net, self.tau, max_frames=frames)

    def __del__(self):
        if hasattr(self, "pipe"):
            self.pipe.close()


def _groups(c):
    """(record length, frames) of a grouped case."""
    n = c["n_samples"]
    return [(n, c["frames_full"]), (n // 2, c["frames_half"]), (n // 4, c["frames_quarter"])]


def _conv_inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, h, w, ci, co = c["batch"], c["h"], c["w"], c["c_in"], c["c_out"]

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    x = normal(B, h, w, ci).relu().to(torch.bfloat16)            # activations after a ReLU
    dy = (normal(B, h, w, co) * 1e-3).to(torch.bfloat16)
    W = normal(9, ci, co) * math.sqrt(2.0 / (9 * ci))
    return x, dy, W, 0.05 * normal(co)


def _train_inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, h, w = c["batch"], c["h"], c["w"]
    feats = torch.zeros((B, h, w, surrogate.C_FEAT), device="cuda")
    feats[..., :surrogate.N_FEAT] = torch.rand((B, h, w, surrogate.N_FEAT), generator=gen, device="cuda")
    target = torch.rand((B, h, w), generator=gen, device="cuda")
    weight = torch.rand((B, h, w), generator=gen, device="cuda")
    return feats.to(torch.bfloat16), target, weight / weight.sum()


def prepare(case, seed):
    call = case["call"]
    s = {"case": case}
    if call == "conv":
        B, h, w, ci, co = case["batch"], case["h"], case["w"], case["c_in"], case["c_out"]
        x, dy, W, b = _conv_inputs(case, seed)
        s.update(x=x, dy=dy, bias=b)
        s["wt"] = torch.empty((co, 9, ci), dtype=torch.bfloat16, device="cuda")
        s["wd"] = torch.empty((ci, 9, co), dtype=torch.bfloat16, device="cuda")
        nn.pack_weights(W.contiguous(), ci, co, s["wt"], s["wd"])
        s["y"] = torch.empty((B, h, w, co), dtype=torch.bfloat16, device="cuda")
        s["g"] = torch.empty_like(dy)
        s["dx"] = torch.empty((B, h, w, ci), dtype=torch.bfloat16, device="cuda")
        s["dw"] = torch.empty((9, ci, co), dtype=torch.float32, device="cuda")
        s["db"] = torch.empty(co, dtype=torch.float32, device="cuda")
        return s
    if call == "train":
        s["x"], s["target"], s["weight"] = _train_inputs(case, seed)
        s["net"] = surrogate.UNet(case["levels"], 32, seed=seed)
        return s
    if call == "surrogate":
        s["rf"] = _rf(case, case["frames"], case["n_samples"], seed)
        s["pipe"] = _Pipe(_geometry(case), case["frames"])
        return s
    s["plan"] = _Plan(_geometry(case), case["precision"])
    plan = s["plan"].plan
    if call == "grouped":
        s["groups"] = _groups(case)
        s["rf"] = torch.cat([_rf(case, F, n, seed + 7919 * k).view(-1) for k, (n, F) in enumerate(s["groups"])])
        F = sum(f for _, f in s["groups"])
        s["ws"] = pam.alloc_workspace_grouped(plan, s["groups"])
    else:
        F = case["frames"]
        s["rf"] = _rf(case, F, case["n_samples"], seed)
        s["ws"] = pam.alloc_workspace(plan, F, case["n_samples"])
    s["image"] = torch.empty((F, plan.n_z, plan.n_x), device="cuda")
    s["nncc"] = torch.empty_like(s["image"])
    return s


def run(s):
    c = s["case"]
    call = c["call"]
    if call == "as_tax":
        pam.pam_as_tax(s["plan"].plan, s["rf"], s["image"], s["nncc"], None, s["ws"])
    elif call == "grouped":
        pam.pam_as_tax_grouped(s["plan"].plan, s["rf"], s["groups"], s["image"], s["nncc"], None, s["ws"])
    elif call == "fd_tea":
        pam.pam_fd_tea_tax(s["plan"].plan, s["rf"], s["image"], s["nncc"], None, s["ws"])
    elif call == "surrogate":
        image, mask, est, fallback = s["pipe"].pipe(s["rf"])
        return {"image": image, "mask": mask, "est": est, "fallback": fallback}
    elif call == "train":
        net = s["net"]
        mask, err = net.forward(s["x"], c["batch"], c["h"], c["w"])
        loss = net.loss_backward(s["target"], s["weight"])
        return {"mask": mask, "err": err, "loss": loss, "grads": net.grads}
    else:
        B, h, w, ci, co = c["batch"], c["h"], c["w"], c["c_in"], c["c_out"]
        nn.conv3x3(s["x"], ci, B, h, w, ci, s["wt"], s["bias"], s["y"], co, co, relu=True)
        s["g"].copy_(s["dy"])
        s["dw"].zero_()
        s["db"].zero_()
        nn.relu_backward(s["y"], co, s["g"], co, B * h * w, co)
        nn.conv3x3_wgrad(s["x"], ci, s["g"], co, B, h, w, ci, co, s["dw"], s["db"])
        nn.conv3x3(s["g"], co, B, h, w, co, s["wd"], None, s["dx"], ci, ci, relu=False, flip=True)
        return {"y": s["y"], "dx": s["dx"], "dw": s["dw"], "db": s["db"]}
    return {"image": s["image"], "nncc": s["nncc"]}


# -- work --------------------------------------------------------------------------------------

def _bins(c, n_t):
    """Number of selected bins of a record of n_t samples on the case's plan."""
    k = np.arange(1, (c["n_samples"] + 1) // 2)
    f = k * (c["fs_mhz"] * MHZ) / c["n_samples"]
    k = k[(f >= c["lo_mhz"] * MHZ) & (f <= c["hi_mhz"] * MHZ)]
    return k[k % (c["n_samples"] // n_t) == 0] // (c["n_samples"] // n_t)


def _as_work(c, frames, n_t, n_sub, outputs=2):
    """The method's operations with 5 N log2 N per complex transform: per (bin, depth, column) the
    inverse lateral transform and the propagator product of each sub-aperture and the sums."""
    nb = len(_bins(c, n_t))
    sums = {1: 4, 2: 12, 3: 24}[n_sub]
    point = n_sub * (5 * math.log2(c["n_x"]) + 6) + sums
    time = 2.5 * n_t * math.log2(n_t) * c["elements"]
    return {"bytes": frames * 4.0 * (c["elements"] * n_t + outputs * c["n_z"] * c["n_x"]),
            "flops": frames * (nb * c["n_z"] * c["n_x"] * point + time)}


def _net_flops(h, w, levels):
    """Multiply-adds (as two operations) of the network's forward pass per frame."""
    total, prev = 0.0, surrogate.N_FEAT
    for l in range(levels):
        p = (h >> l) * (w >> l)
        total += 18.0 * p * CHANNELS[l] * (prev + CHANNELS[l])
        prev = CHANNELS[l]
        if l < levels - 1:
            total += 18.0 * p * CHANNELS[l] * (CHANNELS[l + 1] + 2 * CHANNELS[l])
    return total + 4.0 * h * w * CHANNELS[0]


def _net_params(levels):
    n, prev = 2 * CHANNELS[0], surrogate.N_FEAT
    for l in range(levels):
        n += 9 * CHANNELS[l] * (prev + CHANNELS[l])
        prev = CHANNELS[l]
        if l < levels - 1:
            n += 9 * CHANNELS[l] * (CHANNELS[l + 1] + 2 * CHANNELS[l])
    return n


def work(case):
    c, call = case, case["call"]
    if call == "as_tax":
        return _as_work(c, c["frames"], c["n_samples"], c["n_sub"])
    if call == "grouped":
        w = [_as_work(c, F, n, c["n_sub"]) for n, F in _groups(c)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    if call == "fd_tea":
        nb = len(_bins(c, c["n_samples"]))
        base = _as_work(c, c["frames"], c["n_samples"], c["n_sub"])
        return {"bytes": base["bytes"],
                "flops": c["frames"] * nb * c["n_z"] * c["n_x"] * (8.0 * c["elements"] + 24)}
    if call == "surrogate":
        base = _as_work(c, c["frames"], c["n_samples"], 1)
        return {"bytes": base["bytes"] + 2.0 * _net_params(4),
                "flops": base["flops"] + c["frames"] * _net_flops(c["n_z"], c["n_x"], 4)}
    if call == "train":
        px = c["batch"] * c["h"] * c["w"]
        return {"bytes": px * (2.0 * surrogate.C_FEAT + 16) + 6.0 * _net_params(c["levels"]),
                "flops": 3.0 * c["batch"] * _net_flops(c["h"], c["w"], c["levels"])}
    px = c["batch"] * c["h"] * c["w"]
    return {"bytes": px * 4.0 * (c["c_in"] + c["c_out"]) + 72.0 * c["c_in"] * c["c_out"],
            "flops": 54.0 * px * c["c_in"] * c["c_out"]}


# -- the same outputs in 64 bits -----------------------------------------------------------------

def _placement(c):
    if c["lateral"] == "pad":
        return (c["n_x"] - c["elements"]) // 2, 1, c["pitch_mm"] * MM
    step = c["n_x"] // c["elements"]
    return 0, step, c["pitch_mm"] * MM / step


def _masks(c, n_sub):
    l = torch.arange(c["elements"], device="cuda")
    return torch.stack([((l // 16) % n_sub == i).double() for i in range(n_sub)])


def _spectra(c, rf):
    """In-band spectra [L][bins] of one frame and its bin indices."""
    k = torch.from_numpy(_bins(c, rf.shape[-1])).cuda()
    return torch.fft.rfft(rf.double(), dim=-1)[:, k], k.double()


def _sums(p):
    """S_i and C_ij of fields p [n_sub][bins][...], summed over the bins."""
    n = p.shape[0]
    pairs = {1: [], 2: [(0, 1)], 3: [(0, 1), (1, 2), (2, 0)]}[n]
    S = [p[i].abs().square().sum(0) for i in range(n)]
    C = [(p[i].conj() * p[j]).real.sum(0) for i, j in pairs]
    return torch.stack(S + C)


def _image(acc, n_sub):
    S, C = acc[:n_sub], acc[n_sub:]
    E = S.sum(0) + 2.0 * C.sum(0)
    w = torch.ones_like(E)
    for (i, j), cc in zip({1: [], 2: [(0, 1)], 3: [(0, 1), (1, 2), (2, 0)]}[n_sub], C):
        den = (S[i] * S[j]).sqrt()
        w = w * torch.where(den > 0, cc / den.clamp_min(1e-300), torch.zeros_like(cc)).clamp(1e-3, 1.0)
    if n_sub == 3:
        w = w ** (1.0 / 3.0)
    rho = w / w.max()
    return rho ** 2 * E, rho


def _propagated(c, X, k, n_t, n_sub, reduce):
    """Sum over bins of reduce(fields [n_sub][bins][n_z][n_x]) for one frame's spectra X [L][bins]."""
    col0, step, dx = _placement(c)
    N = c["n_x"]
    z = torch.from_numpy(_geometry(c).depths_m).cuda()
    kx = 2 * math.pi * torch.fft.fftfreq(N, d=dx, dtype=torch.float64, device="cuda")
    masks = _masks(c, n_sub) if n_sub > 1 else torch.ones((1, c["elements"]), dtype=torch.float64, device="cuda")
    total = 0
    chunk = max(1, int(3e7 / (n_sub * c["n_z"] * N)))
    for b in range(0, len(k), chunk):
        kk = 2 * math.pi * k[b:b + chunk] * (c["fs_mhz"] * MHZ) / n_t / c["c_mps"]
        v = torch.zeros((n_sub, len(kk), N), dtype=torch.complex128, device="cuda")
        v[:, :, col0: col0 + step * c["elements"]: step] = masks[:, None, :] * X[:, b:b + chunk].T[None]
        A = torch.fft.fft(v, dim=-1)
        d = kk[:, None] ** 2 - kx[None] ** 2
        kz = torch.where(d >= 0, torch.complex(d.clamp_min(0).sqrt(), torch.zeros_like(d)),
                         torch.complex(torch.zeros_like(d), (-d).clamp_min(0).sqrt()))
        H = torch.exp(1j * kz[:, None, :] * z[None, :, None])
        total = total + reduce(torch.fft.ifft(H[None] * A[:, :, None, :], dim=-1))
    return total


def _delayed(c, X, k, n_t, n_sub):
    """Delay-and-sum fields of one frame, summed over bins."""
    col0, step, dx = _placement(c)
    N, L = c["n_x"], c["elements"]
    z = torch.from_numpy(_geometry(c).depths_m).cuda()
    centre = col0 + step * (L - 1) / 2.0
    x = (torch.arange(N, device="cuda", dtype=torch.float64) - centre) * dx
    xl = (col0 + step * torch.arange(L, device="cuda", dtype=torch.float64) - centre) * dx
    masks = _masks(c, n_sub)
    total = 0
    chunk = max(1, int(2e7 / (c["n_z"] * N)))
    for b in range(0, len(k), chunk):
        om = 2 * math.pi * k[b:b + chunk] * (c["fs_mhz"] * MHZ) / n_t
        p = torch.zeros((n_sub, len(om), c["n_z"], N), dtype=torch.complex128, device="cuda")
        for l in range(L):
            tau = ((x[None] - xl[l]) ** 2 + z[:, None] ** 2).sqrt() / c["c_mps"]
            ph = om[:, None, None] * tau
            v = torch.polar(torch.ones_like(ph), ph) * X[l, b:b + chunk, None, None]
            for i in range(n_sub):
                if masks[i, l] > 0:
                    p[i] += v
        total = total + _sums(p)
    return total


def _conv64(x, W, b=None):
    """3x3 convolution [B][h][w][ci] with W [9][ci][co], zeros outside, as nine products."""
    h, w = x.shape[1:3]
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = 0
    for t in range(9):
        y = y + xp[:, t // 3: t // 3 + h, t % 3: t % 3 + w] @ W[t]
    return y if b is None else y + b


def _network64(P, x, levels):
    """The network on features x in 64 bits: logits of the mask and of the error head."""
    F = torch.nn.functional

    def block(h, name):
        for s in "ab":
            h = _conv64(h, P[f"{name}{s}.w"], P[f"{name}{s}.b"]).relu()
        return h

    skips, h = [], x
    for l in range(levels):
        if l:
            h = F.max_pool2d(h.permute(0, 3, 1, 2), 2).permute(0, 2, 3, 1)
        h = block(h, f"enc{l}")
        skips.append(h)
    for l in range(levels - 2, -1, -1):
        up = h.repeat_interleave(2, 1).repeat_interleave(2, 2)
        h = block(torch.cat([up, skips[l]], -1), f"dec{l}")
    return h @ P["head.w"] + P["head.b"]


def _params64(net, grad=False):
    """The network's parameters in 64 bits, the convolutions' weights as the BF16 operands they are."""
    out = {}
    for k, v in net.params.items():
        v = v.to(torch.bfloat16) if k.endswith(".w") and k != "head.w" else v
        out[k] = v.double().requires_grad_(grad)
    return out


def _surrogate64(c, seed):
    rf = _rf(c, c["frames"], c["n_samples"], seed)
    net, _ = surrogate.UNet.from_weights(WEIGHTS)
    P = _params64(net)
    masks, ests = [], []
    xe, ze = torch.arange(c["n_x"], device="cuda") & ~1, torch.arange(c["n_z"], device="cuda") & ~1

    def reduce(p):
        p = p[0]
        gx = p[..., xe] * p[..., xe + 1].conj()
        gz = p[:, ze] * p[:, ze + 1].conj()
        return torch.stack([p.abs().square().sum(0), gx.real.sum(0), gx.imag.sum(0), gz.real.sum(0), gz.imag.sum(0)])

    for f in range(c["frames"]):
        X, k = _spectra(c, rf[f])
        A = _propagated(c, X, k, c["n_samples"], 1, reduce)
        E = A[0]
        r = E / E.max()
        feats = torch.zeros((1, c["n_z"], c["n_x"], surrogate.C_FEAT), dtype=torch.float64, device="cuda")
        feats[0, ..., 0] = ((r.clamp_min(1e-30)).log10() / 6 + 1).clamp(0, 1)
        feats[0, ..., 1] = r
        for at, (re, im), den in ((2, A[1:3], E[:, xe] * E[:, xe + 1]), (5, A[3:5], E[ze] * E[ze + 1])):
            q = den.clamp_min(1e-300).rsqrt()
            re, im = re * q, im * q
            feats[0, ..., at] = (re ** 2 + im ** 2).sqrt()
            feats[0, ..., at + 1], feats[0, ..., at + 2] = re, im
        out = torch.sigmoid(_network64(P, feats.to(torch.bfloat16).double(), 4))
        m, e = out[0, ..., 0], out[0, ..., 1]
        masks.append(m)
        ests.append((2 * m * e * E).norm() / (m * m * E).norm())
    return {"image": None, "mask": torch.stack(masks), "est": torch.stack(ests), "fallback": None}


def _train64(c, seed):
    x, target, weight = _train_inputs(c, seed)
    net = surrogate.UNet(c["levels"], 32, seed=seed)
    P = _params64(net, grad=True)
    target, weight = target.double(), weight.double()
    mask, err, loss = [], [], torch.zeros(3, dtype=torch.float64, device="cuda")
    sp = torch.nn.functional.softplus
    for b in range(c["batch"]):
        z = _network64(P, x[b:b + 1].double(), c["levels"])[0]
        m, e = torch.sigmoid(z[..., 0]), torch.sigmoid(z[..., 1])
        ae = (m - target[b]).abs().detach()
        l0 = (weight[b] * (target[b] * sp(-z[..., 0]) + (1 - target[b]) * sp(z[..., 0]))).sum()
        l1 = (weight[b] * (ae * sp(-z[..., 1]) + (1 - ae) * sp(z[..., 1]))).sum()
        (l0 + l1).backward()
        loss += torch.stack([l0, l1, (weight[b] * ae).sum()]).detach()
        mask.append(m.detach())
        err.append(e.detach())
    return {"mask": torch.stack(mask), "err": torch.stack(err), "loss": loss, "grads": {k: v.grad for k, v in P.items()}}


def _conv64_layer(c, seed):
    x, dy, W, b = _conv_inputs(c, seed)
    x, dy, W, b = x.double(), dy.double(), W.to(torch.bfloat16).double(), b.double()
    y = _conv64(x, W, b).relu()
    g = dy * (y > 0)
    h, w = c["h"], c["w"]
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    dw = torch.stack([xp[:, t // 3: t // 3 + h, t % 3: t % 3 + w].reshape(-1, c["c_in"]).T @ g.reshape(-1, c["c_out"])
                      for t in range(9)])
    dx = _conv64(g, torch.stack([W[8 - t].T for t in range(9)]))
    return {"y": y, "dx": dx, "dw": dw, "db": g.sum((0, 1, 2))}


def exact(case, seed):
    c, call = case, case["call"]
    if call == "conv":
        return _conv64_layer(c, seed)
    if call == "train":
        return _train64(c, seed)
    if call == "surrogate":
        return _surrogate64(c, seed)
    if call == "grouped":
        parts = [(_rf(c, F, n, seed + 7919 * k), n) for k, (n, F) in enumerate(_groups(c))]
    else:
        parts = [(_rf(c, c["frames"], c["n_samples"], seed), c["n_samples"])]
    images, rhos = [], []
    for rf, n_t in parts:
        for f in range(rf.shape[0]):
            X, k = _spectra(c, rf[f])
            if call == "fd_tea":
                acc = _delayed(c, X, k, n_t, c["n_sub"])
            else:
                acc = _propagated(c, X, k, n_t, c["n_sub"], _sums)
            I, rho = _image(acc, c["n_sub"])
            images.append(I)
            rhos.append(rho)
    return {"image": torch.stack(images), "nncc": torch.stack(rhos)}
