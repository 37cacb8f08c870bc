"""The work that a user of this library has it do, as cases that can be timed and compared.

A case names one call (or the short chain of calls that belongs together) and its sizes.
Sizes are those of the repository's own configurations: the paper-scale ensemble (128 + 128
elements, 9 angles, 300 frames, planes of 250 x 274), its P = 8 sub-block form (35 slabs
per orientation), the tiny ensemble (32 + 32 elements, 4 angles, 20 frames, 64 x 64), and
everything between them in draw().
"""
from __future__ import annotations

import math
import os
from types import SimpleNamespace

import numpy as np
import torch

import paper_2511_21647_amd as ulm

DEV = "cuda"
C0, F0, FS, BANDWIDTH = 1540.0, 6e6, 24e6, 0.65
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(ulm.__file__)), "weights", "cnn_paper.npy")


# ------------------------------------------------------------------ the cases

def _case(op, name=None, **kw):
    c = dict(op=op, shallow=False, elems=128, angles=9, frames=300, nz=250, nu=274, blocks=1,
             cutoff=20, ncc=9, precision="fp64")
    c.update(kw)
    if name:
        c = dict(name=name, **c)
    return c


def listed():
    return [
        # the smallest call: one tiny ensemble, IQ to localisations; launches and latency count
        _case("path", "path_tiny", shallow=True, elems=32, angles=4, frames=20, nz=64, nu=64,
              cutoff=2, ncc=7),
        # the headline: one paper-scale ensemble, IQ to localisations, plain path
        _case("path", "path_paper"),
        # stage 2 of the P = 8 sub-block form: 2 x 35 slab planes from the stage-1 slices
        _case("stage2", "stage2_slabs", blocks=35),
        # the clutter filter of the 70 slab planes, plain (FP64) precision
        _case("filter", "filter_slabs", blocks=35),
        # the clutter filter in the split-BF16 form, one plane per orientation
        _case("filter", "filter_paper_bf16x3", precision="bf16x3"),
        # NCC localisation of one ensemble's two planes
        _case("ncc", "ncc_paper"),
        # the sub-block form's localisation: NCC on 70 slab planes, then the XZ/YZ pairing
        _case("detect3d", "detect3d_slabs", blocks=35),
        # XDoppler: native and cross projections, both filtered, correlated over 3 frames
        _case("xdoppler", "xdoppler_paper", window=3),
        # rigid motion of 300 frames on the 18 stage-1 slices, +-8 pixels
        _case("motion", "motion_paper", lag=8),
        # separation of one ensemble into three speeds up and three down
        _case("separate", "separate_paper", speeds=3),
        # the learned localiser on one ensemble's 600 images with the shipped weights
        _case("cnn_localize", "cnn_localize_paper"),
        # one training step of that network (batch of 16 images, BF16 activations)
        _case("cnn_train", "cnn_train_paper", batch=16, train="bf16"),
    ]


FRAME_COUNTS = (20, 25, 36, 50, 63, 75, 96, 125, 150, 200, 245, 300)   # factors 2, 3, 5, 7


def draw(rng):
    """A case of the same calls between the tiny and the paper-scale configuration."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["path", "stage2", "filter", "filter", "ncc", "detect3d", "xdoppler", "motion",
                     "separate", "cnn_localize", "cnn_train"])
    nz, nu = log_int(48, 250), log_int(48, 274)
    frames = rng.choice(FRAME_COUNTS)
    c = _case(op, shallow=nz < 100, elems=log_int(32, 128), angles=rng.randint(3, 9),
              frames=frames, nz=nz, nu=nu, cutoff=rng.randint(2, min(20, frames // 4)),
              ncc=rng.choice([5, 7, 9, 11]))
    if op in ("stage2", "filter", "ncc", "detect3d"):
        per = -(-nu // min(log_int(1, 35), nu // 8))
        c["blocks"] = -(-nu // per)
    if op in ("path", "filter"):
        c["precision"] = rng.choice(["fp64", "fp64", "bf16x3"])
    if op == "xdoppler":
        c["window"] = rng.choice([1, 3, 5])
    if op == "motion":
        c["lag"] = rng.randint(3, 10)
    if op == "separate":
        c["speeds"] = rng.randint(1, 4)
    if op == "cnn_train":
        c.update(batch=rng.randint(1, 16), train=rng.choice(["bf16", "bf16", "fp32"]))
    return c


# ------------------------------------------------------------------ geometry

def _config(c):
    """The configuration object that ulm.Context takes."""
    nz, nu = c["nz"], c["nu"]
    if c["shallow"]:
        pitch, z0, dz, angles = 0.2e-3, 4e-3, 6e-3 / 64, np.linspace(-6.0, 6.0, c["angles"])
    else:
        pitch, z0, dz, angles = 0.214e-3, 20e-3, 0.1e-3, np.linspace(-8.0, 8.0, c["angles"])
    du = 0.1e-3
    t_start = 2 * z0 / C0 - 0.8e-6
    zmax = z0 + (nz - 1) * dz
    half = 0.5 * (c["elems"] - 1) * pitch
    reach = half + 0.5 * (nu - 1) * du
    tmax = (zmax + half * math.sin(math.radians(abs(float(angles[0])))) +
            math.hypot(zmax, reach)) / C0
    samples = int(math.ceil((tmax - t_start) * FS)) + 24
    if c["elems"] == 128 and nz == 250 and nu == 274 and not c["shallow"]:
        samples = 1024
    if c["elems"] == 32 and nz == 64 and nu == 64 and c["shallow"]:
        samples = 256
    org = -0.5 * (nu - 1) * du
    return SimpleNamespace(
        probe=SimpleNamespace(n_elem=c["elems"], pitch=pitch, f0=F0, fs=FS, c=C0,
                              bandwidth=BANDWIDTH),
        seq=SimpleNamespace(angles_deg=tuple(float(a) for a in angles), n_frames=c["frames"],
                            t_start=t_start, n_samp=samples),
        grid=SimpleNamespace(nu=nu, nz=nz, du=du, dz=dz, u0=org, z0=z0, nv=nu, dv=du, v0=org,
                             n_blocks=c["blocks"], v_ref=0.0),
        svd_cutoff=c["cutoff"],
        loc=SimpleNamespace(ncc_size=c["ncc"], sigma_u=1.2, sigma_z=1.2, tau_ncc=0.5, alpha=0.05))


def _context(c):
    return ulm.Context(_config(c), precision=ulm.ULM_PREC_BF16X3 if c["precision"] == "bf16x3"
                       else ulm.ULM_PREC_FP64GRAM)


def _slab_ranges(c):
    per = -(-c["nu"] // c["blocks"])
    return [(b * per, min((b + 1) * per, c["nu"])) for b in range(c["blocks"])]


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _cnoise(shape, g):
    """Complex Gaussian of unit rms."""
    return torch.randn(shape, dtype=torch.complex64, device=DEV, generator=g)


def _tissue_profiles(c, g, modes):
    """Slow-time course of the tissue modes [modes][F]: a slow rotation with some flicker."""
    f = torch.arange(c["frames"], device=DEV, dtype=torch.float32)
    freq = torch.rand(modes, 1, device=DEV, generator=g) * 0.04 - 0.02
    flick = 1.0 + 0.3 * torch.randn(modes, c["frames"], device=DEV, generator=g)
    return torch.polar(flick, 2 * math.pi * freq * f[None, :])


def _tissue_amps(modes):
    """40 dB above the blood for the first mode, about 10 dB for the last."""
    return [100.0 * 0.03 ** (r / max(1, modes - 1)) for r in range(modes)]


def _add_tissue(x, c, g):
    """Adds the tissue modes in place to x [..][F][rows][columns]."""
    modes = c["cutoff"]
    prof = _tissue_profiles(c, g, modes)
    for r, amp in enumerate(_tissue_amps(modes)):
        field = amp * _cnoise(x.shape[:-3] + (1,) + x.shape[-2:], g)
        x.addcmul_(field.expand_as(x), prof[r].view(-1, 1, 1).expand_as(x))
    return x


def _smooth_(x, sigma=1.2, taps=3):
    """Separable circular Gaussian of x [..][rows][columns] in place, frame block by block: the
    point spread of a beamformed plane."""
    w = [math.exp(-0.5 * (t / sigma) ** 2) for t in range(-taps, taps + 1)]
    n = math.sqrt(sum(v * v for v in w))
    flat = x.view(-1, x.shape[-2], x.shape[-1])
    step = max(1, (1 << 25) // (x.shape[-2] * x.shape[-1]))
    for i in range(0, flat.shape[0], step):
        b = flat[i:i + step]
        for dim in (1, 2):
            b = sum((v / n) * torch.roll(b, t, dims=dim) for t, v in zip(range(-taps, taps + 1), w))
        flat[i:i + step] = b
    return x


def _spots_(x, g, per_image):
    """Adds microbubble spots (one point spread each, exponential strength) in place."""
    flat = x.view(-1, x.shape[-2] * x.shape[-1])
    nz, nu = x.shape[-2], x.shape[-1]
    n, rows = per_image, torch.arange(flat.shape[0], device=DEV)
    for _ in range(n):      # one spot per image and turn: no two writes meet
        cz = torch.rand(flat.shape[0], device=DEV, generator=g) * (nz - 9) + 4
        cu = torch.rand(flat.shape[0], device=DEV, generator=g) * (nu - 9) + 4
        amp = 6.0 - 4.0 * torch.log(torch.rand(flat.shape[0], device=DEV, generator=g) + 1e-6)
        ph = 2 * math.pi * torch.rand(flat.shape[0], device=DEV, generator=g)
        iz, iu = torch.floor(cz).long(), torch.floor(cu).long()
        for a in range(-2, 4):
            for b in range(-2, 4):
                r2 = (iz + a - cz) ** 2 + (iu + b - cu) ** 2
                flat[rows, (iz + a) * nu + iu + b] += torch.polar(
                    amp * torch.exp(-r2 / (2 * 1.2 ** 2)), ph)
    return x


def _planes(c, seed, filtered):
    """[2][B][F][Nz][Nu]: blood speckle with microbubble spots; the tissue is still in it
    unless `filtered`."""
    g = _gen(seed)
    x = _cnoise((2, c["blocks"], c["frames"], c["nz"], c["nu"]), g)
    # blood echoes below the microbubbles': about 370 detections an image on the two full
    # planes and 330 on slab planes, near what simulated ensembles of this library give
    _smooth_(x).mul_(0.5 if c["blocks"] == 1 else 0.34)
    _spots_(x, g, max(2, c["nz"] * c["nu"] // (4000 if c["blocks"] == 1 else 16000)))
    return x if filtered else _add_tissue(x, c, g)


def _slices(c, seed, out):
    """Stage-1 slices [2][K][F][Nz][Nu] into `out`: tissue 40 dB above blood and noise."""
    g = _gen(seed)
    for o in range(2):
        for k in range(c["angles"]):
            out[o, k] = _cnoise(out.shape[2:], g)
    modes = c["cutoff"]
    prof = _tissue_profiles(c, g, modes)
    for o in range(2):
        for r, amp in enumerate(_tissue_amps(modes)):
            field = amp * _cnoise((c["angles"], 1, c["nz"], c["nu"]), g)
            out[o].addcmul_(field.expand_as(out[o]), prof[r].view(-1, 1, 1).expand_as(out[o]))
    return out


def _moving_slices(c, seed, out):
    """Stage-1 slices of one speckle field each that moves by up to 2 pixels over the frames."""
    g = _gen(seed)
    nz, nu, F = c["nz"], c["nu"], c["frames"]
    kz = torch.fft.fftfreq(nz, device=DEV)[:, None]
    ku = torch.fft.fftfreq(nu, device=DEV)[None, :]
    band = torch.exp(-2 * (math.pi * 1.5) ** 2 * (kz ** 2 + ku ** 2))
    t = torch.arange(F, device=DEV) / max(1, F)
    dz = 2.0 * torch.sin(2 * math.pi * t)
    du = 0.5 * torch.sin(4 * math.pi * t)
    ramp = torch.polar(torch.ones((), device=DEV),
                       -2 * math.pi * (kz[None] * dz[:, None, None] + ku[None] * du[:, None, None]))
    for o in range(2):
        for k in range(c["angles"]):
            spec = torch.fft.fft2(_cnoise((nz, nu), g)) * band
            out[o, k] = torch.fft.ifft2(spec[None] * ramp)
            out[o, k] += 0.01 * _cnoise((F, nz, nu), g)
    return out


def _iq(c, seed):
    """IQ channel data [F][2][K][Nc][Ns]: tissue modes, moving microbubbles (each with its true
    wavefront in every channel) and channel noise."""
    cfg = _config(c)
    g = _gen(seed)
    F, K, Nc, Ns = c["frames"], c["angles"], c["elems"], cfg.seq.n_samp
    iq = _cnoise((F, 2, K, Nc, Ns), g).mul_(0.0316)
    modes = max(2, min(6, c["cutoff"]))
    prof = _tissue_profiles(c, g, modes)
    for r, amp in enumerate(_tissue_amps(modes)):
        field = amp * _cnoise((1, 2, K, Nc, Ns), g)
        iq.addcmul_(field.expand_as(iq), prof[r].view(-1, 1, 1, 1, 1).expand_as(iq))
    sig = math.sqrt(2 * math.log(2)) / (math.pi * BANDWIDTH * F0)
    ang = torch.tensor(cfg.seq.angles_deg, device=DEV, dtype=torch.float64) * (math.pi / 180)
    ue = (torch.arange(Nc, device=DEV, dtype=torch.float64) - 0.5 * (Nc - 1)) * cfg.probe.pitch
    L = (Nc - 1) * cfg.probe.pitch
    gr = cfg.grid
    flat = iq.view(-1, Ns)
    rows = torch.arange(F * 2 * K * Nc, device=DEV).view(F, 2, K, Nc, 1)
    half = 0.5 * (c["nu"] - 1) * gr.du
    for _ in range(24):
        p = torch.rand(3, device=DEV, generator=g, dtype=torch.float64)
        v = (torch.rand(3, device=DEV, generator=g, dtype=torch.float64) - 0.5) * 40e-3 / 400.0
        f = torch.arange(F, device=DEV, dtype=torch.float64)
        x = (2 * p[0] - 1) * 0.8 * half + v[0] * f
        y = (2 * p[1] - 1) * 0.8 * half + v[1] * f
        z = gr.z0 + (0.1 + 0.8 * p[2]) * (c["nz"] - 1) * gr.dz + v[2] * f
        u, w = torch.stack([x, y], 1)[:, :, None, None], torch.stack([y, x], 1)[:, :, None, None]
        zz = z[:, None, None, None]
        a = ang[None, None, :, None]
        tau = (zz * torch.cos(a) + w * torch.sin(a) + 0.5 * L * torch.sin(a).abs()
               + torch.sqrt((u - ue) ** 2 + zz ** 2)) / C0                   # [F][2][K][Nc]
        s = (tau - cfg.seq.t_start) * FS
        at = torch.floor(s)[..., None] + torch.arange(-8, 10, device=DEV)
        val = torch.polar(torch.exp(-((at - s[..., None]) / (FS * sig)) ** 2 / 2),
                          (-2 * math.pi * F0 * tau)[..., None].expand_as(at)).to(torch.complex64)
        ok = (at >= 0) & (at < Ns)
        idx = (rows * Ns + at.long())[ok]
        view = flat.view(-1)
        view[idx] = view[idx] + val[ok]
    return iq


def _train_batch(c, seed):
    """Normalised images [B][Nz][Nu], and the microbubbles in them."""
    g = _gen(seed)
    B, nz, nu = c["batch"], c["nz"], c["nu"]
    x = _smooth_(_cnoise((B, nz, nu), g))
    n = max(4, nz * nu // 40)                  # about 1700 a paper-scale image
    zu = torch.rand(B, n, 2, device=DEV, generator=g) * torch.tensor([nz - 1.0, nu - 1.0], device=DEV)
    img = torch.arange(B, device=DEV, dtype=torch.int32).repeat_interleave(n)
    flat = x.view(B, -1)
    b = torch.arange(B, device=DEV)
    for i in range(min(n, 200)):               # the stronger ones leave a spot in the image
        cz, cu = zu[:, i, 0], zu[:, i, 1]
        iz, iu = torch.floor(cz).long(), torch.floor(cu).long()
        for p in range(-2, 4):
            for q in range(-2, 4):
                zi, ui = (iz + p).clamp(0, nz - 1), (iu + q).clamp(0, nu - 1)
                r2 = (zi - cz) ** 2 + (ui - cu) ** 2
                flat[b, zi * nu + ui] += 5.0 * torch.exp(-r2 / (2 * 1.2 ** 2))
    images = x.abs()
    images /= images.amax(dim=(1, 2), keepdim=True)
    return images.contiguous(), zu.view(-1, 2).contiguous(), img


def _weights():
    return torch.from_numpy(np.load(WEIGHTS).astype(np.float32)).to(DEV)


def _adam_state(seed):
    g = _gen(seed + 77)
    m = 1e-5 * torch.randn(ulm.ULM_CNN_PARAMS, device=DEV, generator=g)
    v = 1e-9 * (0.5 + torch.rand(ulm.ULM_CNN_PARAMS, device=DEV, generator=g))
    return m, v


ADAM_STEP, LEARNING_RATE = 1000, 5e-4     # somewhere inside a training run


# ------------------------------------------------------------------ prepare and run

def _capacity(c):
    return 4096 + 2 * c["blocks"] * c["frames"] * c["nz"] * c["nu"] // 24


def _record_buffers(s, c):
    s.cap = _capacity(c)
    s.locs = torch.zeros((s.cap, 8), dtype=torch.int32, device=DEV)
    s.count = torch.zeros(1, dtype=torch.int32, device=DEV)


def prepare(case, seed):
    c, s = case, SimpleNamespace(case=case)
    op = c["op"]
    if op == "cnn_train":
        s.images, s.zu, s.img = _train_batch(c, seed)
        s.params = _weights()
        s.m, s.v = _adam_state(seed)
        s.loss = torch.zeros(1, device=DEV)
        s.prec = ulm.ULM_CNN_FP32 if c["train"] == "fp32" else ulm.ULM_CNN_BF16
        s.ws = ulm.Workspace(ulm.ulm_cnn_workspace_size(c["batch"], c["nz"], c["nu"], s.prec, True),
                             DEV)
        return s
    s.ctx = _context(c)
    if op == "path":
        s.iq = _iq(c, seed)
        s.planes = torch.zeros(s.ctx.proj_shape, dtype=torch.complex64, device=DEV)
        s.eig = torch.zeros(s.ctx.proj_shape[:3], dtype=torch.float64, device=DEV)
        _record_buffers(s, c)
    elif op in ("stage2", "xdoppler"):
        _slices(c, seed, ulm.ulm_stage1_slices(s.ctx))
        s.planes = torch.zeros(s.ctx.proj_shape, dtype=torch.complex64, device=DEV)
        if op == "xdoppler":
            s.cross = torch.zeros_like(s.planes)
            s.out = torch.zeros_like(s.planes)
            s.eig = torch.zeros(s.ctx.proj_shape[:3], dtype=torch.float64, device=DEV)
    elif op == "motion":
        s.slices = _moving_slices(c, seed, ulm.ulm_stage1_slices(s.ctx))
        s.disp = torch.zeros((2, c["angles"], c["frames"], 2), device=DEV)
        s.motion = torch.zeros((c["frames"], 3), device=DEV)
        s.ws = ulm.Workspace(ulm.ulm_motion_workspace_size(s.ctx, c["lag"]), DEV)
    elif op == "filter":
        s.raw = _planes(c, seed, filtered=False)
        s.planes = torch.zeros_like(s.raw)
        s.eig = torch.zeros(s.ctx.proj_shape[:3], dtype=torch.float64, device=DEV)
    else:
        s.planes = _planes(c, seed, filtered=True)
        if op == "separate":
            s.subsets = torch.zeros((2 * c["speeds"],) + tuple(s.ctx.proj_shape),
                                    dtype=torch.complex64, device=DEV)
        else:
            _record_buffers(s, c)
        if op == "detect3d":
            s.out_cap = s.cap // 2
            s.pairs = torch.zeros((s.out_cap, 8), dtype=torch.int32, device=DEV)
            s.pair_count = torch.zeros(1, dtype=torch.int32, device=DEV)
            s.ws = ulm.Workspace(ulm.ulm_pair_workspace_size(s.ctx, s.cap), DEV)
        if op == "cnn_localize":
            s.params = _weights()
            s.ws = ulm.Workspace(ulm.ulm_cnn_localize_workspace_size(s.ctx, 64), DEV)
    return s


def _records(s):
    """The 32-byte records as what they are: four integers and four floats each."""
    return {"where": s.locs[:, :4], "values": s.locs[:, 4:].view(torch.float32), "count": s.count}


def run(s):
    c, op = s.case, s.case["op"]
    if op == "path":
        ulm.ulm_reconstruct_ensemble(s.ctx, s.iq, s.cap, s.planes, s.eig, s.locs, s.count)
        out = {"planes": s.planes, "eigvals": s.eig}
        # Detections are yes/no decisions on the filtered planes.  In a large ensemble some of
        # the millions of pixels always lie within one rounding of a decision, so there the
        # planes stand for them (the localisers' own cases return every record).
        if c["frames"] * c["nz"] * c["nu"] <= 200_000:
            out.update(_records(s))
        return out
    if op == "stage2":
        return ulm.rca_beamform_stage2(s.ctx, s.planes)
    if op == "filter":
        # the filter works in place and this program keeps the unfiltered planes
        s.planes.copy_(s.raw)
        ulm.svd_clutter_filter(s.ctx, s.planes, s.eig)
        return {"planes": s.planes, "eigvals": s.eig}
    if op == "xdoppler":
        ulm.rca_beamform_stage2(s.ctx, s.planes)
        ulm.rca_beamform_cross(s.ctx, s.cross)
        ulm.svd_clutter_filter(s.ctx, s.planes, s.eig)
        ulm.svd_clutter_filter(s.ctx, s.cross, s.eig)
        return ulm.ulm_xdoppler(s.ctx, s.planes, s.cross, c["window"], s.out)
    if op == "motion":
        ulm.ulm_motion_estimate(s.ctx, s.slices, 0, c["lag"], s.disp, s.motion, s.ws)
        return {"disp": s.disp, "motion": s.motion}
    if op == "separate":
        return ulm.ulm_separate(s.ctx, s.planes, c["speeds"], s.subsets)
    if op == "ncc":
        ulm.ncc_localize(s.ctx, s.planes, s.cap, s.locs, s.count)
        return _records(s)
    if op == "detect3d":
        ulm.ncc_localize(s.ctx, s.planes, s.cap, s.locs, s.count)
        ulm.ulm_pair_planes(s.ctx, s.locs, s.count, s.cap, s.out_cap, s.pairs, s.pair_count, s.ws)
        out = _records(s)
        out.update(frame=s.pairs[:, 0], position=s.pairs[:, 1:6].view(torch.float32),
                   members=s.pairs[:, 6:], pair_count=s.pair_count)
        return out
    if op == "cnn_localize":
        ulm.ulm_cnn_localize(s.ctx, s.params, s.planes, s.cap, ulm.CNN_THRESHOLD, 64,
                             ulm.ULM_CNN_BF16, s.locs, s.count, s.ws)
        return _records(s)
    ulm.ulm_cnn_train_step(s.params, s.m, s.v, ADAM_STEP, LEARNING_RATE, s.images, s.zu, s.img,
                           s.prec, s.loss, s.ws)
    return {"params": s.params, "m": s.m, "v": s.v, "loss": s.loss}


# ------------------------------------------------------------------ work

def _taps(c):
    """Stage-2 filter taps per output pixel, over all transmits and slabs."""
    cfg = _config(c)
    n = 0
    for a in cfg.seq.angles_deg:
        t = math.tan(math.radians(a) / 2)
        for lo, hi in _slab_ranges(c):
            sh = [math.floor((cfg.grid.v0 + m * cfg.grid.dv) * t / cfg.grid.dz) for m in range(lo, hi)]
            if sh:
                n += max(sh) - min(sh) + (2 if t != 0.0 else 1)
    return n


def _filter_flops(c, planes):
    npix, F, cut = c["nz"] * c["nu"], c["frames"], c["cutoff"]
    return planes * (8.0 * npix * F * (F + 1) / 2 + 16.0 * npix * F * cut + 16.0 / 3 * F ** 3)


def work(c):
    op = c["op"]
    npix, F, K, B = c["nz"] * c["nu"], c["frames"], c["angles"], c["blocks"]
    stack = 8.0 * 2 * B * F * npix              # one stack of planes
    slices = 8.0 * 2 * K * F * npix
    pixels = 2.0 * B * F * npix                 # image pixels
    ncc_flops = pixels * (12.0 * c["ncc"] + 20)
    if op == "path":
        iq = 8.0 * F * 2 * K * c["elems"] * _config(c).seq.n_samp
        flops = (12.0 * 2 * K * F * npix * c["elems"] + 8.0 * 2 * F * npix * _taps(c)
                 + _filter_flops(c, 2 * B) + ncc_flops)
        return {"bytes": iq + stack + 8.0 * 2 * B * F, "flops": flops}
    if op == "stage2":
        return {"bytes": slices + stack, "flops": 8.0 * 2 * F * npix * _taps(c)}
    if op == "filter":
        return {"bytes": 2 * stack, "flops": _filter_flops(c, 2 * B)}
    if op == "xdoppler":
        return {"bytes": slices + stack, "flops": 2 * _filter_flops(c, 2 * B)
                + 8.0 * 2 * F * npix * _taps(c) + pixels * (8.0 * K * 2 + 20)}
    if op == "motion":
        lags = (2 * c["lag"] + 1) ** 2
        per = min(2.0 * lags, 10.0 * math.log2(npix))
        return {"bytes": slices, "flops": 2.0 * K * F * npix * per}
    if op == "separate":
        sub = 2 * c["speeds"]
        return {"bytes": (1 + sub) * stack, "flops": pixels * (1 + sub) * 5 * math.log2(F)}
    if op in ("ncc", "detect3d"):
        return {"bytes": stack, "flops": ncc_flops}
    macs = 32 * 9 + 5 * 32 * 288 + 64 * 32
    if op == "cnn_localize":
        return {"bytes": stack, "flops": pixels * 2.0 * macs}
    px = float(c["batch"] * npix)
    return {"bytes": 4.0 * px + 7 * 4.0 * ulm.ULM_CNN_PARAMS, "flops": px * 6.0 * macs}


# ------------------------------------------------------------------ exact values

def _fir_matrices(c, lo, hi):
    """[K][Nz][Nz] complex128: stage 2 of the slices v in [lo, hi) as a matrix along depth."""
    cfg = _config(c)
    g, nz = cfg.grid, c["nz"]
    out = np.zeros((c["angles"], nz, nz), dtype=np.complex128)
    row = np.arange(nz)
    for k, a in enumerate(cfg.seq.angles_deg):
        t = math.tan(math.radians(a) / 2)
        for m in range(lo, hi):
            out[k] += _shift_matrix((g.v0 + m * g.dv) * t, g.dz, nz, row)
    return torch.from_numpy(out).to(DEV)


def _shift_matrix(dz_m, dz, nz, row):
    m = np.zeros((nz, nz), dtype=np.complex128)
    phase = np.exp(4j * math.pi * F0 * dz_m / C0)
    shift = dz_m / dz
    n0 = int(math.floor(shift))
    for w, off in ((1.0 - (shift - n0), n0), (shift - n0, n0 + 1)):
        ok = (row + off >= 0) & (row + off < nz)
        m[row[ok], row[ok] + off] += w * phase
    return m


def _exact_stage2(c, slices):
    out = torch.zeros((2, c["blocks"], c["frames"], c["nz"], c["nu"]), dtype=torch.complex128,
                      device=DEV)
    mats = [_fir_matrices(c, lo, hi) if lo < hi else None for lo, hi in _slab_ranges(c)]
    for o in range(2):
        for k in range(c["angles"]):
            s = slices[o, k].to(torch.complex128).permute(1, 0, 2).reshape(c["nz"], -1)
            for b, m in enumerate(mats):
                if m is not None:
                    p = torch.mm(m[k], s).view(c["nz"], c["frames"], c["nu"])
                    out[o, b] += p.permute(1, 0, 2)
    return out


def _exact_cross(c, slices):
    cfg, nz, nu, F = _config(c), c["nz"], c["nu"], c["frames"]
    g, row = cfg.grid, np.arange(nz)
    out = torch.zeros((2, 1, F, nz, nu), dtype=torch.complex128, device=DEV)
    for k, a in enumerate(cfg.seq.angles_deg):
        t = math.tan(math.radians(a) / 2)
        prof = slices[:, k].to(torch.complex128).sum(dim=3)                   # [2][F][Nz]
        m = np.stack([_shift_matrix((g.v0 + i * g.dv) * t, g.dz, nz, row) for i in range(nu)], 1)
        m = torch.from_numpy(m.reshape(nz * nu, nz)).to(DEV)
        for o in range(2):
            out[o, 0] += torch.mm(prof[1 - o].contiguous(), m.t().contiguous()).view(F, nz, nu)
    return out


def _exact_filter(c, planes):
    out = torch.zeros(planes.shape, dtype=torch.complex128, device=DEV)
    eig = torch.zeros(planes.shape[:3], dtype=torch.float64)
    F = c["frames"]
    for o in range(2):
        for b in range(planes.shape[1]):
            x = planes[o, b].to(torch.complex128).reshape(F, -1)
            cov = torch.mm(x.conj().resolve_conj(), x.t().contiguous())       # C = I^H I
            lam, vec = torch.linalg.eigh(cov.cpu())
            eig[o, b] = lam.flip(0)
            v = vec.flip(1)[:, :c["cutoff"]].to(DEV)
            y = torch.mm(v.t().contiguous(), x)                              # (I V)^T
            out[o, b] = (x - torch.mm(v.conj().resolve_conj().contiguous(), y)).view(planes.shape[2:])
    return out, eig


def _exact_stage1(c, iq):
    cfg = _config(c)
    g, F, K, Nc, Ns = cfg.grid, c["frames"], c["angles"], c["elems"], cfg.seq.n_samp
    z = g.z0 + torch.arange(c["nz"], device=DEV, dtype=torch.float64)[:, None] * g.dz
    u = g.u0 + torch.arange(c["nu"], device=DEV, dtype=torch.float64)[None, :] * g.du
    L = (Nc - 1) * cfg.probe.pitch
    out = torch.zeros((2, K, F, c["nz"], c["nu"]), dtype=torch.complex128, device=DEV)
    for k, a in enumerate(cfg.seq.angles_deg):
        th = math.radians(a)
        tx = (z * math.cos(th) + 0.5 * L * abs(math.sin(th))) / C0
        for e in range(Nc):
            ue = (e - 0.5 * (Nc - 1)) * cfg.probe.pitch
            tau = tx + torch.sqrt((u - ue) ** 2 + z ** 2) / C0
            s = (tau - cfg.seq.t_start) * FS
            i0 = torch.floor(s)
            fr = (s - i0).reshape(-1)
            i0 = i0.long().reshape(-1)
            ph = 2 * math.pi * F0 * (tau - 2 * z / C0)
            ph = torch.polar(torch.ones_like(ph), ph).reshape(-1)
            w0 = torch.where((i0 >= 0) & (i0 < Ns), 1 - fr, torch.zeros_like(fr)) * ph
            w1 = torch.where((i0 + 1 >= 0) & (i0 + 1 < Ns), fr, torch.zeros_like(fr)) * ph
            a0, a1 = i0.clamp(0, Ns - 1), (i0 + 1).clamp(0, Ns - 1)
            for o in range(2):
                row = iq[:, o, k, e].to(torch.complex128)
                out[o, k] += (row[:, a0] * w0 + row[:, a1] * w1).view(F, c["nz"], c["nu"])
    return out


def _exact_peak(win, lag):
    """Sub-pixel peak of NCC windows [n][2L+1][2L+1] (float64, decided on their FP32 values)."""
    n, W = win.shape[0], 2 * lag + 1
    w = win.to(torch.float32)
    flat = w.view(n, -1)
    top = flat.max(dim=1, keepdim=True).values
    k = (flat == top).to(torch.int32).argmax(dim=1)
    iz, iu = k // W, k % W
    r = torch.arange(n, device=w.device)

    def fit(lo, mid, hi, edge):
        lo, mid, hi = lo.double(), mid.double(), hi.double()
        pos = (lo > 0) & (mid > 0) & (hi > 0)
        a, b, d = (torch.where(pos, torch.log(torch.where(pos, t, torch.ones_like(t))), t)
                   for t in (lo, mid, hi))
        curv = a - 2 * b + d
        off = torch.where(curv < 0, 0.5 * (a - d) / torch.where(curv < 0, curv, -torch.ones_like(curv)),
                          torch.zeros_like(curv)).clamp(-0.5, 0.5)
        return torch.where(edge, torch.zeros_like(off), off)

    def at(z, u):
        return w[r, z.clamp(0, W - 1), u.clamp(0, W - 1)]

    dz = (iz - lag) + fit(at(iz - 1, iu), at(iz, iu), at(iz + 1, iu), (iz == 0) | (iz == W - 1))
    du = (iu - lag) + fit(at(iz, iu - 1), at(iz, iu), at(iz, iu + 1), (iu == 0) | (iu == W - 1))
    return torch.stack([dz.double(), du.double()], dim=1)


def _exact_motion(c, slices):
    lag, nz, nu = c["lag"], c["nz"], c["nu"]
    disp = torch.zeros((2, c["angles"], c["frames"], 2), dtype=torch.float64, device=DEV)
    lz = torch.arange(-lag, lag + 1, device=DEV) % nz
    lu = torch.arange(-lag, lag + 1, device=DEV) % nu
    for o in range(2):
        for k in range(c["angles"]):
            a = slices[o, k].to(torch.complex128).abs()
            a = a - a.mean(dim=(1, 2), keepdim=True)
            nrm = a.square().sum(dim=(1, 2)).sqrt()
            A = torch.fft.fft2(a.to(torch.complex128))
            cc = torch.fft.ifft2(A * A[0].conj()[None]).real
            win = cc[:, lz][:, :, lu] / (nrm * nrm[0]).view(-1, 1, 1)
            disp[o, k] = _exact_peak(win, lag)
    mean = disp.mean(dim=1)
    return {"disp": disp, "motion": torch.stack(
        [mean[0, :, 1], mean[1, :, 1], 0.5 * (mean[0, :, 0] + mean[1, :, 0])], dim=1)}


def _exact_separate(c, planes):
    F, S = c["frames"], c["speeds"]
    H = (F - 1) // 2
    X = torch.fft.fft(planes.to(torch.complex128), dim=2)
    out = torch.zeros((2 * S,) + tuple(planes.shape), dtype=torch.complex128, device=DEV)
    for d, sign in enumerate((1, -1)):
        for s in range(S):
            mask = torch.zeros(F, device=DEV, dtype=torch.float64)
            mask[[(sign * m) % F for m in range(1 + s * H // S, 1 + (s + 1) * H // S)]] = 1.0
            out[d * S + s] = torch.fft.ifft(X * mask.view(1, 1, F, 1, 1), dim=2)
    return out


def _conv3x3(x, w, b):
    """x [B][H][W][Cin], w [Cout][Cin][3][3]; zero padding."""
    B, H, W, cin = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b
    for i in range(3):
        for j in range(3):
            t = torch.mm(xp[:, i:i + H, j:j + W].reshape(-1, cin), w[:, :, i, j].t().contiguous())
            y = y + t
    return y.view(B, H, W, -1)


def _exact_train(c, seed):
    images, zu, img = _train_batch(c, seed)
    B, nz, nu = images.shape
    params = _weights().double().requires_grad_(True)
    at, p = 0, {}
    for name, shape in ulm.CNN_LAYOUT:
        n = int(np.prod(shape))
        p[name] = params[at:at + n].view(shape)
        at += n
    x = images.double()[..., None]
    for l in range(6):
        x = torch.relu(_conv3x3(x, p["w%d" % l], p["b%d" % l]))
    head = torch.mm(x.reshape(-1, 32), p["wh"].t().contiguous()) + p["bh"]
    heat = head.view(B, nz, nu, 8, 8).permute(0, 1, 3, 2, 4).reshape(B, 8 * nz, 8 * nu)
    T = torch.zeros(B * 64 * nz * nu, dtype=torch.float64, device=DEV)
    cz = 8 * (zu[:, 0].double() + 0.5) - 0.5
    cu = 8 * (zu[:, 1].double() + 0.5) - 0.5
    fz, fu = torch.floor(cz).long(), torch.floor(cu).long()
    for a in range(-4, 6):
        for b in range(-4, 6):
            qz, qu = fz + a, fu + b
            ok = (qz >= 0) & (qz < 8 * nz) & (qu >= 0) & (qu < 8 * nu)
            val = torch.exp(-((qz - cz) ** 2 + (qu - cu) ** 2) / 2)
            idx = (img.long() * 8 * nz + qz) * 8 * nu + qu
            T.scatter_reduce_(0, idx[ok], val[ok], "amax")
    loss = (heat - T.view_as(heat)).square().mean()
    loss.backward()
    gr = params.grad
    m, v = _adam_state(seed)
    m = 0.9 * m.double() + 0.1 * gr
    v = 0.999 * v.double() + 0.001 * gr * gr
    mh, vh = m / (1 - 0.9 ** ADAM_STEP), v / (1 - 0.999 ** ADAM_STEP)
    new = params.detach() - LEARNING_RATE * mh / (vh.sqrt() + 1e-8)
    return {"params": new, "m": m, "v": v, "loss": loss.detach().view(1)}


def exact(case, seed):
    c, op = case, case["op"]
    if op in ("ncc", "detect3d", "cnn_localize"):
        return None                 # decisions; the values belong to the records decided on
    if op == "cnn_train":
        return _exact_train(c, seed)
    shape = (2, c["angles"], c["frames"], c["nz"], c["nu"])
    if op == "path":
        if 2.0 * c["angles"] * c["frames"] * c["nz"] * c["nu"] * c["elems"] > 8e9:
            return None             # minutes in 64 bits
        planes, eig = _exact_filter(c, _exact_stage2(c, _exact_stage1(c, _iq(c, seed))))
        out = {"planes": planes, "eigvals": eig}
        if c["frames"] * c["nz"] * c["nu"] <= 200_000:
            out.update(where=None, values=None, count=None)
        return out
    if op == "filter":
        planes, eig = _exact_filter(c, _planes(c, seed, filtered=False))
        return {"planes": planes, "eigvals": eig}
    if op == "separate":
        return _exact_separate(c, _planes(c, seed, filtered=True))
    slices = torch.zeros(shape, dtype=torch.complex64, device=DEV)
    if op == "motion":
        return _exact_motion(c, _moving_slices(c, seed, slices))
    _slices(c, seed, slices)
    if op == "stage2":
        return _exact_stage2(c, slices)
    P, _ = _exact_filter(c, _exact_stage2(c, slices))
    Q, _ = _exact_filter(c, _exact_cross(c, slices))
    h = (c["window"] - 1) // 2
    prod = P * Q.conj()
    out = torch.zeros_like(prod)
    F = c["frames"]
    for f in range(F):
        out[:, :, f] = prod[:, :, max(0, f - h):min(F, f + h + 1)].sum(dim=2).abs().sqrt()
    return out
