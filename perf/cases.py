"""Performance cases of the event-based 4D-STEM library: what its users run, over the range of
scan sizes, detectors, doses, options and entry points they run it with.

A case is a dict of plain values.  `listed()` names the fixed cases, `draw(rng)` makes one more of
the same ranges, `prepare(case, seed)` builds what a program holds before the call (events on the
GPU, the state buffer, the output buffers), `run(state)` is one pass through the public entry
points, `work(case)` the bytes and operations a pass cannot do without (each input read once, each
output written once) and `exact(case, seed)` the outputs of the same pass in 64-bit torch.

Kinds of case (entry points):
  step      com_dpc (centre of mass + DPC phase) and SsbState.oneshot (sideband phase and T): an
            acquisition reconstructed by both methods
  stream    the same in chunks of scan rows as they arrive: accumulate with the centre of mass from
            the same pass over the events, then the DPC integration and finalize
  refocus   new aberration coefficients and probe phase on a finalized state: the interactive slider
  gradient  loss and gradients through SSBPhase (autograd): one step of an aberration fit
  detect    virtual bright-field / dark-field detectors and the sum of all frames
  recode    run-length events to linear indices, then validation of the CSR arrays (ingest)

Geometries are the repository's (576 x 576 detector with a 60 pixel bright-field disk, 64 x 64 with
16 pixels; 0.2 angstrom steps, 300 kV, 25 mrad).  Events are synthetic: Poisson counts per frame,
hits in the bright-field disk, displaced per frame by a smooth phase gradient, and a few per cent
scattered into the dark field, sorted inside each frame as the detector delivers them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2104_06336_amd as stem

LAM, ALPHA, STEP = 0.0196875, 0.025, 0.2
ABERR = (50.0, 20.0, 20.0, 300.0, 300.0, 300.0, 300.0, 1.0e4)  # of the aberrated workload
NO_ABERR = (0.0,) * 8
DPC = (0.5, 0.0, 0.0, 10)
RADIUS = {64: 16.0, 576: 60.0}
PRECISION = {"fp32": stem.STEM_FFT_FP32, "bf16": stem.STEM_DFT_BF16_SPLIT, "fp16": stem.STEM_DFT_FP16_SPLIT}
G_MODE = {"store": stem.STEM_G_STORE, "recompute": stem.STEM_G_RECOMPUTE}


def _case(kind, ny, nx, det, bin_, mean_e, g="store", precision="fp32", aberr=False, d_bits=8, normalize=0,
          scratch_mib=0, chunk_rows=0, n_det=0, **name):
    return dict(name, kind=kind, ny=ny, nx=nx, det=det, bin=bin_, mean_e=float(mean_e), g=g, precision=precision,
                aberr=aberr, d_bits=d_bits, normalize=normalize, scratch_mib=scratch_mib, chunk_rows=chunk_rows,
                n_det=n_det)


def listed():
    return [
        # the smallest: a live preview of a small scan, latency and launches count
        _case("step", 64, 64, 576, 8, 40, g="recompute", name="preview 64x64"),
        # small and ragged, unbinned: every bright-field pixel kept, 16-bit counts, normalised sum
        _case("step", 96, 160, 64, 1, 20, d_bits=16, normalize=1, name="unbinned 96x160"),
        # ordinary: the 256 x 256 workload with the state class's default options (stored G)
        _case("step", 256, 256, 576, 4, 100, name="step 256x256 stored"),
        # ordinary: aberrated 512 x 512 on the matrix cores, G recomputed in the default scratch
        _case("step", 512, 512, 576, 6, 60, g="recompute", precision="bf16", aberr=True, name="step 512x512 bf16"),
        # the benchmark's workload and options: the largest power-of-two scan
        _case("step", 1024, 1024, 576, 8, 40, g="recompute", scratch_mib=2048, name="step 1024x1024"),
        # a scan whose sides are not powers of two, default options: the largest work
        _case("step", 1000, 1000, 576, 8, 40, name="step 1000x1000 stored"),
        # streaming acquisition, eight chunks of rows, then finalize with aberrations
        _case("stream", 512, 512, 576, 8, 40, aberr=True, chunk_rows=64, name="stream 512x512"),
        # interactive refocus at the largest scan
        _case("refocus", 1024, 1024, 576, 8, 40, aberr=True, name="refocus 1024x1024"),
        # one step of an aberration fit: from the stored values, and with G recomputed
        _case("gradient", 512, 512, 576, 6, 60, aberr=True, name="gradient 512x512 stored"),
        _case("gradient", 256, 256, 576, 6, 60, g="recompute", aberr=True, name="gradient 256x256 recomputed"),
        # Table 1 extras on the largest acquisition: virtual detectors, run-length ingest
        _case("detect", 1024, 1024, 576, 8, 40, n_det=2, name="detectors 1024x1024"),
        _case("recode", 1024, 1024, 576, 8, 40, name="recode 1024x1024"),
    ]


_FAST = (32, 64, 128, 256, 512, 1024)
_OTHER = tuple(n for n in (2 ** a * 3 ** b * 5 ** c for a in range(1, 11) for b in range(5) for c in range(5))
               if 32 <= n <= 2048 and n not in _FAST)


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _near(values, x):
    return min(values, key=lambda v: abs(math.log(v / x)))


def draw(rng):
    while True:
        kind = rng.choice(("step", "step", "step", "stream", "refocus", "gradient", "detect", "recode"))
        fast = rng.random() < 0.6
        ny, nx = (_near(_FAST if fast else _OTHER, _log(rng, 32, 1400)) for _ in range(2))
        if kind in ("detect", "recode"):  # these take any scan
            ny, nx = (int(_log(rng, 32, 1024)) for _ in range(2))
        det = rng.choice((64, 576, 576))
        bin_ = rng.choice((1, 2, 4, 8) if det == 64 else (4, 6, 8, 12))
        c = _case(kind, ny, nx, det, bin_, round(_log(rng, 5, 120), 1), g=rng.choice(("store", "recompute")),
                  precision=rng.choice(("fp32", "fp32", "bf16", "fp16")) if fast else "fp32",
                  aberr=rng.random() < 0.5, d_bits=rng.choice((8, 8, 16)), scratch_mib=rng.choice((0, 0, 256)))
        if kind == "refocus":
            c["g"] = "store"
        if kind == "step" and rng.random() < 0.2:
            c["normalize"] = 1
        if kind == "stream":
            c["chunk_rows"] = max(1, int(_log(rng, ny / 16, ny / 2)))
        if kind == "detect":
            c["n_det"] = rng.choice((1, 2, 4, 8, 16))
        F = ny * nx
        # no costlier than the largest listed case
        if F * c["mean_e"] <= 4.2e7 and F <= 2 ** 20 and F * _num_pixels(c) <= 1.6e8:
            return c


# ----------------------------------------------------------------------------------------------
# geometry


def _optics(case, c=None):
    r = RADIUS[case["det"]]
    c = (ABERR if case["aberr"] else NO_ABERR) if c is None else c
    return stem.Optics.from_values(LAM, r, (ALPHA / LAM) / r, c)


def _structs(case):
    d = case["det"]
    return (stem.Det(d, d, d // 2, d // 2, case["bin"]), stem.Scan(case["ny"], case["nx"], STEP), _optics(case),
            stem.Ssb(PRECISION[case["precision"]], case["normalize"], G_MODE[case["g"]], case["d_bits"],
                     case["scratch_mib"]))


def _centres(case):
    """Kept bins' centres in unbinned pixels (raster order) and the bin index -> kept index table."""
    d, b = case["det"], case["bin"]
    j = np.arange(d // b, dtype=np.float64) * b + 0.5 * (b - 1) - d // 2
    ky, kx = np.meshgrid(j, j, indexing="ij")
    kept = kx * kx + ky * ky < RADIUS[d] ** 2
    lut = np.full(kept.shape, -1, dtype=np.int64)
    lut[kept] = np.arange(int(kept.sum()))
    return kx[kept], ky[kept], lut


def _num_pixels(case):
    return len(_centres(case)[0])


def _annuli(case):
    """Bright field and annular dark field first (the benchmark's), then rings across the detector."""
    r = RADIUS[case["det"]]
    r_in = [0.0, 1.2 * r] + [0.25 * j * r for j in range(14)]
    r_out = [r, 4.0 * r] + [0.25 * (j + 2) * r for j in range(14)]
    return r_in[:case["n_det"]], r_out[:case["n_det"]]


# ----------------------------------------------------------------------------------------------
# inputs


def _events(case, seed, device):
    """CSR events (int32 idx, int64 off): made from the seed alone."""
    g = torch.Generator(device=device)
    g.manual_seed(1000003 * (seed + 1))
    F, d, r = case["ny"] * case["nx"], case["det"], RADIUS[case["det"]]
    # a fixed total over the frames at random: Poisson counts per frame, the same buffer sizes for every seed
    C = round(F * case["mean_e"])
    f = torch.sort(torch.randint(F, (C,), generator=g, device=device))[0]
    off = torch.zeros(F + 1, dtype=torch.int64, device=device)
    torch.cumsum(torch.bincount(f, minlength=F), 0, out=off[1:])
    # the disk's displacement in frame (ry, rx): a smooth phase gradient, up to a tenth of its radius
    a = torch.rand(8, generator=g, device=device, dtype=torch.float64).tolist()
    ry, rx = torch.div(f, case["nx"], rounding_mode="floor").float(), (f % case["nx"]).float()
    w = [0.2 + 0.9 * v for v in a]
    sx = 0.05 * r * (torch.sin(w[0] * rx + 0.3 * w[1] * ry) + torch.sin(0.1 * w[2] * rx - w[3] * ry))
    sy = 0.05 * r * (torch.cos(0.3 * w[4] * rx + w[5] * ry) + torch.sin(w[6] * rx + 0.1 * w[7] * ry))
    rho = r * torch.sqrt(torch.rand(C, generator=g, device=device))
    dark = torch.rand(C, generator=g, device=device) < 0.04
    rho = torch.where(dark, rho * 2.5, rho)
    ang = (2 * math.pi) * torch.rand(C, generator=g, device=device)
    kx = (rho * torch.cos(ang) + sx + (d // 2 + 0.5)).floor().long().clamp_(0, d - 1)
    ky = (rho * torch.sin(ang) + sy + (d // 2 + 0.5)).floor().long().clamp_(0, d - 1)
    key, _ = torch.sort(f * (d * d) + ky * d + kx)
    return (key - f * (d * d)).to(torch.int32).contiguous(), off


def _theta(case, seed, device):
    """A per-pixel probe phase of a few tenths of a radian, and coefficients near the nominal ones."""
    g = torch.Generator(device=device)
    g.manual_seed(7919 * (seed + 1))
    th = 0.2 * torch.randn(_num_pixels(case), generator=g, device=device, dtype=torch.float32)
    u = torch.rand(8, generator=g, device=device, dtype=torch.float64).tolist()
    base = ABERR if case["aberr"] else (10.0,) * 8
    return th, [b * (0.4 + 0.3 * v) for b, v in zip(base, u)]


def prepare(case, seed):
    dev = torch.device("cuda")
    det, scan, optics, ssb = _structs(case)
    F = case["ny"] * case["nx"]
    idx, off = _events(case, seed, dev)
    kind = case["kind"]
    s = {"case": case, "idx": idx, "off": off, "F": F, "det": det, "scan": scan, "optics": optics}

    def out(n, dtype):
        return torch.zeros(n, dtype=dtype, device=dev)

    if kind == "detect":
        s.update(annuli=_annuli(case), det_out=out(case["n_det"] * F, torch.int32),
                 sum=out(case["det"] ** 2, torch.int32), mean=out(case["det"] ** 2, torch.float32),
                 status=stem.status_tensor(dev))
        return s
    if kind == "recode":
        dist = idx.clone()
        dist[1:] -= idx[:-1]
        first = off[:-1][off[1:] > off[:-1]]
        dist[first] = idx[first]
        s.update(dist=dist, idx=torch.empty_like(idx), status=stem.status_tensor(dev))
        return s
    s["st"] = stem.SsbState(det, scan, optics, ssb)
    s["phase"] = out(F, torch.float32)
    if kind in ("step", "stream"):
        s.update(dpc=stem.Dpc(*DPC), T=out(F, torch.complex64), com64=out(2 * F, torch.float64),
                 counts=out(F, torch.int32), dpc_phase=out(F, torch.float32), status=stem.status_tensor(dev),
                 ws=torch.empty(stem.com_dpc_workspace_bytes(scan), dtype=torch.uint8, device=dev))
    else:
        s["theta"], s["c"] = _theta(case, seed, dev)
        if kind == "gradient":
            s["c"] = torch.tensor(s["c"], dtype=torch.float64, requires_grad=True)
            s["theta"].requires_grad_(True)
            s["st"].accumulate(idx, off, 0, F)
        else:
            s["T"] = out(F, torch.complex64)
            s["st"].oneshot(idx, off)
    return s


# ----------------------------------------------------------------------------------------------
# one pass


def run(s):
    case, F = s["case"], s["F"]
    kind = case["kind"]
    if kind == "step":
        stem.com_dpc(s["idx"], s["off"], 0, F, s["det"], s["scan"], s["optics"], s["dpc"], com64=s["com64"],
                     counts=s["counts"], phase=s["dpc_phase"], ws=s["ws"], d_status=s["status"])
        s["st"].oneshot(s["idx"], s["off"], phase=s["phase"], T=s["T"])
    elif kind == "stream":
        rows = case["chunk_rows"]
        for y in range(0, case["ny"], rows):
            n = min(rows, case["ny"] - y)
            s["st"].accumulate(s["idx"], s["off"], y * case["nx"], n * case["nx"], com64=s["com64"],
                               counts=s["counts"])
        stem.com_dpc(s["idx"], s["off"], 0, 0, s["det"], s["scan"], s["optics"], s["dpc"], com64=s["com64"],
                     counts=s["counts"], phase=s["dpc_phase"], ws=s["ws"], d_status=s["status"])
        s["st"].finalize(phase=s["phase"], T=s["T"])
    elif kind == "refocus":
        s["st"].refocus(s["c"], s["theta"], phase=s["phase"], T=s["T"])
        return {"phase": s["phase"], "T": s["T"]}
    elif kind == "gradient":
        phi = stem.SSBPhase.apply(s["c"], s["theta"], s["st"])
        loss = -torch.var(phi, unbiased=False)
        dc, dtheta = torch.autograd.grad(loss, (s["c"], s["theta"]))
        return {"phase": phi.detach(), "dc": dc, "dtheta": dtheta}
    elif kind == "detect":
        r_in, r_out = s["annuli"]
        stem.virtual_annular(s["idx"], s["off"], 0, F, s["det"], s["scan"], r_in, r_out, s["det_out"],
                             d_status=s["status"])
        s["sum"].zero_()
        stem.sum_frames(s["idx"], s["off"], 0, F, s["det"], s["sum"], s["mean"], d_status=s["status"])
        return {"annular": s["det_out"], "sum": s["sum"], "mean": s["mean"], "status": s["status"]}
    else:
        stem.eer_decode_rle(s["dist"], s["off"], 0, F, s["det"], s["idx"], d_status=s["status"])
        stem.eer_load_csr(None, None, 0, F, s["idx"].numel(), s["det"], s["idx"], s["off"], d_status=s["status"])
        return {"idx": s["idx"], "status": s["status"]}
    return {"com64": s["com64"], "counts": s["counts"], "dpc": s["dpc_phase"], "phase": s["phase"], "T": s["T"],
            "status": s["st"].status}


def work(case):
    """Bytes: events and offsets (or the stored double-overlap values) read once, outputs written
    once.  Operations: real 2D FFTs of the kept pixels, 8 per double-overlap pair, one per event."""
    F = case["ny"] * case["nx"]
    C = F * case["mean_e"]
    ev = 4.0 * C + 8.0 * (F + 1)
    kind = case["kind"]
    if kind == "detect":
        return {"bytes": ev + 4.0 * case["n_det"] * F + 8.0 * case["det"] ** 2, "flops": 2.0 * C}
    if kind == "recode":
        return {"bytes": ev + 4.0 * C, "flops": C}
    pairs = _pairs(case)
    fft = 2.5 * _num_pixels(case) * F * math.log2(F)
    if kind == "refocus":
        return {"bytes": 8.0 * pairs + 12.0 * F, "flops": 8.0 * pairs + 5.0 * F * math.log2(F)}
    if kind == "gradient":  # the sum and its adjoint over the stored values, or from the binned counts
        if case["g"] == "store":
            return {"bytes": 16.0 * pairs + 16.0 * F, "flops": 60.0 * pairs}
        return {"bytes": 2.0 * _num_pixels(case) * F * (case["d_bits"] // 8) + 16.0 * F, "flops": fft + 60.0 * pairs}
    return {"bytes": ev + 36.0 * F, "flops": fft + 8.0 * pairs + 2.0 * C}


def _pairs(case):
    """Double-overlap pairs: the scan-frequency lattice's density times, per pixel, the area of the
    disk |K - Q| < r outside |K + Q| < r."""
    r = RADIUS[case["det"]]
    dk = (ALPHA / LAM) / r
    kx, ky, _ = _centres(case)
    h = np.minimum(np.sqrt(kx * kx + ky * ky) / r, 1.0)
    lens = 2 * r * r * (np.arccos(h) - h * np.sqrt(1 - h * h))
    sx, sy = (1.0 / (n * STEP * dk) for n in (case["nx"], case["ny"]))
    return float(np.sum(np.minimum((math.pi * r * r - lens) / (sx * sy), case["ny"] * case["nx"])))


# ----------------------------------------------------------------------------------------------
# the same pass in 64 bits


def _chi(kx, ky, c, dk):
    wx, wy = LAM * (kx * dk), LAM * (ky * dk)
    w2 = wx * wx + wy * wy
    p = (0.5 * c[0] * w2 + 0.5 * c[1] * (wx * wx - wy * wy) + c[2] * wx * wy + c[3] * w2 * wx / 3.0
         + c[4] * w2 * wy / 3.0 + c[5] * (wx * wx * wx - 3.0 * wx * wy * wy) / 3.0
         + c[6] * (3.0 * wx * wx * wy - wy * wy * wy) / 3.0 + 0.25 * c[7] * w2 * w2)
    return (2.0 * math.pi / LAM) * p


def _frequencies(n, device):
    return torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=device).round()


def _com(case, idx, off):
    d, F = case["det"], case["ny"] * case["nx"]
    n = off[1:] - off[:-1]
    f = torch.repeat_interleave(torch.arange(F, device=idx.device), n)
    k = idx.long()
    div = n.clamp(min=1).double()
    out = []
    for v in (k % d - d // 2, torch.div(k, d, rounding_mode="floor") - d // 2):
        out.append(torch.zeros(F, dtype=torch.int64, device=idx.device).index_add_(0, f, v).double() / div)
    return torch.stack(out), n


def _dpc(case, com):
    ny, nx = case["ny"], case["nx"]
    dev = com.device
    mu, lam1, lam2, n_iter = DPC
    gr = 2.0 * math.pi * ((ALPHA / LAM) / RADIUS[case["det"]]) * com.reshape(2, ny, nx)
    Gx, Gy = torch.fft.fft2(gr[0].to(torch.complex128)), torch.fft.fft2(gr[1].to(torch.complex128))
    qy = (2 * math.pi * _frequencies(ny, dev) / (ny * STEP))[:, None]
    qx = (2 * math.pi * _frequencies(nx, dev) / (nx * STEP))[None, :]
    q2 = qx * qx + qy * qy
    den = lam1 + q2 + lam2 * q2 * q2
    live = den != 0
    live[ny // 2, :] = False
    live[:, nx // 2] = False
    den = torch.where(live, den, torch.ones_like(den))
    phi = torch.zeros_like(Gx)
    for _ in range(n_iter):
        step = -1j * qx * (Gx - 1j * qx * phi) - 1j * qy * (Gy - 1j * qy * phi)
        phi = torch.where(live, phi + mu * step / den, torch.zeros_like(phi))
    return torch.fft.ifft2(phi).real


class _Sideband:
    """Pixel by pixel: G (2D FFT of the binned counts), the double-overlap set and the phase psi."""

    def __init__(self, case, idx, off, c, theta):
        dev = idx.device
        self.ny, self.nx = case["ny"], case["nx"]
        F, d, b = self.ny * self.nx, case["det"], case["bin"]
        self.r2 = RADIUS[d] ** 2
        self.dk = (ALPHA / LAM) / RADIUS[d]
        self.kx, self.ky, lut = _centres(case)
        lut = torch.from_numpy(lut).to(dev)
        k = idx.long()
        kd = lut[torch.div(torch.div(k, d, rounding_mode="floor"), b, rounding_mode="floor"),
                 torch.div(k % d, b, rounding_mode="floor")]
        f = torch.repeat_interleave(torch.arange(F, device=dev), off[1:] - off[:-1])
        keep = kd >= 0
        self.D = torch.zeros(len(self.kx) * F, dtype=torch.int32, device=dev)
        self.D.index_add_(0, kd[keep] * F + f[keep], torch.ones(1, dtype=torch.int32, device=dev).expand(int(keep.sum())))
        sx, sy = (1.0 / ((float(n) * STEP) * self.dk) for n in (self.nx, self.ny))
        self.qx = (_frequencies(self.nx, dev) * sx)[None, :]
        self.qy = (_frequencies(self.ny, dev) * sy)[:, None]
        self.c, self.theta = c, theta

    def pixels(self):
        F = self.ny * self.nx
        for j in range(len(self.kx)):
            kx, ky = float(self.kx[j]), float(self.ky[j])
            dx, dy, ux, uy = kx - self.qx, ky - self.qy, kx + self.qx, ky + self.qy
            m = (dx * dx + dy * dy < self.r2) & (ux * ux + uy * uy >= self.r2)
            z = torch.fft.fft2(self.D[j * F:(j + 1) * F].reshape(self.ny, self.nx).to(torch.complex128)) * m
            th = float(self.theta[j]) if self.theta is not None else 0.0
            if self.theta is not None or any(self.c):
                psi = _chi(dx, dy, self.c, self.dk) - _chi(kx, ky, self.c, self.dk) - th
                z = z * torch.polar(torch.ones_like(psi), psi)
            yield j, z, m, (dx, dy, kx, ky)


def exact(case, seed):
    dev = torch.device("cuda")
    F, ny, nx = case["ny"] * case["nx"], case["ny"], case["nx"]
    kind = case["kind"]
    idx, off = _events(case, seed, dev)
    if kind == "recode":
        return {"idx": idx, "status": torch.zeros(1, dtype=torch.int32)}
    if kind == "detect":
        d = case["det"]
        k = idx.long()
        x, y = k % d - d // 2, torch.div(k, d, rounding_mode="floor") - d // 2
        d2 = (x * x + y * y).double()
        f = torch.repeat_interleave(torch.arange(F, device=dev), off[1:] - off[:-1])
        rings = [torch.zeros(F, dtype=torch.int32, device=dev).index_add_(0, f, ((d2 >= a * a) & (d2 < b * b)).int())
                 for a, b in zip(*_annuli(case))]
        total = torch.zeros(d * d, dtype=torch.int64, device=dev).index_add_(0, k, torch.ones_like(k))
        return {"annular": torch.cat(rings), "sum": total.int(), "mean": total.double() / F,
                "status": torch.zeros(1, dtype=torch.int32)}
    th = None
    c = ABERR if case["aberr"] else NO_ABERR
    if kind in ("refocus", "gradient"):
        t, c = _theta(case, seed, dev)
        th = t.double().cpu().numpy()
    sb = _Sideband(case, idx, off, c, th)
    T = torch.zeros(ny, nx, dtype=torch.complex128, device=dev)
    npair = torch.zeros(ny, nx, dtype=torch.int64, device=dev)
    for _, z, m, _ in sb.pixels():
        T += z
        npair += m
    if case["normalize"]:
        T = torch.where(npair > 0, T / npair.clamp(min=1), torch.zeros_like(T))
    phase = torch.fft.ifft2(T).imag
    if kind == "gradient":
        # loss -Var(phase); Tbar = (i/F) FFT2(dL/dphase); w = Re(conj(Tbar) i z) per pair
        g = -(2.0 / F) * (phase - phase.mean())
        tbar = (1j / F) * torch.fft.fft2(g.to(torch.complex128))
        unit = [tuple(1.0 if i == j else 0.0 for i in range(8)) for j in range(8)]
        dc, dth = torch.zeros(8, dtype=torch.float64, device=dev), torch.zeros(len(sb.kx), dtype=torch.float64, device=dev)
        for j, z, _, (dx, dy, kx, ky) in sb.pixels():
            w = (tbar.conj() * 1j * z).real
            for i in range(8):
                dc[i] += (w * (_chi(dx, dy, unit[i], sb.dk) - _chi(kx, ky, unit[i], sb.dk))).sum()
            dth[j] = -w.sum()
        return {"phase": phase, "dc": dc.cpu(), "dtheta": dth}
    if kind == "refocus":
        return {"phase": phase.reshape(-1), "T": T.reshape(-1)}
    com, n = _com(case, idx, off)
    return {"com64": com.reshape(-1), "counts": n.int(), "dpc": _dpc(case, com).reshape(-1), "phase": phase.reshape(-1),
            "T": T.reshape(-1), "status": torch.zeros(1, dtype=torch.int32)}
