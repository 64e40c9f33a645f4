"""The work that users of this framework have it do, as cases that can be timed.

Three kinds of case, each one call of a public entry point on buffers that a
program keeps between calls (plan, S-matrix, workspace, outputs):

  build   Plan.build_smatrix: every plane wave of the beam set through all
          potential slices (returns the S-matrix);
  batch   build_smatrix_batch: the S-matrices of several specimens in one call;
  probe   Plan.probe_outputs (detector sums) or Plan.probe_cbed (diffraction
          patterns) on a resident S-matrix.

Specimens are seeded random atoms in a periodic cell (0.3 A Gaussian phase
blobs, 2 A slices). ``exact`` is the same arithmetic in torch's 64-bit types.
"""
import math

import numpy as np
import torch

DEV = "cuda"
SIGMA_A = 0.3            # standard deviation of an atom's phase blob
Z_CHOICES = (6, 14, 29, 79)
SLICE_A = 2.0


def listed():
    return [
        # --- S-matrix builds, smallest to largest ---------------------------
        # quick look at a small cell: launches and latency count
        dict(name="build_128", kind="build", n=128, H=4, f=2, keV=80.0, alpha=20.0, pixel=0.1),
        # an ordinary small specimen
        dict(name="build_256", kind="build", n=256, H=8, f=2, keV=80.0, alpha=20.0, pixel=0.1),
        # a 3 * 2^k grid of the mixed batches, thick
        dict(name="build_768", kind="build", n=768, H=40, f=6, keV=80.0, alpha=20.0, pixel=0.1),
        # the 1024^2 crystal of the benchmark (200 keV, 25 mrad, 50 slices) at f = 8
        dict(name="build_1024", kind="build", n=1024, H=50, f=8, keV=200.0, alpha=25.0,
             pixel=0.0390625),
        # a large 3 * 2^k grid
        dict(name="build_1536", kind="build", n=1536, H=30, f=12, keV=80.0, alpha=20.0, pixel=0.1),
        # the nanoparticle grid of the benchmark (2048^2, 35 slices) at f = 8
        dict(name="build_2048", kind="build", n=2048, H=35, f=8, keV=80.0, alpha=20.0,
             pixel=0.0390625),
        # several specimens of mixed grids queued together in one call
        dict(name="batch_mixed", kind="batch", sizes="256,384,384,512,576", slices="30,12,24,16,20",
             factors="4,6,8,4,6", keV=80.0, alpha=20.0, pixel=0.1),
        # --- probe steps on a resident S-matrix ------------------------------
        # a few probes of a large specimen (interactive use, serving): latency
        dict(name="probe_few", kind="probe", n=1024, f=4, keV=200.0, alpha=25.0, pixel=0.0390625,
             prec="fp32", out="det", scan="raster", px=5, py=3, bins=16, defocus=0.0),
        # the benchmark's scan: 256 x 256 probes, 16 bins
        dict(name="probe_scan", kind="probe", n=1024, f=4, keV=200.0, alpha=25.0, pixel=0.0390625,
             prec="fp32", out="det", scan="raster", px=256, py=256, bins=16, defocus=0.0),
        # a 3 * 2^k window (W = 96) over a full raster of a mixed-batch specimen
        dict(name="probe_fp16", kind="probe", n=768, f=4, keV=80.0, alpha=20.0, pixel=0.1,
             prec="fp16", out="det", scan="raster", px=192, py=192, bins=3, defocus=0.0),
        # scattered probes over a particle, W = 256, 16-bit operands
        dict(name="probe_bf16", kind="probe", n=2048, f=4, keV=80.0, alpha=20.0, pixel=0.0390625,
             prec="bf16", out="det", scan="disc", px=1024, py=1, bins=1, defocus=30.0),
        # full diffraction patterns (4D-STEM), W = 64, a ragged scan
        dict(name="cbed_64", kind="probe", n=1024, f=8, keV=200.0, alpha=25.0, pixel=0.0390625,
             prec="fp32", out="cbed", scan="raster", px=93, py=61, bins=0, defocus=-40.0),
    ]


GRIDS = (128, 192, 256, 384, 512, 576, 768, 1024, 1152, 1536, 2048)
WINDOWS = (8, 12, 16, 18, 24, 32, 36, 48, 64, 72, 96, 128, 144, 192, 256)


def draw(rng):
    """One more case: any grid and any factor with a supported window."""
    r = rng.random()
    keV, alpha = rng.choice(((80.0, 20.0), (200.0, 25.0)))
    pixel = rng.choice((0.1, 0.08, 0.0390625))
    if r < 0.12:
        sizes = [rng.choice((128, 192, 256, 384, 512, 576)) for _ in range(rng.randint(2, 6))]
        parts = [(n, rng.randint(2, 30), rng.choice(_factors(n, 12))) for n in sizes]
        while True:
            cols = dict(zip(("sizes", "slices", "factors"),
                            (",".join(map(str, c)) for c in zip(*parts))))
            case = dict(kind="batch", **cols, keV=keV, alpha=alpha, pixel=pixel)
            if len(parts) == 1 or work(case)["flops"] <= work(listed()[5])["flops"]:
                return case
            parts.pop()
    n = rng.choice(GRIDS)
    case = dict(kind="build", n=n, f=rng.choice(_factors(n, 16)), keV=keV, alpha=alpha, pixel=pixel)
    while _smatrix_bytes(case) > 3e9:  # many beams on a large grid: a coarser set
        case["f"] = next(g for g in _factors(n, 999) if g > case["f"])
    if r < 0.5:
        case["H"] = round(2 * 30 ** rng.random())
        most = work(listed()[5])["flops"]
        while case["H"] > 1 and work(case)["flops"] > most:
            case["H"] = case["H"] * 2 // 3
        return case
    P = 10 ** (4.6 * rng.random())
    px = max(1, round(math.sqrt(P) * rng.uniform(0.6, 1.6)))
    case.update(kind="probe", prec=rng.choice(("fp32", "fp32", "bf16", "fp16")),
                out=rng.choice(("det", "det", "cbed")), scan=rng.choice(("raster", "disc")), px=px,
                py=max(1, round(P / px)), bins=rng.choice((1, 3, 4, 7, 16, 32)),
                defocus=round(rng.uniform(-60.0, 60.0), 1))
    # scattered probes share less of their windows
    most = work(listed()[8])["flops"] / (6 if case["scan"] == "disc" else 1)

    def large():
        return work(case)["flops"] > most or case["px"] * case["py"] * (n // (2 * case["f"])) ** 2 > 5e8
    while case["py"] > 1 and large():
        case["py"] = case["py"] * 2 // 3
    while case["px"] > 1 and large():
        case["px"] = case["px"] * 2 // 3
    return case


def _smatrix_bytes(case):
    n, f = case["n"], case["f"]
    return 2.0 * n * n * len(_beams(n, f, case["keV"], case["alpha"], case["pixel"])[0])


def _factors(n, most):
    """Interpolation factors that give a supported window (f = 1 only on small grids)."""
    return [f for f in range(1 if n <= 256 else 2 if n <= 576 else 3, most + 1)
            if n % (2 * f) == 0 and n // (2 * f) in WINDOWS]


# ------------------------------------------------------------------ the beam set

def _wavelength(keV):
    return 12.398419843320026 / math.sqrt(keV * (keV + 2.0 * 510.99895000))


def _optics(case):
    return dict(alpha_mrad=case["alpha"], C1_A=case.get("defocus", 0.0), C3_A=0.0)


def _beams(n, f, keV, alpha, pixel):
    """(m, n) pairs of the beam set in lexicographic order and alpha_max (mrad)."""
    dq = 1.0 / (n * pixel)
    ldq = _wavelength(keV) * dq
    amax = alpha + float(f) * ldq * 1e3
    lim = n // (4 * f) + 1
    g = np.arange(-lim, lim + 1)
    m, k = (a.ravel() for a in np.meshgrid(g, g, indexing="ij"))
    k2 = (m * f) ** 2 + (k * f) ** 2
    keep = (16 * k2 < n * n) & (ldq * np.sqrt(k2.astype(np.float64)) <= amax * 1e-3)
    return np.stack([m[keep], k[keep]], axis=1), amax


def _active(n, f, keV, alpha, pixel):
    mn, _ = _beams(n, f, keV, alpha, pixel)
    ldq = _wavelength(keV) / (n * pixel)
    k2 = ((mn * f) ** 2).sum(axis=1).astype(np.float64)
    return np.nonzero(ldq * np.sqrt(k2) <= alpha * 1e-3)[0]


# ------------------------------------------------------------------ inputs

def _phase(n, H, pixel, seed):
    """Projected phases [H][n][n] (float32 values, on the GPU) of random atoms."""
    rng = np.random.default_rng(seed)
    side = n * pixel
    per = max(1, round(0.015 * side * side * SLICE_A))
    xs = torch.arange(n, dtype=torch.float64, device=DEV) * pixel
    out = torch.empty((H, n, n), dtype=torch.float32, device=DEV)
    for p in range(H):
        at = torch.from_numpy(rng.uniform(0.0, side, (2, per))).to(DEV)
        amp = torch.from_numpy(0.05 * rng.choice(np.array(Z_CHOICES), per) ** 0.7).to(DEV)
        d = torch.remainder(xs[None, None, :] - at[:, :, None] + side / 2, side) - side / 2
        g = torch.exp(d * d * (-0.5 / SIGMA_A ** 2))
        out[p] = (g[1].T @ (g[0] * amp[:, None])).to(torch.float32)
    return out


def _smatrix(case, seed):
    """A resident S-matrix [B][n/2][n/2]: the beam set's plane waves through two strong
    slices of a random specimen, at the compact sampling."""
    n, f, pixel = case["n"], case["f"], case["pixel"]
    ns, side = n // 2, n * pixel
    mn, _ = _beams(n, f, case["keV"], case["alpha"], pixel)
    t = torch.exp(1j * _phase(ns, 2, 2 * pixel, seed).to(torch.complex64) * 4.0)
    k = torch.fft.fftfreq(ns, 1.0 / ns, dtype=torch.float64, device=DEV)
    prop = torch.exp(-1j * math.pi * _wavelength(case["keV"]) * 8.0 *
                     (k[:, None] ** 2 + k[None, :] ** 2) / side ** 2).to(torch.complex64)
    x = torch.arange(ns, dtype=torch.float64, device=DEV) * (2.0 * math.pi / ns)
    S = torch.empty((len(mn), ns, ns), dtype=torch.complex64, device=DEV)
    m = torch.from_numpy(mn).to(DEV).to(torch.float64) * f
    step = max(1, (1 << 27) // (ns * ns * 8))
    for b in range(0, len(mn), step):
        ex = torch.exp(1j * m[b:b + step, 0, None] * x[None, :]).to(torch.complex64)
        ey = torch.exp(1j * m[b:b + step, 1, None] * x[None, :]).to(torch.complex64)
        w = ey[:, :, None] * ex[:, None, :] * t[0]
        S[b:b + step] = torch.fft.ifft2(torch.fft.fft2(w) * prop) * t[1]
    return S


def _probes(case, seed):
    """Probe positions (A) as a program hands them over: neighbours together."""
    n, f, pixel = case["n"], case["f"], case["pixel"]
    side, px, py = n * pixel, case["px"], case["py"]
    if case["scan"] == "raster":  # two S-pixels apart, in 8 x 8 patches
        step = min(4 * pixel, side / max(px, py))
        j, i = (a.ravel() for a in np.meshgrid(np.arange(py), np.arange(px), indexing="ij"))
        order = np.lexsort((i, j, i // 8, j // 8))
        origin = np.random.default_rng([seed, 7]).uniform(0.0, side, 2)
        return np.stack([i[order] * step + origin[0], j[order] * step + origin[1]], axis=1)
    rng = np.random.default_rng([seed, 9])
    r = side / 4 * np.sqrt(rng.uniform(0.0, 1.0, px * py))
    t = rng.uniform(0.0, 2.0 * np.pi, px * py)
    xy = np.stack([side / 2 + r * np.cos(t), side / 2 + r * np.sin(t)], axis=1)
    c = (xy / (2 * pixel * max(1, min(16, n // (16 * f))))).astype(np.int64)
    key = np.zeros(len(c), dtype=np.int64)
    for b in range(16):
        key |= (c[:, 0] >> b & 1) << (2 * b) | (c[:, 1] >> b & 1) << (2 * b + 1)
    return xy[np.argsort(key, kind="stable")]


def _edges(case):
    """Contiguous annular bins up to a little past the half-band angle."""
    top = 1.1e3 * _wavelength(case["keV"]) / (4 * case["pixel"])
    e = np.linspace(0.0, top, max(1, case["bins"]) + 1)
    return np.stack([e[:-1], e[1:]], axis=1) if case["bins"] > 1 else np.array([[0.3 * top, top]])


def _parts(case):
    """The (n, H, f) of every specimen of a build or batch case."""
    if case["kind"] == "build":
        return [(case["n"], case["H"], case["f"])]
    return list(zip(*([int(v) for v in case[k].split(",")] for k in ("sizes", "slices", "factors"))))


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    from paper_1702_01904_amd import Plan, build_batch_workspace_bytes
    if case["kind"] == "probe":
        n, f = case["n"], case["f"]
        plan = Plan(n, n * case["pixel"], case["keV"], np.full(2, SLICE_A))
        plan.set_probe_precision(case["prec"])
        amax, o = plan.alpha_max_default(case["alpha"], f), _optics(case)
        xy = torch.from_numpy(_probes(case, seed)).to(DEV)
        P, W = len(xy), n // (2 * f)
        out = torch.empty((P, W, W), dtype=torch.float32, device=DEV) if case["out"] == "cbed" \
            else torch.empty((P, len(_edges(case))), dtype=torch.float64, device=DEV)
        ws = torch.empty(plan.probe_workspace_bytes(f, amax, o)[0], dtype=torch.uint8, device=DEV)
        return dict(case=case, plan=plan, f=f, amax=amax, optics=o, xy=xy, out=out, ws=ws,
                    S=_smatrix(case, seed), edges=_edges(case))
    items = []
    for i, (n, H, f) in enumerate(_parts(case)):
        plan = Plan(n, n * case["pixel"], case["keV"], np.full(H, SLICE_A))
        plan.set_potential_slices(_phase(n, H, case["pixel"], [seed, i]))
        amax = plan.alpha_max_default(case["alpha"], f)
        S = torch.empty((plan.beam_count(f, amax), n // 2, n // 2), dtype=torch.complex64,
                        device=DEV)
        items.append((plan, f, amax, S))
    size = items[0][0].build_workspace_bytes(*items[0][1:3])[0] if case["kind"] == "build" \
        else build_batch_workspace_bytes(items)[0]
    return dict(case=case, items=items, ws=torch.empty(size, dtype=torch.uint8, device=DEV))


def run(state):
    case = state["case"]
    if case["kind"] == "build":
        plan, f, amax, S = state["items"][0]
        plan.build_smatrix(f, amax, S, state["ws"])
        return S
    if case["kind"] == "batch":
        from paper_1702_01904_amd import build_smatrix_batch
        build_smatrix_batch(state["items"], state["ws"])
        return [it[3] for it in state["items"]]
    args = (state["f"], state["amax"], state["S"], state["xy"], state["optics"])
    if case["out"] == "cbed":
        state["plan"].probe_cbed(*args, state["out"], state["ws"])
    else:
        state["plan"].probe_outputs(*args, state["edges"], state["out"], state["ws"])
    return state["out"]


def work(case):
    if case["kind"] != "probe":
        b = fl = 0.0
        for n, H, f in _parts(case):
            B = len(_beams(n, f, case["keV"], case["alpha"], case["pixel"])[0])
            b += 4.0 * H * n * n + 2.0 * B * n * n          # phases in, S-matrix out
            # a slice step: two 2D transforms (half of the columns are kept) and two products
            fl += B * H * (2 * 0.75 * 5.0 * n * n * 2 * math.log2(n) + 6.0 * n * n * 1.5)
        return dict(bytes=b, flops=fl)
    n, f = case["n"], case["f"]
    W, P = n // (2 * f), case["px"] * case["py"]
    BA = len(_active(n, f, case["keV"], case["alpha"], case["pixel"]))
    # the pixels of S under some window, each of them once
    if case["scan"] == "raster":
        seen = min(1.0, (W + 2 * case["px"]) * (W + 2 * case["py"]) / (n / 2) ** 2)
    else:
        seen = min(1.0, (n / 4 + W) ** 2 / (n / 2) ** 2)
    seen = min(seen, P * W * W / (n / 2) ** 2)
    out = 4.0 * P * W * W if case["out"] == "cbed" else 8.0 * P * max(1, case["bins"])
    return dict(bytes=8.0 * BA * seen * (n / 2) ** 2 + 16.0 * P + out,
                flops=P * W * W * (8.0 * BA + 10.0 * math.log2(W) + 4.0))


# ------------------------------------------------------------------ 64 bits

def exact(case, seed):
    if case["kind"] == "build":
        return _exact_build(case, case["n"], case["H"], case["f"], [seed, 0])
    if case["kind"] == "batch":
        return [_exact_build(case, n, H, f, [seed, i]) for i, (n, H, f) in enumerate(_parts(case))]
    return _exact_probe(case, seed)


def _exact_build(case, n, H, f, seed):
    pixel, lam = case["pixel"], _wavelength(case["keV"])
    mn, _ = _beams(n, f, case["keV"], case["alpha"], pixel)
    phase = _phase(n, H, pixel, seed)
    k = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEV)
    k2 = k[:, None] ** 2 + k[None, :] ** 2
    prop = torch.polar((16 * k2 < n * n).to(torch.float64),
                       -math.pi * lam * SLICE_A * k2 / (n * pixel) ** 2)
    x = torch.arange(n, dtype=torch.float64, device=DEV) * (2.0 * math.pi / n)
    m = torch.from_numpy(mn).to(DEV).to(torch.float64) * f
    S = torch.empty((len(mn), n // 2, n // 2), dtype=torch.complex128, device=DEV)
    step = max(1, (1 << 28) // (n * n * 16))
    for b in range(0, len(mn), step):
        w = torch.exp(1j * m[b:b + step, 1, None] * x[None, :])[:, :, None] * \
            torch.exp(1j * m[b:b + step, 0, None] * x[None, :])[:, None, :]
        for p in range(H):
            t = torch.polar(torch.ones_like(k2), phase[p].to(torch.float64))
            w = torch.fft.ifft2(torch.fft.fft2(w * t) * prop)
        S[b:b + step] = w[:, ::2, ::2]
    return S


def _exact_probe(case, seed):
    n, f, pixel = case["n"], case["f"], case["pixel"]
    ns, W, side, lam = n // 2, n // (2 * f), n * pixel, _wavelength(case["keV"])
    act = _active(n, f, case["keV"], case["alpha"], pixel)
    mn = _beams(n, f, case["keV"], case["alpha"], pixel)[0][act]
    S = _smatrix(case, seed)
    act_t = torch.from_numpy(act).to(DEV)
    xy = _probes(case, seed)
    q = torch.from_numpy(mn).to(DEV).to(torch.float64) * (f / side)
    q2 = (q ** 2).sum(dim=1)
    dxs = side / ns
    org = np.mod(np.floor(xy / dxs + 0.5).astype(np.int64) - W // 2, ns)
    kw = torch.fft.fftfreq(W, 1.0 / W, dtype=torch.float64, device=DEV) * f
    th = lam / side * torch.sqrt(kw[:, None] ** 2 + kw[None, :] ** 2)
    bins = torch.stack([((th >= lo * 1e-3) & (th < hi * 1e-3)).flatten()
                        for lo, hi in _edges(case)]).to(torch.float64)
    off = torch.arange(W, device=DEV)
    outs = []
    for p0 in range(0, len(xy), 64):
        pos = torch.from_numpy(xy[p0:p0 + 64]).to(DEV)
        o = org[p0:p0 + 64]
        rel = np.mod(o - o[0] + ns // 2, ns) - ns // 2  # (x, y) of each window from the first
        lo, ext = rel.min(axis=0), W + np.ptp(rel, axis=0)
        a = torch.polar(torch.ones((len(pos), len(mn)), dtype=torch.float64, device=DEV),
                        -(math.pi * lam * case["defocus"]) * q2[None, :] -
                        2.0 * math.pi * (pos @ q.T)) / (W * math.sqrt(len(mn)))
        gx = torch.remainder(torch.arange(int(ext[0]), device=DEV) + int(o[0, 0] + lo[0]), ns)
        gy = torch.remainder(torch.arange(int(ext[1]), device=DEV) + int(o[0, 1] + lo[1]), ns)
        u = torch.empty((len(pos), len(gy), len(gx)), dtype=torch.complex128, device=DEV)
        rows = max(1, (1 << 25) // (len(act) * len(gx)))
        for y in range(0, len(gy), rows):
            s = S[act_t[:, None, None], gy[None, y:y + rows, None], gx[None, None, :]]
            u[:, y:y + rows] = (a @ s.reshape(len(act), -1).to(torch.complex128)).view(
                len(pos), -1, len(gx))
        r = torch.from_numpy(rel - lo).to(DEV)
        i = torch.arange(len(pos), device=DEV)[:, None, None]
        psi = u[i, (r[:, 1, None] + off)[:, :, None], (r[:, 0, None] + off)[:, None, :]]
        z = torch.fft.fft2(psi)
        inten = (z.real ** 2 + z.imag ** 2) / W ** 2
        outs.append(inten if case["out"] == "cbed" else inten.flatten(1) @ bins.T)
    return torch.cat(outs)
