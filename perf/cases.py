"""The work that a user has the EPIC imaging library do, as cases to time.

A case is one call chain on digitised voltages that already sit in device
memory, with the plan, accumulator and (for the batched band) HIP graph that a
program keeps for its array:

- ``image``: reset, accumulate one block or integration, read the images out;
- ``graph``: the same with the accumulate captured once as a HIP graph;
- ``frames``: one image set per ``frame_len`` samples (high-cadence imaging);
- ``staged``: the separate primitives, grids and sky images kept in memory.

A case has one array (elements in a disc with a minimum spacing: a station
does not move between observations).  The kernels of its elements and the
voltages come from the seed: a few point sources with a fresh random phase per
sample and thermal noise, quantised to 4 or 8 bits per part.
"""
import math

import numpy as np
import torch

import paper_2609_03027_amd as E

C_LIGHT = 299792458.0
SIDES = (32, 48, 64, 96, 128, 192, 256, 384, 512)
PRECISION = {"f32": E.EPIC_F32, "f16": E.EPIC_F16_MFMA, "f8": E.EPIC_F8E4M3_MFMA,
             "bf16x2": E.EPIC_BF16X2_MFMA, "fixed16": E.EPIC_FIXED16}
XFORM = {"auto": E.XFORM_AUTO, "fft": E.XFORM_FFT, "direct": E.XFORM_DFT_DIRECT,
         "separable": E.XFORM_DFT_SEPARABLE}


def case(name, **kw):
    c = dict(name=name, kind="image", n_ant=256, n_pol=2, n_chan=128, n_time=1000, disc_m=100.0,
             f_lo=40e6, f_hi=80e6, grid=0, aperture=0, k=3, bits=4, precision="f32", xform="auto",
             jones=False, table=False, frame_len=0, noise=1.0)
    c.update(kw)
    return c


def listed():
    lwa = dict(n_ant=256, n_chan=128, disc_m=100.0, f_lo=40e6, f_hi=80e6, grid=128, aperture=64)
    stream = dict(n_ant=4096, n_chan=64, n_time=256, disc_m=300.0, f_lo=92e6, f_hi=108e6, grid=256)
    return [
        # the smallest call: 16 elements, one feed, one channel; latency and launches
        case("tiny_f32", n_ant=16, n_pol=1, n_chan=1, n_time=64, disc_m=10.0, f_lo=60e6,
             f_hi=60e6, grid=32),
        # one block of a served LWA-like station (1 ms of data), imaged at once
        case("station_block_f32", n_time=25, **lwa),
        # a whole LWA-like integration, the default path
        case("station_integration_f32", n_time=1000, **lwa),
        # the same station with four complex kernels per element (full polarimetry)
        case("station_jones_f32", n_time=250, jones=True, **lwa),
        # high-cadence imaging of the same station, four samples per frame
        case("station_frames_f32", kind="frames", n_time=100, frame_len=4, **lwa),
        # gridding, transform and products called one by one, grids and sky kept
        case("station_staged_f32", kind="staged", n_time=64, **dict(lwa, n_chan=32, f_hi=50e6)),
        # the station's integration on the matrix cores, grid transformed as F G F^T
        case("station_separable_f16", n_time=250, precision="f16", xform="separable", **lwa),
        # a wide band whose grid side grows with frequency, one launch for all of it
        case("band_batch_f32", kind="graph", n_chan=384, n_time=512, disc_m=38.0, f_lo=50e6,
             f_hi=350e6),
        # an AAVS2-like station with 8+8-bit voltages in 16-bit fixed point
        case("station_fixed16", n_chan=64, n_time=1000, disc_m=38.0, f_lo=150e6, f_hi=168e6,
             grid=64, k=2, bits=8, table=True, precision="fixed16", noise=0.0),
        # one block of a 4096-element streaming array, FP32
        case("array_block_f32", **stream),
        # the same block in FP16 on the matrix cores
        case("array_block_f16", precision="f16", **stream),
        # wide-field image of 20 000 elements, 1 ms of one coarse channel
        case("wide_image_f32", n_ant=20000, n_chan=1, n_time=781, disc_m=700.0, f_lo=100e6,
             f_hi=100e6, grid=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, without a name."""
    family = rng.choice(["station", "station", "station", "jones", "frames", "staged", "gemm",
                         "band", "fixed16", "array", "array", "wide"])
    if family in ("station", "jones", "frames", "staged", "gemm"):
        n_chan = _log(rng, 1, 128)
        n_time = _log(rng, 8, 1000)
        f_lo = rng.uniform(40e6, 60e6)
        kw = dict(n_ant=_log(rng, 16, 256), n_chan=n_chan, n_time=n_time,
                  disc_m=rng.uniform(20.0, 100.0), f_lo=f_lo, f_hi=f_lo + rng.uniform(0.5e6, 20e6),
                  k=rng.choice([2, 3, 3]), bits=rng.choice([4, 4, 8]))
        if family == "station":
            grid = rng.choice([(0, 0), (128, 64), (128, 64), (128, 0)])
            kw.update(n_pol=rng.choice([1, 2, 2, 2]), grid=grid[0], aperture=grid[1],
                      table=rng.random() < 0.2)
        elif family == "gemm":
            form = rng.choice([("f16", "separable"), ("bf16x2", "separable"), ("f16", "direct"),
                               ("f8", "direct"), ("bf16x2", "direct")])
            kw.update(precision=form[0], xform=form[1], grid=128, aperture=64,
                      n_time=min(n_time, 250))
            if form[0] == "f8":
                kw.update(bits=4)
        elif family == "jones":
            kw.update(jones=True, grid=128, aperture=64, n_time=min(n_time, 250))
        elif family == "frames":
            fl = rng.choice([1, 2, 4, 8, 25])
            frames = max(1, min(n_time, 100) // fl)
            kw.update(kind="frames", frame_len=fl, n_time=fl * frames, grid=128, aperture=64)
        else:
            kw.update(kind="staged", n_chan=min(n_chan, 32), n_time=min(n_time, 64))
    elif family == "band":
        f_lo = rng.uniform(50e6, 200e6)
        kw = dict(kind=rng.choice(["graph", "image"]), n_ant=_log(rng, 64, 256),
                  n_chan=_log(rng, 8, 192), n_time=_log(rng, 25, 512), disc_m=rng.uniform(25.0, 38.0),
                  f_lo=f_lo, f_hi=f_lo + rng.uniform(10e6, 150e6))
    elif family == "fixed16":
        kw = dict(n_ant=_log(rng, 16, 256), n_chan=_log(rng, 1, 64), n_time=_log(rng, 16, 1000),
                  disc_m=38.0, f_lo=150e6, f_hi=168e6, grid=64, k=rng.choice([2, 3]),
                  bits=rng.choice([4, 8]), table=rng.random() < 0.5, precision="fixed16",
                  noise=rng.choice([0.0, 1.0]))
    elif family == "array":
        f_lo = rng.uniform(80e6, 100e6)
        kw = dict(n_ant=_log(rng, 1000, 4096), n_chan=_log(rng, 2, 64), n_time=_log(rng, 16, 256),
                  disc_m=rng.uniform(200.0, 300.0), f_lo=f_lo, f_hi=f_lo + rng.uniform(0.5e6, 8e6),
                  grid=256, precision=rng.choice(["f32", "f16"]), bits=rng.choice([4, 4, 8]))
    else:
        kw = dict(n_ant=_log(rng, 5000, 20000), n_chan=_log(rng, 1, 2), n_time=_log(rng, 50, 390),
                  disc_m=rng.uniform(450.0, 700.0), f_lo=90e6, f_hi=100e6, grid=512)
    c = case("", **kw)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _freqs(c):
    n = c["n_chan"]
    return c["f_lo"] + (np.arange(n) + 0.5) * (c["f_hi"] - c["f_lo"]) / n


def _layout(c):
    """Uniform in the disc, 1 m apart (closer where the disc is too full)."""
    rng = np.random.default_rng([c["n_ant"], int(c["disc_m"])])
    n, r = c["n_ant"], 0.5 * c["disc_m"]
    gap = min(1.0, 0.7 * c["disc_m"] / math.sqrt(n) / 1.5)
    cells, pts = {}, []
    while len(pts) < n:
        for x, y in rng.uniform(-r, r, size=(2 * n, 2)).tolist():
            if len(pts) == n:
                break
            if x * x + y * y > r * r:
                continue
            i, j = math.floor(x / gap), math.floor(y / gap)
            if any((x - u) ** 2 + (y - v) ** 2 < gap * gap
                   for a in (i - 1, i, i + 1) for b in (j - 1, j, j + 1)
                   for u, v in cells.get((a, b), ())):
                continue
            cells.setdefault((i, j), []).append((x, y))
            pts.append((x, y))
    return np.array(pts)


def _sides(c, pos):
    """The grid side of every channel: the case's, or the library's stated rule."""
    if c["grid"]:
        return np.full(c["n_chan"], c["grid"], dtype=np.int32)
    ext = 2.0 * np.abs(pos).max()
    cell = 0.5 * C_LIGHT / _freqs(c)
    need = 2 * np.ceil(ext / cell + c["k"])
    return np.array([min(s for s in SIDES if s >= m) for m in need], dtype=np.int32)


def _geometry(c, pos, freq, n):
    """Grid position x and first support cell j0 of every element."""
    x = pos / (0.5 * C_LIGHT / freq) + n / 2.0
    return x, np.floor(x - c["k"] / 2.0 + 1.0).astype(np.int64)


def _gauss(c, x, j0):
    """Unit-sum Gaussian kernel [A][K][K] ([dy][dx]) on each support."""
    d = j0[:, :, None] + np.arange(c["k"]) - x[:, :, None]
    g = np.exp(-d * d / (2.0 * 0.5 * 0.5))
    w = g[:, 1, :, None] * g[:, 0, None, :]
    return w / w.sum(axis=(1, 2), keepdims=True)


def _kernels(c, pos, sides, rng):
    """Explicit kernels [C][A](alpha, p)[K][K]: the Gaussian times one complex
    factor per element, or a 2x2 matrix near the identity for Jones plans."""
    A, k = c["n_ant"], c["k"]
    if c["jones"]:
        m = 0.15 * (rng.standard_normal((A, 2, 2)) + 1j * rng.standard_normal((A, 2, 2)))
        m = m + np.eye(2)
    else:
        m = 1.0 + 0.15 * (rng.standard_normal(A) + 1j * rng.standard_normal(A))
    out = np.empty((c["n_chan"],) + m.shape + (k, k), dtype=np.complex64)
    for i, f in enumerate(_freqs(c)):
        w = _gauss(c, *_geometry(c, pos, f, sides[i]))
        out[i] = m[..., None, None] * (w[:, None, None] if c["jones"] else w)
    return out


def _voltages(c, pos, rng):
    """Digitised voltages on the GPU: uint8 [t][c][p][a], or int8 [t][c][p][a][2]."""
    T, P, A, S = c["n_time"], c["n_pol"], c["n_ant"], 3
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(rng.integers(1 << 62)))
    rad, ang = 0.7 * np.sqrt(rng.uniform(size=S)), rng.uniform(0, 2 * np.pi, size=S)
    path = pos @ np.stack([rad * np.cos(ang), rad * np.sin(ang)])            # [A][S]
    top = 7 if c["bits"] == 4 else 127
    scale = (2.0 if c["bits"] == 4 else 32.0) / math.sqrt((S + c["noise"]) / 2.0)
    out = torch.empty((T, c["n_chan"], P, A) + ((2,) if c["bits"] == 8 else ()),
                      dtype=torch.uint8 if c["bits"] == 4 else torch.int8, device=dev)
    for i, f in enumerate(_freqs(c)):
        geo = torch.from_numpy(np.exp(-2j * np.pi * path.T * f / C_LIGHT)).to(torch.complex64).to(dev)
        ph = 2 * math.pi * torch.rand((T, P, S), generator=gen, device=dev)
        if P == 2:
            ph[:, 1, 0] = ph[:, 0, 0] + math.pi / 4      # one polarised source
        v = torch.view_as_real((torch.polar(torch.ones_like(ph), ph).reshape(T * P, S) @ geo))
        if c["noise"]:
            v = v + torch.randn(v.shape, generator=gen, device=dev) * math.sqrt(c["noise"] / 2)
        q = (v * scale).round_().clamp_(-top, top).to(torch.int32).reshape(T, P, A, 2)
        out[:, i] = (((q[..., 0] & 15) << 4) | (q[..., 1] & 15)).to(torch.uint8) \
            if c["bits"] == 4 else q.to(torch.int8)
    return out


def _inputs(c, seed):
    rng = np.random.default_rng([int(seed), 7])
    pos = _layout(c)
    sides = _sides(c, pos)
    kernels = _kernels(c, pos, sides, rng) if c["jones"] or c["table"] else None
    return pos, sides, kernels, _voltages(c, pos, rng)


def prepare(case, seed):
    c = case
    pos, sides, kernels, volt = _inputs(c, seed)
    kw = {}
    if kernels is not None:
        kw["kernel_table"] = np.stack([kernels.real, kernels.imag], axis=-1)
    plan = E.Plan(pos, _freqs(c), sides if c["grid"] else None, c["n_pol"],
                  aperture_n=c["aperture"], kernel_k=c["k"], volt_bits=c["bits"], jones=c["jones"],
                  precision=PRECISION[c["precision"]], xform=XFORM[c["xform"]], **kw)
    acc = E.Accumulator(plan)
    s = dict(kind=c["kind"], plan=plan, acc=acc, volt=volt, n_time=c["n_time"],
             frame_len=c["frame_len"])
    f32 = dict(dtype=torch.float32, device="cuda")
    if c["kind"] == "frames":
        s["out"] = torch.empty((c["n_time"] // c["frame_len"], plan.info["image_floats"]), **f32)
        return s
    s["out"] = torch.empty(plan.info["image_floats"], **f32)
    if c["kind"] == "staged":
        shape = (c["n_time"], plan.info["grid_elems_per_t"])
        s["grid"] = torch.empty(shape, dtype=torch.complex64, device="cuda")
        s["sky"] = torch.empty(shape, dtype=torch.complex64, device="cuda")
    if c["kind"] == "graph":
        s["graph"] = E.Graph(plan, acc, volt)
    return s


def run(state):
    s = state
    plan, acc, volt, out = s["plan"], s["acc"], s["volt"], s["out"]
    if s["kind"] == "frames":
        E.accumulate_frames(plan, acc, volt, s["frame_len"], out)
        return out
    acc.reset()
    if s["kind"] == "graph":
        s["graph"].launch()
    elif s["kind"] == "staged":
        E.grid(plan, volt, s["n_time"], s["grid"])
        E.image(plan, s["grid"], s["n_time"], s["sky"])
        E.accumulate(plan, acc, volt=volt, sky=s["sky"])
    else:
        E.accumulate(plan, acc, volt=volt)
    E.readout(plan, acc, out)
    if s["kind"] == "staged":
        return {"grid": s["grid"], "sky": s["sky"], "image": out}
    return out


def work(case):
    """Voltages in, images (or frames, or grids and skies) out; the transform
    counted as 5 n log2 n per image of n pixels, 16 flops per pixel and sample
    for the products (4 with one feed), 8 per kernel tap and feed pair."""
    c = case
    T, P, C = c["n_time"], c["n_pol"], c["n_chan"]
    # the library's rule on the disc itself, which the elements nearly fill
    pos = np.array([[0.5 * c["disc_m"], 0.0]])
    n2 = [int(n) ** 2 for n in _sides(c, pos)]
    n_prod = 4 if P == 2 else 1
    sets = c["n_time"] // c["frame_len"] if c["kind"] == "frames" else 1
    bytes_ = T * C * P * c["n_ant"] * (1 if c["bits"] == 4 else 2) + 4 * n_prod * sum(n2) * sets
    if c["kind"] == "staged":
        bytes_ += 2 * 8 * T * P * sum(n2)
    taps = c["n_ant"] * c["k"] ** 2 * P * (P if c["jones"] else 1)
    flops = sum(T * (5.0 * P * n * math.log2(n) + (16.0 if P == 2 else 4.0) * n + 8.0 * taps)
                for n in n2)
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------------ 64-bit values
def exact(case, seed):
    """What run() returns, from Eq. 1 and Eq. 2 in double precision."""
    c = case
    pos, sides, kernels, volt = _inputs(c, seed)
    T, P, A, k = c["n_time"], c["n_pol"], c["n_ant"], c["k"]
    dev, f64, c128 = volt.device, torch.float64, torch.complex128
    frames = c["kind"] == "frames"
    fl = c["frame_len"] if frames else T
    images, grids, skies = [], [], []
    for i, f in enumerate(_freqs(c)):
        n = int(sides[i])
        x, j0 = _geometry(c, pos, f, n)
        if kernels is None:
            w = _gauss(c, x, j0)[:, None, None].astype(np.complex128)
        else:
            w = kernels[i].astype(np.complex128).reshape(A, *((2, 2) if c["jones"] else (1, 1)), k, k)
        w = torch.from_numpy(w).to(dev)                                       # [A][al][p][dy][dx]
        v = volt[:, i].to(torch.int32)
        if c["bits"] == 4:
            re, im = (v << 24) >> 28, (v << 28) >> 28
        else:
            re, im = v[..., 0], v[..., 1]
        e = torch.complex(re.to(f64), im.to(f64))                             # [T][P][A]
        cells = [torch.from_numpy((j0[:, 1] + dy) * n + j0[:, 0] + dx).to(dev)
                 for dy in range(k) for dx in range(k)]
        step = max(fl if frames else 1, (1 << 30) // (16 * P * n * n) // fl * fl if frames
                   else (1 << 30) // (16 * P * n * n))
        total = torch.zeros((4 if P == 2 else 1, n, n), dtype=f64, device=dev)
        out = []
        for t0 in range(0, T, step):
            et = e[t0:t0 + step]
            m = et.shape[0]
            g = torch.zeros((m * P, n * n, 2), dtype=f64, device=dev)
            for t, cell in enumerate(cells):
                wt = w[:, :, :, t // k, t % k].conj()                         # [A][al][p]
                if c["jones"]:
                    tap = (et[:, None] * wt.permute(1, 2, 0)).sum(dim=2)      # [m][al][A]
                else:
                    tap = et * wt[:, 0, 0]
                g.index_add_(1, cell, torch.view_as_real(tap.reshape(m * P, A).contiguous()))
            g = torch.view_as_complex(g).reshape(m, P, n, n)
            s = torch.fft.fftshift(torch.fft.ifft2(torch.fft.ifftshift(g, dim=(-2, -1))),
                                   dim=(-2, -1)) * (n * n)
            if c["kind"] == "staged":
                grids.append((t0, i, g.reshape(m, -1)))
                skies.append((t0, i, s.reshape(m, -1)))
            prod = [s[:, 0].abs() ** 2]
            if P == 2:
                xy = s[:, 0] * s[:, 1].conj()
                prod += [s[:, 1].abs() ** 2, xy.real, xy.imag]
            if frames:
                out.append(torch.stack([p.reshape(m // fl, fl, n, n).sum(1) for p in prod], dim=1))
            else:
                total += torch.stack([p.sum(0) for p in prod])
        if frames:
            images.append(torch.cat(out).reshape(T // fl, -1))
            continue
        # self terms: S_a^{pq} B_a^{al p} conj(B_a^{be q}), from the footprint
        # displacements d: sum_j conj(W^{al p}(j)) W^{be q}(j - d)
        cov = torch.einsum("tpa,tqa->pqa", e, e.conj())
        pairs = [(0, 0)] + ([(1, 1), (0, 1)] if P == 2 else [])
        term = []
        for al, be in pairs:
            h = torch.zeros((n, n), dtype=c128, device=dev)
            for jy in range(k):
                for jx in range(k):
                    for iy in range(k):
                        for ix in range(k):
                            if c["jones"]:
                                s = torch.einsum("ap,aq,pqa->", w[:, al, :, jy, jx].conj(),
                                                 w[:, be, :, iy, ix], cov)
                            else:
                                s = (w[:, 0, 0, jy, jx].conj() * w[:, 0, 0, iy, ix] * cov[al, be]).sum()
                            h[(jy - iy) % n, (jx - ix) % n] += s
            term.append(torch.fft.fftshift(torch.fft.ifft2(h)) * (n * n))
        sub = [term[0].real] + ([term[1].real, term[2].real, term[2].imag] if P == 2 else [])
        images.append(((total - torch.stack(sub)) / T).reshape(-1))
    if frames:
        return torch.cat(images, dim=1)
    if c["kind"] != "staged":
        return torch.cat(images)

    def whole(parts):
        rows = {}
        for t0, i, z in parts:
            rows.setdefault(t0, []).append(z)
        return torch.cat([torch.cat(rows[t0], dim=1) for t0 in sorted(rows)])
    return {"grid": whole(grids), "sky": whole(skies), "image": torch.cat(images)}
