"""Performance cases: the work a user of this library has it do, through the
public entry points of paper_1903_06838_amd.pdc.

A case is one pass of a program's steady state: raw frames resident in device
memory go in, photon lists (and what the program asks for beside them) come
out.  Detectors are those of the repository's own workloads (ePix100,
CSPAD-like, auto-ranging ePix10k-like and Jungfrau-like) and two geometries
outside the persistent kernel's fast path (odd and very wide banks).  Inputs
are synthetic and made on the GPU from the seed alone: charge is scattered in
integer units, so the same seed gives the same words every time.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  inputs, calibration, context, network, output buffers
  run(state)           one pass and its outputs
  work(case)           bytes and operations a pass cannot do without
  exact(case, seed)    the floating outputs in 64 bits, in plain torch
"""
import math

import numpy as np
import torch

from paper_1903_06838_amd import pdc

# name: tiles, rows, cols, bank columns, gain mode (0: one range)
DETECTORS = {
    "epix100": (1, 704, 768, 96, 0),
    "cspad": (32, 185, 388, 194, 0),
    "epix10k": (1, 352, 384, 96, 1),
    "jungfrau": (1, 512, 1024, 256, 2),
    "odd_banks": (8, 185, 194, 97, 0),     # odd bank width: the general kernel
    "wide_banks": (1, 512, 1024, 512, 0),  # banks over 256 columns: the general kernel
}
GENERAL = ("odd_banks", "wide_banks")
SIGMA, SEED, NB, ADU = 3.0, 5.0, 3.0, 150.0
RANGE_GAINS = (1.0, 1.0 / 3.0, 1.0 / 100.0)
RANGE_FRACTIONS = (0.95, 0.03, 0.01, 0.01)  # of the pixels: three ranges, invalid codes
CM_MODES = {"median": pdc.CM_MEDIAN, "bank": pdc.CM_BANK_MEAN, "tile": pdc.CM_TILE_MEAN}
MIX = ("epix100", "epix10k", "jungfrau")
NBINS, HIST_LO, HIST_HI = 1024, -50.0, 974.0
ETA_BINS = 256
TRAIN_STEPS, LR = 8, 2e-3
DEV = "cuda"


def _frames_case(name, det, n, occ, cm="median", stages=1, host=False, graph=False):
    return {"name": name, "kind": "frames", "det": det, "n": n, "occ": occ, "cm": cm, "stages": stages, "host": host,
            "graph": graph}


def listed():
    return [
        # online monitoring: one camera frame at a time, photon records to the host
        _frames_case("one_epix100_frame", "epix100", 1, 0.01, host=True),
        # a short acquisition of the large detector, records to the host
        _frames_case("cspad_16_frames", "cspad", 16, 0.01, host=True),
        # offline reduction: the 10,000-frame batch of the headline workload, records stay on the device
        _frames_case("cspad_batch_10000", "cspad", 10000, 0.01),
        # an auto-ranging detector with three gain ranges and invalid codes
        _frames_case("jungfrau_batch_1000", "jungfrau", 1000, 0.005),
        # the paper's thresholded mean, three stacked stages, over banks and over tiles
        _frames_case("cspad_bank_mean_1000", "cspad", 1000, 0.01, cm="bank", stages=3),
        _frames_case("cspad_tile_mean_1000", "cspad", 1000, 0.01, cm="tile", stages=3),
        # a geometry the persistent kernel does not take
        _frames_case("odd_banks_64", "odd_banks", 64, 0.01),
        # several detectors' batches enqueued together
        {"name": "mixed_3_detectors_1000", "kind": "mixed", "n": 1000, "occ": 0.01},
        # an analysis run: Frames2 kept, count map, spectra and the Frames2 histogram beside the photon list
        {"name": "epix100_analysis_100", "kind": "analysis", "det": "epix100", "n": 100, "occ": 0.01},
        # learned subpixel positions of every hit of a batch, with the classical fallback
        {"name": "cspad_positions_64", "kind": "subpixel", "det": "cspad", "n": 64, "occ": 0.005},
        # positions from stored patches: the network, and centroid + eta beside it
        {"name": "patches_1m", "kind": "patches", "n": 1000000},
        # training the network on simulated patches: consecutive steps
        {"name": "train_2048", "kind": "train", "n": 2048},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _pixels(det):
    T, H, W, _, _ = DETECTORS[det]
    return T * H * W


def draw(rng):
    kind = rng.choice(["frames"] * 6 + ["mixed", "analysis", "subpixel", "subpixel", "patches", "train"])
    occ = round(math.exp(rng.uniform(math.log(0.001), math.log(0.05))), 5)
    if kind == "frames":
        det = rng.choice(["epix100", "cspad", "cspad", "epix10k", "jungfrau", "odd_banks", "wide_banks"])
        general = det in GENERAL
        cm, stages = "median", 1
        if not general and DETECTORS[det][4] == 0 and rng.random() < 0.3:
            cm, stages = rng.choice(["bank", "tile"]), rng.randint(1, 3)
        most = 4.0e7 if general else (2.5e9 if cm != "median" else 9.0e9)  # pixels of a pass
        n = _log_int(rng, 1, max(1, int(most / _pixels(det))))
        small = n * _pixels(det) < 4.0e7
        return {"kind": kind, "det": det, "n": n, "occ": occ, "cm": cm, "stages": stages,
                "host": small and rng.random() < 0.5, "graph": small and not general and rng.random() < 0.3}
    if kind == "mixed":
        return {"kind": kind, "n": _log_int(rng, 4, 2000), "occ": min(occ, 0.02)}
    if kind in ("analysis", "subpixel"):
        det = rng.choice(["epix100", "cspad", "jungfrau"])
        return {"kind": kind, "det": det, "n": _log_int(rng, 1, int(1.5e8 / _pixels(det))), "occ": min(occ, 0.03)}
    if kind == "patches":
        return {"kind": kind, "n": _log_int(rng, 37, 10000000)}
    return {"kind": kind, "n": _log_int(rng, 65, 40000)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(*key):
    g = torch.Generator(device=DEV)
    s = 1903
    for k in key:
        s = (s * 1000003 + int(k) + 6838) % (1 << 62)
    g.manual_seed(s)
    return g


def _calibration(det, seed):
    """Pedestal and gain planes, float32 [ranges, T, H, W] on the device."""
    T, H, W, _, gm = DETECTORS[det]
    g = _gen(seed, 1)
    R = 3 if gm else 1
    ped = 1500.0 + 50.0 * torch.randn((R, T, H, W), generator=g, device=DEV)
    gain = 0.95 + 0.1 * torch.rand((R, T, H, W), generator=g, device=DEV)
    if gm:
        gain = gain * torch.tensor(RANGE_GAINS, device=DEV).view(3, 1, 1, 1)
    return ped, gain


def _charge(n, shape, occ, g):
    """Photon charge of n frames in 1/256 ADU, int32 [n, T, H, W]: Poisson photons of 150 ADU at uniform
    positions, each spread as a Gaussian (sigma 0.2 px) over the pixels around it, inside its tile."""
    T, H, W = shape
    cnt = torch.poisson(torch.full((n * T * H * W,), occ, device=DEV), generator=g).to(torch.int64)
    at = torch.nonzero(cnt).view(-1)
    at = torch.repeat_interleave(at, cnt[at])
    pos = torch.rand((2, at.numel()), generator=g, device=DEV)
    r, c = (at // W) % H, at % W
    out = torch.zeros(n * T * H * W, dtype=torch.int32, device=DEV)
    s = 0.2 * math.sqrt(2.0)

    def share(p, d):  # of the charge in the row (column) at distance d
        return 0.5 * (torch.erf((d + 1 - p) / s) - torch.erf((d - p) / s))

    for dr in (-1, 0, 1):
        fy = share(pos[0], dr)
        for dc in (-1, 0, 1):
            q = torch.round(256.0 * ADU * fy * share(pos[1], dc)).to(torch.int32)
            ok = (r + dr >= 0) & (r + dr < H) & (c + dc >= 0) & (c + dc < W)
            out.index_add_(0, (at + dr * W + dc)[ok], q[ok])
    return out.view(n, T, H, W)


def _pool_size(case):
    """Distinct frames: a batch repeats them (each copy at its own address)."""
    return min(case["n"], 64 if _pixels(case["det"]) < 3000000 else 16)


def _pool(case, seed, ped, gain):
    """Distinct raw frames, int16 words [P, T, H, W]."""
    T, H, W, B, gm = DETECTORS[case["det"]]
    cm = case.get("cm", "median")
    P = _pool_size(case)
    words = torch.empty((P, T, H, W), dtype=torch.int16, device=DEV)
    step = max(1, 20000000 // (T * H * W))
    for f in range(0, P, step):
        m = min(step, P - f)
        g = _gen(seed, 2, f)
        sig = _charge(m, (T, H, W), case["occ"], g).float() / 256.0
        # offsets: per bank, or per tile where the tile is the common-mode region; the thresholded mean is for
        # offsets inside its noise threshold
        if cm == "tile":
            off = 2.0 * torch.randn((m, T, 1, 1), generator=g, device=DEV)
        else:
            off = (10.0 if cm == "median" else 2.0) * torch.randn((m, T, H, W // B, 1), generator=g, device=DEV)
            off = off.expand(m, T, H, W // B, B).reshape(m, T, H, W)
        noise = SIGMA * torch.randn((m, T, H, W), generator=g, device=DEV)
        if gm:
            u = torch.rand((m, T, H, W), generator=g, device=DEV)
            a, b, d = RANGE_FRACTIONS[0], sum(RANGE_FRACTIONS[:2]), sum(RANGE_FRACTIONS[:3])
            pick = (u >= a).int() + (u >= b).int() + (u >= d).int()  # 3: invalid code
            rng = pick.clamp(max=2)
            pe = torch.where(rng == 0, ped[0], torch.where(rng == 1, ped[1], ped[2]))
            ga = torch.where(rng == 0, gain[0], torch.where(rng == 1, gain[1], gain[2]))
            codes = torch.tensor((0, 1, 2, 3) if gm == 1 else (0, 1, 3, 2), device=DEV, dtype=torch.int32)
            code = codes[pick.long()] << 14
        else:
            pe, ga, code = ped[0], gain[0], 0
        val = torch.round(pe + ga * sig + off + noise).clamp(0, 16383).to(torch.int32)
        words[f:f + m] = (val | code).to(torch.int16)
    return words


def _frames(pool, n):
    P = pool.shape[0]
    if n == P:
        return pool
    out = torch.empty((n,) + tuple(pool.shape[1:]), dtype=torch.int16, device=DEV)
    for f in range(0, n, P):
        m = min(P, n - f)
        out[f:f + m] = pool[:m]
    return out


def _hit_capacity(case, det):
    """What such a program expects: its occupancy, with room for low-gain noise and split clouds."""
    rate = 1.3 * case["occ"] + (0.02 if DETECTORS[det][4] else 0.0)
    if case.get("cm", "median") != "median":
        rate += 0.01
    return int(rate * case["n"] * _pixels(det)) + 8192


def _patches(n, seed):
    """Corrected 5x5 patches around single-photon hits (float32 [n, 25]) and the true positions [n, 2]."""
    g = _gen(seed, 3)
    truth = torch.rand((n, 2), generator=g, device=DEV) - 0.5
    s = (0.1 + 0.3 * torch.rand((n, 1), generator=g, device=DEV)) * math.sqrt(2.0)
    edges = torch.arange(-2, 4, device=DEV, dtype=torch.float32) - 0.5
    fy = 0.5 * torch.diff(torch.erf((edges - truth[:, :1]) / s), dim=1)
    fx = 0.5 * torch.diff(torch.erf((edges - truth[:, 1:]) / s), dim=1)
    p = ADU * fy[:, :, None] * fx[:, None, :] + SIGMA * torch.randn((n, 5, 5), generator=g, device=DEV)
    return p.reshape(n, 25).contiguous(), truth.contiguous()


def _theta(seed):
    """He-uniform weights and zero biases of the 25-64-64-2 network, in the library's layout."""
    rng = np.random.default_rng([1903, 6838, int(seed)])
    parts = []
    for a, b in ((25, 64), (64, 64), (64, 2)):
        lim = math.sqrt(6.0 / a)
        parts += [rng.uniform(-lim, lim, a * b), np.zeros(b)]
    return np.concatenate(parts).astype(np.float32)


# ---------------------------------------------------------------------------
# state and one pass
# ---------------------------------------------------------------------------
class State:
    """A context and what the program keeps with it; everything goes with the object."""

    def __init__(self, case):
        self.case = case
        self.ctx = pdc.create(0)
        self.net = None
        self.stream = torch.cuda.Stream()

    def __del__(self):
        if getattr(self, "net", None):
            pdc.mlp_destroy(self.net)
            self.net = None
        if getattr(self, "ctx", None):
            pdc.destroy(self.ctx)  # graphs, detectors and buffers go with it
            self.ctx = None


def _detector(st, case, det, seed, flags=0):
    """Calibrated detector and its device frames."""
    T, H, W, B, gm = DETECTORS[det]
    ped, gain = _calibration(det, seed)
    frames = _frames(_pool(dict(case, det=det), seed, ped, gain), case["n"])
    prm = pdc.params(SIGMA, SEED, NB, ADU, flags, CM_MODES[case.get("cm", "median")], case.get("stages", 1), 3.0)
    d = pdc.calibrate(st.ctx, pdc.geometry(T, H, W, B, gm), ped.cpu().numpy(), gain.cpu().numpy(), prm)
    return d, frames


def _records(cap):
    return torch.zeros((cap, 4), dtype=torch.int32, device=DEV)


def prepare(case, seed):
    st = State(case)
    kind, n = case["kind"], case["n"]
    if kind == "frames":
        st.det, st.frames = _detector(st, case, case["det"], seed)
        st.cap = _hit_capacity(case, case["det"])
        st.out = None if case["host"] else _records(st.cap)
        torch.cuda.synchronize()
        st.graph = pdc.graph_create(st.ctx, st.det, st.frames, n, st.cap) if case["graph"] else None
    elif kind == "mixed":
        st.items, st.out = [], []
        for i, det in enumerate(MIX):
            d, fr = _detector(st, case, det, seed + 1000 * i)
            cap = _hit_capacity(case, det)
            st.items.append((d, fr, n, cap))
            st.out.append(_records(cap))
    elif kind == "analysis":
        st.det, st.frames = _detector(st, case, case["det"], seed, pdc.KEEP_CORRECTED)
        st.cap = _hit_capacity(case, case["det"])
        st.out = _records(st.cap)
        px = _pixels(case["det"])
        st.corrected = torch.empty((n, px), dtype=torch.float32, device=DEV)
        st.map = torch.empty(px, dtype=torch.int32, device=DEV)
        st.spectrum = torch.empty(NBINS + 2, dtype=torch.int32, device=DEV)
        st.sizes = torch.empty((9, NBINS + 2), dtype=torch.int32, device=DEV)
        st.hist = torch.empty(NBINS + 2, dtype=torch.int32, device=DEV)
    elif kind == "subpixel":
        st.det, st.frames = _detector(st, case, case["det"], seed, pdc.KEEP_MEDIANS)
        st.cap = _hit_capacity(case, case["det"])
        st.out = _records(st.cap)
        st.inputs = torch.empty((st.cap, pdc.MLP_INPUT_WORDS), dtype=torch.int16, device=DEV)
        st.pos = torch.zeros((st.cap, 2), dtype=torch.float32, device=DEV)
        st.net = pdc.mlp_create(st.ctx, _theta(seed))
    elif kind == "patches":
        st.patches, _ = _patches(n, seed)
        sample, _ = _patches(65536, seed + 1)
        work = torch.empty(2 * ETA_BINS, dtype=torch.int32, device=DEV)
        st.eta = torch.empty((2, ETA_BINS + 1), dtype=torch.float32, device=DEV)
        st.learned = torch.empty((n, 2), dtype=torch.float32, device=DEV)
        st.classical = torch.empty((n, 2), dtype=torch.float32, device=DEV)
        st.net = pdc.mlp_create(st.ctx, _theta(seed))
        torch.cuda.synchronize()
        pdc.eta_table(st.ctx, sample, 65536, NB * SIGMA, ETA_BINS, work, st.eta, st.stream)
    else:
        st.patches, st.truth = _patches(n * TRAIN_STEPS, seed)
        st.net = pdc.mlp_create(st.ctx, _theta(seed))
    torch.cuda.synchronize()
    return st


# Records come as the whole destination (zeros after the last hit), so that batches of one case have one shape.
def _host_result(got):
    hits, total, fh, fp, _ = got
    hits = hits if hits.base is None else hits.base
    return {"frame": hits["frame"], "pixel": hits["pixel"], "charge": hits["charge"], "nphot": hits["nphot"],
            "frame_hits": fh, "frame_photons": fp.view(np.int64), "total": total}


def _device_result(rec, got):
    _, total, fh, fp, _ = got
    return {"frame": rec[:, 0], "pixel": rec[:, 1], "charge": rec.view(torch.float32)[:, 2], "nphot": rec[:, 3],
            "frame_hits": fh, "frame_photons": fp.view(np.int64), "total": total}


def run(st):
    case, ctx = st.case, st.ctx
    kind, n = case["kind"], case["n"]
    if kind == "frames":
        if st.graph:
            b = pdc.graph_launch(ctx, st.graph, st.stream)
        else:
            b = pdc.process_frames(ctx, st.det, st.frames, n, st.cap, st.stream)
        if case["host"]:
            out = _host_result(pdc.get_hits(ctx, b, n, st.cap))
        else:
            out = _device_result(st.out, pdc.get_hits(ctx, b, n, st.cap, st.out))
        pdc.release_batch(ctx, b)
        return out
    if kind == "mixed":
        bs = pdc.process_mixed(ctx, st.items, st.stream)
        outs = []
        for b, (_, _, m, cap), rec in zip(bs, st.items, st.out):
            outs.append(_device_result(rec, pdc.get_hits(ctx, b, m, cap, rec)))
            pdc.release_batch(ctx, b)
        return outs
    if kind == "analysis":
        b = pdc.process_frames(ctx, st.det, st.frames, n, st.cap, st.stream)
        with torch.cuda.stream(st.stream):
            for t in (st.map, st.spectrum, st.sizes, st.hist):
                t.zero_()
        pdc.accumulate_hits(ctx, b, st.map, st.spectrum, st.sizes, 0.0, 1024.0, NBINS, st.stream)
        pdc.histogram_corrected(ctx, b, st.hist, HIST_LO, HIST_HI, NBINS, st.stream)
        pdc.get_corrected(ctx, b, st.corrected)
        out = _device_result(st.out, pdc.get_hits(ctx, b, n, st.cap, st.out))
        pdc.release_batch(ctx, b)
        out.update(corrected=st.corrected, map=st.map, spectrum=st.spectrum, sizes=st.sizes, hist=st.hist)
        return out
    if kind == "subpixel":
        b = pdc.process_frames(ctx, st.det, st.frames, n, st.cap, st.stream)
        m = pdc.capture_inputs(ctx, b, ADU, st.inputs, st.cap)
        pdc.mlp_infer_inputs(st.net, st.inputs, m, st.pos, st.stream)
        st.stream.synchronize()  # the fallback reads the positions on the library's own stream
        pdc.capture_centroids(ctx, b, NB * SIGMA, st.pos, st.cap, only_implausible=True)
        out = _device_result(st.out, pdc.get_hits(ctx, b, n, st.cap, st.out))
        pdc.release_batch(ctx, b)
        out["positions"] = st.pos
        return out
    if kind == "patches":
        pdc.mlp_infer(st.net, st.patches, n, ADU, st.learned, st.stream)
        pdc.centroid(ctx, st.patches, n, NB * SIGMA, st.classical, st.eta, ETA_BINS, st.stream)
        return {"learned": st.learned, "classical": st.classical}
    for k in range(TRAIN_STEPS):
        pdc.mlp_train_step(st.net, st.patches[k * n:], st.truth[k * n:], n, ADU, LR, st.stream)
    return {"theta": pdc.mlp_get_params(st.net), "loss": pdc.mlp_last_loss(st.net)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _frames_work(det, n, occ, extra=0.0):
    T, H, W, B, gm = DETECTORS[det]
    px = T * H * W
    hits = (occ + (0.012 if gm else 0.0)) * n * px
    return 2.0 * n * px + 8.0 * px * (3 if gm else 1) + 16.0 * hits + 12.0 * n + extra, 3.0 * n * px, hits


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "frames":
        b, f, _ = _frames_work(case["det"], n, case["occ"])
        return {"bytes": b, "flops": f}
    if kind == "mixed":
        parts = [_frames_work(d, n, case["occ"]) for d in MIX]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    if kind == "analysis":
        px = _pixels(case["det"])
        b, f, hits = _frames_work(case["det"], n, case["occ"], 4.0 * px + 4.0 * n * px)
        return {"bytes": b, "flops": f + 3.0 * n * px}
    if kind == "subpixel":
        b, f, hits = _frames_work(case["det"], n, case["occ"])
        return {"bytes": b + 8.0 * hits, "flops": f + 11648.0 * hits}
    if kind == "patches":
        return {"bytes": 116.0 * n, "flops": 11648.0 * n}
    return {"bytes": TRAIN_STEPS * (108.0 * n + 6 * 4 * 5954.0), "flops": TRAIN_STEPS * 3 * 11648.0 * n}


# ---------------------------------------------------------------------------
# floating outputs in 64 bits (which pixels are seeds, maxima and noise is decided in binary32, as the
# library's contract defines them; every value is then formed in binary64)
# ---------------------------------------------------------------------------
def _corrected64(case, words, ped, gain):
    """Frames2 of some frames: binary32 values (for decisions) and binary64 ones, [m, T, H, W]."""
    T, H, W, B, gm = DETECTORS[case["det"]]
    m = words.shape[0]
    w = words.to(torch.int32) & 0xFFFF
    adc = (w & 0x3FFF)
    bad = torch.zeros_like(w, dtype=torch.bool)
    if gm:
        code = w >> 14
        table = torch.tensor((0, 1, 2, 3) if gm == 1 else (0, 1, 3, 2), device=DEV)
        r = table[code.long()]
        bad = r == 3
        pe = torch.where(r == 0, ped[0], torch.where(r == 1, ped[1], ped[2]))
        ga = torch.where(r == 0, gain[0], torch.where(r == 1, gain[1], gain[2]))
    else:
        pe, ga = ped[0], gain[0]
    k32 = (1.0 / ga.cpu()).to(DEV) if ga.dim() == 3 else 1.0 / ga
    u32 = (adc.float() - pe) * k32
    u64 = (adc.double() - pe.double()) / ga.double()
    cm = case.get("cm", "median")
    if cm == "median":
        def med(u):
            s = torch.where(bad, torch.full_like(u, math.inf), u).view(m, T, H, W // B, B).sort(dim=-1).values
            nv = (~bad).view(m, T, H, W // B, B).sum(-1, keepdim=True)
            at = ((nv - 1) // 2).clamp(min=0)
            v = torch.where(nv > 0, s.gather(-1, at), torch.zeros_like(s[..., :1]))
            return v.expand(m, T, H, W // B, B).reshape(m, T, H, W)

        v32, v64 = u32 - med(u32), u64 - med(u64)
    else:
        shape = (m, T, 1, 1, H * W) if cm == "tile" else (m, T, H, W // B, B)
        a, b = u32.view(shape), u64.view(shape)
        guard = math.sqrt(shape[-1])
        for _ in range(case.get("stages", 1)):
            noise = (a < 3.0 * SIGMA) & ~bad.view(shape)
            n0 = noise.sum(-1, keepdim=True).double().clamp(min=guard)
            ca = (torch.where(noise, a.double(), 0.0).sum(-1, keepdim=True).float() / n0.float())
            cb = torch.where(noise, b, 0.0).sum(-1, keepdim=True) / n0
            a, b = a - ca, b - cb
        v32, v64 = a.reshape(m, T, H, W), b.reshape(m, T, H, W)
    return torch.where(bad, 0.0, v32), torch.where(bad, 0.0, v64)


def _hits64(v32, v64):
    """Hits in raster order: (frame, tile, row, col) and the charges in binary64."""
    m, T, H, W = v32.shape
    pad = torch.nn.functional.pad(v32, (1, 1, 1, 1), value=-math.inf)
    pad64 = torch.nn.functional.pad(v64, (1, 1, 1, 1))
    ok = v32 > SEED * SIGMA
    q = torch.zeros_like(v64)
    for dr in (0, 1, 2):
        for dc in (0, 1, 2):
            x = pad[:, :, dr:dr + H, dc:dc + W]
            if (dr, dc) < (1, 1):
                ok &= v32 > x
            elif (dr, dc) > (1, 1):
                ok &= v32 >= x
            q += torch.where(x > NB * SIGMA, pad64[:, :, dr:dr + H, dc:dc + W], 0.0)
    at = torch.nonzero(ok)
    return at, q[ok]


def _patches64(v64, at):
    m, T, H, W = v64.shape
    pad = torch.nn.functional.pad(v64, (2, 2, 2, 2))
    f, t, r, c = at.unbind(1)
    return torch.stack([pad[f, t, r + dr, c + dc] for dr in range(5) for dc in range(5)], 1)


def _mlp64(theta, x):
    t = torch.as_tensor(theta, device=DEV).double() if not isinstance(theta, torch.Tensor) else theta
    w1, b1, w2, b2, w3, b3 = t.split([1600, 64, 4096, 64, 128, 2])
    h = torch.relu(x @ w1.view(25, 64) + b1)
    h = torch.relu(h @ w2.view(64, 64) + b2)
    return h @ w3.view(64, 2) + b3


def _centroid64(p):
    s = torch.where(p > NB * SIGMA, p, 0.0).view(-1, 5, 5)[:, 1:4, 1:4]
    d = torch.tensor([-1.0, 0.0, 1.0], device=DEV, dtype=torch.float64)
    tot = s.sum((1, 2))
    c = torch.stack([(s.sum(2) * d).sum(1), (s.sum(1) * d).sum(1)], 1) / tot.clamp(min=1e-300)[:, None]
    return torch.where(tot[:, None] > 0, c, 0.0)


def _exact_frames(case, seed, kind="frames"):
    """Per distinct frame, then repeated as the batch repeats them."""
    ped, gain = _calibration(case["det"], seed)
    pool = _pool(case, seed, ped, gain)
    P, n = pool.shape[0], case["n"]
    T, H, W, _, _ = DETECTORS[case["det"]]
    step = max(1, 20000000 // (T * H * W))
    theta = torch.as_tensor(_theta(seed), device=DEV).double() if kind == "subpixel" else None
    charges, counts, corr, pos = [], [], [], []
    for f in range(0, P, step):
        v32, v64 = _corrected64(case, pool[f:f + step], ped, gain)
        at, q = _hits64(v32, v64)
        charges.append(q)
        counts.append(torch.bincount(at[:, 0], minlength=v32.shape[0]))
        if kind == "analysis":
            corr.append(v64.reshape(v64.shape[0], -1))
        if kind == "subpixel":
            p = _patches64(v64, at)
            y = _mlp64(theta, p / ADU)
            bad = ~((y.abs() <= 1.0).all(1, keepdim=True))
            pos.append(torch.where(bad, _centroid64(p), y))
    q, first = torch.cat(charges), [0] + torch.cat(counts).cumsum(0).tolist()

    def repeat(x, per):  # rows of the pool's frames, `per[f]` the first row of frame f
        whole, rest = n // P, n % P
        return torch.cat([x] * whole + [x[:per[rest]]])

    def fill(x):  # to the size of the destination
        room = torch.zeros((_hit_capacity(case, case["det"]),) + tuple(x.shape[1:]), dtype=x.dtype, device=DEV)
        m = min(len(room), len(x))
        room[:m] = x[:m]
        return room

    out = {"frame": None, "pixel": None, "charge": fill(repeat(q, first)), "nphot": None, "frame_hits": None,
           "frame_photons": None, "total": None}
    if kind == "analysis":
        out.update(corrected=repeat(torch.cat(corr), list(range(P + 1))), map=None, spectrum=None, sizes=None,
                   hist=None)
    if kind == "subpixel":
        out["positions"] = fill(repeat(torch.cat(pos), first))
    return out


def _exact_patches(case, seed):
    p, _ = _patches(case["n"], seed)
    s, _ = _patches(65536, seed + 1)
    nb = ETA_BINS
    # the table's bins are decided in binary32, its values are counts over their number
    c = _centroid64(s.double()).float()
    b = torch.floor((c.clamp(-1.0, 1.0) + 1.0) * 0.5 * float(nb)).long().clamp(max=nb - 1)
    cdf = [torch.cat([torch.zeros(1, device=DEV, dtype=torch.float64),
                      torch.bincount(b[:, a], minlength=nb).double().cumsum(0) / 65536.0]) for a in (0, 1)]
    theta = torch.as_tensor(_theta(seed), device=DEV).double()
    learned, classical = [], []
    for i in range(0, case["n"], 1 << 20):
        x = p[i:i + (1 << 20)].double()
        learned.append(_mlp64(theta, x / ADU))
        t = (_centroid64(x).clamp(-1.0, 1.0) + 1.0) * 0.5 * nb
        k = torch.floor(t).long().clamp(max=nb - 1)
        f = t - k
        classical.append(torch.stack([cdf[a][k[:, a]] * (1 - f[:, a]) + cdf[a][k[:, a] + 1] * f[:, a] - 0.5
                                      for a in (0, 1)], 1))
    return {"learned": torch.cat(learned), "classical": torch.cat(classical)}


def _exact_train(case, seed):
    n = case["n"]
    p, truth = _patches(n * TRAIN_STEPS, seed)
    th = torch.as_tensor(_theta(seed), device=DEV).double().requires_grad_(True)
    m = torch.zeros_like(th)
    v = torch.zeros_like(th)
    loss = None
    for k in range(TRAIN_STEPS):
        x, t = p[k * n:(k + 1) * n].double() / ADU, truth[k * n:(k + 1) * n].double()
        loss = ((_mlp64(th, x) - t) ** 2).sum() / (2 * n)
        (g,) = torch.autograd.grad(loss, th)
        with torch.no_grad():
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            th -= LR * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return {"theta": th.detach().cpu().numpy(), "loss": float(loss)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("frames", "analysis", "subpixel"):
        return _exact_frames(case, seed, kind)
    if kind == "mixed":
        return [_exact_frames(dict(case, kind="frames", det=d), seed + 1000 * i) for i, d in enumerate(MIX)]
    if kind == "patches":
        return _exact_patches(case, seed)
    return _exact_train(case, seed)
