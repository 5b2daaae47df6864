"""The persistent kernel on rows of many banks, bit for bit against the oracles:
every lane layout with as few rows a strip as it takes (one to six own rows
beside the two halo rows), the two-pass layout's first number of banks and the
last one-pass one, and strips over tile edges."""
import numpy as np
import pytest

from oracle import cm_mean as M
from oracle import multigain as G
from paper_1903_06838_amd import synth
from tests.helpers import assert_same, oracle_threads

pytestmark = pytest.mark.gpu

# bank width, banks per row
MANY = [(14, 42), (64, 32), (66, 31), (96, 21), (98, 10), (98, 11), (98, 20), (100, 13), (100, 18), (126, 12), (128, 16),
        (130, 15), (190, 10), (200, 10), (202, 10), (256, 8)]
ODD = [(31, 42), (63, 32), (95, 21), (97, 10), (97, 21), (127, 11), (127, 16), (129, 15), (255, 8)]
FEW_LOW_GAIN = dict(range_frac=(0.985, 0.008, 0.003), invalid_frac=0.01)


@pytest.fixture(scope="module")
def ctx():
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = pdc.create(0)
    yield c
    pdc.destroy(c)


def _case(B, nb, mode, n=3):
    geom, seed = synth.Geometry(2, 21, B * nb, B), 1100 + B
    if mode == "ranges":
        ped, gain = synth.make_calibration_multigain(geom, seed)
        raw = synth.make_frames_multigain(geom, ped, gain, n, 0.02, seed, 1, **FEW_LOW_GAIN)
        return geom, raw, ped, gain, 1, 0, G.process(raw, ped, gain, B, 1, keep_corrected=True)
    ped, gain = synth.make_calibration(geom, seed)
    sim = synth.SimParams(cm_sigma=2.0) if mode == "mean" else synth.SimParams()
    raw = synth.make_frames(geom, ped, gain, n, 0.02, seed, sim=sim)
    if mode == "mean":
        return geom, raw, ped, gain, 0, M.BANK, M.process(raw, ped, gain, B, M.BANK, 2, keep_corrected=True)
    return geom, raw, ped, gain, 0, 0, oracle_threads(raw, ped, gain, B, keep_corrected=True)


@pytest.mark.parametrize("B,nb,mode", [(B, nb, m) for B, nb in MANY for m in ("median", "ranges", "mean")] +
                         [(B, nb, "median") for B, nb in ODD], ids=str)
def test_many_banks(ctx, B, nb, mode):
    import torch

    from paper_1903_06838_amd import pdc

    geom, raw, ped, gain, gm, cm, want = _case(B, nb, mode)
    n = raw.shape[0]
    prm = pdc.params(3.0, 5.0, 3.0, 150.0, pdc.KEEP_CORRECTED, cm_mode=cm, cm_stages=2 if cm else 1)
    det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, B, gm), ped, gain, prm)
    try:
        b = pdc.process_frames(ctx, det, torch.from_numpy(raw).cuda(), n, raw.size // 8)
        hits, total, fh, fp, _ = pdc.get_hits(ctx, b, n)
        corr = np.empty(raw.shape, np.float32)
        pdc.get_corrected(ctx, b, corr)
        path = pdc.debug_batch_path(ctx, b)
        pdc.release_batch(ctx, b)
    finally:
        pdc.release_detector(ctx, det)
    assert path in (2, 3)
    assert_same(dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp, corrected=corr), want, corrected=True)


@pytest.mark.parametrize("B,nb,rows", [(98, 10, 4), (100, 13, 7), (100, 18, 5), (128, 12, 6)])
def test_strip_heights(ctx, B, nb, rows):
    """Own rows a strip: a workgroup holds 128 bank-rows of up to 128 columns in
    two passes (8 rows of 1,536 pixels fit its LDS), 64 in one, less the two
    halo rows."""
    import torch

    from paper_1903_06838_amd import pdc

    geom = synth.Geometry(1, 64, B * nb, B)
    ped, gain = np.full(geom.shape, 1000.0, np.float32), np.ones(geom.shape, np.float32)
    frames = torch.full((2, *geom.shape), 1000, dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, B), ped, gain, pdc.params())
    try:
        got, _, ms = pdc.autotune_strips(ctx, det, frames, 2, 1024)
        assert got == rows and len(ms) == 1
    finally:
        pdc.release_detector(ctx, det)


@pytest.mark.parametrize("other,one", [((100, 13, "median"), True), ((100, 18, "ranges"), True), ((97, 2, "median"), False),
                                       ((300, 2, "median"), False)], ids=str)
def test_mixed(ctx, other, one):
    """Beside a CSPAD-like detector: the two-pass layout shares the one launch,
    an odd-bank or wide-bank detector makes the batches launch on their own."""
    import torch

    from paper_1903_06838_amd import pdc

    cases = [_case(194, 2, "median", 5), _case(*other)]
    dets, devs = [], []
    try:
        for geom, raw, ped, gain, gm, _, _ in cases:
            dets.append(pdc.calibrate(ctx, pdc.geometry(*geom.shape, geom.bank_cols, gm), ped, gain, pdc.params()))
            devs.append(torch.from_numpy(raw).cuda())
        torch.cuda.synchronize()
        batches = pdc.process_mixed(ctx, [(d, f, f.shape[0], 1 << 16) for d, f in zip(dets, devs)])
        for b, case in zip(batches, cases):
            n = case[1].shape[0]
            hits, total, fh, fp, _ = pdc.get_hits(ctx, b, n)
            assert_same(dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp), case[-1])
            assert pdc.debug_batch_path(ctx, b) in ((4, 5) if one else (2, 3))
            pdc.release_batch(ctx, b)
    finally:
        for d in dets:
            pdc.release_detector(ctx, d)
