"""Lane layouts of the persistent kernel at their edges, bit for bit against the
oracles: bank widths around every compiled capacity (64, 96, 128, 200 and 256
pixels), banks that end inside a lane's group of columns, strips of every
height up to the fullest, strips across tile edges, and enough frames for
every buffer that alternates between frames to come round."""
import os

import numpy as np
import pytest

from oracle import cm_mean as M
from oracle import multigain as G
from paper_1903_06838_amd import synth
from tests.helpers import assert_same, oracle_threads

pytestmark = pytest.mark.gpu

# bank widths (even) around the layouts' capacities, and the banks per row
EDGES = [(2, 2), (6, 6), (62, 2), (64, 4), (66, 2), (94, 2), (96, 1), (98, 2), (126, 2), (128, 3), (130, 2), (192, 2),
         (194, 4), (198, 2), (200, 1), (202, 2), (254, 2), (256, 4)]
FEW_LOW_GAIN = dict(range_frac=(0.985, 0.008, 0.003), invalid_frac=0.01)


def _process(raw, ped, gain, B, gain_mode=0, cm_mode=0, stages=1, strip_rows=None):
    import torch

    from paper_1903_06838_amd import pdc

    if strip_rows:
        os.environ["PDC_STRIP_ROWS"] = str(strip_rows)
    try:
        ctx = pdc.create(0)
    finally:
        os.environ.pop("PDC_STRIP_ROWS", None)
    try:
        N, T, H, W = raw.shape
        prm = pdc.params(3.0, 5.0, 3.0, 150.0, pdc.KEEP_CORRECTED, cm_mode=cm_mode, cm_stages=stages)
        det = pdc.calibrate(ctx, pdc.geometry(T, H, W, B, gain_mode), ped, gain, prm)
        b = pdc.process_frames(ctx, det, torch.from_numpy(raw).cuda(), N, max(1024, raw.size // 10))
        hits, total, fh, fp, _ = pdc.get_hits(ctx, b, N)
        corr = np.empty(raw.shape, np.float32)
        pdc.get_corrected(ctx, b, corr)
        path = pdc.debug_batch_path(ctx, b)
        pdc.release_batch(ctx, b)
        return dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp, corrected=corr), path
    finally:
        pdc.destroy(ctx)


@pytest.mark.parametrize("B,nb", EDGES, ids=lambda v: str(v))
@pytest.mark.parametrize("gain_mode,cm_mode", [(0, 0), (1, 0), (0, M.BANK)], ids=["median", "ranges", "mean"])
def test_layout_edges(B, nb, gain_mode, cm_mode):
    W = B * nb
    if gain_mode == 0 and W % 4:
        pytest.skip("single-gain rows of a multiple of 4 columns only")
    geom = synth.Geometry(2, 33, W, B)
    seed = 900 + B
    sim = synth.SimParams(cm_sigma=2.0) if cm_mode else synth.SimParams()
    if gain_mode:
        ped, gain = synth.make_calibration_multigain(geom, seed)
        raw = synth.make_frames_multigain(geom, ped, gain, 6, 0.02, seed, gain_mode, **FEW_LOW_GAIN)
        want = G.process(raw, ped, gain, B, gain_mode, keep_corrected=True)
    else:
        ped, gain = synth.make_calibration(geom, seed)
        raw = synth.make_frames(geom, ped, gain, 6, 0.02, seed, sim=sim)
        if cm_mode:
            want = M.process(raw, ped, gain, B, cm_mode, 2, keep_corrected=True)
        else:
            want = oracle_threads(raw, ped, gain, B, keep_corrected=True)
    got, path = _process(raw, ped, gain, B, gain_mode, cm_mode, 2 if cm_mode else 1)
    assert path in (2, 3)
    assert_same(got, want, corrected=True)


@pytest.mark.parametrize("rows", [1, 2, 7, 29])
def test_short_strips_and_tile_edges(rows):
    geom = synth.Geometry(3, 31, 388, 194)
    ped, gain = synth.make_calibration(geom, 77)
    raw = synth.make_frames(geom, ped, gain, 5, 0.03, 77)
    want = oracle_threads(raw, ped, gain, 194, keep_corrected=True)
    got, path = _process(raw, ped, gain, 194, strip_rows=rows)
    assert path in (2, 3)
    assert_same(got, want, corrected=True)
