"""Per-frame counts, offsets and the raster-ordered list at the edges of the one
launch that forms them for batches of few units: fewer and more units than a
workgroup's 16, frames that start inside one, one unit a frame and more than
its limit, unit counts around the limit, and frame counts around the number
whose totals are kept in pinned memory.  Against the oracle, bit for bit."""
import os

import numpy as np
import pytest

from paper_1903_06838_amd import synth
from tests.helpers import assert_same, oracle_threads

pytestmark = pytest.mark.gpu

# rows of one 8-column tile (one row a strip, so as many units a frame), frames
CASES = [(1, 1), (1, 15), (1, 16), (1, 17), (3, 5), (3, 11), (15, 2), (16, 3), (17, 3), (33, 4), (1023, 2), (1024, 2),
         (1025, 2), (1024, 16), (1024, 17), (2, 8192), (2, 8193), (1, 16384), (1, 16385), (1, 65536), (1, 65537)]


@pytest.mark.parametrize("rows,n", CASES)
def test_tail(rows, n):
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    geom = synth.Geometry(1, rows, 8, 8)
    ped, gain = synth.make_calibration(geom, rows)
    raw = synth.make_frames(geom, ped, gain, n, 0.05, rows)
    want = oracle_threads(raw, ped, gain, 8)
    os.environ["PDC_STRIP_ROWS"] = "1"
    try:
        ctx = pdc.create(0)
    finally:
        del os.environ["PDC_STRIP_ROWS"]
    try:
        det = pdc.calibrate(ctx, pdc.geometry(1, rows, 8, 8), ped, gain, pdc.params(3.0, 5.0, 3.0, 150.0, 0))
        dev = torch.from_numpy(raw).cuda()
        for _ in range(2):  # a fresh batch, then one on its released buffers
            b = pdc.process_frames(ctx, det, dev, n, raw.size)
            hits, total, fh, fp, _ = pdc.get_hits(ctx, b, n)
            assert_same(dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp), want)
            main, whole = pdc.batch_timing(ctx, b)
            assert 0.0 < main < 1e3 and 0.0 < whole < 1e3
            pdc.release_batch(ctx, b)
    finally:
        pdc.destroy(ctx)
