"""Batches that are run again: staging overflow on the general kernel, eager and
replayed from a graph, and strips of wide banks whose lists overflow and are
redone by the general kernel.  Against the oracles, bit for bit."""
import os

import numpy as np
import pytest

from oracle import cm_mean as M
from paper_1903_06838_amd import synth
from tests.helpers import assert_same, oracle_threads

pytestmark = pytest.mark.gpu


def _create(**env):
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    os.environ.update(env)
    try:
        return pdc.create(0)
    finally:
        for k in env:
            del os.environ[k]


def _check(ctx, b, raw, want, path):
    from paper_1903_06838_amd import pdc

    hits, total, fh, fp, _ = pdc.get_hits(ctx, b, raw.shape[0])
    corr = np.empty(raw.shape, np.float32)
    pdc.get_corrected(ctx, b, corr)
    assert pdc.debug_batch_path(ctx, b) == path
    assert_same(dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp, corrected=corr), want, corrected=True)


@pytest.mark.parametrize("B,cm_mode,force", [(514, 0, "0"), (97, M.BANK, "0"), (194, 0, "1"), (194, M.TILE, "1")], ids=str)
def test_general_kernel_overflow(B, cm_mode, force):
    import torch

    from paper_1903_06838_amd import pdc

    geom, n = synth.Geometry(2, 40, 2 * B, B), 5
    ped, gain = synth.make_calibration(geom, 91)
    raw = synth.make_frames(geom, ped, gain, n, 0.04, 91, sim=synth.SimParams(cm_sigma=1.0))
    if cm_mode:
        want = M.process(raw, ped, gain, B, cm_mode, 1, keep_corrected=True)
    else:
        want = oracle_threads(raw, ped, gain, B, keep_corrected=True)
    assert want["total"] > 100
    ctx = _create(PDC_DEBUG_TIGHT_POOL="1", PDC_FORCE_GENERAL=force)
    try:
        det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, B), ped, gain,
                            pdc.params(flags=pdc.KEEP_CORRECTED, cm_mode=cm_mode))
        dev = torch.from_numpy(raw).cuda()
        torch.cuda.synchronize()
        for capacity in (0, 60, raw.size):  # no room, room for some units, room for all
            b = pdc.process_frames(ctx, det, dev, n, capacity)
            _check(ctx, b, raw, want, 1)
            pdc.release_batch(ctx, b)
        for capacity in (0, raw.size):  # the batch leaves the graph's buffers, or not
            graph = pdc.graph_create(ctx, det, dev, n, capacity)
            for _ in range(3):
                b = pdc.graph_launch(ctx, graph)
                _check(ctx, b, raw, want, 1)
                pdc.release_batch(ctx, b)
            pdc.graph_destroy(ctx, graph)
    finally:
        pdc.destroy(ctx)


@pytest.mark.parametrize("tiles", [1, 3])
def test_wide_banks_flood(tiles):
    """Seeds on 485 of 1,024 columns of every row: at least 13 x 485 a strip,
    more than the two fifths of its 15 rows that the lists hold."""
    import torch

    from paper_1903_06838_amd import pdc

    geom, B = synth.Geometry(tiles, 40, 1024, 512), 512
    ped, gain = np.full(geom.shape, 1000.0, np.float32), np.ones(geom.shape, np.float32)
    raw = np.full((3, *geom.shape), 1000, np.uint16)
    bright = np.zeros(1024, bool)
    for k in range(4):
        bright[k::9] = True
    bright[4::36] = True
    assert bright[:512].sum() < 256 and bright[512:].sum() < 256 and 13 * bright.sum() > 2 * 15 * 1024 // 5
    r, c = np.indices((40, 1024))
    raw[1][:, bright[c[0]][None, :].repeat(40, 0)] = (1200 + (7 * c + 13 * r) % 61)[:, bright].reshape(-1)
    want = oracle_threads(raw, ped, gain, B, keep_corrected=True)
    assert want["total"] > 1000
    ctx = _create()
    try:
        det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, B), ped, gain, pdc.params(flags=pdc.KEEP_CORRECTED))
        dev = torch.from_numpy(raw).cuda()
        torch.cuda.synchronize()
        b = pdc.process_frames(ctx, det, dev, 3, raw.size)
        _check(ctx, b, raw, want, 3)
        pdc.release_batch(ctx, b)
    finally:
        pdc.destroy(ctx)
