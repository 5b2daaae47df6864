"""The persistent kernel on widths off its 4-column grid, and on banks wider than
256 columns, bit for bit against the oracles: banks of an odd width (the last column of each has no partner, and
banks and rows start at odd columns and addresses) around every lane layout's
capacity, rows of an even width that is no multiple of 4, with and without
Frames2, one frame and several, at the buffer's last pixel, and where a strip's
seed lists overflow."""
import numpy as np
import pytest

from oracle import cm_mean as M
from paper_1903_06838_amd import synth
from tests.helpers import assert_same, oracle_threads

pytestmark = pytest.mark.gpu

# bank width, banks per row
ODD = [(3, 1), (3, 5), (5, 8), (7, 3), (9, 2), (31, 1), (33, 3), (63, 2), (65, 1), (65, 2), (95, 2), (97, 1), (97, 2),
       (127, 1), (127, 3), (129, 1), (185, 2), (193, 2), (199, 1), (201, 1), (255, 1), (255, 2), (255, 8)]
EVEN = [(6, 1), (6, 3), (62, 1), (66, 1), (98, 1), (126, 3), (130, 1), (194, 1), (202, 1), (254, 1)]


def _process(raw, ped, gain, B, keep, cm_mode=0, stages=1):
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ctx = pdc.create(0)
    try:
        N, T, H, W = raw.shape
        prm = pdc.params(3.0, 5.0, 3.0, 150.0, pdc.KEEP_CORRECTED if keep else 0, cm_mode=cm_mode, cm_stages=stages)
        det = pdc.calibrate(ctx, pdc.geometry(T, H, W, B), ped, gain, prm)
        b = pdc.process_frames(ctx, det, torch.from_numpy(raw).cuda(), N, max(1024, raw.size // 4))
        hits, total, fh, fp, _ = pdc.get_hits(ctx, b, N)
        out = dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp)
        if keep:
            out["corrected"] = np.empty(raw.shape, np.float32)
            pdc.get_corrected(ctx, b, out["corrected"])
        path = pdc.debug_batch_path(ctx, b)
        pdc.release_batch(ctx, b)
        return out, path
    finally:
        pdc.destroy(ctx)


@pytest.mark.parametrize("B,nb", ODD + EVEN, ids=lambda v: str(v))
@pytest.mark.parametrize("n,keep", [(1, True), (5, True), (6, False)])
def test_widths(B, nb, n, keep):
    geom = synth.Geometry(2, 33, B * nb, B)
    ped, gain = synth.make_calibration(geom, 500 + B)
    raw = synth.make_frames(geom, ped, gain, n, 0.03, 500 + B)
    raw[-1, -1, -1, -1] = int(ped[-1, -1, -1]) + 400  # a photon on the buffer's last pixel
    want = oracle_threads(raw, ped, gain, B, keep_corrected=keep)
    got, path = _process(raw, ped, gain, B, keep)
    assert path in (2, 3)
    assert_same(got, want, corrected=keep)


def test_odd_banks_flood():
    """A photon on every fourth pixel of one strip: its lists overflow and the
    general kernel redoes it."""
    geom = synth.Geometry(2, 40, 388, 97)
    ped = np.full(geom.shape, 1000.0, np.float32)
    gain = np.ones(geom.shape, np.float32)
    raw = np.full((3, *geom.shape), 1000, np.uint16)
    raw[1, 0, :, 0::9] = raw[1, 0, :, 1::9] = raw[1, 0, :, 2::9] = raw[1, 0, :, 3::9] = 1200
    want = oracle_threads(raw, ped, gain, 97, keep_corrected=True)
    got, path = _process(raw, ped, gain, 97, True)
    assert path == 3
    assert_same(got, want, corrected=True)


@pytest.mark.parametrize("cm_mode", [M.BANK, M.TILE])
def test_odd_banks_mean(cm_mode):
    """A thresholded mean over odd banks stays on the general kernel; over rows
    off the 4-column grid it takes the persistent one."""
    for B, nb, paths in ((97, 2, (1,)), (66, 1, (2, 3))):
        geom = synth.Geometry(1, 33, B * nb, B)
        ped, gain = synth.make_calibration(geom, 41)
        raw = synth.make_frames(geom, ped, gain, 3, 0.02, 41, sim=synth.SimParams(cm_sigma=1.0))
        want = M.process(raw, ped, gain, B, cm_mode, 2, keep_corrected=True)
        got, path = _process(raw, ped, gain, B, True, cm_mode, 2)
        assert path in paths
        assert_same(got, want, corrected=True)


@pytest.mark.parametrize("B,nb", [(258, 1), (258, 2), (300, 3), (384, 1), (510, 4), (512, 1), (512, 2), (512, 4),
                                  (257, 1), (511, 2), (514, 1)])
@pytest.mark.parametrize("n,keep", [(1, True), (5, True), (6, False)])
def test_wide_banks(B, nb, n, keep):
    """Even widths up to 512 take the persistent kernel, the others the general one."""
    geom = synth.Geometry(2, 33, B * nb, B)
    ped, gain = synth.make_calibration(geom, 700 + B)
    raw = synth.make_frames(geom, ped, gain, n, 0.03, 700 + B)
    want = oracle_threads(raw, ped, gain, B, keep_corrected=keep)
    got, path = _process(raw, ped, gain, B, keep)
    assert path in ((2, 3) if B % 2 == 0 and B <= 512 else (1,))
    assert_same(got, want, corrected=keep)


def test_wide_banks_flood():
    geom = synth.Geometry(1, 40, 1024, 512)
    ped = np.full(geom.shape, 1000.0, np.float32)
    gain = np.ones(geom.shape, np.float32)
    raw = np.full((3, *geom.shape), 1000, np.uint16)
    for k in range(4):
        raw[1, 0, :12, k::9] = 1200
    want = oracle_threads(raw, ped, gain, 512, keep_corrected=True)
    got, path = _process(raw, ped, gain, 512, True)
    assert path in (2, 3)
    assert_same(got, want, corrected=True)


@pytest.mark.parametrize("B,nb", [(97, 2), (199, 1), (300, 2), (512, 2)])
def test_graph_and_kept_medians(B, nb):
    """The same batches replayed from a graph, and their patches from kept
    medians against those from kept Frames2."""
    import torch

    from paper_1903_06838_amd import pdc

    geom, n = synth.Geometry(1, 40, B * nb, B), 4
    ped, gain = synth.make_calibration(geom, 800 + B)
    raw = synth.make_frames(geom, ped, gain, n, 0.03, 800 + B)
    want = oracle_threads(raw, ped, gain, B)
    dev = torch.from_numpy(raw).cuda()
    ctx = pdc.create(0)
    try:
        got = []
        for flag in (pdc.KEEP_CORRECTED, pdc.KEEP_MEDIANS):
            det = pdc.calibrate(ctx, pdc.geometry(1, 40, B * nb, B), ped, gain, pdc.params(3.0, 5.0, 3.0, 150.0, flag))
            graph = pdc.graph_create(ctx, det, dev, n, raw.size)
            for _ in range(3):
                b = pdc.graph_launch(ctx, graph)
                hits, total, fh, fp, _ = pdc.get_hits(ctx, b, n)
                assert_same(dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp), want)
                out = torch.zeros((total, 25), dtype=torch.float32, device="cuda")
                torch.cuda.synchronize()
                assert pdc.capture_patches(ctx, b, out, total) == total
                pdc.release_batch(ctx, b)
            got.append(out.cpu().numpy().view(np.uint32))
        assert np.array_equal(got[0], got[1])
    finally:
        pdc.destroy(ctx)
