"""pdc_process_frames_static at the limits of its arguments and of its scratch:
counts without a record list, and the frame counts it has room for."""
import numpy as np
import pytest

from oracle import cm_mean as M
from paper_1903_06838_amd import synth
from tests.helpers import oracle_threads

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = pdc.create(0)
    yield c
    pdc.destroy(c)


# few units (one launch for totals and offsets), more than it takes, and the general kernel
@pytest.mark.parametrize("geom,n,cm_mode", [
    (synth.Geometry(2, 40, 388, 194), 5, 0),
    (synth.Geometry(1, 8, 16, 8), 17000, 0),
    (synth.Geometry(1, 33, 194, 97), 3, M.BANK),
], ids=["few", "many", "general"])
def test_static_counts_alone(ctx, geom, n, cm_mode):
    """hits_dev NULL with capacity 0: the counts of a call with a list, and its
    status for a list that is too short."""
    import torch

    from paper_1903_06838_amd import pdc

    ped, gain = synth.make_calibration(geom, 63)
    raw = synth.make_frames(geom, ped, gain, n, 0.02, 63)
    if cm_mode:
        want = M.process(raw, ped, gain, geom.bank_cols, cm_mode, 1)
    else:
        want = oracle_threads(raw, ped, gain, geom.bank_cols)
    assert want["total"] > 0
    prm = pdc.params(cm_mode=cm_mode)
    det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, geom.bank_cols), ped, gain, prm)
    dev = torch.from_numpy(raw).cuda()
    fh = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    fp = torch.full((n,), 7, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    st, total = pdc.process_frames_static(ctx, det, dev, n, None, 0, fh, fp)
    assert st == pdc.WARN_TRUNCATED and total == want["total"]
    assert np.array_equal(fh.cpu().numpy().view(np.uint32), want["frame_hits"])
    assert np.array_equal(fp.cpu().numpy().view(np.uint64), want["frame_photons"])


def _compare(ctx, geom, raw, ped, gain):
    """A static call against pdc_process_frames and pdc_get_hits."""
    import torch

    from paper_1903_06838_amd import pdc

    n = raw.shape[0]
    det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, geom.bank_cols), ped, gain, pdc.params())
    dev = torch.from_numpy(raw).cuda()
    b = pdc.process_frames(ctx, det, dev, n, raw.size // 8)
    hits, total, fh, fp, _ = pdc.get_hits(ctx, b, n)
    pdc.release_batch(ctx, b)
    assert total > 0
    recs = torch.full((total, 4), -1, dtype=torch.int32, device="cuda")
    fh_s = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    fp_s = torch.full((n,), 7, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    st, tot_s = pdc.process_frames_static(ctx, det, dev, n, recs, total, fh_s, fp_s)
    assert st == pdc.OK and tot_s == total
    assert np.array_equal(fh_s.cpu().numpy().view(np.uint32), fh)
    assert np.array_equal(fp_s.cpu().numpy().view(np.uint64), fp)
    assert np.array_equal(recs.cpu().numpy().view(np.uint32), np.ascontiguousarray(hits).view(np.uint32).reshape(-1, 4))


# the launch's own frame groups leave the pool no room, then one group's chunks
# of 8,192 hits, then any of the persistent kernel's
@pytest.mark.parametrize("geom,n", [
    (synth.CSPAD, 15),
    (synth.Geometry(8, 512, 1024, 256), 8),
    (synth.Geometry(1, 1024, 1024, 64), 20),
    (synth.Geometry(2, 1313, 2016, 96), 1),
    (synth.Geometry(1, 1436, 1240, 31), 2),
    (synth.Geometry(4, 1620, 574, 14), 1),
    (synth.Geometry(2, 1313, 1900, 100), 1),
], ids=lambda v: "x".join(map(str, v.shape)) if hasattr(v, "shape") else str(v))
def test_static_takes_what_fits(ctx, geom, n):
    ped, gain = np.full(geom.shape, 1000.0, np.float32), np.ones(geom.shape, np.float32)
    one = synth.make_frames(geom, ped, gain, 1, 0.01, 64)
    raw = np.concatenate([np.roll(one, 7 * f, axis=3) for f in range(n)])
    _compare(ctx, geom, raw, ped, gain)


def test_static_overflow_takes_fewer_groups(ctx):
    """A hit on every ninth pixel: with the chunks of several frame groups open
    the pool is too small, with one group's it is not."""
    geom = synth.CSPAD
    ped = np.full(geom.shape, 1000.0, np.float32)
    gain = np.ones(geom.shape, np.float32)
    raw = np.full((15, *geom.shape), 1000, np.uint16)
    raw[:, :, ::3, ::3] = 1200
    _compare(ctx, geom, raw, ped, gain)
