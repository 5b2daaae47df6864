"""Frame groups of detectors of few strips, around the 64 and 128 groups that a
launch has at most: every frame once, bit for bit against the oracle, eager and
through the static call."""
import numpy as np
import pytest

from paper_1903_06838_amd import synth
from tests.helpers import assert_same, oracle_threads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 130, 400])
@pytest.mark.parametrize("T,H,W,B", [(1, 16, 32, 16), (3, 8, 32, 16), (7, 8, 32, 16), (9, 8, 32, 16), (2, 12, 512, 512)], ids=str)
def test_groups(T, H, W, B, n):
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    geom = synth.Geometry(T, H, W, B)
    ped, gain = synth.make_calibration(geom, n)
    raw = synth.make_frames(geom, ped, gain, n, 0.03, n)
    want = oracle_threads(raw, ped, gain, B)
    ctx = pdc.create(0)
    try:
        det = pdc.calibrate(ctx, pdc.geometry(T, H, W, B), ped, gain, pdc.params())
        dev = torch.from_numpy(raw).cuda()
        torch.cuda.synchronize()
        b = pdc.process_frames(ctx, det, dev, n, raw.size // 8)
        hits, total, fh, fp, _ = pdc.get_hits(ctx, b, n)
        assert pdc.debug_batch_path(ctx, b) in (2, 3)
        pdc.release_batch(ctx, b)
        assert_same(dict(hits=hits, total=total, frame_hits=fh, frame_photons=fp), want)
        recs = torch.full((total + 1, 4), -1, dtype=torch.int32, device="cuda")
        fh_s, fp_s = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        assert pdc.process_frames_static(ctx, det, dev, n, recs, total, fh_s, fp_s) == (pdc.OK, total)
        assert np.array_equal(recs[:total].cpu().numpy().view(np.uint32), np.ascontiguousarray(hits).view(np.uint32).reshape(-1, 4))
        assert np.array_equal(fh_s.cpu().numpy().view(np.uint32), want["frame_hits"])
    finally:
        pdc.destroy(ctx)
