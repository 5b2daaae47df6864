"""Frame numbers of the hit records: batches whose frames are empty, sparse or
full, so that one wave's run of hits lies in one frame, crosses a boundary, or
spans many (empty ones included), at frame counts around the 64 probes of the
search, and destinations that hold only the first part.  The frame of every
record follows from the per-frame counts."""
import numpy as np
import pytest

from paper_1903_06838_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129, 4095, 4097])
def test_record_frames(n):
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    geom = synth.Geometry(1, 16, 64, 32)
    ped = np.full(geom.shape, 1000.0, np.float32)
    gain = np.ones(geom.shape, np.float32)
    raw = np.full((n, *geom.shape), 1000, np.uint16)
    rng = np.random.default_rng(n)
    kind = rng.integers(0, 3, n)  # empty, one photon, many
    raw[kind == 1, 0, 8, 31] = 1160
    raw[kind == 2, :, 1::3, 1::5] = 1160
    c = pdc.create(0)
    try:
        det = pdc.calibrate(c, pdc.geometry(1, 16, 64, 32), ped, gain, pdc.params(3.0, 5.0, 3.0, 150.0, 0))
        b = pdc.process_frames(c, det, torch.from_numpy(raw.view(np.int16)).cuda(), n, raw.size)
        hits, total, fh, _, _ = pdc.get_hits(c, b, n)
        assert np.array_equal(fh, np.array([0, 1, 5 * 13])[kind])
        frames = np.repeat(np.arange(n, dtype=np.uint32), fh)
        assert total == len(hits) == len(frames)
        assert np.array_equal(hits["frame"], frames)
        assert np.all(hits["nphot"] == 1) and np.all(hits["charge"] == 160.0)
        for cap in (1, 511, 512, 513):
            if cap < total:
                part = pdc.get_hits(c, b, n, capacity=cap)[0]
                assert np.array_equal(part, hits[:cap])
        pdc.release_batch(c, b)
    finally:
        pdc.destroy(c)


@pytest.mark.parametrize("cap", [1, 4095, 4096, 4097, 16384, 16385, 65536, 65537, 90000])
def test_host_destinations(cap):
    """Host destinations around the sizes of the pinned staging: the records of
    one batch, whole and cut, against its device copy."""
    import torch

    from paper_1903_06838_amd import pdc

    geom = synth.Geometry(2, 60, 388, 194)
    ped, gain = synth.make_calibration(geom, 3)
    raw = synth.make_frames(geom, ped, gain, 40, 0.06, 3)
    c = pdc.create(0)
    try:
        det = pdc.calibrate(c, pdc.geometry(2, 60, 388, 194), ped, gain, pdc.params(3.0, 5.0, 3.0, 150.0, 0))
        b = pdc.process_frames(c, det, torch.from_numpy(raw).cuda(), 40, raw.size // 8)
        total = pdc.get_hits(c, b, 40, capacity=0)[1]
        assert total > 65537
        rec = torch.zeros((total, 4), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        pdc.get_hits(c, b, 40, total, rec)
        want = rec.cpu().numpy().tobytes()
        for n in (cap, total, cap):
            hits = pdc.get_hits(c, b, 40, capacity=n)[0]
            assert hits.tobytes() == want[:16 * min(n, total)]
        pdc.release_batch(c, b)
    finally:
        pdc.destroy(c)
