"""Patches into destinations shorter than the batch's hit list: they end at, just
before and just after a frame's last hit, with empty frames between, and hold
the first patches of the whole capture; nothing past them is written."""
import numpy as np
import pytest

from paper_1903_06838_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flag", [1, 2], ids=["corrected", "medians"])
@pytest.mark.parametrize("B,nb,n", [(194, 2, 40), (97, 2, 40), (8, 4, 3000)], ids=str)
def test_short_destinations(B, nb, n, flag):
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    geom = synth.Geometry(2, 20, B * nb, B)
    ped, gain = synth.make_calibration(geom, 7)
    raw = synth.make_frames(geom, ped, gain, 40, 0.02, 7)
    dark = np.rint(ped).astype(np.uint16)
    for f in (0, 1, 5, 6, 17, 39):
        raw[f] = dark  # no photon
    raw = np.tile(raw, (n // 40 + 1, 1, 1, 1))[:n]
    ctx = pdc.create(0)
    try:
        det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, B), ped, gain, pdc.params(flags=flag))
        dev = torch.from_numpy(raw).cuda()
        torch.cuda.synchronize()
        b = pdc.process_frames(ctx, det, dev, n, raw.size // 8)
        _, total, fh, _, _ = pdc.get_hits(ctx, b, n)
        assert fh[0] == fh[5] == fh[39] == 0 and total > 500
        whole = torch.zeros((total, 25), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        assert pdc.capture_patches(ctx, b, whole, total) == total
        ends = np.cumsum(fh)[[2, 4, 7, 18, n // 2, n - 2]]
        for cap in sorted({0, 1, 11, 12, 13, total - 1} | {int(e) + d for e in ends for d in (-1, 0, 1)}):
            m = min(cap, total)
            out = torch.full((m + 2, 25), -1.0, dtype=torch.float32, device="cuda")
            words = torch.full((m + 2, 32), -1, dtype=torch.int16, device="cuda")
            torch.cuda.synchronize()
            assert pdc.capture_patches(ctx, b, out, m) == m
            assert pdc.capture_inputs(ctx, b, 1.0, words, m) == m
            assert torch.equal(out[:m], whole[:m]) and bool((out[m:] == -1).all())
            assert torch.equal(words[:m, :25], whole[:m].to(torch.bfloat16).view(torch.int16))
            assert bool((words[:m, 25:] == 0).all()) and bool((words[m:] == -1).all())
        pdc.release_batch(ctx, b)
    finally:
        pdc.destroy(ctx)
