"""Hit records in host memory: page-locked destinations around the number of
records from which the copy engine fills them, ordinary ones, destinations
shorter than the list, and more records than its device staging holds, against
the records of a device destination."""
import ctypes

import numpy as np
import pytest

from paper_1903_06838_amd import synth

pytestmark = pytest.mark.gpu

COPY, CHUNK = 1 << 15, 1 << 24  # records


def _batch(n):
    """A hit on every ninth pixel of n CSPAD-like frames; context, batch, number
    of hits and the records of a device destination."""
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    geom = synth.CSPAD
    ctx = pdc.create(0)
    ped, gain = np.full(geom.shape, 1000.0, np.float32), np.ones(geom.shape, np.float32)
    raw = torch.full((n, *geom.shape), 1000, dtype=torch.int16, device="cuda")
    raw[:, :, ::3, ::3] = (1200 + torch.arange(n, device="cuda")).to(torch.int16).view(n, 1, 1, 1)
    det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, geom.bank_cols), ped, gain, pdc.params())
    torch.cuda.synchronize()
    b = pdc.process_frames(ctx, det, raw, n, raw.numel() // 8)
    total = n * 32 * 62 * 130
    dev = torch.empty((total, 4), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    _, got, _, _, st = pdc.get_hits(ctx, b, n, capacity=total, dst_dev=dev)
    assert got == total and st == pdc.OK
    return ctx, b, total, dev


def _host(ctx, b, dst, capacity):
    from paper_1903_06838_amd import pdc

    total = ctypes.c_uint64(0)
    st = pdc._lib.pdc_get_hits(ctx, b, dst.data_ptr(), capacity, 0, ctypes.byref(total), None, None)
    assert st == (pdc.WARN_TRUNCATED if capacity < total.value else pdc.OK)


def test_sizes():
    import torch

    from paper_1903_06838_amd import pdc

    ctx, b, total, dev = _batch(2)
    try:
        want = dev.cpu()
        for pinned in (True, False):
            for n in (1, 4096, 4097, COPY - 1, COPY, COPY + 1, 100001, total - 1, total):
                dst = torch.full((n + 8, 4), -1, dtype=torch.int32, pin_memory=pinned)
                _host(ctx, b, dst[4:], n)
                assert torch.equal(dst[4:n + 4], want[:n]) and bool((dst[:4] == -1).all()) and bool((dst[n + 4:] == -1).all())
    finally:
        pdc.destroy(ctx)


def test_more_than_the_staging():
    import torch

    from paper_1903_06838_amd import pdc

    ctx, b, total, dev = _batch(66)
    try:
        assert total > CHUNK
        dst = torch.full((total, 4), -1, dtype=torch.int32, pin_memory=True)
        _host(ctx, b, dst, total)
        assert torch.equal(dst.cuda(), dev)
    finally:
        pdc.destroy(ctx)


def test_long_lists():
    """Records of frames that are empty, hold one hit or many, in lists around
    the length from which a wave takes two rows of hits."""
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    n, rows = 30000, 1 << 19
    geom = synth.Geometry(1, 16, 64, 32)
    kind = np.random.default_rng(6).integers(0, 3, n)
    raw = np.full((n, *geom.shape), 1000, np.uint16)
    raw[kind == 1, 0, 8, 31] = 1160
    raw[kind == 2, :, 1::3, 1::5] = 1160
    ctx = pdc.create(0)
    try:
        ped, gain = np.full(geom.shape, 1000.0, np.float32), np.ones(geom.shape, np.float32)
        det = pdc.calibrate(ctx, pdc.geometry(*geom.shape, 32), ped, gain, pdc.params())
        b = pdc.process_frames(ctx, det, torch.from_numpy(raw.view(np.int16)).cuda(), n, raw.size // 8)
        total = pdc.get_hits(ctx, b, n, capacity=0)[1]
        frame = torch.from_numpy(np.repeat(np.arange(n), np.array([0, 1, 65])[kind]).astype(np.int32)).cuda()
        one, many = [8 * 64 + 31], [64 * r + c for r in range(1, 16, 3) for c in range(1, 64, 5)]
        pixel = torch.tensor(np.concatenate([([], one, many)[k] for k in kind]).astype(np.int32)).cuda()
        assert total == len(frame) == len(pixel) > rows + 200
        for cap in (rows - 1, rows, rows + 1, rows + 63, rows + 64, rows + 65, rows + 127, rows + 128, rows + 129, total):
            rec = torch.full((cap + 2, 4), -1, dtype=torch.int32, device="cuda")
            torch.cuda.synchronize()
            pdc.get_hits(ctx, b, n, capacity=cap, dst_dev=rec)
            assert torch.equal(rec[:cap, 0], frame[:cap]) and torch.equal(rec[:cap, 1], pixel[:cap])
            assert bool((rec[:cap, 3] == 1).all()) and bool((rec[cap:] == -1).all())
    finally:
        pdc.destroy(ctx)
