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
