"""Seed and neighbour thresholds of zero, with either sign, bit for bit against the
oracle: pixels of exactly 0 are not above them."""
import numpy as np
import pytest

from paper_1903_06838_amd import synth
from tests.helpers import assert_same, oracle_threads, run_pdc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zero", [0.0, -0.0], ids=["plus", "minus"])
@pytest.mark.parametrize("B,nb", [(96, 2), (97, 2), (194, 2), (300, 1), (514, 1)])
def test_zero_threshold(B, nb, zero):
    import torch

    from paper_1903_06838_amd import pdc

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    # few rows, so that the half of the pixels at or above the median fits the lists
    geom = synth.Geometry(1, 4, B * nb, B)
    ped, gain = np.full(geom.shape, 1000.0, np.float32), np.ones(geom.shape, np.float32)
    raw = np.random.default_rng(B).choice(np.array([998, 999, 1000, 1001], np.uint16), (40, *geom.shape),
                                          p=[0.2, 0.25, 0.25, 0.3])
    want = oracle_threads(raw, ped, gain, B, sigma=3.0, n_seed=zero, n_nb=zero)
    ctx = pdc.create(0)
    try:
        got = run_pdc(ctx, raw, ped, gain, B, n_seed=zero, n_nb=zero, hit_capacity=raw.size)
    finally:
        pdc.destroy(ctx)
    assert want["total"] > 0
    assert_same(got, want)
