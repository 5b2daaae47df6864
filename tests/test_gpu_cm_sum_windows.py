"""Exact thresholded sums where their way changes: one pixel's dark of 2^e (raw
0 there is a tiny noise value) moves the lowest bit of the sums through the
widths at which values are added in groups, one by one in two binary64 limbs,
and the general way; tile sizes around the lanes and steps of one workgroup,
with full, single and ragged frame groups.  Bit for bit against the oracle,
whose sum is exact and rounded once."""
import pytest

from oracle import cm_mean as M
from paper_1903_06838_amd import synth
from tests.helpers import assert_same
from tests.test_gpu_cm_mean import _run, ctx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

EXPONENTS = [6, 0, -8, -12, -16, -24, -32, -36, -44]
GEOMS = [
    (synth.Geometry(2, 20, 388, 194), 9),
    (synth.Geometry(1, 24, 768, 96), 3),
    (synth.Geometry(1, 20, 512, 256), 2),
    (synth.Geometry(1, 20, 128, 64), 8),
]
TILES = [(1, 4), (1, 252), (1, 256), (2, 130), (1, 1020), (1, 1024), (2, 514), (2, 1024), (3, 684), (5, 820), (4, 3)]


def _check(ctx, geom, n, region, e, seed):
    ped, gain = synth.make_calibration(geom, seed)
    ped[0, 0, geom.cols // 2] = 2.0**e
    raw = synth.make_frames(geom, ped, gain, n, 0.03, seed, sim=synth.SimParams(cm_sigma=1.0))
    raw[n // 2, 0, 0, geom.cols // 2] = 0
    want = M.process(raw, ped, gain, geom.bank_cols, region, 3, keep_corrected=True)
    assert_same(_run(ctx, raw, ped, gain, geom.bank_cols, region, 3), want, corrected=True)


@pytest.mark.parametrize("e", EXPONENTS)
@pytest.mark.parametrize("geom,n", GEOMS, ids=lambda x: str(x))
def test_sum_window(ctx, geom, n, e):  # noqa: F811
    for region in (M.BANK, M.TILE):
        _check(ctx, geom, n, region, e, 31)


@pytest.mark.parametrize("hw", TILES, ids=lambda x: f"{x[0]}x{x[1]}")
def test_tile_sizes(ctx, hw):  # noqa: F811
    for n in (1, 8, 11):
        _check(ctx, synth.Geometry(3, hw[0], hw[1], hw[1]), n, M.TILE, 6, 32)
