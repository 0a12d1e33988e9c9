"""The FP64 normals against their definition evaluated in extended precision
from the device's Philox words: every value within four units of relative
rounding, 4 x 2^-53 (radius and angle function each below one, their product
and the Philox-exact arguments nothing else).  Needs an MI355X."""
import numpy as np
import pytest

from paper_2602_16486_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu_present():
    assert _lib.device_count() > 0, "no HIP device visible: the gpu tests need an MI355X"


@pytest.mark.parametrize("q", [9, 19, 27])
def test_normals_fp64_to_rounding(q):
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("long double is no wider than double")
    n, seed, step = 200_000, (5 << 32) + 77, 12345
    first = 3 if q == 9 else 4
    got = _lib.noise_sample(q, seed, 0, step, 0, n, fp64=True)[:, first:]
    pi = np.longdouble("3.14159265358979323846264338327950288")
    for blk in range((q - first + 3) // 4):
        ctr = np.zeros((n, 4), dtype=np.uint32)
        ctr[:, 0], ctr[:, 1], ctr[:, 3] = np.arange(n), step, blk
        w = _lib.philox_words(ctr, seed & 0xFFFFFFFF, seed >> 32)
        for pair in range(2):
            a, b = w[:, 2 * pair], w[:, 2 * pair + 1]
            r = np.sqrt(-2 * np.log(((a >> 8).astype(np.longdouble) + 1) / 2 ** 24))
            # the angle reduced to [-pi/4, pi/4] around its quarter turn, so
            # that long double keeps its relative accuracy near the axes
            t = (b >> 8).astype(np.int64)
            quarter = (t + (1 << 21)) >> 22
            x = (t - (quarter << 22)).astype(np.longdouble) * (2 * pi / 2 ** 24)
            s, c = np.sin(x), np.cos(x)
            cos = np.choose(quarter % 4, [c, -s, -c, s])
            sin = np.choose(quarter % 4, [s, c, -s, -c])
            for k, ref in enumerate((r * cos, r * sin)):
                col = 4 * blk + 2 * pair + k
                if col < got.shape[1]:
                    assert np.all(np.abs(got[:, col] - ref) <= 4 * 2.0 ** -53 * np.abs(ref)), col
