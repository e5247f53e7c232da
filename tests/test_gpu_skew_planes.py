"""Skewed rows of spread counters where the planes divide by 4, with rows of tiles that hold no
divisor of 256 bins, and next to them numbers of planes without a skew."""

import pytest

from test_gpu_spread_counters import test_spread_counters as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stable", [False, True])
@pytest.mark.parametrize("n,n_w,images", [
    (250, 36, 2), (1040, 12, 1), (1040, 14, 1), (572, 4, 1), (1100, 4, 1), (208, 28, 1),
])
def test_skew_planes(n, n_w, images, stable):
    check(n, n_w, images, stable)
