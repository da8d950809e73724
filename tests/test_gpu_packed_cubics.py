"""Top-k in magnitude, p = 4/3: the outputs above the block, whose cubics a wavefront solves packed when at most half of
its elements are above (csrc/cubic.hpp): shares around that half, none and all.  Oracle; bar: that of test_gpu_parity."""
import numpy as np
import pytest

from tests.test_gpu_parity import P43, gpu, run_case  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n", [(5, 200), (3, 400), (300, 1500), (2, 4096), (2, 4099), (3, 30001), (2, 40001), (1, 65536)])
def test_shares_above(gpu, oracle, rows, n):
    r = np.random.default_rng(n)
    x = (r.laplace(size=(rows, n)) * 0.02).astype(np.float32)
    x[0, :5] = 0.0
    # the first elements of a row all above, so that some wavefronts hold nothing else
    x[-1, : n // 4] = np.float32(0.5) + np.abs(x[-1, : n // 4])
    t = r.normal(size=x.shape).astype(np.float32)
    for share in (0.02, 0.3, 0.48, 0.5, 0.52, 0.9):
        run_case(gpu, oracle, "mag", x, t, max(1, int(share * n)), P43, 1e-3, check_perm=False)
    run_case(gpu, oracle, "mag", x, t, n, P43, 1e-3, check_perm=False)
