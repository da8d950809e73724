"""Long rows whose candidates are solved without sorting them (csrc/wide_rows.hip).  The exact solve sees the list of those
elements that a threshold may fall next to: up to 2048 one wavefront solves, up to 6144 a workgroup with the list in LDS,
longer ones a workgroup with the list in memory.  Lists of distinct values at these edges, windows of some thousand
candidates (few of which are on the list), ties at the block's ends and around zero.  Oracle; bar: that of test_gpu_parity."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, P43, dev, gpu, host, long_rows_route, run_case  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


# A cluster far narrower than a bin, all of which is on the list; the rest of the row is out of reach.  k = 1 and
# lambda = 1: everything is in the block.  lambda a fraction of the cluster's width: both thresholds are inside.
@pytest.mark.parametrize("length", [2047, 2048, 2049, 6143, 6144, 6145, 39000])
def test_lists_of_distinct_values(gpu, oracle, length):
    n = 40000
    r = np.random.default_rng(length)
    for width, k, lam in ((1e-3, 1, 1.0), (1e-4, length // 2, 4e-5), (1e-4, length // 3, 1e-5)):
        x = np.full((2, n), -100.0, dtype=np.float32)
        for row in x:
            row[r.permutation(n)[:length]] = 1.01 + width * r.random(length)
        t = r.normal(size=x.shape).astype(np.float32)
        run_case(gpu, oracle, "mask", x, t, k, P2, lam, check_perm=False)
        x[x < 0] = 0.0
        run_case(gpu, oracle, "mag", x, t, k, P2, lam, check_perm=False)
        for op in ("mask", "mag"):
            if length < 7000:                                # (the oracle's p = 4/3 pooling is quadratic in the block)
                run_case(gpu, oracle, op, x, t, k, P43, lam, check_perm=False)
            else:
                fn = gpu.topk_mask_jvp if op == "mask" else gpu.topkmag_jvp
                o, j = (host(a) for a in fn(dev(x), dev(t), k, P43, lam))
                with long_rows_route(gpu, "select"):
                    o2, j2 = (host(a) for a in fn(dev(x), dev(t), k, P43, lam))
                assert np.abs(o - o2).max() <= 2.4e-7 * np.abs(o2).max()
                assert np.abs(j - j2).max() <= 2.4e-7 * np.abs(j2).max()


# windows of about `width` candidates, of which the list holds the few next to the block's ends
@pytest.mark.parametrize("n", [40000, 262144, 300001])
@pytest.mark.parametrize("width", [4000, 4200, 16000, 17000, 32700, 33500])
def test_list_lengths(gpu, oracle, n, width):
    r = np.random.default_rng(n + width)
    k = n // 10
    # uniform values: a window of 2 lambda around s_k holds about `width` elements
    x = r.random(size=(2, n)).astype(np.float32) + 1.0
    t = r.normal(size=x.shape).astype(np.float32)
    lam = min(0.5 * width / n, 0.09)
    run_case(gpu, oracle, "mask", x, t, k, P2, lam, check_perm=False)
    run_case(gpu, oracle, "mag", x - 2.0, t, k, P2, lam, check_perm=False)


def test_ties_at_the_ends_and_around_zero(gpu, oracle):
    n = 60000
    r = np.random.default_rng(9)
    x = np.round(r.normal(size=(3, n)) * 64).astype(np.float32) / 64          # binary fractions: exact sums
    x[1] = np.where(x[1] == 0, np.float32(-0.0), x[1])
    t = r.normal(size=x.shape).astype(np.float32)
    for k in (n // 2, n // 2 + 700, n // 2 - 11000, n // 5):
        for lam in (0.125, 0.5, 1.0):
            run_case(gpu, oracle, "mask", x, t, k, P2, lam, check_perm=False)
            run_case(gpu, oracle, "mag", x, t, k, P2, lam, check_perm=False)


# An element x above the block whose singleton minimiser x / (1 + lambda) equals the pooled value exactly does
# not violate: it stays outside, and its output follows its own tangent alone.  lambda = 0.75, gamma = 4 x / 7 is
# no float64 number, and for these x the rounded gamma times the rounded 1 + lambda is above x.  Block of 8 q
# elements: q copies of a < x (top-k positions), 7 q of b > gamma, q a + 7 q b = gamma (8 q + 0.75 q).
@pytest.mark.parametrize("x,a,b", [(29, 26, 17), (58, 52, 34), (123, 118, 71), (253, 250, 145)])
@pytest.mark.parametrize("q", [600, 2400, 5000])
def test_exact_ties_at_the_upper_end(gpu, oracle, x, a, b, q):
    n, copies, above = 60000, 50, 3000
    r = np.random.default_rng(x + q)
    v = np.full(n, 1.0, dtype=np.float32)
    v[:above] = 8 * x
    v[above:above + copies] = x
    v[above + copies:above + copies + q] = a
    v[above + copies + q:above + copies + 8 * q] = b
    rows = np.stack([r.permutation(v) * r.choice([-1.0, 1.0], size=n) for _ in range(2)]).astype(np.float32) / 64
    t = r.normal(size=rows.shape).astype(np.float32)
    run_case(gpu, oracle, "mag", rows, t, above + copies + q, P2, 0.75, check_perm=False)


# gamma = 0 exactly: elements at 0 and at lambda tie with the block and stay outside.  Block of 3 m elements: m copies
# of 0.5 (top-k positions), 2 m of 0.25, 0.5 m + 0.25 (2 m) = lambda m; lambda = 1, and, scaled by an odd number, the
# same with a gamma that is zero up to rounding.
@pytest.mark.parametrize("m", [2000, 8000])
@pytest.mark.parametrize("scale", [1.0, 3.0])
def test_exact_ties_around_zero(gpu, oracle, m, scale):
    n, above, at_lambda, zeros = 60000, 3000, 30, 7000
    v = np.full(n, -2.0, dtype=np.float32)
    for value, count in ((0.0, zeros), (0.25, 2 * m), (0.5, m), (1.0, at_lambda), (5.0, above)):
        v = np.r_[np.full(count, value, dtype=np.float32), v]
    r = np.random.default_rng(m)
    x = np.stack([r.permutation(v[:n]) for _ in range(2)]) * np.float32(scale)
    t = r.normal(size=x.shape).astype(np.float32)
    run_case(gpu, oracle, "mask", x, t, above + at_lambda + m, P2, scale, check_perm=False)
