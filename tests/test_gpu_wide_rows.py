"""Long rows, dense outputs (csrc/wide_rows.hip): row lengths at the edges of the parts that workgroups take, counts added
up directly and in groups, 16-bit and 32-bit counts, lists of every kind (empty middle, one wavefront, one workgroup, longer
than LDS), ties and infinities.  Against the oracle with the bar of test_gpu_parity where it is quick, else bit for
bit against the routes that sort."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, P43, dev, gpu, host, long_rows_route, run_case  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


def _same_as_sorted(gpu, op, x, t, k, p, lam, mode="select"):
    print(f"case op={op} shape={tuple(x.shape)} k={k} p={p:.4f} lam={lam}", flush=True)
    fn = gpu.topk_mask_jvp if op == "mask" else gpu.topkmag_jvp
    o, j = (host(a) for a in fn(x, t, k, p, lam))
    with long_rows_route(gpu, mode):
        o2, j2 = (host(a) for a in fn(x, t, k, p, lam))
    assert np.array_equal(o, o2)
    err = np.abs(j.astype(np.float64) - j2)
    assert (err <= 2.4e-7 * np.abs(j2) + 1e-9).all(), float(err.max())      # (two roundings of d gamma's sum)
    with long_rows_route(gpu, "wide"):
        o3, j3 = (host(a) for a in fn(x, t, k, p, lam))
    assert np.array_equal(o, o3) and np.array_equal(j, j3)                   # and again: the same bits


# parts of 16384 elements; 33 parts (524289 elements) and more are counted in groups
@pytest.mark.parametrize("rows,n", [(1, 32769), (3, 49151), (2, 49153), (1, 524289), (1, 600001)])
def test_row_lengths(gpu, oracle, rows, n):
    r = np.random.default_rng(n)
    x = r.normal(size=(rows, n)).astype(np.float32)
    t = r.normal(size=x.shape).astype(np.float32)
    for k, lam in ((1, 0.01), (n // 10, 0.1), (n - 1, 0.01), (n // 2, 1e-6)):
        run_case(gpu, oracle, "mask", x, t, k, P2, lam, check_perm=False)
        run_case(gpu, oracle, "mag", x, t, k, P2, lam, check_perm=False)
    run_case(gpu, oracle, "mask", x, t, n // 10, P43, 0.003, check_perm=False)
    run_case(gpu, oracle, "mag", x, t, n // 10, P43, 0.003, check_perm=False)


# 34 x 500000: parts of more than 65536 elements, counts of 32 bits.  64 x 262144: parts of 65536 elements, of which
# one holds nothing but one value (a 16-bit count runs over)
@pytest.mark.parametrize("rows,n", [(34, 500000), (64, 262144)])
def test_counts(gpu, rows, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((rows, n), generator=g, device="cuda")
    t = torch.randn((rows, n), generator=g, device="cuda")
    x[1, 65536:131072] = 1.25
    x[2, :65536] = 1.75
    for op, p, lam in (("mask", P2, 0.1), ("mag", P2, 0.05), ("mask", P43, 0.02)):
        _same_as_sorted(gpu, op, x, t, n // 10, p, lam)


# Counts that are added up in groups: 2^24 elements in 256 parts of 65536, eight of which hold nothing but one value of
# the window, in eight neighbouring bins (a 16-bit count runs over, in either half of the words that two share); and more
# elements than that, whose counts take 32 bits.
@pytest.mark.parametrize("n", [1 << 24, (1 << 24) + 4097])
def test_counts_in_groups(gpu, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((1, n), generator=g, device="cuda")
    t = torch.randn((1, n), generator=g, device="cuda")
    for i, part in enumerate((1, 2, 17, 100, 101, 130, 240, 255)):
        x[0, part * 65536:(part + 1) * 65536] = 1.25 + 0.00025 * i          # (the mask's s_k is 1.263)
    for op, k, lam in (("mask", n // 10, 0.1), ("mag", n // 5, 0.05)):
        _same_as_sorted(gpu, op, x, t, k, P2, lam)


# a block that is most of the row; lists of equal values that fit a wavefront, a workgroup, or nothing
@pytest.mark.parametrize("copies", [500, 2049, 6200, 40000])
def test_lists_of_equal_values(gpu, oracle, copies):
    n = 100000
    r = np.random.default_rng(copies)
    x = r.normal(size=(2, n)).astype(np.float32)
    x[:, :copies] = np.float32(1.25)
    x[1] = r.permutation(x[1])
    t = r.normal(size=x.shape).astype(np.float32)
    above = int((x[0] > 1.25).sum())
    for k in (above + 1, above + copies // 2, above + copies):
        for lam in (1e-7, 1e-3, 0.5):
            run_case(gpu, oracle, "mask", x, t, k, P2, lam, check_perm=False)
            run_case(gpu, oracle, "mag", x, t, k, P2, lam, check_perm=False)
        if copies < 7000:                    # (the oracle's p = 4/3 pooling is quadratic in the block)
            run_case(gpu, oracle, "mask", x, t, k, P43, 1e-3, check_perm=False)
            for lam in (1e-7, 1e-3, 0.5):
                run_case(gpu, oracle, "mag", x, t, k, P43, lam, check_perm=False)


def test_wide_blocks_infinities_and_signs_of_zero(gpu, oracle):
    n = 70000
    r = np.random.default_rng(3)
    x = r.normal(size=(4, n)).astype(np.float32)
    x[1] = np.abs(x[1]) * (r.random(n) < 0.02)                # s_k an exact zero
    x[1, ::7] *= -1.0
    x[2, : n // 2] = -np.inf                                  # masked out
    x[3, :3] = np.inf
    t = r.normal(size=x.shape).astype(np.float32)
    for k, lam in ((10, 1.0), (n // 10, 1e-3), (n // 3, 1.0), (n // 10, 30.0)):
        run_case(gpu, oracle, "mask", x, t, k, P2, lam, check_perm=False)
        run_case(gpu, oracle, "mag", x[:2], t[:2], k, P2, lam, check_perm=False)
    run_case(gpu, oracle, "mask", x[:1], t[:1], n // 10, P43, 1e-3, check_perm=False)
    run_case(gpu, oracle, "mag", x[:2], t[:2], n // 10, P43, 1e-3, check_perm=False)
    # (a block of 60000 zeros: the oracle would take 20 s)
    _same_as_sorted(gpu, "mask", dev(x[1:2]), dev(t[1:2]), n // 10, P43, 1e-3)


# Scores masked out by a large negative number, with more top-k positions than scores that are left: the block is the
# masked elements, exact ties, and lambda is lost beside their value, or beside the width of the window that holds it.
# Of `tied` equal elements that share m positions each gets m / tied, whatever p (float64: one rounding); in
# magnitude v / (1 + lambda m / tied) m / tied (p = 2), resp. w^3 with w^3 = (v - lambda w) m / tied (p = 4/3).
@pytest.mark.parametrize("value", [-1e4, -1e9, -1e30, float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("lam", [1e-6, 1e-2, 1.0, 100.0])
def test_masked_out_scores_share_what_is_left(gpu, value, lam):
    n, left, k = 33000, 3000, 9000
    r = np.random.default_rng(11)
    x = np.full((2, n), value, dtype=np.float32)
    x[0, r.permutation(n)[:left]] = r.normal(size=left)
    x[1] = value                                             # a row of nothing else
    t = r.normal(size=x.shape).astype(np.float32)
    masked = x == np.float32(value)
    for p in (P2, P43):
        print(f"case value={value} lam={lam} p={p:.4f}", flush=True)
        o, j = (host(a).astype(np.float64) for a in gpu.topk_mask_jvp(dev(x), dev(t), k, p, lam))
        for row in range(2):
            here, tied = masked[row], int(masked[row].sum())
            y = (k - (n - tied)) / tied
            assert np.array_equal(o[row, ~here], np.ones(n - tied))
            assert np.abs(o[row, here] - y).max() <= 1.2e-7 * y
            slope = (1.0 if p == P2 else 3.0 * y ** (2.0 / 3.0)) / lam
            want = slope * (t[row].astype(np.float64) - t[row, here].astype(np.float64).mean())
            assert np.abs(j[row, here] - want[here]).max() <= 2.4e-7 * np.abs(want[here]).max()
            assert not j[row, ~here].any()
        mag = np.abs(x)
        mag[0, ~masked[0]] = 0.0                             # the tied elements are the largest
        o, _ = gpu.topkmag_jvp(dev(mag), dev(t), k, p, lam)
        o = host(o).astype(np.float64)
        for row in range(2):
            tied, v = int(masked[row].sum()), float(mag[row].max())
            share = k / tied
            if p == P2:
                want = share * v / (1.0 + lam * share)
            else:                                            # g = v - lambda w with w^3 = share g
                w = np.cbrt(np.longdouble(share) * v)        # (from above: Newton falls to the root)
                for _ in range(100):
                    w -= (w ** 3 - share * (v - lam * w)) / (3 * w ** 2 + lam * share)
                want = float(w ** 3)
            assert np.abs(o[row, masked[row]] - want).max() <= 2.4e-7 * want, (o[row, masked[row]][:3], want)
            assert not o[row, ~masked[row]].any()


# the largest float32 values above the block, whose cubes and products with lambda are in no float32 (csrc/cubic.hpp)
@pytest.mark.parametrize("lam", [1e-3, 1.0, 1e12, 1e25])
def test_largest_values_above_the_block(gpu, lam):
    n, k = 33000, 3000
    r = np.random.default_rng(12)
    x = np.zeros((2, n), dtype=np.float32)
    x[:, :k] = (2.0 + 1.4 * r.random((2, k))) * 1e38
    x[1, k:] = r.random(n - k) * 1e-3 + 1e-3
    t = np.ones_like(x)
    o, j = (host(a).astype(np.float64) for a in gpu.topkmag_jvp(dev(x), dev(t), k, P43, lam))
    s = x[:, :k].astype(np.longdouble)
    w = np.minimum(s / lam, np.cbrt(s))                      # w^3 + lambda w = s
    for _ in range(60):
        w -= (w ** 3 + lam * w - s) / (3 * w ** 2 + lam)
    assert np.array_equal(o[:, :k], (w ** 3).astype(np.float32).astype(np.float64))
    slope = (3 * w ** 2 / (3 * w ** 2 + lam)).astype(np.float64)
    assert np.abs(j[:, :k] - slope).max() <= 1.2e-7
    assert not o[:, k:].any()


# Outputs above the block are float64 solutions, rounded once (csrc/cubic.hpp): elements whose solution lies within 4e-13
# of the middle between two floats, where a solve to 5e-13 rounds some to the wrong one and one in float64 none.  They
# are near s = lambda^(3/2), where the float32 start of the solve is worst.
@pytest.mark.parametrize("lam", [0.011, 0.07, 0.3, 1.7, 4.5, 11.0, 29.0, 73.0])
def test_cubics_above_the_block_to_rounding(gpu, lam):
    n = 40000
    s = np.unique((lam ** 1.5 * np.linspace(0.97, 1.04, 1 << 21)).astype(np.float32))

    def solve(v, of):
        v = v.astype(of)
        w = np.minimum(v / lam, np.cbrt(v))                  # w^3 + lambda w = s
        for _ in range(8):
            w -= (w * (w * w + lam) - v) / (3 * w * w + lam)
        return w ** 3

    def from_middle(g):
        f = g.astype(np.float32)
        step = np.where(g > f, np.nextafter(f, np.float32(np.inf)), np.nextafter(f, np.float32(0.0)))
        return np.abs(g - (f.astype(g.dtype) + step.astype(g.dtype)) / 2) / g

    s = s[from_middle(solve(s, np.float64)) < 4e-13]
    g = solve(s, np.longdouble)
    keep = from_middle(g) > 2e-15
    s, g = s[keep], g[keep]
    assert 1 <= len(s) <= n // 2
    x = np.zeros((1, n), dtype=np.float32)
    x[0, ::n // len(s)][:len(s)] = s
    o = host(gpu.topkmag_fwd(dev(x), len(s), P43, lam))
    assert np.array_equal(o[0, ::n // len(s)][:len(s)], g.astype(np.float32))
