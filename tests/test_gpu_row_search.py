"""The kernel that finds a row's pooled value by root search in registers (csrc/row_search.hpp): row
lengths at the edges of its shapes for few rows and for many, rows whose values are far from its first
guess, unaligned arrays, blocks from none to most of the row, ties at the block's ends and around zero,
every route.  Bar: that of test_gpu_parity (1e-5 + one float32 ulp)."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, P43, close, dev, gpu, host, run_case  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu

EDGES = [129, 255, 256, 509, 512, 513, 1021, 1024, 1533, 1537, 2045, 2046, 2047, 2048, 2049, 3069, 3072, 3073, 4093,
         4094, 4095, 4096,
         5117, 5120, 6141, 8189, 8192, 10237, 12285, 16381, 16384, 20477, 24573, 32765, 32766, 32768]


# (three rows: the shapes of up to 256 rows, 8 or 16 elements per thread up to 16384 elements)
@pytest.mark.parametrize("n", EDGES)
def test_lengths_at_the_edges_of_the_shapes(gpu, oracle, n):
    r = np.random.default_rng(n)
    x = r.normal(size=(3, n)).astype(np.float32)
    x[1] = np.round(x[1] * 4) / 4                                   # ties
    t = r.normal(size=x.shape).astype(np.float32)
    # (tiny lambda: rows without a block, or blocks of two; the oracle is quadratic in a p = 4/3 block)
    for k in (65, n // 2, n - 1):
        for p, lam in ((P2, 1e-5), (P2, 0.1), (P43, 1e-3)):
            run_case(gpu, oracle, "mask", x, t, k, p, lam, check_perm=False)
            run_case(gpu, oracle, "mag", x, t, k, p, lam, check_perm=False)
    run_case(gpu, oracle, "mask", x, t, n // 3, P2, 20.0, check_perm=False)     # a block longer than the list
    run_case(gpu, oracle, "mag", x, t, n // 3, P2, 20.0, check_perm=False)


# Every shape (threads per row x elements per thread) that more than 256 rows select, at the longest row that fits it
# with aligned and with unaligned rows; the row counts are just above a threshold and no multiple of four.
SHAPES = [(259, 512), (259, 1024), (259, 2045), (1541, 1536), (1541, 2048), (259, 3072), (259, 4096), (259, 5120),
          (259, 6144), (259, 8192), (1027, 8192), (259, 10240), (259, 12288), (259, 16384), (515, 16384), (259, 20480),
          (259, 24576), (259, 32768)]


@pytest.mark.parametrize("rows,n", SHAPES + [(rows, n - 3) for rows, n in SHAPES if n % 4 == 0])
def test_every_shape_at_its_longest_rows(gpu, oracle, rows, n):
    r = np.random.default_rng(rows + n)
    x = r.normal(size=(rows, n)).astype(np.float32)
    t = r.normal(size=x.shape).astype(np.float32)
    some = sorted({0, 1, 2, rows // 2, rows - 3, rows - 2, rows - 1})          # (all of the last workgroup)
    xd, td, k = dev(x), dev(t), n // 10
    for p, lam in ((P2, 0.02), (P43, 0.02)):
        for op in (gpu.topk_mask_jvp, gpu.topkmag_jvp):
            print(op.__name__, rows, n, k, p, lam, flush=True)
            ref = (oracle.topk_mask if op is gpu.topk_mask_jvp else oracle.topkmag)(x[some], k, p, lam, tangent=t[some])
            o, j = (host(a) for a in op(xd, td, k, p, lam))
            close(o[some], ref["out"], (op.__name__, p))
            close(j[some], ref["jvp"], (op.__name__, p, "jvp"))


@pytest.mark.parametrize("rows,n", [(259, 600), (259, 1021), (259, 1533), (1541, 1533), (1541, 1536), (1541, 2045), (259, 3069)])
def test_operators_built_on_the_mask_and_the_loss_many_rows(gpu, oracle, rows, n):
    r = np.random.default_rng(rows + n)
    x = r.normal(size=(rows, n)).astype(np.float32)
    t = r.normal(size=x.shape).astype(np.float32)
    some = sorted({0, 1, 2, rows // 2, rows - 3, rows - 2, rows - 1})
    xd, td, k = dev(x), dev(t), n // 5
    for p, lam in ((P2, 0.3), (P43, 0.05)):
        for name in ("topk_signed_mask", "topk_masked_value"):
            print(name, rows, n, k, p, lam, flush=True)
            ref = getattr(oracle, name)(x[some], k, p, lam, tangent=t[some])
            o, j = (host(a) for a in getattr(gpu, name + "_jvp")(xd, td, k, p, lam))
            close(o[some], ref["out"], name)
            close(j[some], ref["jvp"], name + " jvp")
        ref_loss, ref_grad = oracle.fenchel_young_loss(x[some], t[some], k, p, lam)
        loss, grad = (host(a) for a in gpu.topk_mask_loss(xd, td, k, p, lam))
        close(grad[some], ref_grad, "grad")
        close(loss[some], ref_loss, "loss")


@pytest.mark.parametrize("rows,n", [(300, 1000), (300, 2000), (300, 3000), (300, 4096), (600, 8190), (1100, 8192),
                                    (520, 12289), (270, 20001)])
def test_many_rows(gpu, oracle, rows, n):
    r = np.random.default_rng(rows + n)
    x = r.normal(size=(rows, n)).astype(np.float32)
    t = r.normal(size=x.shape).astype(np.float32)
    for p in (P2, P43):
        run_case(gpu, oracle, "mask", x, t, n // 10, p, 0.02, check_perm=False)
        run_case(gpu, oracle, "mag", x, t, n // 10, p, 0.02, check_perm=False)


@pytest.mark.parametrize("n", [700, 2500, 9001])
def test_operators_built_on_the_mask_and_the_loss(gpu, oracle, n):
    r = np.random.default_rng(n)
    x = r.normal(size=(5, n)).astype(np.float32)
    t = r.normal(size=x.shape).astype(np.float32)
    hot = np.zeros_like(x)
    hot[np.arange(5), r.integers(0, n, size=5)] = 1.0
    for p, lam in ((P2, 0.3), (P43, 0.01)):
        for k in (100, n // 3):
            for name in ("topk_signed_mask", "topk_masked_value"):
                ref = getattr(oracle, name)(x, k, p, lam, tangent=t)
                o, j = (host(a) for a in getattr(gpu, name + "_jvp")(dev(x), dev(t), k, p, lam))
                close(o, ref["out"], name)
                close(j, ref["jvp"], name + " jvp")
            ref_loss, ref_grad = oracle.fenchel_young_loss(x, hot, k, p, lam)
            loss, grad = (host(a) for a in gpu.topk_mask_loss(dev(x), dev(hot), k, p, lam))
            close(grad, ref_grad, "grad")
            # (float32 rounding of the stored value, and a small absolute term)
            assert (np.abs(loss - ref_loss) <= 2e-6 + 1.2e-7 * np.abs(ref_loss)).all()


@pytest.mark.parametrize("n", [1000, 4097, 9000])
def test_unaligned_arrays_and_special_values(gpu, oracle, n):
    import torch
    r = np.random.default_rng(n)
    x = r.normal(size=(4, n)).astype(np.float32)
    x[1] = x[1] * (r.random(n) < 0.05)                             # mostly zeros: s_{k+1} = 0
    x[2] = 2.5                                                     # constant
    x[3] = np.round(x[3] * 2) * np.float32(1e-38)                  # denormals
    t = r.normal(size=x.shape).astype(np.float32)
    run_case(gpu, oracle, "mask", x, t, n // 4, P2, 0.5, check_perm=False)
    run_case(gpu, oracle, "mag", x, t, n // 4, P2, 0.1, check_perm=False)
    run_case(gpu, oracle, "mag", x[:2], t[:2], n // 4, P43, 0.1, check_perm=False)
    ref = oracle.topk_mask(x, n // 4, P2, 0.5, tangent=t)
    for off in ((1, 1, 1, 1), (0, 1, 2, 3)):                       # offsets of the four arrays, in elements
        bufs = [torch.empty(4 * n + 8, device="cuda") for _ in range(4)]
        v = [b[o:o + 4 * n].view(4, n) for b, o in zip(bufs, off)]
        v[0].copy_(torch.from_numpy(x))
        v[1].copy_(torch.from_numpy(t))
        gpu.topk_mask_jvp(v[0], v[1], n // 4, P2, 0.5, out=v[2], jvp_out=v[3])
        close(host(v[2]), ref["out"], "unaligned fwd")
        close(host(v[3]), ref["jvp"], "unaligned jvp")


# Magnitude, p = 2, up to 2048 elements: a kept entry above the block is x / (1 + lambda) with one float32 rounding,
# whatever shape of the kernel the number of rows selects (1 / (1 + lambda) itself is rounded to float64: one
# output in 2^28 may round the other way, none of these do).
@pytest.mark.parametrize("n", [600, 1000, 1500, 1537, 2000, 2046])
def test_kept_entries_are_rounded_once(gpu, n):
    r = np.random.default_rng(n)
    x = r.normal(size=(300, n)).astype(np.float32)
    t = r.normal(size=x.shape).astype(np.float32)
    k, lam = 200, 1e-3
    inv = 1.0 / (1.0 + lam)
    many, d_many = (host(a) for a in gpu.topkmag_jvp(dev(x), dev(t), k, P2, lam))
    few, d_few = (host(a) for a in gpu.topkmag_jvp(dev(x[:4]), dev(t[:4]), k, P2, lam))
    # (clear of the block, which reaches up to s_{k+1} (1 + lambda))
    top = np.abs(x) > 1.01 * np.sort(np.abs(x), axis=1)[:, [n - k]]
    for y, d, rows in ((many, d_many, 300), (few, d_few, 4)):
        m = top[:rows]
        assert np.array_equal(y[m], (x[:rows][m].astype(np.float64) * inv).astype(np.float32))
        if n > 1024:                                                # (shorter ones: a float32 product)
            assert np.array_equal(d[m], (t[:rows][m].astype(np.float64) * inv).astype(np.float32))


# The header promises the same results on every route; rows of up to 2048 elements of these operators take no
# long-row route, whatever is set, and the ones that the root search takes are those with k = 0 or k > 48.
@pytest.mark.parametrize("n", [600, 1025, 1500, 2048])
def test_operators_built_on_the_mask_on_every_route(gpu, oracle, n):
    r = np.random.default_rng(n)
    x = r.normal(size=(3, n)).astype(np.float32)
    t = r.normal(size=x.shape).astype(np.float32)
    routes = [(gpu.TOPK_ROUTE_LONG_ROWS, v) for v in range(5)] + [(gpu.TOPK_ROUTE_SHORT_ROW_KERNEL, v) for v in range(3)]
    for k in (0, 48, 65, n // 3, n):
        for p, lam in ((P2, 0.3), (P43, 0.05)):
            refs = {name: getattr(oracle, name)(x, k, p, lam, tangent=t) for name in ("topk_signed_mask", "topk_masked_value")}
            ref_loss, ref_grad = oracle.fenchel_young_loss(x, t, k, p, lam)
            for which, value in routes:
                gpu.set_route(which, value)
                try:
                    for name, ref in refs.items():
                        o, j = (host(a) for a in getattr(gpu, name + "_jvp")(dev(x), dev(t), k, p, lam))
                        close(o, ref["out"], (name, k, which, value))
                        close(j, ref["jvp"], (name + " jvp", k, which, value))
                        close(host(getattr(gpu, name + "_fwd")(dev(x), k, p, lam)), ref["out"], (name, k, which, value))
                    loss, grad = (host(a) for a in gpu.topk_mask_loss(dev(x), dev(t), k, p, lam))
                    close(grad, ref_grad, ("grad", k, which, value))
                    close(loss, ref_loss, ("loss", k, which, value))
                finally:
                    gpu.set_route(which, 0)


def hard_rows(r, n):
    """Rows whose values are far from what a guess from a few order statistics says, and a lambda for each."""
    x = r.normal(size=n)
    return {"masked": (np.where(r.random(n) < 0.5, -1e9, x), 0.1),
            "masked, lowest float": (np.where(r.random(n) < 0.85, -3.4028235e38, x), 0.1),
            "heavy tails": (x * np.exp(4 * r.normal(size=n)), 0.1),
            "one far value": (np.r_[x[:-1], 1e9], 0.1),
            "whole numbers": (np.round(2 * x), 1e-3),
            "two values": ((r.random(n) < 0.5) * 1.0, 0.05),
            "probabilities": (np.exp(3 * x) / np.exp(3 * x).sum(), 1e-6),
            "few non-zeros": (x * (r.random(n) < 0.05), 0.1),
            "sorted": (np.sort(x), 0.1),
            "far from zero": (300 * x + 5000, 0.1),
            "much smaller than lambda": (1e-30 * x, 0.1)}


# Few and many rows; 4094: fewer elements than four per thread.
@pytest.mark.parametrize("rows,n", [(3, 1500), (300, 3000), (3, 4094), (3, 20000)])
def test_values_far_from_the_guess(gpu, oracle, rows, n):
    r = np.random.default_rng(rows * n)
    t = r.normal(size=(rows, n)).astype(np.float32)
    for name, (v, lam) in hard_rows(r, n).items():
        print(name, flush=True)
        x = np.stack([r.permutation(v) if name != "sorted" else v for _ in range(rows)]).astype(np.float32)
        for k in (65, n // 10, n // 2):
            # (a block of lowest floats: lambda is lost beside them in the oracle's float64 sums)
            if "lowest" in name and k > n // 10:
                continue
            run_case(gpu, oracle, "mask", x, t, k, P2, lam, check_perm=False)
            if "lowest" in name:
                continue
            run_case(gpu, oracle, "mag", x, t, k, P2, lam, check_perm=False)
            if rows == 3 and n < 5000 and lam < 0.01:
                run_case(gpu, oracle, "mask", x, t, k, P43, lam, check_perm=False)


# The search takes some dozens of passes over a row at most, whatever the values: 2 ms for a few rows is more
# than ten times what any of these takes (growing the block of a row of 32768 elements one value at a time: 275 ms).
def test_time_does_not_depend_on_the_values(gpu):
    import torch
    n = 32768
    r = np.random.default_rng(3)
    t = torch.zeros((8, n), device="cuda")
    for name, (v, lam) in hard_rows(r, n).items():
        x = dev(np.broadcast_to(v.astype(np.float32), (8, n)).copy())
        for p in (P2, P43):
            for k in (65, n // 10, n // 2):
                for f in (gpu.topk_mask_jvp, gpu.topkmag_jvp):
                    f(x, t, k, p, lam)
                    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    a.record()
                    f(x, t, k, p, lam)
                    b.record()
                    b.synchronize()
                    assert a.elapsed_time(b) < 2.0, (name, p, k, f.__name__, a.elapsed_time(b))


# gamma = 0 exactly: elements at 0 and at lambda tie with the block and stay outside, their outputs follow their own
# tangents (0 and, above, 0).  Block: m copies of 0.5 (top-k positions), 2 m of 0.25: 0.5 m + 0.25 (2 m) = lambda m.
# The sums of the search are taken relative to its first guess: gamma comes out some 1e-17 off zero, where floats
# are dense.  60000: candidate lists of long rows (csrc/wide_rows.hip) of 6050 and 24050 members and more.
@pytest.mark.parametrize("rows,n,m", [(3, 1500, 100), (300, 1500, 100), (300, 3000, 40), (3, 20000, 3000), (2, 60000, 2000),
                                      (2, 60000, 8000)])
def test_ties_around_zero(gpu, oracle, rows, n, m):
    above, at_lambda, zeros = n // 20, 30, n // 8
    v = np.full(n, -2.0, dtype=np.float32)
    for value, count in ((0.0, zeros), (0.25, 2 * m), (0.5, m), (1.0, at_lambda), (5.0, above)):
        v = np.r_[np.full(count, value, dtype=np.float32), v]
    v = v[:n]
    for seed in range(4):
        r = np.random.default_rng(rows + n + seed)
        x = np.stack([r.permutation(v) for _ in range(rows)])
        t = r.normal(size=x.shape).astype(np.float32)
        run_case(gpu, oracle, "mask", x, t, above + at_lambda + m, P2, 1.0, check_perm=False)
