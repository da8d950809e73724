"""General weights, identity form, p = 2, forward: the kernel that does not sort the row
(csrc/general_search.hip) against the oracle, and against the kernel that sorts it where that one takes
over.  Bar: that of test_gpu_parity (1e-5 + one float32 ulp)."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, close, dev, gpu, host  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


def weight_rows(n):
    i = np.arange(n)
    return {"ranks": (n - i), "ones_k": (i < n // 7), "steps": np.floor((n - i) / 97.0), "constant": np.full(n, 2.5),
            "inverse": 1.0 / (1.0 + i), "negative": -0.01 * i}


# edges of the tiles of weights (2048), of the loops over the row, odd lengths
@pytest.mark.parametrize("n", [1025, 2047, 2048, 2049, 4095, 5001, 8192, 16388, 40000, 65536, 131071, 131072])
def test_lengths_weights_and_lambdas(gpu, oracle, n):
    r = np.random.default_rng(n)
    x = r.normal(size=(3, n)).astype(np.float32)
    x[1] = np.round(x[1] * 8) / 8                                   # ties, both zeros
    x[2] = (x[2] * np.exp(r.normal(size=n) * 4)).astype(np.float32)  # many bins
    for name, w in weight_rows(n).items():
        w = w.astype(np.float32)
        for lam in (1e-6, 1e-3, 0.1, 3.0):
            print(n, name, lam, flush=True)
            ref = oracle.topk_general(x, w, P2, lam, "id")["out"]
            close(host(gpu.topk_general_fwd(dev(x), dev(w), gpu.TOPK_PHI_IDENTITY, P2, lam)), ref, f"{name} {lam}")
    ws = np.sort(r.normal(size=(3, n)).astype(np.float32))[:, ::-1].copy()      # a row of weights per row
    ref = oracle.topk_general(x, ws, P2, 0.05, "id")["out"]
    close(host(gpu.topk_general_fwd(dev(x), dev(ws), gpu.TOPK_PHI_IDENTITY, P2, 0.05)), ref, "weights per row")


def test_values_at_the_ends_of_the_type(gpu, oracle):
    n = 3001
    r = np.random.default_rng(5)
    x = np.stack([r.normal(size=n) * 1e-41, r.normal(size=n) * 1e10, np.full(n, 0.7), np.where(np.arange(n) % 2, 0.0, -0.0),
                  1.0 + 1e-6 * r.random(size=n), np.r_[r.normal(size=n - 1), 1e9]]).astype(np.float32)
    w = np.arange(n, 0, -1, dtype=np.float32)
    for lam in (1e-4, 1.0):
        ref = oracle.topk_general(x, w, P2, lam, "id")["out"]
        close(host(gpu.topk_general_fwd(dev(x), dev(w), gpu.TOPK_PHI_IDENTITY, P2, lam)), ref, f"lambda {lam}")


def test_rows_and_weights_left_to_the_kernel_that_sorts(gpu):
    n = 6000
    r = np.random.default_rng(6)
    x = r.normal(size=(6, n)).astype(np.float32)
    x[1, 17] = np.inf
    x[2, 5] = np.nan
    x[3] = np.float32(1e4) * np.exp(r.normal(size=n) * 20).astype(np.float32)
    w = np.arange(n, 0, -1, dtype=np.float32)
    up = w[::-1].copy()                                             # increasing: everything is one block
    for weights in (w, up):
        for lam in (1e-7, 1e-3, 1.0):
            got = host(gpu.topk_general_fwd(dev(x), dev(weights), gpu.TOPK_PHI_IDENTITY, P2, lam))
            ref, _ = gpu.topk_general_jvp(dev(x), dev(weights), dev(np.zeros_like(x)), gpu.TOPK_PHI_IDENTITY, P2, lam)
            ref = host(ref)
            assert np.array_equal(np.isfinite(got), np.isfinite(ref))
            ok = np.isfinite(ref)
            assert (np.abs(got[ok] - ref[ok]) <= 1e-5 + 1.2e-7 * np.abs(ref[ok])).all()


# Bins whose values are ordered by counting (up to 64) and by a network over all items, the most items that a row
# may have (2816), rows of one value: equal and different values that share a bin.
@pytest.mark.parametrize("m", [2, 63, 64, 65, 66, 700, 2047, 2800, 2815, 2816, 2817])
def test_full_bins(gpu, oracle, m):
    n = 6000
    r = np.random.default_rng(m)
    base = np.where(np.arange(n) < n // 2, -40.0, 40.0) + r.normal(size=n)
    x = np.stack([base, base, base, np.full(n, 0.7)]).astype(np.float32)
    x[0, r.choice(n, m, replace=False)] = 0.7                                  # equal values
    x[1, r.choice(n, m, replace=False)] = 1.0 + 0.1 * r.random(size=m)         # different ones, one bin of 1/8
    x[2, r.choice(n, m, replace=False)] = np.round(1.0 + 0.1 * r.random(size=m), 2)
    for name, w in weight_rows(n).items():
        for lam in (1e-6, 1e-3, 0.1, 3.0):
            w32 = w.astype(np.float32)
            ref = oracle.topk_general(x, w32, P2, lam, "id")["out"]
            close(host(gpu.topk_general_fwd(dev(x), dev(w32), gpu.TOPK_PHI_IDENTITY, P2, lam)), ref, f"{name} {lam}")


# 1000 rows of 2000 equal values: 1200 us when the bin's values are ordered by counting, 200 us with a complete sort
def test_time_of_rows_of_one_value(gpu):
    import torch
    x = torch.full((1000, 2000), 0.7, device="cuda")
    w = torch.arange(2000, 0, -1, device="cuda", dtype=torch.float32)
    times = []
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        gpu.topk_general_fwd(x, w, gpu.TOPK_PHI_IDENTITY, P2, 0.1)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    assert min(times) < 0.6, times


# Rows that are left to the kernel that sorts: lengths around the longest one that a network in LDS sorts (8192) and
# powers of two, with ties (equal keys keep their index order); against the oracle.
@pytest.mark.parametrize("n", [1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193])
def test_rows_left_over_are_sorted(gpu, oracle, n):
    r = np.random.default_rng(n)
    x = np.stack([r.normal(size=n), np.round(r.normal(size=n) * 8) / 8, np.full(n, 0.5), np.sort(r.normal(size=n))]).astype(np.float32)
    up = np.arange(1, n + 1, dtype=np.float32)                                 # increasing: every row is left over
    few = (1.0 / (1.0 + np.arange(n))).astype(np.float32)
    for w, lam in ((up, 0.01), (up, 3.0), (few, 1e-7)):
        ref = oracle.topk_general(x, w, P2, lam, "id")["out"]
        close(host(gpu.topk_general_fwd(dev(x), dev(w), gpu.TOPK_PHI_IDENTITY, P2, lam)), ref, f"{lam}")
