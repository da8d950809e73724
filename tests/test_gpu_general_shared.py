"""General weights, p = 2, one weight vector for all rows, rows of up to 1024 elements (the kernel with
shared prefix sums in csrc/general_w.hip): lengths at the edges of its shapes, partial workgroups, ties,
rows that need many rounds.  Oracle; and the same rows with a row of weights each (the other kernel).
Bar: that of test_gpu_parity (1e-5 + one float32 ulp)."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, close, dev, gpu, host  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 32, 33, 63, 64, 65, 128, 129, 255, 256, 257, 512, 513, 1000, 1023, 1024]


@pytest.mark.parametrize("n", EDGES)
def test_lengths_at_the_edges_of_the_shapes(gpu, oracle, n):
    r = np.random.default_rng(n)
    for rows in (1, 2 * 4 * max(1, 512 // n) + 3):
        x = r.normal(size=(rows, n)).astype(np.float32)
        x[rows // 2] = np.round(x[rows // 2] * 4) / 4                          # ties
        t = r.normal(size=x.shape).astype(np.float32)
        for w in (np.arange(n, 0, -1), np.arange(n) < n // 3, 1.0 / (1.0 + np.arange(n))):
            w = w.astype(np.float32)
            for phi, code in (("id", gpu.TOPK_PHI_IDENTITY), ("half_sq", gpu.TOPK_PHI_HALF_SQUARE)):
                for lam in (1.0 / 512, 0.25):
                    ref = oracle.topk_general(x, w, P2, lam, phi, tangent=t)
                    o, j = (host(a) for a in gpu.topk_general_jvp(dev(x), dev(w), dev(t), code, P2, lam))
                    close(o, ref["out"], f"{phi} {lam}")
                    close(j, ref["jvp"], f"{phi} {lam} jvp")
                    f = host(gpu.topk_general_fwd(dev(x), dev(w), code, P2, lam))
                    assert np.array_equal(f, o)
                    each = np.ascontiguousarray(np.broadcast_to(w, x.shape))
                    o2, j2 = (host(a) for a in gpu.topk_general_jvp(dev(x), dev(each), dev(t), code, P2, lam))
                    close(o2, ref["out"], "weights per row")
                    close(j2, ref["jvp"], "weights per row, jvp")


def test_rows_that_lose_one_boundary_per_round(gpu, oracle):
    # one heavy first weight in front of a slowly falling ramp: the block takes in one neighbour per round
    n = 1024
    w = np.ones(n, dtype=np.float32)
    x = (1.0 - 1e-3 * np.arange(n)).astype(np.float32)
    x = np.stack([x, np.sort(np.random.default_rng(1).normal(size=n)).astype(np.float32)[::-1] * 1e-3])
    w[0] = 700.0
    t = np.random.default_rng(2).normal(size=x.shape).astype(np.float32)
    for lam in (0.5, 1.0):
        ref = oracle.topk_general(x, w, P2, lam, "id", tangent=t)
        o, j = (host(a) for a in gpu.topk_general_jvp(dev(x), dev(w), dev(t), gpu.TOPK_PHI_IDENTITY, P2, lam))
        close(o, ref["out"], "out")
        close(j, ref["jvp"], "jvp")
