"""General weights, p = 2, rows of 257..1024 elements: the sort on 32-bit words (csrc/general_w.hip), where the leading bits of
the values decide, where neighbours have to be exchanged, where neither is enough and the row is sorted by complete keys, and
where that is seen beforehand; shorter rows, which are sorted by complete keys.  Against the oracle with the bar of test_gpu_parity, and bit
for bit against the kernel that is used when rounds are asked for."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, close, dev, gpu, host  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


def _rows(r, n):
    near = 1.0 + np.arange(n) * 2.0 ** -23                       # agree in all but the last bits
    wide = r.normal(size=n)
    wide[r.permutation(n)[: n // 8]] *= 1e30
    inf = r.normal(size=n)
    inf[::5] = -1e38
    rows = [r.normal(size=n), r.permutation(near), 100.0 + 1e-3 * r.normal(size=n),
            np.where(r.random(n) < 0.5, 1e-3 * r.normal(size=n), 100.0 + 1e-3 * r.normal(size=n)),
            np.sort(r.normal(size=n)), wide, inf, np.maximum(r.normal(size=n), 0.0),
            np.full(n, 0.75)]
    late = r.normal(size=n)                                      # a cluster that the first 64 elements do not show
    late[n // 2:] = 100.0 + 1e-3 * late[n // 2:]
    few = r.normal(size=n)                                       # one that takes more exchanges than are made
    few[n - 20:] = 100.0 + 1e-3 * few[n - 20:]
    masked = np.where(np.arange(n) % 3 > 0, np.round(r.normal(size=n) * 4096) / 4096, -2.0 ** 30)      # (exact sums)
    zeros = np.where(np.arange(n) % 2 > 0, 0.0, -0.0)
    return np.stack(rows + [late, few, masked, zeros]).astype(np.float32)


@pytest.mark.parametrize("n", [129, 256, 257, 512, 513, 1000, 1024])
def test_every_way_to_the_order(gpu, oracle, n):
    r = np.random.default_rng(n)
    x = _rows(r, n)
    t = r.normal(size=x.shape).astype(np.float32)
    w = np.arange(n, 0, -1).astype(np.float32)
    for phi, phic in (("id", gpu.TOPK_PHI_IDENTITY), ("half_sq", gpu.TOPK_PHI_HALF_SQUARE)):
        for lam in (1e-6, 0.1):
            # (rows of few values have pooled values that tie in real arithmetic only, and 1e30 has no absolute bar)
            rows = [0, 1, 2, 3, 4, 9, 10]
            ref = oracle.topk_general(x[rows], w, P2, lam, phi, tangent=t[rows])
            o, j = (host(a) for a in gpu.topk_general_jvp(dev(x), dev(w), dev(t), phic, P2, lam))
            if lam > 1e-3 or phi == "half_sq":
                close(o[rows], ref["out"], "fwd")
                if phi == "id":
                    close(j[rows], ref["jvp"], "jvp")
            gpu.set_route(gpu.TOPK_ROUTE_GENERAL_ROUNDS, 4096)
            try:
                o2, j2 = (host(a) for a in gpu.topk_general_jvp(dev(x), dev(w), dev(t), phic, P2, lam))
            finally:
                gpu.set_route(gpu.TOPK_ROUTE_GENERAL_ROUNDS, 0)
            assert np.array_equal(o, o2), (phi, lam, np.argwhere(o != o2)[:4])
            assert np.array_equal(j, j2), (phi, lam, np.argwhere(j != j2)[:4])
