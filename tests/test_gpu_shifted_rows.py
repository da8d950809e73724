"""Rows of 192 .. 2045 elements that do not start at 16-byte boundaries, with a tangent or a target: 16-byte accesses at
the addresses' own alignment (csrc/short_rows_value.hpp, SHIFT).  Lengths on both sides of every limit of that rule, arrays
starting at every word of 16 bytes, the words beside the arrays untouched; against the oracle (bar: that of test_gpu_parity)
and against arrays that disagree modulo 16 bytes, which are accessed element by element."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, P43, close, gpu, host  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu
ROWS, MARK = 5, 77.0


def place(a, shape, word):
    """`a` (None: marks) as a view that starts `word` words past a 16-byte boundary, in a buffer full of marks."""
    import torch
    size = int(np.prod(shape))
    buf = torch.full((size + 16,), MARK, device="cuda")
    v = buf[8 + word:8 + word + size].view(shape)
    if a is not None:
        v.copy_(torch.from_numpy(a))
    return buf, v


def untouched(buf, word, size):
    b = host(buf)
    assert (b[:8 + word] == MARK).all() and (b[8 + word + size:] == MARK).all(), "a word beside the array was written"


@pytest.mark.parametrize("n", [191, 192, 193, 253, 254, 381, 384, 387, 509, 510, 513, 516, 575, 577, 1020, 1021, 1022, 1025,
                               1151, 1153, 2042, 2045, 2046])
def test_rows_at_every_word(gpu, oracle, n):
    r = np.random.default_rng(n)
    shape = (ROWS, n)
    x = r.normal(size=shape).astype(np.float32)
    x[1] = np.round(x[1] * 4) / 4                                    # ties
    t = r.normal(size=shape).astype(np.float32)
    ks = (3, 70 if n < 1024 else 30)                                 # (above and below the lanes of a row)
    for word in range(4):
        words = [(word,) * 4, (word, word, word, (word + 1) % 4)]    # x, tangent, out, jvp
        for k in ks:
            for p, lam in ((P2, 0.5), (P43, 0.05)):
                for name in ("topk_mask", "topkmag", "topk_signed_mask", "topk_masked_value"):
                    print(name, n, word, k, p, lam, flush=True)
                    got = []
                    for at in words:
                        (_, xv), (_, tv) = place(x, shape, at[0]), place(t, shape, at[1])
                        (ob, ov), (jb, jv) = place(None, shape, at[2]), place(None, shape, at[3])
                        getattr(gpu, name + "_jvp")(xv, tv, k, p, lam, out=ov, jvp_out=jv)
                        got.append((host(ov), host(jv)))
                        untouched(ob, at[2], ROWS * n)
                        untouched(jb, at[3], ROWS * n)
                    ref = getattr(oracle, name)(x, k, p, lam, tangent=t)
                    for o, j in got:
                        close(o, ref["out"], name)
                        close(j, ref["jvp"], name + " jvp")
                    assert np.array_equal(got[0][0], got[1][0]), name
                ref_loss, ref_grad = oracle.fenchel_young_loss(x, t, k, p, lam)
                for at in words:
                    (_, xv), (_, tv), (gb, gv) = place(x, shape, at[0]), place(t, shape, at[1]), place(None, shape, at[3])
                    loss, _ = gpu.topk_mask_loss(xv, tv, k, p, lam, grad_out=gv)
                    close(host(gv), ref_grad, "grad")
                    close(host(loss), ref_loss, "loss")
                    untouched(gb, at[3], ROWS * n)
