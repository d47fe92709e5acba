"""The one-pass d am / d lm kernel at the edges of its variants: token rows
around 64, 128, 192 and 320 (past it the two separate kernels), frames around
its 32-frame steps, odd and short vocabularies (more targets in a column tile
than one gather round lists), one and several frame ranges, a spread of logits
whose exponentials reach e^-60, and the smoothed joiner.

The plain gradients are compared with the same sums in fp64 over the kernel's
own occupations, d = sum (gx + gy) p - targets and blanks. Bound: W and p carry
the rounding of Z, of the exponentials' arguments and of the hardware exp2
(2^-22 (8 + |argument|) of a term), the contraction one fp32 rounding per 16
frames or rows, and the target terms one per target, each of the sum of the
terms' absolute values. The smoothed ones go against the oracle at the tolerance
that its other tests use."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2206_13236_amd as P
from gpu_common import assert_close, dev_f32, host, make_dev_batch, say
from workloads import make_batch

pytestmark = pytest.mark.gpu


def _case(N, T, U, V, spread=1.0):
    b = make_batch("bpe", seed=T + U + V, N=N, T_range=(T, T), U_range=(U, U), V=V, J=8, S=5, with_joiner=False)
    b.t_len[1], b.u_len[1] = max(1, T - 33), U // 2
    b.am *= np.float32(spread)
    b.lm *= np.float32(spread)
    return b


@pytest.mark.parametrize("N,T,U,V,spread", [
    (2, 31, 63, 70, 1.0), (2, 33, 64, 65, 1.0), (2, 65, 127, 16, 1.0), (2, 40, 128, 131, 1.0), (2, 64, 191, 64, 1.0),
    (2, 34, 192, 100, 1.0), (2, 5, 319, 130, 1.0), (2, 70, 319, 33, 1.0), (2, 34, 320, 70, 1.0), (2, 400, 20, 66, 1.0),
    (2, 97, 90, 9000, 1.0), (2, 1, 1, 3, 1.0), (2, 100, 40, 129, 10.0), (2, 90, 150, 67, 10.0), (300, 40, 5, 20, 1.0),
    # more than 256 items: one group a workgroup, more targets than one gather round lists
    (300, 70, 60, 20, 1.0), (300, 66, 63, 3, 10.0), (300, 65, 100, 30, 1.0), (300, 34, 127, 60, 10.0)])
def test_simple_gradients_over_own_occupations(N, T, U, V, spread):
    say(f"[simple_grad] N={N} T={T} U={U} V={V} spread={spread}")
    b = _case(N, T, U, V, spread)
    r = P.rnnt_simple_loss(make_dev_batch(b), V, dev_f32(b.am), dev_f32(b.lm), want_logprobs=True, want_grads=True)
    torch.cuda.synchronize()
    r = {k: host(r[k]).astype(np.float64) for k in ("px_occ", "py_occ", "am_grad", "lm_grad")}
    big = float(np.abs(b.am).max() + np.abs(b.lm).max())
    eps = 2.0**-22 * (8 + 2 * big) + (T + 2 * U) * 2.0**-25
    for n in (0, 1, N - 1):
        t, u = int(b.t_len[n]), int(b.u_len[n])
        a, l, y = b.am[n, :t].astype(np.float64), b.lm[n, :u + 1].astype(np.float64), b.symbols[n, :u]
        gx, gy = r["px_occ"][n, :t, :u + 1].copy(), r["py_occ"][n, :t, :u + 1]
        gx[:, u] = 0.0
        ma, ml = a.max(1, keepdims=True), l.max(1, keepdims=True)
        ea, el = np.exp(a - ma), np.exp(l - ml)
        w = (gx + gy) / (ea @ el.T)
        dam, dlm = ea * (w @ el), el * (w.T @ ea)
        sam, slm = np.zeros_like(dam), np.zeros_like(dlm)
        np.add.at(sam.T, y, gx[:, :u].T)
        sam[:, b.wl.blank] += gy.sum(1)
        slm[np.arange(u), y] += gx[:, :u].sum(0)
        slm[:, b.wl.blank] += gy.sum(0)
        for name, got, dense, sparse in (("am", r["am_grad"][n], dam, sam), ("lm", r["lm_grad"][n], dlm, slm)):
            k = dense.shape[0]
            err = np.abs(got[:k] - (dense - sparse))
            assert (err <= eps * (dense + sparse) + 1e-12).all(), (name, n, float((err / (dense + sparse + 1e-30)).max()), eps)
            assert not got[k:].any(), (name, n, "padding")


@pytest.mark.parametrize("w", [(0.25, 0.1), (0.4, 0.0), (0.0, 0.3)], ids=["both", "lm", "am"])
@pytest.mark.parametrize("N,T,U,V", [(2, 33, 63, 37), (2, 40, 64, 130), (2, 34, 128, 66), (2, 33, 200, 65),
                                     (2, 34, 63, 8300), (2, 33, 100, 8300)])  # more than 256 items
def test_smoothed_gradients(N, T, U, V, w):
    say(f"[simple_grad] smoothed {w} N={N} T={T} U={U} V={V}")
    b = _case(N, T, U, V)
    sc = np.linspace(0.5, 2.0, N)
    ref = O.smoothed_simple_stage(b.am, b.lm, b.symbols, b.t_len, b.u_len, b.wl.blank, *w, scale=sc)
    got = P.rnnt_simple_loss(make_dev_batch(b), V, dev_f32(b.am), dev_f32(b.lm), dev_f32(sc), want_logprobs=True,
                             want_grads=True, lm_only_scale=w[0], am_only_scale=w[1])
    torch.cuda.synchronize()
    assert_close("am_grad", host(got["am_grad"]), ref["am_grad"], atol=1e-4)
    assert_close("lm_grad", host(got["lm_grad"]), ref["lm_grad"], atol=1e-4)
