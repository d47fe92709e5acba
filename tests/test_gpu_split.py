"""The fp32 joiner's contractions on split operands (two fp16 planes per
element): sizes around the 32-element groups and 128-wide tiles, W of any
magnitude and with outliers, occupations and scales of any magnitude.

Bounds. Splitting an element leaves at most 2^-23 of it, the dropped lo lo
product 2^-22 of a product: 2^-21 of a product in all. The fp32 accumulation of
K products in three MFMAs per 32 leaves at most (3 K / 32) 2^-24 of the sum of
their magnitudes; h itself is within 2e-7 (hardware exp2 and reciprocal).
Gradients are compared with the sum of the magnitudes of their products times
2^-20 (a product's 2^-21 and as much for their sum), the log-probs and softmax
that enter them having errors of about 2e-6."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2206_13236_amd as P
from gpu_common import assert_close, dev_f32, dev_i32, host, make_dev_batch, say
from workloads import make_batch

pytestmark = pytest.mark.gpu

# J around the 32-element group, V around groups, tiles and the wide forward's threshold
SIZES = [(8, 31, 2), (24, 33, 3), (32, 64, 4), (40, 127, 5), (96, 129, 5), (136, 257, 7), (64, 2049, 3)]


def _setup(J, V, S, wscale=1.0, outlier=False):
    b = make_batch("bpe", seed=J + V, N=3, T_range=(17, 41), U_range=(1, 11), V=V, J=J, S=S)
    b.W *= np.float32(wscale)
    if outlier:
        b.W[J // 2, V // 3] *= np.float32(300.0)
    ranges = np.zeros((b.N, b.T, S), np.int32)
    for n in range(b.N):
        top = max(0, int(b.u_len[n]) - S + 1)
        p = np.minimum((np.arange(b.T) * top) // max(1, int(b.t_len[n]) - 1), top)
        ranges[n] = p[:, None] + np.arange(S)
    return b, ranges


def _run(b, ranges, S, gscale=1.0, **kw):
    args = [dev_f32(x) for x in (b.enc, b.dec, b.W, b.bias)]
    batch, rg = make_dev_batch(b), dev_i32(ranges)
    jo = P.rnnt_pruned_joiner(batch, S, *args, rg, keep_logits=True)
    pl = P.rnnt_pruned_loss(batch, S, jo["px"], jo["py"], rg)
    g = P.rnnt_pruned_joiner_backward(batch, S, *args, rg, jo["lse"], pl["px_occ"] * gscale, pl["py_occ"] * gscale, **kw)
    torch.cuda.synchronize()
    return jo, pl, g


@pytest.mark.parametrize("J,V,S", SIZES)
@pytest.mark.parametrize("wscale,outlier", [(1.0, False), (1e-6, False), (1.0, True)], ids=["unit", "tiny", "outlier"])
def test_split_joiner_against_oracle(J, V, S, wscale, outlier):
    say(f"[split] J={J} V={V} S={S} W x {wscale} outlier={outlier}")
    b, ranges = _setup(J, V, S, wscale, outlier)
    jo, pl, g = _run(b, ranges, S)
    st = O.pruned_stage(b.enc, b.dec, b.W, b.bias, ranges, b.symbols, b.t_len, b.u_len, b.wl.blank)
    W = np.abs(b.W.astype(np.float64))
    # logits: the largest of |h| |W| summed over J (|h| <= 1), and h's own error
    bound = (3 * (J / 32 + 1) * 2.0**-24 + 2.0**-21) * W.sum(0) + 2e-7 * W.sum(0)
    ref = O.pruned_joiner_logits(b.enc, b.dec, b.W, b.bias, ranges, b.t_len, b.u_len)
    got = host(jo["logits"])
    for n in range(b.N):
        on = np.zeros((b.T, S), bool)
        on[:b.t_len[n]] = ranges[n, :b.t_len[n]] <= b.u_len[n]
        err = np.abs(got[n][on] - np.asarray(ref[n])[on])
        assert np.all(err <= bound + 1e-30), float((err - bound).max())
    assert_close("pruned_loss", host(pl["loss"]), st["loss"], rtol=1e-5)
    gsum = (st["gx"] + st["gy"]).sum()
    # |d(logits)| summed over a row is at most 2 (gx + gy): the gradients' products sum to at most this
    for k, mag in (("W_grad", 2 * gsum), ("bias_grad", 2 * gsum), ("enc_grad", 2 * S * W.max()), ("dec_grad", 2 * gsum * W.max())):
        atol = (2.0**-20 + 2e-6) * mag
        assert_close(k, host(g[k]), st[k], atol=atol)


@pytest.mark.parametrize("gscale", [1e-9, 1e5], ids=["tiny", "huge"])
def test_split_backward_scales_with_the_occupations(gscale):
    """d(logits) of any magnitude: the backward is linear in the occupations
    (and in scale), to the rounding of the scaled occupations."""
    say(f"[split] occupations x {gscale}")
    b, ranges = _setup(96, 129, 5)
    _, _, ref = _run(b, ranges, 5)
    _, _, got = _run(b, ranges, 5, gscale=gscale)
    _, _, sc = _run(b, ranges, 5, scale=torch.full((b.N,), gscale, device="cuda"))
    for out in (got, sc):
        for k in ("W_grad", "bias_grad", "enc_grad", "dec_grad"):
            r = host(ref[k])
            assert_close(k, host(out[k]) / gscale, r, atol=4e-6 * np.abs(r).max())


# d(logits) of the backward's three producers: recomputed, streamed from the head, streamed from stored logits
PATHS = ["recomputed", "head", "logits"]


def _backward(b, ranges, S, path, scale):
    args = [dev_f32(x) for x in (b.enc, b.dec, b.W, b.bias)]
    batch, rg = make_dev_batch(b), dev_i32(ranges)
    C = P.backward_chunk_rows(b.N, b.T, S, b.wl.J, b.V, P.RNNT_F32)
    kw = dict(head=torch.empty(C, (b.V + 7) // 8 * 8, device="cuda"), head_rows=C) if path == "head" else {}
    jo = P.rnnt_pruned_joiner(batch, S, *args, rg, keep_logits=path == "logits", **kw)
    pl = P.rnnt_pruned_loss(batch, S, jo["px"], jo["py"], rg)
    g = P.rnnt_pruned_joiner_backward(batch, S, *args, rg, jo["lse"], pl["px_occ"], pl["py_occ"],
                                      scale=dev_f32(np.asarray(scale)), logits=jo["logits"], **kw)
    torch.cuda.synchronize()
    return g


def _rel(got, ref):
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("path", PATHS)
def test_split_backward_keeps_each_utterance_its_own_magnitude(path):
    """Utterances whose scales differ by 1e5 and 1e10: each one's d enc and d
    dec against 64 bits, relative to its own norm. Bound: 2^-21 a product, the
    fp32 sums over V and S rows and the 2e-6 of the softmax that enters
    d(logits), which adds up along a row at worst: 2e-5."""
    b, ranges = _setup(96, 129, 5)
    scale = np.array([1.0, 1e-5, 1e-10])
    say(f"[split] scales {scale} {path}")
    g = _backward(b, ranges, 5, path, scale)
    st = O.pruned_stage(b.enc, b.dec, b.W, b.bias, ranges, b.symbols, b.t_len, b.u_len, b.wl.blank, scale=scale)
    for k in ("enc_grad", "dec_grad"):
        got = host(g[k])
        for n in range(b.N):
            assert _rel(got[n], st[k][n]) < 2e-5, (k, n)


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("J,V", [(40, 127), (96, 300)])
def test_split_weight_gradient_of_improbable_tokens(J, V, path):
    """Tokens of probability e^-15 to e^-45 at every row, that are no target or
    one only in an utterance of scale 1e-6: each one's column of d W against
    64 bits, relative to its own norm. Bound: as above, and the 1e-6 relative
    error that 2^-24 of a logit of 45 gives its exponential times its sum: 4e-5."""
    say(f"[split] improbable tokens J={J} V={V} {path}")
    b, ranges = _setup(J, V, 5)
    cols = [v for v in range(1, V) if v not in b.symbols][:6]
    b.bias[cols] -= np.array([15, 20, 25, 30, 35, 45][:len(cols)], np.float32)
    scale = np.ones(b.N)
    scale[2] = 1e-6
    b.symbols[b.symbols == cols[0]] = cols[-1]
    b.symbols[2, 0] = cols[2]
    g = _backward(b, ranges, 5, path, scale)
    st = O.pruned_stage(b.enc, b.dec, b.W, b.bias, ranges, b.symbols, b.t_len, b.u_len, b.wl.blank, scale=scale)
    got = host(g["W_grad"])
    for v in range(V):
        assert _rel(got[:, v], st["W_grad"][:, v]) < 4e-5, (v, v in cols)


@pytest.mark.parametrize("J,V", [(40, 127), (64, 2100)])
def test_split_forward_with_an_infinite_weight(J, V):
    """W = -inf where h > 0 at every row masks a token: its logit is -inf, the
    others and the loss are those of 64 bits. A NaN makes the logits of its
    column NaN and no others. (rtol and atol as for finite W.)"""
    say(f"[split] infinite weight J={J} V={V}")
    b, ranges = _setup(J, V, 5)
    v0 = next(v for v in range(1, V) if v not in b.symbols)
    b.enc[..., 3] = np.abs(b.enc[..., 3])
    b.dec[..., 3] = np.abs(b.dec[..., 3])
    b.W[3, v0] = -np.inf
    jo, pl, _ = _run(b, ranges, 5)
    with np.errstate(invalid="ignore"):
        px, py, lse = O.pruned_joiner_logprobs(b.enc, b.dec, b.W, b.bias, ranges, b.symbols, b.t_len, b.u_len, 0)
    loss, _, _ = O.pruned_loss(px, py, ranges, b.t_len, b.u_len)
    assert np.isfinite(loss).all()
    assert_close("lse", host(jo["lse"]), lse, atol=5e-5)
    assert_close("px", host(jo["px"]), px, atol=5e-5)
    assert_close("pruned_loss", host(pl["loss"]), loss, rtol=1e-5)
    b.W[3, v0] = np.nan
    jo, pl, _ = _run(b, ranges, 5)
    on = np.arange(b.T)[None, :, None] < b.t_len[:, None, None]
    on = on & (ranges <= b.u_len[:, None, None])
    nan = np.isnan(host(jo["logits"])[on])
    assert nan[:, v0].all() and nan.sum() == on.sum() and np.isnan(host(pl["loss"])).all()


@pytest.mark.parametrize("T,dtype", [(1300, "f32"), (1700, "f32"), (2900, "bf16")], ids=["four_chunks", "five_chunks", "bf16"])
def test_forward_of_many_row_chunks(T, dtype):
    """Padded rows of up to four forward chunks, whose first h pass runs in the prep kernel's blocks, and of more, where
    it is a launch of its own: bitwise the same as each utterance in a batch of its own (one chunk)."""
    N, U, S, J, V = 6, 9, 8, 16, 19
    say(f"[split] {N * T * S} rows {dtype}")
    g = torch.Generator(device="cuda").manual_seed(T)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    enc, dec, W, bias = (torch.randn(s, generator=g, device="cuda").to(dt) for s in ((N, T, J), (N, U + 1, J), (J, V), (V,)))
    t_len = dev_i32([T, T - 700, T, 5, T - 1, T - 300])
    u_len, sym = dev_i32([U, 3, U, 4, 0, U]), torch.randint(1, V, (N, U), generator=g, device="cuda", dtype=torch.int32)
    rg = (torch.arange(T, device="cuda")[None, :, None] * (u_len[:, None, None] - S + 1).clamp(min=0) // T).int()
    rg = (rg + torch.arange(S, device="cuda", dtype=torch.int32)).contiguous()
    jo = P.rnnt_pruned_joiner(P.Batch(t_len, u_len, sym, T, U), S, enc, dec, W, bias, rg)
    for n in range(N):
        one = P.Batch(t_len[n:n + 1], u_len[n:n + 1], sym[n:n + 1], T, U)
        ref = P.rnnt_pruned_joiner(one, S, enc[n:n + 1], dec[n:n + 1], W, bias, rg[n:n + 1])
        torch.cuda.synchronize()
        for k in ("px", "py", "lse"):
            assert torch.equal(jo[k][n:n + 1], ref[k]), (k, n)
