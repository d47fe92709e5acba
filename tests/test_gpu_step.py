"""The whole step in one call against the stages called one by one, on one
stream and with the second stream (forced at sizes below its threshold), and
the scaling of stored gradients: bitwise equal in both cases."""
import pytest
import torch

import paper_2206_13236_amd as P
from gpu_common import dev_f32, dev_joiner, make_dev_batch, say
from workloads import make_batch

pytestmark = pytest.mark.gpu


def _stages(b, batch, S, args):
    """The stages of a step by their own entry points (simple scale 0.5, sum)."""
    am, lm, enc, dec, W, bias = args
    N, T, U, V, J = batch.N, batch.T, batch.U, b.V, int(W.shape[0])
    dt = P.RNNT_BF16 if W.dtype == torch.bfloat16 else P.RNNT_F32
    sc = torch.full((N,), 0.5, device="cuda")
    sim = P.rnnt_simple_loss(batch, V, am, lm, sc, want_grads=True)
    rg = P.rnnt_prune_ranges(batch, S, sim["px_occ"], sim["py_occ"])
    C = P.backward_chunk_rows(N, T, S, J, V, dt)
    head = torch.empty(C, (V + 7) // 8 * 8, device="cuda")
    jo = P.rnnt_pruned_joiner(batch, S, enc, dec, W, bias, rg, head=head, head_rows=C)
    pl = P.rnnt_pruned_loss(batch, S, jo["px"], jo["py"], rg)
    g = P.rnnt_pruned_joiner_backward(batch, S, enc, dec, W, bias, rg, jo["lse"], pl["px_occ"], pl["py_occ"],
                                      head=head, head_rows=C)
    c = P.rnnt_combine_losses(sim["loss"], pl["loss"], 0.5, 1.0)
    return {"simple_loss": sim["loss"], "am_grad": sim["am_grad"], "lm_grad": sim["lm_grad"], "ranges": rg,
            "pruned_loss": pl["loss"], "loss": c["loss"], "total": c["total"],
            **{k: g[k] for k in ("enc_grad", "dec_grad", "W_grad", "bias_grad")}}


@pytest.mark.parametrize("work", [0, 1 << 62], ids=["two_streams", "one_stream"])
@pytest.mark.parametrize("wl", ["tiny", "bpe", "long"])
def test_step_equals_its_stages(wl, work, monkeypatch):
    say(f"[step] {wl} overlap from {work}")
    monkeypatch.setattr(P, "_OVERLAP_WORK", work)
    b = make_batch("tiny") if wl == "tiny" else make_batch(wl, seed=3, N=3, T_range=(30, 61), U_range=(5, 17), V=133, J=72)
    bf, S = b.wl.joiner_dtype == "bf16", b.wl.S
    args = (dev_f32(b.am), dev_f32(b.lm), *(dev_joiner(x, bf) for x in (b.enc, b.dec, b.W, b.bias)))
    batch = make_dev_batch(b)
    ref = _stages(b, batch, S, args)
    step = P.PrunedRnntLoss(S)
    for _ in range(3):
        out = step.step(batch, *args)
    torch.cuda.synchronize()
    for k, r in ref.items():
        assert torch.equal(out[k], r), k


@pytest.mark.parametrize("pruned_scale", [1.0, 0.0])
def test_first_step_of_each_size_equals_the_kept_one(pruned_scale, monkeypatch):
    """A module's first step, and its first of other sizes, runs its stages up to the joiner by their own calls: every
    output bitwise that of a module that has its buffers; sizes that come back too."""
    monkeypatch.setattr(P, "_OVERLAP_WORK", 0)
    cases = [("bpe", dict(seed=3, N=3, T_range=(30, 61), U_range=(5, 17), V=133, J=72)),
             ("long", dict(seed=4, N=2, T_range=(20, 41), U_range=(5, 9), V=70, J=40))]
    step = P.PrunedRnntLoss(5, pruned_scale=pruned_scale)
    for wl, kw in (cases + cases)[:3]:
        say(f"[step] first of {wl} {kw} pruned scale {pruned_scale}")
        b = make_batch(wl, **kw)
        bf = b.wl.joiner_dtype == "bf16"
        args = (dev_f32(b.am), dev_f32(b.lm), *(dev_joiner(x, bf) for x in (b.enc, b.dec, b.W, b.bias)))
        batch, kept = make_dev_batch(b), P.PrunedRnntLoss(5, pruned_scale=pruned_scale)
        for _ in range(2):
            ref = kept.step(batch, *args)
        got = step.step(batch, *args)
        torch.cuda.synchronize()
        assert got.keys() == ref.keys()
        for k, r in ref.items():
            assert torch.equal(got[k], r), k


def test_step_refuses_mismatched_arguments():
    b = make_batch("tiny")
    args = [dev_f32(b.am), dev_f32(b.lm), *(dev_joiner(x, False) for x in (b.enc, b.dec, b.W, b.bias))]
    batch, step = make_dev_batch(b), P.PrunedRnntLoss(b.wl.S)
    for i in range(6):
        bad = list(args)
        bad[i] = bad[i][..., :-1].contiguous()
        with pytest.raises((ValueError, TypeError)):
            step.step(batch, *bad)
    with pytest.raises(ValueError):
        step.step(batch, *args, out={"px": torch.empty(1, device="cuda")})
    # W with the right shape but another layout (a linear layer's transposed weight) or in host memory
    W = args[4]
    for bad in (W.t().contiguous().t(), W.cpu()):
        with pytest.raises(ValueError):
            step.step(batch, *args[:4], bad, args[5])
        with pytest.raises(ValueError):
            P.rnnt_full_loss(batch, args[2], args[3], bad, args[5])
        r = P.rnnt_prune_ranges(batch, b.wl.S, *(torch.rand(b.N, b.T, b.U + 1, device="cuda") for _ in range(2)))
        with pytest.raises(ValueError):
            P.rnnt_pruned_joiner(batch, b.wl.S, args[2], args[3], bad, args[5], r)
        one = torch.zeros(b.N, b.T, b.wl.S, device="cuda")
        with pytest.raises(ValueError):
            P.rnnt_pruned_joiner_backward(batch, b.wl.S, args[2], args[3], bad, args[5], r, one, one, one)


OUTPUTS = ["am_grad", "lm_grad", "enc_grad", "dec_grad", "W_grad", "bias_grad", "loss", "simple_loss", "pruned_loss"]


@pytest.mark.parametrize("pruned_scale", [1.0, 0.0])
def test_step_refuses_outputs_that_do_not_fit(pruned_scale):
    """An output array too short, of another type, strided or in host memory is refused before anything is launched;
    one of the right size in another shape is written."""
    b = make_batch("tiny")
    args = [dev_f32(b.am), dev_f32(b.lm), *(dev_joiner(x, False) for x in (b.enc, b.dec, b.W, b.bias))]
    batch = make_dev_batch(b)
    step = P.PrunedRnntLoss(b.wl.S, pruned_scale=pruned_scale)
    ref = {k: v.clone() for k, v in step.step(batch, *args).items()}
    for key in OUTPUTS:
        good = torch.empty_like(ref[key])
        bad = [good.flatten()[:-1].clone(), good.double(), good.cpu(),
               torch.empty(2 * good.numel(), device="cuda")[::2].view_as(good)]
        if pruned_scale == 0.0 and key in ("enc_grad", "dec_grad", "W_grad", "bias_grad", "pruned_loss"):
            continue  # zeroed by torch, in whatever form
        for t in bad:
            with pytest.raises((ValueError, TypeError)):
                step.step(batch, *args, out={key: t})
    flat = {k: torch.empty(ref[k].numel(), device="cuda") for k in ("am_grad", "W_grad", "total")}
    out = step.step(batch, *args, out=flat)
    torch.cuda.synchronize()
    for k, t in flat.items():
        assert out[k] is t and torch.equal(t.view(ref[k].shape), ref[k]), k


@pytest.mark.parametrize("divisor", [1.0, 13.0])
def test_scaled_gradients(divisor):
    """Counts around the vector width and a block, both types, an offset source (not 16-byte aligned)."""
    say(f"[step] scaled gradients / {divisor}")
    g = torch.tensor(0.37, device="cuda")
    src = [torch.randn(n + 1, device="cuda")[off:off + n] for n, off in ((1, 0), (3, 0), (4097, 0), (8192, 1), (5, 1), (4096, 0))]
    types = (torch.float32, torch.bfloat16, torch.bfloat16, torch.float32, torch.bfloat16, torch.bfloat16)
    dst = [torch.empty(s.shape, dtype=t, device="cuda") for s, t in zip(src, types)]
    arr = (P.RnntScaled * 6)(*[(s.data_ptr(), d.data_ptr(), s.numel(), int(d.dtype == torch.bfloat16))
                               for s, d in zip(src, dst)])
    P.check(P.lib().rnnt_scale_gradients(6, arr, g.data_ptr(), divisor, None))
    torch.cuda.synchronize()
    for s, d in zip(src, dst):
        assert torch.equal(d, (s * (g / divisor)).to(d.dtype))


def test_backward_through_hooks_and_create_graph():
    """Saved-tensor hooks and a second differentiation take torch's own products, with the same result."""
    b = make_batch("tiny")
    batch = make_dev_batch(b)
    leaves = [t.requires_grad_(True) for t in (dev_f32(b.am), dev_f32(b.lm), *(dev_joiner(x, False) for x in
                                                                               (b.enc, b.dec, b.W, b.bias)))]
    ref = torch.autograd.grad(P.pruned_rnnt_loss(*leaves, batch, b.wl.S, reduction="mean"), leaves)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.double(), lambda t: t.float()):
        got = torch.autograd.grad(P.pruned_rnnt_loss(*leaves, batch, b.wl.S, reduction="mean"), leaves)
    w = torch.tensor(2.0, device="cuda", requires_grad=True)
    loss = P.pruned_rnnt_loss(*leaves, batch, b.wl.S, reduction="mean") * w
    first = torch.autograd.grad(loss, leaves, create_graph=True)
    dw, = torch.autograd.grad(first[0].sum(), w)
    for r, a, f in zip(ref, got, first):
        assert torch.equal(a, r) and torch.allclose(f, 2 * r, rtol=1e-6)
    assert torch.allclose(dw, ref[0].sum(), rtol=1e-4, atol=1e-5)


def test_backward_of_batched_and_dual_gradients():
    """Incoming gradients that are no plain arrays take torch's own products: a batch of them (vmap has no storage
    to point at) and a forward-mode dual (whose tangent is the gradients' tangent)."""
    b = make_batch("tiny")
    batch = make_dev_batch(b)
    leaves = [t.requires_grad_(True) for t in (dev_f32(b.am), dev_f32(b.lm), *(dev_joiner(x, False) for x in
                                                                               (b.enc, b.dec, b.W, b.bias)))]
    loss = P.pruned_rnnt_loss(*leaves, batch, b.wl.S, reduction="mean")
    ref = torch.autograd.grad(loss, leaves, retain_graph=True)
    gs = torch.tensor([1.0, -0.5, 3.0], device="cuda")
    got = torch.autograd.grad(loss, leaves, gs, is_grads_batched=True, retain_graph=True)
    for r, x in zip(ref, got):
        assert x.shape == (3, *r.shape)
        for k, f in enumerate(gs.tolist()):
            assert torch.allclose(x[k], f * r, rtol=1e-6, atol=0)
    with torch.autograd.forward_ad.dual_level():
        g = torch.autograd.forward_ad.make_dual(torch.ones((), device="cuda"), torch.full((), 0.25, device="cuda"))
        got = torch.autograd.grad(loss, leaves, g)
        for r, x in zip(ref, got):
            v, t = torch.autograd.forward_ad.unpack_dual(x)
            assert torch.allclose(v, r, rtol=1e-6, atol=0) and torch.allclose(t, 0.25 * r, rtol=1e-6, atol=0)
