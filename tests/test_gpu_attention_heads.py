"""Matrix-instruction attention at both head sizes (64 and 128) and at the edges of its tiles, forward and backward,
against attention in fp64 on the same bf16 values; and head size 64 in packed batches.  The outputs are rounded to bf16
(2^-9 relative) and the probabilities and score gradients to bf16 before their products, each 2^-9 off at most and in
random directions: 1 % of the largest value bounds what was seen (0.3 %) three times over."""
import math

import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, stream, sync

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2602_05145_amd import binding
    return binding


def _reference(qkv, dout, n, nh, nkv, dh):
    x = qkv.double().cpu().requires_grad_()
    q, k, v = (t.transpose(0, 1) for t in x.view(n, nh + 2 * nkv, dh).split([nh, nkv, nkv], 1))
    k, v = (t.repeat_interleave(nh // nkv, 0) for t in (k, v))
    s = q @ k.transpose(1, 2) / math.sqrt(dh)
    s = s.masked_fill(torch.ones(n, n, dtype=torch.bool).triu(1), -math.inf)
    o = (torch.softmax(s, -1) @ v).transpose(0, 1).reshape(n, nh * dh)
    o.backward(dout.double().cpu())
    return o.detach(), torch.logsumexp(s, -1).detach(), x.grad


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("S,nh,nkv", [(1, 2, 1), (31, 2, 2), (64, 4, 2), (65, 3, 1), (127, 4, 4), (128, 8, 8), (129, 16, 8), (333, 8, 2), (777, 4, 1)])
def test_attention_at_the_edges_of_its_tiles(B, dh, S, nh, nkv):
    bt = 2
    g = torch.Generator(device=DEV).manual_seed(S * dh + nh)
    qkv = torch.randn(bt * S, (nh + 2 * nkv) * dh, device=DEV, generator=g).bfloat16()
    dout = torch.randn(bt * S, nh * dh, device=DEV, generator=g).bfloat16()
    out, dqkv = torch.full_like(dout, float("nan")), torch.full_like(qkv, float("nan"))
    lse, delta = (torch.full((bt, nh, S), float("nan"), device=DEV) for _ in range(2))
    print(f"attention S={S} nh={nh} nkv={nkv} dh={dh}", flush=True)
    B.tide_attention_fwd(bt, S, nh, nkv, dh, qkv, out, lse, 1, stream())
    sync()
    B.tide_attention_bwd(bt, S, nh, nkv, dh, qkv, out, dout, lse, delta, dqkv, 1, stream())
    sync()
    for b in range(bt):
        rows = slice(b * S, (b + 1) * S)
        ro, rl, rg = _reference(qkv[rows], dout[rows], S, nh, nkv, dh)
        assert float((out[rows].double().cpu() - ro).abs().max()) < 1e-2 * float(ro.abs().max())
        assert float((lse[b].double().cpu() - rl).abs().max()) < 1e-5 * max(1.0, float(rl.abs().max()))
        w = nh * dh
        for part in (slice(0, w), slice(w, w + nkv * dh), slice(w + nkv * dh, None)):   # dq, dk, dv
            assert float((dqkv[rows, part].double().cpu() - rg[:, part]).abs().max()) < 1e-2 * max(1e-30, float(rg[:, part].abs().max())) or S == 1


@pytest.mark.parametrize("lens,tail", [([200, 56, 129, 3], 12), ([1] * 9 + [250], 5)])
def test_head_size_64_in_a_packed_training_step(lens, tail):
    from oracle import tide_oracle as O
    from paper_2602_05145_amd import runtime, workloads as W
    T = sum(lens) + tail
    cfg = W.get_config("small", batch=1, seq=T, target_hidden=256, hidden=256, n_heads=4, n_kv_heads=2, head_dim=64, ffn=512, vocab=2048,
                       mask="none", seed=77)
    wl = W.make_workload(cfg)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    tr = runtime.trainer_from_workload(cfg, wl)
    tr.set_packed(cu)
    tr.workspace.fill_(0xFF)
    print(f"packed head size 64 lens={lens}", flush=True)
    tr.train_step_packed(cfg["lr"])
    sync()
    p0 = {k: np.asarray(v, np.float64) for k, v in wl["params"].items()}
    loss, grads = O.train_quantities_packed(cfg, p0, wl["hidden"].astype(np.float64), wl["tokens"], wl["mask"], cu)[:2]
    assert abs(float(tr.loss.item()) - loss) < 1e-2 * abs(loss)
    for k, ref in grads.items():
        a, b = tr.host(tr.grads)[k].reshape(-1), ref.reshape(-1)
        assert a @ b / (np.linalg.norm(a) * np.linalg.norm(b)) > 0.999, k


def test_both_forms_of_the_key_gradient_passes_agree(B):
    """The dK / dV passes take four sets of waves per block when blocks are few, four waves otherwise: the same sequence
    alone (one sequence: few) and as one of many (the other form) gives the same gradients up to the order of the fp32 sums."""
    S, nh, nkv, dh, many = 300, 8, 8, 128, 48
    g = torch.Generator(device=DEV).manual_seed(3)
    qkv = torch.randn(S, (nh + 2 * nkv) * dh, device=DEV, generator=g).bfloat16()
    dout = torch.randn(S, nh * dh, device=DEV, generator=g).bfloat16()
    got = []
    for bt in (1, many):
        q, do = qkv.repeat(bt, 1), dout.repeat(bt, 1)
        out, dq = torch.empty_like(do), torch.full_like(q, float("nan"))
        lse, delta = torch.empty(bt, nh, S, device=DEV), torch.empty(bt, nh, S, device=DEV)
        print(f"dK/dV forms batch={bt}", flush=True)
        B.tide_attention_fwd(bt, S, nh, nkv, dh, q, out, lse, 1, stream())
        B.tide_attention_bwd(bt, S, nh, nkv, dh, q, out, do, lse, delta, dq, 1, stream())
        sync()
        got.append(dq.view(bt, S, -1).double())
    assert float((got[1] - got[1][:1]).abs().max()) == 0.0
    diff, top = (got[0][0] - got[1][0]).abs(), got[1][0].abs().max()
    assert float(diff.max()) < 2.0 ** -7 * float(top)      # one step of bf16 at most


_SHAPES = [(1, 1, 1, 2), (15, 2, 1, 64), (16, 4, 2, 64), (17, 2, 2, 20), (64, 3, 1, 24), (65, 4, 2, 66), (130, 2, 1, 80), (200, 2, 1, 129), (150, 2, 2, 256)]


@pytest.mark.parametrize("dtype,S,nh,nkv,dh", [(t, *s) for t in ("fp32", "bf16") for s in _SHAPES if t == "fp32" or s[3] != 64])
def test_attention_in_fp32_arithmetic(B, dtype, S, nh, nkv, dh):
    """The kernels of fp32 mode and of the other head sizes: tiles of 16 rows and 64, channel groups of 16 (padded, unaligned
    and at the widest head), against fp64.  fp32: 1e-5 of the largest value (sums of up to 256 products and of S probabilities);
    bf16: half a step of the result (2^-8)."""
    bt, dt, code, tol = 2, *((torch.float32, 0, 1e-5) if dtype == "fp32" else (torch.bfloat16, 1, 2.0 ** -8))
    g = torch.Generator(device=DEV).manual_seed(S + dh)
    qkv = torch.randn(bt * S, (nh + 2 * nkv) * dh, device=DEV, generator=g).to(dt)
    dout = torch.randn(bt * S, nh * dh, device=DEV, generator=g).to(dt)
    out, dqkv = torch.full_like(dout, float("nan")), torch.full_like(qkv, float("nan"))
    lse, delta = (torch.full((bt, nh, S), float("nan"), device=DEV) for _ in range(2))
    print(f"attention {dtype} S={S} nh={nh} nkv={nkv} dh={dh}", flush=True)
    B.tide_attention_fwd(bt, S, nh, nkv, dh, qkv, out, lse, code, stream())
    sync()
    B.tide_attention_bwd(bt, S, nh, nkv, dh, qkv, out, dout, lse, delta, dqkv, code, stream())
    sync()
    for b in range(bt):
        rows = slice(b * S, (b + 1) * S)
        ro, rl, rg = _reference(qkv[rows], dout[rows], S, nh, nkv, dh)
        assert float((out[rows].double().cpu() - ro).abs().max()) < tol * float(ro.abs().max())
        assert float((lse[b].double().cpu() - rl).abs().max()) < 1e-5 * max(1.0, float(rl.abs().max()))
        # delta is made from the rounded output, which the reference does not see: 2^-8 of it on top in bf16
        assert float((dqkv[rows].double().cpu() - rg).abs().max()) < 2 * tol * float(rg.abs().max())


@pytest.mark.parametrize("bf16", [0, 1])
def test_later_positions_reach_nothing_before_them(B, bf16):
    """NaN and infinities from position 50 on leave the outputs of the positions before it as they are (in bf16: up to
    a step of the result's type, at most 2^-7 of it: the rows of such a tile are summed in another order)."""
    S, nh, nkv, dh = 100, 2, 1, 64
    qkv = torch.randn(S, (nh + 2 * nkv) * dh, device=DEV).to(torch.bfloat16 if bf16 else torch.float32)
    bad = qkv.clone()
    bad[50:, :] = float("nan")
    bad[51::2, -7:] = float("inf")
    got = []
    for x in (qkv, bad):
        out, lse = torch.empty(S, nh * dh, device=DEV, dtype=x.dtype), torch.empty(1, nh, S, device=DEV)
        print("attention later NaN", flush=True)
        B.tide_attention_fwd(1, S, nh, nkv, dh, x, out, lse, bf16, stream())
        sync()
        got.append(out[:50].float())
        assert x is qkv or bool(torch.isnan(out[50:]).all())
    assert bool(torch.isfinite(got[1]).all()) and bool(((got[0] - got[1]).abs() <= (2 ** -7 * got[0].abs() if bf16 else 0) + 1e-5).all())


@pytest.mark.parametrize("dtype,dh,bt", [("fp32", 64, 1), ("fp32", 80, 1), ("bf16", 80, 1), ("bf16", 64, 1), ("bf16", 64, 70)])
def test_no_position_reaches_a_gradient_it_has_no_part_in(B, dtype, dh, bt):
    """Causality of the backward pass where values are not finite: from a later key, value or query nothing reaches the query
    gradients of the positions before it, and from an earlier query or output gradient nothing the key and value gradients
    of the positions after it.  (70 sequences: the four-wave form of the matrix-instruction dK / dV passes.)  Other tiles than
    the clean ones sum in another order: 1e-5 of the largest value in fp32, one step of the type (2^-7) on top in bf16."""
    S, nh, nkv, dt = 100, 4, 2, torch.bfloat16 if dtype == "bf16" else torch.float32
    code, cut = int(dtype == "bf16"), 50
    g = torch.Generator(device=DEV).manual_seed(dh)
    qkv = torch.randn(S, (nh + 2 * nkv) * dh, device=DEV, generator=g).to(dt).repeat(bt, 1)
    dout = torch.randn(S, nh * dh, device=DEV, generator=g).to(dt).repeat(bt, 1)
    out, lse = torch.empty_like(dout), torch.empty(bt, nh, S, device=DEV)
    B.tide_attention_fwd(bt, S, nh, nkv, dh, qkv, out, lse, code, stream())
    sync()

    def backward(bad, what):
        q, o, do, l = (x.clone() for x in (qkv.view(bt, S, -1), out.view(bt, S, -1), dout.view(bt, S, -1), lse))
        if bad is not None:
            q[:, bad], o[:, bad], do[:, bad], l[:, :, bad] = (float("nan"),) * 4
            q[:, bad[1::2], 3:9] = float("inf")
            do[:, bad[1::2], -9:] = float("-inf")
        dqkv, delta = torch.empty_like(q), torch.empty_like(l)
        print(f"attention backward {dtype} dh={dh} batch={bt} {what}", flush=True)
        B.tide_attention_bwd(bt, S, nh, nkv, dh, q, o, do, l, delta, dqkv, code, stream())
        sync()
        return dqkv.float()

    def same(a, b):
        assert bool(torch.isfinite(a).all())
        assert bool(((a - b).abs() <= (2.0 ** -7 * b.abs() if code else 0) + 1e-5 * b.abs().max()).all())

    at, w, clean = torch.arange(S, device=DEV), nh * dh, backward(None, "clean")
    later, earlier = backward(at[cut:], "later"), backward(at[:cut], "earlier")
    same(later[:, :cut, :w], clean[:, :cut, :w])
    same(earlier[:, cut:, w:], clean[:, cut:, w:])
    assert bool(torch.isnan(later[:, cut:, :w]).all()) and bool(torch.isnan(earlier[:, :cut, w:]).all())
