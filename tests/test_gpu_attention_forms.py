"""The forms of the bf16 attention kernels: blocks of four waves that walk every key, and sets of waves that share the keys (forward, dQ) or
the queries (dK / dV) where blocks are few.  Each against fp64 at the edges of its items (32 queries of one head, several heads side by side)
and of its steps; and one sequence alone against the same sequence as one of many."""
import pytest
import torch

from tests import internal_attention as ia
from tests.gpu_util import DEV, stream, sync
from tests.test_gpu_attention_heads import _reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2602_05145_amd import binding
    return binding


def _run(B, qkv, dout, bt, S, nh, nkv, dh):
    out, dqkv = torch.full_like(dout, float("nan")), torch.full_like(qkv, float("nan"))
    lse, delta = (torch.full((bt, nh, S), float("nan"), device=DEV) for _ in range(2))
    print(f"attention forms batch={bt} S={S} heads={nh}/{nkv} dh={dh}", flush=True)
    B.tide_attention_fwd(bt, S, nh, nkv, dh, qkv, out, lse, 1, stream())
    sync()
    B.tide_attention_bwd(bt, S, nh, nkv, dh, qkv, out, dout, lse, delta, dqkv, 1, stream())
    sync()
    return out, lse, dqkv


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("bt,S,nh,nkv", ia.EDGES)
def test_every_form_at_its_edges(B, dh, bt, S, nh, nkv):
    qkv, dout = ia.inputs(S, nh, nkv, dh, S + nh + dh)
    out, lse, dqkv = _run(B, qkv.repeat(bt, 1), dout.repeat(bt, 1), bt, S, nh, nkv, dh)
    for x, shape in ((out, (bt, S, -1)), (lse, (bt, nh, S)), (dqkv, (bt, S, -1))):   # every sequence of the batch the same bits
        assert float((x.view(*shape) - x.view(*shape)[:1]).abs().max()) == 0.0
    ia.check((out[:S], lse[0], dqkv[:S]), nh, nkv, dh, qkv=qkv, dout=dout)


@pytest.mark.parametrize("bt,S,nh,nkv", ia.PAIRS)
def test_pairs_of_waves_at_their_edges(B, bt, S, nh, nkv):
    test_every_form_at_its_edges(B, 128, bt, S, nh, nkv)


@pytest.mark.parametrize("dh", [64, 128])
def test_sets_and_single_waves_agree(B, dh):
    """A sequence alone takes the sets, as one of 90 the four-wave blocks: the same results but for the order of the fp32 sums and what the
    running maximum was when a probability was rounded (one step of bf16, 2^-7 of the largest value, at most)."""
    S, nh, nkv = 420, 8, 2
    g = torch.Generator(device=DEV).manual_seed(dh)
    qkv = torch.randn(S, (nh + 2 * nkv) * dh, device=DEV, generator=g).bfloat16()
    dout = torch.randn(S, nh * dh, device=DEV, generator=g).bfloat16()
    one = _run(B, qkv, dout, 1, S, nh, nkv, dh)
    many = _run(B, qkv.repeat(90, 1), dout.repeat(90, 1), 90, S, nh, nkv, dh)
    for a, b, n in zip(one, many, (S, 1, S)):
        a, b = a.double(), b[:n].double()
        assert float((a - b).abs().max()) < 2.0 ** -7 * float(b.abs().max())
    ref = ia.reference(qkv, dout, nh, nkv, dh)   # and of every row each within its own bound
    ia.check((one[0], one[1][0], one[2]), nh, nkv, dh, ref)
    ia.check((many[0][:S], many[1][0], many[2][:S]), nh, nkv, dh, ref)


def test_later_positions_reach_nothing_before_them_across_sets(B):
    """As for one set: NaN from position 200 on leave the outputs of the rows before it as they are up to a step of the type, also where
    the sets' sums are merged (head size 64)."""
    S, nh, nkv, dh, cut = 333, 4, 2, 64, 200
    g = torch.Generator(device=DEV).manual_seed(1)
    qkv = torch.randn(S, (nh + 2 * nkv) * dh, device=DEV, generator=g).bfloat16()
    dout = torch.randn(S, nh * dh, device=DEV, generator=g).bfloat16()
    bad = qkv.clone()
    bad[cut:] = float("nan")
    bad[cut + 1::2, -7:] = float("inf")
    clean, got = _run(B, qkv, dout, 1, S, nh, nkv, dh), _run(B, bad, dout, 1, S, nh, nkv, dh)
    assert bool(torch.isnan(got[0][cut:]).all())
    for a, b in ((got[0][:cut].float(), clean[0][:cut].float()), (got[2][:cut, :nh * dh].float(), clean[2][:cut, :nh * dh].float())):
        assert bool(torch.isfinite(a).all()) and bool(((a - b).abs() <= 2.0 ** -7 * b.abs() + 1e-5 * b.abs().max()).all())


@pytest.mark.parametrize("dh,nh,nkv,lens,form", ia.PACKED)
def test_packed_sequences_in_every_form(B, dh, nh, nkv, lens, form):
    """Sequences shorter than the launch's longest, empty ones, blocks without rows, sets with fewer steps than others, and heads that keep all XCDs busy (8) or not: each
    sequence as it is by itself in fp64."""
    qkv, dout = ia.inputs(sum(lens), nh, nkv, dh, sum(lens) + nh + dh)
    offsets = [0]
    for n in lens:
        offsets.append(offsets[-1] + n)
    print(f"packed attention of {len(lens)} sequences heads={nh}/{nkv} dh={dh} {form}", flush=True)
    assert ia.forms(len(lens), max(lens), nh, nkv, dh, sum(lens)) == form
    out, lse, dqkv = ia.packed(qkv, dout, offsets, max(lens), nh, nkv, dh)
    for i, (a, b) in enumerate(zip(offsets, offsets[1:])):
        if b > a and (i < 24 or i % 7 == 0):
            ia.check((out[a:b], lse[:, a:b], dqkv[a:b]), nh, nkv, dh, qkv=qkv[a:b], dout=dout[a:b])
    assert bool(torch.isfinite(out).all()) and bool(torch.isfinite(dqkv).all())


@pytest.mark.parametrize("dh,nh,nkv", [(64, 10, 2), (128, 6, 2)])
def test_packed_lengths_in_a_training_step(B, dh, nh, nkv):
    """Sequences of many lengths, from one row to several items, with groups of five and three heads, against the oracle."""
    from paper_2602_05145_amd import runtime, workloads as W
    import numpy as np
    lens = [1, 31, 32, 33, 95, 250, 64, 7]
    T = sum(lens)
    cfg = W.get_config("small", batch=1, seq=T, target_hidden=256, hidden=nh * dh, n_heads=nh, n_kv_heads=nkv, head_dim=dh, ffn=512, vocab=1024, mask="none", seed=5)
    wl = W.make_workload(cfg)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    tr = runtime.trainer_from_workload(cfg, wl)
    tr.set_packed(cu)
    print(f"packed forms dh={dh}", flush=True)
    tr.train_step_packed(cfg["lr"])
    sync()
    from oracle import tide_oracle as O
    p0 = {k: np.asarray(v, np.float64) for k, v in wl["params"].items()}
    loss, grads = O.train_quantities_packed(cfg, p0, wl["hidden"].astype(np.float64), wl["tokens"], wl["mask"], cu)[:2]
    assert abs(float(tr.loss.item()) - loss) < 1e-2 * abs(loss)
    for k, ref in grads.items():
        a, b = tr.host(tr.grads)[k].reshape(-1), ref.reshape(-1)
        assert a @ b / (np.linalg.norm(a) * np.linalg.norm(b)) > 0.999, k


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("bt,S,nh,nkv", [(1, 160, 2, 2), (1, 700, 8, 2), (80, 160, 8, 2)])
def test_a_first_step_whose_scores_are_all_minus_infinity(B, dh, bt, S, nh, nkv):
    """The products of the queries with the first 32 keys overflow to -inf: those keys weigh nothing with the queries that see others too, in
    the blocks of four waves as in the sets."""
    g = torch.Generator(device=DEV).manual_seed(3)
    qkv = torch.randn(S, (nh + 2 * nkv) * dh, device=DEV, generator=g).bfloat16()
    heads = qkv.view(S, nh + 2 * nkv, dh)
    heads[:, :nh, 0], heads[:, nh:nh + nkv, 0], heads[:32, nh:nh + nkv, 0] = 1e20, 0.0, -3e38
    dout = torch.randn(S, nh * dh, device=DEV, generator=g).bfloat16()
    out, lse, dqkv = _run(B, qkv.repeat(bt, 1), dout.repeat(bt, 1), bt, S, nh, nkv, dh)
    ro, rl, rg = (x[..., 32:] if x.shape == (nh, S) else x[32:] for x in _reference(qkv, dout, S, nh, nkv, dh))
    w = nh * dh
    for got, want, tol in ((out[32:S], ro, 1e-2), (lse[0, :, 32:], rl, 1e-5), (dqkv[32:S, :w], rg[:, :w], 1e-2)):   # as in the tests above
        assert float((got.double().cpu() - want).abs().max()) < tol * float(want.abs().max())


@pytest.mark.parametrize("dh", [64, 128])
def test_a_packed_batch_of_more_blocks_than_a_launch_has(B, dh):
    """The most sequences that a call takes, nearly all of them empty, and a longest length of 16384: 2^32 threads by their bounds in the forward pass,
    twice that for dK / dV at head size 128.  The three that have rows as by themselves (sums in another order, see above)."""
    nh, nkv, rows, longest = 2, 2, 1200, 16384
    g = torch.Generator(device=DEV).manual_seed(dh)
    qkv = torch.randn(rows, (nh + 2 * nkv) * dh, device=DEV, generator=g).bfloat16()
    dout = torch.randn(rows, nh * dh, device=DEV, generator=g).bfloat16()
    ends, offsets = {7: 300, 40000: 1123, 65535: 1200}, [0]
    for i in range(1, 65536):
        offsets.append(ends.get(i, offsets[-1]))
    print(f"packed batch of {len(offsets) - 1} sequences dh={dh}", flush=True)
    many, few = ia.packed(qkv, dout, offsets, longest, nh, nkv, dh), ia.packed(qkv, dout, [0, 300, 1123, 1200], 823, nh, nkv, dh)
    for a, b in zip(many, few):
        assert float((a.double() - b.double()).abs().max()) < 2.0 ** -7 * float(b.double().abs().max())
