"""The bounds that the tests of the attention kernels hold them to, on the host: an emulation of the kernels' roundings is inside them, and a row that is
missing, 2 % off, or made from probabilities in one bf16 value where two are due is not.  And which forms of the kernels those tests run."""
import math

import pytest
import torch

from tests import internal_attention as ia


def _round(x):
    return x.float().bfloat16().double()


def _emulated(qkv, dout, nh, nkv, dh, parts):
    """fp64, with values rounded where the kernels round them; parts: bf16 values that hold a probability or a score gradient."""
    n, g, scale = qkv.shape[0], nh // nkv, 1.0 / math.sqrt(dh)
    held = _round if parts == 1 else lambda t: _round(t) + _round(t - _round(t))
    x, do = qkv.double().view(n, nh + 2 * nkv, dh).transpose(0, 1), dout.double().view(n, nh, dh).transpose(0, 1)
    q, k, v = x[:nh], x[nh:nh + nkv].repeat_interleave(g, 0), x[nh + nkv:].repeat_interleave(g, 0)
    s = (q @ k.transpose(1, 2) * scale).masked_fill(torch.ones(n, n, dtype=torch.bool).triu(1), -math.inf)
    lse, w = torch.logsumexp(s, -1), torch.exp(s - s.max(-1, keepdim=True)[0])
    o = _round((held(w) @ v) / w.sum(-1, keepdim=True))
    w = torch.exp(s - lse[..., None])
    ds = held(w * (do @ v.transpose(1, 2) - (do * o).sum(-1, keepdim=True)))
    heads = lambda t: t.view(nkv, g, n, dh).sum(1)  # noqa: E731
    grads = (scale * (ds @ k), heads(scale * (ds.transpose(1, 2) @ q)), heads(held(w).transpose(1, 2) @ do))
    rows = lambda *ts: torch.cat([t.transpose(0, 1) for t in ts], 1).reshape(n, -1)  # noqa: E731
    return rows(o), lse, rows(*(_round(t) for t in grads))


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("bt,S,nh,nkv", [s for s in ia.EDGES + ia.PAIRS if s[1] * s[2] < 5000])
def test_bounds_of_a_row(dh, bt, S, nh, nkv):
    qkv, dout = ia.inputs(S, nh, nkv, dh, S + nh + dh, "cpu")
    ref = ia.reference(qkv, dout, nh, nkv, dh)
    out, lse, dqkv = _emulated(qkv, dout, nh, nkv, dh, 2 if dh == 64 else 1)
    ia.check((out, lse, dqkv), nh, nkv, dh, ref)

    def refused(o, d):
        with pytest.raises(AssertionError):
            ia.check((o, lse, d), nh, nkv, dh, ref)
    w, k = nh * dh, nkv * dh
    for part in (slice(0, w), slice(w, w + k), slice(w + k, None)):   # dq, dk, dv of the last position
        for factor in (0.0, 1.02):
            bad = dqkv.clone()
            bad[-1, part] *= factor
            refused(out, bad)
    for factor in (0.0, 1.02):
        bad = out.clone()
        bad[-1] *= factor
        refused(bad, dqkv)
    if dh == 64 and S >= 64:
        one = _emulated(qkv, dout, nh, nkv, dh, 1)
        refused(one[0], dqkv)
        for part in (slice(0, w), slice(w, w + k), slice(w + k, None)):
            bad = dqkv.clone()
            bad[:, part] = one[2][:, part]
            refused(out, bad)


def test_every_form_is_among_the_cases():
    want = {64: ({(2, 2), (4, 1)}, {(2, 4), (2, 2), (4, 1)}, {(2, 4), (2, 2), (2, 1)}),
            128: ({(2, 2), (4, 2), (4, 1)}, {(2, 2), (4, 1)}, {(1, 2), (2, 2), (2, 1)})}
    for dh, sets in want.items():
        for k in range(3):
            assert {ia.forms(bt, S, nh, nkv, dh)[k] for bt, S, nh, nkv in ia.EDGES + (ia.PAIRS if dh == 128 else [])} == sets[k], (dh, k)
            assert {form[k] for d, *_, form in ia.PACKED if d == dh} == sets[k], (dh, k)
    for dh, nh, nkv, lens, form in ia.PACKED:
        assert ia.forms(len(lens), max(lens), nh, nkv, dh, sum(lens)) == form, (dh, nh, nkv, ia.forms(len(lens), max(lens), nh, nkv, dh, sum(lens)))
