"""The library's internal attention launchers, which a training step calls with packed sequences (device offsets) that the public calls
do not have.  Mirrors struct AttnArgs of csrc/kernels.h."""
import ctypes as C
import math

import torch

from paper_2602_05145_amd import binding as B
from tests.gpu_util import DEV, stream, sync


class AttnArgs(C.Structure):
    _fields_ = [("B", C.c_int), ("S", C.c_int), ("nh", C.c_int), ("nkv", C.c_int), ("dh", C.c_int), ("qkv", C.c_void_p), ("out", C.c_void_p),
                ("lse", C.c_void_p), ("dout", C.c_void_p), ("delta", C.c_void_p), ("dqkv", C.c_void_p), ("dtype", C.c_int), ("cu_seqlens", C.c_void_p),
                ("total_rows", C.c_int64)]


def _symbol(name):
    f = getattr(B._lib, name)
    f.restype, f.argtypes = C.c_int, [C.POINTER(AttnArgs), C.c_void_p]
    return f


_fwd = _symbol("_ZN4tide15launch_attn_fwdERKNS_8AttnArgsEP12ihipStream_t")
_form = B._lib._ZN4tide14attn_mfma_formERKNS_8AttnArgsEi
_form.restype, _form.argtypes = C.c_int, [C.POINTER(AttnArgs), C.c_int]
_bwd = _symbol("_ZN4tide15launch_attn_bwdERKNS_8AttnArgsEP12ihipStream_t")


def forms(bt, S, nh, nkv, dh, rows=0):
    """Waves (dK / dV of head size 128: pairs of waves) and sets of the forward, the dQ and the dK / dV kernel; rows: of a packed batch."""
    a = AttnArgs(B=bt, S=S, nh=nh, nkv=nkv, dh=dh, dtype=1, cu_seqlens=256 if rows else None, total_rows=rows)
    return tuple(divmod(_form(a, k), 10) for k in range(3))


def packed(qkv, dout, offsets, longest, nh, nkv, dh):
    """bf16 attention of the packed sequences [offsets[i], offsets[i + 1]), forward and backward: out, lse [nh, rows], dqkv; NaN where nothing was written."""
    rows = qkv.shape[0]
    cu = torch.tensor(offsets, dtype=torch.int32, device=DEV)
    out, dqkv = torch.full_like(dout, float("nan")), torch.full_like(qkv, float("nan"))
    lse, delta = (torch.full((nh, rows), float("nan"), device=DEV) for _ in range(2))
    a = AttnArgs(B=len(offsets) - 1, S=longest, nh=nh, nkv=nkv, dh=dh, qkv=qkv.data_ptr(), out=out.data_ptr(), lse=lse.data_ptr(), dout=dout.data_ptr(),
                 delta=delta.data_ptr(), dqkv=dqkv.data_ptr(), dtype=1, cu_seqlens=cu.data_ptr(), total_rows=rows)
    for launch in (_fwd, _bwd):
        assert launch(a, stream()) == 0
        sync()
    return out, lse, dqkv


U = 2.0 ** -8   # the most that a value moves when it is rounded to bf16, relative to it


def reference(qkv, dout, nh, nkv, dh):
    """Attention of one sequence in fp64: out, lse [nh, S], dqkv; and how far each of their rows of one head may be from it ([S, heads of out | of dqkv]).
    A kernel rounds its results once, by U of each at most.  Before that it rounds probabilities and score gradients, by p = U of each at head
    size 128 and in two parts, U U, at 64; and it takes delta from the rounded outputs.  These roundings are in random directions: the squares
    of their products with the other operand add up, and the root of that is over twice what a row shows (a rounding is 0.41 U in the mean).  Delta is one
    number for a whole row, which no channel averages: twice as much, i.e. nearly five times its mean."""
    n, g, scale = qkv.shape[0], nh // nkv, 1.0 / math.sqrt(dh)
    p = U if dh == 128 else U * U
    x, do = qkv.double().cpu().view(n, nh + 2 * nkv, dh).transpose(0, 1), dout.double().cpu().view(n, nh, dh).transpose(0, 1)
    q, (k, v) = x[:nh], (t.repeat_interleave(g, 0) for t in (x[nh:nh + nkv], x[nh + nkv:]))
    s = (q @ k.transpose(1, 2) * scale).masked_fill(torch.ones(n, n, dtype=torch.bool).triu(1), -math.inf)
    lse = torch.logsumexp(s, -1)
    w = torch.exp(s - lse[..., None])
    o = w @ v
    ds = w * (do @ v.transpose(1, 2) - (do * o).sum(-1, keepdim=True))
    ddelta2 = (2 * U * do * o).square().sum(-1, keepdim=True)     # of delta, squared
    heads = lambda t: t.view(nkv, g, n, dh).sum(1)  # noqa: E731
    wt, dst = w.transpose(1, 2), ds.transpose(1, 2)
    dq, dk, dv = scale * (ds @ k), heads(scale * (dst @ q)), heads(wt @ do)
    off = dict(o=(U * o).square() + p * p * (w.square() @ v.square()), dv=(U * dv).square() + heads(p * p * (wt.square() @ do.square())),
               dq=(U * dq).square() + scale ** 2 * (p * p * (ds.square() @ k.square()) + ddelta2 * (w @ k).square()),
               dk=(U * dk).square() + heads(scale ** 2 * (p * p * (dst.square() @ q.square()) + (wt.square() @ (ddelta2 * q.square())))))
    rows = lambda *ts: torch.cat([t.transpose(0, 1) for t in ts], 1)  # noqa: E731
    bound = lambda *ts: torch.sqrt(rows(*ts).sum(-1)) + 1e-6 * max(float(t.abs().max()) for t in (o, dq, dk, dv))  # noqa: E731  (fp32 sums)
    return (rows(o).reshape(n, -1), lse, rows(dq, dk, dv).reshape(n, -1)), (bound(off["o"]), bound(off["dq"], off["dk"], off["dv"]))


def worst_row(got, want, bound):
    """The largest error of a row of one head, in its bound (NaN counts as infinite)."""
    n, h = bound.shape
    e = (got.double().cpu() - want).view(n, h, -1).norm(dim=-1) / bound
    return float(torch.where(torch.isnan(e), torch.full_like(e, math.inf), e).max())


def relative(got, want):
    return float((got.double().cpu() - want).norm() / want.norm())


def check(got, nh, nkv, dh, ref=None, qkv=None, dout=None):
    """out, lse and dqkv of one sequence, every row of every head and all of them together."""
    (out, lse, dqkv), ((ro, rl, rg), (bo, bg)) = got, ref or reference(qkv, dout, nh, nkv, dh)
    assert worst_row(out, ro, bo) < 1.0, ("out", worst_row(out, ro, bo))
    assert float((lse.double().cpu() - rl).abs().max()) < 1e-5 * max(1.0, float(rl.abs().max()))
    parts = dict(dq=(0, nh), dk=(nh, nh + nkv), dv=(nh + nkv, nh + 2 * nkv))
    for name, (a, b) in parts.items():
        w = worst_row(dqkv[:, a * dh:b * dh], rg[:, a * dh:b * dh], bg[:, a:b])
        assert w < 1.0, (name, w)
    for name, e in dict(out=relative(out, ro), **{k: relative(dqkv[:, a * dh:b * dh], rg[:, a * dh:b * dh]) for k, (a, b) in parts.items()}).items():
        assert ro.shape[0] < 64 or e < MOST[dh][name], (name, e)


# Root mean square over all rows of 64 positions or more, relative: one rounding to bf16 is 1.5e-3 to 1.7e-3, by where the values lie in their octaves.  Emulated for
# the cases below, out / dq, dk / dv: 1.60e-3 / 1.95e-3 / 1.72e-3 at most with probabilities and score gradients in two parts, in one 1.85e-3 to 1.99e-3 / 2.43e-3 to 2.73e-3 /
# 2.19e-3 to 2.36e-3: the lines for head size 64 are between.
MOST = {64: dict(out=1.72e-3, dq=2.2e-3, dk=2.2e-3, dv=1.95e-3), 128: dict(out=2.2e-3, dq=3e-3, dk=3e-3, dv=2.6e-3)}

# batch, positions, heads, kv heads: items of a block from several heads and query blocks (groups of 3, 5 and 7 heads), steps that the sets share unevenly, one step fewer than sets
EDGES = [(1, 97, 3, 1), (1, 161, 5, 1), (3, 225, 7, 1), (1, 321, 10, 2), (2, 650, 20, 4), (9, 640, 8, 2), (40, 33, 6, 2), (33, 70, 4, 4), (66, 257, 2, 2), (260, 65, 10, 1), (100, 129, 8, 4), (4, 900, 16, 4)]
# dK / dV at head size 128: pairs of waves in two sets of one pair, of two pairs and in one set; the last keys with fewer tiles than sets, a pair without keys.  (From 32 positions on: over one, gradients of queries and keys are zero, and
# over a few they are the rest of a cancellation against delta.)
PAIRS = [(1, 32, 8, 1), (1, 33, 8, 1), (1, 257, 2, 2), (1, 288, 2, 2), (33, 270, 4, 2), (33, 289, 4, 2), (130, 65, 10, 1), (66, 257, 2, 2), (200, 96, 3, 1), (16, 289, 8, 4), (14, 270, 8, 4)]

# head size, heads, kv heads, lengths of packed sequences; waves and sets of the forward, the dQ and the dK / dV kernel that such a batch takes
_FEW, _MANY = [1, 31, 32, 33, 95, 250, 64, 7], [1, 31, 33, 65, 129, 0, 64, 97]
_RAGGED = [201, 1075, 261, 118, 13, 38, 293]
PACKED = [(128, 32, 8, _RAGGED, ((4, 1), (2, 2), (2, 2))), (128, 24, 8, _RAGGED, ((4, 2), (2, 2), (2, 2))), (128, 16, 4, _RAGGED, ((2, 2), (2, 2), (1, 2))),
          (128, 16, 4, _MANY * 22, ((4, 1), (4, 1), (2, 1))), (64, 6, 2, _FEW, ((2, 2), (2, 4), (2, 4))), (64, 16, 4, _MANY * 22, ((4, 1), (4, 1), (2, 1))),
          (64, 32, 8, [201, 700, 261, 118, 13, 38, 293, 1, 33], ((2, 2), (2, 2), (2, 4))), (64, 16, 8, _MANY * 5 + [400], ((4, 1), (2, 2), (2, 2))),
          (128, 3, 3, _FEW + [0] * 30, ((2, 2), (2, 2), (1, 2))), (64, 20, 10, [0] * 9 + [517] + [0] * 8, ((2, 2), (2, 4), (2, 4)))]


def inputs(S, nh, nkv, dh, seed, device=DEV):
    g = torch.Generator(device=device).manual_seed(seed)
    return (torch.randn(S, (nh + 2 * nkv) * dh, device=device, generator=g).bfloat16(), torch.randn(S, nh * dh, device=device, generator=g).bfloat16())
