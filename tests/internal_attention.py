"""The library's internal attention launchers, which a training step calls with packed sequences (device offsets) that the public calls
do not have.  Mirrors struct AttnArgs of csrc/kernels.h."""
import ctypes as C

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
_bwd = _symbol("_ZN4tide15launch_attn_bwdERKNS_8AttnArgsEP12ihipStream_t")


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
