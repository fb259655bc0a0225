"""The library's internal product launcher and its plan, which a training step calls with device-side sizes, leading dimensions
and second operand pairs that the public call does not have.  Mirrors struct GemmArgs of csrc/kernels.h."""
import ctypes as C

from paper_2602_05145_amd import binding as B

NT, NN, TN = 0, 1, 2
F32, BF16 = 0, 1


class GemmArgs(C.Structure):
    _fields_ = [("layout", C.c_int), ("M", C.c_int64), ("N", C.c_int64), ("K", C.c_int64), ("A", C.c_void_p), ("lda", C.c_int64),
                ("B", C.c_void_p), ("ldb", C.c_int64), ("A2", C.c_void_p), ("B2", C.c_void_p), ("K2", C.c_int64), ("C", C.c_void_p),
                ("ldc", C.c_int64), ("residual", C.c_void_p), ("ldr", C.c_int64), ("alpha", C.c_float), ("alpha_dev", C.c_void_p),
                ("in_dtype", C.c_int), ("out_dtype", C.c_int), ("accumulate", C.c_int), ("m_dev", C.c_void_p), ("m_off", C.c_int64),
                ("k_dev", C.c_void_p), ("k_off", C.c_int64), ("scratch", C.c_void_p), ("scratch_bytes", C.c_size_t)]


def _symbol(name, restype, argtypes):
    f = getattr(B._lib, name)
    f.restype, f.argtypes = restype, argtypes
    return f


scratch_bytes = _symbol("_ZN4tide25gemm_splitk_scratch_bytesERKNS_8GemmArgsE", C.c_size_t, [C.POINTER(GemmArgs)])
scratch_bound = _symbol("_ZN4tide25gemm_splitk_scratch_boundERKNS_8GemmArgsE", C.c_size_t, [C.POINTER(GemmArgs)])
kernel_name = _symbol("_ZN4tide16gemm_kernel_nameERKNS_8GemmArgsE", C.c_char_p, [C.POINTER(GemmArgs)])
long_rings = _symbol("_ZN4tide15gemm_long_ringsERKNS_8GemmArgsE", C.c_bool, [C.POINTER(GemmArgs)])
launch = _symbol("_ZN4tide11launch_gemmERKNS_8GemmArgsEP12ihipStream_t", C.c_int, [C.POINTER(GemmArgs), C.c_void_p])


def args(layout, M, N, K, out=BF16, K2=0, lda=None, ldb=None, ldc=None, a=256, b=256, c=256, in_dtype=BF16, **more):
    """Pointers default to an address that is only looked at for its alignment."""
    g = GemmArgs(layout=layout, M=M, N=N, K=K, A=a, B=b, C=c, K2=K2, alpha=1.0, in_dtype=in_dtype, out_dtype=out,
                 lda=lda or (M if layout == TN else K), ldb=ldb or (K if layout == NT else N), ldc=ldc or N)
    if K2:
        g.A2, g.B2 = a, b
    for k, v in more.items():
        setattr(g, k, v)
    return g
