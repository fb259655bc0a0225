"""Matrix products at the sizes where a dispatch rule or a kernel changes its form, against an fp64 product of the same
values.  Bounds: K products of fp32 rounding 2^-24 each, added in fp32 in any order, are at most K 2^-24 off the sum of
the magnitudes; the observed error grows with sqrt(K), and 2e-5 of the largest result is the bound the other product tests use
(2e-6 for fp32 operands)."""
import pytest
import torch

from tests.gpu_util import DEV, stream, sync

pytestmark = pytest.mark.gpu

DT = {"fp32": (0, torch.float32), "bf16": (1, torch.bfloat16)}


def _operands(B, layout, M, N, K, dtype, seed, pad=0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    shape_a = (K, M) if layout == B.LAYOUT_TN else (M, K)
    shape_b = (N, K) if layout == B.LAYOUT_NT else (K, N)
    a, b = (torch.randn(s, device=DEV, generator=g).to(DT[dtype][1]) for s in (shape_a, shape_b))
    ad, bd = a.double(), b.double()
    ref = (ad.t() if layout == B.LAYOUT_TN else ad) @ (bd.t().contiguous() if layout == B.LAYOUT_NT else bd)
    return a, b, ref


def _gemm(B, layout, M, N, K, a, b, c, in_dt, out_dt, alpha=1.0, residual=None, accumulate=0):
    need = B.tide_gemm_workspace_bytes(layout, M, N, K, DT[out_dt][0])
    ws = torch.full((max(need, 16),), 0xFF, dtype=torch.uint8, device=DEV)   # NaN patterns
    print(f"gemm layout={layout} M={M} N={N} K={K} {in_dt}->{out_dt} acc={accumulate} res={residual is not None} ws={need}", flush=True)
    B.tide_gemm(layout, M, N, K, alpha, a, b, c, residual, DT[in_dt][0], DT[out_dt][0], accumulate, stream(),
                workspace=ws if need else None, workspace_bytes=need)
    sync()


@pytest.fixture(scope="module")
def B():
    from paper_2602_05145_amd import binding
    return binding


@pytest.mark.parametrize("M,N,K", [(264, 520, 1), (264, 520, 31), (264, 520, 33), (136, 72, 1999), (3720, 3656, 65), (3720, 3656, 127),
                                   (4312, 4088, 2051)])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_weight_gradient_over_any_number_of_rows(B, M, N, K, accumulate):
    """TN with K (the rows of a batch) of any remainder, on the small- and the large-tile kernel, split and not split."""
    a, b, ref = _operands(B, B.LAYOUT_TN, M, N, K, "bf16", 3 * K + M)
    c = torch.full((M, N), 0.5 if accumulate else float("nan"), device=DEV)
    _gemm(B, B.LAYOUT_TN, M, N, K, a, b, c, "bf16", "fp32", accumulate=accumulate)
    ref = ref + (0.5 if accumulate else 0.0)
    assert float((c.double() - ref).abs().max()) < 2e-5 * float(ref.abs().max())


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 31, 7), (40, 100, 515), (128, 256, 4096),     # split over waves
                                   (897, 832, 37), (1000, 1001, 130),                             # tiles of 64
                                   (2048, 2060, 96), (2050, 2047, 33)])                           # tiles of 128
def test_fp32_products_at_the_edges_of_their_tiles(B, layout, M, N, K):
    """fp32 operands on the three forms of the fp32 kernel: aligned rows (16-byte loads) and odd ones, ragged tiles and K
    remainders, with residual, accumulation and alpha."""
    a, b, ref = _operands(B, layout, M, N, K, "fp32", M + K)
    g = torch.Generator(device=DEV).manual_seed(5)
    res, c0 = torch.randn(M, N, device=DEV, generator=g), torch.randn(M, N, device=DEV, generator=g)
    c = torch.full((M, N), float("nan"), device=DEV)
    _gemm(B, layout, M, N, K, a, b, c, "fp32", "fp32")
    assert float((c.double() - ref).abs().max()) < 2e-6 * max(1.0, float(ref.abs().max()))
    c = c0.clone()
    _gemm(B, layout, M, N, K, a, b, c, "fp32", "fp32", alpha=-1.5, residual=res, accumulate=1)
    want = -1.5 * ref + res.double() + c0.double()
    assert float((c.double() - want).abs().max()) < 2e-6 * max(1.0, float(want.abs().max()))
