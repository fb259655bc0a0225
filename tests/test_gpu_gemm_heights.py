"""Tiles of 128 to 224 rows x 256 columns: the smallest ragged products that the plan gives to each of them, against a float
reference of the same bf16 operands."""
import pytest
import torch

from tests import internal_gemm as ig
from tests.internal_gemm import kernel_name

# layout, M, N, K: a last tile row and column that are partly filled, one slab or (TN) one and a remainder
CASES = [(ig.NT, 521, 6608, 64, 128), (ig.NT, 7405, 1040, 64, 160), (ig.NT, 5830, 1544, 64, 192), (ig.NT, 7037, 1544, 64, 224),
         (ig.NN, 530, 6736, 64, 128), (ig.NN, 6542, 1176, 64, 160), (ig.NN, 6831, 1288, 64, 192), (ig.NN, 8151, 1296, 64, 224),
         (ig.TN, 5456, 656, 65, 128), (ig.TN, 1048, 7192, 65, 160), (ig.TN, 1288, 7240, 301, 192), (ig.TN, 2192, 5392, 515, 224),
         (ig.NN, 1665, 5632, 2048, 160), (ig.NT, 2040, 4096, 576, 128), (ig.TN, 5632, 2048, 1333, 192)]


@pytest.mark.parametrize("layout,M,N,K,height", CASES)
def test_the_plan_takes_the_height(layout, M, N, K, height):
    got = kernel_name(ig.args(layout, M, N, K, out=ig.F32 if layout == ig.TN else ig.BF16)).decode()
    assert got.startswith(f"gemm_mfma_{('nt', 'nn', 'tn')[layout]}_{height}x256_"), got


def test_heights_between_the_squares_are_kept_from_what_they_do_not_serve():
    ragged = [ig.args(ig.NT, 521, 6608, 72), ig.args(ig.NN, 6831, 1288, 8), ig.args(ig.NT, 521, 6608, 64, K2=72), ig.args(ig.NT, 521, 6608, 64, k_dev=256),
              ig.args(ig.NT, 521, 6608, 64, out=ig.F32), ig.args(ig.TN, 5456, 656, 65, out=ig.BF16),
              ig.args(ig.NT, 521, 6608, 64, accumulate=1)]
    for g in ragged:
        assert b"x256" not in kernel_name(g)


def planned(layout, M, N, K, **more):
    """The kernel of a product that is given the scratch it asks for."""
    g = ig.args(layout, M, N, K, out=ig.F32 if layout == ig.TN else ig.BF16, **more)
    g.scratch, g.scratch_bytes = 256, ig.scratch_bytes(g)
    return kernel_name(g).decode()


@pytest.mark.parametrize("layout,M,N,K", [(ig.NT, 39, 32000, 6144), (ig.NN, 25, 32000, 5632), (ig.NT, 103, 32000, 6144), (ig.NN, 157, 32000, 25600),
                                          (ig.NT, 160, 32000, 14336), (ig.NT, 688, 5120, 5632), (ig.NT, 3887, 1024, 5632)])
def test_a_split_is_kept_where_it_is_faster(layout, M, N, K):
    """One row of 125 tiles that streams its operand from memory on half the CUs; small tiles whose split is nearly as cheap by the model."""
    assert "x256" not in planned(layout, M, N, K)


@pytest.mark.parametrize("layout,M,N,K,height", [(ig.NT, 127, 50304, 14336, 128), (ig.NT, 76, 128256, 2048, 128), (ig.NN, 140, 25600, 4096, 160),
                                                 (ig.NT, 1283, 5120, 12288, 128), (ig.TN, 1024, 5120, 6041, 128)])
def test_a_split_gives_way_where_a_height_is_faster(layout, M, N, K, height):
    assert f"_{height}x256_" in planned(layout, M, N, K)


@pytest.mark.parametrize("M", [4096, 3999])
def test_a_height_pays_over_the_row_counts_that_a_bound_stands_for(M):
    """Gate product of a padded batch: 60 % of the rows just fill a round of squares, 62 % no round of 224 x 256 tiles, though 60, 85 and 100 % do."""
    assert planned(ig.NT, M, 5632, 2048, m_dev=256) == "gemm_mfma_nt_256_bf16out"


@pytest.mark.gpu
@pytest.mark.parametrize("layout,M,N,K,height", CASES)
def test_products_of_every_height(layout, M, N, K, height):
    """With a residual and old values where the layout of the step has them.  bf16 results: one rounding, half a step of 8 significant bits
    (up to 2^-8 of the value), plus that of the sums (below 1e-6 of their scale); float results: the sums' own, K eps at most."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    sh = {ig.NT: ((M, K), (N, K)), ig.NN: ((M, K), (K, N)), ig.TN: ((K, M), (K, N))}[layout]
    a, b = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in sh)
    f32 = layout == ig.TN
    ref = {ig.NT: lambda: a.double() @ b.double().t(), ig.NN: lambda: a.double() @ b.double(), ig.TN: lambda: a.double().t() @ b.double()}[layout]()
    extra = torch.randn(M, N, device="cuda", generator=g).to(torch.float32 if f32 else torch.bfloat16)
    for add in (0, 1):
        c = extra.clone() if f32 and add else torch.full((M, N), float("nan"), device="cuda", dtype=extra.dtype)
        args = ig.args(layout, M, N, K, out=ig.F32 if f32 else ig.BF16, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr(), accumulate=add if f32 else 0)
        if add and not f32:
            args.residual, args.ldr = extra.data_ptr(), N
        assert b"x256" in kernel_name(args)
        print("height", height, layout, M, N, K, "add", add, flush=True)
        assert ig.launch(args, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        want = ref + extra.double() if add else ref
        err = (c.double() - want).abs()
        bound = 2e-6 * K ** 0.5 * 4 + (0 if f32 else want.abs() * 2.0 ** -8)
        assert bool((err <= bound).all()), float((err - bound).max())


# numbers of slabs that end in every phase of the ring of three and two units and of its loop of six; TN has one row in the last slab
RING = [(ig.NT, 397, 8248, 128), (ig.NT, 1029, 7224, 160), (ig.NT, 8240, 1032, 192), (ig.NT, 8077, 1296, 224),
        (ig.NN, 385, 8480, 128), (ig.NN, 1038, 7192, 160), (ig.NN, 8305, 1032, 192), (ig.NN, 8148, 1296, 224),
        (ig.TN, 8272, 392, 128), (ig.TN, 7176, 1032, 160), (ig.TN, 8408, 1032, 192), (ig.TN, 8200, 1416, 224)]


def _depths(layout):
    return [64 * slabs - 63 for slabs in range(9, 15)] if layout == ig.TN else [64 * slabs for slabs in range(7, 13)]


def _run(g):
    assert ig.launch(g, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


def _bound(K, want, bf16):
    return 2e-6 * K ** 0.5 * 4 + (want.abs() * 2.0 ** -8 if bf16 else 0)     # as above


@pytest.mark.gpu
@pytest.mark.parametrize("layout,M,N,height,K", [(*x, k) for x in RING for k in _depths(x[0])])
def test_every_phase_of_the_ring(layout, M, N, height, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    sh = {ig.NT: ((M, K), (N, K)), ig.NN: ((M, K), (K, N)), ig.TN: ((K, M), (K, N))}[layout]
    a, b = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in sh)
    f32 = layout == ig.TN
    c = torch.full((M, N), float("nan"), device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
    args = ig.args(layout, M, N, K, out=ig.F32 if f32 else ig.BF16, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr())
    assert f"_{height}x256_" in kernel_name(args).decode()
    print("ring", height, layout, M, N, K, flush=True)
    _run(args)
    ad, bd = a.double(), b.double()
    want = (ad.t() if f32 else ad) @ (bd.t() if layout == ig.NT else bd)
    assert bool(((c.double() - want).abs() <= _bound(K, want, not f32)).all())


ROWS = [(ig.NT, 705, 8256, 128), (ig.NT, 1026, 7200, 160), (ig.NT, 5809, 1560, 192), (ig.NT, 1371, 8216, 224),
        (ig.NN, 707, 8432, 128), (ig.NN, 1044, 7272, 160), (ig.NN, 5140, 1800, 192), (ig.NN, 3668, 3104, 224)]


@pytest.mark.gpu
@pytest.mark.parametrize("layout,M,N,height", ROWS)
def test_a_number_of_rows_known_on_the_device(layout, M, N, height):
    """None, one, up to inside a tile, the bound and beyond it, less an offset; the rows from there on stay as they are."""
    K, off = 448, 5
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, b = torch.randn(M, K, device="cuda", generator=g).bfloat16(), torch.randn((N, K) if layout == ig.NT else (K, N), device="cuda", generator=g).bfloat16()
    res = torch.randn(M, N, device="cuda", generator=g).bfloat16()
    product = a.double() @ (b.double().t() if layout == ig.NT else b.double())
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    for rows, r in ((0, None), (1, None), (height + 37, None), (height + 37, res), (M - 1, None), (M, res), (M + 9, None), (-3, None)):
        c = torch.full((M, N), 7.0, device="cuda", dtype=torch.bfloat16)
        cnt.fill_(rows + off)
        args = ig.args(layout, M, N, K, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr(), m_dev=cnt.data_ptr(), m_off=off)
        if r is not None:
            args.residual, args.ldr = r.data_ptr(), N
        assert f"_{height}x256_" in kernel_name(args).decode()
        print("rows on the device", height, layout, M, N, rows, r is not None, flush=True)
        _run(args)
        n = max(0, min(M, rows))
        want = product[:n] + (0 if r is None else r[:n].double())
        assert bool(((c[:n].double() - want).abs() <= _bound(K, want, True)).all())
        assert bool((c[n:] == 7.0).all())


PAIRS = [(ig.NT, 389, 8240, 128), (ig.NT, 1159, 6416, 160), (ig.NT, 5870, 1560, 192), (ig.NT, 1734, 6448, 224),
         (ig.NN, 386, 8344, 128), (ig.NN, 899, 8200, 160), (ig.NN, 5863, 1544, 192), (ig.NN, 5428, 2056, 224)]


@pytest.mark.gpu
@pytest.mark.parametrize("K,K2", [(448, 192), (192, 448), (64, 448)])
@pytest.mark.parametrize("layout,M,N,height", PAIRS)
def test_a_second_operand_pair(layout, M, N, height, K, K2):
    """Pairs of unequal depth, whose seam falls into another phase of the ring each time."""
    lda, g = max(K, K2), torch.Generator(device="cuda").manual_seed(M + N + K)
    a, a2 = (torch.randn(M, lda, device="cuda", generator=g).bfloat16() for _ in range(2))
    b, b2 = (torch.randn((N, lda) if layout == ig.NT else (k, N), device="cuda", generator=g).bfloat16() for k in (K, K2))
    c = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
    args = ig.args(layout, M, N, K, K2=K2, lda=lda, ldb=lda if layout == ig.NT else N, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr())
    args.A2, args.B2 = a2.data_ptr(), b2.data_ptr()
    assert f"_{height}x256_" in kernel_name(args).decode()
    print("pairs", height, layout, M, N, K, K2, flush=True)
    _run(args)
    want = sum(x[:, :k].double() @ (y[:, :k].double().t() if layout == ig.NT else y.double()) for x, y, k in ((a, b, K), (a2, b2, K2)))
    assert bool(((c.double() - want).abs() <= _bound(K + K2, want, True)).all())


def test_the_cases_above_are_what_they_say():
    for layout, M, N, height in RING:
        for K in _depths(layout):
            g = ig.args(layout, M, N, K, out=ig.F32 if layout == ig.TN else ig.BF16)
            assert f"_{height}x256_" in kernel_name(g).decode(), (layout, M, N, K, kernel_name(g))
    for layout, M, N, height in ROWS:
        assert f"_{height}x256_" in kernel_name(ig.args(layout, M, N, 448, m_dev=256)).decode(), (layout, M, N)
    for layout, M, N, height in PAIRS:
        for k, k2 in ((448, 192), (192, 448), (64, 448)):
            g = ig.args(layout, M, N, k, K2=k2, lda=max(k, k2), ldb=max(k, k2) if layout == ig.NT else N)
            assert f"_{height}x256_" in kernel_name(g).decode(), (layout, M, N, k, k2, kernel_name(g))


# Squares of 128 on at most 224 CUs, 16 slabs or more: rings of five units for either operand.  Numbers of slabs in every phase of them, whole and with
# a remainder of 8 (TN: 1); a depth on the device of no, one and a few slabs; a seam between operand pairs in every phase.
@pytest.mark.gpu
@pytest.mark.parametrize("layout", [ig.NT, ig.NN, ig.TN])
@pytest.mark.parametrize("slabs", range(16, 21))
def test_every_phase_of_the_long_rings(layout, slabs):
    M, N = (264, 264)
    g = torch.Generator(device="cuda").manual_seed(slabs)
    for K in (64 * slabs, 64 * slabs - (63 if layout == ig.TN else 56)):
        sh = {ig.NT: ((M, K), (N, K)), ig.NN: ((M, K), (K, N)), ig.TN: ((K, M), (K, N))}[layout]
        a, b = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in sh)
        ad, bd = a.double(), b.double()
        for out in (ig.F32, ig.BF16):
            for k in (None, 0, 1, 200, K - 1) if layout == ig.TN else (None,):
                c = torch.full((M, N), float("nan"), device="cuda", dtype=torch.float32 if out == ig.F32 else torch.bfloat16)
                args = ig.args(layout, M, N, K, out=out, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr())
                cnt = torch.tensor([k or 0], dtype=torch.int32, device="cuda")
                if k is not None:
                    args.k_dev = cnt.data_ptr()
                assert ig.long_rings(args) and "_128_" in kernel_name(args).decode()
                print("long rings", layout, K, out, k, flush=True)
                _run(args)
                n = K if k is None else k
                want = ad[:n].t() @ bd[:n] if layout == ig.TN else ad @ (bd.t() if layout == ig.NT else bd)
                assert bool(((c.double() - want).abs() <= _bound(K, want, out == ig.BF16)).all())


@pytest.mark.gpu
@pytest.mark.parametrize("layout", [ig.NT, ig.NN])
@pytest.mark.parametrize("K,K2", [(64, 1216), (640, 576), (704, 512), (832, 640), (960, 320), (1032, 200)])
def test_a_second_operand_pair_on_the_long_rings(layout, K, K2):
    M, N, rows, lda, g = 300, 264, 141, max(K, K2), torch.Generator(device="cuda").manual_seed(K)
    a, a2 = (torch.randn(M, lda, device="cuda", generator=g).bfloat16() for _ in range(2))
    b, b2 = (torch.randn((N, lda) if layout == ig.NT else (k, N), device="cuda", generator=g).bfloat16() for k in (K, K2))
    c = torch.full((M, N), 7.0, device="cuda", dtype=torch.bfloat16)
    cnt = torch.tensor([rows], dtype=torch.int32, device="cuda")
    args = ig.args(layout, M, N, K, K2=K2, lda=lda, ldb=lda if layout == ig.NT else N, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr(), m_dev=cnt.data_ptr())
    args.A2, args.B2 = a2.data_ptr(), b2.data_ptr()
    assert ig.long_rings(args) and "_128_" in kernel_name(args).decode()
    print("pairs on the long rings", layout, K, K2, flush=True)
    _run(args)
    want = sum(x[:rows, :k].double() @ (y[:, :k].double().t() if layout == ig.NT else y.double()) for x, y, k in ((a, b, K), (a2, b2, K2)))
    assert bool(((c[:rows].double() - want).abs() <= _bound(K + K2, want, True)).all()) and bool((c[rows:] == 7.0).all())


def test_the_long_rings_are_for_few_blocks_of_many_slabs():
    """At most 224 squares of 128 and 16 slabs or more, also over two operand pairs: both sides of either limit; and no launch that is split."""
    def plan(layout, M, N, K, **more):
        g = ig.args(layout, M, N, K, out=ig.F32 if layout == ig.TN else ig.BF16, **more)
        assert "_128_" in kernel_name(g).decode(), (layout, M, N, K, more)
        return g
    for layout in (ig.NT, ig.NN):
        for K, K2, long in ((1024, 0, True), (968, 0, True), (960, 0, False), (960, 64, True), (896, 64, False)):
            assert ig.long_rings(plan(layout, 264, 264, K, K2=K2, lda=1024, ldb=1024)) == long, (layout, K, K2)
        for rows, columns, long in ((16, 14, True), (15, 15, False)):     # (bf16 results added to old ones: on squares alone)
            assert ig.long_rings(plan(layout, 128 * rows, 128 * columns, 1024, accumulate=1)) == long, (layout, rows, columns)
    assert ig.long_rings(plan(ig.TN, 264, 264, 961)) and not ig.long_rings(plan(ig.TN, 264, 264, 960))
    for layout, M, N, K in ((ig.NT, 264, 264, 4096), (ig.NN, 104, 512, 5632), (ig.TN, 256, 1024, 4000)):
        for more in ({}, dict(k_dev=256) if layout == ig.TN else dict(m_dev=256)):
            g = plan(layout, M, N, K, **more)
            assert ig.long_rings(g)
            g.scratch, g.scratch_bytes = 256, ig.scratch_bytes(g)
            assert g.scratch_bytes > 0 and not ig.long_rings(plan(layout, M, N, K, scratch=g.scratch, scratch_bytes=g.scratch_bytes, **more))
