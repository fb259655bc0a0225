"""Matrix products at the sizes where a dispatch rule or a kernel changes its form, against an fp64 product of the same
values.  Bounds: K products of fp32 rounding 2^-24 each, added in fp32 in any order, are at most K 2^-24 off the sum of
the magnitudes; the observed error grows with sqrt(K), and 2e-5 of the largest result is the bound the other product tests use
(2e-6 for fp32 operands)."""
import pytest
import torch

from tests import internal_gemm as ig
from tests.gpu_util import DEV, stream, sync

pytestmark = pytest.mark.gpu

DT = {"fp32": (0, torch.float32), "bf16": (1, torch.bfloat16)}


def _operands(B, layout, M, N, K, dtype, seed):
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


@pytest.mark.parametrize("M,N,K,tile,split", [(264, 520, 1, "128", False), (264, 520, 31, "128", False), (264, 520, 33, "128", False),
                                              (136, 72, 1999, "128", True), (3720, 3656, 65, "256", False), (3720, 3656, 127, "256", False),
                                              (4312, 4088, 2051, "160x256", False), (4344, 4096, 4099, "256", True)])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_weight_gradient_over_any_number_of_rows(B, M, N, K, tile, split, accumulate):
    """TN with K (the rows of a batch) of any remainder, on the small, the large and an intermediate tile, whole, split into parts
    everywhere (136 x 72) and in the last round alone (4344 x 4096)."""
    plan = ig.args(ig.TN, M, N, K, out=ig.F32, accumulate=accumulate)
    plan.scratch, plan.scratch_bytes = 256, B.tide_gemm_workspace_bytes(B.LAYOUT_TN, M, N, K, 0)
    assert ig.kernel_name(plan).decode() == f"gemm_mfma_tn_{tile}_f32out" and (plan.scratch_bytes > 0 and "x" not in tile) == split
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


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K,split", [(8, 8, 704, False), (8, 8, 1408, True), (136, 264, 2056, True), (304, 4096, 4104, True),
                                         (169, 688, 2560, True), (1024, 1000, 8000, True), (3000, 1032, 800, False)])
def test_small_results_split_over_k(B, layout, M, N, K, split):
    """Fewer tiles of 128 than the chip runs at a time: with a workspace each tile's K range is shared by several blocks
    and a second kernel adds the partial sums.  Odd M, ragged K; residual, alpha and accumulation in the second kernel; and
    the same call without a workspace."""
    if layout == B.LAYOUT_TN and M % 8:
        M += 8 - M % 8
    a, b, ref = _operands(B, layout, M, N, K, "bf16", M + 7 * K)
    g = torch.Generator(device=DEV).manual_seed(9)
    top = float(ref.abs().max())
    tiles, slabs = ((M + 127) // 128) * ((N + 127) // 128), (K + 63) // 64
    need = B.tide_gemm_workspace_bytes(layout, M, N, K, 0)
    assert need % (tiles * 65536) == 0 and (need > 0) == split     # whole partial sums, and two parts or more
    assert need <= min(512, tiles * slabs // 4) * 65536
    for out in ("fp32", "bf16"):
        dt = DT[out][1]
        res, c0 = (torch.randn(M, N, device=DEV, generator=g).to(dt) for _ in range(2))
        tol = 2e-5 if out == "fp32" else 6e-3      # bf16: the rounding of the result
        c = torch.full((M, N), float("nan"), device=DEV, dtype=dt)
        _gemm(B, layout, M, N, K, a, b, c, "bf16", out)
        assert float((c.double() - ref).abs().max()) < tol * top
        plain = torch.full((M, N), float("nan"), device=DEV, dtype=dt)
        B.tide_gemm(layout, M, N, K, 1.0, a, b, plain, None, 1, DT[out][0], 0, stream())
        sync()
        assert float((plain.double() - c.double()).abs().max()) < (5e-6 if out == "fp32" else tol) * top
        c = c0.clone()
        _gemm(B, layout, M, N, K, a, b, c, "bf16", out, alpha=0.5, residual=res, accumulate=1)
        want = 0.5 * ref + res.double() + c0.double()
        assert float((c.double() - want).abs().max()) < tol * float(want.abs().max())


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(1000, 512, 32008), (2040, 1544, 20000), (2296, 1016, 12288)])
def test_large_tiles_split_over_k(B, layout, M, N, K):
    """Few tiles with a long contraction, where the split runs on 256 x 256 tiles (the first: sixteen parts of small ones).  Ragged M, N and K, bf16 and fp32 results,
    residual and alpha in the second kernel."""
    assert B.tide_gemm_workspace_bytes(layout, M, N, K, 1) > 0
    a, b, ref = _operands(B, layout, M, N, K, "bf16", M + K)
    for out, tol in (("fp32", 2e-5), ("bf16", 6e-3)):
        dt = DT[out][1]
        res = torch.randn(M, N, device=DEV).to(dt)
        c = torch.full((M, N), float("nan"), device=DEV, dtype=dt)
        _gemm(B, layout, M, N, K, a, b, c, "bf16", out, alpha=0.25, residual=res)
        want = 0.25 * ref + res.double()
        assert float((c.double() - want).abs().max()) < tol * float(want.abs().max())


@pytest.mark.parametrize("layout,M,N,K,out", [(0, 4352, 4096, 2048, "bf16"), (1, 4315, 4096, 2056, "bf16"), (2, 4096, 4352, 1999, "fp32"),
                                              (2, 2048, 4096, 20000, "fp32")])
def test_a_product_without_workspace_need_leaves_any_workspace_alone(B, layout, M, N, K, out):
    """A size of 0 says that the call is never split: a large buffer that other products share is neither read nor written,
    and the result is bit for bit that of the call without one."""
    assert B.tide_gemm_workspace_bytes(layout, M, N, K, DT[out][0]) == 0
    g = torch.Generator(device=DEV).manual_seed(M + K)
    a = torch.randn((K, M) if layout == B.LAYOUT_TN else (M, K), device=DEV, generator=g).bfloat16()
    b = torch.randn((N, K) if layout == B.LAYOUT_NT else (K, N), device=DEV, generator=g).bfloat16()
    ws = torch.full((96 << 20,), 0xA5, dtype=torch.uint8, device=DEV)
    got = [torch.full((M, N), float("nan"), device=DEV, dtype=DT[out][1]) for _ in range(2)]
    for c, w in zip(got, (ws, None)):
        print(f"gemm told 0: layout={layout} M={M} N={N} K={K} {out} workspace={w is not None}", flush=True)
        B.tide_gemm(layout, M, N, K, 1.0, a, b, c, None, 1, DT[out][0], 0, stream(), workspace=w, workspace_bytes=0 if w is None else w.numel())
        sync()
    untouched, finite, same = bool((ws == 0xA5).all()), not bool(torch.isnan(got[0]).any()), torch.equal(got[0], got[1])
    assert untouched and finite and same     # (plain values: a failing assertion prints the tensors it names)


def _launch(what, g):
    print(f"internal gemm {what}: layout={g.layout} M={g.M} N={g.N} K={g.K}+{g.K2} out={g.out_dtype} scratch={g.scratch_bytes}", flush=True)
    assert ig.launch(g, stream()) == 0
    sync()


@pytest.mark.parametrize("layout,M,N,K,pair", [(0, 4315, 4096, 2056, 0), (1, 4352, 4088, 2048, 1), (2, 4344, 4096, 4099, 0), (0, 8450, 4096, 2048, 0)])
@pytest.mark.parametrize("out", ["bf16", "fp32"])
def test_only_the_last_round_of_large_tiles_split(layout, M, N, K, pair, out):
    """256 or 512 whole tiles and a few more, as a training step launches them: the whole ones first, the parts of the others
    behind them, and the sums in a second launch with the residual (and, of bf16, the old values).  Ragged M, N and K, one and
    two operand pairs.  fp32 results without a residual have a split of their own."""
    dt = DT[out][1]
    g = torch.Generator(device=DEV).manual_seed(M + N)
    a, a2 = (torch.randn((K, M) if layout == ig.TN else (M, K), device=DEV, generator=g).bfloat16() for _ in range(2))
    b, b2 = (torch.randn((N, K) if layout == ig.NT else (K, N), device=DEV, generator=g).bfloat16() for _ in range(2))
    res, c0 = (torch.randn(M, N, device=DEV, generator=g).to(dt) for _ in range(2))

    def product(x, y):
        x, y = x.double(), y.double()
        return (x.t().contiguous() if layout == ig.TN else x) @ (y.t().contiguous() if layout == ig.NT else y)

    want = -0.5 * (product(a, b) + (product(a2, b2) if pair else 0.0)) + res.double() + (c0.double() if out == "bf16" else 0.0)
    ws, got = torch.full((64 << 20,), 0xFF, dtype=torch.uint8, device=DEV), []     # NaN patterns
    for split in (True, False):
        c = c0.clone()
        p = ig.args(layout, M, N, K, out=DT[out][0], K2=K if pair else 0, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr(), alpha=-0.5,
                    residual=res.data_ptr(), ldr=N, accumulate=int(out == "bf16"))
        if pair:
            p.A2, p.B2 = a2.data_ptr(), b2.data_ptr()
        if split:
            p.scratch, p.scratch_bytes = ws.data_ptr(), ws.numel()
            tail = -(-M // 256) * -(-N // 256) % 256
            need = ig.scratch_bytes(p)
            assert need > 0 and need % (tail * 262144) == 0 and need // (tail * 262144) >= 2    # two parts or more of the last tiles alone
        _launch("last round", p)
        got.append(c.double())
        assert float((got[-1] - want).abs().max()) < (2e-5 if out == "fp32" else 6e-3) * float(want.abs().max())
    same = torch.equal(got[0], got[1])
    assert not same                             # the split happened: another order of the sums


@pytest.mark.parametrize("m_off", [0, 640])
def test_last_round_of_a_row_count_known_on_the_device(m_off):
    """The same launch, planned for 85 % of 5376 rows, with row counts on both sides of whole rounds: none, a few tiles all of
    which are split, 192 that are not, one whole round, one and a tail, the bound.  Rows past the count stay as they were."""
    M, N, K = 5376, 4096, 4096
    g = torch.Generator(device=DEV).manual_seed(3)
    a, b = torch.randn(M, K, device=DEV, generator=g).bfloat16(), torch.randn(K, N, device=DEV, generator=g).bfloat16()
    want, ws = a.double() @ b.double(), torch.empty(64 << 20, dtype=torch.uint8, device=DEV)
    for rows in (0, 1, 300, 1000, 3000, 4096, 4097, 4359, 5376, 6000):
        cnt, n = torch.tensor([rows + m_off], dtype=torch.int32, device=DEV), min(rows, M)
        c = torch.full((M, N), 7.0, device=DEV, dtype=torch.bfloat16)
        ws.fill_(0xFF)
        p = ig.args(ig.NN, M, N, K, a=a.data_ptr(), b=b.data_ptr(), c=c.data_ptr(), m_dev=cnt.data_ptr(), m_off=m_off,
                    scratch=ws.data_ptr(), scratch_bytes=ws.numel())
        assert ig.scratch_bytes(p) > 0
        _launch(f"{rows} rows on the device", p)
        assert n == 0 or float((c[:n].double() - want[:n]).abs().max()) < 6e-3 * float(want.abs().max()), rows
        untouched = bool((c[n:] == 7.0).all())
        assert untouched, rows


def test_split_products_of_a_training_step_with_few_kept_rows():
    """The number of rows behind the attention is on the device only: with one sequence in eight carrying loss, the same
    launches come out with other numbers of parts.  Against the oracle."""
    import numpy as np
    from oracle import tide_oracle as O
    from paper_2602_05145_amd import runtime, workloads as W
    cfg = W.get_config("small", batch=8, seq=96, target_hidden=512, hidden=512, n_heads=4, n_kv_heads=2, head_dim=128, ffn=2048, vocab=8008,
                       mask="none", seed=31)
    wl = W.make_workload(cfg)
    for kept in (8, 1, 0):
        mask = np.zeros_like(wl["mask"])
        mask[:kept] = 1
        tr = runtime.DraftTrainer(cfg, wl["params"])
        tr.set_batch(wl["hidden"], wl["tokens"], mask)
        tr.workspace.fill_(0xFF)
        print(f"split step kept={kept}", flush=True)
        tr.train_step(cfg["lr"])
        sync()
        p0 = {k: np.asarray(v, np.float64) for k, v in wl["params"].items()}
        z = {k: np.zeros_like(v) for k, v in p0.items()}
        loss, grads, *_ = O.train_step(cfg, p0, z, z, 0, wl["hidden"].astype(np.float64), wl["tokens"], mask, cfg["lr"])
        assert abs(float(tr.loss.item()) - loss) <= 1e-2 * abs(loss)
        for k, r in grads.items():
            g, r = tr.host(tr.grads)[k].reshape(-1), r.reshape(-1)
            if kept:
                assert g @ r / (np.linalg.norm(g) * np.linalg.norm(r)) > 0.999, (kept, k)
            else:
                assert not g.any(), k


@pytest.mark.parametrize("kw", [dict(), dict(batch=3, seq=37, target_hidden=20, hidden=36, n_heads=2, n_kv_heads=1, head_dim=18, ffn=50, vocab=77),
                                dict(batch=2, seq=520)])
def test_grouped_weight_gradients_of_an_fp32_step(kw):
    """The layer's weight gradients of an fp32 step in one launch (aligned and unaligned rows), and one by one where the
    batch is too long for that (1040 rows).  Against the oracle, as the other fp32 steps: 1e-4 of the largest gradient."""
    import numpy as np
    from oracle import tide_oracle as O
    from paper_2602_05145_amd import runtime, workloads as W
    cfg = W.get_config("tiny", **dict(dict(vocab=512), **kw))
    wl = W.make_workload(cfg)
    tr = runtime.trainer_from_workload(cfg, wl)
    tr.workspace.fill_(0xFF)
    print(f"fp32 grouped step {kw}", flush=True)
    tr.train_step(cfg["lr"])
    sync()
    p0 = {k: np.asarray(v, np.float64) for k, v in wl["params"].items()}
    z = {k: np.zeros_like(v) for k, v in p0.items()}
    _, grads, *_ = O.train_step(cfg, p0, z, z, 0, wl["hidden"].astype(np.float64), wl["tokens"], wl["mask"], cfg["lr"])
    got = tr.host(tr.grads)
    for k, r in grads.items():
        assert np.abs(got[k] - r).max() <= 1e-4 * np.abs(r).max(), k


def test_the_profile_names_the_tile_that_ran(B):
    """Large tiles chosen for their split over K: without a workspace the launch runs small ones, and is reported so."""
    M, N, K = 2040, 1544, 20000
    need = B.tide_gemm_workspace_bytes(B.LAYOUT_NN, M, N, K, 1)
    assert need > 0
    a, b, _ = _operands(B, B.LAYOUT_NN, M, N, K, "bf16", 1)
    c, ws = torch.empty(M, N, device=DEV, dtype=torch.bfloat16), torch.empty(need, dtype=torch.uint8, device=DEV)
    for w, name in ((ws, "gemm_mfma_nn_256_bf16out"), (None, "gemm_mfma_nn_128_bf16out")):
        print(f"profiled gemm workspace={w is not None}", flush=True)
        B.tide_profile_start()
        B.tide_gemm(B.LAYOUT_NN, M, N, K, 1.0, a, b, c, None, 1, 1, 0, stream(), workspace=w, workspace_bytes=0 if w is None else need)
        assert [r["kernel"] for r in B.tide_profile_stop()] == [name]


def test_profile_of_an_fp32_step_counts_the_rows_that_ran(B):
    """The grouped products work on the rows that carry loss, whose number is on the device; the report's flops are of those.
    Against the count from the configuration; and the launch that folds the norms' partial sums is in the report."""
    import numpy as np
    from paper_2602_05145_amd import runtime, workloads as W
    cfg = W.get_config("tiny", batch=2, seq=64)
    wl = W.make_workload(cfg)
    mask = np.zeros_like(wl["mask"])
    mask[:, :13] = 1
    tr = runtime.DraftTrainer(cfg, wl["params"])
    tr.set_batch(wl["hidden"], np.abs(wl["tokens"]) % cfg["vocab"], mask)
    print("profiled fp32 step", flush=True)
    B.tide_profile_start()
    tr.train_step(cfg["lr"])
    got = {r["kernel"]: r for r in B.tide_profile_stop()}
    t, rows, p = 128, 26, {k: int(np.prod(s)) for k, s in W.param_shapes(cfg).items()}
    late = p["w_o"] + p["w_gate"] + p["w_up"] + p["w_down"] + p["w_lm"]
    want = 4.0 * t * p["w_fc"] + 6.0 * t * p["w_qkv"] + 6.0 * rows * late
    assert "gemm_fp32_group" in got and got["colsums"]["launches"] == 1
    assert abs(sum(r["flops"] for k, r in got.items() if k.startswith("gemm")) - want) < 1e-5 * want
