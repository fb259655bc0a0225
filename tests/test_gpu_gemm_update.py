"""Weight gradients whose AdamW update follows in the same launch: the gradient against a float64 product, the update against the
formula in float64 on the gradient that was written."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2602_05145_amd import workloads as W
from tests import internal_gemm as ig


class AdamTarget(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("m", "v", "master", "w", "dyn")] + [(n, C.c_float) for n in ("lr", "decay", "beta1", "beta2", "eps", "c1", "c2")]


supported = ig._symbol("_ZN4tide19gemm_adam_supportedERKNS_8GemmArgsERKNS_10AdamTargetE", C.c_bool, [C.POINTER(ig.GemmArgs), C.POINTER(AdamTarget)])
launch = ig._symbol("_ZN4tide16launch_gemm_adamERKNS_8GemmArgsERKNS_10AdamTargetEP12ihipStream_t", C.c_int,
                    [C.POINTER(ig.GemmArgs), C.POINTER(AdamTarget), C.c_void_p])
pays = ig._symbol("_ZN4tide14gemm_adam_paysERKNS_8GemmArgsE", C.c_bool, [C.POINTER(ig.GemmArgs)])
name = ig._symbol("_ZN4tide21gemm_adam_kernel_nameERKNS_8GemmArgsE", C.c_char_p, [C.POINTER(ig.GemmArgs)])
launch_group = ig._symbol("_ZN4tide22launch_gemm_adam_groupEPKNS_8GemmArgsEPKNS_10AdamTargetEiP12ihipStream_t", C.c_int,
                          [C.POINTER(ig.GemmArgs), C.POINTER(AdamTarget), C.c_int, C.c_void_p])
RATE = dict(lr=1e-3, decay=1 - 1e-5, beta1=0.9, beta2=0.999, eps=1e-8, c1=1 / (1 - 0.9 ** 3), c2=(1 - 0.999 ** 3) ** -0.5)


def test_what_a_product_with_update_serves():
    ok = AdamTarget(m=256, v=256, master=256, w=256)
    assert supported(ig.args(ig.TN, 264, 136, 77, out=ig.F32), ok)
    for g in (ig.args(ig.NT, 264, 136, 64, out=ig.F32), ig.args(ig.TN, 264, 136, 77), ig.args(ig.TN, 260, 136, 77, out=ig.F32),
              ig.args(ig.TN, 264, 132, 77, out=ig.F32), ig.args(ig.TN, 264, 136, 77, out=ig.F32, ldc=140), ig.args(ig.TN, 264, 136, 77, out=ig.F32, c=264),
              ig.args(ig.TN, 264, 136, 77, out=ig.F32, residual=256), ig.args(ig.TN, 264, 136, 77, out=ig.F32, in_dtype=ig.F32)):
        assert not supported(g, ok)
    for f in ("m", "v", "master", "w"):
        assert not supported(ig.args(ig.TN, 264, 136, 77, out=ig.F32), AdamTarget(**dict(dict(m=256, v=256, master=256, w=256), **{f: 264})))


def test_few_tiles_and_split_ones_leave_the_update_to_the_pass_over_all_weights():
    """A tile's update keeps its CU busy for 8 us and more however idle the others are: not with less than half of them at work."""
    for m, n, k in ((256, 256, 64), (688, 256, 1000), (1376, 512, 300), (1024, 1024, 5000), (2048, 1024, 64)):
        assert not pays(ig.args(ig.TN, m, n, k, out=ig.F32)), (m, n, k)
    for m, n, k in ((2816, 1024, 64), (1536, 1536, 300), (5632, 2048, 2560), (128256, 4096, 1700)):
        assert pays(ig.args(ig.TN, m, n, k, out=ig.F32)), (m, n, k)
    ok = AdamTarget(m=256, v=256, master=256, w=256)
    for m, n, k, k_dev in ((248, 688, 30000, 0), (2040, 1544, 8000, 256), (2816, 1024, 5000, 0), (3440, 1280, 8000, 0)):
        g = ig.args(ig.TN, m, n, k, out=ig.F32, k_dev=k_dev)
        assert supported(g, ok)
        g.scratch, g.scratch_bytes = 256, ig.scratch_bytes(g)
        assert g.scratch_bytes > 0 and not supported(g, ok), (m, n, k)     # all tiles split: a kernel of its own adds the parts
    g = ig.args(ig.TN, 4344, 4096, 8000, out=ig.F32)
    g.scratch, g.scratch_bytes = 256, ig.scratch_bytes(g)
    assert g.scratch_bytes > 0 and supported(g, ok)                        # the last round alone: 16 of 272 tiles


# M, N, K, the number of rows on the device (None: known to the host), old values, columns of the weight, kernel, scratch
CASES = [(264, 136, 77, None, 0, 136, "128", 0), (264, 136, 77, None, 1, 272, "128", 0), (264, 136, 77, 13, 1, 136, "128", 0), (264, 136, 77, 0, 0, 136, "128", 0),
         (264, 136, 77, 0, 1, 136, "128", 0), (4096, 4104, 40, 33, 0, 4104, "128", 0), (5456, 656, 65, None, 1, 656, "128x256", 0),
         (1048, 7192, 65, None, 0, 7192, "160x256", 0), (1288, 7240, 301, 1, 1, 7240, "192x256", 0), (2192, 5392, 515, None, 0, 5392, "224x256", 0),
         (248, 688, 30000, None, 1, 688, "128", 0), (2040, 1544, 8000, 4321, 0, 1544, "128", 0), (4344, 4096, 8000, None, 1, 4096, "256", 1),
         (4344, 4096, 8000, 4321, 0, 4096, "256", 1), (4344, 4096, 8000, 70, 1, 4096, "256", 1), (4344, 4096, 8000, 0, 1, 4096, "256", 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,rows,add,ld,kernel,split", CASES)
def test_gradient_and_update(M, N, K, rows, add, ld, kernel, split):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    dev = dict(device="cuda")
    a, b = torch.randn(K, M, generator=g, **dev).bfloat16(), (torch.randn(K, N, generator=g, **dev) * 0.1).bfloat16()
    k = K if rows is None else rows
    grad, m, v, master = (torch.randn(M, ld, generator=g, **dev) * s for s in (1.0, 0.1, 1.0, 0.02))
    v = v.square() * 1e-2
    w = master.bfloat16()
    col = ld - N                                          # a column half of a wider weight, as a two-part input projection has it
    old = [x.clone() for x in (grad, m, v, master, w)]
    cnt = torch.tensor([k], dtype=torch.int32, **dev)
    dyn = torch.tensor([RATE["lr"], RATE["decay"], RATE["c1"], RATE["c2"]], **dev) if rows is not None else None
    scratch = torch.full((64 << 20,), 0xFF, dtype=torch.uint8, **dev)
    p = ig.args(ig.TN, M, N, K, out=ig.F32, ldc=ld, a=a.data_ptr(), b=b.data_ptr(), c=grad[:, col:].data_ptr(), alpha=-0.5, accumulate=add)
    if rows is not None:
        p.k_dev = cnt.data_ptr()
    if split:
        p.scratch, p.scratch_bytes = scratch.data_ptr(), scratch.numel()
        assert ig.scratch_bytes(p) > 0
    t = AdamTarget(m=m[:, col:].data_ptr(), v=v[:, col:].data_ptr(), master=master[:, col:].data_ptr(), w=w[:, col:].data_ptr(),
                   dyn=None if dyn is None else dyn.data_ptr(), **(RATE if dyn is None else dict(beta1=0.9, beta2=0.999, eps=1e-8)))
    assert name(p).decode() == f"gemm_mfma_tn_{kernel}_adamw"
    print("update", M, N, K, rows, add, kernel, flush=True)
    assert launch(p, t, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    for x, y in zip((grad, m, v, master, w), old):
        assert torch.equal(x[:, :col], y[:, :col])       # the other columns are not this product's
    grad, m, v, master, w = (x[:, col:] for x in (grad, m, v, master, w))
    g0, m0, v0, th0 = (x[:, col:].double() for x in old[:4])
    want = -0.5 * (a[:k].double().t() @ b[:k].double()) + add * g0
    # a float sum of k products of size 0.1, whose partial sums are of size sqrt(k) 0.1: k roundings of 6e-8 of that, which add up as a root
    # of their number; times four.  (4: the old values)
    partial, roundings = 0.1 * max(k, 1) ** 0.5, max(k, 1)
    assert float((grad.double() - want).abs().max()) < 4 * 6e-8 * (roundings ** 0.5 * partial + 4)
    gd = grad.double()
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
    m1, v1 = b1 * m0 + (1 - b1) * gd, b2 * v0 + (1 - b2) * gd * gd
    u = RATE["lr"] * m1 * RATE["c1"] / (v1.sqrt() * RATE["c2"] + 1e-8)
    th1 = th0 * RATE["decay"] - u
    eps = 2.0 ** -22                                      # the constants' own rounding and three or four of the formula's
    assert bool(((m.double() - m1).abs() <= eps * (m0.abs() + gd.abs())).all())
    assert bool(((v.double() - v1).abs() <= eps * (v0 + gd * gd)).all())
    assert bool(((master.double() - th1).abs() <= eps * (th0.abs() + 4 * u.abs() + 4 * RATE["lr"] * RATE["c1"] * (m0.abs() + gd.abs()) / (v1.sqrt() * RATE["c2"] + 1e-8))).all())
    assert torch.equal(w, master.bfloat16())


def test_a_group_takes_products_that_it_can_update_alone():
    ok, bad = ig.args(ig.TN, 264, 136, 77, out=ig.F32), ig.args(ig.NT, 264, 136, 64, out=ig.F32)
    t = AdamTarget(m=256, v=256, master=256, w=256)
    for gs in ((), (ok, bad), (ok,) * 7):
        assert launch_group((ig.GemmArgs * 7)(*gs), (AdamTarget * 7)(*[t] * len(gs)), len(gs), None) != 0


# (M, N, old values, rows of the batch rather than all) of each product; upper bound of the rows (4096 is where the tiles change), rows on the device
GROUPS = [([(264, 136, 0, 0)], 77, 70), ([(8, 8, 0, 1), (1288, 1544, 1, 0), (160, 256, 0, 1), (168, 264, 0, 1), (2056, 520, 0, 0), (320, 512, 1, 1)], 65, 0),
          ([(8, 8, 0, 1), (1288, 1544, 1, 0), (160, 256, 0, 1), (168, 264, 0, 1), (2056, 520, 0, 0), (320, 512, 1, 1)], 4096, 3001),
          ([(8, 8, 0, 1), (1288, 1544, 1, 0), (256, 256, 0, 1), (264, 264, 0, 1), (2056, 520, 0, 0), (512, 512, 1, 1)], 4097, 4001)]


@pytest.mark.gpu
@pytest.mark.parametrize("shapes,K,rows", GROUPS)
def test_a_group_gives_what_a_launch_each_gives(shapes, K, rows):
    """Bit for bit: an element's sum runs over the rows in the same order on every tile."""
    g = torch.Generator(device="cuda").manual_seed(K + rows)
    dev = dict(device="cuda")
    cnt = torch.tensor([rows], dtype=torch.int32, **dev)
    group, single = [], []
    stream = torch.cuda.current_stream().cuda_stream
    for M, N, add, trimmed in shapes:
        a, b = torch.randn(K, M, generator=g, **dev).bfloat16(), (torch.randn(K, N, generator=g, **dev) * 0.1).bfloat16()
        grad, m, v, master = (torch.randn(M, N, generator=g, **dev) * s for s in (1.0, 0.1, 1.0, 0.02))
        state = [grad, m, v.square() * 1e-2, master, master.bfloat16()]
        for out in (group, single):
            out.append([x.clone() for x in state] + [a, b])
    def arguments(state, shape):
        M, N, add, trimmed = shape
        grad, m, v, master, w, a, b = (x.data_ptr() for x in state)
        p = ig.args(ig.TN, M, N, K, out=ig.F32, a=a, b=b, c=grad, alpha=-0.5, accumulate=add)
        if trimmed:
            p.k_dev = cnt.data_ptr()
        return p, AdamTarget(m=m, v=v, master=master, w=w, **RATE)
    print("group", len(shapes), K, rows, flush=True)
    for state, shape in zip(single, shapes):
        assert launch(*arguments(state, shape), stream) == 0
    gs, ts = zip(*(arguments(state, shape) for state, shape in zip(group, shapes)))
    assert launch_group((ig.GemmArgs * len(gs))(*gs), (AdamTarget * len(ts))(*ts), len(gs), stream) == 0
    torch.cuda.synchronize()
    for x, y, shape in zip(group, single, shapes):
        assert all(torch.equal(p, q) for p, q in zip(x, y)), shape


@pytest.mark.gpu
@pytest.mark.parametrize("kw,block", [(dict(), 0), (dict(batch=3, seq=37), 64), (dict(hidden=264, n_heads=2, n_kv_heads=1, head_dim=132, ffn=332), 0),
                                      (dict(ffn=16640, vocab=512), 0), (dict(ffn=16652), 0)])
def test_a_step_updates_every_weight_once(kw, block):
    """Weights whose product carries the update (W_lm; with ffn 16640 the MLP's) and weights whose product does not (few tiles; ffn 332 and 16652:
    rows no 16-byte piece fits), in one step; LM head in blocks, of which the last carries it.  Against the update in float64 from the gradients that the step returned."""
    from paper_2602_05145_amd import runtime
    cfg = W.get_config("small", **dict(dict(batch=2, seq=64, target_hidden=256, hidden=256, n_heads=2, n_kv_heads=1, head_dim=128, ffn=512, vocab=16640), **kw))
    wl = W.make_workload(cfg)
    cfg["lm_block_rows"] = block
    assert pays(ig.args(ig.TN, max(cfg["vocab"], cfg["ffn"]), cfg["hidden"], cfg["batch"] * cfg["seq"], out=ig.F32))
    tr = runtime.trainer_from_workload(cfg, wl)
    before = {k: x.astype(np.float64) for k, x in tr.host(tr.master).items()}
    print("step", kw, block, flush=True)
    tr.train_step(cfg["lr"])
    torch.cuda.synchronize()
    grads, master, params = (tr.host(x) for x in (tr.grads, tr.master, tr.params))
    for k, g in grads.items():
        g = g.astype(np.float64)
        want = before[k] * (1 - cfg["lr"] * cfg["weight_decay"]) - cfg["lr"] * g / (np.abs(g) + cfg["adam_eps"])
        # the first step divides a gradient by its own magnitude: a rounding of either counts against lr; float gradients below
        # 1e-18 have squares that underflow (a gradient of zero is exact: the weight decays)
        ok = (np.abs(master[k] - want) <= 2.0 ** -22 * (np.abs(before[k]) + 4 * cfg["lr"])) | ((np.abs(g) < 1e-16) & (g != 0))
        assert ok.all(), (k, np.abs(master[k] - want).max())
        assert np.array_equal(params[k], W.round_to_bf16(master[k])), k


@pytest.mark.gpu
def test_an_input_projection_is_updated_by_its_two_products():
    """W_in, whose column halves are two products (144 tiles each), against the update in float64 from the gradient that the step returned."""
    from tests.test_gpu_token_input import _setup
    cfg = W.get_config("small", batch=2, seq=33, target_hidden=64, hidden=1536, n_heads=12, n_kv_heads=4, head_dim=128, ffn=256, vocab=512)
    assert pays(ig.args(ig.TN, cfg["hidden"], cfg["hidden"], 66, out=ig.F32, ldc=2 * cfg["hidden"]))
    wl, ti, tr, *_ = _setup(cfg, embed_rows=57)
    tr.set_token_input(ti["embed"], ti["input_ids"], ti["w_in"])
    before = tr.master_w_in.double()
    print("token-input step", flush=True)
    tr.train_step_tok(cfg["lr"])
    torch.cuda.synchronize()
    g = tr.grad_w_in.double()
    want = before * (1 - cfg["lr"] * cfg["weight_decay"]) - cfg["lr"] * g / (g.abs() + cfg["adam_eps"])
    # as above
    ok = ((tr.master_w_in.double() - want).abs() <= 2.0 ** -22 * (before.abs() + 4 * cfg["lr"])) | ((g.abs() < 1e-16) & (g != 0))
    assert bool(ok.all()) and float(g.abs().max()) > 0
    assert torch.equal(tr.w_in, tr.master_w_in.bfloat16())
