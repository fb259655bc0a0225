"""The work that users of the draft-training library have it do, as cases that can be timed one by one.

Whole calls (a training step on fixed-length or packed batches, an evaluation pass) and the building blocks a
program can call by themselves (matrix products in the three layouts, attention, cross-entropy, RMSNorm), each
through the C ABI's names in `paper_2602_05145_amd.binding`.  Widths come from the configurations of
`paper_2602_05145_amd.workloads`; row counts run over what a serving system hands over: a few requests (hundreds
of rows, ragged) up to full training batches.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2602_05145_amd import binding as B
from paper_2602_05145_amd import workloads as W

DEV = "cuda:0"
DTYPE = {"fp32": torch.float32, "bf16": torch.bfloat16}
CODE = {"fp32": B.TIDE_DTYPE_FP32, "bf16": B.TIDE_DTYPE_BF16}
LAYOUT = {"nt": B.LAYOUT_NT, "nn": B.LAYOUT_NN, "tn": B.LAYOUT_TN}


def listed():
    return [
        # the smallest call: the fp32 configuration used to check a setup, 128 rows (launches and latency count)
        dict(name="train_tiny_fp32", kind="train", preset="tiny", batch=2, seq=64, n_seqs=0),
        # an ordinary fine-tuning step of a small draft: 8 right-padded requests
        dict(name="train_small", kind="train", preset="small", batch=8, seq=512, n_seqs=0),
        # the training step of the 8B-shaped draft on a full batch: the largest call
        dict(name="train_8b", kind="train", preset="8b", batch=16, seq=2048, n_seqs=0),
        # an online adaptation step on a handful of requests, packed back to back without padding: ragged
        # lengths, a row count that is no multiple of anything
        dict(name="train_8b_packed", kind="train", preset="8b", batch=1, seq=1999, n_seqs=7),
        # the deployment gate: evaluation of the draft on held-out requests of an odd length
        dict(name="forward_8b", kind="forward", preset="8b", batch=3, seq=1333, n_seqs=0),
        # gate / up projection of a full batch's loss-carrying rows (forward products)
        dict(name="gemm_nt_gate", kind="gemm", layout="nt", m=27852, n=14336, k=4096, dtype="bf16"),
        # input gradient of a small draft's down projection on an odd number of rows
        dict(name="gemm_nn_small", kind="gemm", layout="nn", m=1665, n=5632, k=2048, dtype="bf16"),
        # weight gradient (fp32 result) of the feature projection over an odd number of rows
        dict(name="gemm_tn_fc", kind="gemm", layout="tn", m=4096, n=12288, k=3999, dtype="bf16"),
        # attention layer of the 8B-shaped draft, forward and backward
        dict(name="attn_8b", kind="attn", batch=16, seq=2048, n_heads=32, n_kv_heads=8, head_dim=128, dtype="bf16"),
        # attention layer of a draft with the other usual head size, odd length
        dict(name="attn_d64", kind="attn", batch=6, seq=777, n_heads=16, n_kv_heads=4, head_dim=64, dtype="bf16"),
        # cross-entropy statistics and logit gradient of one block of logits
        dict(name="ce_8b", kind="ce", rows=8192, vocab=128256, dtype="bf16"),
        # RMSNorm forward and backward with the residual gradient, a full batch
        dict(name="rmsnorm_8b", kind="rmsnorm", rows=27852, d=4096, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_WIDTHS = (256, 688, 1024, 2048, 2560, 4096, 5120, 5632, 6144, 12288, 14336, 25600, 32000)


def draw(rng):
    kind = rng.choice(("train", "train", "train", "forward", "gemm", "gemm", "gemm", "attn", "attn", "ce", "rmsnorm"))
    if kind in ("train", "forward"):
        preset = rng.choice(("tiny", "small", "small", "8b"))
        rows = {"tiny": (32, 1024), "small": (128, 6144), "8b": (256, 2500)}[preset]
        t = _log_int(rng, *rows)
        if kind == "train" and rng.random() < 0.4:
            return dict(kind=kind, preset=preset, batch=1, seq=t, n_seqs=rng.randint(2, max(2, min(24, t // 16))))
        batch = rng.randint(1, max(1, min(12, t // 32)))
        return dict(kind=kind, preset=preset, batch=batch, seq=max(1, t // batch), n_seqs=0)
    if kind == "gemm":
        layout, dtype = rng.choice(("nt", "nn", "tn")), rng.choice(("bf16", "bf16", "bf16", "fp32"))
        while True:
            rows, a, b = _log_int(rng, 32, 32768), rng.choice(_WIDTHS), rng.choice(_WIDTHS)
            flops = 2.0 * rows * a * b
            if 1e7 < flops < (2e12 if dtype == "bf16" else 5e10):
                break
        if layout == "tn":
            return dict(kind=kind, layout=layout, m=a, n=b, k=rows, dtype=dtype)
        return dict(kind=kind, layout=layout, m=rows, n=a, k=b, dtype=dtype)
    if kind == "attn":
        head_dim = rng.choice((64, 128, 128))
        seq = _log_int(rng, 48, 8192 if head_dim == 128 else 2500)
        tokens = _log_int(rng, seq, max(seq, min(16384, (24 if head_dim == 128 else 8) * 1024 * 1024 // seq)))
        n_heads, n_kv_heads = rng.choice(((16, 8), (32, 8), (40, 8), (16, 4), (32, 32)))
        return dict(kind=kind, batch=max(1, min(64, tokens // seq)), seq=seq, n_heads=n_heads, n_kv_heads=n_kv_heads,
                    head_dim=head_dim, dtype="bf16")
    if kind == "ce":
        dtype = rng.choice(("bf16", "bf16", "bf16", "fp32"))
        return dict(kind=kind, rows=_log_int(rng, 48, 8192), vocab=rng.choice((4096, 32000, 50257, 128256, 152064)), dtype=dtype)
    return dict(kind=kind, rows=_log_int(rng, 48, 32768), d=rng.choice((256, 1024, 2048, 2560, 4096, 5120, 8192)),
                dtype=rng.choice(("bf16", "bf16", "bf16", "fp32")))


# ---- inputs ----------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, *shape, dtype, scale=1.0):
    return (torch.randn(shape, device=DEV, generator=g) * scale).to(dtype)


def _cfg(case):
    return W.get_config(case["preset"], batch=case["batch"], seq=case["seq"])


def _lengths(case):
    """Lengths of the packed sequences, by the case alone: requests differ, and they fill the rows."""
    t, n = case["batch"] * case["seq"], case["n_seqs"]
    cuts = sorted(random.Random(1000003 * t + n).sample(range(1, t), n - 1))
    return [b - a for a, b in zip([0] + cuts, cuts + [t])]


def _sequences(case):
    """(first row, length) of every sequence."""
    if not case["n_seqs"]:
        return [(b * case["seq"], case["seq"]) for b in range(case["batch"])]
    out, at = [], 0
    for n in _lengths(case):
        out.append((at, n))
        at += n
    return out


def _zipf(g, shape, vocab, s):
    w = torch.arange(1, vocab + 1, device=DEV, dtype=torch.float64) ** (-s)
    cdf = torch.cumsum(w / w.sum(), 0)
    ranks = torch.searchsorted(cdf, torch.rand(shape, device=DEV, dtype=torch.float64, generator=g), right=True)
    return torch.randperm(vocab, device=DEV, generator=g)[ranks.clamp_(max=vocab - 1)].to(torch.int32)


def _model_inputs(case, seed):
    """Weights, captured hidden states (a few channels carry massive activations), emitted tokens and loss mask."""
    cfg, g = _cfg(case), _gen(seed)
    dt, t = DTYPE[cfg["dtype"]], case["batch"] * case["seq"]
    params = {}
    for name, shape in W.param_shapes(cfg).items():
        params[name] = (1.0 + torch.randn(shape, device=DEV, generator=g) * 0.05).to(dt) if len(shape) == 1 else _randn(g, *shape, dtype=dt, scale=0.02)
    ht = cfg["target_hidden"]
    hidden = torch.randn((t, cfg["n_capture"] * ht), device=DEV, generator=g)
    for k in range(cfg["n_capture"]):
        idx = torch.randperm(ht, device=DEV, generator=g)[: int(round(cfg["outlier_frac"] * ht))] + k * ht
        hidden[:, idx] *= cfg["outlier_scale"]
    tokens = _zipf(g, (t,), cfg["vocab"], cfg["zipf_s"])
    mask = torch.ones(t, dtype=torch.uint8, device=DEV)
    if cfg["mask"] == "bernoulli":
        mask = (torch.rand(t, device=DEV, generator=g) >= cfg["mask_p"]).to(torch.uint8)
    elif cfg["mask"] == "lengths" and not case["n_seqs"]:  # right-padded requests, a quarter of the length or more
        pos = torch.arange(t, device=DEV) % case["seq"]
        length = torch.randint(max(1, case["seq"] // 4), case["seq"] + 1, (case["batch"],), device=DEV, generator=g)
        mask = (pos < length.repeat_interleave(case["seq"])).to(torch.uint8)
        hidden[mask == 0] = 0.0
        tokens[mask == 0] = 0
    else:  # the prompt's part of every request carries no loss
        for at, n in _sequences(case):
            mask[at: at + int(0.15 * n)] = 0
    return cfg, params, hidden.to(dt), tokens, mask


def _prepare_model(case, seed):
    cfg, params, hidden, tokens, mask = _model_inputs(case, seed)
    s = dict(cfg=cfg, ccfg=B.make_config(cfg), params=params, hidden=hidden, tokens=tokens, mask=mask)
    s["c_params"] = B.make_tensors(params)
    s["ws_bytes"] = B.tide_draft_workspace_bytes(s["ccfg"])
    s["workspace"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV)
    s["loss"] = torch.zeros(1, device=DEV)
    if case["n_seqs"]:
        lengths = _lengths(case)
        s["cu"] = torch.tensor([0] + lengths, device=DEV).cumsum(0).to(torch.int32)
        s["n_seqs"], s["max_seqlen"] = len(lengths), max(lengths)
    if case["kind"] == "train":
        zeros = lambda: {k: torch.zeros(v.shape, device=DEV) for k, v in params.items()}  # noqa: E731
        s["grads"], s["m"], s["v"] = zeros(), zeros(), zeros()
        s["master"] = {k: v.float() for k, v in params.items()} if cfg["dtype"] == "bf16" else None
        s["c_grads"], s["adam"] = B.make_tensors(s["grads"]), B.TideAdamState()
        s["adam"].m, s["adam"].v, s["adam"].master = B.make_tensors(s["m"]), B.make_tensors(s["v"]), B.make_tensors(s["master"])
        s["adam"].step = 0
    else:
        kept = int(((mask != 0) & (tokens >= 0) & (tokens < cfg["vocab"])).sum())

        def view(name, n, dtype):  # a named result that the call leaves in its workspace
            off = B.tide_draft_workspace_offset(s["ccfg"], name)
            return s["workspace"][off: off + n * dtype.itemsize].view(dtype)

        s["rows"] = dict(loss_rows=view("loss_rows", kept, torch.float32), lse=view("lse", kept, torch.float32),
                         yhat=view("yhat", kept * cfg["hidden"], DTYPE[cfg["dtype"]]).view(kept, cfg["hidden"]))
    return s


def _gemm_shapes(case):
    m, n, k = case["m"], case["n"], case["k"]
    return {"nt": ((m, k), (n, k)), "nn": ((m, k), (k, n)), "tn": ((k, m), (k, n))}[case["layout"]]


def _gemm_out(case):
    return "fp32" if case["layout"] == "tn" else case["dtype"]  # weight gradients are fp32


def _block_inputs(case, seed):
    g, dt = _gen(seed), DTYPE[case["dtype"]]
    if case["kind"] == "gemm":
        a, b = _gemm_shapes(case)
        return dict(a=_randn(g, *a, dtype=dt), b=_randn(g, *b, dtype=dt, scale=0.02))
    if case["kind"] == "attn":
        t, nh, nkv, dh = case["batch"] * case["seq"], case["n_heads"], case["n_kv_heads"], case["head_dim"]
        return dict(qkv=_randn(g, t, (nh + 2 * nkv) * dh, dtype=dt), dout=_randn(g, t, nh * dh, dtype=dt, scale=0.1))
    if case["kind"] == "ce":
        ldz = (case["vocab"] + 63) // 64 * 64
        return dict(z=_randn(g, case["rows"], ldz, dtype=dt, scale=1.3), tokens=_zipf(g, (case["rows"],), case["vocab"], 1.05),
                    mask=torch.ones(case["rows"], dtype=torch.uint8, device=DEV))
    r, d = case["rows"], case["d"]
    return dict(x=_randn(g, r, d, dtype=dt), dy=_randn(g, r, d, dtype=dt, scale=0.1), res=_randn(g, r, d, dtype=dt, scale=0.1),
                gain=(1.0 + torch.randn(d, device=DEV, generator=g) * 0.05).to(dt))


def prepare(case, seed):
    if case["kind"] in ("train", "forward"):
        s = _prepare_model(case, seed)
    else:
        s, dt = _block_inputs(case, seed), DTYPE[case["dtype"]]
        f32 = dict(device=DEV, dtype=torch.float32)
        if case["kind"] == "gemm":
            out = _gemm_out(case)
            s["c"] = torch.empty(case["m"], case["n"], device=DEV, dtype=DTYPE[out])
            s["ws_bytes"] = B.tide_gemm_workspace_bytes(LAYOUT[case["layout"]], case["m"], case["n"], case["k"], CODE[out])
            s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV) if s["ws_bytes"] else None
        elif case["kind"] == "attn":
            b, n, nh = case["batch"], case["seq"], case["n_heads"]
            s["out"], s["dqkv"] = torch.empty_like(s["dout"]), torch.empty_like(s["qkv"])
            s["lse"], s["delta"] = torch.empty(b, nh, n, **f32), torch.empty(b, nh, n, **f32)
        elif case["kind"] == "ce":
            s["lse"], s["loss_rows"] = torch.empty(case["rows"], **f32), torch.empty(case["rows"], **f32)
        else:
            r, d = case["rows"], case["d"]
            s["y"], s["dx"] = torch.empty(r, d, device=DEV, dtype=dt), torch.empty(r, d, device=DEV, dtype=dt)
            s["rstd"], s["dg"] = torch.empty(r, **f32), torch.empty(d, **f32)
            s["scratch"] = torch.empty(B.tide_rmsnorm_bwd_scratch_bytes(r, d), dtype=torch.uint8, device=DEV)
    s["case"] = dict(case)
    return s


# ---- one pass --------------------------------------------------------------------------------------------------
def run(s):
    c, stream = s["case"], torch.cuda.current_stream().cuda_stream
    if c["kind"] == "train":
        lr = s["cfg"]["lr"]
        if c["n_seqs"]:
            B.tide_draft_train_step_packed(s["ccfg"], s["c_params"], s["c_grads"], s["adam"], s["hidden"], s["tokens"], s["mask"],
                                           s["cu"], s["n_seqs"], s["max_seqlen"], lr, s["loss"], s["workspace"], s["ws_bytes"], stream)
        else:
            B.tide_draft_train_step(s["ccfg"], s["c_params"], s["c_grads"], s["adam"], s["hidden"], s["tokens"], s["mask"], lr,
                                    s["loss"], s["workspace"], s["ws_bytes"], stream)
        out = dict(loss=s["loss"], grads=s["grads"], params=s["params"])
        if s["master"] is not None:
            out["master"] = s["master"]
        return out
    if c["kind"] == "forward":
        B.tide_draft_forward(s["ccfg"], s["c_params"], s["hidden"], s["tokens"], s["mask"], s["loss"], None, s["workspace"],
                             s["ws_bytes"], stream)
        return dict(s["rows"], loss=s["loss"])
    code = CODE[c["dtype"]]
    if c["kind"] == "gemm":
        B.tide_gemm(LAYOUT[c["layout"]], c["m"], c["n"], c["k"], 1.0, s["a"], s["b"], s["c"], None, code, CODE[_gemm_out(c)], 0, stream,
                    workspace=s["ws"], workspace_bytes=s["ws_bytes"])
        return s["c"]
    if c["kind"] == "attn":
        shape = (c["batch"], c["seq"], c["n_heads"], c["n_kv_heads"], c["head_dim"])
        B.tide_attention_fwd(*shape, s["qkv"], s["out"], s["lse"], code, stream)
        B.tide_attention_bwd(*shape, s["qkv"], s["out"], s["dout"], s["lse"], s["delta"], s["dqkv"], code, stream)
        return dict(out=s["out"], lse=s["lse"], dqkv=s["dqkv"])
    if c["kind"] == "ce":
        # in place, as in training; a repeated pass takes what the pass before left as its logits
        B.tide_ce_train(c["rows"], c["vocab"], s["z"], s["z"].shape[1], s["tokens"], s["mask"], s["lse"], s["loss_rows"], code, stream)
        return dict(dz=s["z"], lse=s["lse"], loss_rows=s["loss_rows"])
    B.tide_rmsnorm_fwd(c["rows"], c["d"], s["x"], s["gain"], 1e-5, s["y"], s["rstd"], code, stream)
    B.tide_rmsnorm_bwd(c["rows"], c["d"], s["dy"], s["x"], s["gain"], s["rstd"], s["res"], s["dx"], s["dg"], s["scratch"], code, stream)
    return dict(y=s["y"], rstd=s["rstd"], dx=s["dx"], dg=s["dg"])


# ---- what a pass cannot do without -----------------------------------------------------------------------------
def work(case):
    if case["kind"] in ("train", "forward"):
        cfg, train = _cfg(case), case["kind"] == "train"
        es = DTYPE[cfg["dtype"]].itemsize
        t = case["batch"] * case["seq"]
        share = {"bernoulli": 0.9, "lengths": 0.85 if case["n_seqs"] else 0.625, "prefix": 0.85}[cfg["mask"]]
        p = {k: math.prod(v) for k, v in W.param_shapes(cfg).items()}
        late = p["w_o"] + p["w_gate"] + p["w_up"] + p["w_down"] + p["w_lm"]   # run on the rows that carry loss
        pairs = sum(n * (n + 1) / 2 for _, n in _sequences(case)) * cfg["n_heads"] * cfg["head_dim"]
        n = sum(p.values())
        if train:
            # weights read, gradients, both moments and (bf16) master and weight written, the fp32 state read
            state = 12 if cfg["dtype"] == "fp32" else 16
            return dict(flops=t * (4.0 * p["w_fc"] + 6.0 * p["w_qkv"]) + share * t * 6.0 * late + 14.0 * pairs,
                        bytes=n * (2.0 * es + 4 + 8 + 8 + (8 if state == 16 else 0)) + t * p["w_fc"] / cfg["hidden"] * es)
        return dict(flops=t * 2.0 * (p["w_fc"] + p["w_qkv"]) + share * t * 2.0 * late + 4.0 * pairs,
                    bytes=n * es + t * (p["w_fc"] / cfg["hidden"] + share * cfg["hidden"]) * es)
    es = DTYPE[case["dtype"]].itemsize
    if case["kind"] == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(flops=2.0 * m * n * k, bytes=es * k * (m + n) + DTYPE[_gemm_out(case)].itemsize * m * n)
    if case["kind"] == "attn":
        t, nh, nkv, dh = case["batch"] * case["seq"], case["n_heads"], case["n_kv_heads"], case["head_dim"]
        pairs = case["batch"] * nh * dh * case["seq"] * (case["seq"] + 1) / 2.0
        return dict(flops=14.0 * pairs, bytes=es * t * dh * (2.0 * (nh + 2 * nkv) + 2 * nh) + 4.0 * t * nh)
    if case["kind"] == "ce":
        return dict(flops=0.0, bytes=2.0 * es * case["rows"] * case["vocab"])
    return dict(flops=0.0, bytes=5.0 * es * case["rows"] * case["d"])   # x, dy, residual gradient; y, dx


def tolerance(case):
    dtype = _cfg(case)["dtype"] if case["kind"] in ("train", "forward") else case["dtype"]
    if case["kind"] in ("train", "forward"):
        # fp32: gradients are 1e-6 to 1.5e-6 off 64 bits.  bf16: 0.3 to 0.9 %, the roundings of the activations.  A
        # draft's first AdamW update divides a gradient by its own magnitude, so the small ones flip by 2 lr (1 % of a
        # weight at most); and most of dW_lm is nearly zero beside the rows of the frequent labels, whose elements are
        # up to 1.4 times its root mean square off.
        return dict(rel=8e-6, max=2e-3) if dtype == "fp32" else dict(rel=2e-2, max=0.99)
    if case["kind"] == "gemm":
        return dict(rel=4e-6, max=4e-5) if _gemm_out(case) == "fp32" else dict(rel=4e-3, max=2e-2)
    if dtype == "fp32":
        return dict(rel=2e-6, max=1e-4)
    # largest difference: one step of bf16 on either side
    return {"attn": dict(rel=1e-2, max=0.1), "ce": dict(rel=1e-4, max=2e-2), "rmsnorm": dict(rel=7e-3, max=2e-2)}[case["kind"]]


# ---- the same in 64 bits ---------------------------------------------------------------------------------------
def _rms(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g


def _rope(x, theta):
    n, _, dh = x.shape
    inv = theta ** (-2.0 * torch.arange(dh // 2, device=DEV, dtype=torch.float64) / dh)
    ang = torch.arange(n, device=DEV, dtype=torch.float64)[:, None] * inv
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    x1, x2 = x[..., : dh // 2], x[..., dh // 2:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _attend(q, k, v):
    """q [n, nh, dh], k and v [n, nkv, dh] in 64 bits -> (out [n, nh, dh], lse [nh, n])."""
    n, nh, dh = q.shape
    rep = nh // k.shape[1]
    qt, kt, vt = q.transpose(0, 1), k.repeat_interleave(rep, 1).transpose(0, 1), v.repeat_interleave(rep, 1).transpose(0, 1)
    s = (qt @ kt.transpose(1, 2).contiguous()) / math.sqrt(dh)
    s = s.masked_fill(torch.ones(n, n, dtype=torch.bool, device=DEV).triu(1), -math.inf)
    lse = torch.logsumexp(s, -1)
    return (torch.exp(s - lse[..., None]) @ vt).transpose(0, 1), lse


def _exact_model(case, seed):
    cfg, params, hidden, tokens, mask = _model_inputs(case, seed)
    train = case["kind"] == "train"
    p = {k: v.double().requires_grad_(train and k != "w_lm") for k, v in params.items()}
    nq, nk, dh = cfg["n_heads"] * cfg["head_dim"], cfg["n_kv_heads"] * cfg["head_dim"], cfg["head_dim"]
    kept = ((mask != 0) & (tokens >= 0) & (tokens < cfg["vocab"])).nonzero().flatten()
    with torch.set_grad_enabled(train):
        x0 = hidden.double() @ p["w_fc"].t()
        qkv = _rms(x0, p["g1"], cfg["rms_eps"]) @ p["w_qkv"].t()

        def one(part):
            n = part.shape[0]
            q, k = _rope(part[:, :nq].view(n, -1, dh), cfg["rope_theta"]), _rope(part[:, nq: nq + nk].view(n, -1, dh), cfg["rope_theta"])
            return _attend(q, k, part[:, nq + nk:].view(n, -1, dh))[0].reshape(n, nq)

        parts = [qkv[at: at + n] for at, n in _sequences(case)]
        if train:
            from torch.utils.checkpoint import checkpoint
            att = torch.cat([checkpoint(one, part, use_reentrant=False) for part in parts])
        else:
            att = torch.cat([one(part) for part in parts])
        x1 = x0[kept] + att[kept] @ p["w_o"].t()
        b = _rms(x1, p["g2"], cfg["rms_eps"])
        x2 = x1 + (torch.nn.functional.silu(b @ p["w_gate"].t()) * (b @ p["w_up"].t())) @ p["w_down"].t()
        y = _rms(x2, p["g3"], cfg["rms_eps"])
    n, w = max(1, len(kept)), p["w_lm"]
    yd, labels = y.detach(), tokens[kept].long()
    dy, dw = (torch.zeros_like(yd), torch.zeros_like(w)) if train else (None, None)
    lse, terms = [], []
    for r in range(0, len(kept), 2048):
        z = yd[r: r + 2048] @ w.t()
        lse.append(torch.logsumexp(z, -1))
        at = labels[r: r + 2048, None]
        terms.append(lse[-1] - z.gather(1, at).flatten())
        if train:
            z = torch.exp(z - lse[-1][:, None]).scatter_add_(1, at, torch.full_like(at, -1, dtype=torch.float64)) / n
            dy[r: r + 2048] = z @ w
            dw += z.t() @ yd[r: r + 2048]
        del z
    loss = torch.cat(terms).sum().reshape(1) / n
    if not train:
        return dict(loss=loss, lse=torch.cat(lse), loss_rows=torch.cat(terms), yhat=yd)
    y.backward(dy)
    grads = {k: (dw if k == "w_lm" else v.grad) for k, v in p.items()}
    lr, new = cfg["lr"], {}
    for k, v in p.items():   # the first AdamW step: both bias-corrected moments are the gradient's own
        new[k] = v.detach() * (1 - lr * cfg["weight_decay"]) - lr * grads[k] / (grads[k].abs() + cfg["adam_eps"])
    out = dict(loss=loss, grads=grads, params=new)
    if cfg["dtype"] == "bf16":
        out["master"] = new
    return out


def exact(case, seed):
    if case["kind"] in ("train", "forward"):
        return _exact_model(case, seed)
    s = _block_inputs(case, seed)
    if case["kind"] == "gemm":
        a, b = s["a"].double(), s["b"].double()
        return {"nt": lambda: a @ b.t(), "nn": lambda: a @ b, "tn": lambda: a.t() @ b}[case["layout"]]()
    if case["kind"] == "attn":
        bt, n, nh, nkv, dh = case["batch"], case["seq"], case["n_heads"], case["n_kv_heads"], case["head_dim"]
        rep = nh // nkv
        out, dqkv = torch.empty(bt * n, nh * dh, dtype=torch.float64, device=DEV), torch.empty(bt * n, (nh + 2 * nkv) * dh, dtype=torch.float64, device=DEV)
        lse = torch.empty(bt, nh, n, dtype=torch.float64, device=DEV)
        for b in range(bt):
            for h in range(nkv):   # one key/value head and its query heads
                rows = slice(b * n, (b + 1) * n)
                cols = [slice(h * rep * dh, (h + 1) * rep * dh)] + [slice((nh + o + h) * dh, (nh + o + h + 1) * dh) for o in (0, nkv)]
                q, k, v = (s["qkv"][rows, c].double().reshape(n, -1, dh).requires_grad_() for c in cols)
                with torch.enable_grad():
                    o, l = _attend(q, k, v)
                    o = o.reshape(n, rep * dh)
                    o.backward(s["dout"][rows, cols[0]].double())
                out[rows, cols[0]], lse[b, h * rep: (h + 1) * rep] = o.detach(), l.detach()
                for c, x in zip(cols, (q, k, v)):
                    dqkv[rows, c] = x.grad.reshape(n, -1)
                del o, l
        return dict(out=out, lse=lse, dqkv=dqkv)
    if case["kind"] == "ce":
        v, at = case["vocab"], s["tokens"].long()[:, None]
        lse = torch.cat([torch.logsumexp(z[:, :v].double(), -1) for z in s["z"].split(1024)])
        terms = lse - s["z"].gather(1, at).flatten().double()
        dz = torch.zeros(s["z"].shape, dtype=torch.float64, device=DEV)
        for r in range(0, case["rows"], 1024):
            dz[r: r + 1024, :v] = torch.exp(s["z"][r: r + 1024, :v].double() - lse[r: r + 1024, None])
        dz.scatter_add_(1, at, torch.full_like(at, -1, dtype=torch.float64))
        return dict(dz=dz, lse=lse, loss_rows=terms)
    x, dy, res, g = (s[k].double() for k in ("x", "dy", "res", "gain"))
    rstd = torch.rsqrt(x.square().mean(-1) + 1e-5)
    u, r = dy * g, rstd[:, None]
    dx = res + r * u - x * r ** 3 * (u * x).mean(-1, keepdim=True)
    return dict(y=x * r * g, rstd=rstd, dx=dx, dg=(dy * x * r).sum(0))
