"""fp32 step: SwiGLU inside the products, the gains updated where their gradients are summed.  Every tensor of a step against the float64 oracle on the same inputs, and the
update against its formula on the gradients that the step returned; sizes on either side of where the products are one launch."""
import numpy as np
import pytest
import torch

from oracle import tide_oracle as O
from paper_2602_05145_amd import runtime, workloads as W

SMALL = dict(target_hidden=20, hidden=36, n_heads=2, n_kv_heads=1, head_dim=18, ffn=50, vocab=77)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(), dict(batch=1, seq=1), dict(batch=3, seq=37, **SMALL), dict(batch=2, seq=520, vocab=512),
                                dict(batch=5, seq=203, ffn=1100, vocab=300), dict(batch=2, seq=33, ffn=8, vocab=20000), dict(batch=1, seq=33, mask_p=1.0)])
def test_fp32_step(kw):
    cfg = W.get_config("tiny", **kw)
    wl = W.make_workload(cfg)
    tr = runtime.trainer_from_workload(cfg, wl)
    tr.workspace.fill_(0xFF)
    print("fp32 step", kw, flush=True)
    tr.train_step(cfg["lr"])
    torch.cuda.synchronize()
    p0 = {k: np.asarray(v, np.float64) for k, v in wl["params"].items()}
    z = {k: np.zeros_like(v) for k, v in p0.items()}
    _, ref, *_ = O.train_step(cfg, p0, z, z, 0, wl["hidden"].astype(np.float64), wl["tokens"], wl["mask"], cfg["lr"])
    grads, params, m, v = (tr.host(x) for x in (tr.grads, tr.params, tr.m, tr.v))
    for k, r in ref.items():
        g = grads[k].astype(np.float64)
        assert np.abs(g - r).max() <= 1e-4 * np.abs(r).max() + 1e-30, k            # as the other fp32 steps
        b1, b2 = (float(np.float32(cfg[x])) for x in ("beta1", "beta2"))
        assert (np.abs(m[k] - (1 - b1) * g) <= 2.0 ** -22 * np.abs(g)).all(), k
        assert (np.abs(v[k] - (1 - b2) * g * g) <= 2.0 ** -22 * g * g + 1e-44).all(), k
        want = p0[k] * (1 - cfg["lr"] * cfg["weight_decay"]) - cfg["lr"] * g / (np.abs(g) + cfg["adam_eps"])
        # the update divides the gradient by its own magnitude: a few roundings of lr; squares of gradients below 1e-16 underflow (a gradient
        # of zero is exact: the weight decays)
        ok = (np.abs(params[k] - want) <= 2.0 ** -22 * (np.abs(p0[k]) + 4 * cfg["lr"])) | ((np.abs(g) < 1e-16) & (g != 0))
        assert ok.all(), (k, np.abs(params[k] - want).max())
