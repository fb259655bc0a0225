"""The row plan on both sides of the size where it becomes two launches, and the gain gradients of the three norms, which
one launch folds.  The plan is whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_2602_05145_amd import binding as B, runtime, workloads as W
from tests.gpu_util import sync

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,seq", [(1, 1), (1, 1023), (1, 1025), (8, 1024), (1, 8193), (3, 3001)])
def test_row_plan(batch, seq):
    T = batch * seq
    cfg = W.get_config("tiny", batch=batch, seq=seq, target_hidden=8, hidden=16, n_heads=2, n_kv_heads=1, head_dim=8, ffn=16, vocab=50)
    rng = np.random.default_rng(T)
    wl = W.make_workload(W.get_config("tiny", batch=1, seq=4, target_hidden=8, hidden=16, n_heads=2, n_kv_heads=1, head_dim=8, ffn=16, vocab=50))
    tokens = rng.integers(-2, 53, (batch, seq)).astype(np.int32)      # some labels outside the vocabulary
    mask = (rng.random((batch, seq)) < 0.6).astype(np.uint8)
    tr = runtime.DraftTrainer(cfg, wl["params"])
    tr.set_batch(rng.standard_normal((batch, seq, 24)).astype(np.float32), tokens, mask)
    tr.workspace.fill_(0xFF)
    print(f"row plan T={T}", flush=True)
    tr.forward()
    sync()
    keep = ((mask != 0) & (tokens >= 0) & (tokens < 50)).reshape(-1)

    def ints(name, n):
        off = B.tide_draft_workspace_offset(tr.ccfg, name)
        return tr.workspace[off:off + 4 * n].view(torch.int32).cpu().numpy()

    kept = np.flatnonzero(keep)
    assert ints("cnt", 1)[0] == len(kept)
    assert np.array_equal(ints("kept_idx", len(kept)), kept)
    assert np.array_equal(ints("row_pos", T), np.where(keep, np.cumsum(keep) - 1, -1))
    scal = tr.intermediate("scal", (2,), "f32").cpu().numpy()
    assert scal[0] == max(1, len(kept)) and scal[1] == np.float32(1.0) / np.float32(max(1, len(kept)))
