"""Sizes that callers allocate by, on the host: a buffer made for a batch has to serve every smaller one."""
import random

import pytest

from paper_2602_05145_amd import binding as B
from paper_2602_05145_amd import workloads as W
from tests import internal_gemm as ig


@pytest.mark.parametrize("d", [8, 256, 1000, 1023, 2048, 2056, 4096, 8192])
def test_rmsnorm_scratch_never_falls_as_rows_grow(d):
    sizes = [B.tide_rmsnorm_bwd_scratch_bytes(rows, d) for rows in range(1, 16500)]
    assert sizes == sorted(sizes)
    assert sizes[0] == 4 * d and sizes[479] >= 480 * 4 * d      # a partial sum per block, a block per row up to 480
    assert sizes[-1] <= 16 << 20                                # the fixed array of tide_rmsnorm_bwd_static


@pytest.mark.parametrize("preset,seqs,batches", [("tiny", (1, 7, 117), 300), ("small", (5, 33, 64, 128, 333, 512), 200),
                                                 ("8b", (3, 17, 64, 509, 2048), 90), ("32b", (64, 513), 60)])
def test_step_workspaces_never_shrink_as_batches_grow(preset, seqs, batches):
    """A workspace made for some batch size is enough for every smaller batch of the same configuration."""
    for seq in seqs:
        sizes = [B.tide_draft_workspace_bytes(B.make_config(W.get_config(preset, batch=b, seq=seq))) for b in range(1, batches + 1)]
        assert sizes[0] > 0 and sizes == sorted(sizes), (preset, seq)


def _step_products(cfg, ccfg):
    """Every bf16 product of a training step, as its GemmArgs: over all rows, over the selected ones, by blocks of the LM head."""
    d, f, v, kh = cfg["hidden"], cfg["ffn"], cfg["vocab"], cfg["n_capture"] * cfg["target_hidden"]
    nq, nqkv = cfg["n_heads"] * cfg["head_dim"], (cfg["n_heads"] + 2 * cfg["n_kv_heads"]) * cfg["head_dim"]
    t, ldz, block = cfg["batch"] * cfg["seq"], (v + 63) // 64 * 64, B.tide_draft_workspace_offset(ccfg, "lm_rows")
    for n, k in ((d, kh), (nqkv, d)):
        yield ig.args(ig.NT, t, n, k)
    yield ig.args(ig.NT, t, d, d, K2=d, ldb=2 * d)
    for n, k in ((d, nq), (f, d), (d, f)):
        yield ig.args(ig.NT, t, n, k, m_dev=256)
    for n, k, k2 in ((f, d, 0), (d, f, f), (nq, d, 0)):
        yield ig.args(ig.NN, t, n, k, K2=k2, m_dev=256)
    yield ig.args(ig.NN, t, d, nqkv)
    for m, n in ((d, f), (f, d), (d, nq), (nqkv, d), (d, kh)):
        yield ig.args(ig.TN, m, n, t, out=ig.F32)
    for r0 in (0, (t - 1) // block * block):
        rows = min(block, t - r0)
        yield ig.args(ig.NT, rows, v, d, ldc=ldz, m_dev=256)
        yield ig.args(ig.NN, rows, d, v, lda=ldz, m_dev=256)
        yield ig.args(ig.TN, v, d, rows, lda=ldz, out=ig.F32)


@pytest.mark.parametrize("preset", ["small", "8b", "32b"])
def test_every_product_of_a_step_finds_the_scratch_it_was_planned_with(preset):
    """A block of the LM head can ask for more than the product over all rows, which fills the chip by itself."""
    rng, asked = random.Random(5), 0
    shapes = [(4672, 576), (32768, 0), (3999, 0), (2500, 0)] + [(int(2 ** rng.uniform(5, 15)), rng.choice((0, 0, 256, 576, 4096))) for _ in range(150)]
    for t, block in shapes:
        cfg = W.get_config(preset, batch=1, seq=t)
        ccfg = B.make_config(cfg)
        ccfg.lm_block_rows = block
        have = B.tide_draft_workspace_offset(ccfg, "splitk_bytes")
        assert 0 <= have <= 64 << 20
        for g in _step_products(cfg, ccfg):
            need = ig.scratch_bytes(g)
            assert need <= have, (t, block, g.layout, g.M, g.N, g.K, need, have)
            asked += need > 0
    assert asked > 300


def test_the_bound_on_split_scratch_covers_every_number_of_rows():
    """Random products, at their number of rows and at smaller ones, on the host and (known on the device alone) as a bound."""
    rng, split = random.Random(17), 0
    for _ in range(3000):
        layout, out = rng.randrange(3), rng.randrange(2)
        rows, n, k = int(2 ** rng.uniform(3, 15)), *(int(2 ** rng.uniform(3, 15)) // 8 * 8 for _ in range(2))
        k2, dev = (k if layout != ig.TN and out == ig.BF16 and rng.random() < 0.3 else 0), layout != ig.TN and rng.random() < 0.5

        def product(r):
            m, kk = (n, r) if layout == ig.TN else (r, k)
            return ig.args(layout, m, k if layout == ig.TN else n, kk, out=out, K2=k2, **(dict(m_dev=256) if dev else {}))

        bound = ig.scratch_bound(product(rows))
        assert bound <= 64 << 20
        last = bound
        for r in sorted({rows, *(rng.randint(1, rows) for _ in range(6))}, reverse=True):
            need, b = ig.scratch_bytes(product(r)), ig.scratch_bound(product(r))
            assert need <= b <= last, (layout, out, r, n, k, need, b)
            last = b
            split += need > 0
    assert split > 1500
