"""RMSNorm forward and backward where the row count or the width changes the grid or the kernel: one row per block up to
480 rows, 480 blocks up to 3360, 8 rows per block, a full chip; widths of one, two and four pieces per thread, the widest one, and a
forward-only width above it.  Against fp64 on the same values; the outputs are rounded once (2^-9 relative in bf16), sums of d
or of the rows in fp32 are 1e-5 off at most."""
import pytest
import torch

from paper_2602_05145_amd import binding as B
from tests.gpu_util import DEV, stream, sync

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("rows,d", [(1, 8), (3, 2048), (479, 264), (481, 2056), (3360, 264), (3361, 256), (5000, 1000), (11000, 512), (600, 4104), (530, 8192)])
def test_rmsnorm_over_row_counts_and_widths(rows, d, dtype):
    dt, code = (torch.bfloat16, 1) if dtype == "bf16" else (torch.float32, 0)
    g = torch.Generator(device=DEV).manual_seed(rows + d)
    x, dy, res = (torch.randn(rows, d, device=DEV, generator=g).to(dt) for _ in range(3))
    gain = (1.0 + 0.1 * torch.randn(d, device=DEV, generator=g)).to(dt)
    y, dx = (torch.full((rows, d), float("nan"), dtype=dt, device=DEV) for _ in range(2))
    rstd, dg = torch.full((rows,), float("nan"), device=DEV), torch.full((d,), float("nan"), device=DEV)
    scratch = torch.full((B.tide_rmsnorm_bwd_scratch_bytes(rows, d),), 0xFF, dtype=torch.uint8, device=DEV)
    print(f"rmsnorm rows={rows} d={d} {dtype}", flush=True)
    B.tide_rmsnorm_fwd(rows, d, x, gain, 1e-5, y, rstd, code, stream())
    B.tide_rmsnorm_bwd(rows, d, dy, x, gain, rstd, res, dx, dg, scratch, code, stream())
    sync()
    xd, dyd, gd = x.double(), dy.double(), gain.double()
    r = torch.rsqrt(xd.square().mean(-1, keepdim=True) + 1e-5)
    u = dyd * gd
    want = dict(y=xd * r * gd, rstd=r.flatten(), dx=res.double() + r * u - xd * r ** 3 * (u * xd).mean(-1, keepdim=True), dg=(dyd * xd * r).sum(0))
    for name, got in dict(y=y, rstd=rstd, dx=dx, dg=dg).items():
        tol = 2.0 ** -8 if dtype == "bf16" and name in ("y", "dx") else 1e-5
        assert float((got.double() - want[name]).abs().max()) < tol * float(want[name].abs().max()), name


# a row per wave: forward up to 2048 columns (512, 1024 and 2048 per form), backward up to 2 KB; blocks whose rows are no multiple of its four waves
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("rows,d", [(1, 512), (2, 520), (5, 1024), (481, 504), (1443, 1016), (3365, 1032), (10246, 512), (3, 2040)])
def test_rmsnorm_with_a_row_per_wave(rows, d, dtype):
    test_rmsnorm_over_row_counts_and_widths(rows, d, dtype)


# fp32 rows of more than 768 columns, a wave each below 6000 of them, a block each from there on, and past the caches
@pytest.mark.parametrize("rows,d", [(5999, 776), (6000, 776), (6000, 768), (6001, 2048), (36900, 1024)])
def test_rmsnorm_of_wide_fp32_rows(rows, d):
    test_rmsnorm_over_row_counts_and_widths(rows, d, "fp32")


# arrays that the last cache does not hold, in the backward pass (four above 288 MB) and in the forward one (two), and a little less than that; one, two and four pieces per thread
@pytest.mark.parametrize("rows,d,dtype", [(36700, 1032, "bf16"), (18400, 2056, "bf16"), (36750, 2056, "bf16"), (18400, 4104, "bf16"), (18400, 2056, "fp32"), (9200, 4104, "fp32"),
                                          (32770, 1032, "bf16"), (16387, 2056, "bf16"), (32801, 2056, "bf16"), (16400, 4104, "bf16"), (32900, 1032, "fp32"), (16390, 2056, "fp32"), (8200, 4104, "fp32")])
def test_rmsnorm_past_the_caches(rows, d, dtype):
    test_rmsnorm_over_row_counts_and_widths(rows, d, dtype)


def test_rmsnorm_forward_of_wide_rows():
    rows, d = 5, 8200
    x, gain = torch.randn(rows, d, device=DEV), torch.randn(d, device=DEV)
    y, rstd = torch.empty_like(x), torch.empty(rows, device=DEV)
    print("rmsnorm wide", flush=True)
    B.tide_rmsnorm_fwd(rows, d, x, gain, 1e-5, y, rstd, 0, stream())
    sync()
    want = x.double() * torch.rsqrt(x.double().square().mean(-1, keepdim=True) + 1e-5) * gain.double()
    assert float((y.double() - want).abs().max()) < 1e-5 * float(want.abs().max())


def test_rmsnorm_backward_of_fewer_rows_than_its_scratch_was_made_for():
    """3500 rows are walked by fewer blocks than 1000: the buffer made for them serves both, and nothing past it is written."""
    d, made_for = 264, 3500
    size = B.tide_rmsnorm_bwd_scratch_bytes(made_for, d)
    buf = torch.full((size + 64 * 1024,), 0xA5, dtype=torch.uint8, device=DEV)
    for rows in (3500, 1000, 479):
        x, dy = (torch.randn(rows, d, device=DEV) for _ in range(2))
        gain = torch.ones(d, device=DEV)
        y, dx, rstd, dg = torch.empty_like(x), torch.empty_like(x), torch.empty(rows, device=DEV), torch.empty(d, device=DEV)
        print(f"rmsnorm scratch of {made_for} rows, rows={rows}", flush=True)
        B.tide_rmsnorm_fwd(rows, d, x, gain, 1e-5, y, rstd, 0, stream())
        B.tide_rmsnorm_bwd(rows, d, dy, x, gain, rstd, None, dx, dg, buf, 0, stream())
        sync()
        want = (dy.double() * x.double() * torch.rsqrt(x.double().square().mean(-1, keepdim=True) + 1e-5)).sum(0)
        assert float((dg.double() - want).abs().max()) < 1e-5 * float(want.abs().max())
        assert bool((buf[size:] == 0xA5).all())


@pytest.mark.parametrize("d,dtype,per_cu", [(512, "bf16", 5), (520, "bf16", 4), (1024, "bf16", 4), (504, "fp32", 4), (1032, "bf16", 5)])
def test_a_full_chip_is_one_round_of_blocks(d, dtype, per_cu):
    """A block leaves a row of partial sums; of the blocks that a CU holds at the kernel's registers there are one round, and no part of a second."""
    rows, (dt, code) = 11000, (torch.bfloat16, 1) if dtype == "bf16" else (torch.float32, 0)
    x, dy = (torch.randn(rows, d, device=DEV).to(dt) for _ in range(2))
    gain, rstd = torch.ones(d, device=DEV, dtype=dt), torch.ones(rows, device=DEV)
    dx, dg = torch.empty_like(x), torch.empty(d, device=DEV)
    part = torch.full((B.tide_rmsnorm_bwd_scratch_bytes(rows, d) // (4 * d), d), float("nan"), device=DEV)
    print(f"rmsnorm blocks d={d} {dtype}", flush=True)
    B.tide_rmsnorm_bwd(rows, d, dy, x, gain, rstd, None, dx, dg, part, code, stream())
    sync()
    assert int(torch.isfinite(part).all(1).sum()) == 256 * per_cu
