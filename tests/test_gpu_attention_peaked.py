"""One key in the second tile outweighs the first tile's: its probability relative to the row's maximum is exactly 1 and costs the result
no rounding of its own."""
import math

import pytest
import torch


@pytest.mark.gpu
@pytest.mark.parametrize("dh", [128, 64])
def test_the_probability_of_the_largest_score_is_not_rounded(dh):
    from paper_2602_05145_amd import binding as B
    b, nh, nkv, s = 64, 8, 8, 65
    g = torch.Generator(device="cuda").manual_seed(dh)
    u = torch.full((dh,), 0.25, device="cuda")
    gap = torch.rand(b, nh, device="cuda", generator=g) * 5.0 + 0.1                  # of the two scores, natural log
    k = torch.full((b, s, nkv, 1), -400.0, device="cuda")                            # the other keys weigh nothing
    k[:, 0] = 0.0
    k[:, 64, :, 0] = gap * math.sqrt(dh) / (dh * 0.25 * 0.25)
    q, k = u.expand(b, s, nh, dh), k * u
    v = torch.zeros(b, s, nkv, dh, device="cuda")
    v[:, 64] = torch.randn(b, nkv, dh, device="cuda", generator=g)
    qkv = torch.cat([x.reshape(b * s, -1) for x in (q, k, v)], 1).bfloat16().contiguous()
    out, lse = torch.empty(b * s, nh * dh, device="cuda", dtype=torch.bfloat16), torch.empty(b, nh, s, device="cuda")
    print("peaked attention", dh, flush=True)
    B.tide_attention_fwd(b, s, nh, nkv, dh, qkv, out, lse, 1, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    x = qkv.double().view(b, s, 3 * nh, dh)
    q, k, v = x[:, 64, :nh], x[:, 64, nh: 2 * nh], x[:, 64, 2 * nh:]
    score = (q * k).sum(-1) / math.sqrt(dh)
    want = v / (1 + torch.exp(-score))[..., None]
    got = out.view(b, s, nh, dh)[:, 64].double()
    # The result's own rounding: half a step of bf16, whose significand has 8 bits, so 2^-8 of the power of two below the value (up to 2^-8 of
    # the value itself).  Beside it a score, a float sum of dh products, is off by at most dh 2^-24 of itself (5 x 128 x 2^-24 < 2^-14, half of
    # which reaches the quotient), and a probability kept in two parts by 2^-16.  One bf16 probability that is no power of two adds up to 2^-8.
    half_step = torch.exp2(torch.floor(torch.log2(want.abs().clamp_min(1e-30))) - 8)
    excess = ((got - want).abs() - half_step) / want.abs().clamp_min(1e-30)
    print("beyond half a step, of the value:", float(excess.max()), flush=True)
    assert float(excess.max()) <= 2.0 ** -14
