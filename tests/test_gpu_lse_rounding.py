"""Row log-sum-exp of the bf16 dense kernel against 64 bits, rows of a few flat logits: its reference lies eight log2 units above the
first maximum, so that the sum of the weights is small, and its exponent has to go into the reference before the logarithm is rounded."""
import math

import pytest
import torch

from paper_2605_20813_amd import pulsecol as pc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [17, 30])
def test_log_sum_exp_of_short_flat_rows(d, n):
    H = 64
    print(f"log-sum-exp of {n} rows, D = {d}", flush=True)
    g = torch.Generator().manual_seed(7 * n + d)
    Q, K, V = (torch.randn(1, H, n, d, generator=g) for _ in range(3))
    Q, K, V = Q.to(torch.bfloat16), (0.1 * K).to(torch.bfloat16), V.to(torch.bfloat16)
    lse = torch.empty(1, H, n, device=DEV)
    with pc.Context(1, H, n, d, torch.bfloat16) as ctx:
        ctx.attn_dense(Q.to(DEV), K.to(DEV), V.to(DEV), lse_out=lse)
        torch.cuda.synchronize()
    want = torch.logsumexp(Q[0].double() @ K[0].double().transpose(1, 2).contiguous() / math.sqrt(d), -1)
    rms = (lse[0].cpu().double() - want).square().mean().sqrt().item()
    # log2 units: reference plus exponent, and that plus a logarithm below one, are rounded between 4 and 8 (unit 4.8e-7, rms of a
    # rounding 0.29 of it), the shifted logits between 8 and 16 (9.5e-7, averaged over the keys); then times ln 2, rounded between 2 and 4 (2.4e-7)
    rounding = 0.29 * 4.8e-7
    bound = math.hypot(math.log(2) * math.sqrt(2 * rounding ** 2 + 4 * rounding ** 2 / n), 0.29 * 2.4e-7)
    assert rms <= bound, f"{rms:.2e} > {bound:.2e}"
