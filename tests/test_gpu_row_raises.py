"""The row pass raises a row's reference by that row's own sums: a row's log-sum-exp, and with it the bits of its head's scores, does
not depend on the rows that share its wave (64 of them in blocks of 256 rows, 32 in blocks of 128)."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from parity_util import f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("H,n,d", [(2, 500, 128), (2, 513, 64), (24, 1000, 128), (40, 1000, 64), (24, 1217, 128)])
def test_bits_of_scores_whose_references_rise_late(H, n, d):
    """Every 37th query meets a key of its own, late in the head, that outgrows its reference; its neighbours do not."""
    print(f"row raises H={H} n={n} d={d}", flush=True)
    long = 4100
    g = torch.Generator(device="cpu")
    g.manual_seed(n + d)
    Q, K = (torch.randn(2, H, long, d, generator=g) for _ in range(2))
    rows = torch.arange(5, n, 37)
    keys = n - 1 - 3 * torch.arange(len(rows))
    K[1, :, keys] = Q[1, :, rows] * (13.0 * d ** 0.5 / (Q[1, :, rows] ** 2).sum(-1, keepdim=True))
    Q, K = (t.to(torch.bfloat16).to(DEV) for t in (Q, K))
    q, k = Q[1:, :, :n].contiguous(), K[1:, :, :n].contiguous()
    with pc.Context(1, H, n, d, torch.bfloat16) as ctx:
        alone = ctx.scores(q, k)[0]
    with pc.Context(2, H, long, d, torch.bfloat16) as ctx:
        ctx.set_seq_lens([long, n])
        among = ctx.scores(Q, K)[1]
        torch.cuda.synchronize()
    assert torch.equal(alone[:, 0], among[:, 0, :n])
    want = oracle.column_scores(f64(q[0, H - 1]), f64(k[0, H - 1]))
    assert (np.abs(f64(alone[H - 1]) - want) / want).max() < 2e-5
