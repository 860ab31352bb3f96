"""The fp32 kernels whose waves share out the tiles of a 32-row (32-key) block: fewer tiles than waves, tile counts
around multiples of the wave count, ragged ends, both workgroup sizes and the line to the 128-row kernels.  Against the
fp64 oracle, tolerances of the fp32 mode."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from parity_util import assert_close, f64, random_idx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # H, n, d, G, k
    (1, 1, 64, 0, 1),
    (2, 33, 128, 0, 31),       # one or two tiles for eight or four waves
    (2, 129, 64, 0, 97),
    (3, 255, 128, 0, 255),
    (2, 289, 128, 128, 160),   # three groups of four tiles, the last one ragged
    (1, 700, 64, 256, 130),
    (9, 1000, 64, 0, 200),     # more blocks than CUs: four waves
    (5, 2040, 128, 0, 300),
    (33, 1024, 64, 0, 64),     # the 128-row kernels
]


@pytest.mark.parametrize("H,n,d,G,k", CASES)
def test_f32_against_the_oracle(H, n, d, G, k):
    print(f"f32 split H={H} n={n} d={d} G={G} k={k}", flush=True)
    g = torch.Generator(device="cpu")
    g.manual_seed(n + d + k)
    Q, K, V = (torch.randn(1, H, n, d, generator=g) for _ in range(3))
    with pc.Context(1, H, n, d, torch.float32, group_size=G) as ctx:
        U = ctx.groups
        idx = random_idx(n, k, H * U, seed=n).view(1, H, U, k)
        q, k_, v = Q.to(DEV), K.to(DEV), V.to(DEV)
        sc = f64(ctx.scores(q, k_))[0]
        O = ctx.attn(q, k_, v, idx.to(DEV))
        lse = torch.empty(1, H, n, device=DEV)
        Od = ctx.attn_dense(q, k_, v, lse_out=lse)
        torch.cuda.synchronize()
    for h in sorted({0, H - 1}):
        qh, kh, vh = f64(Q[0, h]), f64(K[0, h]), f64(V[0, h])
        want = oracle.column_scores(qh, kh, group_size=G)
        assert (np.abs(sc[h] - want) / want).max() < 2e-5
        assert_close(O[0, h], oracle.sparse_attention_masked(qh, kh, vh, idx[0, h].numpy(), group_size=G), "f32", "sparse")
        assert_close(Od[0, h], oracle.dense_attention(qh, kh, vh), "f32", "dense")
        Z = oracle.attention_logits(qh, kh)
        top = Z.max(axis=1)
        assert np.abs(f64(lse[0, h]) - (top + np.log(np.exp(Z - top[:, None]).sum(axis=1)))).max() < 1e-5
