"""The hand-scheduled attention kernel hands its query blocks out by workgroup id first and by counters behind that: fewer
blocks than workgroups, as many, one more, several rounds, queues of unequal length, rows of padding among the
dealt blocks, and a captured launch that is replayed (the counters are zero again after every launch)."""
import numpy as np
import pytest
import torch

from paper_2605_20813_amd import pulsecol as pc
from parity_util import assert_close, f64, random_idx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _case(B, H, n, d, k, seed):
    g = torch.Generator().manual_seed(seed)
    Q, K, V = (torch.randn(B, H, n, d, generator=g).to(torch.bfloat16) for _ in range(3))
    idx = random_idx(n, k, B * H, seed=seed + 1).view(B, H, 1, k)
    return Q, K, V, idx


# blocks of 256 rows on 256 CUs: 1; 255 (five queues of five heads' worth); 256; 257 blocks of a single head; two uneven rounds
@pytest.mark.parametrize("H,n", [(1, 200), (5, 51 * 256), (8, 32 * 256), (1, 257 * 256), (9, 60 * 256 - 3)])
def test_rounds_of_the_scheduled_kernel(H, n):
    k, d = 70, 128
    print(f"scheduled kernel, {H} heads of {n} rows", flush=True)
    Q, K, V, idx = _case(1, H, n, d, k, 4100 + H)
    with pc.Context(1, H, n, d, torch.bfloat16) as ctx:
        ctx.set_attn_block(256)
        q, k_, v, ix = (t.to(DEV) for t in (Q, K, V, idx))
        outs = []
        for _ in range(3):
            O = torch.full_like(q, float("nan"))
            ctx.attn(q, k_, v, ix, O)
            outs.append(O)
        torch.cuda.synchronize()
    for O in outs:
        assert not torch.isnan(O.float()).any() and torch.equal(O, outs[0])
    rows = torch.cat([torch.arange(0, min(n, 64)), torch.arange(max(0, n - 64), n)])        # first and last rows of the last head
    q64, k64, v64 = f64(Q[0, H - 1]), f64(K[0, H - 1]), f64(V[0, H - 1])
    cols = idx[0, H - 1, 0].numpy()
    z = q64[rows.numpy()] @ k64[cols].T / np.sqrt(d)
    p = np.exp(z - z.max(axis=1, keepdims=True))
    assert_close(outs[0][0, H - 1][rows.to(DEV)], (p / p.sum(axis=1, keepdims=True)) @ v64[cols], "bf16", "rounds")


def test_padding_among_the_dealt_blocks():
    B, H, n, d, k = 3, 4, 30 * 256, 128, 60
    lens = (300, n, 1)
    print("scheduled kernel, ragged batch", flush=True)
    Q, K, V, _ = _case(B, H, n, d, k, 4200)
    idx = torch.full((B, H, 1, k), -1, dtype=torch.int32)
    for b, L in enumerate(lens):
        idx[b, :, 0, :min(k, L)] = random_idx(L, min(k, L), H, seed=50 + b).view(H, -1)
    with pc.Context(B, H, n, d, torch.bfloat16) as ctx:
        ctx.set_seq_lens(lens)
        q, k_, v, ix = (t.to(DEV) for t in (Q, K, V, idx))
        outs = {}
        for bm in (256, 128, 256):
            ctx.set_attn_block(bm)
            O = torch.full_like(q, 7.0)
            ctx.attn(q, k_, v, ix, O)
            if bm in outs:
                assert torch.equal(outs[bm], O)
            outs[bm] = O
        torch.cuda.synchronize()
    for b, L in enumerate(lens):
        assert (outs[256][b, :, L:] == 7.0).all()
        # the same weights in either kernel but for the reference: two bf16 roundings of O(1) outputs apart
        assert (outs[256][b, :, :L].float() - outs[128][b, :, :L].float()).abs().max() <= 2e-2


def test_replayed_launch():
    B, H, n, d, k = 1, 9, 40 * 256, 128, 64
    print("scheduled kernel, captured", flush=True)
    Q, K, V, idx = _case(B, H, n, d, k, 4300)
    with pc.Context(B, H, n, d, torch.bfloat16) as ctx:
        ctx.set_attn_block(256)
        q, k_, v, ix = (t.to(DEV) for t in (Q, K, V, idx))
        want = ctx.attn(q, k_, v, ix).clone()
        O = torch.zeros_like(q)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ctx.attn(q, k_, v, ix, O)
        for rep in range(4):
            O.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(O, want), f"replay {rep}"
            if rep == 1:
                assert torch.equal(ctx.attn(q, k_, v, ix), want)         # the program's own launches in between
        torch.cuda.synchronize()
