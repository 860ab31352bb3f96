"""Shapes on the far side of the lines that send small calls to other kernels: the 128-row fp32 kernels (ragged rows and
tiles, query groups, grouped-query K/V, a padded batch, steep logits), the plain attention kernel with one team and lists of
blocks on steep logits, and the streaming top-k (padded batches, the cached pattern).  Against the fp64 oracle, on sampled heads
and rows."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from paper_2605_20813_amd import workloads as wl
from parity_util import assert_close, f64, random_idx
from test_gpu_logit_range import steep_qkv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check_f32(Q, K, V, G, k, lens=None, rel=2e-5):
    """Scores, column-sparse and dense attention of a context, first and last element and head."""
    B, H, n, d = Q.shape
    Hkv = K.shape[1]
    lens = lens or [n] * B
    kept = [max(1, k * L // n) for L in lens]
    rng = np.random.default_rng(n)
    with pc.Context(B, H, n, d, torch.float32, group_size=G, kv_heads=Hkv if Hkv != H else 0) as ctx:
        U = ctx.groups
        idx = torch.full((B, H, U, k), -1, dtype=torch.int32)
        for b in range(B):
            Ub = U if U == 1 else -(-lens[b] // G)
            idx[b, :, :Ub, :kept[b]] = random_idx(lens[b], kept[b], H * Ub, seed=n + b).view(H, Ub, kept[b])
        if min(lens) < n:
            ctx.set_seq_lens(lens)
        assert ctx.tile_shape(k)[0] == 128
        q, k_, v = Q.to(DEV), K.to(DEV), V.to(DEV)
        sc, O = ctx.scores(q, k_), ctx.attn(q, k_, v, idx.to(DEV))
        lse = torch.empty(B, H, n, device=DEV)
        Od = ctx.attn_dense(q, k_, v, lse_out=lse)
        torch.cuda.synchronize()
    for b, h in sorted({(0, 0), (B - 1, H - 1)}):
        L, hk = lens[b], h * Hkv // H
        qh, kh, vh = f64(Q[b, h, :L]), f64(K[b, hk, :L]), f64(V[b, hk, :L])
        want = oracle.column_scores(qh, kh, group_size=G)
        got = f64(sc[b, h])[:want.shape[0], :L]
        big = want > 1e-6 * want.max()
        assert (np.abs(got - want)[big] / want[big]).max() < rel
        rows = np.unique(np.concatenate([[0, L - 1, min(127, L - 1), min(128, L - 1), (L - 1) // 128 * 128], rng.integers(0, L, 40)]))
        assert_close(O[b, h][rows], oracle.sparse_attention_masked(qh, kh, vh, idx[b, h, :want.shape[0], :kept[b]].numpy(),
                                                                   group_size=G, rows=rows), "f32", f"sparse b={b} h={h}")
        assert_close(Od[b, h][rows], oracle.dense_attention(qh, kh, vh, rows=rows), "f32", f"dense b={b} h={h}")
        Z = oracle.attention_logits(qh, kh)[rows]
        top = Z.max(axis=1)
        want_lse = top + np.log(np.exp(Z - top[:, None]).sum(axis=1))
        assert np.abs(f64(lse[b, h])[rows] - want_lse).max() < 2e-5 * max(1.0, np.abs(want_lse).max())


@pytest.mark.parametrize("B,H,Hkv,n,d,G,k,lens", [
    (1, 17, 17, 2043, 128, 0, 301, None),
    (1, 17, 17, 2043, 128, 128, 300, None),
    (1, 18, 6, 2043, 64, 0, 333, None),
    (1, 18, 3, 2000, 128, 256, 97, None),
    (3, 12, 12, 1500, 128, 0, 200, [1500, 777, 33]),
    (3, 12, 4, 1500, 64, 128, 200, [1500, 130, 1400]),
])
def test_128_row_f32_kernels(B, H, Hkv, n, d, G, k, lens):
    print(f"128-row f32 B={B} H={H} Hkv={Hkv} n={n} d={d} G={G}", flush=True)
    g = torch.Generator(device="cpu")
    g.manual_seed(n + d + G)
    Q = torch.randn(B, H, n, d, generator=g)
    K, V = (torch.randn(B, Hkv, n, d, generator=g) for _ in range(2))
    if lens:
        for b, L in enumerate(lens):
            for t in (Q, K, V):
                t[b, :, L:] = float("nan")
    check_f32(Q, K, V, G, k, lens)


@pytest.mark.parametrize("shape", ["up", "down", "late", "saw"])
@pytest.mark.parametrize("d", [64, 128])
def test_128_row_f32_kernels_with_steep_logits(shape, d):
    """(the span and the tolerance of the scores as in test_gpu_logit_range.py)"""
    print(f"128-row f32 steep {shape} d={d}", flush=True)
    Q, K, V = steep_qkv(1, 17, 2001, d, torch.float32, seed=d, shape=shape, span=25.0)
    check_f32(Q, K, V, 0, 300, rel=2e-4)


@pytest.mark.parametrize("shape", ["up", "down", "late", "saw"])
@pytest.mark.parametrize("d,G", [(128, 0), (64, 0), (128, 128)])
def test_plain_attention_kernel_with_one_team_and_steep_logits(shape, d, G):
    H, n, k = 20, 2000, 300
    print(f"plain kernel, one team, steep {shape} d={d} G={G}", flush=True)
    Q, K, V = steep_qkv(1, H, n, d, torch.bfloat16, seed=d + G, shape=shape, span=60.0 if d == 128 else 40.0)
    U = 1 if G == 0 else -(-n // G)
    idx = random_idx(n, k, H * U, seed=n).view(1, H, U, k)
    with pc.Context(1, H, n, d, torch.bfloat16, group_size=G) as ctx:
        ctx.set_attn_block(128)
        O = ctx.attn(Q.to(DEV), K.to(DEV), V.to(DEV), idx.to(DEV))
        torch.cuda.synchronize()
    rows = np.unique(np.concatenate([[0, 127, 128, n - 1, (n - 1) // 128 * 128], np.random.default_rng(d).integers(0, n, 60)]))
    for h in (0, 7, H - 1):
        want = oracle.sparse_attention_masked(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h]), idx[0, h].numpy(), group_size=G, rows=rows)
        assert_close(O[0, h][rows], want, "bf16", f"{shape} h={h}")


def test_streaming_topk_in_a_padded_batch():
    B, H, n, k, lens = 3, 2, 65541, 6000, (65541, 40000, 3)
    print("streaming top-k, padded batch", flush=True)
    scores = wl.random_scores(B * H, n, seed=3, ties=True).view(B, H, 1, n)
    for b, L in enumerate(lens):
        scores[b, :, :, L:] = float("nan")
    with pc.Context(B, H, n, 64, torch.bfloat16, max_keep_ratio=0.1) as ctx:
        ctx.set_seq_lens(lens)
        idx = ctx.topk(scores.to(DEV), k).cpu().numpy()
    for b, L in enumerate(lens):
        kb = min(k, L)
        for h in range(H):
            assert np.array_equal(idx[b, h, 0, :kb], oracle.topk_columns(f64(scores[b, h, 0, :L])[None], kb)[0])
            assert (idx[b, h, 0, kb:] == -1).all()


@pytest.mark.parametrize("lens", [None, (65600, 700)])
def test_streaming_topk_writes_the_cached_pattern(lens):
    B, H, n, d, keep = (len(lens) if lens else 1), 1, 65600, 64, 0.05
    print(f"streaming top-k, cached pattern lens={lens}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    Q, K = (torch.randn(B, H, n, d, device=DEV, generator=g).to(torch.bfloat16) for _ in range(2))
    with pc.Context(B, H, n, d, torch.bfloat16, max_keep_ratio=keep) as ctx:
        if lens:
            ctx.set_seq_lens(lens)
        sc = f64(ctx.scores(Q, K))
        idx = ctx.select(Q, K, keep)
        again = ctx.select(None, None, keep, refresh=False)
        torch.cuda.synchronize()
    assert torch.equal(idx, again)
    for b in range(B):
        L = lens[b] if lens else n
        kb = oracle.num_keep(L, keep)
        assert np.array_equal(idx[b, 0, 0, :kb].cpu().numpy(), oracle.topk_columns(sc[b, 0, :, :L], kb)[0])
        assert (idx[b, 0, 0, kb:] == -1).all()
