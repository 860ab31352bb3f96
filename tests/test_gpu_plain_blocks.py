"""The plain column-sparse kernel where a workgroup works through several 128-row blocks (more of them than the chip
holds at a time) and where two teams share a block: every remainder of the tile count by the tile slots, ragged last
blocks, a ragged batch.  Against the fp64 oracle on sampled rows."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from parity_util import assert_close, f64, random_idx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run(B, H, n, d, k, lens=None, seed=0):
    g = torch.Generator(device="cpu")
    g.manual_seed(seed + n + k)
    Q, K, V = (torch.randn(B, H, n, d, generator=g).to(torch.bfloat16) for _ in range(3))
    idx = torch.full((B, H, 1, k), -1, dtype=torch.int32)
    kept = [max(1, k * L // n) for L in (lens or [n] * B)]
    for b in range(B):
        idx[b, :, 0, :kept[b]] = random_idx((lens or [n] * B)[b], kept[b], H, seed=seed + b)
    with pc.Context(B, H, n, d, torch.bfloat16) as ctx:
        ctx.set_attn_block(128)
        if lens:
            ctx.set_seq_lens(lens)
        O = ctx.attn(Q.to(DEV), K.to(DEV), V.to(DEV), idx.to(DEV))
        torch.cuda.synchronize()
    rng = np.random.default_rng(seed)
    for b in range(B):
        L = lens[b] if lens else n
        for h in sorted({0, H // 2 + 1, H - 1} & set(range(H))):
            rows = np.unique(np.concatenate([[0, L - 1, min(128, L - 1), (L - 1) // 128 * 128], rng.integers(0, L, 24)]))
            want = oracle.sparse_attention_masked(f64(Q[b, h, :L]), f64(K[b, h, :L]), f64(V[b, h, :L]),
                                                  idx[b, h, :, :kept[b]].numpy(), rows=rows)
            assert_close(O[b, h][rows], want, "bf16", f"n={n} d={d} k={k} b={b} h={h}")


@pytest.mark.parametrize("k", [1, 20, 41, 70, 128, 150])         # 1, 1, 2, 3, 4, 5 tiles
@pytest.mark.parametrize("H,n,d", [(32, 4100, 128), (20, 8200, 64)])
def test_several_blocks_per_workgroup(H, n, d, k):
    print(f"plain blocks H={H} n={n} d={d} k={k}", flush=True)
    run(1, H, n, d, k)


def test_several_blocks_per_workgroup_in_a_ragged_batch():
    print("plain blocks, ragged batch", flush=True)
    run(3, 20, 4100, 128, 130, lens=[4100, 2050, 77])


@pytest.mark.parametrize("k", [128, 129, 161, 224])              # 4, 5, 6, 7 tiles: the teams' shares even and uneven
@pytest.mark.parametrize("H,n,d", [(3, 500, 128), (2, 333, 64)])
def test_two_teams_per_block(H, n, d, k):
    print(f"two teams H={H} n={n} d={d} k={k}", flush=True)
    run(1, H, n, d, k)


@pytest.mark.parametrize("H,n,d,k,copies", [(2, 1000, 128, 200, 20), (3, 500, 128, 161, 30), (2, 333, 64, 129, 50)])
def test_two_teams_form_the_weights_that_one_team_forms(H, n, d, k, copies):
    """The same heads alone (two teams per block) and many times over in one launch (one team).  The weights and their
    16-bit roundings are the same in both, the fp32 sums run in another order: relative differences of some 1e-6 move a
    rounding boundary of the output under about 1e-6 / 2^-8 of the values, by 2^-8 of the value, 6e-5 of the norm.  (Weights
    rounded against two references differ by some 2e-3.)"""
    print(f"two teams against one H={H} n={n} d={d} k={k}", flush=True)
    g = torch.Generator(device="cpu")
    g.manual_seed(n + k)
    Q, K, V = (torch.randn(1, H, n, d, generator=g).to(torch.bfloat16).to(DEV) for _ in range(3))
    idx = random_idx(n, k, H, seed=n).view(1, H, 1, k).to(DEV)
    outs = []
    for r in (1, copies):
        with pc.Context(1, H * r, n, d, torch.bfloat16) as ctx:
            ctx.set_attn_block(128)
            assert (H * r * -(-n // 128) <= 256) == (r == 1)
            O = ctx.attn(*(t.repeat(1, r, 1, 1).contiguous() for t in (Q, K, V)), idx.repeat(1, r, 1, 1).contiguous())
            torch.cuda.synchronize()
        outs.append(f64(O[0, :H]))
    assert np.linalg.norm(outs[0] - outs[1]) <= 5e-4 * np.linalg.norm(outs[1])


@pytest.mark.parametrize("k", [1, 20, 33, 70, 100, 129, 170, 200, 230, 300])         # 1 to 10 tiles
@pytest.mark.parametrize("d", [128, 64])
def test_two_wave_blocks(d, k):
    """Groups of 64 rows: at D = 128 two V slots instead of three, every tile count up to the second round of the unrolled
    iterations, a ragged last group."""
    H, n, G = 2, 333, 64
    print(f"two-wave blocks d={d} k={k}", flush=True)
    g = torch.Generator(device="cpu")
    g.manual_seed(d + k)
    Q, K, V = (torch.randn(1, H, n, d, generator=g).to(torch.bfloat16) for _ in range(3))
    U = -(-n // G)
    idx = random_idx(n, k, H * U, seed=k).view(1, H, U, k)
    with pc.Context(1, H, n, d, torch.bfloat16, group_size=G) as ctx:
        O = ctx.attn(Q.to(DEV), K.to(DEV), V.to(DEV), idx.to(DEV))
        torch.cuda.synchronize()
    for h in range(H):
        want = oracle.sparse_attention_masked(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h]), idx[0, h].numpy(), group_size=G)
        assert_close(O[0, h], want, "bf16", f"d={d} k={k} h={h}")
