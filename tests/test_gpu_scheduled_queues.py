"""The hand-scheduled attention kernel hands its query blocks out by workgroup id first and by counters behind that: fewer
blocks than workgroups, as many, one more, several rounds, queues of unequal length, rows of padding among the
dealt blocks, and captured launches that are replayed between direct ones (a launch finds its counters at zero whatever the ones
before it left).  A row of every query block is compared with 64 bits, in each mode that takes blocks from the counters."""
import numpy as np
import pytest
import torch

from paper_2605_20813_amd import pulsecol as pc
from parity_util import assert_close, f64, random_idx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MODES = ["sparse", "dense", "block"]


def _case(B, H, n, d, k, seed, mode="sparse"):
    """Q, K, V, and the pattern of the mode: column numbers, key-block numbers, none."""
    g = torch.Generator().manual_seed(seed)
    Q, K, V = (torch.randn(B, H, n, d, generator=g).to(torch.bfloat16) for _ in range(3))
    if mode == "dense":
        return Q, K, V, None
    entries = (n // 64, max(1, k // 64)) if mode == "block" else (n, k)
    return Q, K, V, random_idx(*entries, B * H, seed=seed + 1).view(B, H, 1, -1)


def _call(ctx, mode, q, k, v, idx, O):
    if mode == "dense":
        return ctx.attn_dense(q, k, v, O=O)
    return (ctx.attn_block if mode == "block" else ctx.attn)(q, k, v, idx, O=O)


def _columns(mode, idx, n):
    """Key positions of one head's pattern."""
    if mode == "dense":
        return np.arange(n)
    idx = idx[idx >= 0].numpy()
    return (idx[:, None] * 64 + np.arange(64)).ravel() if mode == "block" else idx


def _assert_a_row_of_every_block(O, Q, K, V, idx, mode, lens=None):
    B, H, n, d = Q.shape
    for b in range(B):
        length = lens[b] if lens else n
        each = np.arange(0, length, 256)
        each = np.minimum(each + 37 * (np.arange(each.size) + 1) % 256, length - 1)         # another row of each block
        for h in range(H):
            ends = np.r_[0:min(64, length), max(0, length - 64):length]                     # of the last head the first and last rows too
            rows = np.unique(np.r_[each, ends]) if h == H - 1 else each
            cols = _columns(mode, None if idx is None else idx[b, h, 0], n)
            q64, k64, v64 = f64(Q[b, h][rows]), f64(K[b, h][cols]), f64(V[b, h][cols])
            z = q64 @ k64.T / np.sqrt(d)
            p = np.exp(z - z.max(axis=1, keepdims=True))
            assert_close(O[b, h][torch.from_numpy(rows).to(O.device)], (p / p.sum(axis=1, keepdims=True)) @ v64, "bf16",
                         f"{mode}, element {b}, head {h}")


# blocks of 256 rows on 256 CUs: 1; 255 (five queues of five heads' worth); 256; 257 blocks of a single head; two uneven rounds
ROUNDS = [(1, 200), (5, 51 * 256), (8, 32 * 256), (1, 257 * 256), (9, 60 * 256 - 3)]


@pytest.mark.parametrize("mode,d,H,n", [
    *[("sparse", 128, H, n) for H, n in ROUNDS],
    ("sparse", 64, 5, 51 * 256), ("sparse", 64, 9, 60 * 256 - 3),
    ("block", 128, 5, 51 * 256), ("block", 64, 9, 60 * 256),
    ("dense", 128, 3, 5000), ("dense", 64, 9, 31 * 256 - 3),
])
def test_rounds_of_the_scheduled_kernel(mode, d, H, n):
    print(f"scheduled kernel, {mode}, D = {d}, {H} heads of {n} rows", flush=True)
    Q, K, V, idx = _case(1, H, n, d, 70, 4100 + H, mode)
    with pc.Context(1, H, n, d, torch.bfloat16) as ctx:
        ctx.set_attn_block(256)
        q, k_, v = (t.to(DEV) for t in (Q, K, V))
        ix = None if idx is None else idx.to(DEV)
        outs = []
        for _ in range(3):
            O = torch.full_like(q, float("nan"))
            _call(ctx, mode, q, k_, v, ix, O)
            outs.append(O)
        torch.cuda.synchronize()
    for O in outs:
        assert not torch.isnan(O.float()).any() and torch.equal(O, outs[0])
    _assert_a_row_of_every_block(outs[0], Q, K, V, idx, mode)


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
    _assert_a_row_of_every_block(outs[256], Q, K, V, idx, "sparse", lens)


@pytest.mark.parametrize("mode,d", [("sparse", 128), ("sparse", 64), ("dense", 128), ("block", 128)])
def test_replayed_launch(mode, d):
    B, H, n = 1, 9, 40 * 256
    print(f"scheduled kernel, captured, {mode}, D = {d}", flush=True)
    Q, K, V, idx = _case(B, H, n, d, 64, 4300, mode)
    with pc.Context(B, H, n, d, torch.bfloat16) as ctx:
        ctx.set_attn_block(256)
        q, k_, v = (t.to(DEV) for t in (Q, K, V))
        ix = None if idx is None else idx.to(DEV)
        want = _call(ctx, mode, q, k_, v, ix, torch.empty_like(q)).clone()
        O, O2 = torch.zeros_like(q), torch.zeros_like(q)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _call(ctx, mode, q, k_, v, ix, O)
            _call(ctx, mode, q, k_, v, ix, O2)          # two launches of one graph
        for rep in range(4):
            O.fill_(float("nan"))
            O2.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(O, want) and torch.equal(O2, want), f"replay {rep}"
            if rep % 2:
                eager = torch.full_like(q, float("nan"))
                assert torch.equal(_call(ctx, mode, q, k_, v, ix, eager), want)         # the program's own launches in between
        torch.cuda.synchronize()


def test_more_launches_than_sets_of_counters():
    """Launches of different sizes of work one behind the other, twenty on one context: each finds what an earlier one has cleared."""
    H, n, d = 3, 30 * 256, 128
    print("scheduled kernel, twenty launches in a row", flush=True)
    Q, K, V, idx = _case(1, H, n, d, 96, 4400)
    blocks = random_idx(n // 64, 2, H, seed=4402).view(1, H, 1, -1)
    with pc.Context(1, H, n, d, torch.bfloat16) as ctx:
        ctx.set_attn_block(256)
        q, k_, v = (t.to(DEV) for t in (Q, K, V))
        patterns = {"sparse": idx.to(DEV), "block": blocks.to(DEV), "dense": None}
        outs = [(m, _call(ctx, m, q, k_, v, patterns[m], torch.full_like(q, float("nan")))) for m in (["sparse", "block"] * 9 + ["dense"] + ["sparse"])]
        torch.cuda.synchronize()
    first = {}
    for m, O in outs:
        assert not torch.isnan(O.float()).any() and torch.equal(O, first.setdefault(m, O))
    _assert_a_row_of_every_block(first["sparse"], Q, K, V, idx, "sparse")
    _assert_a_row_of_every_block(first["block"], Q, K, V, blocks, "block")
