"""The scoring passes where the streamed range of a head is cut into runs (few heads, short contexts): run
boundaries at ragged ends, runs past the end, runs of whole query groups, and the row pass's way out when a row's
sum overflows.  Against the fp64 oracle; tolerance as in the other score tests."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from parity_util import f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rand_qk(B, H, n, d, dtype, seed):
    g = torch.Generator(device="cpu")
    g.manual_seed(seed)
    Q, K = (torch.randn(B, H, n, d, generator=g, dtype=torch.float32) for _ in range(2))
    K[:, :, ::13] *= 2.5
    return Q.to(dtype), K.to(dtype)


CASES = [
    # H, n, d, G: 64-row tiles and the runs they are cut into (bf16)
    (1, 511, 128, 0),      # 8 tiles: two runs, the second one ragged
    (1, 769, 64, 0),       # 13 tiles: three runs, one row in the last tile
    (2, 2049, 128, 0),     # 33 tiles, 8 runs of 5: the last run lies past the end
    (1, 2049, 64, 0),
    (1, 500, 128, 32),     # runs of two groups (a group ends inside a tile)
    (2, 777, 64, 96),      # ... of 96 rows: three tiles, ragged last group
    (1, 1030, 128, 256),   # fewer groups than runs would fit
]


@pytest.mark.parametrize("H,n,d,G", CASES)
def test_split_scores_match_oracle(H, n, d, G):
    print(f"split scores H={H} n={n} d={d} G={G}", flush=True)
    Q, K = rand_qk(1, H, n, d, torch.bfloat16, seed=n + d + G)
    with pc.Context(1, H, n, d, torch.bfloat16, group_size=G) as ctx:
        got = f64(ctx.scores(Q.to(DEV), K.to(DEV)))[0]
    for h in range(H):
        want = oracle.column_scores(f64(Q[0, h]), f64(K[0, h]), group_size=G)
        assert np.abs(got[h].sum(axis=-1) - 1.0).max() < 1e-5
        assert (np.abs(got[h] - want) / want).max() < 2e-5


@pytest.mark.parametrize("H,n,d", [(40, 2000, 64), (36, 4100, 128)])
def test_runs_of_grids_larger_than_half_the_chip(H, n, d):
    """Three runs per block where 320 blocks would fill part of the chip only, two where 612 blocks would leave most
    of it idle in the last round.  First and last head against the oracle, every head's sum, and the entry point without
    allocations, which cuts the shape alike, against the context."""
    print(f"split scores H={H} n={n} d={d}", flush=True)
    Q, K = rand_qk(1, H, n, d, torch.bfloat16, seed=H)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    with pc.Context(1, H, n, d, torch.bfloat16) as ctx:
        got = f64(ctx.scores(Qd, Kd))[0, :, 0]
        kept = ctx.select(Qd, Kd, 0.1)
    same = torch.empty_like(kept)
    pc.select_noalloc(pc.make_shape(1, H, n, d, torch.bfloat16), Qd, Kd, 0.1, same)
    assert torch.equal(same, kept)
    assert np.abs(got.sum(axis=-1) - 1.0).max() < 1e-5
    for h in (0, H - 1):
        want = oracle.column_scores(f64(Q[0, h]), f64(K[0, h]))[0]
        assert (np.abs(got[h] - want) / want).max() < 2e-5


def test_runs_past_the_end_of_a_short_batch_element():
    n, lens, d = 2049, (2049, 70, 1), 128
    print(f"split scores n={n} lens={lens}", flush=True)
    Q, K = rand_qk(3, 1, n, d, torch.bfloat16, seed=11)
    for b, length in enumerate(lens):
        Q[b, :, length:] = float("nan")
        K[b, :, length:] = float("nan")
    with pc.Context(3, 1, n, d, torch.bfloat16) as ctx:
        ctx.set_seq_lens(lens)
        sc = torch.full((3, 1, 1, n), -7.0, device=DEV)
        got = f64(ctx.scores(Q.to(DEV), K.to(DEV), scores_out=sc))[:, 0, 0]
    for b, length in enumerate(lens):
        want = oracle.column_scores(f64(Q[b, 0, :length]), f64(K[b, 0, :length]))[0]
        assert (np.abs(got[b, :length] - want) / want).max() < 2e-5
        assert (got[b, length:] == -7.0).all()


@pytest.mark.parametrize("n,d", [(300, 128), (1500, 64)])
def test_row_sums_that_overflow(n, d):
    """Logits that rise more than 127 log2 units above a row's first 32 (for half of the rows; the other half falls)."""
    print(f"overflowing row sums n={n} d={d}", flush=True)
    Q, K = rand_qk(1, 1, n, d, torch.float32, seed=n)
    lift = torch.zeros(n)
    lift[40:] = torch.linspace(0.0, 240.0, n - 40)                       # natural-log units, d^0.5 per unit of K[..., 0]
    Q[..., 0] = torch.where(torch.arange(n) % 2 == 0, 1.0, -1.0)
    K[..., 0] = lift * d ** 0.5
    Q, K = Q.to(torch.bfloat16), K.to(torch.bfloat16)
    with pc.Context(1, 1, n, d, torch.bfloat16) as ctx:
        got = f64(ctx.scores(Q.to(DEV), K.to(DEV)))[0, 0, 0]
    want = oracle.column_scores(f64(Q[0, 0]), f64(K[0, 0]))[0]
    # fp32 dot products of magnitude M = 240 d^0.5 carry an absolute error of some 2^-24 M d^0.5 (rounding of a running
    # sum), times the scale d^-0.5: 240 d^0.5 2^-24 = 1.6e-4 of a weight, relative
    assert abs(got.sum() - 1.0) < 1e-3
    assert np.abs(got - want).max() <= 1e-3 * want.max()
