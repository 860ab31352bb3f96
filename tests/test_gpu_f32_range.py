"""fp32 mode outside the range in which three bf16 parts carry a number: small numbers of Q and K against large ones of the other (or
a large scale), small V, large V under weights that are next to nothing."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from parity_util import f64, random_idx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# factors of Q and K, and what is left for the scale: parts of the smaller one flushed in part, altogether; the scale alone
FACTORS = [(2.0 ** 112, 2.0 ** -112, 1.0), (2.0 ** -112, 2.0 ** 112, 1.0), (2.0 ** 118, 2.0 ** -118, 1.0), (2.0 ** -119, 2.0 ** 119, 1.0), (2.0 ** -60, 2.0 ** -60, 2.0 ** 120),
           (2.0 ** 124, 2.0 ** -124, 1.0), (1.0, 2.0 ** -116, 2.0 ** 116), (2.0 ** 40, 2.0 ** -40, 1.0), (2.0 ** 55, 2.0 ** -55, 1.0), (2.0 ** 40, 2.0 ** 30, 2.0 ** -70)]


def tensors(H, n, d, seed):
    g = torch.Generator(device="cpu")
    g.manual_seed(seed)
    return [torch.randn(1, H, n, d, generator=g) for _ in range(3)]


# A power of two changes no digit of an ordinary fp32 product.  The error of a weight is that of its logit: 2^-24 sqrt(d) of a few units,
# 2e-6 (4e-7 measured in a mean over some hundred rows); the parts lose that much from factors of 2^114 on.
@pytest.mark.parametrize("fq,fk,fs", FACTORS)
@pytest.mark.parametrize("H,n,d,G", [(2, 1100, 128, 0), (2, 1100, 64, 0), (40, 700, 128, 0), (2, 1300, 128, 256), (2, 300, 64, 0)])
def test_scores_of_scaled_queries_and_keys(H, n, d, G, fq, fk, fs):
    print(f"f32 range scores H={H} n={n} d={d} G={G} {fq} {fk} {fs}", flush=True)
    Q, K, _ = tensors(H, n, d, n + d)
    with pc.Context(1, H, n, d, torch.float32, group_size=G, scale=fs / d ** 0.5) as ctx:
        sc = f64(ctx.scores((Q * fq).to(DEV), (K * fk).to(DEV)))[0]
    for h in sorted({0, H - 1}):
        want = oracle.column_scores(f64(Q[0, h]), f64(K[0, h]), group_size=G)
        assert (np.abs(sc[h] - want) / want).max() < 2e-6


@pytest.mark.parametrize("which", ["Q", "K"])
def test_scores_of_one_large_number(which):
    """One element of Q or K beyond the range, in a head whose other columns are small: all columns of its row's segment."""
    n, d = 1500, 128
    print("f32 range scores, one large number", which, flush=True)
    Q, K, _ = tensors(1, n, d, 2)
    small, large = (K, Q) if which == "Q" else (Q, K)
    small[..., 7] *= 2.0 ** -110
    large[0, 0, 701, 7] = 2.0 ** 110
    with pc.Context(1, 1, n, d, torch.float32) as ctx:
        sc = f64(ctx.scores(Q.to(DEV), K.to(DEV)))[0, 0, 0]
    want = oracle.column_scores(f64(Q[0, 0]), f64(K[0, 0]))[0]
    assert (np.abs(sc - want) / want).max() < 2e-6


SHAPES = [(2, 300, 128, 77), (2, 300, 64, 77), (40, 700, 128, 225), (70, 520, 64, 129)]       # workgroups of 32 rows, of 128


def attention(Q, K, V, idx, scale=0.0):
    """Sparse and dense attention and the row log-sum-exp, in 64 bits: (got, wanted) of the first and the last head."""
    _, H, n, d = Q.shape
    k = idx.shape[1]
    with pc.Context(1, H, n, d, torch.float32, scale=scale) as ctx:
        q, k_, v = Q.to(DEV), K.to(DEV), V.to(DEV)
        O = ctx.attn(q, k_, v, idx.view(1, H, 1, k).to(DEV))
        lse = torch.empty(1, H, n, device=DEV)
        Od = ctx.attn_dense(q, k_, v, lse_out=lse)
        torch.cuda.synchronize()
    factor = scale * d ** 0.5 if scale else 1.0
    for h in sorted({0, H - 1}):
        qh, kh, vh, cols = f64(Q[0, h]) * factor, f64(K[0, h]), f64(V[0, h]), idx[h].numpy()
        Z = oracle.attention_logits(qh, kh)
        top = Z.max(axis=1)
        yield [(f64(O[0, h]), oracle.dense_attention(qh, kh[cols], vh[cols])), (f64(Od[0, h]), oracle.dense_attention(qh, kh, vh)),
               (f64(lse[0, h])[:, None], (top + np.log(np.exp(Z - top[:, None]).sum(axis=1)))[:, None])]


def columns_off(got, want):
    return (np.linalg.norm(got - want, axis=0) / np.linalg.norm(want, axis=0)).max()


# (an output hangs on fewer weights than a score: twice the bound)
@pytest.mark.parametrize("fq,fk,fs", FACTORS)
@pytest.mark.parametrize("H,n,d,k", SHAPES)
def test_attention_of_scaled_queries_and_keys(H, n, d, k, fq, fk, fs):
    print(f"f32 range attention H={H} n={n} d={d} k={k} {fq} {fk} {fs}", flush=True)
    Q, K, V = tensors(H, n, d, n + d + k)
    for pairs in attention(Q * fq, K * fk, V, random_idx(n, k, H, seed=n), fs / d ** 0.5):
        for got, want in pairs:
            assert columns_off(got, want) < 4e-6


@pytest.mark.parametrize("H,n,d,k", SHAPES)
def test_attention_of_one_large_key(H, n, d, k):
    """An element of one kept key beyond the range, against queries that are small there."""
    print(f"f32 range attention, one large key H={H} n={n} d={d} k={k}", flush=True)
    Q, K, V = tensors(H, n, d, n + d)
    idx = random_idx(n, k, H, seed=n)
    Q[..., 7] *= 2.0 ** -110
    for h in range(H):
        K[0, h, idx[h, k // 2].long(), 7] = 2.0 ** 110
    for pairs in attention(Q, K, V, idx):
        for got, want in pairs:
            assert columns_off(got, want) < 4e-6


# One column of V small, one zero, the others ordinary.  Sums of numbers below 2^-126 are rounded to multiples of 2^-149: the fp32 instruction's
# n / 2 times, by a third of one each, sqrt(n / 2) / 3 = 6 of them over 700 rows, and divided by the sum of the weights, ten and more; the
# result once more.  Four allowed.
@pytest.mark.parametrize("exponent", [-144, -141, -136, -133, -130, -126, -120, -100])
@pytest.mark.parametrize("H,n,d,k", SHAPES)
def test_small_values(H, n, d, k, exponent):
    print(f"f32 range, small values H={H} n={n} d={d} k={k} 2^{exponent}", flush=True)
    Q, K, V = tensors(H, n, d, n + d)
    V[..., 3] = (1.0 + V[..., 3].abs()) * 2.0 ** exponent
    V[..., 4] = 0.0
    for pairs in attention(Q, K, V, random_idx(n, k, H, seed=n)):
        for got, want in pairs[:2]:
            assert (got[:, 4] == 0.0).all()
            assert (np.abs(got[:, 3] - want[:, 3]) <= 2e-5 * want[:, 3] + 2.0 ** -147).all()


# A value that rounds to an infinity, in every place of a tile and in columns of every piece of it: seen by the largest magnitude of its column.
@pytest.mark.parametrize("H,n,d,k", [(32, 260, 128, 65), (32, 200, 64, 64), (40, 700, 128, 225), (70, 520, 64, 129)])
def test_one_huge_value_anywhere(H, n, d, k):
    print(f"f32 range, one huge value H={H} n={n} d={d} k={k}", flush=True)
    Q, K, V = tensors(H, n, d, n + d)
    idx = random_idx(n, k, H, seed=n)
    columns = [(11 * h + 3) % d for h in range(H)]
    for h in range(H):
        V[0, h, idx[h, (k - 1 - h) % k].long(), columns[h]] = 3.4e38
    with pc.Context(1, H, n, d, torch.float32) as ctx:
        O = ctx.attn(Q.to(DEV), K.to(DEV), V.to(DEV), idx.view(1, H, 1, k).to(DEV))
        torch.cuda.synchronize()
    for h in range(H):
        cols = idx[h].numpy()
        want = oracle.dense_attention(f64(Q[0, h]), f64(K[0, h])[cols], f64(V[0, h])[cols])
        assert columns_off(f64(O[0, h]), want) < 2e-5, (h, columns[h])


# Logits of -87 units: 2^-24 of them times sqrt(d) is an error of 6e-5 of a weight.
@pytest.mark.parametrize("H,n,d,k", SHAPES)
@pytest.mark.parametrize("depth", [60.0, 72.0, 80.0, 87.0])
def test_large_values_under_small_weights(H, n, d, k, depth):
    """One key has all but e^-depth of the weight and values of order one; the others' values make up for theirs."""
    print(f"f32 range, small weights H={H} n={n} d={d} k={k} {depth}", flush=True)
    Q, K, V = tensors(H, n, d, n + d)
    idx = random_idx(n, k, H, seed=n)
    Q *= 0.1
    Q[..., 0] = 1.0
    K[..., 0] = -depth * d ** 0.5
    V[..., 3] = (1.0 + V[..., 3].abs()) * float(np.exp(depth)) / n
    for h in range(H):
        first = idx[h, 0].long()
        K[0, h, first] = 0.0
        V[0, h, first, 3] = 0.5
    for pairs in attention(Q, K, V, idx):
        for got, want in pairs[:2]:
            assert (np.abs(got[:, 3] / want[:, 3] - 1.0)).max() < 2e-4
