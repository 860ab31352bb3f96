"""fp32 mode outside the range in which three bf16 parts carry a number: small numbers of Q and K against large ones of the other (or
a large scale)."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from parity_util import f64

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
