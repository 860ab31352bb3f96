"""The reference of the row pass (bf16): rows whose dominating logits come late and far above the first keys, and blocks of
keys whose logits are all -inf, at the start of a head and where a pass is cut into runs.  One component of Q and K carries
the logits, so that every dot product is exact and what is measured is the softmax alone."""

import numpy as np
import pytest
import torch

from paper_2605_20813_amd import pulsecol as pc
from parity_util import assert_close, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def scores_of(k0, n, d, heads=1):
    """Column scores [heads, n] on the GPU and in fp64 for identical rows whose logit against key j is k0[h, j] / sqrt(d)."""
    Q, K = torch.zeros(1, heads, n, d), torch.zeros(1, heads, n, d)
    Q[..., 0] = 1.0
    K[0, :, :, 0] = torch.as_tensor(np.asarray(k0), dtype=torch.float32)
    K = K.to(torch.bfloat16)
    with pc.Context(1, heads, n, d, torch.bfloat16) as ctx:
        got = f64(ctx.scores(Q.to(torch.bfloat16).to(DEV), K.to(DEV)))[0, :, 0]
    # (log2 units per unit of K: the product of two fp32 numbers, rounded to fp32, as in the kernels)
    c2 = float(np.float32(np.float32(1.0 / np.float32(np.sqrt(np.float32(d)))) * np.float32(1.4426950408889634)))
    z = f64(K[0, :, :, 0]) * c2
    w = np.exp2(z - z.max(axis=1, keepdims=True))
    return got, w / w.sum(axis=1, keepdims=True)


@pytest.mark.parametrize("n,d,heads", [(200, 128, 40), (260, 64, 40), (511, 128, 16)])
def test_late_logits_keep_the_precision_of_early_ones(n, d, heads):
    """One key per head carries the row; it lies 20 to 120 log2 units above the first keys.  Its score is off by the
    rounding of log2(sum) + reference below one, 2^-24, of the exponentials and the logarithm of the hardware, about one
    unit of 2^-23 each, and of the division: 4e-7.  (Weighed against the first keys, z - reference alone is rounded by up to
    2^-18, 2.6e-6 of the score.  Few rows: the rows are equal, so the rounding of a sum over them does not average out.)"""
    print(f"late logits n={n} d={d}", flush=True)
    rng = np.random.default_rng(n)
    unit = np.sqrt(d) / 1.4426950408889634                          # of K per log2 unit
    k0 = np.full((heads, n), -140.0 * unit)
    late = rng.integers(n // 3, n, heads)
    k0[:, :32] = -np.linspace(20.0, 120.0, heads)[:, None] * unit
    k0[np.arange(heads), late] = rng.uniform(-0.9, 0.9, heads) * unit
    got, want = scores_of(k0, n, d, heads)
    err = np.abs(got - want)[np.arange(heads), late]
    print("worst", err.max())
    assert err.max() < 4e-7


@pytest.mark.parametrize("first,last", [(320, 352), (0, 32), (0, 400), (1000, 2049), (640, 1280)])
def test_keys_without_a_finite_logit(first, last):
    """Keys first .. last-1 have logits of -inf; 33 tiles of 64 keys in runs of a few tiles each.  Their score is zero, that of the
    others the softmax over them."""
    n, d = 2049, 128
    print(f"-inf logits {first}..{last}", flush=True)
    rng = np.random.default_rng(first)
    k0 = rng.normal(size=(1, n)) * np.sqrt(d)
    k0[:, first:last] = -np.inf
    got, want = scores_of(k0, n, d)
    assert (got[:, first:last] == 0.0).all()
    assert np.isfinite(got).all()
    ok = want > 0
    assert (np.abs(got - want)[ok] / want[ok]).max() < 2e-5


def test_error_of_long_sums():
    """Scores of a long head against fp64, rms relative error.  Left are the weights (one rounding of z - log-sum-exp of up to 2^-22 for
    each, which average out over the rows), the row sums' rounding, 3e-8, and that of the result, 2^-24 / 3^0.5 = 3.4e-8: 5e-8
    altogether.  (24 segments added up one after the other without what their roundings leave out: 9e-8.)"""
    n, d = 16384, 128
    print("error of long sums", flush=True)
    err = []
    for seed in range(3):
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        Q, K = (torch.randn(1, 1, n, d, device=DEV, generator=g) for _ in range(2))
        K *= torch.where(torch.rand(1, 1, n, 1, device=DEV, generator=g) < 0.05, 2.5, 1.0)
        Q, K = Q.to(torch.bfloat16), K.to(torch.bfloat16)
        with pc.Context(1, 1, n, d, torch.bfloat16) as ctx:
            got = ctx.scores(Q, K)[0, 0, 0].double()
        q, k = Q[0, 0].double(), K[0, 0].double()
        want = sum(torch.softmax(q[a:a + 2048] @ k.t() / d ** 0.5, dim=-1).sum(0) for a in range(0, n, 2048)) / n
        err.append((((got - want) / want) ** 2).mean().item())
    rms = (sum(err) / len(err)) ** 0.5
    print("rms", rms)
    assert rms < 6e-8


def one_component(k0, n, d, dtype):
    Q, K = torch.zeros(1, 1, n, d), torch.zeros(1, 1, n, d)
    Q[..., 0] = 1.0
    K[0, 0, :, 0] = torch.as_tensor(k0, dtype=torch.float32)
    g = torch.Generator(device="cpu")
    g.manual_seed(n)
    return Q.to(dtype), K.to(dtype), torch.randn(1, 1, n, d, generator=g).to(dtype)


# (the 32-row fp32 kernels: wave w takes the tiles w, w + 4 or w + 8, ...)
@pytest.mark.parametrize("first,last", [(32, 64), (0, 32), (64, 200), (224, 256), (0, 290)])
@pytest.mark.parametrize("d", [64, 128])
def test_f32_keys_without_a_finite_logit(d, first, last):
    n = 300
    print(f"f32 -inf logits d={d} {first}..{last}", flush=True)
    k0 = np.random.default_rng(first).normal(size=n) * np.sqrt(d)
    k0[first:last] = -np.inf
    Q, K, V = one_component(k0, n, d, torch.float32)
    z = f64(K[0, 0, :, 0]) / np.sqrt(d)
    w = np.exp(z - z.max())
    w /= w.sum()
    with pc.Context(1, 1, n, d, torch.float32) as ctx:
        q, k, v = Q.to(DEV), K.to(DEV), V.to(DEV)
        sc = f64(ctx.scores(q, k))[0, 0, 0]
        idx = torch.arange(n, dtype=torch.int32, device=DEV).view(1, 1, 1, n)
        outs = [ctx.attn(q, k, v, idx), ctx.attn_dense(q, k, v)]
    assert np.abs(sc - w).max() < 1e-5 * w.max()
    for O in outs:
        assert np.abs(f64(O[0, 0]) - w @ f64(V[0, 0])).max() < 1e-4


@pytest.mark.parametrize("copies", [1, 130])                 # two teams, one team
@pytest.mark.parametrize("G", [0, 32, 64, 128])
def test_first_tile_without_a_finite_logit(G, copies):
    """The plain bf16 attention kernel: the first 32 columns' logits are -inf, what follows lies beyond 2^127 as weights against zero."""
    n, d, k = 256, 128, 160
    print(f"-inf first tile G={G} copies={copies}", flush=True)
    k0 = np.full(n, -np.inf)
    k0[32:k] = (200.0 + np.random.default_rng(G).uniform(-3.0, 3.0, k - 32)) * np.sqrt(d)
    Q, K, V = one_component(k0, n, d, torch.bfloat16)
    z = f64(K[0, 0, :k, 0]) / np.sqrt(d)
    w = np.exp(z - z.max())
    w /= w.sum()
    with pc.Context(1, copies, n, d, torch.bfloat16, group_size=G) as ctx:
        ctx.set_attn_block(128)
        idx = torch.arange(k, dtype=torch.int32, device=DEV).expand(1, copies, ctx.groups, k).contiguous()
        O = ctx.attn(*(t.to(DEV).repeat(1, copies, 1, 1).contiguous() for t in (Q, K, V)), idx)
    want = np.broadcast_to(w @ f64(V[0, 0, :k]), (n, d))
    assert_close(O[0, 0], want, "bf16", "first head")
    assert_close(O[0, -1], want, "bf16", "last head")
