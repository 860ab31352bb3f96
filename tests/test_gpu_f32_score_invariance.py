"""fp32 scores of a head, in blocks of 128 rows, have the same bits whether the scoring passes cut the head into runs or not: alone
and among other heads, as an element of a padded batch, with and without a context."""

import pytest
import torch

from paper_2605_20813_amd import pulsecol as pc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(n, d, seed):
    g = torch.Generator(device="cpu")
    g.manual_seed(seed)
    Q, K = (torch.randn(1, 1, n, d, generator=g) for _ in range(2))
    K[:, :, ::13] *= 2.5
    return Q, K


def check_copies(Q, K, G, copies):
    n, d = Q.shape[2:]
    want = None
    for r in copies:
        with pc.Context(1, r, n, d, torch.float32, group_size=G) as ctx:
            got = ctx.scores(*(t.repeat(1, r, 1, 1).to(DEV) for t in (Q, K)))
            torch.cuda.synchronize()
        if want is None:
            want = got[0, 0].clone()
        assert torch.equal(got, want.expand_as(got)), f"{r} heads"


# copies of a head on 256 compute units: ten runs, five, two, one; twelve, four, two, one; groups of 4 and of 12 blocks of 32 rows
@pytest.mark.parametrize("n,d,G,copies", [
    (1500, 128, 0, (1, 8, 32, 40)),
    (1500, 64, 0, (1, 8, 32, 40)),
    (3000, 128, 0, (1, 4, 32, 40)),
    (2333, 64, 0, (1, 8, 40, 60)),
    (14001, 128, 0, (1, 3, 10)),            # segments of more than sixteen blocks
    (1500, 128, 128, (1, 8, 40)),
    (3001, 64, 384, (1, 8, 40)),
    (5000, 128, 1280, (1, 4, 40)),
])
def test_a_head_alone_and_among_others(n, d, G, copies):
    print(f"f32 score invariance n={n} d={d} G={G}", flush=True)
    check_copies(*inputs(n, d, n + d), G, copies)


def test_an_element_of_a_padded_batch():
    n, d, H = 3000, 128, 4
    print("f32 score invariance, padded batch", flush=True)
    g = torch.Generator(device="cpu")
    g.manual_seed(5)
    Q, K = (torch.randn(4, H, n, d, generator=g).to(DEV) for _ in range(2))
    alone = {}
    for lens in ([3000] * 4, [3000, 1711, 902, 130], [3000, 1, 902, 3000], [64, 1711, 1902, 3000]):
        with pc.Context(4, H, n, d, torch.float32) as ctx:
            ctx.set_seq_lens(lens)
            got = ctx.scores(Q, K)
            torch.cuda.synchronize()
        for b, length in enumerate(lens):
            if (b, length) not in alone:
                alone[b, length] = got[b, :, 0, :length].clone()
                if length > 512:            # (shorter ones run in blocks of 32 rows when they are alone)
                    with pc.Context(1, H, length, d, torch.float32) as one:
                        alone[b, length] = one.scores(Q[b:b + 1, :, :length].contiguous(), K[b:b + 1, :, :length].contiguous())[0, :, 0]
            assert torch.equal(got[b, :, 0, :length], alone[b, length]), (lens, b)


def test_columns_with_and_without_a_context():
    """56 heads of 3000 rows: three runs in a context, none in the scratch of the call without one.  Pairs of keys whose scores differ by
    roundings only lie at the threshold of about half of the heads."""
    H, n, d = 56, 3000, 128
    print("f32 select with and without a context", flush=True)
    g = torch.Generator(device="cpu")
    g.manual_seed(9)
    Q, K = (torch.randn(1, H, n, d, generator=g) for _ in range(2))
    Q[..., d // 2:] = Q[..., :d // 2]
    K[:, :, 1::2] = K[:, :, 0::2].roll(d // 2, dims=-1)
    Q, K = Q.to(DEV), K.to(DEV)
    with pc.Context(1, H, n, d, torch.float32) as ctx:
        idx = ctx.select(Q, K, 0.1003)          # 300 columns
        odd = ctx.select(Q, K, 0.1004)          # 301
    for keep, want in ((0.1003, idx), (0.1004, odd)):
        got = torch.empty_like(want)
        pc.select_noalloc(pc.make_shape(1, H, n, d, torch.float32), Q, K, keep, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want), keep


@pytest.mark.parametrize("d,G,copies", [(128, 0, (4, 32, 40)), (64, 0, (4, 32, 40)), (128, 256, (4, 40))])
def test_masses_that_underflow_in_single_segments(d, G, copies):
    """Some columns' masses over the first 700 queries lie far below 2^-90 and are formed again with the fp32 instruction; the other
    segments and groups keep the sums that they have in every layout."""
    n = 3000
    print(f"f32 score invariance, small masses d={d} G={G}", flush=True)
    Q, K = inputs(n, d, 3)
    Q[..., 0] = 0.0
    Q[:, :, :700, 0] = 4.0
    K[..., 0] = 0.0
    K[:, :, 100:200, 0] = -82.0 * d ** 0.5 / 4.0
    check_copies(Q, K, G, copies)


@pytest.mark.parametrize("d,G,copies", [(128, 0, (4, 32, 40)), (64, 0, (4, 32, 40)), (128, 256, (4, 40))])
def test_large_and_infinite_numbers(d, G, copies):
    n = 3000
    print(f"f32 score invariance, large and infinite numbers d={d} G={G}", flush=True)
    Q, K = inputs(n, d, 4)
    Q[..., 0] = Q[..., 0].abs().clamp(0.5, 1.0)
    K[:, :, 1000:1040, 0] = -float("inf")
    K[:, :, 2500, 0] = -3.4e38
    K[..., 1] *= 1e-30
    Q[:, :, 300, 1] = 1e30
    check_copies(Q, K, G, copies)
