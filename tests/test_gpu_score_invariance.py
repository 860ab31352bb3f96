"""A head's scores (bf16) have the same bits in every launch that holds it: alone, where the passes are cut into runs, and
among many heads, where they are not; whatever the other elements of a padded batch; with and without a context."""

import pytest
import torch

from paper_2605_20813_amd import pulsecol as pc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(B, H, n, d, seed):
    g = torch.Generator(device="cpu")
    g.manual_seed(seed)
    Q, K = (torch.randn(B, H, n, d, generator=g) for _ in range(2))
    K[:, :, ::13] *= 2.5
    return Q.to(torch.bfloat16).to(DEV), K.to(torch.bfloat16).to(DEV)


@pytest.mark.parametrize("n,d,G,copies", [
    (200, 128, 0, (1, 600)),            # one segment
    (1000, 128, 0, (1, 30, 70, 300)),   # four segments: four runs, two, none
    (2049, 64, 0, (1, 20, 130)),        # eight, ragged
    (4100, 128, 0, (1, 7, 9, 16, 31)),  # twelve of five and six tiles
    (8192, 128, 0, (1, 4, 16)),
    (1000, 128, 96, (1, 30, 130)),      # groups of three blocks of 32 rows
    (4100, 64, 256, (1, 9, 31)),
])
def test_a_head_alone_and_among_others(n, d, G, copies):
    print(f"score invariance n={n} d={d} G={G}", flush=True)
    Q, K = inputs(1, 1, n, d, seed=n + d)
    want = None
    for r in copies:
        with pc.Context(1, r, n, d, torch.bfloat16, group_size=G) as ctx:
            q, k = (t.repeat(1, r, 1, 1).contiguous() for t in (Q, K))
            got = ctx.scores(q, k)
            idx = ctx.select(q, k, 0.1)
            if (1 + ctx.groups) * r * n <= 4 << 20:
                same = torch.empty_like(idx)
                pc.select_noalloc(pc.make_shape(1, r, n, d, torch.bfloat16, group_size=G), q, k, 0.1, same)
                assert torch.equal(same, idx)
            torch.cuda.synchronize()
        if want is None:
            want = got[0, 0].clone()
        assert torch.equal(got, want.expand_as(got)), f"{r} heads"


def test_an_element_of_a_padded_batch():
    n, d, H = 3000, 128, 4
    print("score invariance, padded batch", flush=True)
    Q, K = inputs(4, H, n, d, seed=5)
    alone = {}
    for lens in ([3000] * 4, [3000, 1711, 902, 130], [3000, 1, 902, 3000], [64, 1711, 902, 3000]):
        with pc.Context(4, H, n, d, torch.bfloat16) as ctx:
            ctx.set_seq_lens(lens)
            got = ctx.scores(Q, K)
            torch.cuda.synchronize()
        for b, length in enumerate(lens):
            if (b, length) not in alone:
                with pc.Context(1, H, length, d, torch.bfloat16) as one:
                    alone[b, length] = one.scores(Q[b:b + 1, :, :length].contiguous(), K[b:b + 1, :, :length].contiguous())[0, :, 0]
            assert torch.equal(got[b, :, 0, :length], alone[b, length]), (lens, b)
