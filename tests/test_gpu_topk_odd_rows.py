"""Top-k over score rows whose length or alignment is not a multiple of 16 bytes: every remainder of the row length,
the smallest and largest rows of each register size, many rows per workgroup, ties at the row's end, a base pointer off
by one element; ragged batches over such rows.  Integer work: bit-exact against the oracle on identical scores."""

import numpy as np
import pytest
import torch

import oracle
from paper_2605_20813_amd import pulsecol as pc
from paper_2605_20813_amd import workloads as wl
from parity_util import assert_idx_matches, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows,n,k", [
    (3, 5, 2), (3, 6, 6), (2, 7, 7), (2, 1023, 100), (3, 4097, 409), (300, 4097, 800), (700, 1501, 150),
    (2, 8191, 819), (5, 16385, 1638), (3, 32770, 6000), (600, 5003, 500), (2, 65535, 6553),
])
@pytest.mark.parametrize("ties", [False, True])
def test_odd_rows_are_bit_exact(rows, n, k, ties):
    print(f"topk odd rows={rows} n={n} k={k} ties={ties}", flush=True)
    s = wl.random_scores(rows, n, seed=rows * n + k, ties=ties)
    if ties:
        s[:, -3:] = s[:, :1]                       # the row's end equals its first score
        s[::2] = s[::2] * 0.0 + 0.5                # every other row is one tie
    with pc.Context(1, rows, n, 64, torch.bfloat16) as ctx:
        idx = ctx.topk(s.view(1, rows, 1, n).to(DEV), k)
        torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy().reshape(rows, k), oracle.topk_columns(f64(s), k))


@pytest.mark.parametrize("n", [1024, 4099])
def test_rows_off_by_one_element(n):
    rows, k = 40, n // 7
    print(f"topk base off by one element n={n}", flush=True)
    s = wl.random_scores(rows, n, seed=n)
    buf = torch.zeros(rows * n + 1, device=DEV)
    buf[1:] = s.view(-1).to(DEV)
    with pc.Context(1, rows, n, 64, torch.bfloat16) as ctx:
        idx = ctx.topk(buf[1:].view(1, rows, 1, n), k)
        torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy().reshape(rows, k), oracle.topk_columns(f64(s), k))


@pytest.mark.parametrize("G", [0, 64])
def test_select_in_a_ragged_batch_of_odd_length(G):
    B, H, n, d, lens, keep = 3, 2, 1021, 64, (1021, 518, 3), 0.2
    print(f"select, ragged batch of odd length G={G}", flush=True)
    g = torch.Generator(device="cpu")
    g.manual_seed(7)
    Q, K = (torch.randn(B, H, n, d, generator=g).to(torch.bfloat16) for _ in range(2))
    with pc.Context(B, H, n, d, torch.bfloat16, group_size=G) as ctx:
        ctx.set_seq_lens(lens)
        idx = ctx.select(Q.to(DEV), K.to(DEV), keep)
        again = ctx.select(None, None, keep, refresh=False)
        torch.cuda.synchronize()
        assert torch.equal(idx, again)
    got = idx.cpu().numpy()
    for b, L in enumerate(lens):
        kb = oracle.num_keep(L, keep)
        for h in range(H):
            s64 = oracle.column_scores(f64(Q[b, h, :L]), f64(K[b, h, :L]), group_size=G)
            for u in range(got.shape[2]):
                if u < s64.shape[0]:
                    assert_idx_matches(got[b, h, u, :kb], s64[u], kb, f"b={b} h={h} u={u}")
                    assert (got[b, h, u, kb:] == -1).all()
                else:
                    assert (got[b, h, u] == -1).all()


@pytest.mark.parametrize("rows,n,k,offset", [(3, 5, 4, 0), (4, 1021, 1000, 0), (4, 1024, 1000, 1), (300, 5003, 500, 0), (300, 5004, 5000, 1),
                                             (3, 32771, 32770, 0)])
def test_odd_rows_with_every_bit_pattern(rows, n, k, offset):
    """Scores of any bits, the NaN with all bits set among them (the smallest key there is): kept by key, the lower index first.  The
    first pass over a row counts digits without a test, so its bounds have to be those of the elements."""
    print(f"topk any bits rows={rows} n={n} k={k} offset={offset}", flush=True)
    rng = np.random.default_rng(n + k)
    bits = rng.uniform(0.5, 0.5001, (rows, n)).astype(np.float32).view(np.uint32)          # one exponent: few digits differ
    lots = rng.random((rows, n)) < 0.02
    bits[lots] = rng.integers(0, 2**32, int(lots.sum()), dtype=np.uint64).astype(np.uint32)
    bits[:, [n // 2, n - 1]] = 0xFFFFFFFF
    bits[::3, 0] = 0xFFFFFFFF
    buf = torch.zeros(rows * n + offset, dtype=torch.int32, device=DEV)
    buf[offset:] = torch.from_numpy(bits.view(np.int32).reshape(-1)).to(DEV)
    scores = buf.view(torch.float32)[offset:].view(1, rows, 1, n)
    with pc.Context(1, rows, n, 64, torch.bfloat16) as ctx:
        idx = ctx.topk(scores, k)
        torch.cuda.synchronize()
    key = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000)).astype(np.int64)
    want = np.sort(np.argsort(-key, axis=1, kind="stable")[:, :k], axis=1)
    assert np.array_equal(idx.cpu().numpy().reshape(rows, k), want)
