"""Top-k of more rows than one line of a grid holds: a last line that is not full, and a launch of 2^32 threads."""

import pytest
import torch

from paper_2605_20813_amd import pulsecol as pc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# heads, elements, groups: a little more than 2^20 rows; 2^24 rows of four waves each (67 GB)
@pytest.mark.parametrize("heads,n,groups", [((1 << 19) + 3, 33, 2), (1 << 20, 500, 16)])
def test_largest_of_many_rows(heads, n, groups):
    print(f"topk many rows heads={heads} n={n} groups={groups}", flush=True)
    if torch.cuda.mem_get_info()[0] < 3 * 4 * heads * groups * n:
        pytest.skip("needs more memory")
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    scores = torch.rand(1, heads, groups, n, generator=g, device=DEV)
    with pc.Context(1, heads, n, 64, torch.bfloat16, group_size=32, max_keep_ratio=1.5 / n) as ctx:
        assert ctx.groups == groups
        idx = torch.full((1, heads, groups, 1), -1, dtype=torch.int32, device=DEV)
        ctx.topk(scores, 1, idx_out=idx)
        torch.cuda.synchronize()
    assert int(idx.min()) >= 0 and int(idx.max()) < n
    at = idx.long()
    largest = scores.amax(-1, keepdim=True)
    assert bool((scores.gather(-1, at) == largest).all())
    # (equal ones: the first)
    column = torch.arange(n, device=DEV)
    for part, of, here in zip(scores.split(1 << 16, 1), largest.split(1 << 16, 1), at.split(1 << 16, 1)):
        assert not bool(((part == of) & (column < here)).any())
