"""The permutation in three kernels (more than 4096 assignments): bucket order, queue lengths and the unit list, the host's and
the device's, against a stable sort, at the smallest such batches, a last block of one assignment, and one to 256 experts (2 to
512 ranges of blocks per bucket); the same of the kernel for fewer."""
import numpy as np
import pytest
import torch

import paper_2503_09304_amd as q

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("E,k,N", [(1, 1, 8193), (3, 3, 2731), (64, 8, 1025), (256, 8, 1025), (255, 5, 4096), (8, 2, 8192),
                                   (1, 1, 1), (64, 8, 1024), (256, 2, 1000)])
def test_three_kernels_sort_like_one(E, k, N):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(E + N)
    H = 64
    x = torch.randn((N, H), generator=gen, device=DEV).bfloat16()
    Wg = torch.randn((H, E), generator=gen, device=DEV).bfloat16()
    dummy = torch.empty(64, dtype=torch.bfloat16, device=DEV)
    w = q.Context.weights(Wg, dummy, dummy, dummy)
    prio = (torch.rand(N, generator=gen, device=DEV) < 0.3).to(torch.uint8)
    ctx = q.Context(E, k, H, 64, q.MOE_BF16, 100, N, device=DEV)
    for _ in range(2):                                   # the second time over what the first has left
        ctx.route(x, w)
        ctx.permute(prio)
        key = ctx.get("topk_idx").cpu().numpy().reshape(-1).astype(np.int64) * 2 + np.repeat(1 - prio.cpu().numpy().astype(np.int64), k)
        want = np.argsort(key, kind="stable")
        assert np.array_equal(ctx.get("perm").cpu().numpy(), want)
        lens = np.bincount(key, minlength=2 * E)
        first = np.concatenate(([0], np.cumsum(lens)))
        units = [(e, c, int(first[2 * e + c]) + r, min(100, int(lens[2 * e + c]) - r))
                 for c in (0, 1) for e in range(E) for r in range(0, int(lens[2 * e + c]), 100)]
        assert [tuple(int(v) for v in u) for u in ctx.units()] == units
        # nothing reports what the device's list holds, the host makes its own from the reported lengths: the list, and its length behind the counts
        assert [tuple(u) for u in ctx.get("units").cpu().tolist()] == units
        at = ctx.get("counts").data_ptr() - ctx.ws.data_ptr() + 8 * E
        assert int(ctx.ws[at: at + 4].view(torch.int32)) == len(units)


@pytest.mark.parametrize("E,k,N", [(1, 1, 4096), (1, 1, 4097), (256, 8, 512), (256, 3, 1366), (64, 1, 5121), (8, 2, 3584)])
def test_either_side_of_4096_assignments(E, k, N):
    """The line between the kernel for few assignments and the three for more."""
    test_three_kernels_sort_like_one(E, k, N)
