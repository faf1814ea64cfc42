"""The router kernels at the edges of their tiles: expert counts around 4, 8, 16, 64, ragged hidden sizes and
token counts, ties, -inf logits (an expert switched off by its bias), k = 1 .. E, on both sides of the k from which
up to 64 experts are ranked instead of chosen in k rounds."""
import numpy as np
import pytest
import torch

import paper_2503_09304_amd as q

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _route(dtype, E, k, H, x, Wg, bias):
    N = x.shape[0]
    logits = torch.empty((N, E), device=DEV)
    idx = torch.full((N, k), -1, dtype=torch.int32, device=DEV)
    w = torch.empty((N, k), device=DEV)
    cfg = q.MoeConfig(E, k, H, 64, q.MOE_F32 if dtype == torch.float32 else q.MOE_BF16, 16, N, 0)
    q.moe_route_noalloc(cfg, x, N, Wg, bias, logits, idx, w)
    torch.cuda.synchronize()
    return logits.cpu().numpy(), idx.cpu().numpy(), w.cpu().numpy()


def _check(logits, idx, w, k):
    order = np.lexsort((np.broadcast_to(np.arange(logits.shape[1]), logits.shape), -logits), axis=1)[:, :k]
    assert np.array_equal(order, idx)
    top = np.take_along_axis(logits, order, 1).astype(np.float64)
    p = np.exp(top - top[:, :1])
    # fp32 exponential, sum of at most 32 terms and division: each within a few 2^-24 of its value
    assert np.abs(w - p / p.sum(1, keepdims=True)).max() <= 64 * 2.0 ** -24


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("E,k", [(1, 1), (3, 2), (4, 4), (5, 2), (8, 2), (12, 3), (16, 16), (17, 5), (32, 6), (63, 8), (64, 8), (65, 9),
                                 (100, 32), (128, 4), (200, 7), (256, 32)])
def test_selection_and_logits(dtype, E, k):
    rng = np.random.default_rng(E * 37 + k)
    H = 192 if dtype == torch.bfloat16 else int(rng.integers(1, 700))
    N = int(rng.integers(1, 40))
    x = torch.from_numpy(rng.standard_normal((N, H)).astype(np.float32)).to(dtype).to(DEV)
    Wg = torch.from_numpy((0.2 * rng.standard_normal((H, E))).astype(np.float32)).to(dtype).to(DEV)
    bias = torch.from_numpy(rng.standard_normal(E).astype(np.float32)).to(DEV)
    logits, idx, w = _route(dtype, E, k, H, x, Wg, bias)
    xd, wd, bd = (t.double().cpu().numpy() for t in (x, Wg, bias))
    # any order of H fp32 additions: (H + 1) roundings of at most 2^-24 of the sum of magnitudes (MFMA adds truncate: twice that)
    bar = 2 * (H + 1) * 2.0 ** -24 * (np.abs(xd) @ np.abs(wd) + np.abs(bd))
    assert (np.abs(logits - (xd @ wd + bd)) <= bar).all()
    _check(logits, idx, w, k)

    # x = 0: the logits are the biases, with ties and switched-off experts among them
    tied = rng.integers(0, 3, E).astype(np.float32)
    off = rng.random(E) < 0.3
    off[0] = False
    tied[off] = -np.inf
    logits, idx, w = _route(dtype, E, k, H, torch.zeros_like(x), Wg, torch.from_numpy(tied).to(DEV))
    assert np.array_equal(logits, np.broadcast_to(tied, logits.shape))
    _check(logits, idx, w, k)


@pytest.mark.parametrize("E", [1, 2, 7, 8, 15, 16, 17, 31, 32, 33, 56, 57, 63, 64, 65])
def test_rounds_and_ranks_choose_alike(E):
    """Every k of one set of logits with ties, both zeros, infinities and, in the second set, NaNs (chosen last, the
    lowest index first): the first k of the order, by rounds below E / 4 and by ranks from there on."""
    rng = np.random.default_rng(E)
    H, N = 64, 19
    x = torch.zeros((N, H), dtype=torch.bfloat16, device=DEV)
    Wg = torch.zeros((H, E), dtype=torch.bfloat16, device=DEV)
    for values in ([-np.inf, -1.5, -0.0, 0.0, 2.0], [-np.inf, -1.0, 0.0, 1.0, np.inf, np.nan]):
        bias = torch.from_numpy(rng.choice(np.array(values, dtype=np.float32), E)).to(DEV)
        if not np.isnan(values).any():
            bias[0] = 2.0                             # the largest logit is finite: the weights are numbers
        for k in range(1, min(E, 32) + 1):
            logits, idx, w = _route(torch.bfloat16, E, k, H, x, Wg, bias)
            order = np.lexsort((np.arange(E), -logits[0]))
            assert np.array_equal(idx, np.broadcast_to(order[:k], (N, k))), (k, bias)
            if not np.isnan(values).any():
                _check(logits, idx, w, k)


@pytest.mark.parametrize("E,k,H", [(8, 2, 64), (8, 2, 8192), (16, 4, 4096), (17, 3, 320), (64, 8, 1088), (100, 5, 704), (256, 6, 512),
                                   (256, 6, 576), (24, 3, 1088), (4, 2, 2112)])
def test_two_launches_give_the_bits_of_one(E, k, H):
    """moe_route deals the gate GEMM of up to 1024 tokens to workgroups per K range where that is faster; moe_route_noalloc never does."""
    g = torch.Generator(device=DEV)
    g.manual_seed(E + H)
    Wg = (torch.randn((H, E), generator=g, device=DEV) * H ** -0.5).bfloat16()
    bias = torch.randn(E, generator=g, device=DEV)
    dummy = torch.empty(64, dtype=torch.bfloat16, device=DEV)
    w = q.Context.weights(Wg, dummy, dummy, dummy)
    for N in (1, 2, 5, 6, 8, 9, 16, 17, 1023, 1024, 1025):
        x = torch.randn((N, H), generator=g, device=DEV).bfloat16()
        ctx = q.Context(E, k, H, 64, q.MOE_BF16, 16, N, device=DEV)
        ctx.route(x, w, bias)
        logits, idx, wt = _route(torch.bfloat16, E, k, H, x, Wg, bias)
        assert np.array_equal(ctx.get("logits").cpu().numpy(), logits), N
        assert np.array_equal(ctx.get("topk_idx").cpu().numpy(), idx) and np.array_equal(ctx.get("topk_w").cpu().numpy(), wt), N
