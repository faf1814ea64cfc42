"""The combine at the edges of its loops: top-k beside the row groups it requests together (1, 2, 4, 8, 16, 32),
every number of K ranges, hidden sizes beside its 1024-column workgroups, no multiple of 4, few tokens (a workgroup
takes 1024 columns) and more than 1024 (it takes all of a token's); by class and by completeness."""
import numpy as np
import pytest
import torch

import paper_2503_09304_amd as q

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [  # dtype, E, k, H, F, N, K ranges
    ("f32", 4, 1, 1, 3, 5, 1),
    ("f32", 4, 3, 255, 5, 7, 1),
    ("f32", 20, 15, 1023, 4, 9, 1),
    ("f32", 32, 32, 1028, 4, 3, 1),
    ("f32", 16, 9, 1024, 4, 3, 1),
    ("f32", 2, 2, 16645, 1, 2, 1),
    ("f32", 1, 1, 66564, 1, 2, 1),
    ("bf16", 8, 1, 64, 128, 17, 2),
    ("bf16", 16, 7, 1088, 256, 5, 4),
    ("bf16", 32, 31, 1024, 128, 5, 2),
    ("bf16", 16, 13, 2112, 256, 6, 4),
    ("bf16", 32, 23, 960, 64, 5, 1),
    ("bf16", 2, 2, 65600, 64, 2, 1),
    ("bf16", 8, 2, 2112, 64, 682, 1),
    ("bf16", 8, 3, 2112, 256, 683, 4),
    ("bf16", 8, 1, 1088, 128, 1025, 2),
    ("f32", 4, 2, 1030, 3, 1024, 1),
    ("f32", 16, 5, 2052, 2, 1100, 1),
]


@pytest.mark.parametrize("dtype,E,k,H,F,N,ks", CASES)
def test_combine(dtype, E, k, H, F, N, ks):
    print("case", dtype, E, k, H, F, N, ks, flush=True)
    rng = np.random.default_rng(H * 7 + k)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def t(shape, std):
        return torch.from_numpy((std * rng.standard_normal(shape)).astype(np.float32)).to(dt).to(DEV)

    x, Wg = t((N, H), 1.0), t((H, E), 0.02)
    held = [t((E, F, H), 0.02), t((E, F, H), 0.02), t((E, H, F), 0.02)]
    w = q.Context.weights(Wg, *held)
    ctx = q.Context(E, k, H, F, q.MOE_F32 if dtype == "f32" else q.MOE_BF16, 16, N, device=DEV, down_ksplit=ks)
    prio = torch.from_numpy((np.arange(N) % 2).astype(np.uint8)).to(DEV)
    ctx.route(x, w, None)
    ctx.permute(prio)
    yc, done = torch.full((N, H), 3.0, dtype=dt, device=DEV), torch.full((N,), 7, dtype=torch.uint8, device=DEV)
    units = ctx.units()
    ctx.expert_run(x, w, len(units) // 2)
    ctx.combine_complete(yc, done)                # the tokens whose rows are all among these units
    row_done = np.zeros(N * k, dtype=bool)
    for _, _, row0, rows in units[: len(units) // 2]:
        row_done[row0: row0 + rows] = True
    want = row_done[ctx.get("inv").cpu().numpy().reshape(N, k)].all(1)
    assert np.array_equal(done.cpu().numpy(), want)
    some = yc.clone()
    if len(units) // 2 < len(units):
        ctx.expert_run(x, w)
    y = torch.full((N, H), 3.0, dtype=dt, device=DEV)
    ctx.combine(y, q.MOE_CLASS_LS)                # the odd tokens only
    torch.cuda.synchronize()
    assert (y[0::2] == 3.0).all()
    ls = y.clone()
    ctx.combine(y)
    y32 = torch.zeros((N, H), device=DEV)
    ctx.combine(y32, q.MOE_CLASS_ALL | q.MOE_Y_F32)
    assert torch.equal(some[torch.from_numpy(want).to(DEV)], y[torch.from_numpy(want).to(DEV)])
    assert (some[torch.from_numpy(~want).to(DEV)] == 3.0).all()
    yc.zero_()
    ctx.combine_complete(yc, done)
    torch.cuda.synchronize()
    assert torch.equal(ls[1::2], y[1::2]) and torch.equal(yc, y) and done.bool().all()
    assert torch.equal(y32.to(dt), y)             # one rounding to the output type

    out = ctx.get("expert_out").reshape(N * k, H).double()
    inv = ctx.get("inv").reshape(N, k).long()
    g = ctx.get("topk_w").reshape(N, k).double()
    terms = g[:, :, None] * out[inv]
    # k fused multiply-adds, each rounded once: at most k * 2^-24 of the sum of the terms' magnitudes
    bar = k * 2.0 ** -24 * terms.abs().sum(1)
    assert ((y32.double() - terms.sum(1)).abs() <= bar).all()
