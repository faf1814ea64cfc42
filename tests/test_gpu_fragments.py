"""bf16 expert kernels at every count of 16-token fragments: a batch in units of c rows, one unit a launch, gives the bits of
one launch of the whole batch (16 fragments), for c at and beside the multiples of 16, in every weight format; the whole
launch against plain products in fp64."""
import pytest
import torch

import paper_2503_09304_amd as q
from test_gpu_unit_list import bar

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("fmt,H,F,ksplit", [("rowmajor", 192, 320, 1), ("packed", 320, 512, 4), ("mxfp4", 256, 384, 2)])
def test_every_fragment_count(fmt, H, F, ksplit):
    N = 256
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)

    def t(shape, std):
        return (torch.randn(shape, generator=gen, device=DEV) * std).bfloat16()

    x, Wg = t((N, H), 1.0), t((H, 1), 0.02)
    shapes = ((1, F, H), (1, F, H), (1, H, F))
    if fmt == "mxfp4":
        codes = [torch.randint(0, 256, s[:2] + (s[2] // 2,), generator=gen, device=DEV, dtype=torch.uint8) for s in shapes]
        scales = [torch.randint(121, 124, s[:2] + (s[2] // 32,), generator=gen, device=DEV, dtype=torch.uint8) for s in shapes]
        table = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64, device=DEV)
        W = [(table[torch.stack((c & 15, c >> 4), -1).long()].reshape(c.shape[:2] + (-1, 32)) * torch.exp2(s.double() - 127)[..., None]).reshape(sh)
             for c, s, sh in zip(codes, scales, shapes)]
        src = q.Context.weights(Wg, *codes, q.MOE_W_MXFP4_ROWMAJOR, *scales)
        hold = [torch.empty((16, H), dtype=torch.bfloat16, device=DEV)] + [torch.empty_like(v) for v in codes + scales]
        w = q.Context.weights(*hold[:4], q.MOE_W_MXFP4_ROWMAJOR, *hold[4:])
    else:
        hold = [t(s, s[2] ** -0.5) for s in shapes]
        W = [v.double() for v in hold]
        src = w = q.Context.weights(Wg, *hold)
        if fmt == "packed":
            keep = hold
            hold = [torch.empty((16, H), dtype=torch.bfloat16, device=DEV)] + [torch.empty_like(v) for v in keep]
            w = q.Context.weights(*hold)
    if fmt != "rowmajor":
        q.moe_pack_weights(q.MoeConfig(1, 1, H, F, q.MOE_BF16, 1, 0), src, w)
    prio = torch.zeros(N, dtype=torch.uint8, device=DEV)

    def run(chunk, units):
        ctx = q.Context(1, 1, H, F, q.MOE_BF16, chunk, N, device=DEV, down_ksplit=ksplit)
        ctx.route(x, w)
        ctx.permute(prio)
        while ctx.expert_run(x, w, units) != q.MOE_DONE:
            pass
        out = ctx.get("expert_out").clone()
        torch.cuda.synchronize()
        return out

    whole = run(256, q.UINT32_MAX)
    g, u = x.double() @ W[0][0].t(), x.double() @ W[1][0].t()
    ref = (g / (1 + torch.exp(-g)) * u) @ W[2][0].t()
    assert ((whole.double() - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= bar("bf16", H, F)
    for c in sorted({1, 15} | {16 * i + d for i in range(1, 16) for d in (0, 1)} | {255}):
        print("case", fmt, "rows", c, flush=True)
        assert torch.equal(run(c, 1), whole), (fmt, c)


@pytest.mark.parametrize("fmt,E,H,F,rows", [("rowmajor", 1, 192, 320, 1), ("packed", 2, 320, 256, 17), ("packed", 3, 64, 512, 32), ("packed", 1, 2048, 256, 16)])
def test_narrow_down_projection(fmt, E, H, F, rows):
    """Small launches put 128 columns of the down projection in a workgroup: `rows` rows per expert (k = E, every token on
    every expert) against plain products, and against the enqueued form, which keeps 256."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + H)

    def t(shape, std):
        return (torch.randn(shape, generator=gen, device=DEV) * std).bfloat16()

    x, Wg = t((rows, H), 1.0), t((H, E), 0.02)
    src = [t((E, F, H), H ** -0.5), t((E, F, H), H ** -0.5), t((E, H, F), F ** -0.5)]
    w = q.Context.weights(Wg, *src)
    if fmt == "packed":
        hold = [torch.empty((16, H), dtype=torch.bfloat16, device=DEV)] + [torch.empty_like(v) for v in src]
        p = q.Context.weights(*hold)
        q.moe_pack_weights(q.MoeConfig(E, 1, H, F, q.MOE_BF16, 1, 0), w, p)
        w = p
    prio = torch.zeros(rows, dtype=torch.uint8, device=DEV)
    outs = []
    for enqueued in (False, True):
        ctx = q.Context(E, E, H, F, q.MOE_BF16, 256, rows, device=DEV)
        ctx.route(x, w)
        ctx.permute(prio)
        if enqueued:
            ctx.expert_enqueue(x, w, q.UINT32_MAX)
            assert ctx.expert_collect() == q.MOE_DONE
        else:
            assert ctx.expert_run(x, w) == q.MOE_DONE
        outs.append(ctx.get("expert_out").clone())
        torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    for e in range(E):                                  # sorted order: expert by expert, tokens ascending
        g, u = x.double() @ src[0][e].double().t(), x.double() @ src[1][e].double().t()
        ref = (g / (1 + torch.exp(-g)) * u) @ src[2][e].double().t()
        got = outs[0][e * rows: (e + 1) * rows].double()
        assert ((got - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= bar("bf16", H, F)
