"""bf16 expert kernels at every count of 16-token fragments, in every weight format.  Launches that stream: a batch in units of c
rows, one unit a launch, gives the bits of one launch of the whole batch (16 fragments), for c at and beside the multiples
of 16; the whole launch against plain products in fp64.  Launches that do not: c rows of one expert beside two segments of
another give the same bits again.  The narrow form of the down projection against plain products and the wide form."""
import pytest
import torch

import paper_2503_09304_amd as q
from test_gpu_unit_list import bar

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
COUNTS = sorted({1, 15} | {16 * i + d for i in range(1, 16) for d in (0, 1)} | {255})


def make(fmt, Wg, E, H, F, gen):
    """(weights as the library reads them, W1, W3, W2 as plain tensors, the tensors that hold their memory)"""
    shapes = ((E, F, H), (E, F, H), (E, H, F))
    if fmt == "mxfp4":
        codes = [torch.randint(0, 256, s[:2] + (s[2] // 2,), generator=gen, device=DEV, dtype=torch.uint8) for s in shapes]
        scales = [torch.randint(121, 124, s[:2] + (s[2] // 32,), generator=gen, device=DEV, dtype=torch.uint8) for s in shapes]
        table = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64, device=DEV)
        W = [(table[torch.stack((c & 15, c >> 4), -1).long()].reshape(c.shape[:2] + (-1, 32)) * torch.exp2(s.double() - 127)[..., None]).reshape(sh)
             for c, s, sh in zip(codes, scales, shapes)]
        src = q.Context.weights(Wg, *codes, q.MOE_W_MXFP4_ROWMAJOR, *scales)
        given = codes + scales
    else:
        W = given = [(torch.randn(s, generator=gen, device=DEV) * s[2] ** -0.5).bfloat16() for s in shapes]
        src = q.Context.weights(Wg, *given)
        if fmt == "rowmajor":
            return src, W, given
    hold = [torch.empty(((E + 15) // 16 * 16, H), dtype=torch.bfloat16, device=DEV)] + [torch.empty_like(v) for v in given]
    args = (q.MOE_W_MXFP4_ROWMAJOR,) if fmt == "mxfp4" else ()
    w = q.Context.weights(*hold[:4], *args, *hold[4:])
    q.moe_pack_weights(q.MoeConfig(E, 1, H, F, q.MOE_BF16, 1, 0), src, w)
    torch.cuda.synchronize()
    return w, W, hold


def error(got, x, W, e):
    """max|err| / RMS of the outputs of expert e for the rows x."""
    g, u = x.double() @ W[0][e].double().t(), x.double() @ W[1][e].double().t()
    ref = (g / (1 + torch.exp(-g)) * u) @ W[2][e].double().t()
    return ((got.double() - ref).abs().max() / ref.pow(2).mean().sqrt()).item()


@pytest.mark.parametrize("fmt,H,F,ksplit", [("rowmajor", 192, 320, 1), ("packed", 320, 512, 4), ("mxfp4", 256, 384, 2)])
def test_every_fragment_count(fmt, H, F, ksplit):
    N = 256
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)
    x, Wg = torch.randn((N, H), generator=gen, device=DEV).bfloat16(), (torch.randn((H, 1), generator=gen, device=DEV) * 0.02).bfloat16()
    w, W, hold = make(fmt, Wg, 1, H, F, gen)
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
    assert error(whole, x, W, 0) <= bar("bf16", H, F)
    for c in COUNTS:
        print("case", fmt, "rows", c, flush=True)
        assert torch.equal(run(c, 1), whole), (fmt, c)


# chunk: rows of the other expert's two segments, units 0 and 2 of three, which do not join: with 256 every count runs in the kernel
# for up to 256 rows, with 16 in the one for its own
@pytest.mark.parametrize("chunk", [16, 256])
@pytest.mark.parametrize("fmt,H,F,ksplit", [("rowmajor", 192, 320, 1), ("packed", 320, 512, 4), ("mxfp4", 192, 384, 2), ("mxfp4", 320, 448, 1)])
def test_every_fragment_count_beside_shared_weights(fmt, H, F, ksplit, chunk):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(12)
    N = 255 + 3 * chunk
    x = torch.randn((N, H), generator=gen, device=DEV).bfloat16()
    x[:255, 0], x[255:, 0] = 1.0, -1.0                  # the first 255 tokens go to expert 0, the others to expert 1
    Wg = torch.zeros((H, 2), dtype=torch.bfloat16, device=DEV)
    Wg[0, 0] = 1.0
    w, W, hold = make(fmt, Wg, 2, H, F, gen)

    def run(xs, pick):
        ctx = q.Context(2, 1, H, F, q.MOE_BF16, chunk, xs.shape[0], device=DEV, down_ksplit=ksplit)
        ctx.route(xs, w)
        ctx.permute(torch.zeros(xs.shape[0], dtype=torch.uint8, device=DEV))
        units = ctx.units()
        ctx.expert_run_units(xs, w, pick(units))
        out = ctx.get("expert_out").clone()
        torch.cuda.synchronize()
        return out, units

    alone, _ = run(x[:255].contiguous(), lambda units: range(len(units)))       # one segment, streamed
    assert error(alone, x[:255], W, 0) <= bar("bf16", H, F)
    for c in COUNTS:
        print("case", fmt, H, "chunk", chunk, "rows", c, flush=True)

        def pick(units):
            other = [i for i, u in enumerate(units) if u[0] == 1]
            assert len(other) == 3
            return [i for i, u in enumerate(units) if u[0] == 0] + [other[0], other[2]]

        out, _ = run(torch.cat((x[:c], x[255:])), pick)
        assert torch.equal(out[:c], alone[:c]), (fmt, c)
        for at in (0, 2 * chunk):
            assert error(out[c + at: c + at + chunk], x[255 + at: 255 + at + chunk], W, 1) <= bar("bf16", H, F)


# the last three: 320 workgroups of 256 columns, two rounds of 256 CUs, as 608 of 128, three rounds
@pytest.mark.parametrize("fmt,E,H,F,rows", [("rowmajor", 1, 192, 320, 1), ("packed", 2, 320, 256, 17), ("packed", 3, 64, 512, 32), ("packed", 1, 2048, 256, 16),
                                            ("mxfp4", 1, 192, 320, 1), ("mxfp4", 2, 320, 256, 17), ("mxfp4", 3, 64, 512, 32),
                                            ("rowmajor", 32, 2432, 64, 3), ("packed", 32, 2432, 64, 32), ("mxfp4", 32, 2432, 64, 17)])
def test_narrow_down_projection(fmt, E, H, F, rows):
    """Small launches put 128 columns of the down projection in a workgroup: `rows` rows per expert (k = E, every token on
    every expert) against plain products, and against the enqueued form, which keeps 256."""
    print("case", fmt, E, H, F, rows, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + H)
    x, Wg = torch.randn((rows, H), generator=gen, device=DEV).bfloat16(), (torch.randn((H, E), generator=gen, device=DEV) * 0.02).bfloat16()
    w, W, hold = make(fmt, Wg, E, H, F, gen)
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
        assert error(outs[0][e * rows: (e + 1) * rows], x, W, e) <= bar("bf16", H, F)


# E experts of `rows` rows each and the columns that the launch rule gives a gate-up wave on 256 CUs (test_expert_items.py asks the rule
# itself): launches of one round, two and more, row-major also beyond 96 rows, of equal cost (row-major of few rows goes to 16 columns)
WAVE_COLUMNS = [("packed", 3, 128, 512, 1, 16), ("packed", 8, 64, 2176, 33, 20), ("rowmajor", 3, 128, 192, 97, 16), ("rowmajor", 8, 64, 4608, 129, 20),
                ("rowmajor", 8, 64, 4608, 256, 20), ("packed", 8, 64, 4608, 96, 20), ("rowmajor", 64, 64, 1408, 5, 16),
                ("packed", 8, 64, 2624, 17, 24), ("packed", 16, 64, 1408, 64, 24), ("packed", 8, 64, 3584, 32, 28), ("packed", 16, 64, 3136, 1, 28),
                ("rowmajor", 8, 64, 3072, 33, 24), ("rowmajor", 16, 64, 1664, 160, 28), ("rowmajor", 8, 64, 3136, 97, 28),
                ("packed", 8, 64, 3648, 96, 32), ("packed", 8, 64, 3584, 97, 32), ("rowmajor", 8, 64, 3648, 97, 32), ("mxfp4", 8, 64, 3584, 32, 32)]


@pytest.mark.parametrize("fmt,E,H,F,rows,width", WAVE_COLUMNS)
def test_wave_columns_of_the_rule(fmt, E, H, F, rows, width, monkeypatch):
    """Narrower gate-up waves than 32 columns, as the launch rule takes them, give the bits of 32 columns, and plain products."""
    print("case", fmt, E, H, F, rows, "columns", width, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + F)
    x, Wg = torch.randn((rows, H), generator=gen, device=DEV).bfloat16(), (torch.randn((H, E), generator=gen, device=DEV) * 0.02).bfloat16()
    k = min(E, 32)
    w, W, hold = make(fmt, Wg, E, H, F, gen)
    prio = torch.zeros(rows, dtype=torch.uint8, device=DEV)
    outs = []
    for cols in (None, "32"):
        if cols:
            monkeypatch.setenv("QMOE_GATE_UP_WAVE_COLUMNS", cols)
        ctx = q.Context(E, k, H, F, q.MOE_BF16, 256, rows, device=DEV)
        ctx.route(x, w)
        ctx.permute(prio)
        assert ctx.expert_run(x, w) == q.MOE_DONE
        outs.append((ctx.get("act").clone(), ctx.get("expert_out").clone()))
        torch.cuda.synchronize()
    assert torch.equal(outs[0][0].view(torch.int16), outs[1][0].view(torch.int16)) and torch.equal(outs[0][1], outs[1][1])
    if k == E:
        for e in range(E):                              # sorted order: expert by expert, tokens ascending
            assert error(outs[0][1][e * rows: (e + 1) * rows], x, W, e) <= bar("bf16", H, F)
