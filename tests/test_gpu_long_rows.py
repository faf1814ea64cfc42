"""Weight rows so long that the rows of one wave span more than 4 GiB: bf16 expert kernels against plain products in fp64.
Weights of 13 to 27 GB."""
import pytest
import torch

import paper_2503_09304_amd as q

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def product(a, w):
    """a [N, K] times w [R, K] transposed in float64, a slice of K at a time."""
    out = torch.zeros((a.shape[0], w.shape[0]), dtype=torch.float64, device=DEV)
    for k in range(0, a.shape[1], 1 << 22):
        out += a[:, k: k + (1 << 22)].double() @ w[:, k: k + (1 << 22)].double().t()
    return out


def close(got, ref, K, rounding):
    """fp32 sums of K terms of random signs: off by about 2^-24 * sqrt(K) of their RMS, the largest by 6 times that, and twice over
    (two factors in the activation); rounding: of the value itself, 2^-8 if it is a bf16."""
    sums = 2 * 6 * 2.0 ** -24 * K ** 0.5
    return bool(((got.double() - ref).abs() <= rounding * ref.abs() + sums * ref.pow(2).mean().sqrt()).all())


# down projection with 64 rows of W2 a wave, with 32; gate-up; gate-up with waves that lie in two row tiles
@pytest.mark.parametrize("fmt,H,F,N,cols", [("rowmajor", 64, 34_560_000, 33, 0), ("rowmajor", 64, 69_312_512, 2, 0), ("rowmajor", 69_312_512, 64, 2, 0),
                                            ("packed", 69_312_512, 64, 2, 28)])
def test_long_rows(fmt, H, F, N, cols, monkeypatch):
    print("case", fmt, H, F, N, cols, flush=True)
    if torch.cuda.mem_get_info()[0] < 70e9:
        pytest.skip("needs 70 GB of free GPU memory")
    if cols:
        monkeypatch.setenv("QMOE_GATE_UP_WAVE_COLUMNS", str(cols))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(H + F)

    def t(shape, std):
        return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=gen)

    x, Wg = t((N, H), 1.0), t((H, 1), 0.02)
    W = [t((1, F, H), H ** -0.5), t((1, F, H), H ** -0.5), t((1, H, F), F ** -0.5)]
    w = q.Context.weights(Wg, *W)
    if fmt == "packed":
        hold = [torch.empty((16, H), dtype=torch.bfloat16, device=DEV)] + [torch.empty_like(v) for v in W]
        p = q.Context.weights(*hold)
        q.moe_pack_weights(q.MoeConfig(1, 1, H, F, q.MOE_BF16, 1, 0), w, p)
        w = p
    ctx = q.Context(1, 1, H, F, q.MOE_BF16, 256, N, device=DEV)
    ctx.route(x, w)
    ctx.permute(torch.zeros(N, dtype=torch.uint8, device=DEV))
    assert ctx.expert_run(x, w) == q.MOE_DONE
    act, out = ctx.get("act").clone(), ctx.get("expert_out").clone()     # one expert: sorted rows are the tokens in order
    torch.cuda.synchronize()
    for f in range(0, F, 1 << 22):
        g, u = (product(x, v[0, f: f + (1 << 22)]) for v in W[:2])
        assert close(act[:, f: f + (1 << 22)], g / (1 + torch.exp(-g)) * u, H, 2.0 ** -8)
    assert close(out, product(act, W[2][0]), F, 0.0)
    del x, Wg, W, w, ctx, act, out, g, u
    torch.cuda.empty_cache()
