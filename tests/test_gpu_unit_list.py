"""Expert kernels over the device's unit list (more row segments than fit the kernel arguments)."""
import pytest
import torch

import paper_2503_09304_amd as q

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def make(dtype, E, k, H, F, N, n_ls, chunk, seed):
    print("case", dtype, E, k, H, F, N, n_ls, chunk, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def t(shape, std):
        return (torch.randn(shape, generator=g, device=DEV) * std).to(dt)

    x, Wg, W1, W3, W2 = t((N, H), 1.0), t((H, E), 0.02), t((E, F, H), H ** -0.5), t((E, F, H), H ** -0.5), t((E, H, F), F ** -0.5)
    prio = torch.zeros(N, dtype=torch.uint8, device=DEV)
    prio[torch.randperm(N, generator=g, device=DEV)[:n_ls]] = 1
    ctx = q.Context(E, k, H, F, q.MOE_F32 if dtype == "f32" else q.MOE_BF16, chunk, N, device=DEV)
    w = q.Context.weights(Wg, W1, W3, W2)
    ctx.route(x, w)
    ctx.permute(prio)
    counts = ctx.get("counts").sum(1)
    assert int(((counts + 255) // 256).sum()) > 384                  # so a launch of everything reads the unit list
    return ctx, x, w, (W1, W3, W2), prio, Wg


def expert_out(ctx, x, W, k):
    """The expert outputs of the batch in float64, in sorted order, from plain products."""
    W1, W3, W2 = W
    E = W1.shape[0]
    off = ctx.get("offsets").tolist()
    tok = ctx.get("perm").long() // k
    out = torch.empty((tok.numel(), x.shape[1]), dtype=torch.float64, device=DEV)
    for e in range(E):
        rows = slice(off[2 * e], off[2 * e + 2])
        xe = x[tok[rows]].double()
        g, u = xe @ W1[e].double().t(), xe @ W3[e].double().t()
        out[rows] = (g / (1 + torch.exp(-g)) * u) @ W2[e].double().t()
    return out


def bar(dtype, H, F):
    """max|err| / RMS.  fp32: a sum of K terms of random signs is off by about 2^-24 * sqrt(K), the largest of a tensor's
    errors by 6 times that, and twice over for the two products.  bf16: the rounding of the activation, 2e-2 as for
    the named workloads."""
    return 4 * 2.0 ** -24 * 6 * (H ** 0.5 + F ** 0.5) if dtype == "f32" else 2e-2


def check(ctx, x, W, k, dtype):
    got, ref = ctx.get("expert_out").double(), expert_out(ctx, x, W, k)
    assert ((got - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= bar(dtype, x.shape[1], W[0].shape[1])


@pytest.mark.parametrize("dtype,H,F,cols", [("f32", 32, 8192, 32), ("bf16", 64, 32768, 128)])
def test_more_workgroups_than_one_launch_holds(dtype, H, F, cols):
    """70000 units of one row x 256 column tiles are 2^24.1 workgroups of 256 threads: more than a launch can hold."""
    ctx, x, w, W, _, _ = make(dtype, 256, 1, H, F, 70000, 0, 1, 3)
    assert ctx.cursor.n_units * ((F + cols - 1) // cols) >= 1 << 24
    assert ctx.expert_run(x, w) == q.MOE_DONE
    torch.cuda.synchronize()
    check(ctx, x, W, 1, dtype)


@pytest.mark.parametrize("dtype,H,F", [("f32", 64, 100), ("f32", 33, 72), ("bf16", 512, 1408), ("bf16", 320, 1152)])
def test_same_bits_whole_cut_enqueued_and_scattered(dtype, H, F):
    """One launch over the unit list, its first 100 units as segments, the enqueued (counted) launch, and scattered units
    in launches of at most 384 segments: the same outputs, bit for bit; the first against plain products."""
    k, N = 8, 16384
    ctx, x, w, W, prio, Wg = make(dtype, 64, k, H, F, N, 4000, 256, 5)
    nu = ctx.cursor.n_units
    y = torch.zeros_like(x)

    def result():
        ctx.combine(y)
        out = ctx.get("expert_out").clone()
        torch.cuda.synchronize()
        return out, y.clone()

    def again():
        ctx.get("expert_out").fill_(float("nan"))
        ctx.route(x, w)
        ctx.permute(prio)

    assert ctx.expert_run(x, w) == q.MOE_DONE
    base = result()
    check(ctx, x, W, k, dtype)

    again()
    assert ctx.expert_run(x, w, 100) == q.MOE_OK and ctx.expert_run(x, w) == q.MOE_DONE
    cut = result()
    again()
    assert ctx.expert_enqueue(x, w, q.UINT32_MAX) == q.MOE_OK and ctx.expert_collect() == q.MOE_DONE
    queued = result()
    again()
    rest = [u for u in range(nu) if u % 5]                       # 4 of 5 units: runs of rows broken up, in several launches
    assert len(rest) > 384
    assert ctx.expert_run_units(x, w, rest) == q.MOE_OK and ctx.expert_run(x, w) == q.MOE_DONE
    scattered = result()
    for other in (cut, queued, scattered):
        assert all(torch.equal(a, b) for a, b in zip(base, other))
