"""fp32 expert kernels over the device's unit list (more row segments than fit the kernel arguments)."""
import pytest
import torch

import paper_2503_09304_amd as q

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def make(E, k, H, F, N, n_ls, chunk, seed):
    print("case", E, k, H, F, N, n_ls, chunk, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)

    def t(shape, std):
        return torch.randn(shape, generator=g, device=DEV) * std

    x, Wg, W1, W3, W2 = t((N, H), 1.0), t((H, E), 0.02), t((E, F, H), H ** -0.5), t((E, F, H), H ** -0.5), t((E, H, F), F ** -0.5)
    prio = torch.zeros(N, dtype=torch.uint8, device=DEV)
    prio[torch.randperm(N, generator=g, device=DEV)[:n_ls]] = 1
    ctx = q.Context(E, k, H, F, q.MOE_F32, chunk, N, device=DEV)
    w = q.Context.weights(Wg, W1, W3, W2)
    ctx.route(x, w)
    ctx.permute(prio)
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


# A sum of K fp32 terms is off by at most K * 2^-24 of the sum of their magnitudes; for random signs the largest
# of a tensor's errors is about 2^-24 * sqrt(K) * 6 of its RMS, twice over for the two products.
def bar(H, F):
    return 4 * 2.0 ** -24 * 6 * (H ** 0.5 + F ** 0.5)


def test_more_workgroups_than_one_launch_takes():
    """70000 units of one row x 8192 columns are 2^24.1 workgroups of 256 threads: more than a launch can hold."""
    E, H, F, N = 256, 32, 8192, 70000
    ctx, x, w, W, _, _ = make(E, 1, H, F, N, 0, 1, 3)
    counts = ctx.get("counts").sum(1)
    assert int(((counts + 255) // 256).sum()) > 384                  # so the launch reads the unit list
    assert ctx.cursor.n_units * ((F + 31) // 32) >= 1 << 24
    assert ctx.expert_run(x, w) == q.MOE_DONE
    torch.cuda.synchronize()
    got, ref = ctx.get("expert_out").double(), expert_out(ctx, x, W, 1)
    assert ((got - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= bar(H, F)
