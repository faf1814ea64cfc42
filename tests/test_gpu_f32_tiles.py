"""fp32 expert kernels at the edges of their tiles: rows per unit around 16, 32, 64 and 256, K (H for
gate-up, F for the down projection) below, at and beside multiples of 32 (the remainder of K is a
guarded tile of its own), output columns beside multiples of 64, rows that are only 4-byte aligned.

Bar: an fp32 sum of K terms has an error of at most about K * 2^-24 times the sum of the terms'
magnitudes; for random signs max|err|/RMS stays near 2^-24 * sqrt(K) * (largest of the elements, 6), twice
over for the two chained products: 2e-5 covers K = 520 four times over."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from gpu_util import GpuLayer, rel_err, to_host
from test_gpu_parity import bits

pytestmark = pytest.mark.gpu

CASES = [  # E, k, H, F, N, n_ls, chunk
    (1, 1, 1, 1, 1, 0, 1),
    (1, 1, 31, 33, 15, 3, 256),
    (2, 1, 32, 64, 40, 8, 16),
    (1, 1, 64, 32, 65, 1, 64),
    (3, 2, 33, 95, 100, 17, 33),
    (4, 2, 97, 130, 129, 40, 256),
    (1, 1, 63, 520, 257, 0, 256),
    (8, 8, 100, 65, 300, 300, 255),
    (16, 1, 128, 96, 33, 7, 17),
]


@pytest.mark.parametrize("E,k,H,F,N,n_ls,chunk", CASES)
def test_f32_tiles(E, k, H, F, N, n_ls, chunk):
    cfg = wl.LayerConfig("f32_tiles", dtype="f32", seed=77, E=E, k=k, H=H, F=F, N=N, n_ls=n_ls, chunk_rows=chunk)
    print("case", wl.describe(cfg), flush=True)
    inp = wl.make_inputs(cfg)
    g = GpuLayer(inp).full()
    r = g.fetch("logits", "topk_idx", "perm", "y")
    lay = oracle.OracleLayer(inp.x, inp.w, inp.prio, inp.bias, k, chunk, logits=r["logits"].astype(np.float64))
    lay.run()
    y_ref, comp = lay.y()
    assert comp.all()
    assert np.array_equal(lay.idx, r["topk_idx"]) and np.array_equal(lay.perm, r["perm"])
    assert rel_err(to_host(g.ctx.get("expert_out")), lay.O) <= 2e-5
    assert rel_err(wl.as_f64(r["y"]), y_ref) <= 2e-5
    nu = g.ctx.cursor.n_units                    # every unit on its own: the same bits
    h = GpuLayer(inp).full(tuple(range(1, nu))[:20])
    assert torch.equal(bits(h.y), bits(g.y))
