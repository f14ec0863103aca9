"""The mean-of-logits score of calls with few heads, where all waves of a workgroup
share one head: the same bits as the one-wave-per-head kernel that larger batches
take, at the edges of key batches (8 x 4 rows for 16-bit d = 128, 4 x 4 for fp32,
twice that for d = 64), of the shares of the stores (64 tokens) and of the query
rows requested at once, near-uniform and spread out."""
import pytest

import synth
from _helpers import log, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2608_23253_amd")

COPIES = 64          # x 32 heads: enough units for one wave per head


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f16", 128), ("f32", 128),
                                     ("f32", 64)])
@pytest.mark.parametrize("std", [-1.0, 1.0])
def test_few_heads_equal_many(dtype, d, std):
    for grid, nt in (((1, 63), 1), ((8, 8), 63), ((5, 13), 64), ((1, 127), 65), ((3, 43), 3),
                     ((16, 16), 129), ((1, 257), 2), ((24, 24), 64), ((25, 41), 17)):
        cfg = synth.Config("split", 140, batch=1, num_layers=1, num_heads=32, num_kv_heads=32,
                           head_dim=d, num_text=nt, grid_h=grid[0], grid_w=grid[1], keep=1,
                           lambdas=(0.1,), cells=1, dtype=dtype, salient_count=2, clusters=0,
                           value_std=std)
        q, k, _ = synth.gen_batch(cfg)
        qd, kd = to_device(q, dtype), to_device(k, dtype)
        log(f"  {dtype} d={d} std={std} {grid} N_T={nt}")
        e1, r1 = E.score_heads(qd, kd, *grid, want_r=True)
        rep = (COPIES, 1, 1, 1, 1)
        em, rm = E.score_heads(qd.repeat(rep), kd.repeat(rep), *grid, want_r=True)
        torch.cuda.synchronize()
        for b in (0, COPIES - 1):
            assert torch.equal(em[b], e1[0]) and torch.equal(rm[b], r1[0])
