"""Grouped-query heads with fp16 keys: the query means split into three fp16 terms
after a power-of-two scaling.  Means from far below fp16's smallest normal to its
largest, a head without any query value, chunks of 1 to 16 heads, token counts at
the edges of a 16-key tile.

Tolerance of e against the float64 oracle: a few float32 roundings of a dot product,
|d e| <= 1e-7 + 4 * 2^-24 A with A = max_{h,n} scale sum_i |qbar_i k_i|."""
import numpy as np
import pytest

import oracle as O
import synth
from _helpers import log, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2608_23253_amd")


@pytest.mark.parametrize("heads,kv", [(2, 1), (14, 2), (16, 1), (34, 2)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("gain", [2.0 ** -13, 1.0, 2.0 ** 9])
def test_query_magnitudes(heads, kv, d, gain):
    for grid in ((1, 1), (3, 5), (4, 4), (1, 17), (11, 12)):
        cfg = synth.Config("f16group", 141, batch=1, num_layers=1, num_heads=heads,
                           num_kv_heads=kv, head_dim=d, num_text=5, grid_h=grid[0],
                           grid_w=grid[1], keep=1, lambdas=(0.1,), cells=1, dtype="f16",
                           salient_count=1, clusters=0)
        q, k, _ = synth.gen_batch(cfg)
        q = (q * np.float32(gain)).astype(np.float16).astype(np.float32)
        q[:, :, heads - 1] = 0.0
        scale = 1.0 / np.sqrt(d)
        e, _ = E.score_heads(to_device(q, "f16"), to_device(k, "f16"), *grid)
        torch.cuda.synchronize()
        ref = O.prune_image(q[0], k[0], *grid, 1, 1, 0.1, "mean_logit").p - 0.5
        qbar = np.abs(q[0].astype(np.float64).mean(2))                   # [L, H, d]
        kk = np.abs(np.repeat(k[0].astype(np.float64), heads // kv, axis=1))
        a = float(np.einsum("lhd,lhnd->lhn", qbar, kk).max()) * scale
        err = float(np.abs(e[0].cpu().numpy().astype(np.float64) - ref).max())
        bound = 1e-7 + 4 * 2.0 ** -24 * a
        log(f"  H={heads}/{kv} d={d} gain={gain} {grid}: {err:.2e} (bound {bound:.2e})")
        assert err <= bound
        assert (e[0, :, heads - 1] == 0).all()


@pytest.mark.parametrize("heads,kv", [(2, 1), (14, 2), (16, 1)])
def test_keys_masked_by_infinity(heads, kv):
    """Tokens masked by keys of -inf (all elements, or one) under positive queries: their
    logits are -inf, their attention 0 (e = -1/2), the others' as without them."""
    d, grid, masked = 64, (5, 13), (0, 17, 40)
    cfg = synth.Config("f16mask", 142, batch=1, num_layers=1, num_heads=heads, num_kv_heads=kv,
                       head_dim=d, num_text=5, grid_h=grid[0], grid_w=grid[1], keep=1,
                       lambdas=(0.1,), cells=1, dtype="f16", salient_count=1, clusters=0,
                       value_std=1.0)
    q, k, _ = synth.gen_batch(cfg)
    q = np.maximum(np.abs(q), np.float32(2.0 ** -4))
    k[:, :, :, masked[:2]] = -np.inf
    k[:, :, :, masked[2], 3] = -np.inf
    e, r = E.score_heads(to_device(q, "f16"), to_device(k, "f16"), *grid, want_r=True)
    torch.cuda.synchronize()
    e, r = e[0].cpu().numpy().astype(np.float64), r[0].cpu().numpy()
    assert (e[..., list(masked)] == -0.5).all() and (r[..., list(masked)] == 0).all()
    _, p = O.score_heads(q[0], k[0])
    # the bound above, A over the keys that count
    kk = np.abs(np.repeat(np.where(np.isfinite(k[0]), k[0], 0).astype(np.float64), heads // kv, axis=1))
    a = float(np.einsum("lhd,lhnd->lhn", q[0].astype(np.float64).mean(2), kk).max()) / np.sqrt(d)
    err = float(np.abs(e - (p - 0.5)).max())
    log(f"  H={heads}/{kv}: {err:.2e}")
    assert err <= 1e-7 + 4 * 2.0 ** -24 * a


@pytest.mark.parametrize("heads,kv", [(7, 1), (16, 1)])
@pytest.mark.parametrize("outlier", [2.0 ** 10, 2.0 ** 18])
def test_outlier_dimension(heads, kv, outlier):
    """One dimension of the queries far above the others, where the keys are 0, so that the
    logits are the small dimensions' alone: the bound above over these, and what the split
    drops, 2^-38 of the largest mean per dimension."""
    d, grid = 64, (11, 12)
    cfg = synth.Config("f16out", 143, batch=1, num_layers=1, num_heads=heads, num_kv_heads=kv,
                       head_dim=d, num_text=5, grid_h=grid[0], grid_w=grid[1], keep=1,
                       lambdas=(0.1,), cells=1, dtype="f16", salient_count=1, clusters=0,
                       value_std=1.0)
    q, k, _ = synth.gen_batch(cfg)
    q = (q * np.float32(2.0 ** -4)).astype(np.float16).astype(np.float32)
    q[..., 5] = np.float32(outlier * 2.0 ** -4)
    k[..., 5] = 0.0
    e, _ = E.score_heads(to_device(q, "f16"), to_device(k, "f16"), *grid)
    torch.cuda.synchronize()
    ref = O.prune_image(q[0], k[0], *grid, 1, 1, 0.1, "mean_logit").p - 0.5
    qbar = np.abs(q[0].astype(np.float64).mean(2))
    kk = np.abs(np.repeat(k[0].astype(np.float64), heads // kv, axis=1))
    small = float(np.einsum("lhd,lhnd->lhn", qbar, kk).max()) / np.sqrt(d)
    dropped = float(kk.sum(-1).max()) * float(qbar.max()) / np.sqrt(d)
    err = float(np.abs(e[0].cpu().numpy().astype(np.float64) - ref).max())
    log(f"  H={heads} outlier {outlier}: {err:.2e}")
    assert err <= 1e-7 + 4 * 2.0 ** -24 * small + 2.0 ** -38 * dropped


@pytest.mark.parametrize("heads,kv", [(7, 1), (16, 1)])
def test_subnormal_keys(heads, kv):
    """Keys below fp16's smallest normal number (2^-14) count at their values."""
    d, grid = 64, (11, 12)
    cfg = synth.Config("f16sub", 144, batch=1, num_layers=1, num_heads=heads, num_kv_heads=kv,
                       head_dim=d, num_text=5, grid_h=grid[0], grid_w=grid[1], keep=1,
                       lambdas=(0.1,), cells=1, dtype="f16", salient_count=1, clusters=0,
                       value_std=1.0)
    q, k, _ = synth.gen_batch(cfg)
    q = (q * np.float32(2.0 ** 12)).astype(np.float16).astype(np.float32)
    k = (k * np.float32(2.0 ** -17)).astype(np.float16).astype(np.float32)
    assert np.abs(k).max() < 2.0 ** -14
    e, _ = E.score_heads(to_device(q, "f16"), to_device(k, "f16"), *grid)
    torch.cuda.synchronize()
    ref = O.prune_image(q[0], k[0], *grid, 1, 1, 0.1, "mean_logit").p - 0.5
    qbar = np.abs(q[0].astype(np.float64).mean(2))
    kk = np.abs(np.repeat(k[0].astype(np.float64), heads // kv, axis=1))
    a = float(np.einsum("lhd,lhnd->lhn", qbar, kk).max()) / np.sqrt(d)
    err = float(np.abs(e[0].cpu().numpy().astype(np.float64) - ref).max())
    log(f"  H={heads}: {err:.2e} of {np.abs(ref).max():.2e}")
    assert np.abs(ref).max() > 1e-3 and err <= 1e-7 + 4 * 2.0 ** -24 * a
