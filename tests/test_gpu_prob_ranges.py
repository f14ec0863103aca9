"""Mean-of-probabilities stage over the forms its terms take, by the spread of the
logits: the series of degree 4 (|s y| <= 1/16), 5 / 6 (<= 1/8), 8 (<= 1/2), the
exponential, and the exponential with the row maximum as reference (beyond 60), in
the register-resident and the two-pass kernel.

Tolerance of e = p - 1/2 against the float64 oracle: a logit carries the rounding of
a float32 dot product, at most a few 2^-24 of A = max_{t,n} s sum_i |q_i k_i|; it
moves a probability by that much relatively and e by at most a quarter of it:
|d e| <= 1e-7 + 4 * 2^-24 A.
"""
import numpy as np
import pytest

import oracle as O
import synth
from _helpers import log, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2608_23253_amd")

# (head_dim, num_text, grid): resident with 4, 3, 2 and 1 query blocks (385 and 576
# tokens at its ends), two-pass with one and two query chunks, one token, a tile and
# one key more than a tile
SHAPES = [(128, 64, (24, 24)), (64, 37, (23, 19)), (128, 20, (5, 77)), (64, 3, (24, 24)),
          (128, 65, (24, 24)), (64, 150, (9, 11)), (128, 8, (1, 1)), (64, 5, (4, 4)),
          (128, 33, (1, 17))]
# element deviation: s y within 1/16; to 1/8; to 1/2; beyond; beyond 60
SPREADS = [0.06, 0.14, 0.25, 1.0, 5.0]


def _cfg(d, nt, grid, dtype, std):
    return synth.Config("ranges", 130, batch=1, num_layers=1, num_heads=2, num_kv_heads=1,
                        head_dim=d, num_text=nt, grid_h=grid[0], grid_w=grid[1], keep=1,
                        lambdas=(0.1,), cells=1, dtype=dtype, salient_count=1, clusters=0,
                        value_std=std)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("shape", SHAPES, ids=[f"d{d}_q{t}_{g[0]}x{g[1]}" for d, t, g in SHAPES])
def test_spread_of_the_logits(shape, dtype):
    d, nt, grid = shape
    for std in SPREADS:
        cfg = _cfg(d, nt, grid, dtype, std)
        q, k, _ = synth.gen_batch(cfg)
        e, _ = E.score_heads(to_device(q, dtype), to_device(k, dtype), *grid, "mean_prob")
        torch.cuda.synchronize()
        ref = O.prune_image(q[0], k[0], *grid, 1, 1, 0.1, "mean_prob").p - 0.5
        a = float(np.einsum("lhtd,lgnd->lhtgn", np.abs(q[0]), np.abs(k[0])).max()) / np.sqrt(d)
        err = float(np.abs(e[0].cpu().numpy().astype(np.float64) - ref).max())
        bound = 1e-7 + 4 * 2.0 ** -24 * a
        log(f"  {shape} {dtype} std {std}: max|de| = {err:.2e} (bound {bound:.2e})")
        assert err <= bound


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("std", SPREADS)
def test_resident_heads_of_a_mixed_batch(dtype, std):
    """Images the register-resident kernel takes alone give the same bits in a ragged
    batch with images it does not take (where the two-pass kernel runs them)."""
    dims = [(24, 24, 64, 30), (9, 11, 30, 9), (5, 77, 17, 20), (20, 22, 48, 12), (24, 24, 70, 9)]
    gens = []
    for gh, gw, nt, keep in dims:
        cfg = synth.Config("mixed", 131, batch=1, num_layers=2, num_heads=4, num_kv_heads=2,
                           head_dim=64, num_text=nt, grid_h=gh, grid_w=gw, keep=keep,
                           lambdas=(0.1,), dtype=dtype, salient_count=4, clusters=0,
                           value_std=std)
        q, k, _ = synth.gen_batch(cfg)
        gens.append((to_device(q, dtype), to_device(k, dtype)))
    images, *_ = E.packed_images(dims, 2, 4, 2, 64)
    qa = torch.cat([q.reshape(-1) for q, _ in gens])
    ka = torch.cat([k.reshape(-1) for _, k in gens])
    keep, fused, prio = E.prune_ragged(qa, ka, images, 2, 4, 2, 64, mode="mean_prob",
                                       want_fused=True, want_prio=True)
    for im, (q, k) in zip(images, gens):
        n = im.grid_h * im.grid_w
        kb, fb, pb = E.prune(q, k, im.grid_h, im.grid_w, im.keep, mode="mean_prob",
                             want_fused=True, want_prio=True)
        torch.cuda.synchronize()
        assert torch.equal(prio[im.token_offset:im.token_offset + n], pb[0])
        assert torch.equal(fused[im.token_offset:im.token_offset + n], fb[0])
        assert torch.equal(keep[im.keep_offset:im.keep_offset + im.keep], kb[0])


@pytest.mark.parametrize("power", [-40, -20, -15, 18, 20, 24])
@pytest.mark.parametrize("shape", [(64, 64, (24, 24)), (64, 70, (24, 24)), (64, 18, (5, 77))],
                         ids=lambda s: f"q{s[1]}_{s[2][0]}x{s[2][1]}")
def test_scale_far_from_one(shape, power):
    """The same logits with a scale 2^power / sqrt(d) and the queries divided by 2^power
    (exact in bf16): the powers of the scale in a series' coefficients must not leave
    float32's range.  Tolerance as above."""
    d, nt, grid = shape
    for std in SPREADS:
        cfg = _cfg(d, nt, grid, "bf16", std)
        q, k, _ = synth.gen_batch(cfg)
        scale = 2.0 ** power / np.sqrt(d)
        e, _ = E.score_heads(to_device(q * np.float32(2.0 ** -power), "bf16"), to_device(k, "bf16"),
                             *grid, "mean_prob", scale=scale)
        torch.cuda.synchronize()
        ref = O.prune_image(q[0], k[0], *grid, 1, 1, 0.1, "mean_prob").p - 0.5
        a = float(np.einsum("lhtd,lgnd->lhtgn", np.abs(q[0]), np.abs(k[0])).max()) / np.sqrt(d)
        err = float(np.abs(e[0].cpu().numpy().astype(np.float64) - ref).max())
        log(f"  {shape} scale 2^{power}/8 std {std}: max|de| = {err:.2e}")
        assert err <= 1e-7 + 4 * 2.0 ** -24 * a
