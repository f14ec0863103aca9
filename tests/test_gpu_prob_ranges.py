"""Mean-of-probabilities stage over the forms its terms take, by the spread of the
logits: the series of degree 4 (|s y| <= 1/16), 5 / 6 (<= 1/8), 8 (<= 1/2), the
exponential or, for chunks with a row near its mean, expm1, and the exponential with the row maximum as reference (beyond 60), in
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


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("std", SPREADS)
@pytest.mark.parametrize("nt", [64, 40, 20, 9])
def test_small_heads_of_a_resident_batch(nt, std, dtype):
    """Images too small for the register-resident kernel by themselves (one token, fewer
    tiles than waves, 384 tokens) that it takes beside larger ones, and those beside so
    many small ones that the two-pass kernel takes the batch: the bits of each alone."""
    large = [(24, 24, nt), (5, 77, nt // 2 + 1)]
    small = [(1, 1, 3), (3, 5, nt), (4, 4, 1), (1, 17, nt), (9, 11, nt // 2), (16, 24, nt), (5, 13, 7)]
    alone = {}

    def image(i, dims):
        gh, gw, t = dims
        cfg = synth.Config("small", 132 + i, batch=1, num_layers=1, num_heads=2, num_kv_heads=1,
                           head_dim=64, num_text=t, grid_h=gh, grid_w=gw, keep=1, lambdas=(0.1,),
                           cells=1, dtype=dtype, salient_count=1, clusters=0, value_std=std)
        q, k = [to_device(x, dtype) for x in synth.gen_batch(cfg)[:2]]
        return q, k, E.prune(q, k, gh, gw, 1, cells=1, mode="mean_prob", want_fused=True)[1][0]

    # the fullest eighth of the heads: all 36 and 25 tiles; an eighth of 16 large images;
    # few large ones among the small
    for batch in (large + small[:1] + small, large * 8 + small * 16, small * 17 + large):
        gens = []
        for dims in batch:
            if dims not in alone:
                alone[dims] = image(len(alone), dims)
            gens.append(alone[dims])
        images, *_ = E.packed_images([(*d, 1) for d in batch], 1, 2, 1, 64)
        q, k = [torch.cat([g[i].reshape(-1) for g in gens]) for i in (0, 1)]
        _, fused, _ = E.prune_ragged(q, k, images, 1, 2, 1, 64, cells=1, mode="mean_prob",
                                     want_fused=True)
        torch.cuda.synchronize()
        for im, g in zip(images, gens):
            n = im.grid_h * im.grid_w
            assert torch.equal(fused[im.token_offset:im.token_offset + n], g[2])


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


# Deviations of the queries' elements (keys: 1), so of the rows' logits: just beyond the
# degree-8 series, rows near their mean among spread ones, chunks of different forms
# (128 queries each) in both orders.
ROWS = {"0.13": [.13] * 64, "0.2": [.2] * 64, "0.3": [.3] * 64, "1": [1.] * 64,
        "60x0.01,4x0.5": [.01] * 60 + [.5] * 4, "63x0.005,0.2": [.005] * 63 + [.2],
        "63x0.02,2": [.02] * 63 + [2.], "32x0.1,32x1": [.1] * 32 + [1.] * 32,
        "128x0.01,22x1": [.01] * 128 + [1.] * 22, "22x1,128x0.01": [1.] * 22 + [.01] * 128,
        "128x1,22x0.01": [1.] * 128 + [.01] * 22, "20x0.2": [.2] * 20,
        "47x0.01,0.7": [.01] * 47 + [.7]}


def _rows(stds, grid, dtype, heads, seed):
    """q [1, 1, heads, N_T, 64] of the given deviations and k [1, 1, heads, N, 64], as stored."""
    rng = np.random.default_rng(seed)
    q = rng.normal(size=(1, 1, heads, len(stds), 64)) * np.asarray(stds)[:, None]
    k = rng.normal(size=(1, 1, heads, grid[0] * grid[1], 64))
    return [synth._round_storage(x.astype(np.float32), dtype) for x in (q, k)]


def _u64(q, k):
    """u = N r - 1 in float64, and the rounding its terms carry: about ten roundings of half
    an ulp (the product's sums, the argument, the term, the weight, the column sums) of
    values of the size of s z N P and N P - 1, independent over the rows: their rms is
    below 2 * 2^-24 of the returned mean."""
    z = np.einsum("hti,hni->htn", q[0, 0].astype(np.float64), k[0, 0].astype(np.float64)) / 8.0
    x = z.shape[-1] * O.softmax_over_visual(z)
    size = np.sqrt(((z * x) ** 2).mean(-1) + ((x - 1) ** 2).mean(-1))
    return x.mean(1) - 1, float(np.sqrt((size ** 2).sum(-1) / z.shape[1] ** 2).max())


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("grid", [(24, 24), (32, 32), (9, 11)])
def test_rows_of_different_spread(grid, dtype):
    for name, stds in ROWS.items():
        q, k = _rows(stds, grid, dtype, 8, 150)
        e, _ = E.score_heads(to_device(q, dtype), to_device(k, dtype), *grid, "mean_prob")
        torch.cuda.synchronize()
        e = e[0, 0].cpu().numpy().astype(np.float64)
        ref, size = _u64(q, k)
        err = float(np.sqrt(((4 * e / (1 - 2 * e) - ref) ** 2).mean()))
        log(f"  {grid} {dtype} {name}: rms du = {err:.2e}, {err / size * 2 ** 24:.2f} * 2^-24")
        assert err <= 4 * 2.0 ** -24 * size


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_rows_of_different_spread_in_both_kernels(dtype):
    """A register-resident head and the same head beside one of 70 queries (the two-pass
    kernel) have the same bits."""
    for name, stds in ROWS.items():
        if len(stds) > 64:
            continue
        heads = [_rows(s, (24, 24), dtype, 4, 151) for s in (stds, [.1] * 70)]
        images, *_ = E.packed_images([(24, 24, len(stds), 9), (24, 24, 70, 9)], 1, 4, 4, 64)
        q, k = [to_device(np.concatenate([h[i].ravel() for h in heads]), dtype) for i in (0, 1)]
        _, fused, prio = E.prune_ragged(q, k, images, 1, 4, 4, 64, mode="mean_prob",
                                        want_fused=True, want_prio=True)
        _, fa, pa = E.prune(to_device(heads[0][0], dtype), to_device(heads[0][1], dtype), 24, 24, 9,
                            mode="mean_prob", want_fused=True, want_prio=True)
        torch.cuda.synchronize()
        log(f"  {dtype} {name}")
        assert torch.equal(prio[:576], pa[0]) and torch.equal(fused[:576], fa[0])


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("stds", [[1.] * 64, [.01] * 63 + [1.], [1.] * 16], ids=len)
@pytest.mark.parametrize("grid", [(24, 24), (32, 32), (5, 7)])
def test_keys_of_infinity_and_nan(grid, stds, dtype):
    """Keys of -inf under positive queries have attention 0 (the maximum becomes the
    reference); keys of +inf or NaN make their own head NaN and no other."""
    q, k = _rows(stds, grid, dtype, 4, 152)
    q = np.maximum(np.abs(q), np.float32(2.0 ** -14))
    k[:, :, 0, (0, 20)] = -np.inf
    k[:, :, 1, 33] = np.nan
    k[:, :, 2, 2] = np.inf
    e, _ = E.score_heads(to_device(q, dtype), to_device(k, dtype), *grid, "mean_prob")
    torch.cuda.synchronize()
    e = e[0, 0].cpu().numpy().astype(np.float64)
    assert np.isnan(e[1:3]).all()
    for h in (0, 3):
        ref, _ = _u64(q[:, :, h:h + 1], np.where(np.isinf(k[:, :, h:h + 1]), -1e9, k[:, :, h:h + 1]))
        # (every logit rounds by a few 2^-24 of s sum |q k| <= 30 here, and u = -1 as well)
        err = float(np.abs(4 * e[h] / (1 - 2 * e[h]) - ref[0]).max())
        log(f"  {grid} {dtype} {len(stds)} head {h}: max du = {err:.2e}")
        assert err <= 4 * 2.0 ** -24 * 30 * (1 + np.abs(ref).max())
    assert np.abs(e[0, [0, 20]] + 0.5).max() <= 2.0 ** -22
