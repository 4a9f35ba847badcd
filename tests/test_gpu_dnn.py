"""GPU parity of the first fully-connected layer under DES (Section 4.3): the matrix-core kernels,
through the C interface, against the CPU oracle on the same seeded inputs.  Shapes span several
128x128 output tiles with ragged edges in every dimension, shards with unequal numbers of fields,
shards with none, and enough samples that the weight gradient is computed in slices."""
import numpy as np
import pytest

from paper_1909_04823_amd import synth
from _harness import assert_close, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def des():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1909_04823_amd import des as d
    return d


SHAPES = [
    # B, F, D, H, K
    (1, 2, 4, 4, 4),          # one sample, more shards than fields
    (300, 7, 8, 200, 3),      # ragged everywhere, D below the k tile
    (257, 26, 16, 256, 8),    # Criteo-like layer
    (130, 5, 64, 132, 2),     # D of several k tiles
    (5000, 3, 4, 132, 1),     # many samples: sliced weight gradient
    (2049, 10, 32, 64, 16),
    # contractions deeper than 1024 products take the two-level summation kernel
    (40000, 2, 4, 8, 1),      # weight gradient, 2512 samples per slice
    (64, 40, 32, 16, 1),      # forward, 1280 products per shard
    (8, 2, 4, 1100, 2),       # g_pool, 1100 hidden units
]


@pytest.mark.parametrize("B,F,D,H,K", SHAPES)
def test_dnn_layer_matches_oracle(oracle, des, B, F, D, H, K):
    import torch
    pool, W, dY = synth.dnn_layer_inputs(B * 31 + F, B, F, D, H)
    Y_ref = oracle.dnn_partial_forward(pool, W, K)
    g_ref, dW_ref = oracle.dnn_backward(pool, W, dY)
    print(f"dnn case B={B} F={F} D={D} H={H} K={K}", flush=True)
    pool_g, W_g, dY_g = dev(pool, torch), dev(W, torch), dev(dY, torch)
    nan = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    Yp = des.dnn_partial_forward(pool_g, W_g, K, out=nan(K, B, H))
    Y = des.aggregate_partials(Yp)
    g_pool, dW = nan(B, F, D), nan(F * D, H)
    ws = torch.empty(des.dnn_backward_bytes(B, F, D, H), dtype=torch.uint8, device="cuda")
    des.dnn_backward(pool_g, W_g, dY_g, g_pool, dW, ws)
    torch.cuda.synchronize()
    assert_close(Yp.cpu().numpy(), Y_ref, "Y_partial")
    assert_close(Y.cpu().numpy(), oracle.aggregate(Y_ref), "Y")
    assert_close(g_pool.cpu().numpy(), g_ref, "g_pool")
    assert_close(dW.cpu().numpy(), dW_ref, "dW")
    # each output alone
    g2, dW2 = nan(B, F, D), nan(F * D, H)
    des.dnn_backward(pool_g, W_g, dY_g, g2, None, None)
    des.dnn_backward(pool_g, W_g, dY_g, None, dW2, ws)
    torch.cuda.synchronize()
    assert torch.equal(g2, g_pool) and torch.equal(dW2, dW)


def test_dnn_layer_argument_checks(des):
    import torch
    pool = torch.zeros((4, 2, 4), device="cuda"); W = torch.zeros((8, 8), device="cuda")
    with pytest.raises(des.DesError):
        des.dnn_partial_forward(pool, W, 0)                       # K < 1
    with pytest.raises(des.DesError):
        des.dnn_partial_forward(torch.zeros((4, 2, 6), device="cuda"), torch.zeros((12, 8), device="cuda"), 2)  # D % 4
    with pytest.raises(des.DesError):
        des.dnn_partial_forward(pool, torch.zeros((8, 6), device="cuda"), 2)   # H % 4
    dY = torch.zeros((4, 8), device="cuda")
    with pytest.raises(des.DesError):
        des.dnn_backward(pool, W, dY, None, None)                  # no output asked for
    big = torch.zeros((5000, 2, 4), device="cuda")
    with pytest.raises(des.DesError) as e:                         # dW summed over slices of samples needs the workspace
        des.dnn_backward(big, W, torch.zeros((5000, 8), device="cuda"), None, torch.zeros((8, 8), device="cuda"), None)
    assert e.value.code == des.ERR_WORKSPACE
    # empty batch: nothing launched, nothing written
    out = des.dnn_partial_forward(torch.zeros((0, 2, 4), device="cuda"), W, 2)
    assert out.shape == (2, 0, 8)


def test_dnn_forward_of_more_workgroups_than_a_row_of_the_grid(des):
    """65537 row tiles times 256 shards, one of them with a field: 2^24 and some workgroups, more threads than a launch takes along one
    dimension."""
    import torch
    B, K = 4194304 + 64, 256
    pool, W, _ = synth.dnn_layer_inputs(1, B, 1, 4, 4)
    Y = torch.full((K, B, 4), float("nan"), dtype=torch.float32, device="cuda")
    des.dnn_partial_forward(dev(pool, torch), dev(W, torch), K, out=Y)
    torch.cuda.synchronize()
    assert_close(Y[0].cpu().numpy(), pool.reshape(B, 4).astype(np.float64) @ W.astype(np.float64), "Y_partial of the shard with a field")
    for s in range(1, K):
        assert not Y[s].any(), s
    del Y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("F,D,bound", [(300, 4, 1.6e-7), (200, 8, 1.8e-7), (150, 12, 2.0e-7), (100, 16, 2.2e-7), (100, 20, 1.93e-7), (50, 36, 2.0e-7)])
def test_dnn_forward_sums_deep_shards_in_short_runs(des, F, D, bound):
    """A sum of more than 1024 products is taken in runs of at most 8 * D / ceil(D/16) products, 128 where D fills 16-deep tiles: its
    2-norm error, which grows with the run's length, stays within 4 % of what a chain of that length leaves (1.54, 1.73, 1.94,
    2.14, 1.87 and 1.95 e-7 on inputs of this kind)."""
    import torch
    pool, W, _ = synth.dnn_layer_inputs(F, 4096, F, D, 128)
    Y = des.dnn_partial_forward(dev(pool, torch), dev(W, torch), 1).cpu().numpy()[0]
    ref = pool.reshape(4096, F * D).astype(np.float64) @ W.astype(np.float64)
    assert np.linalg.norm(Y - ref) <= bound * np.linalg.norm(ref)


def _gradients(des, torch, pool, W, dY):
    B, F, D = pool.shape
    g_pool = torch.full((B, F, D), float("nan"), dtype=torch.float32, device="cuda")
    dW = torch.full(W.shape, float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(des.dnn_backward_bytes(B, F, D, W.shape[1]), dtype=torch.uint8, device="cuda")
    des.dnn_backward(dev(pool, torch), dev(W, torch), dev(dY, torch), g_pool, dW, ws)
    torch.cuda.synchronize()
    return g_pool.cpu().numpy().reshape(B, F * D), dW.cpu().numpy()


# both tile sizes, ragged in every dimension; fields that are not a multiple of the k tile, several fields per k tile
@pytest.mark.parametrize("B,F,D,H,K", [(12801, 8, 100, 128, 3), (1601, 9, 20, 388, 7), (65, 33, 4, 68, 2), (4097, 3, 12, 36, 5)])
def test_dnn_products_at_tile_edges(des, B, F, D, H, K):
    import torch
    pool, W, dY = synth.dnn_layer_inputs(B + F, B, F, D, H)
    x, w, g = pool.reshape(B, F * D).astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    Y = des.dnn_partial_forward(dev(pool, torch), dev(W, torch), K).cpu().numpy()
    for s in range(K):
        cols = np.concatenate([np.arange(f * D, (f + 1) * D) for f in range(s, F, K)]) if s < F else np.zeros(0, int)
        assert_close(Y[s], x[:, cols] @ w[cols], f"Y_partial shard {s}")
    g_pool, dW = _gradients(des, torch, pool, W, dY)
    assert_close(g_pool, g @ w.T, "g_pool")
    assert_close(dW, x.T @ g, "dW")


@pytest.mark.parametrize("B,F,D,H", [(300, 7, 8, 200), (12801, 8, 100, 128)])     # small and large tiles
def test_dnn_gradients_of_infinities_nans_and_extreme_magnitudes(des, B, F, D, H):
    """Infinities and NaN reach exactly the outputs that plain fp32 arithmetic sends them to; operands so small that bf16
    parts cannot hold them, and so large that their leading part would round up to infinity, lose nothing."""
    import torch
    pool, W, dY = synth.dnn_layer_inputs(B + 1, B, F, D, H)
    pool.reshape(B, -1)[5, 3] = np.inf
    dY[7, 2] = -np.inf
    dY[B - 1, H - 1] = np.nan
    W[1, 1] = np.inf
    x, w, g = pool.reshape(B, F * D).astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    with np.errstate(invalid="ignore"):
        refs = g @ w.T, x.T @ g
    for got, ref, what in zip(_gradients(des, torch, pool, W, dY), refs, ("g_pool", "dW")):
        fin = np.isfinite(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~fin & ~np.isnan(ref)], ref[~fin & ~np.isnan(ref)]), what
        assert_close(got[fin], ref[fin], what)
    # a power of two on one operand and its inverse on the other leave every product as it is
    pool, W, dY = synth.dnn_layer_inputs(B + 2, B, F, D, H)
    up, down = np.float32(2.0 ** 112), np.float32(2.0 ** -112)
    x, w, g = pool.reshape(B, F * D).astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    g_pool, _ = _gradients(des, torch, pool, W * up, dY * down)
    assert_close(g_pool, g @ w.T, "g_pool, dY tiny")
    _, dW = _gradients(des, torch, pool * up, W, dY * down)
    assert_close(dW, x.T @ g, "dW, dY tiny")
    W[0, 0] = np.float32(3.4e38)
    g_pool, _ = _gradients(des, torch, pool, W, dY * np.float32(1e-3))
    ref = (g * 1e-3) @ W.astype(np.float64).T
    assert np.isfinite(g_pool).all()
    assert np.all(np.abs(g_pool - ref) <= np.maximum(1e-5 * np.abs(ref), 1e-6))


@pytest.mark.parametrize("B,F,D,H", [(300, 7, 8, 200), (12801, 8, 100, 128)])     # small and large tiles
def test_dnn_gradients_that_overflow_are_infinite(des, B, F, D, H):
    """A product beyond fp32's range, and a sum of finite products that leaves it, make an infinity of the sign that fp32
    arithmetic gives; no NaN, and the other outputs keep their values."""
    import torch
    pool, W, dY = synth.dnn_layer_inputs(B + 3, B, F, D, H)
    dY[7, 5], dY[9, 6] = 1.37 * 2.0 ** 70, 1.37 * 2.0 ** 100
    W[3, 5], W[4, 6] = 1.21 * 2.0 ** 70, -1.21 * 2.0 ** 60
    pool.reshape(B, -1)[7, 2], pool.reshape(B, -1)[9, 1] = 1.43 * 2.0 ** 79, -1.11 * 2.0 ** 75
    dY[200, :], W[-1, :] = 2.0 ** 63, 2.0 ** 64           # each product 2^127, their sum past the range (in a tile of its own)
    x, w, g = pool.reshape(B, F * D).astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    with np.errstate(over="ignore"):
        refs = (g @ w.T).astype(np.float32), (x.T @ g).astype(np.float32)
    assert np.isinf(refs[0]).sum() >= 3 and np.isinf(refs[1]).sum() >= 2
    for got, ref, what in zip(_gradients(des, torch, pool, W, dY), refs, ("g_pool", "dW")):
        fin = np.isfinite(ref)
        assert np.array_equal(got[~fin], ref[~fin]), what
        # 2^-21 of the sum of the magnitudes: a chain of up to 12801 products, each huge element met by ordinary ones
        mag = (np.abs(g) @ np.abs(w.T)) if what == "g_pool" else (np.abs(x.T) @ np.abs(g))
        assert np.all(np.abs(got[fin].astype(np.float64) - ref[fin]) <= 2.0 ** -21 * mag[fin]), what


@pytest.mark.parametrize("exponent", [-112, -110, -109, -108, -107, -105, -103, -102, -100])
def test_dnn_gradients_of_operands_with_subnormal_parts(des, exponent):
    """Operands of one binade whose third bf16 part is subnormal, or (below 2^-110) cannot hold what is left, against large ones: the sums
    of 64 and 512 products keep the error of ordinary operands (1.45e-7 and 1.3e-7 in fp32 arithmetic, 3 % added; without
    the third part it would be some 1e-6)."""
    import torch
    rng = np.random.default_rng(-exponent)
    one = lambda *s: (rng.uniform(1, 2, s) * rng.choice([-1.0, 1.0], s)).astype(np.float32)
    pool, W, dY = one(512, 8, 16), one(128, 64), one(512, 64)
    small, large = np.float32(2.0 ** exponent), np.float32(2.0 ** 40)
    x, w, g = pool.reshape(512, 128).astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    g_pool, _ = _gradients(des, torch, pool, W * large, dY * small)
    _, dW = _gradients(des, torch, pool * large, W, dY * small)
    for got, ref, bound in ((g_pool, g @ w.T, 1.5e-7), (dW, x.T @ g, 1.35e-7)):
        assert np.linalg.norm(got.astype(np.float64) * 2.0 ** (-40 - exponent) - ref) <= bound * np.linalg.norm(ref)


@pytest.mark.parametrize("B,F,D,H", [
    (300, 7, 8, 60), (300, 7, 8, 64), (300, 7, 8, 68), (300, 7, 8, 96),            # g_pool: thirds, halves, a last half tile, none
    (300, 7, 8, 1024), (300, 7, 8, 1028), (300, 7, 8, 1536),                       # ... one stretch, several of 512 and a short one, whole ones
    (2000, 130, 16, 132), (2000, 130, 16, 1060),                                   # large tiles
    (1024, 7, 8, 36), (16400, 3, 4, 36), (17000, 30, 64, 260),                     # dW: slices of 64, 1040 and 1072 samples or more
])
def test_dnn_gradients_of_rows_of_any_magnitude(des, B, F, D, H):
    """Operand rows from 1 down to 2^-90 of each other, in both products; rows that begin with zeros, and go on small; single elements
    that are 2^20 times their row's others.  Bound, for each output by the sum of its products' magnitudes: a product from halves is off by
    up to 3 * 2^-24 (two cuts and the term left out), one in fp32 by 2^-24, and each of at most min(k, 1024) roundings of a partial sum,
    which is no larger than that sum, by 2^-24 (to nearest; the 16-bit instruction's by 2^-23, one per 16 products); taken as independent,
    six standard deviations.  Without the rests of a cut it would be 2^-12 per product."""
    rng = np.random.default_rng(B + H)
    pool, W, dY = synth.dnn_layer_inputs(B + H, B, F, D, H)
    pool = pool.reshape(B, F * D)
    dY *= np.exp2(-rng.integers(0, 30, (B, 1)) * rng.integers(0, 4, (B, 1))).astype(np.float32)   # a sample's gradients
    pool *= np.exp2(-rng.integers(0, 20, (1, F * D))).astype(np.float32)                          # a column's embeddings
    W *= np.exp2(-rng.integers(0, 20, (F * D, 1))).astype(np.float32)
    dY[5, :40], pool[:40, 3], W[2, :40] = 0, 0, 0
    dY[6, 34], W[4, 35] = dY[6, 34] * np.float32(2 ** 20), W[4, 35] * np.float32(2 ** 20)
    dY[7, :40] = 0
    dY[7, 40:] = rng.standard_normal(H - 40).astype(np.float32) * np.float32(2.0 ** -80) if H > 40 else 0     # (products stay normal)
    x, w, g = pool.astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    g_pool, dW = _gradients(des, __import__("torch"), pool.reshape(B, F, D), W, dY)
    for got, ref, mag, k, what in ((g_pool, g @ w.T, np.abs(g) @ np.abs(w.T), H, "g_pool"), (dW, x.T @ g, np.abs(x.T) @ np.abs(g), B, "dW")):
        assert np.all(np.abs(got - ref) <= 6 * 2.0 ** -24 * np.sqrt(9 + min(k, 1024)) * mag), what


@pytest.mark.parametrize("B,F,D,H", [
    (64, 4, 8, 16), (64, 4, 8, 64), (1100, 4, 8, 32), (1100, 4, 8, 64),      # small tiles; thirds or halves for either product
    (2000, 60, 16, 256),                                                    # large tiles for dW alone, small ones for g_pool alone
    (5003, 27, 20, 300), (16640, 26, 16, 256), (20000, 50, 32, 256),        # large tiles; dW of several stretches per slice
    (131072, 2, 16, 64), (1100, 100, 32, 16),                               # two launches
    (2, 7, 8, 64),
])
def test_dnn_gradients_together_and_alone(des, B, F, D, H):
    """Both gradients from one launch have the bits that each has from a launch of its own."""
    import torch
    pool, W, dY = (dev(a, torch) for a in synth.dnn_layer_inputs(B, B, F, D, H))
    ws = torch.empty(des.dnn_backward_bytes(B, F, D, H), dtype=torch.uint8, device="cuda")
    out = [torch.full((B, F, D), float("nan"), device="cuda") for _ in range(2)], [torch.full((F * D, H), float("nan"), device="cuda") for _ in range(2)]
    des.dnn_backward(pool, W, dY, out[0][0], out[1][0], ws)
    des.dnn_backward(pool, W, dY, out[0][1], None, None)
    des.dnn_backward(pool, W, dY, None, out[1][1], ws)
    assert torch.equal(out[0][0], out[0][1]) and torch.equal(out[1][0], out[1][1])
    rows = slice(0, 500)
    assert_close(out[0][0].view(B, -1)[rows].cpu().numpy(), (dY[rows].double() @ W.double().t()).cpu().numpy(), "g_pool")
    assert_close(out[1][0][rows].cpu().numpy(), (pool.view(B, -1)[:, rows].double().t() @ dY.double()).cpu().numpy(), "dW")


@pytest.mark.parametrize("B", [1, 2, 3])
def test_dnn_weight_gradient_of_a_few_samples(des, B):
    """One product is rounded once, to nearest; the sum of two or three loses no more than fp32 arithmetic does (2-norm errors 3.1e-8
    and 3.6e-8, 3 % added)."""
    import torch
    pool, W, dY = synth.dnn_layer_inputs(B, B, 26, 16, 256)
    _, dW = _gradients(des, torch, pool, W, dY)
    ref = pool.reshape(B, 416).astype(np.float64).T @ dY.astype(np.float64)
    if B == 1:
        assert np.array_equal(dW, ref.astype(np.float32))
    assert np.linalg.norm(dW - ref) <= {1: 2.6e-8, 2: 3.2e-8, 3: 3.7e-8}[B] * np.linalg.norm(ref)


@pytest.mark.parametrize("H", [64, 128, 200, 256, 300, 400, 1100])     # one run of 128 products, odd and even numbers of them
def test_dnn_gradients_of_zeros_are_plus_zero(des, H):
    import torch
    pool, W, dY = synth.dnn_layer_inputs(H, 300, 7, 8, H)
    dY[:] = 0
    for got, what in zip(_gradients(des, torch, pool, W, dY), ("g_pool", "dW")):
        assert not got.view(np.int32).any(), what


@pytest.mark.parametrize("B,F,D,H", [(4096, 26, 16, 64), (4096, 26, 16, 128), (4096, 26, 16, 300), (4096, 26, 16, 1100),   # g_pool: 1, 1, 3, 9 runs
                                     (2048, 26, 16, 256), (300, 26, 16, 256)])   # dW: slices of one or two runs
def test_dnn_gradients_have_no_mean_error(des, B, F, D, H):
    """Also where the number of runs is odd.  The mean of n independent errors of the size `err` is within 6 err / sqrt(n); with the
    instruction's rounding towards minus infinity left in, it is up to 100 times err / sqrt(n) here."""
    import torch
    pool, W, dY = synth.dnn_layer_inputs(B + H, B, F, D, H)
    x, w, g = pool.reshape(B, F * D).astype(np.float64), W.astype(np.float64), dY.astype(np.float64)
    for got, ref, what in zip(_gradients(des, torch, pool, W, dY), (g @ w.T, x.T @ g), ("g_pool", "dW")):
        err = got - ref
        assert abs(err.mean()) <= 6 * np.sqrt((err * err).mean() / err.size), what


def test_dnn_weight_gradient_has_no_drift(des):
    """The matrix instruction's rounding towards minus infinity must not pile up over a long sum: the mean error over 4096 sums of
    3344 products per slice (uncorrected -3e-7 of the results' root mean square, its standard error 4e-9) stays below 3e-8."""
    import torch
    pool, W, dY = synth.dnn_layer_inputs(3, 40003, 4, 16, 64)
    _, dW = _gradients(des, torch, pool, W, dY)
    ref = pool.reshape(40003, 64).astype(np.float64).T @ dY.astype(np.float64)
    assert abs((dW - ref).mean()) < 3e-8 * np.sqrt((ref * ref).mean())


@pytest.mark.parametrize("opt", ["OPT_SGD", "OPT_ADAGRAD", "OPT_ADAM", "OPT_FTRL"])
def test_dense_update_of_many_arrays(des, opt):
    """The same bits as one call per array, over more arrays than a launch takes: empty ones, single values, edges of workgroups."""
    import torch
    sizes = [1, 0, 255, 256, 257, 1000, 3, 70000, 1, 511, 512, 513, 2, 4096, 4097, 65, 64, 0, 12345, 7]
    gen = torch.Generator(device="cuda").manual_seed(3)

    def arrays():
        gen.manual_seed(3)
        return [tuple(torch.rand(n, generator=gen, device="cuda") + 0.1 for _ in range(4)) for n in sizes]

    o = des.Optimizer(opt_emb=getattr(des, opt), lr=0.05, eps=1e-8, beta1=0.9, beta2=0.999, step=3, ftrl_alpha=0.05, ftrl_beta=1.0,
                      ftrl_l1=0.01, ftrl_l2=0.1)
    one, many = arrays(), arrays()
    for theta, g, s1, s2 in one:
        des.dense_update(theta, g, o, s1, s2)
    des.dense_update_many(many, o)
    for a, b in zip(one, many):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
