"""GPU kernels at the sizes where they can go wrong: edges of tiles, remainders, the smallest and largest of a range."""
import numpy as np
import pytest

import coe_workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_02354_amd import binding
    return binding


@pytest.mark.parametrize("n,E", [(1, 2048), (63, 511), (64, 512), (65, 513), (511, 1), (2047, 370), (2048, 370), (2049, 370),
                                 (4097, 2048), (100003, 370), (262144, 33), (262145, 33), (300001, 600)])
def test_regroup_range_edges(B, oracle, n, E):
    """One workgroup up to 2048 keys, then ranges of 2048, then longer ranges beyond 128 workgroups."""
    rng = np.random.default_rng(n + E)
    cur = np.where(rng.random(n) < 0.8, rng.choice(E, size=n, p=W.zipf_probs(E, 1.1)), rng.choice([-1, E, E + 5], size=n)).astype(np.int32)
    ctx = B.Context(max_requests=n)
    got = ctx.coe_debug_regroup(cur, E)
    ctx.close()
    want = oracle.regroup(np.where(cur < E, cur, -1).astype(np.int32), E)
    for k in ("cnt", "off", "perm", "inv"):
        assert np.array_equal(got[k], want[k]), k


@pytest.mark.parametrize("n,H,Wd,C,K,R,stride,pad,use_res,act", [
    (2, 64, 64, 3, 16, 3, 1, 1, False, 1),        # contiguous patch rows, fewer than 32 filters
    (3, 17, 15, 16, 32, 3, 1, 1, True, 0),        # one block of 16 channels, ragged tiles
    (2, 33, 20, 32, 64, 3, 1, 1, False, 1),       # two filter blocks
    (600, 7, 7, 64, 128, 3, 1, 1, True, 1),       # more tiles than resident workgroups, several channel blocks
    (700, 5, 9, 8, 40, 3, 1, 1, False, 0),        # resident workgroups walk several tiles and two filter tiles of 64
    (2, 31, 31, 24, 66, 3, 2, 1, True, 3),        # channels in blocks of 8, stride 2, filters not a multiple of 4
    (2, 40, 37, 3, 64, 7, 2, 3, False, 2),        # 7x7 stride 2 on an image
    (1, 6, 5, 5, 7, 1, 1, 0, True, 1),            # 1x1, odd everything
    (1, 3, 3, 256, 10, 3, 1, 1, False, 0),        # one small tile
])
def test_conv_f32_elementwise(B, oracle, n, H, Wd, C, K, R, stride, pad, use_res, act):
    rng = np.random.default_rng(n * 1000 + H * 10 + K)
    x = rng.standard_normal((n, H, Wd, C)).astype(np.float32)
    w = (rng.standard_normal((K, R, R, C)) * np.sqrt(2.0 / (R * R * C))).astype(np.float32)
    bias = rng.standard_normal(K).astype(np.float32)
    P = (H + 2 * pad - R) // stride + 1; Q = (Wd + 2 * pad - R) // stride + 1
    res = rng.standard_normal((n, P, Q, K)).astype(np.float32) if use_res else None
    ctx = B.Context(max_requests=1)
    got, _ = ctx.coe_debug_conv(0, x, w, bias, res, stride, pad, act)
    ctx.close()
    some = range(n) if n <= 8 else sorted(set([0, 1, n - 1] + list(rng.integers(0, n, 20))))
    for i in some:
        r = None if res is None else res[i]
        want = oracle.conv2d(x[i], w, bias, r, stride, pad, act, 0)
        # a sum of m fp32 products in any order is off by at most m * 2^-24 times the sum of the absolute products (first
        # order); bias and residual are two terms more; the activations' slopes stay below 1.13, their own evaluation adds
        # a few roundings of the result
        mag = oracle.conv2d(np.abs(x[i]), np.abs(w), np.abs(bias), None if r is None else np.abs(r), stride, pad, 0, 0)
        bound = 1.13 * (R * R * C + 2) * 2.0 ** -24 * mag + 8 * 2.0 ** -24 * np.abs(want) + (1e-6 * mag if act >= 2 else 0)
        assert np.all(np.abs(got[i] - want) <= bound), float((np.abs(got[i] - want) / bound).max())


def _spread(bad, R, stride, pad, P, Q):
    """Outputs whose window holds one of the image positions `bad` (h, w)."""
    hit = np.zeros((P, Q), bool)
    for h, w in bad:
        for p in range(P):
            for q in range(Q):
                hit[p, q] |= 0 <= h - (p * stride - pad) < R and 0 <= w - (q * stride - pad) < R
    return hit


@pytest.mark.parametrize("H,Wd,C,K,R,stride,pad,act", [
    (20, 21, 3, 16, 3, 1, 1, 0), (20, 21, 3, 40, 3, 1, 1, 1), (19, 33, 5, 7, 3, 1, 1, 0), (18, 18, 5, 64, 5, 1, 2, 1),
    (40, 37, 3, 64, 7, 2, 3, 1), (9, 9, 3, 8, 1, 1, 0, 0), (17, 18, 16, 32, 3, 1, 1, 0), (17, 18, 8, 64, 3, 2, 1, 1),
])
def test_conv_f32_keeps_non_finite_pixels_to_their_windows(B, oracle, H, Wd, C, K, R, stride, pad, act):
    """An infinite or NaN pixel reaches the outputs whose window holds it and no other: those have the bits they have with
    the pixel replaced."""
    rng = np.random.default_rng(H * 10 + C)
    x = rng.standard_normal((1, H, Wd, C)).astype(np.float32)
    w = (rng.standard_normal((K, R, R, C)) * np.sqrt(2.0 / (R * R * C))).astype(np.float32)
    bias = rng.standard_normal(K).astype(np.float32)
    P = (H + 2 * pad - R) // stride + 1; Q = (Wd + 2 * pad - R) // stride + 1
    bad = [(3, 5), (H - 1, Wd - 1), (0, Wd // 2), (H // 2, 0)]
    ctx = B.Context(max_requests=1)
    base, _ = ctx.coe_debug_conv(0, x, w, bias, None, stride, pad, act)
    for value in (np.inf, -np.inf, np.nan):
        xb = x.copy()
        for i, (h, wd) in enumerate(bad):
            xb[0, h, wd, i % C] = value
        got, _ = ctx.coe_debug_conv(0, xb, w, bias, None, stride, pad, act)
        hit = _spread(bad, R, stride, pad, P, Q)
        assert np.array_equal(got[0][~hit], base[0][~hit]), value
        if act == 0:
            want = oracle.conv2d(xb[0], w, bias, None, stride, pad, act, 0)
            assert np.array_equal(np.isnan(got[0][hit]), np.isnan(want[hit])) and np.array_equal(got[0][hit] > 0, want[hit] > 0)
            assert not np.isfinite(got[0][hit]).any()
    ctx.close()


@pytest.mark.parametrize("H,Wd,C,K,R,stride,pad,act", [
    (20, 21, 3, 40, 3, 1, 1, 0), (33, 18, 16, 64, 3, 1, 1, 1), (40, 37, 3, 64, 7, 2, 3, 2), (50, 50, 136, 32, 3, 1, 1, 0),
])
def test_conv_f32_keeps_non_finite_filters_off_the_padding(B, oracle, H, Wd, C, K, R, stride, pad, act):
    """A filter value that is not finite does not reach outputs for which it falls on the zero padding."""
    rng = np.random.default_rng(H * 10 + C)
    x = rng.standard_normal((2, H, Wd, C)).astype(np.float32)
    w = (rng.standard_normal((K, R, R, C)) * np.sqrt(2.0 / (R * R * C))).astype(np.float32)
    w[1, 0, 1, C - 1], w[K - 1, R - 1, R - 1, 0] = np.inf, np.nan
    bias = rng.standard_normal(K).astype(np.float32)
    ctx = B.Context(max_requests=1)
    got, _ = ctx.coe_debug_conv(0, x, w, bias, None, stride, pad, act)
    ctx.close()
    for i in range(2):
        want = oracle.conv2d(x[i], w, bias, None, stride, pad, act, 0)
        finite = np.isfinite(want)
        assert finite[0, :, 1].all() and finite[-1, :, K - 1].all()
        assert not np.isfinite(want[2, 2, [1, K - 1]]).any() or act
        assert np.array_equal(np.isnan(got[i]), np.isnan(want)) and np.array_equal(np.isinf(got[i]), np.isinf(want))
        wf = np.where(np.isfinite(w), np.abs(w), 0)
        mag = oracle.conv2d(np.abs(x[i]), wf, np.abs(bias), None, stride, pad, 0, 0)
        # as in test_conv_f32_elementwise
        bound = 1.13 * (R * R * C + 2) * 2.0 ** -24 * mag + 8 * 2.0 ** -24 * np.abs(want) + (1e-6 * mag if act >= 2 else 0)
        assert np.all(np.abs(got[i][finite] - want[finite]) <= bound[finite])


@pytest.mark.parametrize("H,Wd,C,K,R,stride,pad,n", [
    (20, 14, 64, 64, 3, 1, 1, 300),       # channel blocks that 32-filter tiles alone would make larger
    (7, 7, 32, 128, 3, 1, 1, 300), (2, 2, 16, 72, 3, 1, 1, 600), (30, 17, 3, 64, 7, 2, 3, 150), (3, 3, 64, 100, 1, 1, 0, 260),
    (17, 1, 24, 64, 3, 1, 1, 300),
])
def test_conv_f32_bits_do_not_depend_on_the_batch(B, H, Wd, C, K, R, stride, pad, n):
    """Few images run on tiles of 32 filters, many on tiles of 64, and rows of a tile below a small map are left out: the same
    image gives the same bits alone and among many."""
    rng = np.random.default_rng(H + C + K)
    x = rng.standard_normal((3, H, Wd, C)).astype(np.float32)
    w = rng.standard_normal((K, R, R, C)).astype(np.float32)
    bias = rng.standard_normal(K).astype(np.float32)
    ctx = B.Context(max_requests=1)
    one, _ = ctx.coe_debug_conv(0, x[:1], w, bias, None, stride, pad, 1)
    many, _ = ctx.coe_debug_conv(0, x[np.arange(n) % 3], w, bias, None, stride, pad, 1)
    ctx.close()
    assert np.array_equal(many[0], one[0]) and np.array_equal(many, many[np.arange(n) % 3])


@pytest.mark.parametrize("H,C,K,R,pad,n", [(1, 64, 40, 3, 1, 70), (1, 100, 16, 5, 2, 3), (2, 8, 24, 4, 1, 5)])
def test_conv_f32_of_one_pixel_on_padding(B, H, C, K, R, pad, n):
    """An output of one pixel whose window lies on the padding for the most part goes to the plain kernel: one chain of
    multiply-adds over the window positions inside the image (1 x 1 map, 3 x 3 window, 512 -> 512, 512 images: 276 us, 4813 in tiles)."""
    rng = np.random.default_rng(C + K)
    x = rng.standard_normal((n, H, H, C)).astype(np.float32)
    w = rng.standard_normal((K, R, R, C)).astype(np.float32)
    bias = rng.standard_normal(K).astype(np.float32)
    ctx = B.Context(max_requests=1)
    got, _ = ctx.coe_debug_conv(0, x, w, bias, None, 1, pad, 0)
    ctx.close()
    acc = np.zeros((n, K), np.float32)
    for r in range(R):
        for t in range(R):
            if 0 <= r - pad < H and 0 <= t - pad < H:
                for c in range(C):       # the product of two fp32 numbers is exact in 64 bits
                    acc = (acc.astype(np.float64) + x[:, r - pad, t - pad, c, None].astype(np.float64) * w[:, r, t, c]).astype(np.float32)
    assert got.shape == (n, 1, 1, K)
    # 64-bit sums rounded to fp32 twice: a tie in 2^29 of them may fall differently
    assert np.mean(got[:, 0, 0] == acc + bias) > 0.999


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_expert_with_a_non_finite_filter(B, oracle, value):
    """The same through an expert that is registered with such a filter, beside one without."""
    import torch
    arch = W.tiny_cnn(4, 32)
    blob = W.make_expert_blob(arch, 7, 0).copy()
    sp = next(sp for sp in W.blob_layout(arch)[0] if sp.layer == 0 and sp.name == "w")
    clean = blob.copy()
    w = blob[sp.offset:sp.offset + sp.nbytes].view(np.float32).reshape(sp.shape)
    w[2, 0, 0, 1] = value
    x = np.random.default_rng(3).standard_normal((2, 32, 32, 3)).astype(np.float32)
    dev = torch.from_numpy(x).cuda()
    ctx = B.Context(max_requests=2, max_batch=2)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, blob, 1.0)
    ctx.coe_register_expert(1, aid, clean, 1.0)
    shape = (2, 32, 32, sp.shape[0])
    got = [ctx.coe_debug_layer_output(e, 2, dev.data_ptr(), 0, shape, np.float32).reshape(shape) for e in (0, 1)]
    ctx.close()
    act = int(arch.layers[0][9])
    for i in range(2):
        want = oracle.conv2d(x[i], w, W.blob_tensor(arch, blob, 0, "b"), None, 1, 1, act, 0)
        assert np.isfinite(want[0, :, 2]).all() and np.array_equal(np.isfinite(got[0][i]), np.isfinite(want))
        np.testing.assert_allclose(np.where(np.isfinite(want), got[0][i], 0), np.where(np.isfinite(want), want, 0), rtol=1e-5, atol=1e-5)
        assert np.isfinite(got[1][i]).all()


def _bf16(rng, *shape, scale=1.0):
    return W.f32_to_bf16_bits((rng.standard_normal(shape) * scale).astype(np.float32)).reshape(shape)


@pytest.mark.parametrize("use_res", [True, False])
@pytest.mark.parametrize("H,Wd,C,K,R,stride,pad,act,few,some,many", [
    (7, 7, 64, 128, 3, 1, 1, 1, 1, 200, 1200),        # slab order: 32 x 32 tiles, 64 x 64 tiles, 256-row tiles
    (9, 11, 32, 64, 3, 1, 1, 0, 3, 300, 1200),        # one channel block (the loop over block pairs ends in its middle)
    (14, 13, 96, 192, 3, 1, 1, 3, 1, 60, 400),        # three channel blocks, filters not a multiple of 128
    (15, 15, 64, 128, 3, 2, 1, 1, 2, 250, 1300),      # stride 2: window positions outside, two channel blocks a stage
    (14, 14, 128, 256, 1, 2, 0, 0, 1, 200, 1400),     # 1x1 projection, four channel blocks a stage
    (50, 1, 192, 64, 1, 1, 0, 2, 3, 600, 2400),       # token GEMM, odd number of stages
    (10, 10, 64, 96, 1, 1, 0, 0, 2, 0, 500),          # filters not a multiple of 64: no 64 x 64 tiles
    (12, 12, 64, 64, 5, 1, 2, 1, 1, 200, 900),        # 5x5 window
    (14, 14, 512, 256, 1, 1, 0, 1, 1, 129, 255),      # 256 x 256 tiles: 16 steps, 196 tiles, the last one ragged
    (50, 1, 768, 512, 1, 1, 0, 2, 2, 400, 2995),      # GELU, workgroups with four and with five tiles, two filter tiles
    (15, 13, 64, 256, 3, 2, 1, 3, 1, 300, 931),       # stride 2 at odd sizes, two channel blocks a window position
    (14, 14, 544, 256, 1, 2, 0, 0, 1, 400, 1045),     # strided rows, 17 steps
    (14, 14, 512, 256, 1, 1, 0, 1, 1, 120, 180),      # 192 x 256 tiles (184 of them) and 128 x 256 ones
    (50, 1, 512, 768, 1, 1, 0, 2, 2, 190, 514),       # 192 x 256 tiles in two turns, three filter tiles; 128 x 256 ones
    (9, 9, 64, 256, 3, 1, 0, 0, 1, 220, 480),         # 3x3 without padding, the same two heights
])
def test_few_tiles_give_the_bits_of_many(B, oracle, H, Wd, C, K, R, stride, pad, act, few, some, many, use_res):
    """Launches with few output tiles run on smaller tiles.  A request's result must not depend on how many requests run
    beside it: the same images alone, among some and among many give the same bits, and those of a few are the oracle's."""
    rng = np.random.default_rng(H * 100 + C + R)
    x = _bf16(rng, few + 1, H, Wd, C)
    w = _bf16(rng, K, R, R, C, scale=np.sqrt(2.0 / (R * R * C)))
    bias = (0.1 * rng.standard_normal(K)).astype(np.float32)
    P = (H + 2 * pad - R) // stride + 1; Q = (Wd + 2 * pad - R) // stride + 1
    res = _bf16(rng, few + 1, P, Q, K) if use_res else None
    ctx = B.Context(max_requests=1)
    outs = {}
    for n in (few, some, many):
        if n:
            idx = np.arange(n) % (few + 1)
            outs[n], _ = ctx.coe_debug_conv(1, x[idx], w, bias, res[idx] if use_res else None, stride, pad, act)
    ctx.close()
    for n, y in outs.items():
        for r in range(1 if n > few else 0, n // (few + 1)):
            assert np.array_equal(y[r * (few + 1):(r + 1) * (few + 1)], y[:few + 1]), (n, r)
        assert np.array_equal(y[:few], outs[few]), n
    xf, wf = (W.bf16_bits_to_f32(a).reshape(a.shape) for a in (x, w))
    rf = W.bf16_bits_to_f32(res).reshape(res.shape) if use_res else [None] * few
    want = np.stack([oracle.conv2d(xf[i], wf, bias, rf[i], stride, pad, act, 1) for i in range(few)])
    got = W.bf16_bits_to_f32(outs[few]).reshape(want.shape)
    # one bf16 ulp where fp32 and fp64 sums round to different sides; 1e-5 absolute where the terms cancel (the fp32 error
    # of a sum of up to 1600 terms of size ~0.05)
    assert np.all(np.abs(got - want) <= np.maximum(np.abs(want) * 2.0 ** -7, 1e-5))


@pytest.mark.parametrize("values", ["exponents", "cancelling", "denormal", "bits"])
@pytest.mark.parametrize("hw,C,K,R,few,some,many", [(14, 128, 256, 1, 1, 40, 300), (14, 64, 128, 3, 1, 60, 400), (7, 512, 512, 3, 2, 60, 150)])
def test_products_of_few_tiles_sum_like_those_of_many(B, hw, C, K, R, few, some, many, values):
    """A 16 x 16 x 32 product (32 x 32 tiles: few images) sums in the order of two 32 x 32 x 16 ones (64 x 64 tiles, and the kernels of many
    tiles), whatever the operands: exponents 24 powers of two apart, terms that cancel but for their last bits, products and sums in
    fp32's denormals, any finite bit patterns."""
    rng = np.random.default_rng(hw + C + R)

    def operands(*shape):
        n = int(np.prod(shape))
        if values == "bits":
            b = rng.integers(0, 1 << 16, n).astype(np.uint16)
            b[(b & 0x7F80) > 0x5D80] &= 0xBFFF                       # below 2^61: products and sums stay finite
            return b.reshape(shape)
        v = rng.standard_normal(n).astype(np.float32)
        if values == "exponents":
            v *= np.exp2(rng.integers(-12, 13, n)).astype(np.float32)
        return W.f32_to_bf16_bits(v).reshape(shape)
    x, w = operands(few + 1, hw, hw, C), operands(K, R, R, C)
    if values == "cancelling":                                       # neighbouring channels: pixels equal but for a bit, filters opposite
        x[..., 1::2] = x[..., ::2] ^ (rng.random(x[..., ::2].shape) < 0.3)
        w[..., 1::2] = w[..., ::2] ^ 0x8000
    if values == "denormal":
        x = W.f32_to_bf16_bits(np.ldexp(W.bf16_bits_to_f32(x), -128)).reshape(x.shape)
        w = W.f32_to_bf16_bits(np.ldexp(W.bf16_bits_to_f32(w), -8)).reshape(w.shape)
    bias = np.zeros(K, np.float32)
    ctx = B.Context(max_requests=1)
    outs = [ctx.coe_debug_conv(1, x[np.arange(n) % (few + 1)], w, bias, None, 1, R // 2, 0)[0] for n in (few, some, many)]
    ctx.close()
    assert np.count_nonzero(outs[0] & 0x7FFF) > outs[0].size // 2
    for y in outs[1:]:
        for i in range(0, len(y) - few, few + 1):
            assert np.array_equal(y[i:i + few], outs[0]), i


def _tiles(n, P, Q, K, side):
    return -(-n * P * Q // side) * (K // side)


@pytest.mark.parametrize("n,H,Wd,C,K,R,stride,pad,use_res,act", [
    (70, 28, 28, 64, 64, 3, 1, 1, True, 3),       # conv3x3_slab_kernel: 256 x 64 tiles, residual, SiLU
    (71, 28, 27, 64, 64, 3, 1, 1, False, 1),      # ragged rows
    (110, 14, 15, 128, 256, 3, 1, 1, False, 1),   # 256 x 128 tiles, two filter tiles
    (300, 7, 7, 64, 512, 3, 1, 1, True, 0),       # an image is less than a tile
    (90, 29, 29, 64, 128, 3, 2, 1, False, 1),     # conv_igemm_dma_kernel: stride 2 at an odd size, 128 x 128 tiles
    (41, 29, 31, 64, 64, 1, 1, 0, True, 1),       # 128 x 64 tiles, ragged
    (160, 14, 14, 128, 512, 1, 2, 0, False, 2),   # strided rows, GELU
])
def test_kernels_of_many_tiles_elementwise(B, oracle, n, H, Wd, C, K, R, stride, pad, use_res, act):
    """The slab and implicit-GEMM kernels, which launches of few tiles no longer reach: more tiles than conv_ring takes, every output
    of some images against the oracle (the first, the last and those that straddle tiles)."""
    rng = np.random.default_rng(n * 10 + K)
    P = (H + 2 * pad - R) // stride + 1; Q = (Wd + 2 * pad - R) // stride + 1
    slab = R == 3 and stride == 1
    assert _tiles(n, P, Q, K, 32) > 512 and _tiles(n, P, Q, K, 64) > (768 if slab else 512)        # kRingTiles32, kRingTiles64(Slab)
    x = _bf16(rng, n, H, Wd, C)
    w = _bf16(rng, K, R, R, C, scale=np.sqrt(2.0 / (R * R * C)))
    bias = (0.1 * rng.standard_normal(K)).astype(np.float32)
    res = _bf16(rng, n, P, Q, K) if use_res else None
    ctx = B.Context(max_requests=1)
    got, cls = ctx.coe_debug_conv(1, x, w, bias, res, stride, pad, act)
    ctx.close()
    assert B.KERNEL_CLASS_NAMES[cls] == ("conv_slab" if slab else "conv_mfma")
    wf = W.bf16_bits_to_f32(w).reshape(w.shape)
    for i in sorted({0, 1, n // 2, n - 2, n - 1} | set(rng.integers(0, n, 4).tolist())):
        r = None if res is None else W.bf16_bits_to_f32(res[i]).reshape(res[i].shape)
        want = oracle.conv2d(W.bf16_bits_to_f32(x[i]).reshape(x[i].shape), wf, bias, r, stride, pad, act, 1)
        g = W.bf16_bits_to_f32(got[i]).reshape(want.shape)
        # as in test_few_tiles_give_the_bits_of_many
        assert np.all(np.abs(g - want) <= np.maximum(np.abs(want) * 2.0 ** -7, 1e-5)), i
        assert np.mean(g == want) > 0.995


@pytest.mark.parametrize("C,pixels", [(64, 200), (64, 6000), (64, 40000), (96, 3000), (512, 33000)])
def test_gelu_rounds_like_the_fp32_path(B, C, pixels):
    """GELU in the bf16 epilogues (32 x 32 tiles, 64 x 64 tiles, 128 x 64 tiles, the register-staged kernel, persistent tiles) gives the
    rounded value of the plain formula, which fp32 experts evaluate, bit for bit: an identity convolution, so that the value before
    the activation is one fp32 sum of a bf16 number and a bias on both paths."""
    rng = np.random.default_rng(C + pixels)
    scale = np.exp(rng.uniform(np.log(1e-3), np.log(6.0), (1, pixels, 1, C)))
    x = W.f32_to_bf16_bits((rng.standard_normal((1, pixels, 1, C)) * scale).astype(np.float32)).reshape(1, pixels, 1, C)
    bias = rng.standard_normal(C).astype(np.float32)
    bias[:10] = [-np.inf, np.inf, np.nan, -13.0, -12.0, -30.0, 80.0, 1e30, -1e30, 0.0]
    eye = np.eye(C, dtype=np.float32).reshape(C, 1, 1, C)
    ctx = B.Context(max_requests=1)
    got, _ = ctx.coe_debug_conv(1, x, W.f32_to_bf16_bits(eye).reshape(eye.shape), bias, None, 1, 0, W.ACT_GELU)
    plain, _ = ctx.coe_debug_conv(0, W.bf16_bits_to_f32(x).reshape(x.shape), eye, bias, None, 1, 0, W.ACT_GELU)
    ctx.close()
    nan = np.isnan(plain)
    assert nan[..., 0].all() and nan[..., 2].all() and not nan[..., 3:].any()          # -inf * 0, as in the plain formula
    assert np.array_equal(np.isnan(W.bf16_bits_to_f32(got).reshape(got.shape)), nan)
    want = W.f32_to_bf16_bits(np.where(nan, 0, plain)).reshape(got.shape)
    assert int(np.sum((got != want) & ~nan)) == 0


@pytest.mark.parametrize("C,K,pixels", [(64, 64, 200), (64, 64, 6000), (64, 64, 40000), (96, 96, 3000), (512, 512, 33000), (4, 32, 5000)])
def test_silu_rounds_like_the_fp32_path(B, C, K, pixels):
    """SiLU in the bf16 epilogues (the kernels of the GELU test, then the one for few input channels) gives the rounded value of the plain
    formula, which fp32 experts evaluate, bit for bit: an identity convolution, so that the value before the activation is one fp32 sum of
    a bf16 number and a bias on both paths."""
    rng = np.random.default_rng(C + pixels)
    scale = np.exp(rng.uniform(np.log(1e-3), np.log(12.0), (1, pixels, 1, C)))
    x = W.f32_to_bf16_bits((rng.standard_normal((1, pixels, 1, C)) * scale).astype(np.float32)).reshape(1, pixels, 1, C)
    bias = rng.standard_normal(K).astype(np.float32)
    bias[:12] = [-np.inf, np.inf, np.nan, -9.9, 10.1, -30.0, 80.0, 1e30, -1e30, 0.0, -87.5, -89.0]
    eye = np.eye(K, C, dtype=np.float32).reshape(K, 1, 1, C)
    ctx = B.Context(max_requests=1)
    got, _ = ctx.coe_debug_conv(1, x, W.f32_to_bf16_bits(eye).reshape(eye.shape), bias, None, 1, 0, W.ACT_SILU)
    plain, _ = ctx.coe_debug_conv(0, W.bf16_bits_to_f32(x).reshape(x.shape), eye, bias, None, 1, 0, W.ACT_SILU)
    ctx.close()
    same, nan = got == W.f32_to_bf16_bits(plain).reshape(got.shape), np.isnan(plain)
    assert np.all(same | nan) and np.isnan(W.bf16_bits_to_f32(got[nan])).all() and nan[..., 2].all()


@pytest.mark.parametrize("beside", [0.0, -20.0])
@pytest.mark.parametrize("lo,hi", [(-10.0, -1.3), (-1.25, 0.0), (0.0, 10.0), (10.0, 1e6), (-20.0, -10.0), (-79.0, -20.0), (-88.0, -79.0)])
def test_silu_next_to_rounding_ties(B, lo, hi, beside):
    """Where SiLU's short form could tip a bf16 rounding: the arguments nearest to the middle of two bf16 values, and 20 on either side.
    An argument is the sum of three bf16 channels, 24 bits in all, which the matrix cores add without rounding; -20 `beside` the
    arguments makes every wavefront take the form for low values.  The bits of the plain formula, rounded."""
    rng = np.random.default_rng(abs(int(lo)) + 1)
    n = 100000
    mag = np.exp(rng.uniform(np.log(max(min(abs(lo), abs(hi)), 1e-20)), np.log(max(abs(lo), abs(hi))), n))
    x = np.where(hi <= 0, -mag, mag)
    with np.errstate(over="ignore"):
        for _ in range(4):                               # to the tie next to the result
            s = 1 / (1 + np.exp(-x))
            y = (x * s).astype(np.float32)
            tie = ((y.view(np.uint32) & 0xFFFF0000) | 0x8000).view(np.float32).astype(np.float64)
            x = np.clip(x + (tie - x * s) / (s * (1 + x * (1 - s))), lo, hi)
    x = (x.astype(np.float32).view(np.int32)[:, None] + np.arange(-20, 20, dtype=np.int32)).view(np.float32).ravel()
    x = x[np.isfinite(x)]
    args = 10                                            # a pixel
    x = x[:len(x) // args * args].reshape(-1, args)
    cols = [0, 1, 2, 3, 4, 5, 6, 8, 9, 10]               # of 16 filters; the others are `beside`
    filters = np.zeros((32, 1, 1, 32), np.float32)
    pieces, rest = np.zeros((len(x), 32), np.float32), x.copy()
    for part in range(3):
        top = (rest.view(np.uint32) & 0xFFFF0000).view(np.float32)
        pieces[:, part * args:(part + 1) * args] = top
        rest = rest - top
        filters[cols, 0, 0, part * args + np.arange(args)] = 1
    assert not rest.any()
    bias = np.full(32, beside, np.float32)
    bias[cols] = 0
    ctx = B.Context(max_requests=1)
    bits = lambda a: W.f32_to_bf16_bits(a).reshape(a.shape)
    got, _ = ctx.coe_debug_conv(1, bits(pieces)[None, :, None, :], bits(filters), bias, None, 1, 0, W.ACT_SILU)
    eye = np.eye(args, dtype=np.float32).reshape(args, 1, 1, args)
    plain, _ = ctx.coe_debug_conv(0, x[None, :, None, :], eye, np.zeros(args, np.float32), None, 1, 0, W.ACT_SILU)
    ctx.close()
    assert np.abs(plain.view(np.int32) % 65536 - 32768).min() <= 2       # ties were met
    assert np.array_equal(got[0, :, 0, cols].T, bits(plain)[0, :, 0])


@pytest.mark.parametrize("H,Wd,C,R,pad", [(14, 14, 256, 5, 2), (7, 9, 64, 5, 2), (22, 23, 32, 5, 2), (20, 20, 96, 5, 2), (13, 13, 64, 7, 3),
                                          (9, 9, 64, 5, 1), (5, 5, 32, 5, 0), (60, 60, 64, 5, 2), (14, 14, 64, 3, 1), (6, 6, 40, 5, 2)])
def test_pools_with_stride_one(B, H, Wd, C, R, pad):
    """Stride-1 pools in LDS (eight and four chunks of channels, windows larger than the rest of the map) and those that stay on the kernel
    for all pools (a map that does not fit, small windows, odd channel counts): the maximum of the window's numbers, minus infinity
    where there is none."""
    n = 3
    p = W._Prog(H, Wd, C); p.maxpool(0, 1, R, 1, pad); p.head(1, 4)
    arch = W.Arch("pool", W.DT_BF16, H, Wd, C, 4, np.array(p.layers, dtype=np.int32), p.gains)
    rng = np.random.default_rng(H * C + R)
    x = W.bf16_bits_to_f32(_bf16(rng, n, H, Wd, C)).reshape(n, H, Wd, C).copy()
    x[rng.random(x.shape) < 0.2] = -np.inf
    x[rng.random(x.shape) < 0.1] = np.nan
    x[rng.random(x.shape) < 0.1] = -3.3895e38
    x[0, :, :, 0], x[1, :, :, 1], x[2, :, :, 2] = np.nan, -np.inf, np.inf
    bits = W.f32_to_bf16_bits(x).reshape(x.shape)
    x = W.bf16_bits_to_f32(bits).reshape(x.shape)
    ctx = B.Context(max_requests=n, max_batch=n)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, W.make_expert_blob(arch, 7, 0), 1.0)
    import torch
    dev = torch.from_numpy(bits.view(np.int16)).cuda()
    P, Q = H + 2 * pad - R + 1, Wd + 2 * pad - R + 1
    got = ctx.coe_debug_layer_output(0, n, dev.data_ptr(), 0, (n, P, Q, C), np.uint16)
    ctx.close()
    padded = np.full((n, H + 2 * pad, Wd + 2 * pad, C), -np.inf, np.float32)
    padded[:, pad:pad + H, pad:pad + Wd] = x
    want = np.full((n, P, Q, C), -np.inf, np.float32)
    for r in range(R):
        for s in range(R):
            want = np.fmax(want, padded[:, r:r + P, s:s + Q])
    assert np.array_equal(W.bf16_bits_to_f32(got).reshape(want.shape), want)


@pytest.mark.parametrize("H,Wd,C,R,pad,many", [(14, 14, 64, 5, 2, 300), (14, 14, 256, 5, 2, 70), (22, 23, 32, 5, 2, 300), (20, 20, 96, 5, 2, 100),
                                               (13, 14, 128, 5, 1, 200), (7, 7, 64, 5, 2, 300), (13, 13, 64, 7, 3, 40)])
def test_pools_of_few_and_many_images_give_the_same_bits(B, H, Wd, C, R, pad, many):
    """Whether a stride-1 pool runs in LDS goes by the size of the launch too (few images not, many in eight and in four chunks of channels;
    the last two always): the same bits, of zeros of either sign, infinities and numbers, NaN passed over."""
    import torch
    p = W._Prog(H, Wd, C); p.maxpool(0, 1, R, 1, pad); p.head(1, 4)
    arch = W.Arch("pool", W.DT_BF16, H, Wd, C, 4, np.array(p.layers, dtype=np.int32), p.gains)
    rng = np.random.default_rng(H * C + R)
    x = W.bf16_bits_to_f32(_bf16(rng, 4, H, Wd, C)).reshape(4, H, Wd, C).copy()
    for value, share in ((-np.inf, 0.2), (np.nan, 0.1), (np.inf, 0.002)):
        x[rng.random(x.shape) < share] = value
    x[1] = np.where(rng.random(x[1].shape) < 0.1, 0.0, np.where(rng.random(x[1].shape) < 0.5, -0.0, -1.0))
    x[2, :, :, ::3] = np.nan
    bits = W.f32_to_bf16_bits(x).reshape(x.shape)[np.arange(many) % 4]
    dev = torch.from_numpy(bits.view(np.int16)).cuda()
    P, Q = H + 2 * pad - R + 1, Wd + 2 * pad - R + 1
    ctx = B.Context(max_requests=many, max_batch=many)
    ctx.coe_register_expert(0, ctx.coe_register_arch(arch), W.make_expert_blob(arch, 7, 0), 1.0)
    few, all_of_them = (ctx.coe_debug_layer_output(0, n, dev.data_ptr(), 0, (n, P, Q, C), np.uint16) for n in (4, many))
    ctx.close()
    for i in range(many):
        assert np.array_equal(all_of_them[i], few[i % 4]), i


@pytest.mark.parametrize("n,H,Wd,C,K,R,stride,pad,act", [
    (3, 45, 50, 3, 64, 6, 2, 2, 3),      # reduction unrolled, outputs through LDS, ragged tiles
    (2, 16, 16, 3, 64, 6, 2, 2, 1),      # less than a tile
    (2, 33, 30, 4, 32, 3, 1, 1, 2),      # 32 filters through LDS
    (2, 20, 20, 4, 64, 9, 1, 4, 0),      # filters and patch leave no room: stores out of the accumulators
    (60, 40, 40, 4, 64, 3, 1, 1, 1),     # through LDS: workgroups of one tile and of two
    (116, 40, 40, 4, 32, 3, 1, 1, 3),    # the same with 32 filters
])
def test_few_channels_without_pool(B, oracle, n, H, Wd, C, K, R, stride, pad, act):
    """The kernel for few input channels without the fused pool, every output against the oracle."""
    rng = np.random.default_rng(H + K + R)
    x = _bf16(rng, n, H, Wd, C)
    w = _bf16(rng, K, R, R, C, scale=np.sqrt(2.0 / (R * R * C)))
    bias = (0.1 * rng.standard_normal(K)).astype(np.float32)
    ctx = B.Context(max_requests=1)
    got, cls = ctx.coe_debug_conv(1, x, w, bias, None, stride, pad, act)
    ctx.close()
    assert B.KERNEL_CLASS_NAMES[cls] == "conv_stem"
    xf, wf = (W.bf16_bits_to_f32(a).reshape(a.shape) for a in (x, w))
    want = np.stack([oracle.conv2d(xf[i], wf, bias, None, stride, pad, act, 1) for i in range(n)])
    g = W.bf16_bits_to_f32(got).reshape(want.shape)
    # as in test_few_tiles_give_the_bits_of_many
    assert np.all(np.abs(g - want) <= np.maximum(np.abs(want) * 2.0 ** -7, 1e-5))
    assert np.mean(g == want) > 0.995


@pytest.mark.parametrize("T,heads,n", [(17, 12, 5), (31, 3, 1), (33, 2, 3), (65, 12, 2), (97, 1, 5), (129, 3, 2), (160, 2, 1), (192, 1, 3),
                                       (193, 3, 2), (197, 12, 29)])
def test_attention_block_counts(B, oracle, T, heads, n):
    """Every number of 32-token blocks: heads packed into one unit of work (with an incomplete last one), workgroups that
    do one unit and several, ragged last blocks."""
    D = 64 * heads
    rng = np.random.default_rng(T * 10 + heads)
    x = _bf16(rng, n, T, 3 * D)
    p = W._Prog(T, 1, 3 * D)
    p.raw([W.OP_ATTENTION, 0, 1, -1, D, 0, 0, 0, 0, 0, heads, 0])
    p.shape[1] = (T, 1, D)
    p.head(1, 4)
    arch = W.Arch("attention", W.DT_BF16, T, 1, 3 * D, 4, np.array(p.layers, dtype=np.int32), p.gains)
    import torch
    dev = torch.from_numpy(x.view(np.int16)).cuda()
    ctx = B.Context(max_requests=n, max_batch=n)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, W.make_expert_blob(arch, 3, 0), 1.0)
    got = W.bf16_bits_to_f32(ctx.coe_debug_layer_output(0, n, dev.data_ptr(), 0, (n, T, D), np.uint16)).reshape(n, T, D)
    ctx.close()
    xf = W.bf16_bits_to_f32(x).reshape(n, T, 3 * D)
    for i in sorted({0, n - 1, n // 2}):
        want = oracle.attention(xf[i], heads, 1)
        # the output is one rounding (2^-8 of a value at most) of sum_j p_j v_j; an fp32 and an fp64 softmax may round a few
        # p_j to neighbouring bf16 values, 2^-8 p_j each: at most 2^-8 sum_j p_j |v_j| in all, and |v| < 5 here
        assert np.all(np.abs(got[i] - want) <= 2.0 ** -8 * (np.abs(want) + 5.0))
        assert np.sqrt(np.mean((got[i] - want) ** 2)) <= 2.0 ** -8 * np.sqrt(np.mean(want ** 2))
        assert np.mean(got[i] == want) > 0.9


@pytest.mark.parametrize("D", [1024, 1280, 1282, 2048])
def test_layer_norms_of_few_and_many_tokens_give_the_same_bits(B, D):
    """Beyond 1280 channels and the tokens that the chip holds at once (7168), the sums of a layer norm take another road, in the same order."""
    import torch
    T, few, many = 200, 3, 37
    p = W._Prog(T, 1, D)
    p.raw([W.OP_LAYERNORM, 0, 1, -1, D, 0, 0, 0, 0, 0, 0, 0])
    p.shape[1] = (T, 1, D)
    p.head(1, 4)
    arch = W.Arch("layernorm", W.DT_BF16, T, 1, D, 4, np.array(p.layers, dtype=np.int32), p.gains)
    x = _bf16(np.random.default_rng(D), few, T, 1, D)[np.arange(many) % few]
    dev = torch.from_numpy(x.view(np.int16)).cuda()
    ctx = B.Context(max_requests=many, max_batch=many)
    ctx.coe_register_expert(0, ctx.coe_register_arch(arch), W.make_expert_blob(arch, 7, 0), 1.0)
    small, large = (ctx.coe_debug_layer_output(0, n, dev.data_ptr(), 0, (n, T, D), np.uint16) for n in (few, many))
    ctx.close()
    xf = W.bf16_bits_to_f32(x[:few]).reshape(few, T, D).astype(np.float64)
    assert W.bf16_bits_to_f32(small).std() > 0.5 * xf.std() > 0
    assert all(np.array_equal(large[i], small[i % few]) for i in range(many))


@pytest.mark.parametrize("H,Wd,n", [
    (224, 224, 3),        # the image of most experts: four strips of 14 pooled columns
    (64, 64, 1300),       # two strips of 8; wavefronts that take several strips
    (38, 58, 2),          # one full strip of 15
    (33, 62, 2),          # 31 conv columns and 17 rows, both odd: a column and a row that do not exist
    (35, 60, 20),         # one strip of 15, its last column's right neighbour does not exist; 18 rows
    (224, 120, 1),        # two full strips
    (21, 122, 3),         # three strips, the last one narrower
    (5, 6, 4),            # three conv rows, segments of one pooled row
    (1, 4, 1), (9, 2, 2), # fewer rows and columns than the window: only the general kernels take some of these
])
def test_stem_with_pool(B, oracle, H, Wd, n):
    """7x7 stride 2 on three channels, ReLU, 3x3 stride 2 max pool: pooled values read back through an identity convolution
    (bit-exact), images at both ends of the batch against the oracle and equal images equal everywhere."""
    import torch
    rng = np.random.default_rng(H * 1000 + Wd)
    few = min(n, 3)
    x = _bf16(rng, few, H, Wd, 3)
    p = W._Prog(H, Wd, 3)
    p.conv(0, 1, 64, 7, 2, 3, W.ACT_RELU)
    p.maxpool(1, 2, 3, 2, 1)
    p.conv(2, 3, 64, 1, 1, 0, 0)
    p.head(3, 4)
    arch = W.Arch("stem", W.DT_BF16, H, Wd, 3, 4, np.array(p.layers, dtype=np.int32), p.gains)
    w = _bf16(rng, 64, 7, 7, 3, scale=np.sqrt(2.0 / 147))
    bias = (0.3 * rng.standard_normal(64)).astype(np.float32)
    blob = W.make_expert_blob(arch, 5, 0).copy()
    for sp in W.blob_layout(arch)[0]:
        value = {(0, "w"): w, (0, "b"): bias, (2, "w"): W.f32_to_bf16_bits(np.eye(64, dtype=np.float32)),
                 (2, "b"): np.zeros(64, np.float32)}.get((sp.layer, sp.name))
        if value is not None:
            blob[sp.offset:sp.offset + sp.nbytes] = np.ascontiguousarray(value).view(np.uint8).reshape(-1)
    P, Q = p.shape[1][:2]
    PP, PQ = p.shape[2][:2]
    idx = np.arange(n) % few
    dev = torch.from_numpy(x[idx].view(np.int16)).cuda()
    ctx = B.Context(max_requests=n, max_batch=n)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, blob, 1.0)
    got = W.bf16_bits_to_f32(ctx.coe_debug_layer_output(0, n, dev.data_ptr(), 2, (n, PP, PQ, 64), np.uint16)).reshape(n, PP, PQ, 64)
    ctx.close()
    assert np.array_equal(got, got[idx])
    xf, wf = W.bf16_bits_to_f32(x).reshape(x.shape), W.bf16_bits_to_f32(w).reshape(w.shape)
    for i in range(few):
        conv = oracle.conv2d(xf[i], wf, bias, None, 2, 3, 1, 1)
        wide = np.full((2 * PP + 1, 2 * PQ + 1, 64), -np.inf, np.float32)
        wide[1:P + 1, 1:Q + 1] = conv
        want = np.max([wide[r:r + 2 * PP - 1:2, c:c + 2 * PQ - 1:2] for r in range(3) for c in range(3)], axis=0)
        # one bf16 ulp where fp32 and fp64 sums round to different sides, 1e-5 where the terms cancel; rounding and the
        # maximum are monotonic, so the pool adds nothing
        assert np.all(np.abs(got[i] - want) <= np.maximum(np.abs(want) * 2.0 ** -7, 1e-5)), i


@pytest.mark.parametrize("H,Wd,n", [(224, 224, 2), (64, 64, 300), (38, 58, 2), (33, 62, 2), (35, 60, 5), (21, 122, 3), (5, 6, 4), (4, 4, 1)])
def test_stem_with_pool_gives_the_bits_of_the_general_kernel(B, H, Wd, n):
    """The fused stem adds the products of a window in the order of the general few-channel kernel: its pooled values are the
    maxima of that kernel's convolution, bit for bit."""
    import torch
    rng = np.random.default_rng(H * 100 + Wd)
    few = min(n, 3)
    x = _bf16(rng, few, H, Wd, 3)
    w = _bf16(rng, 64, 7, 7, 3, scale=np.sqrt(2.0 / 147))
    bias = (0.3 * rng.standard_normal(64)).astype(np.float32)
    p = W._Prog(H, Wd, 3)
    p.conv(0, 1, 64, 7, 2, 3, W.ACT_RELU)
    p.maxpool(1, 2, 3, 2, 1)
    p.conv(2, 3, 64, 1, 1, 0, 0)
    p.head(3, 4)
    arch = W.Arch("stem", W.DT_BF16, H, Wd, 3, 4, np.array(p.layers, dtype=np.int32), p.gains)
    blob = W.make_expert_blob(arch, 5, 0).copy()
    for sp in W.blob_layout(arch)[0]:
        value = {(0, "w"): w, (0, "b"): bias, (2, "w"): W.f32_to_bf16_bits(np.eye(64, dtype=np.float32)),
                 (2, "b"): np.zeros(64, np.float32)}.get((sp.layer, sp.name))
        if value is not None:
            blob[sp.offset:sp.offset + sp.nbytes] = np.ascontiguousarray(value).view(np.uint8).reshape(-1)
    P, Q = p.shape[1][:2]
    PP, PQ = p.shape[2][:2]
    idx = np.arange(n) % few
    dev = torch.from_numpy(x[idx].view(np.int16)).cuda()
    ctx = B.Context(max_requests=n, max_batch=n)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, blob, 1.0)
    got = ctx.coe_debug_layer_output(0, n, dev.data_ptr(), 2, (n, PP, PQ, 64), np.uint16).reshape(n, PP, PQ, 64)
    conv, cls = ctx.coe_debug_conv(1, x, w, bias, None, 2, 3, W.ACT_RELU)
    ctx.close()
    assert cls == B.K_CONV_STEM
    wide = np.zeros((few, 2 * PP + 1, 2 * PQ + 1, 64), np.uint16)         # after ReLU bf16 orders like its bits, 0 is the least
    wide[:, 1:P + 1, 1:Q + 1] = conv
    want = np.max([wide[:, r:r + 2 * PP - 1:2, c:c + 2 * PQ - 1:2] for r in range(3) for c in range(3)], axis=0)
    # (the identity convolution turns -0 into 0; there is none after ReLU)
    assert np.array_equal(got, want[idx])


@pytest.mark.parametrize("H,Wd,C", [(64, 64, 64), (33, 31, 512), (16, 16, 16), (1, 1, 64), (3, 5, 1024), (255, 1, 64), (257, 1, 32),
                                    (20, 13, 48), (9, 9, 12)])
def test_fp32_head_pooling(B, H, Wd, C):
    """Average pool and classifier of fp32 experts: sixteen positions in flight per thread and their remainders, one position,
    one position group (1024 channels), and channel counts that keep the plain loads (48, 12)."""
    import torch
    n = 3
    p = W._Prog(H, Wd, C)
    p.head(0, 5)
    arch = W.Arch("head", W.DT_F32, H, Wd, C, 5, np.array(p.layers, dtype=np.int32), p.gains)
    blob = W.make_expert_blob(arch, 7, 0)
    rng = np.random.default_rng(H * 7 + C)
    x = rng.standard_normal((n, H, Wd, C)).astype(np.float32)
    dev = torch.from_numpy(x).cuda()
    ctx = B.Context(max_requests=n, max_stages=1, max_batch=n)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, blob, 1.0)
    g = W.graph_from_lists([[]])
    ctx.coe_set_dependency_graph(g.succ_off, g.succ)
    ctx.coe_submit(n, dev.data_ptr(), True)
    while ctx.coe_step()[0] != B.COE_DONE:
        pass
    _, logits, _ = ctx.coe_collect(n)
    ctx.close()
    w, b = W.blob_tensor(arch, blob, 0, "w").astype(np.float64).reshape(5, C), W.blob_tensor(arch, blob, 0, "b").astype(np.float64)
    want = x.astype(np.float64).mean((1, 2)) @ w.T + b
    # first order: HW - 1 additions, a division, C products and additions, each 2^-24 of the absolute terms
    bound = (H * Wd + 2 * C + 4) * 2.0 ** -24 * (np.abs(x).astype(np.float64).mean((1, 2)) @ np.abs(w).T + np.abs(b))
    assert np.all(np.abs(logits[:, :5] - want) <= bound)


@pytest.mark.parametrize("H,Wd,C,n_cls", [(7, 7, 512, 16), (7, 7, 2048, 65), (1, 1, 64, 1), (8, 16, 64, 5), (43, 3, 64, 17), (4, 4, 2048, 4), (1, 17, 2048, 3),
                                          (33, 31, 512, 9), (5, 5, 96, 6), (65, 1, 512, 2), (16, 8, 256, 4), (12, 12, 256, 4), (29, 5, 256, 4), (127, 1, 256, 4),
                                          (11, 11, 256, 4)])
def test_bf16_head_pooling(B, H, Wd, C, n_cls):
    """Average pool and classifier of bf16 experts: sixteen positions in flight per thread, one less and one more, one position group
    (2048 channels), remainders of none, two and three rounds of the groups, ones that some groups have and others not, more classes than one round of the wavefronts takes, and a channel count that keeps the plain loads (96)."""
    import torch
    n = 3
    p = W._Prog(H, Wd, C)
    p.head(0, n_cls)
    arch = W.Arch("head", W.DT_BF16, H, Wd, C, n_cls, np.array(p.layers, dtype=np.int32), p.gains)
    blob = W.make_expert_blob(arch, 7, 0)
    x = torch.randn((n, H, Wd, C), generator=torch.Generator().manual_seed(H * 7 + C)).bfloat16().cuda()
    ctx = B.Context(max_requests=n, max_stages=1, max_batch=n)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, blob, 1.0)
    g = W.graph_from_lists([[]])
    ctx.coe_set_dependency_graph(g.succ_off, g.succ)
    ctx.coe_submit(n, x.data_ptr(), True)
    while ctx.coe_step()[0] != B.COE_DONE:
        pass
    _, logits, path = ctx.coe_collect(n)
    ctx.close()
    xd = x.cpu().double().numpy()
    w, b = W.blob_tensor(arch, blob, 0, "w").astype(np.float64).reshape(n_cls, C), W.blob_tensor(arch, blob, 0, "b").astype(np.float64)
    want = xd.mean((1, 2)) @ w.T + b
    # first order: HW - 1 additions, a division, C products and additions, each 2^-24 of the absolute terms
    bound = (H * Wd + 2 * C + 4) * 2.0 ** -24 * (np.abs(xd).mean((1, 2)) @ np.abs(w).T + np.abs(b))
    assert np.all(np.abs(logits[:, :n_cls] - want) <= bound) and np.all(path[:, 0] == 0)


@pytest.mark.parametrize("n", [341, 342, 700])
def test_pageable_inputs_arrive_whole(B, n):
    """Inputs from pageable memory (below 16 MB by the runtime's copy, from there through the pinned ring: eight chunks and a
    remainder, more chunks than the ring holds) and from pinned memory give the bits of inputs in device memory, twice over."""
    import torch
    arch = W.tiny_cnn(4, 64)
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, 64, 64, 3)).astype(np.float32)
    pinned = torch.from_numpy(x).pin_memory()
    ctx = B.Context(max_requests=n, max_stages=1, max_batch=256)
    aid = ctx.coe_register_arch(arch)
    ctx.coe_register_expert(0, aid, W.make_expert_blob(arch, 7, 0), 1.0)
    g = W.graph_from_lists([[]])
    ctx.coe_set_dependency_graph(g.succ_off, g.succ)
    dev = torch.from_numpy(x).cuda()
    out = []
    for src, on_device in ((dev.data_ptr(), True), (x, False), (x[::-1].copy(), False), (pinned.numpy(), False)):
        ctx.coe_submit(n, src, on_device)
        while ctx.coe_step()[0] != B.COE_DONE:
            pass
        out.append(ctx.coe_collect(n)[1])
    ctx.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2][::-1]) and np.array_equal(out[0], out[3])


@pytest.mark.parametrize("parts", [(342, 342), (700, 342, 500), (345, 1, 345)])
def test_submits_in_a_row_through_the_pinned_ring(B, parts):
    """Submits that follow each other without a step between them share the ring's chunks: every image arrives as it was, also
    when the caller's memory is written over as soon as a submit returns."""
    import torch
    arch = W.tiny_cnn(4, 64)
    n = sum(parts)
    x = np.random.default_rng(n).standard_normal((n, 64, 64, 3)).astype(np.float32)
    dev = torch.from_numpy(x).cuda()
    out = []
    for host in (False, True):
        ctx = B.Context(max_requests=n, max_stages=1, max_batch=256)
        aid = ctx.coe_register_arch(arch)
        ctx.coe_register_expert(0, aid, W.make_expert_blob(arch, 7, 0), 1.0)
        g = W.graph_from_lists([[]])
        ctx.coe_set_dependency_graph(g.succ_off, g.succ)
        at = 0
        for m in parts:
            if host:
                mine = x[at:at + m].copy()
                ctx.coe_submit(m, mine, False)
                mine[:] = np.nan
            else:
                ctx.coe_submit(m, dev[at].data_ptr(), True)
            at += m
        while ctx.coe_step()[0] != B.COE_DONE:
            pass
        out.append(ctx.coe_collect(n)[1])
        ctx.close()
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1])


@pytest.mark.parametrize("n,hw,shift", [(1, 16, 0), (1, 5, 0), (9, 16, 4), (130, 5, 0), (130, 16, 0), (5463, 16, 0), (200, 64, 16)])
def test_device_inputs_and_known_counts(B, n, hw, shift):
    """Submits from device memory that move in the launch which sets the store up (a multiple of 16 bytes from a 16-byte boundary on, at
    most 16 MB) and those that do not (5 x 5 images, a shifted start, 16.8 MB) give the bits of host inputs.  A step regroups by the
    counts the host knows (two submits into an empty store) as by those it reads back (a submit beside requests that have run), and a
    store that was collected starts over."""
    import torch
    arch, E = W.tiny_cnn(4, hw), 3
    rng = np.random.default_rng(n + hw)
    x = rng.standard_normal((n, hw, hw, 3)).astype(np.float32)
    first = rng.integers(0, E, n).astype(np.int32)
    raw = torch.zeros(x.size + 8, dtype=torch.float32, device="cuda")
    raw[shift // 4:shift // 4 + x.size] = torch.from_numpy(x.reshape(-1)).cuda()
    torch.cuda.synchronize()
    at = lambda i: raw.data_ptr() + shift + i * hw * hw * 3 * 4
    out, cut = [], max(1, n // 3)
    for on_device in (False, True):
        ctx = B.Context(max_requests=2 * n, max_stages=1, max_batch=256)
        aid = ctx.coe_register_arch(arch)
        for e in range(E):
            ctx.coe_register_expert(e, aid, W.make_expert_blob(arch, 7, e), 1.0 / E)
        g = W.graph_from_lists([[]] * E)
        ctx.coe_set_dependency_graph(g.succ_off, g.succ)
        for _ in range(2):
            for a, b in ((0, cut), (cut, n)):
                if b > a:
                    ctx.coe_submit(b - a, at(a) if on_device else x[a:b], on_device, first[a:b])
            assert ctx.coe_step()[0] == B.COE_OK
            r = ctx.coe_debug_last_regroup(2 * n)
            assert np.array_equal(r["cnt"], np.bincount(first, minlength=E)) and np.array_equal(r["perm"], np.argsort(first, kind="stable"))
            ctx.coe_submit(n, at(0) if on_device else x, on_device, first[::-1].copy())
            assert ctx.coe_step()[0] == B.COE_OK
            r = ctx.coe_debug_last_regroup(2 * n)
            assert np.array_equal(r["cnt"], np.bincount(first, minlength=E)) and np.array_equal(r["perm"], n + np.argsort(first[::-1], kind="stable"))
            assert ctx.coe_step()[0] == B.COE_DONE
            ids, logits, path = ctx.coe_collect(2 * n)
            assert np.array_equal(path[:, 0], np.concatenate([first, first[::-1]])) and len(ids) == 2 * n
            out.append(logits)
        ctx.close()
    assert np.isfinite(out[0]).all() and all(np.array_equal(out[0], o) for o in out[1:])


def test_collects_beyond_the_pinned_memory(B):
    """A store whose results may exceed the pinned memory (5000 requests, 1000 classes): all at once by copies, in halves through
    it, the same results."""
    import torch
    arch, n = W.tiny_cnn(1000, 8), 5000
    x = torch.randn((n, 8, 8, 3), generator=torch.Generator().manual_seed(3)).cuda()
    ctx = B.Context(max_requests=n, max_stages=1, max_batch=512)
    ctx.coe_register_expert(0, ctx.coe_register_arch(arch), W.make_expert_blob(arch, 7, 0), 1.0)
    g = W.graph_from_lists([[]])
    ctx.coe_set_dependency_graph(g.succ_off, g.succ)
    out = []
    for parts in ((n,), (n // 2, n // 2)):
        logits = []
        for i, m in enumerate(parts):
            ctx.coe_submit(m, x[i * parts[0]].data_ptr(), True)
            while ctx.coe_step()[0] != B.COE_DONE:
                pass
            ids, lg, path = ctx.coe_collect(m)
            assert np.array_equal(ids, ids[0] + np.arange(m)) and not path.any()
            logits.append(lg)
        out.append(np.concatenate(logits))
    ctx.close()
    assert out[0].shape == (n, 1000) and np.isfinite(out[0]).all() and out[0].std() > 0 and np.array_equal(out[0], out[1])


@pytest.mark.parametrize("C,hw,n", [(64, 16, 1), (64, 16, 33), (128, 16, 7), (128, 16, 20), (128, 16, 200), (128, 20, 150), (96, 16, 5)])
def test_independent_convolutions_share_a_launch_with_the_same_bits(B, C, hw, n):
    """Neighbouring convolutions that do not depend on each other run in one launch where both have few tiles (32 x 32 tiles with two or
    four channel blocks to a stage, those deep or, where both together are more than the compute units, shallower; 64 x 64 tiles), alone and in groups: the bits of a batch of 700, whose launches are apart.  96
    channels have no such tiles.  Neighbours that read or overwrite each other's outputs stay in order."""
    import torch
    K, many, E = 128, 700, 3
    p = W._Prog(hw, hw, 3, n_scratch=7)
    p.conv(0, 1, 64, 3, 1, 1, W.ACT_RELU)
    p.conv(1, 2, C, 1, 1, 0, W.ACT_RELU)
    p.conv(2, 3, K, 3, 2, 1, W.ACT_RELU)                 # a strided convolution and the projection beside it
    p.conv(2, 4, K, 1, 2, 0, W.ACT_NONE)
    p.conv(3, 5, K, 3, 1, 1, W.ACT_RELU, res=4, gain=0.5)
    p.conv(5, 1, K // 2, 1, 1, 0, W.ACT_SILU)            # two branches
    p.conv(5, 2, K // 2, 1, 1, 0, W.ACT_SILU)
    p.conv(1, 3, K, 1, 1, 0, W.ACT_NONE)                 # the second reads the first as its residual
    p.conv(2, 4, K, 1, 1, 0, W.ACT_RELU, res=3)
    p.conv(4, 6, 2 * K, 1, 2, 0, W.ACT_NONE)             # unlike shapes
    p.conv(4, 7, K // 2, 1, 1, 0, W.ACT_RELU)
    p.conv(7, 1, K, 1, 1, 0, W.ACT_RELU)                 # the second overwrites what the first reads
    p.conv(4, 7, K // 2, 1, 1, 0, W.ACT_RELU)
    p.conv(7, 2, K, 1, 1, 0, W.ACT_RELU, res=1)
    p.conv(2, 3, 2 * K, 3, 2, 1, W.ACT_RELU, res=6, gain=0.5)
    p.head(3, 6)
    arch = W.Arch("pairs", W.DT_BF16, hw, hw, 3, 6, np.array(p.layers, dtype=np.int32), p.gains)
    blobs = [W.make_expert_blob(arch, 11, e) for e in range(E)]
    x = torch.randn((many, hw, hw, 3), generator=torch.Generator().manual_seed(C + hw)).bfloat16().cuda()
    first = np.random.default_rng(n).integers(0, E, n).astype(np.int32)
    got = {}
    for small in (-1, 64):
        ctx = B.Context(max_requests=many, max_stages=1, max_batch=many, group_small=small)
        aid = ctx.coe_register_arch(arch)
        for e, blob in enumerate(blobs):
            ctx.coe_register_expert(e, aid, blob, 1.0 / E)
        g = W.graph_from_lists([[]] * E)
        ctx.coe_set_dependency_graph(g.succ_off, g.succ)
        ctx.coe_submit(n, x.data_ptr(), True, first)
        while ctx.coe_step()[0] != B.COE_DONE:
            pass
        got[small] = ctx.coe_collect(n)[1]
        if small < 0:
            want = np.stack([ctx.coe_debug_forward(e, many, x.data_ptr()) for e in range(E)])
            few = np.stack([ctx.coe_debug_forward(e, n, x.data_ptr()) for e in range(E)])
        ctx.close()
    assert np.isfinite(want).all() and want.std() > 0
    assert np.array_equal(few, want[:, :n])
    for logits in got.values():
        assert np.array_equal(logits, want[first, np.arange(n)])


@pytest.mark.parametrize("c,K,hw,n", [(32, 64, 8, 3), (32, 128, 8, 900), (64, 64, 8, 1), (64, 256, 7, 40), (64, 64, 12, 300), (128, 128, 8, 2), (128, 256, 9, 700),
                                      (256, 512, 14, 128), (48, 64, 8, 5), (64, 96, 8, 5)])
def test_concatenations_read_in_place(B, c, K, hw, n):
    """A 1x1 convolution over a concatenation reads the concatenated maps themselves: two, four (chained), three, with residual, beside
    readers that need the concatenated map, and over the parts of unequal size that it leaves alone.  Same bits as with a 1x1 pool in between,
    which makes the map.  Sizes: few tiles (32 x 32 of two and four channel blocks to a stage, 64 x 64), 128-row tiles of 64 and 128 filters,
    persistent tiles; 48 channels and 96 filters keep the concatenation."""
    import torch
    def build(direct):
        p = W._Prog(hw, hw, 3, n_scratch=7)
        def fuse(src, dst, spare, k, act, res=-1):
            if direct:
                p.conv(src, dst, k, 1, 1, 0, act, res=res)
            else:
                p.maxpool(src, spare, 1, 1, 0)
                p.conv(spare, dst, k, 1, 1, 0, act, res=res)
        p.conv(0, 1, 64, 3, 1, 1, W.ACT_RELU)
        p.conv(1, 2, c, 1, 1, 0, W.ACT_SILU)
        p.conv(1, 3, c, 1, 1, 0, W.ACT_RELU)
        p.concat(2, 3, 1)
        fuse(1, 7, 5, K, W.ACT_RELU)                        # two maps; 7 stays
        p.maxpool(2, 4, 3, 1, 1)
        p.concat(1, 4, 5)
        fuse(5, 6, 3, K, W.ACT_NONE, res=7)                 # three maps, residual
        p.conv(6, 7, c, 1, 1, 0, W.ACT_RELU)
        p.concat(5, 7, 1)
        fuse(1, 6, 3, K, W.ACT_SILU)                        # four maps, the first two kept from the start
        p.concat(7, 6, 2)
        fuse(2, 5, 3, 64, W.ACT_RELU)                       # parts of unequal size where K is not c
        p.concat(5, 5, 3)
        p.maxpool(3, 4, 3, 1, 1)                         # a reader that needs the map, and one that does not
        fuse(3, 6, 1, 128, W.ACT_NONE, res=4)
        p.head(6, 5)
        return W.Arch("cat", W.DT_BF16, hw, hw, 3, 5, np.array(p.layers, dtype=np.int32), p.gains)
    archs = [build(True), build(False)]
    blob = W.make_expert_blob(archs[0], 5, 0)
    x = torch.randn((n, hw, hw, 3), generator=torch.Generator().manual_seed(c + K)).bfloat16().cuda()
    out = []
    for arch in archs:
        assert W.blob_layout(arch)[1] == blob.nbytes
        ctx = B.Context(max_requests=n, max_stages=1, max_batch=n)
        ctx.coe_register_expert(0, ctx.coe_register_arch(arch), blob, 1.0)
        g = W.graph_from_lists([[]])
        ctx.coe_set_dependency_graph(g.succ_off, g.succ)
        out.append(ctx.coe_debug_forward(0, n, x.data_ptr()))
        if arch is archs[0]:                             # layer by layer every map is made
            at = [i for i, l in enumerate(arch.layers) if l[0] == W.OP_CONCAT]
            maps = [ctx.coe_debug_layer_output(0, n, x.data_ptr(), i, (n, hw, hw, w), np.uint16) for i, w in ((at[0], 2 * c), (at[0] - 2, c), (at[0] - 1, c))]
            assert np.array_equal(maps[0], np.concatenate(maps[1:], -1))
        ctx.close()
    assert np.isfinite(out[0]).all() and out[0].std() > 0 and np.array_equal(out[0], out[1])


@pytest.mark.parametrize("dst,res", [(8, -1), (99, -1), (-1, 40), (5, 3)])
def test_buffers_that_an_operation_does_not_have_change_nothing(B, dst, res):
    """The destination of a head and the residual of a pool or an upsampling may hold anything: same logits as with -1."""
    import torch
    arch = W.detector(27, 64)
    blob, n = W.make_expert_blob(arch, 5, 0), 3
    x = torch.randn((n, 64, 64, 3), generator=torch.Generator().manual_seed(1)).bfloat16().cuda()
    layers = arch.layers.copy()
    for l in layers:
        if l[0] == W.OP_HEAD_DET:
            l[2] = dst
        if l[0] in (W.OP_MAXPOOL, W.OP_UPSAMPLE):
            l[3] = res
    out = []
    for a in (arch, W.Arch("stray", arch.dtype, 64, 64, 3, 27, layers, arch.gains)):
        ctx = B.Context(max_requests=n, max_stages=1, max_batch=n)
        ctx.coe_register_expert(0, ctx.coe_register_arch(a), blob, 1.0)
        g = W.graph_from_lists([[]])
        ctx.coe_set_dependency_graph(g.succ_off, g.succ)
        out.append(ctx.coe_debug_forward(0, n, x.data_ptr()))
        ctx.close()
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1])


@pytest.mark.parametrize("n,experts,cap", [(30, 6, 0), (300, 9, 0), (60, 8, 5)])
def test_grouped_transformers_give_the_same_bits(B, n, experts, cap):
    """Small groups of several transformer-shaped experts share launches: same logits, routes and switches, bit for bit, as one
    launch per group."""
    import torch
    from oracle import guard as G
    wl = W.config5(n, hw=64, n_experts=experts, cap=cap, dim=128, depth=2, heads=2, mlp=256, calibrated=False)
    G.calibrate_workload(wl, n_cal=48)        # spreads the routes
    blobs = [wl.blob(e) for e in range(experts)]
    x = wl.inputs(range(n))
    dev = torch.from_numpy(x.view(np.int16)).cuda()
    out = {}
    for small in (-1, 0):
        ctx = B.Context(max_requests=n, max_stages=2, max_batch=256, cache_cap_experts=cap, group_small=small)
        B.setup_workload(ctx, wl, blobs)
        runs = []
        for _ in range(2):                    # the first pass waits for the experts' first copies
            ctx.coe_submit(n, dev.data_ptr(), True)
            stats = []
            while True:
                rc, st = ctx.coe_step()
                if rc == B.COE_DONE:
                    break
                stats.append(st)
            _, logits, path = ctx.coe_collect(n)
            runs.append((logits, path, [st.n_groups for st in stats], [st.n_misses for st in stats], sum(st.n_grouped for st in stats)))
        ctx.close()
        out[small] = runs
    for a, b in zip(out[-1], out[0]):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[2:4] == b[2:4]
        assert a[4] == 0
    assert out[0][1][4] >= 2


@pytest.mark.parametrize("kind,n,experts", [("vit", 1500, 8), ("resnet", 1400, 6), ("vit", 400, 20)])
def test_large_groups_share_launches_with_the_same_bits(B, kind, n, experts):
    """Groups of 60 to 300 requests in shared launches of more tiles than conv_ring takes: persistent tiles of token GEMMs whose
    workgroups go on from one group's rows to the next, slab tiles and strided tiles that start anew in every group."""
    import torch
    from oracle import guard as G
    if kind == "vit":
        wl = W.config5(n, hw=64, n_experts=experts, cap=0, dim=512, depth=1, heads=8, mlp=1024, calibrated=False)
        sizes = [(n * 17, k) for k in (512, 1024, 1536)]
    else:
        wl = W.config2(n, hw=128, n_experts=experts, width=64, calibrated=False)
        sizes = [(n * 32 * 32, 64), (n * 16 * 16, 128), (n * 8 * 8, 256)]
    assert all(rows * k // 4096 > 768 for rows, k in sizes)
    G.calibrate_workload(wl, n_cal=48)
    blobs = [wl.blob(e) for e in range(experts)]
    dev = torch.from_numpy(wl.inputs(range(n)).view(np.int16)).cuda()
    out = []
    for small in (-1, 1024):
        ctx = B.Context(max_requests=n, max_stages=2, max_batch=4096, group_small=small)
        B.setup_workload(ctx, wl, blobs)
        for _ in range(2):
            ctx.coe_submit(n, dev.data_ptr(), True)
            grouped = 0
            while True:
                rc, st = ctx.coe_step()
                if rc == B.COE_DONE:
                    break
                grouped += st.n_grouped
            _, logits, path = ctx.coe_collect(n)
        ctx.close()
        assert (grouped >= experts // 2) == (small > 0)
        out.append((logits, path))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_experts_beyond_two_gib_run_group_by_group(B):
    """Transformer-shaped experts whose last tensors lie more than 2 GiB into their weights, out of reach of a group table's
    offsets: their small groups run one by one, with the result of a context that groups nothing."""
    import torch
    T, D, n_cls, n = 2, 1024, 4, 6
    p = W._Prog(16, 16, 3, n_scratch=5)
    p.conv(0, 1, D, 16, 16, 0, W.ACT_NONE)
    p.raw([W.OP_TOKENS, 1, 2, -1, D, 0, 0, 0, 0, 0, 0, 0]); p.shape[2] = (T, 1, D)
    p.conv(2, 3, 32768, 1, 1, 0, W.ACT_RELU)
    p.conv(3, 4, 32704, 1, 1, 0, W.ACT_RELU)
    p.conv(4, 1, D, 1, 1, 0, W.ACT_NONE)
    p.raw([W.OP_HEAD_CLS, 1, -1, -1, n_cls, 0, 0, 0, 0, 0, 0, 0])
    big = W.Arch("wide", W.DT_BF16, 16, 16, 3, n_cls, np.array(p.layers, dtype=np.int32), p.gains)
    specs, nbytes = W.blob_layout(big)
    assert specs[-1].offset > 2 ** 31
    rng = np.random.default_rng(0)
    blob = np.zeros(nbytes, np.uint8)
    for sp in specs:                             # every tensor from a few hundred thousand values: its contents do not matter
        bits = W.f32_to_bf16_bits((rng.standard_normal(300007) * 0.02).astype(np.float32)) if sp.is_param_dtype else \
            rng.standard_normal(4099).astype(np.float32)
        raw = bits.view(np.uint8)
        blob[sp.offset:sp.offset + sp.nbytes] = np.resize(raw, sp.nbytes)
    root = W.vit(n_cls, 16, 16, 64, 1, 1, 64)
    x = W.make_inputs(root, 5, range(n))
    dev = torch.from_numpy(x.view(np.int16)).cuda()
    g = W.graph_from_lists([[1, 2], [], []])
    out = []
    for small in (-1, 0):
        ctx = B.Context(max_requests=n, max_stages=2, max_batch=64, group_small=small)
        ids = [ctx.coe_register_arch(root), ctx.coe_register_arch(big)]
        ctx.coe_register_expert(0, ids[0], W.make_expert_blob(root, 7, 0), 1.0)
        for e in (1, 2):
            ctx.coe_register_expert(e, ids[1], blob, 0.5)
        ctx.coe_set_dependency_graph(g.succ_off, g.succ)
        for _ in range(2):
            first = np.array([0, 0, 1, 1, 2, 2], np.int32)             # both wide experts have a group in either step
            ctx.coe_submit(n, dev.data_ptr(), True, first)
            grouped = 0
            while True:
                rc, st = ctx.coe_step()
                if rc == B.COE_DONE:
                    break
                grouped += st.n_grouped
            _, logits, path = ctx.coe_collect(n)
        ctx.close()
        assert grouped == 0
        out.append((logits, path))
    assert np.isfinite(out[0][0]).all() and np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
