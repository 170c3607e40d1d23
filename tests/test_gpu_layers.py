"""GPU parity of the per-layer entry points against the oracle (Section 5 "Reuse")."""
import numpy as np
import pytest
import torch

from paper_1712_01670_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _to_dev(a, bf16):
    t = torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    return t.to(torch.bfloat16) if bf16 else t


def _to_np(t):
    return t.float().cpu().numpy()


def _rel_err(got, want):
    scale = max(float(np.abs(want).max()), 1e-30)
    return float(np.abs(got - want).max()) / scale


def _layer(cin, cout, k, s, p, relu):
    return dict(type=synth.CONV, k=k, s=s, p=p, cin=cin, cout=cout, relu=int(relu), in0=0, in1=-1)


CONV_CASES = [
    # H, W, cin, cout, k, s, p, relu
    (20, 37, 3, 16, 3, 1, 1, True),      # first-layer shape, ragged tiles
    (33, 18, 16, 32, 3, 2, 1, True),     # stride 2
    (16, 16, 32, 32, 3, 1, 1, False),
    (29, 31, 64, 64, 3, 1, 1, True),     # 64-channel, several tiles and a ragged tail
    (14, 14, 128, 256, 3, 1, 1, True),   # small map, wide
    (28, 28, 64, 128, 1, 1, 0, True),    # 1x1
    (28, 28, 128, 64, 1, 2, 0, False),   # 1x1 stride 2 (projection shortcut)
    (40, 40, 3, 64, 7, 2, 3, True),      # stem
    (9, 11, 5, 7, 3, 1, 0, True),        # odd channel counts: scalar load path
    (10, 10, 40, 136, 3, 1, 1, True),    # cin not a multiple of the chunk, cout ragged
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", CONV_CASES)
def test_full_conv_matches_oracle(oracle, case, bf16):
    H, W, cin, cout, k, s, p, relu = case
    print(f"[conv] case={case} bf16={bf16}", flush=True)
    rng = np.random.default_rng(abs(hash(case)) % 2 ** 31)
    x = rng.standard_normal((2, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, k, k, cin)) * np.sqrt(2.0 / (cin * k * k))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    if bf16:
        x, w = oracle.round_bf16(x), oracle.round_bf16(w)
    got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, k, s, p, relu), _to_dev(x, bf16), _to_dev(w, bf16),
                                              torch.from_numpy(b).to(DEV)))
    for n in range(2):
        want = oracle.conv_cached(x[n], w, b, k, s, p, relu, bf16=bf16)
        assert got[n].shape == want.shape
        assert _rel_err(got[n], want) <= (2e-2 if bf16 else 1e-4), (case, n)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", [(40, 52, 16, 64, 3, 1, 1), (31, 45, 32, 32, 3, 2, 1), (24, 24, 64, 160, 1, 1, 0)])
def test_cached_conv_matches_oracle(oracle, case, bf16):
    H, W, cin, cout, k, s, p = case
    print(f"[cached conv] case={case} bf16={bf16}", flush=True)
    rng = np.random.default_rng(sum(case))
    n = 3
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, k, k, cin)) * np.sqrt(2.0 / (cin * k * k))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    Ho, Wo = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    cache = rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    # per-stream regions: stream 0 large rect + sliver, stream 1 nothing, stream 2 everything that fits
    regions = [
        (np.array([[2, 1, Wo - 9, Ho - 9], [Wo - 6, 3, 2, 5]], np.int32), (3, -1)),
        (np.zeros((0, 4), np.int32), (0, 0)),
        (np.array([[0, 0, Wo - 2, Ho - 1]], np.int32), (2, 1)),
    ]
    got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, k, s, p, True), _to_dev(x, bf16), _to_dev(w, bf16),
                                              torch.from_numpy(b).to(DEV), cache_prev=_to_dev(cache, bf16),
                                              regions=regions))
    for i in range(n):
        mask = oracle.rasterize(regions[i][0], Ho, Wo)
        want = oracle.conv_cached(x[i], w, b, k, s, p, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16)
        m = mask.astype(bool)
        assert np.array_equal(got[i][m], want[m]), "copied pixels must be bit-identical"
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (case, i)


def _random_regions(rng, oracle, Ho, Wo):
    """Disjoint rectangles (merged from a random grid mask) whose sources stay inside the map."""
    cell = int(rng.choice([2, 3, 5]))
    mask = (rng.random((Ho // cell, Wo // cell)) < rng.choice([0.3, 0.6, 0.9])).astype(np.uint8)
    rects = oracle.merge_blocks(mask, cell)
    dx, dy = int(rng.integers(-4, 5)), int(rng.integers(-4, 5))
    out = []
    for x, y, w, h in rects.tolist():
        x0, y0 = max(x, -dx, 0), max(y, -dy, 0)
        x1, y1 = min(x + w, Wo - dx, Wo), min(y + h, Ho - dy, Ho)
        if x1 > x0 and y1 > y0:
            out.append([x0, y0, x1 - x0, y1 - y0])
    return np.array(out, np.int32).reshape(-1, 4), (dx, dy)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("seed", range(6))
def test_cached_conv_random_regions(oracle, seed, bf16):
    """Random layer shapes of both kernel families with random disjoint reusable rectangles per stream:
    copied pixels bit-identical, recomputed ones within tolerance, nothing else touched."""
    rng = np.random.default_rng(100 + seed)
    k, s, p = [(3, 1, 1), (3, 1, 1), (1, 1, 0), (3, 2, 1), (5, 1, 2), (3, 1, 0)][seed]
    cin = int(rng.choice([16, 32, 64])) if seed < 2 else int(rng.choice([8, 16, 24]))
    cout = int(rng.choice([64, 128])) if seed < 2 else int(rng.choice([16, 40, 64]))
    H, W = int(rng.integers(18, 40)), int(rng.integers(18, 44))
    print(f"[cached conv random] seed={seed} bf16={bf16} {H}x{W} cin={cin} cout={cout} k={k} s={s} p={p}", flush=True)
    n = 3
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, k, k, cin)) * np.sqrt(2.0 / (cin * k * k))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    Ho, Wo = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    cache = rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = [_random_regions(rng, oracle, Ho, Wo) for _ in range(n)]
    got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, k, s, p, True), _to_dev(x, bf16), _to_dev(w, bf16),
                                              torch.from_numpy(b).to(DEV), cache_prev=_to_dev(cache, bf16),
                                              regions=regions))
    for i in range(n):
        mask = oracle.rasterize(regions[i][0], Ho, Wo)
        want = oracle.conv_cached(x[i], w, b, k, s, p, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16)
        m = mask.astype(bool)
        assert np.array_equal(got[i][m], want[m]), "copied pixels must be bit-identical"
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (seed, i)


# 3x3 stride-1 layers with whole 64-byte channel rows take the compile-time-shaped GEMM kernel; the launch
# heuristics are overridden so that every shape of that kernel is exercised at a size the oracle handles:
# (arrangement, units per workgroup, K split, chunk index); arrangement 1 exists for bf16 only.
FAST_CASES = [
    # H, W, cin, cout, tuning
    (22, 30, 32, 64, (0, 1, -1, 0)),     # one unit per workgroup
    (22, 30, 64, 64, (0, 5, -1, 1)),     # odd unit count, longer channel chunk
    (22, 30, 64, 128, (0, 16, 1, 0)),    # full workgroup tile, more units in the tile than in the map's last group
    (14, 14, 128, 64, (0, 3, 4, 0)),     # K split among 4 workgroups + reduction kernel
    (13, 17, 256, 128, (0, 2, 8, 1)),    # K split, ragged map
    (22, 30, 64, 128, (1, 7, 1, 0)),     # 128 channels per workgroup
    (22, 30, 64, 256, (1, 16, 2, 0)),    # ... with a K split
    (22, 30, 64, 64, (2, 11, 1, 0)),     # 64 channels per workgroup in two blocks per wavefront (bf16)
    (14, 14, 128, 192, (2, 4, 2, 1)),
    (19, 23, 128, 128, (-1, -1, -1, -1)),  # the library's own choice
    (22, 30, 64, 64, (3, -1, -1, -1)),    # bf16: persistent kernel with the weights in registers (plain weights)
    (37, 41, 64, 128, (3, -1, -1, -1)),   # ... two channel tiles, more unit groups than one step, ragged map
    (22, 30, 64, 128, (4, 18, 1, 0)),     # bf16: twelve wavefronts, 18 units per workgroup (96 units: the last group holds 6)
    (45, 61, 32, 256, (4, 13, 1, 0)),     # ... 13 units: one row of wavefronts with three units, five with two
    (30, 34, 96, 128, (4, 17, 3, 0)),     # ... with a K split
]


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", FAST_CASES)
def test_fast_conv_kernel_shapes(oracle, case, bf16, cached):
    H, W, cin, cout, tuning = case
    print(f"[fast conv] case={case} bf16={bf16} cached={cached}", flush=True)
    rng = np.random.default_rng(H * 1000 + W * 10 + cin + cout)
    n = 2
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, 3, 3, cin)) * np.sqrt(2.0 / (cin * 9))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    cache = rng.standard_normal((n, H, W, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = None
    if cached:
        regions = [(np.array([[1, 2, W - 7, H - 6], [W - 5, 1, 3, 4]], np.int32), (2, -1)),
                   (np.array([[0, 0, W - 1, H - 3]], np.int32), (1, 2))]
    binding.dc_conv_tuning(*tuning)
    try:
        layer, wd = _layer(cin, cout, 3, 1, 1, True), _to_dev(w, bf16)
        got = _to_np(binding.dc_cached_conv_layer(layer, _to_dev(x, bf16), wd, torch.from_numpy(b).to(DEV),
                                                  cache_prev=_to_dev(cache, bf16) if cached else None, regions=regions))
        # the same layer reading the packed copy of the weights: same products in the same order
        wp = binding.dc_pack_conv_weights(layer, wd)
        assert wp is not None
        es = 2 if bf16 else 4
        raw = wd.view(torch.uint8).cpu().numpy().reshape(cout // 16, 16, 9, cin * es // 64, 64)
        assert np.array_equal(wp.view(torch.uint8).cpu().numpy().reshape(cout // 16, cin * es // 64, 9, 16, 64),
                              raw.transpose(0, 3, 2, 1, 4)), "layout [cout/16][64-byte chunk][tap][16][64 bytes]"
        # plain weights zeroed: the result shows that the kernel reads the packed copy
        plain = wd if tuning[0] == 3 else torch.zeros_like(wd)     # arrangement 3 reads the plain layout
        got_p = _to_np(binding.dc_cached_conv_layer(layer, _to_dev(x, bf16), plain, torch.from_numpy(b).to(DEV),
                                                    cache_prev=_to_dev(cache, bf16) if cached else None, regions=regions,
                                                    packed=wp))
    finally:
        binding.dc_conv_tuning()
    assert np.array_equal(got, got_p), "packed weights must not change a bit"
    for i in range(n):
        if cached:
            mask = oracle.rasterize(regions[i][0], H, W)
            want = oracle.conv_cached(x[i], w, b, 3, 1, 1, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16)
            m = mask.astype(bool)
            assert np.array_equal(got[i][m], want[m]), "copied pixels must be bit-identical"
        else:
            want = oracle.conv_cached(x[i], w, b, 3, 1, 1, True, bf16=bf16)
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (case, i)


def test_register_weight_kernel_without_relu_and_bias(oracle):
    """The persistent bf16 kernel for 64 input channels: negative outputs survive when the layer has no ReLU,
    and a missing bias is zero."""
    H, W, cin, cout = 26, 34, 64, 64
    rng = np.random.default_rng(5)
    x = oracle.round_bf16(rng.standard_normal((3, H, W, cin)).astype(np.float32))
    w = oracle.round_bf16((rng.standard_normal((cout, 3, 3, cin)) * np.sqrt(2.0 / (cin * 9))).astype(np.float32))
    binding.dc_conv_tuning(3, -1, -1, -1)
    try:
        got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, 3, 1, 1, False), _to_dev(x, True), _to_dev(w, True), None))
    finally:
        binding.dc_conv_tuning()
    assert (got < 0).mean() > 0.3
    for i in range(3):
        want = oracle.conv_cached(x[i], w, None, 3, 1, 1, False, bf16=True)
        assert _rel_err(got[i], want) <= 2e-2


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("cout", [16, 32, 64, 128])
def test_first_layer_kernel(oracle, cout, bf16, cached):
    """Input pixels of one 16-byte vector (4 fp32 / 8 bf16 channels): the kernel without LDS staging."""
    H, W = 21, 26
    cin = 8 if bf16 else 4
    print(f"[first layer] cout={cout} bf16={bf16} cached={cached}", flush=True)
    rng = np.random.default_rng(cout + 7)
    n = 2
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, 3, 3, cin)) * np.sqrt(2.0 / (cin * 9))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    cache = rng.standard_normal((n, H, W, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = None
    if cached:
        regions = [(np.array([[3, 1, W - 8, H - 5]], np.int32), (-2, 1)), (np.zeros((0, 4), np.int32), (0, 0))]
    got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, 3, 1, 1, True), _to_dev(x, bf16), _to_dev(w, bf16),
                                              torch.from_numpy(b).to(DEV),
                                              cache_prev=_to_dev(cache, bf16) if cached else None, regions=regions))
    for i in range(n):
        if cached:
            mask = oracle.rasterize(regions[i][0], H, W)
            want = oracle.conv_cached(x[i], w, b, 3, 1, 1, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16)
            m = mask.astype(bool)
            assert np.array_equal(got[i][m], want[m])
        else:
            want = oracle.conv_cached(x[i], w, b, 3, 1, 1, True, bf16=bf16)
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (cout, i)


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("cout", [16, 64, 96])
@pytest.mark.parametrize("geom", [(7, 2, 3), (11, 4, 0), (11, 4, 2)])
def test_stem_kernel(oracle, geom, cout, bf16, cached):
    """7x7 stride-2 and 11x11 stride-4 convolutions over 16-byte input pixels (the first layers of the residual and
    the AlexNet-style networks); odd and even sizes, so that the last output row reads past the input on one side
    only."""
    H, W = (45, 54) if geom[0] == 7 else (75, 91)
    k, s, p = geom
    Ho, Wo = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    cin = 8 if bf16 else 4
    print(f"[stem] geom={geom} cout={cout} bf16={bf16} cached={cached}", flush=True)
    rng = np.random.default_rng(cout + 11)
    n = 2
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, k, k, cin)) * np.sqrt(2.0 / (cin * k * k))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    cache = rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = None
    if cached:
        regions = [(np.zeros((0, 4), np.int32), (0, 0)), (np.array([[2, 3, Wo - 9, Ho - 6], [Wo - 6, 4, 3, 6]], np.int32), (1, -2))]
    got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, k, s, p, True), _to_dev(x, bf16), _to_dev(w, bf16),
                                              torch.from_numpy(b).to(DEV),
                                              cache_prev=_to_dev(cache, bf16) if cached else None, regions=regions))
    assert got.shape == (n, Ho, Wo, cout)
    for i in range(n):
        if cached:
            mask = oracle.rasterize(regions[i][0], Ho, Wo)
            want = oracle.conv_cached(x[i], w, b, k, s, p, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16)
            m = mask.astype(bool)
            assert np.array_equal(got[i][m], want[m])
        else:
            want = oracle.conv_cached(x[i], w, b, k, s, p, True, bf16=bf16)
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (cout, i)


def test_cached_conv_everything_reusable_launches_no_gemm(oracle):
    rng = np.random.default_rng(1)
    x = rng.standard_normal((1, 16, 16, 16)).astype(np.float32)
    w = rng.standard_normal((32, 3, 3, 16)).astype(np.float32)
    cache = rng.standard_normal((1, 16, 16, 32)).astype(np.float32)
    got = _to_np(binding.dc_cached_conv_layer(_layer(16, 32, 3, 1, 1, True), _to_dev(x, False), _to_dev(w, False), None,
                                              cache_prev=_to_dev(cache, False),
                                              regions=[(np.array([[0, 0, 16, 16]], np.int32), (0, 0))]))
    assert np.array_equal(got, cache)


@pytest.mark.parametrize("bf16", [False, True])
def test_uncached_layers(oracle, bf16):
    rng = np.random.default_rng(2)
    x = rng.standard_normal((2, 23, 30, 24)).astype(np.float32)
    y = rng.standard_normal((2, 23, 30, 24)).astype(np.float32)
    if bf16:
        x, y = oracle.round_bf16(x), oracle.round_bf16(y)
    for k, s, p in [(2, 2, 0), (3, 2, 1)]:
        got = _to_np(binding.dc_maxpool_layer(_to_dev(x, bf16), k, s, p))
        for n in range(2):
            assert np.array_equal(got[n], oracle.maxpool(x[n], k, s, p))
    for relu in (0, 1):
        got = _to_np(binding.dc_add_layer(_to_dev(x, bf16), _to_dev(y, bf16), relu))
        assert np.array_equal(got, oracle.add(x, y, relu, bf16=bf16))
    f = rng.integers(0, 256, (2, 9, 11, 3)).astype(np.uint8)
    dt = binding.DC_BF16 if bf16 else binding.DC_F32
    got = _to_np(binding.dc_frame_to_tensor(torch.from_numpy(f).to(DEV), dt))
    assert np.array_equal(got, oracle.frame_to_tensor(f))
    for ct in (4, 8):      # a tensor pixel of exactly 16 bytes (fp32 x 4, bf16 x 8) takes the per-pixel kernel
        got = _to_np(binding.dc_frame_to_tensor(torch.from_numpy(f).to(DEV), dt, c_tensor=ct))
        assert np.array_equal(got[..., :3], oracle.frame_to_tensor(f)) and not got[..., 3:].any()
    # element counts that are not whole 16-byte vectors
    xs, ys = x[:, :5, :7, :3].copy(), y[:, :5, :7, :3].copy()
    for relu in (0, 1):
        got = _to_np(binding.dc_add_layer(_to_dev(xs, bf16), _to_dev(ys, bf16), relu))
        assert np.array_equal(got, oracle.add(xs, ys, relu, bf16=bf16))


@pytest.mark.parametrize("bf16", [False, True])
def test_lrn_avgpool_concat_softmax_layers(oracle, bf16):
    """The un-cached layer types of Table 2 besides pooling and add, each against the oracle."""
    print(f"[more layers] bf16={bf16}", flush=True)
    rng = np.random.default_rng(9)
    tol = 2e-2 if bf16 else 1e-4
    n = 2
    for ch in (24, 7, 8):          # whole 16-byte vectors per pixel (several, one) and an odd channel count
        x = (rng.standard_normal((n, 13, 17, ch)) * 2).astype(np.float32)
        if bf16:
            x = oracle.round_bf16(x)
        xd = _to_dev(x, bf16)
        for size, within in [(5, False), (3, False), (1, False), (7, False), (3, True), (5, True)]:
            got = _to_np(binding.dc_lrn_layer(xd, size, 0.5, 0.75, 2.0, within))
            for i in range(n):
                assert _rel_err(got[i], oracle.lrn(x[i], size, 0.5, 0.75, 2.0, within, bf16=bf16)) <= tol, (ch, size, within)
        for k, s, p in [(3, 2, 1), (2, 2, 0), (13, 1, 0), (5, 3, 2)]:
            got = _to_np(binding.dc_avgpool_layer(xd, k, s, p))
            for i in range(n):
                assert _rel_err(got[i], oracle.avgpool(x[i], k, s, p, bf16=bf16)) <= tol, (ch, k, s, p)
            got = _to_np(binding.dc_maxpool_layer(xd, k, s, p))
            for i in range(n):
                assert np.array_equal(got[i], oracle.maxpool(x[i], k, s, p)), (ch, k, s, p)
    for cs in [(24, 8, 16), (24, 3), (5, 7, 24, 1), (8, 8)]:       # whole 16-byte vectors and odd channel counts
        parts = [np.ascontiguousarray(rng.standard_normal((n, 13, 17, c)).astype(np.float32)) for c in cs]
        if bf16:
            parts = [oracle.round_bf16(q) for q in parts]
        got = _to_np(binding.dc_concat_layer([_to_dev(q, bf16) for q in parts]))
        for i in range(n):
            assert np.array_equal(got[i], oracle.concat([q[i] for q in parts])), cs
    for c in (10, 64, 1000, 1024, 1500):      # up to 1024 channels stay in registers
        v = (rng.standard_normal((n, 2, 3, c)) * 4).astype(np.float32)
        if bf16:
            v = oracle.round_bf16(v)
        got = _to_np(binding.dc_softmax_layer(_to_dev(v, bf16)))
        for i in range(n):
            want = oracle.softmax(v[i], bf16=bf16)
            assert np.abs(got[i] - want).max() <= tol * max(float(want.max()), 1e-30), c


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,shape,cout", [(1, (6, 6, 32), 100), (3, (5, 5, 7), 33), (20, (1, 1, 256), 64), (5, (2, 3, 24), 1),
                                          (16, (2, 2, 64), 30), (37, (3, 3, 16), 50), (18, (1, 1, 40), 3)])
def test_fully_connected_layer(oracle, n, shape, cout, bf16):
    print(f"[fc] n={n} shape={shape} cout={cout} bf16={bf16}", flush=True)
    rng = np.random.default_rng(n * 100 + cout)
    K = int(np.prod(shape))
    x = rng.standard_normal((n,) + shape).astype(np.float32)
    w = (rng.standard_normal((cout, K)) * np.sqrt(2.0 / K)).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    if bf16:
        x, w = oracle.round_bf16(x), oracle.round_bf16(w)
    for relu, bias in [(True, b), (False, None)]:
        got = _to_np(binding.dc_fc_layer(_to_dev(x, bf16), _to_dev(w, bf16), None if bias is None else torch.from_numpy(bias).to(DEV), relu))
        assert got.shape == (n, 1, 1, cout)
        want = np.stack([oracle.fc(x[i], w, bias, relu, bf16=bf16) for i in range(n)])
        assert _rel_err(got, want) <= (2e-2 if bf16 else 1e-4)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,K,cout", [(4, 64, 40), (5, 8, 1), (16, 1032, 15), (17, 1024, 16), (32, 2056, 17), (33, 520, 48), (64, 1096, 33),
                                      (65, 2048, 31), (130, 72, 20)])
def test_fully_connected_layer_on_the_matrix_cores(oracle, n, K, cout, bf16):
    """Edges of the stream blocks (16, 32, 64), of the neuron block (16) and of the wavefronts' chunks of K (16 x 128 bytes).
    fp32: a sum of K products, partly in order: its error is below K 2^-24 of the sum of their magnitudes; bf16 adds one rounding."""
    print(f"[fc mfma] n={n} K={K} cout={cout} bf16={bf16}", flush=True)
    rng = np.random.default_rng(K + n)
    x = rng.standard_normal((n, 1, 1, K)).astype(np.float32)
    w = rng.standard_normal((cout, K)).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    if bf16:
        x, w = oracle.round_bf16(x), oracle.round_bf16(w)
    for relu, bias in [(True, b), (False, None)]:
        got = _to_np(binding.dc_fc_layer(_to_dev(x, bf16), _to_dev(w, bf16), None if bias is None else torch.from_numpy(bias).to(DEV), relu))
        x2, w2 = x.reshape(n, K).astype(np.float64), w.astype(np.float64)
        want = x2 @ w2.T + (0.0 if bias is None else bias)
        bound = (K + 2) * 2.0 ** -24 * (np.abs(x2) @ np.abs(w2).T + (0.0 if bias is None else np.abs(bias)))
        if relu:
            want = np.maximum(want, 0.0)
        if bf16:
            bound = bound + 2.0 ** -8 * np.abs(want)
        assert (np.abs(got.reshape(n, cout) - want) <= bound).all()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n", [9, 20, 64])
def test_fully_connected_rounds_and_the_rows_end(n, bf16):
    """One to five rounds of the wavefronts, ending on a chunk, a vector short of it and a vector behind it.  Whole numbers of
    few bits, so every sum is exact.  Vectors behind a row's end repeat its last one and must not count: an infinity there
    belongs to its stream and to neurons with a weight of their own sign alone."""
    print(f"[fc rounds] n={n} bf16={bf16}", flush=True)
    rng = np.random.default_rng(n)
    ve, cout = (8 if bf16 else 4), 18
    step = (8 if bf16 or n > 16 else 16) * 16 * ve
    for rounds in range(1, 6):
        for K in (rounds * step - ve, rounds * step, rounds * step + ve, (rounds - 1) * step + 16 * ve):
            x = rng.integers(-1, 2, (n, 1, 1, K)).astype(np.float32)
            w = rng.integers(-1, 2, (cout, K)).astype(np.float32)
            w[:, -1] = np.where(w[:, -1] == 0, 1, w[:, -1])
            want = x.reshape(n, K) @ w.T
            if bf16:
                want = torch.from_numpy(want).bfloat16().float().numpy()
            x[n // 2, 0, 0, -1] = np.inf
            want[n // 2] = np.where(w[:, -1] > 0, np.inf, -np.inf)
            got = _to_np(binding.dc_fc_layer(_to_dev(x, bf16), _to_dev(w, bf16), None, False)).reshape(n, cout)
            assert np.array_equal(got, want), K


@pytest.mark.parametrize("K", [1536, 1544, 2040, 2176, 4096, 9208, 9216])
def test_bf16_fully_connected_outputs_do_not_depend_on_the_number_of_streams(K):
    """Four streams take another kernel than nine and more, whose wavefronts fetch K in other pieces: the sums are the same bit for bit."""
    print(f"[fc order] K={K}", flush=True)
    gen = torch.Generator(DEV)
    gen.manual_seed(K)
    x = torch.randn((70, 1, 1, K), generator=gen, device=DEV).bfloat16()
    w = (torch.randn((37, K), generator=gen, device=DEV) * K ** -0.5).bfloat16()
    b = torch.randn(37, generator=gen, device=DEV) * 0.1
    want = torch.cat([binding.dc_fc_layer(x[s:s + 4].contiguous(), w, b, False) for s in range(0, 68, 4)])
    for n in (9, 16, 17, 32, 33, 64, 68):
        assert torch.equal(binding.dc_fc_layer(x[:n].contiguous(), w, b, False), want[:n]), n


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("H,W,ch,k,s,p", [(13, 17, 24, 3, 1, 1), (14, 9, 8, 3, 2, 0), (5, 6, 520, 3, 2, 2), (1, 1, 8, 3, 1, 1), (2, 7, 2056, 3, 3, 2),
                                          (7, 7, 1024, 7, 1, 0), (9, 5, 16, 5, 1, 2), (8, 11, 8, 4, 3, 1), (11, 12, 40, 9, 2, 4)])
def test_pooling_windows(oracle, H, W, ch, k, s, p, bf16):
    """3x3 windows on every side of the padding, windows with whole and partial groups of columns, rows longer than a workgroup;
    values of the type's extremes and infinities."""
    print(f"[pool] {H}x{W}x{ch} k={k} s={s} p={p} bf16={bf16}", flush=True)
    rng = np.random.default_rng(H * 100 + ch)
    x = (rng.standard_normal((3, H, W, ch)) * 4).astype(np.float32)
    if bf16:
        x = oracle.round_bf16(x)
    got = _to_np(binding.dc_avgpool_layer(_to_dev(x, bf16), k, s, p))
    for i in range(3):
        assert _rel_err(got[i], oracle.avgpool(x[i], k, s, p, bf16=bf16)) <= (2e-2 if bf16 else 1e-4)
    x[0, 0, 0, :4] = [-np.inf, np.inf, -3.3895314e38, 3.3895314e38]
    x[1, :, :, 0] = -np.inf
    x[2, :, :, 1] = -3.3895314e38
    if bf16:
        x = oracle.round_bf16(x)
    got = _to_np(binding.dc_maxpool_layer(_to_dev(x, bf16), k, s, p))
    for i in range(3):
        assert np.array_equal(got[i], oracle.maxpool(x[i], k, s, p))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("ch,size,beta,kappa", [(8, 5, 0.75, 2.0), (96, 5, 0.75, 1.0), (24, 3, 0.75, 1e-3), (40, 5, 0.5, 1.0)])
def test_lrn_power(oracle, ch, size, beta, kappa, bf16):
    """The exponent 3/4 (two roots) and another one (logarithm).  fp32: the sum of at most five squares, two roots and two
    products are each off by at most a few 2^-24; the logarithm form by |beta log2 x| 2^-22 more."""
    print(f"[lrn] ch={ch} size={size} beta={beta} kappa={kappa} bf16={bf16}", flush=True)
    rng = np.random.default_rng(ch)
    x = (rng.standard_normal((2, 9, 11, ch)) * np.exp(rng.uniform(-6, 6, (2, 9, 11, 1)))).astype(np.float32)
    if bf16:
        x = oracle.round_bf16(x)
    got = _to_np(binding.dc_lrn_layer(_to_dev(x, bf16), size, 0.7, beta, kappa, False))
    want = np.stack([oracle.lrn(x[i], size, 0.7, beta, kappa, False, bf16=bf16) for i in range(2)]).astype(np.float64)
    rel = 2.0 ** -7 if bf16 else (16 * 2.0 ** -24 if beta == 0.75 else 40 * 2.0 ** -24)
    assert (np.abs(got - want) <= rel * np.abs(want)).all()


@pytest.mark.parametrize("size,alpha,kappa,ch", [(5, 1e-4, 2.0, 192), (5, 1.0, 1.0, 64), (3, 5e-2, 1.0, 64)])
def test_lrn_fp32_is_rounded_like_three_operations(size, alpha, kappa, ch):
    """fp32, exponent 3/4, against 64 bits: what is left is the rounding of the product (rms at most 2^-24 / sqrt(3) of the
    value), of the power (the same) and of the denominator and its sum of squares (three roundings, times 3/4): together
    2^-24 / sqrt(3) * sqrt(1 + 1 + 3 * 9/16) = 6.6e-8.  Two hardware roots without correction: 7.2e-8 to 7.9e-8."""
    print(f"[lrn precision] size={size} alpha={alpha} kappa={kappa} ch={ch}", flush=True)
    x = (np.random.default_rng(ch).standard_normal((2, 32, 32, ch)) * 8).astype(np.float32)
    got = _to_np(binding.dc_lrn_layer(_to_dev(x, False), size, alpha, 0.75, kappa, False)).astype(np.float64)
    sq = np.pad(x.astype(np.float64) ** 2, ((0, 0), (0, 0), (0, 0), (size // 2, size // 2)))
    total = sum(sq[..., i:i + ch] for i in range(size))
    want = x * (np.float64(np.float32(kappa)) + np.float64(np.float32(alpha) / np.float32(size)) * total) ** -0.75
    rms = float(np.sqrt(np.mean(((got - want) / want) ** 2)))
    assert rms <= 6.6e-8, rms


# 5x5 stride-1 bf16 layers on the 3x3 GEMM kernel's frame: both arrangements, every number of units per wavefront, a wavefront
# row with a unit less, paddings other than 2, ragged maps, one and several chunks, a K split.
@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("case", [(22, 30, 32, 128, 2, (1, 3, 1, 0)), (22, 30, 96, 128, 2, (1, 8, 1, 0)), (13, 17, 64, 256, 2, (1, 7, 1, 0)),
                                  (22, 30, 96, 64, 2, (2, 4, 1, 0)), (19, 23, 32, 192, 0, (2, 7, 1, 0)), (19, 23, 64, 64, 4, (2, 12, 1, 0)),
                                  (14, 14, 128, 128, 1, (1, 5, 3, 0)), (22, 30, 64, 64, 2, (-1, -1, -1, -1)), (21, 13, 96, 256, 2, (-1, -1, -1, -1))])
def test_5x5_conv_kernel_shapes(oracle, case, cached):
    H, W, cin, cout, p, tuning = case
    print(f"[5x5 conv] case={case} cached={cached}", flush=True)
    rng = np.random.default_rng(H * 1000 + W * 10 + cin + cout)
    n, Ho, Wo = 3, H + 2 * p - 4, W + 2 * p - 4
    x = oracle.round_bf16(rng.standard_normal((n, H, W, cin)).astype(np.float32))
    w = oracle.round_bf16((rng.standard_normal((cout, 5, 5, cin)) * np.sqrt(2.0 / (cin * 25))).astype(np.float32))
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    cache = oracle.round_bf16(rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32))
    regions = None
    if cached:
        regions = [(np.array([[1, 2, Wo - 7, Ho - 6], [Wo - 5, 1, 3, 4]], np.int32), (2, -1)),
                   (np.array([[0, 0, Wo - 1, Ho - 3]], np.int32), (1, 2)), (np.zeros((0, 4), np.int32), (0, 0))]
    binding.dc_conv_tuning(*tuning)
    try:
        got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, 5, 1, p, True), _to_dev(x, True), _to_dev(w, True), torch.from_numpy(b).to(DEV),
                                                  cache_prev=_to_dev(cache, True) if cached else None, regions=regions))
    finally:
        binding.dc_conv_tuning()
    for i in range(n):
        if cached:
            mask = oracle.rasterize(regions[i][0], Ho, Wo)
            want = oracle.conv_cached(x[i], w, b, 5, 1, p, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=True)
            m = mask.astype(bool)
            assert np.array_equal(got[i][m], want[m]), "copied pixels must be bit-identical"
        else:
            want = oracle.conv_cached(x[i], w, b, 5, 1, p, True, bf16=True)
        # a bf16 rounding of the result (2^-9) and fp32 sums that may round to the neighbour
        assert (np.abs(got[i].astype(np.float64) - want) <= 2.0 ** -7 * np.abs(want) + 1e-5 * np.abs(want).max()).all(), (case, i)


@pytest.mark.parametrize("cin,cout,tuning", [(128, 128, (1, 8, 1, 0)), (128, 64, (2, 12, 1, 0)), (192, 128, (1, 3, 1, 0))])
def test_5x5_sums_are_rounded_once_per_stage(cin, cout, tuning):
    """Inputs whose second half of channels repeats the first with negated weights: the exact output is zero and the stored
    value is what the fp32 sums lost.  Expected: every stage (5 taps x 32 channels) rounds its own running sum five times and
    the total once, each by at most 2^-24 / sqrt(3) of the sum (rms); half as much again is allowed.  One chain over all of K
    rounds the total at every tap: at least sqrt(5) of that, measured 3.2."""
    H, W, p = 22, 30, 2
    print(f"[5x5 sums] cin={cin} cout={cout} tuning={tuning}", flush=True)
    rng = np.random.default_rng(cin + cout)
    x = _to_dev(np.abs(rng.standard_normal((1, H, W, cin // 2))).astype(np.float32), True)
    w = _to_dev(np.abs(rng.standard_normal((cout, 5, 5, cin // 2))).astype(np.float32), True)
    x, w = torch.cat([x, x], 3).contiguous(), torch.cat([w, -w], 3).contiguous()
    binding.dc_conv_tuning(*tuning)
    try:
        got = binding.dc_cached_conv_layer(_layer(cin, cout, 5, 1, p, False), x, w, None)
    finally:
        binding.dc_conv_tuning()
    xd, wd = x[0, H // 2 - 2:H // 2 + 3, W // 2 - 2:W // 2 + 3].double().cpu().numpy(), w[0].double().cpu().numpy()
    taps = (xd * wd).reshape(5, 5, cin // 32, 32).sum(-1)                      # [ky][kx][chunk]
    run = np.cumsum(taps.sum(1).T.reshape(-1))                                # after every stage: [chunk][ky]
    in_stage = np.cumsum(taps, axis=1)
    rms = 2.0 ** -24 / np.sqrt(3.0) * np.sqrt((run ** 2).sum() + (in_stage ** 2).sum())
    inner = got[0, 2:-2, 2:-2].double().cpu().numpy()
    assert np.sqrt((inner ** 2).mean()) <= 1.5 * rms, np.sqrt((inner ** 2).mean()) / rms


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("H,W", [(4, 4), (2, 3), (9, 4), (5, 1), (1, 7), (4, 13)])
@pytest.mark.parametrize("cin,cout,k,tuning", [(0, 64, 3, None), (64, 64, 3, None), (64, 64, 3, (3, 4, 1, 1)), (64, 128, 1, None), (128, 128, 5, None),
                                               (64, 64, 3, (0, 2, 1, 0)), (64, 64, 3, (0, 1, 2, 0)), (64, 128, 1, (-1, 4, -1, -1)), (64, 128, 1, (-1, 8, -1, -1))])
def test_conv_on_maps_of_one_unit_column(oracle, cin, cout, k, tuning, H, W, bf16):
    """Maps of a single 4x4 unit, unit column or unit row, several streams, in full: every pixel of every stream is written."""
    cin = cin or (8 if bf16 else 4)                   # (a pixel of one 16-byte vector: the first-layer kernel)
    print(f"[one unit column] {H}x{W} {cin}->{cout} k={k} bf16={bf16} tuning={tuning}", flush=True)
    rng = np.random.default_rng(H * 100 + W + cin + k)
    x = rng.standard_normal((5, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, k, k, cin)) * np.sqrt(2.0 / (cin * k * k))).astype(np.float32)
    if bf16:
        x, w = oracle.round_bf16(x), oracle.round_bf16(w)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    if tuning:
        binding.dc_conv_tuning(*tuning)
    try:
        got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, k, 1, k // 2, True), _to_dev(x, bf16), _to_dev(w, bf16), torch.from_numpy(b).to(DEV)))
    finally:
        binding.dc_conv_tuning()
    for i in range(5):
        assert _rel_err(got[i], oracle.conv_cached(x[i], w, b, k, 1, k // 2, True, bf16=bf16)) <= (2e-2 if bf16 else 1e-4), i


PW_CASES = [
    # H, W, cin, cout, stride
    (13, 18, 64, 64, 1),       # one chunk in bf16, two in fp32
    (13, 18, 96, 24, 1),       # last chunk half empty (bf16), cout below one channel tile
    (9, 9, 1024, 72, 1),       # more chunks than ring stages; channel tile with a tail
    (14, 14, 256, 200, 1),
    (8, 8, 8, 8, 1),           # a single 16-byte vector per pixel (bf16)
    (27, 21, 128, 136, 2),     # strided projection, odd map
    (28, 28, 64, 256, 2),
]


@pytest.fixture
def pw_tile(request):
    """Forces the 1x1 kernel's tile (units per workgroup) for one test."""
    binding.dc_conv_tuning(units_per_workgroup=request.param)
    yield request.param
    binding.dc_conv_tuning()


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("pw_tile", [4, 8], indirect=True)
@pytest.mark.parametrize("case", PW_CASES)
def test_pointwise_kernel(oracle, case, pw_tile, bf16, cached):
    """1x1 convolutions (stride 1 and 2) on the GEMM kernel with the staged K ring, both tile sizes."""
    H, W, cin, cout, s = case
    print(f"[pointwise] case={case} tile={pw_tile} bf16={bf16} cached={cached}", flush=True)
    rng = np.random.default_rng(sum(case) + 3)
    n = 3
    Ho, Wo = (H - 1) // s + 1, (W - 1) // s + 1
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, 1, 1, cin)) * np.sqrt(2.0 / cin)).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    cache = rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = None
    if cached:
        regions = [(np.array([[1, 0, Wo - 3, Ho - 2]], np.int32), (1, 1)), (np.zeros((0, 4), np.int32), (0, 0)),
                   (np.array([[0, 1, 2, Ho - 2], [3, 2, Wo - 4, 3]], np.int32), (1, 0))]
    got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, 1, s, 0, True), _to_dev(x, bf16), _to_dev(w, bf16),
                                              torch.from_numpy(b).to(DEV),
                                              cache_prev=_to_dev(cache, bf16) if cached else None, regions=regions))
    assert got.shape == (n, Ho, Wo, cout)
    for i in range(n):
        if cached:
            mask = oracle.rasterize(regions[i][0], Ho, Wo)
            want = oracle.conv_cached(x[i], w, b, 1, s, 0, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16)
            m = mask.astype(bool)
            assert np.array_equal(got[i][m], want[m])
        else:
            want = oracle.conv_cached(x[i], w, b, 1, s, 0, True, bf16=bf16)
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (case, i)


# The kernel whose four wavefronts split K in pieces of 128 bytes, which takes layers of few units: fewer pieces than wavefronts, a last
# piece that is not whole, more than two pieces per wavefront, channels that end inside a 32-channel tile; from (14, 14, 256, 200) on
# some with two units per workgroup, the last ones with one unit in the last.
@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", PW_CASES + [(7, 7, 1096, 40, 1), (15, 13, 840, 8, 2), (8, 5, 192, 264, 1), (12, 12, 840, 328, 1), (9, 9, 40, 1000, 1)])
def test_pointwise_kernel_with_split_k(oracle, case, bf16, cached):
    test_pointwise_kernel(oracle, case, None, bf16, cached)


@pytest.mark.parametrize("bf16", [False, True])
def test_tuning_values_of_3x3_layers_leave_1x1_layers_alone(bf16):
    """Units per workgroup that the 1x1 kernel has no tile for are ignored: the same bits, whatever another layer is tuned to."""
    gen = torch.Generator(DEV)
    gen.manual_seed(4)
    dt = torch.bfloat16 if bf16 else torch.float32
    x = torch.randn((4, 56, 56, 256), generator=gen, device=DEV).to(dt)
    w = torch.randn((256, 1, 1, 256), generator=gen, device=DEV).to(dt)
    run = lambda: binding.dc_cached_conv_layer(_layer(256, 256, 1, 1, 0, True), x, w, None)
    want = run()
    for units in (1, 2, 3, 5, 18):
        binding.dc_conv_tuning(units_per_workgroup=units)
        try:
            assert torch.equal(run(), want), units
        finally:
            binding.dc_conv_tuning()


# 3x3 layers of few units: channels that end inside a tile, rows that are no whole chunks, windows without padding and with stride 2,
# maps of a few units with deep rows.
FEW_UNIT_CASES = [  # (streams, H, W, cin, cout, s, p)
    (2, 5, 9, 8, 8, 1, 1),
    (1, 13, 11, 40, 24, 2, 1),
    (3, 8, 6, 96, 72, 1, 0),
    (2, 7, 7, 512, 128, 1, 1),
    (1, 16, 16, 256, 256, 1, 1),
    (1, 17, 13, 256, 264, 1, 1),
    (4, 14, 14, 64, 264, 2, 1),
    (2, 9, 10, 24, 136, 2, 2),
]


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", FEW_UNIT_CASES)
def test_3x3_layers_of_few_units(oracle, case, bf16, cached):
    """Tolerance: both sides sum at least in fp32 (9 cin terms: below 1e-5 of the map); bf16 results are rounded, 2^-8 each."""
    n, H, W, cin, cout, s, p = case
    print(f"[few-unit 3x3] case={case} bf16={bf16} cached={cached}", flush=True)
    rng = np.random.default_rng(sum(case) + 11)
    Ho, Wo = (H + 2 * p - 3) // s + 1, (W + 2 * p - 3) // s + 1
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, 3, 3, cin)) * np.sqrt(2.0 / (cin * 9))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    cache = rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = [_random_regions(rng, oracle, Ho, Wo) for _ in range(n)] if cached else None
    layer, wd = _layer(cin, cout, 3, s, p, True), _to_dev(w, bf16)
    run = lambda weights, packed: _to_np(binding.dc_cached_conv_layer(
        layer, _to_dev(x, bf16), weights, torch.from_numpy(b).to(DEV), cache_prev=_to_dev(cache, bf16) if cached else None,
        regions=regions, packed=packed))
    got, packed = run(wd, None), binding.dc_pack_conv_weights(layer, wd)
    if packed is not None:
        assert np.array_equal(got, run(torch.zeros_like(wd), packed)), "packed weights must not change a bit"
    for i in range(n):
        mask = oracle.rasterize(regions[i][0], Ho, Wo) if cached else np.zeros((Ho, Wo), np.uint8)
        want = oracle.conv_cached(x[i], w, b, 3, s, p, True, cache_prev=cache[i], mask=mask, bf16=bf16,
                                  dxy=regions[i][1] if cached else (0, 0))
        m = mask.astype(bool)
        assert np.array_equal(got[i][m], want[m])
        assert _rel_err(got[i], want) <= (1e-2 if bf16 else 1e-5), (case, i)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case,tuning", [((20, 24, 4, 32, 3, 1, 1), None), ((20, 24, 64, 64, 3, 1, 1), None), ((20, 24, 64, 128, 1, 1, 0), None),
                                         ((21, 25, 32, 48, 5, 2, 2), None), ((21, 25, 6, 10, 3, 1, 1), None), ((12, 12, 512, 64, 3, 1, 1), None),
                                         ((20, 24, 64, 64, 3, 1, 1), (0, 2, 1, 0)), ((12, 12, 512, 64, 3, 1, 1), (0, 2, 4, 0)),
                                         ((20, 24, 64, 128, 1, 1, 0), (-1, 4, -1, -1)), ((20, 24, 64, 128, 1, 1, 0), (-1, 8, -1, -1))])
def test_leaky_relu_in_every_conv_kernel(oracle, case, tuning, bf16):
    """relu = 2 (leaky, slope 0.1) in the epilogue of the first-layer, 3x3, 1x1 (fp32: split K as well), general, element-load and
    split-K kernels; the tuned cases name the 3x3 kernel, its split of K with the reduction, and the 1x1 ring's two tiles."""
    H, W, cin, cout, k, s, p = case
    if bf16 and cin == 4:
        cin = 8
    print(f"[leaky] case={case} tuning={tuning} bf16={bf16}", flush=True)
    rng = np.random.default_rng(sum(case) + 1)
    x = rng.standard_normal((2, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, k, k, cin)) * np.sqrt(2.0 / (cin * k * k))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    if bf16:
        x, w = oracle.round_bf16(x), oracle.round_bf16(w)
    if tuning:
        binding.dc_conv_tuning(*tuning)
    try:
        got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, k, s, p, 2), _to_dev(x, bf16), _to_dev(w, bf16), torch.from_numpy(b).to(DEV)))
    finally:
        binding.dc_conv_tuning()
    for i in range(2):
        want = oracle.conv_cached(x[i], w, b, k, s, p, 2, bf16=bf16)
        assert (want < 0).any()
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (case, i)


# Launches of the general kernel with at least three workgroups on every two CUs switch to short stages of the
# narrowest channel chunk (one kernel row of taps, or about a dozen taps where four wavefronts share a stage):
# shapes that reach that many workgroups at a size the oracle still handles.
SHORT_STAGE_CASES = [
    # n, H, W, cin, cout, k, s, p
    (12, 64, 64, 32, 128, 3, 2, 1),     # 384 workgroups of 4 units x 64 channels: 3 taps per stage
    (6, 48, 48, 16, 128, 5, 1, 2),      # 432 workgroups: 5 taps per stage
    (16, 28, 28, 16, 32, 5, 1, 2),      # 392 workgroups of 2 units x 32 channels: 13 + 12 taps (tap tail)
    (12, 62, 66, 40, 72, 3, 2, 0),      # channel tail in the chunk, ragged channel tile, no padding
]


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", SHORT_STAGE_CASES)
def test_general_kernel_short_stages(oracle, case, bf16, cached):
    n, H, W, cin, cout, k, s, p = case
    print(f"[short stages] case={case} bf16={bf16} cached={cached}", flush=True)
    rng = np.random.default_rng(sum(case) + 7)
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, k, k, cin)) * np.sqrt(2.0 / (cin * k * k))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    Ho, Wo = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    cache = rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = None
    if cached:      # few reusable pixels, so that the launch keeps its many workgroups
        regions = []
        for i in range(n):
            rw, rh = int(rng.integers(2, 7)), int(rng.integers(2, 7))
            rx, ry = int(rng.integers(2, Wo - rw - 2)), int(rng.integers(2, Ho - rh - 2))
            regions.append((np.array([[rx, ry, rw, rh]], np.int32), (int(rng.integers(-2, 3)), int(rng.integers(-2, 3)))))
    got = _to_np(binding.dc_cached_conv_layer(_layer(cin, cout, k, s, p, True), _to_dev(x, bf16), _to_dev(w, bf16),
                                              torch.from_numpy(b).to(DEV),
                                              cache_prev=_to_dev(cache, bf16) if cached else None, regions=regions))
    for i in range(n):
        if cached:
            mask = oracle.rasterize(regions[i][0], Ho, Wo)
            want = oracle.conv_cached(x[i], w, b, k, s, p, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16)
            m = mask.astype(bool)
            assert np.array_equal(got[i][m], want[m]), "copied pixels must be bit-identical"
        else:
            want = oracle.conv_cached(x[i], w, b, k, s, p, True, bf16=bf16)
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (case, i)


KERNEL_SHAPE_CASES = [
    # H, W, cin, cout, kh, kw, s, ph, pw, dil
    (23, 31, 16, 32, 1, 7, 1, 0, 3, 1),      # a row kernel
    (23, 31, 16, 32, 7, 1, 1, 3, 0, 1),      # a column kernel
    (26, 30, 32, 64, 3, 3, 1, 2, 2, 2),      # dilated by 2, same size
    (33, 29, 32, 32, 3, 1, 2, 1, 0, 1),      # column kernel with stride 2
    (24, 28, 16, 48, 5, 3, 1, 4, 2, 2),      # not square and dilated
    (19, 21, 5, 7, 2, 5, 3, 0, 1, 1),        # odd channel counts (element loads), stride 3
    (30, 30, 8, 16, 3, 3, 1, 3, 3, 3),       # dilated by 3
]


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", KERNEL_SHAPE_CASES)
def test_kernels_that_are_not_square_or_dilated(oracle, case, bf16, cached):
    """dc_layer.k2 / p2 / dil: the general conv kernels with a kernel of k rows x k2 columns and taps dil pixels apart."""
    H, W, cin, cout, kh, kw, s, ph, pw, dil = case
    print(f"[kernel shapes] case={case} bf16={bf16} cached={cached}", flush=True)
    rng = np.random.default_rng(sum(case))
    n = 2
    x = rng.standard_normal((n, H, W, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, kh, kw, cin)) * np.sqrt(2.0 / (cin * kh * kw))).astype(np.float32)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    layer = dict(type=synth.CONV, k=kh, s=s, p=ph, cin=cin, cout=cout, relu=1, in0=0, in1=-1, k2=kw, p2=pw, dil=dil)
    Ho, Wo, _ = synth.tensor_shapes([layer], H, W, cin)[1]
    cache = rng.standard_normal((n, Ho, Wo, cout)).astype(np.float32)
    if bf16:
        x, w, cache = oracle.round_bf16(x), oracle.round_bf16(w), oracle.round_bf16(cache)
    regions = None
    if cached:
        regions = [(np.array([[1, 2, Wo - 4, Ho - 5]], np.int32), (1, -1)), (np.array([[0, 0, Wo - 2, Ho - 1]], np.int32), (1, 0))]
    got = _to_np(binding.dc_cached_conv_layer(layer, _to_dev(x, bf16), _to_dev(w, bf16), torch.from_numpy(b).to(DEV),
                                              cache_prev=_to_dev(cache, bf16) if cached else None, regions=regions))
    assert got.shape == (n, Ho, Wo, cout)
    for i in range(n):
        if cached:
            mask = oracle.rasterize(regions[i][0], Ho, Wo)
            want = oracle.conv_cached(x[i], w, b, kh, s, ph, True, cache_prev=cache[i], mask=mask, dxy=regions[i][1], bf16=bf16,
                                      k2=kw, p2=pw, dil=dil)
            m = mask.astype(bool)
            assert np.array_equal(got[i][m], want[m])
        else:
            want = oracle.conv_cached(x[i], w, b, kh, s, ph, True, bf16=bf16, k2=kw, p2=pw, dil=dil)
        assert _rel_err(got[i], want) <= (2e-2 if bf16 else 1e-4), (case, i)


def test_raster_positions_of_a_large_batch(oracle):
    """40 streams of 416 x 416: the product of a unit's raster position and the units per map passes 2^32, where the
    kernels' division by a magic number is one too large and is corrected.  First-layer shape and a 3x3 layer; the first
    and the last stream against the oracle."""
    n, H, W = 40, 416, 416
    for cin, cout in ((8, 32), (32, 64)):
        rng = np.random.default_rng(cin)
        x = oracle.round_bf16(rng.standard_normal((n, H, W, cin)).astype(np.float32))
        w = oracle.round_bf16((rng.standard_normal((cout, 3, 3, cin)) * np.sqrt(2.0 / (cin * 9))).astype(np.float32))
        got = binding.dc_cached_conv_layer(_layer(cin, cout, 3, 1, 1, True), _to_dev(x, True), _to_dev(w, True), None)
        torch.cuda.synchronize()
        for s in (0, n - 1):
            want = oracle.conv_cached(x[s], w, None, 3, 1, 1, True, bf16=True)
            assert _rel_err(got[s].float().cpu().numpy(), want) <= 2e-2, (cin, s)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("H,W,ch,k,s,p,n", [(33, 41, 48, 3, 1, 1, 5), (40, 24, 64, 3, 2, 1, 7), (17, 19, 8, 3, 2, 0, 9), (30, 30, 96, 2, 1, 0, 3),
                                             (9, 9, 16, 9, 1, 0, 11), (64, 64, 32, 3, 1, 2, 1)])
def test_pooling_workgroups_cover_every_stream(oracle, H, W, ch, k, s, p, n, bf16):
    """Workgroups dealt to the XCDs in runs: numbers of them that are no multiple of eight, maps of one and of many workgroups,
    a partial last one per stream."""
    print(f"[pool groups] {H}x{W}x{ch} k={k} s={s} p={p} n={n} bf16={bf16}", flush=True)
    x = (np.random.default_rng(H + ch).standard_normal((n, H, W, ch)) * 4).astype(np.float32)
    if bf16:
        x = oracle.round_bf16(x)
    got_max, got_avg = (_to_np(f(_to_dev(x, bf16), k, s, p)) for f in (binding.dc_maxpool_layer, binding.dc_avgpool_layer))
    for i in range(n):
        assert np.array_equal(got_max[i], oracle.maxpool(x[i], k, s, p)), i
        assert _rel_err(got_avg[i], oracle.avgpool(x[i], k, s, p, bf16=bf16)) <= (2e-2 if bf16 else 1e-4), i


@pytest.mark.parametrize("n,K,cout", [(2, 1024, 100), (2, 9216, 256), (3, 4096, 255), (4, 4096, 512), (4, 4100, 3), (2, 4096, 1024), (2, 1028, 1)])
def test_fc_few_fp32_streams_and_neurons(n, K, cout):
    """A wavefront per neuron for two to four fp32 streams: against 64 bits.  A lane adds K / 256 products to each of its four
    sums, each rounded once, then eight levels of pairs, the bias: rms error at most 2^-24 / sqrt(3) sqrt(K / 256 + 10) of the root of the sum
    of the squared products, by which the result is compared; five of those for the largest of n cout values."""
    print(f"[fc few] n={n} K={K} cout={cout}", flush=True)
    rng = np.random.default_rng(K + cout)
    x = np.maximum(rng.standard_normal((n, 1, 1, K)), 0).astype(np.float32)
    w = rng.standard_normal((cout, K)).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    got = _to_np(binding.dc_fc_layer(_to_dev(x, False), _to_dev(w, False), torch.from_numpy(b).to(DEV), False)).reshape(n, cout)
    xd, wd = x.reshape(n, K).astype(np.float64), w.astype(np.float64)
    want = xd @ wd.T + b
    scale = np.sqrt((xd ** 2) @ (wd ** 2).T) + np.abs(want)
    err = (got - want) / scale
    bound = 2.0 ** -24 / np.sqrt(3.0) * np.sqrt(K / 256 + 10)
    assert np.sqrt((err ** 2).mean()) <= bound and np.abs(err).max() <= 5 * bound, (np.sqrt((err ** 2).mean()) / bound, np.abs(err).max() / bound)


# Single-layer calls take turns on two workspaces; the plan travels with the copies in one launch while those take at most 32
# rectangles of whole 16-byte vectors.  Calls one behind the other, and from three threads on streams of their own, against calls that
# are waited for: 32 rectangles, 33, channel runs that are no whole vectors, no rectangle at all.
@pytest.mark.parametrize("per_stream,cout,bf16", [(8, 64, True), (8, 64, False), (11, 64, True), (8, 20, True), (0, 64, True)])
def test_single_layer_calls_without_a_wait_in_between(per_stream, cout, bf16):
    import threading
    n, H, W, cin = 4, 24, 28, 32
    dt = torch.bfloat16 if bf16 else torch.float32
    gen = torch.Generator(DEV)
    gen.manual_seed(per_stream + cout)
    w = torch.randn((cout, 3, 3, cin), generator=gen, device=DEV).to(dt) * 0.1
    layer = _layer(cin, cout, 3, 1, 1, True)
    rng = np.random.default_rng(7)
    calls = []
    for c in range(10):
        regions = []
        for s in range(n - 1):
            rects = [[1 + 2 * j, 1 + int(rng.integers(0, 4)), 2, int(rng.integers(1, 16))] for j in range(per_stream)]
            regions.append((np.array(rects, np.int32).reshape(-1, 4), (int(rng.integers(-1, 2)), int(rng.integers(-1, 2)))))
        regions.append((np.array([[2, 3, 9, 11]] * (1 if per_stream == 11 else 0), np.int32).reshape(-1, 4), (1, 0)))
        if per_stream == 8:
            regions[-1] = (np.array([[3 * j, 0, 3, 24] for j in range(8)], np.int32), (0, 0))
        x = torch.randn((n, H, W, cin), generator=gen, device=DEV).to(dt)
        prev = torch.randn((n, H, W, cout), generator=gen, device=DEV).to(dt)
        calls.append((x, prev, regions))
    torch.cuda.synchronize()

    def run(i):
        x, prev, regions = calls[i]
        return binding.dc_cached_conv_layer(layer, x, w, None, prev, regions)
    want = []
    for i in range(10):
        want.append(run(i))
        torch.cuda.synchronize()
        x, prev, regions = calls[i]
        for s, (rects, (dx, dy)) in enumerate(regions):
            for rx, ry, rw, rh in rects.tolist():
                assert torch.equal(want[i][s, ry:ry + rh, rx:rx + rw], prev[s, ry + dy:ry + dy + rh, rx + dx:rx + dx + rw])
    got = [run(i) for i in range(10)]
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    bad = []

    def worker():
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            res = [run(i) for i in range(10)]
            st.synchronize()
        bad.extend(i for i in range(10) if not torch.equal(res[i], want[i]))
    threads = [threading.Thread(target=worker) for _ in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not bad and len(binding._conv_ws.free) <= binding._conv_ws.KEPT


# The bf16 kernel whose weights go straight to registers (arrangement 5; a K split of 2 selects its 128-channel workgroups):
# 6 to 8 units per workgroup, a last workgroup that is not full, one channel chunk (first and last at once), two and more,
# ragged maps, both widths of a workgroup.
DEEP_CASES = [
    (22, 30, 32, 256, (5, 8, -1, -1)), (22, 30, 64, 256, (5, 7, -1, -1)), (13, 17, 96, 256, (5, 6, -1, -1)),
    (14, 14, 128, 512, (5, 8, 2, -1)), (37, 41, 32, 128, (5, 7, -1, -1)), (5, 3, 160, 384, (5, 6, -1, -1)),
    (45, 61, 64, 128, (5, 8, -1, -1)),
]


def _kernel_of(cin, cout, n, H, W, tuning):
    """The kernel that a 3x3 bf16 layer of this shape takes under a tuning (a full frame of a stack of this layer alone)."""
    layer = dict(_layer(cin, cout, 3, 1, 1, True), in0=0, in1=-1)
    binding.dc_conv_tuning(*tuning)
    try:
        runner = binding.StackRunner([layer], [np.zeros((cout, 3, 3, cin), np.float32)], [np.zeros(cout, np.float32)], n, H, W, cin,
                                     block=1, radius=1, dtype=binding.DC_BF16, overlap=False)
        runner.step(torch.zeros((n, H, W, cin), dtype=torch.uint8, device=DEV))
        torch.cuda.synchronize()
        return binding.conv_kernel_name(runner.layer_stats()["kernel_id"][0])
    finally:
        binding.dc_conv_tuning()


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("case", DEEP_CASES)
def test_deep_conv_kernel_shapes(oracle, case, cached):
    if cached and case[1] < 8:
        pytest.skip("the rectangles of the cached case need a wider map")
    H, W, cin, cout, tuning = case
    assert _kernel_of(cin, cout, 2, H, W, tuning) == f"conv_deep_kernel<{2 if cout % 256 or tuning[2] == 2 else 4}, {tuning[1]}>"
    test_fast_conv_kernel_shapes(oracle, case, True, cached)


def test_deep_conv_kernel_bits_and_borders():
    """The same sums in the same order as the kernel it stands in for (chunks of 32 channels, K not split), leaky and no
    activation, no bias, infinities in the padding's neighbours and a NaN: the same bits."""
    n, H, W, cin, cout = 3, 23, 21, 96, 256
    g = torch.Generator(DEV)
    g.manual_seed(5)
    x = torch.randn((n, H, W, cin), generator=g, device=DEV).bfloat16()
    x[0, 0, 0, 5], x[1, H - 1, W - 1, 7], x[2, 4, 4, 0] = float("inf"), float("-inf"), float("nan")
    w = (torch.randn((cout, 3, 3, cin), generator=g, device=DEV) * 0.05).bfloat16()
    b = torch.randn(cout, generator=g, device=DEV)
    assert _kernel_of(cin, cout, n, H, W, (1, 8, 1, 0)).startswith("conv_fast_kernel")
    for tuning, name in (((5, 8, -1, -1), "conv_deep_kernel<4, 8>"), ((5, 7, -1, -1), "conv_deep_kernel<4, 7>"), ((5, 6, 2, -1), "conv_deep_kernel<2, 6>")):
        assert _kernel_of(cin, cout, n, H, W, tuning) == name
    for relu, bias in ((0, b), (1, b), (2, None)):
        layer = dict(_layer(cin, cout, 3, 1, 1, True), relu=relu)
        wp = binding.dc_pack_conv_weights(layer, w)
        out = {}
        for tuning in ((1, 8, 1, 0), (5, 8, -1, -1), (5, 7, -1, -1), (5, 6, 2, -1)):
            print(f"[deep bits] relu={relu} {tuning}", flush=True)
            binding.dc_conv_tuning(*tuning)
            try:
                out[tuning] = binding.dc_cached_conv_layer(layer, x, w, bias, packed=wp).view(torch.int16)
            finally:
                binding.dc_conv_tuning()
        base = out.pop((1, 8, 1, 0))
        for tuning, got in out.items():
            assert torch.equal(got, base), tuning


# The bf16 kernel that takes whole maps (arrangement 6): one tile of pixels per row of wavefronts to four, tiles that end
# inside the map, one channel chunk and more, 64 and 128 channels per workgroup.  Same bits as the kernel it stands in for.
@pytest.mark.parametrize("H,W,cin,cout,n", [(13, 13, 64, 128, 3), (14, 14, 32, 64, 2), (14, 9, 96, 192, 1), (1, 1, 32, 64, 4), (5, 14, 160, 128, 2),
                                            (14, 3, 64, 256, 2), (7, 7, 128, 64, 3)])
def test_whole_map_kernel(oracle, H, W, cin, cout, n):
    rng = np.random.default_rng(H * 100 + W)
    x = oracle.round_bf16(rng.standard_normal((n, H, W, cin)).astype(np.float32))
    w = oracle.round_bf16((rng.standard_normal((cout, 3, 3, cin)) * np.sqrt(2.0 / (cin * 9))).astype(np.float32))
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    xd, wd, bd = _to_dev(x, True), _to_dev(w, True), torch.from_numpy(b).to(DEV)
    assert _kernel_of(cin, cout, n, H, W, (0, 4, 1, 0)).startswith("conv_fast_kernel")
    for units, blocks in ((2, 2), (4, 2 if cout % 128 else 4)):
        assert _kernel_of(cin, cout, n, H, W, (6, units, -1, -1)) == f"conv_map_kernel<{((H * W + 15) // 16 + 3) // 4}, {blocks}>"
    for relu, bias in ((1, bd), (2, bd), (0, None)):
        layer = dict(_layer(cin, cout, 3, 1, 1, True), relu=relu)
        wp = binding.dc_pack_conv_weights(layer, wd)
        out = {}
        for tuning in ((0, 4, 1, 0), (6, 2, -1, -1), (6, 4, -1, -1)):
            for packed in (None, wp):
                print(f"[whole map] {H}x{W} {cin}->{cout} n={n} relu={relu} {tuning} packed={packed is not None}", flush=True)
                binding.dc_conv_tuning(*tuning)
                try:
                    out[tuning, packed is None] = binding.dc_cached_conv_layer(layer, xd, wd, bias, packed=packed)
                finally:
                    binding.dc_conv_tuning()
        base = out[(0, 4, 1, 0), True]
        for key, got in out.items():
            assert torch.equal(got.view(torch.int16), base.view(torch.int16)), key
        if relu == 1:
            for i in range(n):
                assert _rel_err(_to_np(base)[i], oracle.conv_cached(x[i], w, b, 3, 1, 1, True, bf16=True)) <= 2e-2


@pytest.mark.parametrize("H,W,cin,cout,kernels", [
    (13, 13, 384, 384, {16: None, 40: (3, 2), 64: (3, 4), 107: (3, 2), 160: (3, 4)}),
    (13, 13, 512, 1024, {8: None, 16: (3, 2), 34: None, 44: (3, 2)}),
    (14, 14, 512, 512, {28: (4, 2), 40: None, 64: (4, 4), 144: None}),
    (11, 13, 256, 512, {30: (3, 2), 40: None, 64: (3, 4), 160: None}), (12, 12, 384, 384, {64: None})])
def test_where_whole_maps_are_taken(H, W, cin, cout, kernels):
    """The kernel that takes whole maps runs where its rounds of workgroups cost less than the other kernels' (numbers of streams
    on both sides of the line, measured); maps that its tiles save nothing on never take it."""
    for n, want in kernels.items():
        print(f"[whole maps] {H}x{W} {cin}->{cout} n={n}", flush=True)
        name = _kernel_of(cin, cout, n, H, W, (-1, -1, -1, -1))
        assert name == f"conv_map_kernel<{want[0]}, {want[1]}>" if want else not name.startswith("conv_map_kernel"), (n, name)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("pw_tile", [4, 8], indirect=True)
@pytest.mark.parametrize("cin,cout", [(8, 8), (64, 72), (96, 200), (320, 136)])
def test_pointwise_kernel_without_a_bias(cin, cout, pw_tile, bf16):
    """No bias is a bias of zeros, and a bias that is not aligned to a channel tile is read to its end and no further: the last
    channel's value lies before a NaN."""
    g = torch.Generator(DEV)
    g.manual_seed(cin + cout)
    x = torch.randn((3, 13, 11, cin), generator=g, device=DEV)
    w = torch.randn((cout, 1, 1, cin), generator=g, device=DEV) * 0.1
    store = torch.full((cout + 64,), float("nan"), device=DEV)
    store[:cout] = torch.randn(cout, generator=g, device=DEV)
    if bf16:
        x, w = x.bfloat16(), w.bfloat16()
    layer = _layer(cin, cout, 1, 1, 0, False)
    run = lambda bias: binding.dc_cached_conv_layer(layer, x, w, bias)
    none, zero, some = run(None), run(torch.zeros(cout, device=DEV)), run(store[:cout])
    assert torch.equal(none, zero)
    want = x.double().reshape(-1, cin) @ w.double().reshape(cout, cin).T + store[:cout].double()
    got = some.double().reshape(-1, cout)
    # K + 2 roundings to 2^-24 of the terms' absolute sum, and one to the storage type
    bound = (cin + 2) * 2.0 ** -24 * (x.double().abs().reshape(-1, cin) @ w.double().abs().reshape(cout, cin).T + store[:cout].double().abs())
    assert bool(((got - want).abs() <= bound + (2.0 ** -8 if bf16 else 0.0) * want.abs()).all())
