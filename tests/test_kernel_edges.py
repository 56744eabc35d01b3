"""Kernels at the sizes where their dispatch or their tiles change: edges of
tiles, remainders, the smallest and the largest of a range, against the CPU
oracle (or the plain definition) on the same inputs."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eg():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2201_06227_amd import binding
    binding.lib()                      # raises if the HIP library has not been built
    return binding


# Rows in registers (up to 768 and 3072 floats, twice that in bf16), longer rows read twice, odd lengths and 3x3
# kernels through LDS, rows of codes beyond the LDS row gathered.
PER_CHANNEL_SHAPES = [(1, 4), (5, 768), (3, 772), (4, 3072), (6, 3080), (9, 6152), (7, 13), (2, 3077), (3, 8200), (2, 8203),
                      (5, 16, 3, 3), (4, 20, 3, 3), (3, 7, 3, 3), (2, 288, 3, 3), (2, 900, 3, 3), (3, 1000, 3, 3), (2, 5, 2, 2)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_per_channel_snapshot_row_lengths(eg, orc, dtype):
    rng = np.random.default_rng(31)
    ws = [torch.from_numpy(rng.standard_normal(s).astype(np.float32)) for s in PER_CHANNEL_SHAPES]
    if dtype == "bf16":
        ws = [w.to(torch.bfloat16) for w in ws]
    ws[1][2] = 0                                                   # a channel of zeros: scale 1, codes 0
    codes, scales = eg.quantize_weights([w.cuda() for w in ws], per_channel=True)
    for w, q, s in zip(ws, codes, scales):
        wq, sw = orc.quantize_per_channel(w.float().numpy())
        assert np.array_equal(s.cpu().numpy(), sw), w.shape
        got = q.cpu().numpy()
        c = w.shape[1]
        want = np.transpose(wq, (0, 2, 3, 1)) if w.dim() == 4 else wq
        assert np.array_equal(got[..., :c], want), w.shape
        assert not got[..., c:].any(), w.shape


# The metric: one block of samples, two, three, four (with ragged last ones), one workgroup doing the whole score (up to
# 512 features, up to 128 where the rows are filled element by element) and its first neighbour, whole slabs of 16 features
# and ragged ones, rows at 16-, 4- and 2-byte boundaries.  Bar as in the parity tests: fp32 products and sums, quadratic in the difference.
@pytest.mark.parametrize("types", ["f32 f32", "bf16 f32", "f32 bf16", "bf16 bf16"])
@pytest.mark.parametrize("b", [1, 5, 31, 32, 33, 64, 65, 96, 97, 128])
def test_metric_block_and_slab_edges(eg, orc, b, types):
    import synth_inputs as si
    kinds = [torch.bfloat16 if k == "bf16" else torch.float32 for k in types.split()]
    for D in (3, 16, 18, 127, 129, 512, 514, 1024, 1025, 1040, 5003, 16388):
        a_t, a_r = (torch.from_numpy(a).to(k) for a, k in zip(si.noisy_pair(b, D, seed=7 + b + D), kinds))
        want = orc.sp_loss(a_t.float().numpy(), a_r.float().numpy())
        got = eg.plasticity(a_t.cuda(), a_r.cuda()).item()
        assert abs(got - want) <= 1e-4 * abs(want) + 1e-12 * 4.0 / b, (b, D, types, got, want)


# Rows of 2^24 features and more, which are addressed with 64 bits: one, two and three blocks of samples, whole slabs and
# ragged ones, rows at 16-, 8-, 4- and 2-byte boundaries, the last size below the line.  Reference in fp64 on the same values.
@pytest.mark.parametrize("b,D,types", [(3, (1 << 24) - 4112, "f32 f32"), (3, (1 << 24) - 4096, "f32 f32"), (2, (1 << 24) + 1, "f32 f32"),
                                       (5, (1 << 24) + 18, "bf16 f32"), (2, (1 << 24) + 1, "f32 bf16"), (33, 1 << 24, "bf16 bf16"),
                                       (70, (1 << 24) + 16, "f32 f32")])
def test_metric_long_rows(eg, b, D, types):
    kinds = [torch.bfloat16 if k == "bf16" else torch.float32 for k in types.split()]
    g = torch.Generator(device="cuda").manual_seed(b)
    r = torch.randn(b, D, generator=g, device="cuda")
    t = (r + 0.05 * torch.randn(b, D, generator=g, device="cuda")).to(kinds[0])
    r = r.to(kinds[1])
    grams = [torch.zeros(b, b, dtype=torch.float64, device="cuda") for _ in range(2)]
    for k in range(0, D, 1 << 21):
        for gram, a in zip(grams, (t, r)):
            part = a[:, k:k + (1 << 21)].double()                  # as a batch of short products: one long one is slow
            part = torch.nn.functional.pad(part, (0, -part.shape[1] % 256)).reshape(b, 256, -1).permute(1, 0, 2).contiguous()
            gram += torch.bmm(part, part.permute(0, 2, 1).contiguous()).sum(0)
    want = (torch.nn.functional.normalize(grams[0]) - torch.nn.functional.normalize(grams[1])).square().sum().item() / (b * b)
    got = eg.plasticity(t, r).item()
    assert abs(got - want) <= 1e-4 * want, (got, want)


# One row of more than 2^34 features: nothing but the last one is set, so the score is 1 if it is seen and 0 if not.
def test_metric_longest_row(eg):
    D = (1 << 34) + 40
    if torch.cuda.mem_get_info()[0] < 5 * D:
        pytest.skip("needs 80 GB of device memory")
    t, r = (torch.zeros(1, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    t[0, -1] = 1.0
    assert eg.plasticity(t, r).item() == 1.0
    del t, r
    torch.cuda.empty_cache()


# Partials of 38, 79, 64, 65, 128, 129, 256 and 244 chunks: the finaliser requests 4 (up to 64 chunks) or 8 of them
# per thread together.  fp32 partial sums: 1e-4 relative.
@pytest.mark.parametrize("b,D", [(100, 9000), (70, 30000), (40, 8192), (64, 8208), (33, 16384), (64, 16400), (50, 32768), (64, 70001)])
def test_metric_chunk_counts(eg, b, D):
    g = torch.Generator(device="cuda").manual_seed(D)
    r = torch.randn(b, D, generator=g, device="cuda")
    t = r + 0.05 * torch.randn(b, D, generator=g, device="cuda")
    grams = [a.double() @ a.double().t() for a in (t, r)]
    want = (torch.nn.functional.normalize(grams[0]) - torch.nn.functional.normalize(grams[1])).square().sum().item() / (b * b)
    assert abs(eg.plasticity(t, r).item() - want) <= 1e-4 * want
    assert eg.plasticity(r, r).item() == 0.0


# A non-finite activation makes the score NaN, also where the other activation's rows are all zeros (their Gram rows have
# no norm, which takes the other branch of a row's share).
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("b,D", [(5, 40), (32, 4096), (64, 3001), (100, 640)])
def test_metric_non_finite(eg, b, D, value):
    for which in (0, 1):
        for kind in (torch.float32, torch.bfloat16):
            for other in (0.0, 1.0):
                pair = [torch.full((b, D), other, dtype=kind, device="cuda") for _ in range(2)]
                pair[which] = torch.randn(b, D, device="cuda").to(kind)
                pair[which][b // 2, D // 3] = value
                assert np.isnan(eg.plasticity(*pair).item()), (which, kind, other)


# Activations whose Gram rows have norms below the 1e-12 at which a norm is clamped: the score is the squared difference of
# the rows over 1e-24, and must not be lost among the rows' own squares.  fp32 sums of at most 4099 terms: 1e-4 relative.
@pytest.mark.parametrize("b,D", [(1, 16), (4, 16), (32, 100), (33, 64), (64, 4099), (100, 300)])
def test_metric_tiny_activations(eg, orc, b, D):
    rng = np.random.default_rng(b + D)
    size = 2e-7 / np.sqrt(D * b)                                   # row norms of about 5e-14
    a_r = (size * rng.uniform(0.5, 1.0, (b, D))).astype(np.float32)
    a_t = (a_r * (1.0 + 1e-6 * rng.standard_normal((b, D)))).astype(np.float32)
    want = orc.sp_loss(a_t, a_r)
    got = eg.plasticity(torch.from_numpy(a_t).cuda(), torch.from_numpy(a_r).cuda()).item()
    assert want > 0.0 and abs(got - want) <= 1e-4 * want, (got, want)


# A batch of one: both rows normalise to the same single entry, so the score is 0 exactly, whatever the sums round to.
@pytest.mark.parametrize("types", ["f32 f32", "bf16 f32", "bf16 bf16"])
@pytest.mark.parametrize("D", [1, 7, 100, 1000, 5003, 100000])
def test_metric_batch_of_one(eg, D, types):
    kinds = [torch.bfloat16 if k == "bf16" else torch.float32 for k in types.split()]
    for seed in range(8):
        g = torch.Generator().manual_seed(seed)
        r = torch.randn(1, D, generator=g)
        t = r * (1.0 + 0.1 * seed) + 0.01 * torch.randn(1, D, generator=g)
        assert eg.plasticity(t.to(kinds[0]).cuda(), r.to(kinds[1]).cuda()).item() == 0.0, seed


# Every output tile of the int8 GEMM with rows and columns that end inside it (the tile is asked for, so that a case
# cannot come to run on another one), against the CPU oracle: fully connected layers (columns in whole groups of four
# and ragged), with symmetric and affine codes.
LINEAR_TILES = [((128, 32, 64), 1000, 20, 100), ((128, 64, 128), 257, 48, 100), ((128, 64, 64), 49805, 68, 64),
                ((128, 128, 64), 44382, 140, 64), ((128, 128, 128), 49294, 68, 520), ((128, 192, 64), 43978, 132, 512),
                ((256, 128, 64), 49395, 196, 512), ((256, 192, 128), 16240, 580, 2048), ((256, 256, 128), 16426, 652, 2048)]


@pytest.mark.parametrize("mode", ["dynamic", "affine"])
@pytest.mark.parametrize("ragged", [0, 3])
@pytest.mark.parametrize("tile,M,N,K", LINEAR_TILES, ids=["x".join(map(str, t[0])) for t in LINEAR_TILES])
def test_linear_tiles_at_edges(eg, orc, tile, M, N, K, ragged, mode):
    import gpu_common as gc
    import synth_inputs as si
    from oracle import affine_oracle as ao
    from test_affine import _gpu_affine
    N += ragged
    assert eg.gemm_tile(M, N, eg.padded(K)) == tile
    wl = si.make_fc(b=M, k=K, n=N, seed=9)
    wl.biases[0] = np.linspace(-1.0, 1.0, N).astype(np.float32)
    if mode == "affine":
        got, want = _gpu_affine(wl, with_taps=False)[0], ao.ref_forward(wl)["a_ref"]
    else:
        got, want = gc.run_forward(wl, with_taps=False)[0], orc.ref_forward(wl)["a_ref"]
    assert np.array_equal(got.reshape(M, N), want)


# Tiles that come with two stages of whole lines (chosen by price) and with three (by rule).
LINEAR_STAGES = [((64, 64, 128), 3, 700, 200, 520), ((128, 64, 128), 2, 4000, 772, 520), ((128, 64, 128), 3, 3970, 484, 100),
                 ((128, 64, 128), 3, 10500, 260, 1030), ((128, 128, 128), 3, 5990, 484, 1030), ((128, 128, 128), 3, 7990, 484, 1030)]


@pytest.mark.parametrize("mode", ["dynamic", "affine"])
@pytest.mark.parametrize("ragged", [0, 3])
@pytest.mark.parametrize("tile,stages,M,N,K", LINEAR_STAGES, ids=["x".join(map(str, t[0])) + f"_{t[1]}stages_M{t[2]}" for t in LINEAR_STAGES])
def test_linear_stages_at_edges(eg, orc, tile, stages, M, N, K, ragged, mode):
    assert eg.gemm_stages(M, N + ragged, eg.padded(K)) == stages
    test_linear_tiles_at_edges(eg, orc, tile, M, N, K, ragged, mode)


# The same for 3x3 convolutions (whose affine codes look up the class of a border pixel per row of the tile): the block's first layer writes the maximum (dynamic), int8 codes (static scales) or fp32
# for affine codes, its second one adds the skip connection.
CONV_TILES = [((128, 64, 128), 1, 44, 15, 15), ((128, 64, 64), 11, 132, 54, 56), ((128, 128, 128), 12, 68, 64, 65),
              ((128, 128, 64), 16, 68, 64, 65), ((128, 192, 64), 11, 132, 63, 64), ((256, 128, 64), 12, 196, 64, 65)]


@pytest.mark.parametrize("mode", ["dynamic", "static", "affine", "affine ragged"])
@pytest.mark.parametrize("tile,b,c,h,w", CONV_TILES, ids=["x".join(map(str, t[0])) for t in CONV_TILES])
def test_conv_tiles_at_edges(eg, orc, tile, b, c, h, w, mode):
    import gpu_common as gc
    import synth_inputs as si
    from oracle import affine_oracle as ao
    from test_affine import _gpu_affine
    c -= 2 if "ragged" in mode else 0
    assert eg.gemm_tile(b * h * w, c, 9 * eg.padded(c), True) == tile
    wl = si.make_basic_block(b=b, c=c, h=h, w=w, seed=10)
    if "affine" in mode:
        got, want = _gpu_affine(wl, with_taps=False)[0], ao.ref_forward(wl)["a_ref"]
    else:
        scales = np.array([0.03, 0.02], np.float32) if mode == "static" else None
        got, want = gc.run_forward(wl, with_taps=False, act_scales=scales)[0], orc.ref_forward(wl, act_scales=scales)["a_ref"]
    assert np.array_equal(got.reshape(-1, c), gc.nhwc(want))


# (c = 132 and 260: window positions of more than a K step that end inside one.)
CONV_STAGES = [((64, 64, 128), 3, 4, 44, 15, 15), ((64, 64, 128), 3, 3, 132, 15, 17), ((128, 64, 128), 2, 36, 132, 29, 28),
               ((128, 64, 128), 3, 40, 132, 14, 15), ((128, 128, 128), 3, 50, 260, 14, 15)]


@pytest.mark.parametrize("mode", ["dynamic", "static", "affine", "affine ragged"])
@pytest.mark.parametrize("tile,stages,b,c,h,w", CONV_STAGES, ids=["x".join(map(str, t[0])) + f"_{t[1]}stages_b{t[2]}" for t in CONV_STAGES])
def test_conv_stages_at_edges(eg, orc, tile, stages, b, c, h, w, mode):
    assert eg.gemm_stages(b * h * w, c, 9 * eg.padded(c), True) == stages
    test_conv_tiles_at_edges(eg, orc, tile, b, c, h, w, mode)


# float16 layers choose among the same tiles (a K of half as many values has as many bytes): every one of them with rows and
# columns that end inside, layer by layer against fp64 sums of the operands that the run itself recorded (products of float16
# values are exact in fp32; sums of up to 2340 of them, 4e-6 of the largest output).  The observed and the unobserved run agree bit
# for bit (asserted by the helper).
def _check_float16(wl, eg, conv):
    from test_float_ref import _gpu_float_forward
    a_ref, taps, _ref, _ws = _gpu_float_forward(wl, "f16")
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda().double()  # noqa: E731
    for i, t in enumerate(taps):
        x, w = dev(t["x"]), dev(wl.weights[i].astype(np.float16).astype(np.float32))
        if conv:
            b, c, h, wd = wl.x.shape
            p = torch.nn.functional.pad(x.reshape(b, h, wd, c), (0, 0, 1, 1, 1, 1))
            y = sum(p[:, kh:kh + h, kw:kw + wd].reshape(-1, c) @ w[:, :, kh, kw].t().contiguous() for kh in range(3) for kw in range(3))
        else:
            y = x @ w.t().contiguous()
        y += dev(wl.biases[i])
        if conv and i == 1:
            y += dev(taps[0]["x"])                                # the skip connection
        y = y.clamp_min(0.0).float().cpu().numpy()
        tol = 4e-6 * np.abs(y).max()
        assert np.abs(t["y"] - y).max() <= tol, i
    assert np.abs(a_ref.reshape(y.shape) - y).max() <= tol


@pytest.mark.parametrize("ragged", [0, 3])
@pytest.mark.parametrize("tile,stages,M,N,K", [(t, None, M, N, K) for t, M, N, K in LINEAR_TILES] + LINEAR_STAGES)
def test_float16_linear_tiles_at_edges(eg, tile, stages, M, N, K, ragged):
    import synth_inputs as si
    N, K = N + ragged, K // 2
    k_bytes = eg.op_row_bytes(K, eg.REF_F16)
    assert eg.gemm_tile(M, N, k_bytes) == tile and stages in (None, eg.gemm_stages(M, N, k_bytes))
    wl = si.make_fc(b=M, k=K, n=N, seed=9)
    wl.biases[0] = np.linspace(-1.0, 1.0, N).astype(np.float32)
    _check_float16(wl, eg, False)


@pytest.mark.parametrize("ragged", [0, 3])
@pytest.mark.parametrize("tile,stages,b,c,h,w", [(t, None, *d) for t, *d in CONV_TILES] + CONV_STAGES)
def test_float16_conv_tiles_at_edges(eg, tile, stages, b, c, h, w, ragged):
    import synth_inputs as si
    c -= ragged                                                   # (twice the bytes of K keep all of these tiles)
    k_bytes = 9 * eg.op_row_bytes(c, eg.REF_F16)
    assert eg.gemm_tile(b * h * w, c, k_bytes, True) == tile and stages in (None, eg.gemm_stages(b * h * w, c, k_bytes, True))
    _check_float16(si.make_basic_block(b=b, c=c, h=h, w=w, seed=10), eg, True)


# ... and for the layers of an encoder (no activation, with and without the maximum) at a ragged number of tokens.
def test_encoder_tiles_at_edges(eg, orc):
    import gpu_common as gc
    import synth_inputs as si
    M = 24 * 197
    assert [eg.gemm_tile(M, n, k)[:2] for n, k in ((2304, 768), (3072, 768), (768, 3072))] == [(128, 192), (256, 128), (128, 64)]
    wl = si.make_bert(b=24, s=197, seed=11, train_act_dtype="f32")
    got = gc.run_forward(wl, with_taps=False)[0]
    gc.assert_within_ulp(got, orc.ref_forward(wl)["a_ref"][0], 1, "encoder layer")


# ... and the tiles of eight waves without an activation, in an encoder layer of 16 x 257 tokens (sums of up to 4096 products).
def test_float16_encoder_tiles_at_edges(eg):
    import synth_inputs as si
    from test_float_ref import _gpu_float_forward
    M, H = 16 * 257, 1024
    assert [eg.gemm_tile(M, n, 2 * k) for n, k in ((3 * H, H), (H, H), (4 * H, H))] == [(256, 256, 128), (128, 64, 128), (256, 192, 128)]
    wl = si.make_bert(b=16, s=257, hidden=H, heads=16, ffn=4 * H, seed=13, train_act_dtype="f32")
    _a, taps, _ref, _ws = _gpu_float_forward(wl, "f16")          # (the unobserved run agrees bit for bit)
    for i, t in enumerate(taps):
        x, w = (torch.from_numpy(a).cuda().double() for a in (t["x"], wl.weights[i].astype(np.float16).astype(np.float32)))
        y = x @ w.t().contiguous()
        tol = 6e-6 * y.abs().max().item()
        assert np.abs(t["acc"] - y.float().cpu().numpy()).max() <= tol, i
        if wl.biases[i] is not None:
            y += torch.from_numpy(wl.biases[i]).cuda().double()
        if i == 2:
            y = torch.nn.functional.gelu(y)
        assert np.abs(t["y"] - y.float().cpu().numpy()).max() <= tol, i


# GEMM epilogue of small modules: rows and columns that end inside, at and just past a tile or a group of four columns, with
# and without a residual, for the dynamic, static, per-channel and affine paths.  The parity tests hold observed runs to the
# oracle; here the observed run, which takes the general form of the epilogue, is the reference for the straight-line one.
# (All of these run on 64x64 or 128x64 tiles; the others are above.)
@pytest.mark.parametrize("mode", ["dynamic", "static", "affine", "per_channel"])
@pytest.mark.parametrize("b,c,h,w", [(1, 36, 3, 5), (2, 64, 8, 8), (3, 33, 11, 12), (5, 68, 16, 13), (4, 130, 16, 16), (9, 64, 15, 17)])
def test_conv_epilogue_edges(eg, b, c, h, w, mode):
    import gpu_common as gc
    import synth_inputs as si
    for wl in (si.make_basic_block(b=b, c=c, h=h, w=w, seed=5), si.make_bottleneck(b=b, c_in=2 * c, c_mid=c, h=h, w=w, seed=6)):
        W = [gc.to_dev(t) for t in wl.weights]
        B = [gc.to_dev(t) for t in wl.biases]
        scales = torch.full((len(W),), 0.03, device="cuda") if mode == "static" else None
        ref = eg.make_reference(wl.kind, wl.dims, W, B, scales, per_channel=mode == "per_channel",
                                act_scheme=eg.ACT_AFFINE if mode == "affine" else eg.ACT_SYMMETRIC)
        x = gc.to_dev(wl.x)
        ws = eg.workspace(eg.workspace_bytes(ref.desc))
        plain, seen = (torch.full((gc.a_ref_numel(wl) + 64,), 7.0, device="cuda") for _ in range(2))
        taps, _bufs, _keep = eg.make_taps(ref, gc.tap_shapes(wl))
        eg.ref_forward(ref, x, seen, ws, taps)
        eg.ref_forward(ref, x, plain, ws)
        assert torch.equal(plain, seen), (wl.name, mode)
        assert bool((plain[-64:] == 7.0).all()), "written past the end"


# Extrema of a tensor: at most four 16-byte units per thread, one more, ragged ends, the extrema among the last values.
@pytest.mark.parametrize("n", [1, 3, 5, 1023, 4100, (1 << 22) - 1, 1 << 22, (1 << 22) + 4, (1 << 22) + 4099])
def test_affine_extrema(eg, n):
    from oracle import affine_oracle as ao
    rng = np.random.default_rng(n % 89)
    for at in (0, n // 2, n - 1):
        x = rng.uniform(-1.0, 1.0, n).astype(np.float32)
        x[at], x[(at + 7) % n] = 5.0, -3.0
        q, s, zp = eg.quantize_affine(torch.from_numpy(x).cuda())
        wq, ws, wzp = ao.quantize(x)
        assert s.item() == ws and zp.item() == wzp and np.array_equal(q.cpu().numpy(), wq), at


# Operands made of whole 16-byte units (rows of 4 k values, planes of 4 k pixels) and of everything else; channel counts
# with and without pad channels.
@pytest.mark.parametrize("b,c,h,w", [(1, 36, 3, 5), (2, 64, 8, 8), (3, 33, 4, 3), (2, 17, 7, 7), (5, 68, 2, 2), (300, 20, 1, 1)])
def test_operand_layouts(eg, b, c, h, w):
    import gpu_common as gc
    import synth_inputs as si
    from oracle import affine_oracle as ao
    from test_affine import _gpu_affine
    from test_float_ref import _gpu_float_forward
    wl = si.make_basic_block(b=b, c=c, h=h, w=w, seed=12)
    q, s, zp = ao.quantize(wl.x)
    _, taps, _, _ = _gpu_affine(wl)
    got = taps[0]["x_q"].astype(np.int16) + 128
    assert taps[0]["x_scale"][0] == s and taps[0]["x_zp"][0] == zp
    assert np.array_equal(got[:, :c], gc.nhwc(q).reshape(-1, c)) and not taps[0]["x_q"][:, c:].any()
    for precision, kind in (("f16", np.float16), ("f32", np.float32)):
        _, taps, _, _ = _gpu_float_forward(wl, precision)
        assert np.array_equal(taps[0]["x"], gc.nhwc(wl.x.astype(kind).astype(np.float32)).reshape(-1, c)), precision


# The operand of the second feed-forward layer written by the GELU's own pass (unobserved runs) against the plain
# sequence (observed runs): rows of whole and of ragged units, pre-activations from the table's lower end to beyond its
# upper one and many near zero, where most values take the fp64 form.
@pytest.mark.parametrize("precision", ["f16", "f32"])
@pytest.mark.parametrize("ffn,spread", [(64, 1.0), (68, 12.0), (97, 3.0), (328, 0.01), (1, 1.0)])
def test_gelu_operand(eg, precision, ffn, spread):
    import gpu_common as gc
    import synth_inputs as si
    wl = si.make_bert(b=3, s=19, hidden=64, heads=2, ffn=ffn, n_layers=2, seed=21, train_act_dtype="f32")
    W = [gc.to_dev(w * (spread if i % 4 == 2 else 1.0)) for i, w in enumerate(wl.weights)]
    B = [None if t is None else gc.to_dev(t) for t in wl.biases]
    ref = eg.make_float_reference(wl.kind, wl.dims, W, B, {"f16": eg.REF_F16, "f32": eg.REF_F32}[precision])
    ws = eg.workspace(eg.workspace_bytes(ref.desc))
    x = gc.to_dev(wl.x)
    plain, seen = (torch.full((gc.a_ref_numel(wl),), 7.0, device="cuda") for _ in range(2))
    shapes = gc.tap_shapes(wl)
    for t in shapes:
        t["kp"] = t["kp"] * 4                              # room for rows of either precision
    taps, _bufs, _keep = eg.make_taps(ref, shapes)
    eg.ref_forward(ref, x, seen, ws, taps)
    eg.ref_forward(ref, x, plain, ws)
    assert torch.equal(plain, seen)


# Attention and the layer norms write the float16 operands of unobserved layers themselves: rows of one and of many 16-byte units,
# past the width of the vector layer norm, with parameters off its alignment, and rows with pad columns (which are cast).
@pytest.mark.parametrize("hidden,heads,off", [(8, 1, 0), (72, 3, 0), (72, 3, 1), (264, 11, 0), (768, 12, 0), (1032, 24, 0), (68, 2, 0)])
def test_float16_operands_of_a_layer(eg, hidden, heads, off):
    import gpu_common as gc
    from paper_2201_06227_amd.binding import Norm
    import synth_inputs as si
    wl = si.make_bert(b=3, s=67, hidden=hidden, heads=heads, ffn=2 * hidden + 4, n_layers=3, seed=23, train_act_dtype="f32")
    W, B = [gc.to_dev(w) for w in wl.weights], [None if t is None else gc.to_dev(t) for t in wl.biases]
    gen = torch.Generator(device="cuda").manual_seed(hidden)
    gamma, beta = (torch.randn(hidden + 4, device="cuda", generator=gen)[off:off + hidden] for _ in range(2))
    ref = eg.make_float_reference(wl.kind, wl.dims, W, B, eg.REF_F16)
    norms = (Norm * 6)(*[Norm(gamma.data_ptr(), beta.data_ptr())] * 6)
    ref.qweights.n_norm, ref.qweights.norm = 6, norms
    ws = eg.workspace(eg.workspace_bytes(ref.desc))
    x = gc.to_dev(wl.x)
    plain, seen = (torch.full((gc.a_ref_numel(wl),), 7.0, device="cuda") for _ in range(2))
    shapes = gc.tap_shapes(wl)
    for t in shapes:
        t["kp"] = t["kp"] * 4
    taps, _bufs, _keep = eg.make_taps(ref, shapes)
    eg.ref_forward(ref, x, seen, ws, taps)
    eg.ref_forward(ref, x, plain, ws)
    assert torch.equal(plain, seen)


# The work of a launch is dealt in pieces, an eighth of them to each XCD: fewer pieces than XCDs, a multiple of eight and its
# neighbours, pieces of one and of several units per thread.  The largest value sits in the last place, then in the first.
@pytest.mark.parametrize("rows,cols", [(1, 16), (3, 16), (7, 4096), (8, 4096), (9, 4096), (255, 16), (257, 16), (17, 4112), (1031, 48),
                                       (5, 30), (700, 20), (4099, 16384)])
def test_codes_of_rows_in_pieces(eg, rows, cols):
    x = torch.randn(rows, cols, device="cuda", generator=torch.Generator(device="cuda").manual_seed(rows + cols)).clamp_(-4, 4)
    for at in (-1, 0):
        y = x.clone()
        y.view(-1)[at] = 5.0
        q, scale = eg.quantize_rows(y)
        assert scale.item() == np.float32(5.0 / 127.0)
        want = torch.clamp(torch.round(y * torch.tensor(127.0 / 5.0, dtype=torch.float64).float().item()), -127, 127).to(torch.int8)
        assert torch.equal(q[:, :cols], want)
        assert not q[:, cols:].any()


# The first feed-forward layer that writes the codes of its GELU itself (two passes over its sums), on each of its tiles with rows
# and columns that end inside: the observed run keeps the fp32 tensor and the row quantiser, A_R has to be the same bit for bit.
# spread: pre-activations so small that the largest |gelu| is a negative value's, ordinary ones, some beyond the table's ends.
GELU_TILES = [((64, 64), 2, 37, 200), ((128, 64), 20, 65, 1540), ((128, 192), 32, 60, 2308), ((128, 128), 40, 65, 2308),
              ((256, 192), 40, 65, 3083), ((256, 256), 100, 70, 2056)]


def _gelu_tile(M, N, cu):
    cost = {}
    for bm, bn, resident, penalty in ((256, 256, 1, 1.0), (256, 192, 1, 1.0), (128, 192, 1, 1.07), (128, 128, 2, 1.07), (128, 64, 2, 1.07),
                                      (64, 64, 2, 1.07)):
        tiles = -(-M // bm) * -(-N // bn)
        cost[(bm, bn)] = -(-tiles // (cu * resident)) * (bm * bn * resident + 14336) * penalty
    return min(cost, key=cost.get)


def _same_observed_and_not(eg, wl, per_channel=False, biases=True, prepare=lambda ref: None, status=0):
    import gpu_common as gc
    ref = eg.make_reference(wl.kind, wl.dims, [gc.to_dev(w) for w in wl.weights], [gc.to_dev(b) if biases else None for b in wl.biases],
                            per_channel=per_channel)
    prepare(ref)
    x, ws = gc.to_dev(wl.x), eg.workspace(eg.workspace_bytes(ref.desc), "cuda")
    got = [torch.empty(gc.a_ref_numel(wl), device="cuda") for _ in range(2)]
    taps, bufs, _keep = eg.make_taps(ref, gc.tap_shapes(wl), "cuda")
    eg.ref_forward(ref, x, got[0], ws, taps)
    eg.ref_forward(ref, x, got[1], ws)
    assert eg.check(ws) == status
    assert torch.equal(got[0], got[1])
    return bufs


@pytest.mark.parametrize("spread,per_channel,biases", [(1.0, False, False), (0.03, False, False), (12.0, False, True), (0.03, True, True)])
@pytest.mark.parametrize("tile,b,s,ffn", GELU_TILES, ids=["x".join(map(str, t[0])) for t in GELU_TILES])
def test_gelu_codes_from_the_gemm(eg, tile, b, s, ffn, spread, per_channel, biases):
    import synth_inputs as si
    assert _gelu_tile(b * s, ffn, torch.cuda.get_device_properties(0).multi_processor_count) == tile
    wl = si.make_bert(b=b, s=s, hidden=68, heads=2, ffn=ffn, seed=17, train_act_dtype="f32")
    wl.weights[2] *= np.float32(spread)
    wl.biases[2] = np.linspace(-0.3, 0.2 * spread, ffn).astype(np.float32)
    bufs = _same_observed_and_not(eg, wl, per_channel, biases)
    top = bufs[2]["y"].max().item()                                # of gelu(v): 0.35 at the shortcut's line
    assert (top < 0.3) == (spread < 1.0) and (top > 9.0) == (spread > 1.0), top


# Values that all sit on the border of two codes: a wave's list overflows and it takes its sums through the cubic pieces.  Equal
# tokens have equal sums, which the biases lift to the border (largest value 3, code 60.5).
@pytest.mark.parametrize("b,s,ffn", [(3, 33, 100), (40, 65, 3083)])
def test_gelu_codes_on_the_border(eg, b, s, ffn):
    import math
    import synth_inputs as si
    wl = si.make_bert(b=b, s=s, hidden=64, heads=2, ffn=ffn, seed=19, train_act_dtype="f32")
    wl.x[:] = wl.x[:1, :1]
    bufs = _same_observed_and_not(eg, wl, biases=False)
    acc = bufs[2]["acc"][0].cpu().numpy().astype(np.float64)
    scale = np.float64(np.float32(bufs[2]["x_scale"].item()) * np.float32(np.abs(wl.weights[2]).max() / np.float64(127.0)))
    gelu = lambda v: 0.5 * v * (1.0 + math.erf(v / math.sqrt(2.0)))  # noqa: E731
    lo, hi = 0.0, 3.0
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if gelu(mid) / gelu(3.0) * 127.0 < 60.5 else (lo, mid)
    v = np.full(ffn, lo)
    v[0] = 3.0
    wl.biases[2] = (v - acc * scale).astype(np.float32)
    bufs = _same_observed_and_not(eg, wl)
    codes = bufs[3]["x_q"][:, 1:ffn]
    assert set(torch.unique(codes).tolist()) <= {60, 61}


# Images whose planes are no whole 16-byte units, through LDS by groups of 64, 32 and 16 channels with all their pixels: the borders
# of the groups' rule, pad channels, planes shorter than a unit, the longest, and the sizes that stay with the tile of 64 pixels.
@pytest.mark.parametrize("n,c,h,w", [(1, 4, 1, 2), (2, 20, 1, 3), (3, 64, 7, 7), (2, 68, 7, 9), (2, 132, 5, 13), (1, 36, 1, 127), (2, 40, 3, 43),
                                     (1, 20, 31, 33), (1, 20, 25, 41), (2, 33, 7, 7), (50, 260, 7, 7)])
@pytest.mark.parametrize("static", [False, True])
def test_odd_planes(eg, n, c, h, w, static):
    x = torch.randn(n, c, h, w, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n * c + h)).clamp_(-4, 4)
    x.view(-1)[-1] = -5.0
    q, scale = eg.quantize_nchw(x, torch.tensor([5.0 / 127.0], device="cuda") if static else None)
    inv = torch.tensor(1.0 / np.float64(np.float32(5.0 / 127.0)) if static else 127.0 / 5.0, dtype=torch.float64).float().item()
    want = torch.clamp(torch.round(x * inv), -127, 127).to(torch.int8).permute(0, 2, 3, 1)
    assert scale.item() == np.float32(5.0 / 127.0)
    assert torch.equal(q[..., :c], want)
    assert not q[..., c:].any()


# A small FC mini-batch beside a snapshot of one launch and of two, per tensor and per channel: the same as the two calls.
@pytest.mark.parametrize("b,k,n,per_channel", [(5, 40, 30, False), (32, 512, 512, False), (32, 512, 512, True), (7, 100, 700, False), (64, 250, 66, False)])
def test_fc_refresh_is_the_two_calls(eg, b, k, n, per_channel):
    from paper_2201_06227_amd.evaluator import PlasticityEvaluator
    gen = torch.Generator(device="cuda").manual_seed(b + k)
    for dt in (torch.float32, torch.bfloat16):
        x, wt = torch.randn(b, k, device="cuda", generator=gen).to(dt), torch.randn(n, k, device="cuda", generator=gen) * k ** -0.5
        a_t = [torch.relu(x.float() @ (wt * 1.01).t())]
        ev = PlasticityEvaluator(eg.FC_RELU, dict(batch=b, c_in=k, c_out=n), [wt], [None], per_channel=per_channel)
        one = ev.step(x, a_t).clone()
        codes, scales = ev.w_q[0].clone(), ev.scales[0].clone()
        ev.w_q[0].zero_(); ev.scales[0].zero_()
        two = ev.step_two_calls(x, a_t)
        assert torch.equal(one, two) and torch.equal(codes, ev.w_q[0]) and torch.equal(scales, ev.scales[0])
        assert eg.check(ev.ws) == eg.OK


# Pre-activations that are no numbers: units whose bias is -infinity (masked out) or a NaN with its sign set, neither of which the
# maximum tracks.  Their code is 0 where the largest value sets the scale; below the shortcut the fp64 maximum takes them in and no
# scale is left (1, every code 0).  Infinity and NaN leave no scale either, and the run is flagged.
@pytest.mark.parametrize("bits", [0xff800000, 0xffc00000, 0x7f800000, 0x7fc00000], ids=["-inf", "-nan", "inf", "nan"])
@pytest.mark.parametrize("spread", [1.0, 0.03])
@pytest.mark.parametrize("b,s,ffn", [(2, 37, 200), (100, 70, 2056)])
def test_gelu_codes_of_masked_units(eg, b, s, ffn, spread, bits):
    import synth_inputs as si
    wl = si.make_bert(b=b, s=s, hidden=68, heads=2, ffn=ffn, seed=29, train_act_dtype="f32")
    wl.weights[2] *= np.float32(spread)
    masked = [0, 5, 37, ffn // 2, ffn - 1]
    wl.biases[2] = np.linspace(-0.3, 0.2 * spread, ffn).astype(np.float32)
    wl.biases[2][masked] = np.array([bits], np.uint32).view(np.float32)
    bufs = _same_observed_and_not(eg, wl, status=eg.OK if bits >> 31 else eg.ERR_NONFINITE)
    codes = bufs[3]["x_q"]
    if bits != 0x7f800000:
        assert not codes[:, masked].any()
    codes[:, masked] = 0
    scaled = spread == 1.0 and bits >> 31 == 1
    assert (bufs[3]["x_scale"].item() == 1.0) != scaled and bool(codes.any()) == scaled


# Pad columns of the codes are zero, however small the tensor's largest value: the next layer's weights get codes in their pad
# columns here, which any other code would multiply.
@pytest.mark.parametrize("spread", [1.0, 1e-3, 1e-4, 1e-5])
@pytest.mark.parametrize("b,s,ffn", [(2, 37, 200), (100, 70, 2056)])
def test_gelu_codes_leave_the_pad_zero(eg, b, s, ffn, spread):
    import gpu_common as gc
    import synth_inputs as si
    wl = si.make_bert(b=b, s=s, hidden=68, heads=2, ffn=ffn, seed=31, train_act_dtype="f32")
    wl.weights[2] *= np.float32(spread)

    def mark(ref):
        assert ref.w_q[3].shape[1] == eg.padded(ffn) > ffn
        ref.w_q[3][:, ffn:] = 127
    bufs = _same_observed_and_not(eg, wl, prepare=mark)
    assert not bufs[3]["x_q"][:, ffn:].any()


# Small pre-activations, for which the straight lines leave more and more codes open, then the cubic pieces, at last all of them: the
# same codes on every tile, with one scale and with one per column and a bias, and a pass takes no more than twice what one of
# ordinary values does (with the fp32 tensor and the row quantiser it took up to 1.4 times as long; waves that worked out again
# what their lists could not hold, 40 times).
SMALL_SPREADS = (1.0, 1e-2, 5e-3, 2e-3, 1e-3, 1e-4, 1e-6, 1e-20)


@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("tile,b,s,ffn", GELU_TILES, ids=["x".join(map(str, t[0])) for t in GELU_TILES])
def test_gelu_codes_of_small_values(eg, tile, b, s, ffn, per_channel):
    import synth_inputs as si
    wl = si.make_bert(b=b, s=s, hidden=68, heads=2, ffn=ffn, seed=37, train_act_dtype="f32")
    plain = wl.weights[2].copy()
    for spread in SMALL_SPREADS[1:]:
        wl.weights[2] = plain * np.float32(spread)
        wl.biases[2] = np.linspace(-0.5, 0.5, ffn).astype(np.float32) * np.float32(spread)
        bufs = _same_observed_and_not(eg, wl, per_channel, biases=per_channel)
        assert bufs[3]["x_q"].abs().max().item() == 127


def test_gelu_codes_of_small_values_take_no_longer(eg):
    import gpu_common as gc
    import synth_inputs as si
    wl = si.make_bert(b=64, s=128, seed=37, train_act_dtype="f32")
    W = [gc.to_dev(w) for w in wl.weights]
    x, out = gc.to_dev(wl.x), torch.empty(gc.a_ref_numel(wl), device="cuda")
    times = {}
    for spread in SMALL_SPREADS:
        ref = eg.make_reference(wl.kind, wl.dims, [W[0], W[1], W[2] * spread, W[3]], [None] * 4)
        ws = eg.workspace(eg.workspace_bytes(ref.desc), "cuda")
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        times[spread] = float("inf")
        for _ in range(5):
            ev[0].record()
            eg.ref_forward(ref, x, out, ws)
            ev[1].record()
            ev[1].synchronize()
            times[spread] = min(times[spread], ev[0].elapsed_time(ev[1]))
    assert max(times.values()) < 2.0 * times[1.0], times


# The longest rows whose sums are made twice, and the next longer ones, which are not.
@pytest.mark.parametrize("hidden,heads", [(1008, 16), (1024, 16), (1040, 20)])
@pytest.mark.parametrize("b,s,ffn", [(3, 45, 300), (40, 65, 3083)])
def test_gelu_codes_of_the_longest_rows(eg, b, s, ffn, hidden, heads):
    import synth_inputs as si
    _same_observed_and_not(eg, si.make_bert(b=b, s=s, hidden=hidden, heads=heads, ffn=ffn, seed=41, train_act_dtype="f32"))


# Layers whose padded output is too wide for the GEMM that writes the codes, and the widest that is not.
@pytest.mark.parametrize("ffn", [4194288, 4194289, 4194300])
def test_gelu_codes_of_the_widest_layers(eg, ffn):
    import gpu_common as gc
    import synth_inputs as si
    gen = torch.Generator(device="cuda").manual_seed(ffn)
    W = [torch.randn(o, i, device="cuda", generator=gen) * (2.0 / (o + i)) ** 0.5 for o, i in ((48, 16), (16, 16), (ffn, 16), (16, ffn))]
    W[2] *= 500.0
    dims = dict(batch=1, seq=3, hidden=16, heads=1, ffn=ffn, n_layers=1, ln_eps=1e-12)
    ref = eg.make_reference(si.KIND_BERT_LAYER, dims, W, [None] * 4)
    x, ws = torch.randn(1, 3, 16, device="cuda", generator=gen), eg.workspace(eg.workspace_bytes(ref.desc), "cuda")
    plain, seen = (torch.empty(48, device="cuda") for _ in range(2))
    shapes = [dict(M=3, kp=eg.padded(k), N=n) for k, n in ((16, 48), (16, 16), (16, ffn), (ffn, 16))]
    taps, _bufs, _keep = eg.make_taps(ref, shapes, "cuda")
    eg.ref_forward(ref, x, seen, ws, taps)
    eg.ref_forward(ref, x, plain, ws)
    assert eg.check(ws) == eg.OK
    assert torch.equal(plain, seen)
