"""Affine (asymmetric) uint8 activations (Section 5 of the paper: the framework's quantisation, whose
default activation code has a zero point): pins of the CPU oracle, then the library against the oracle
through the C-ABI."""
from fractions import Fraction

import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import affine_oracle as ao
from oracle import oracle as orc


# ----------------------------------------------------------------------------- oracle pins

def test_worked_example():
    # extrema -1 and 3: scale = 4/255, lo/scale = -63.75 -> zero point 64; 3 * 63.75 = 191.25 -> 191 + 64 = 255
    x = np.array([-1.0, 0.0, 0.5, 3.0], np.float32)
    q, s, zp = ao.quantize(x)
    assert s == np.float32(np.float32(4.0) / np.float32(255.0)) and zp == 64
    assert q.tolist() == [0, 64, 96, 255]                         # 0.5 * 63.75 = 31.875 -> 32
    assert ao.dequantize(q, s, zp)[1] == 0.0                       # zero is a code
    # all values positive: the range still starts at zero, zero point 0
    q, s, zp = ao.quantize(np.array([2.0, 5.0], np.float32))
    assert zp == 0 and s == np.float32(np.float32(5.0) / np.float32(255.0)) and q.tolist() == [102, 255]
    # all values negative: zero point 255
    q, s, zp = ao.quantize(np.array([-2.0, -5.0], np.float32))
    assert zp == 255 and q.tolist() == [153, 0]
    # a tensor of zeros: the smallest scale, zero point 0, codes 0
    q, s, zp = ao.quantize(np.zeros(5, np.float32))
    assert s == np.float32(2.0 ** -23) and zp == 0 and not q.any()


@pytest.mark.parametrize("seed", range(6))
def test_against_the_frameworks_observer_and_quantiser(seed):
    """The reading is the framework's min/max observer and per-tensor quantiser: same scale, same zero point,
    same codes (another implementation of the same float32 operations)."""
    from torch.ao.quantization.observer import MinMaxObserver
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal(20000) * rng.uniform(0.01, 30) + rng.uniform(-3, 3)).astype(np.float32)
    if seed == 4:
        x = np.abs(x)
    if seed == 5:
        x = -np.abs(x)
    q, s, zp = ao.quantize(x)
    obs = MinMaxObserver(dtype=torch.quint8, qscheme=torch.per_tensor_affine, reduce_range=False)
    obs(torch.from_numpy(x))
    ts, tz = obs.calculate_qparams()
    assert np.float32(ts.item()) == s and int(tz.item()) == zp
    tq = torch.quantize_per_tensor(torch.from_numpy(x), float(s), zp, torch.quint8).int_repr().numpy()
    assert np.array_equal(tq, q)


def test_round_trip_and_monotonicity():
    rng = np.random.default_rng(11)
    x = np.sort((rng.standard_normal(5000) * 2 - 0.7).astype(np.float32))
    q, s, zp = ao.quantize(x)
    assert (np.diff(q.astype(np.int32)) >= 0).all()                # codes are monotone in x
    assert q.min() == 0 and q.max() == 255                         # both ends of the range are used
    err = np.abs(ao.dequantize(q, s, zp).astype(np.float64) - x)
    assert err.max() <= 0.5 * float(s) * (1 + 1e-5) + 1e-7         # half a step inside the range


def test_linear_against_exact_rational_arithmetic():
    """acc = sum (q - zp) w exactly; y = one fma of (float) acc with the float32 product of the scales."""
    rng = np.random.default_rng(12)
    x = rng.standard_normal((3, 7)).astype(np.float32) + 0.4
    w = rng.standard_normal((4, 7)).astype(np.float32)
    b = rng.standard_normal(4).astype(np.float32)
    wq, sw = orc.quantize(w)
    taps = {}
    y = ao.linear(x, wq, sw, b, ao.ACT_NONE, taps, "")
    q, s, zp = ao.quantize(x)
    for m in range(3):
        for n in range(4):
            acc = sum((int(q[m, k]) - zp) * int(wq[n, k]) for k in range(7))
            assert taps["acc"][m, n] == acc
            exact = Fraction(acc) * Fraction(float(np.float32(s * sw))) + Fraction(float(b[n]))
            want = np.float32(float(exact))                         # the fma rounds once
            assert y[m, n] == want
    # the centred codes times the scale reproduce x to half a step, so y is close to the fp32 layer
    assert np.abs(y - (x @ w.T + b)).max() <= 0.5 * float(s) * np.abs(w).sum(axis=1).max() + 0.5 * float(sw) * np.abs(x).sum(axis=1).max() + 1e-3


def test_padding_is_the_real_value_zero():
    """A 3x3 window over the image border sees centred code 0 there: with weights of ones the accumulator of a
    corner pixel is the sum of the four centred codes inside the image."""
    x = (np.arange(16, dtype=np.float32).reshape(1, 1, 4, 4) - 5.0)
    q, s, zp = ao.quantize(x)
    w = np.ones((1, 1, 3, 3), np.float32)
    wq, sw = orc.quantize(w)
    taps = {}
    ao._conv(q, s, zp, wq, sw, None, 1, ao.ACT_NONE, None, taps, "")
    c = q.astype(np.int32) - zp
    assert zp != 0 and zp != 128
    assert taps["acc"][0, 0, 0, 0] == 127 * (c[0, 0, 0, 0] + c[0, 0, 0, 1] + c[0, 0, 1, 0] + c[0, 0, 1, 1])
    assert taps["acc"][0, 0, 1, 1] == 127 * c[0, 0, :3, :3].sum()


SMALL = [("fc", lambda: si.make_fc(b=5, k=100, n=7, seed=41)),
         ("basic", lambda: si.make_basic_block(b=2, c=20, h=9, w=11, seed=42)),
         ("bottleneck", lambda: si.make_bottleneck(b=2, c_in=24, c_mid=12, h=6, w=5, seed=43)),
         ("bert", lambda: si.make_bert(b=2, s=9, hidden=48, heads=3, ffn=80, n_layers=2, seed=44, train_act_dtype="f32"))]


@pytest.mark.parametrize("name,make", SMALL, ids=[s[0] for s in SMALL])
def test_affine_reference_tracks_the_fp32_model(name, make):
    """End to end the affine reference stays as close to the fp32 module as the symmetric one does (the
    plasticity of identical weights is small), and is not the same computation as the symmetric one."""
    wl = make()
    a = ao.ref_forward(wl)["a_ref"]
    b_ = orc.ref_forward(wl)["a_ref"]
    a = a[-1] if isinstance(a, list) else a
    b_ = b_[-1] if isinstance(b_, list) else b_
    assert a.shape == b_.shape and not np.array_equal(a, b_)
    assert np.abs(a - b_).max() <= 0.2 * np.abs(b_).max()


# ----------------------------------------------------------------------------- GPU parity (through the C-ABI)
# Codes, scales, zero points and accumulators are integers or single IEEE operations: equal bit for bit.  Outputs of
# the FC / convolution modules are one fma of those: equal.  In the encoder layers the fp32 glue (attention, layer
# norm, GELU) is evaluated in fp64 on both sides and rounded once: at most one unit in the last place.

def _gpu_affine(wl, with_taps=True):
    from paper_2201_06227_amd import binding as eg
    import tests.gpu_common as gc
    W = [gc.to_dev(w) for w in wl.weights]
    B = [None if b is None else gc.to_dev(b) for b in wl.biases]
    ref = eg.make_reference(wl.kind, wl.dims, W, B, act_scheme=eg.ACT_AFFINE)
    a_ref = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    taps = bufs = None
    if with_taps:
        taps, bufs, _keep = eg.make_taps(ref, gc.tap_shapes(wl), gc.DEV)
    eg.ref_forward(ref, gc.to_dev(wl.x), a_ref, ws, taps)
    torch.cuda.synchronize()
    assert eg.check(ws) == eg.OK
    np_taps = [{k: v.cpu().numpy() for k, v in b.items()} for b in bufs] if with_taps else None
    return a_ref.cpu().numpy(), np_taps, ref, ws


@pytest.mark.gpu
@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 4096, 4097, 100003, 1 << 20])
def test_quantize_affine_bit_exact(n):
    from paper_2201_06227_amd import binding as eg
    import tests.gpu_common as gc
    rng = np.random.default_rng(500 + n % 97)
    for variant in range(4):
        x = (rng.standard_normal(n) * 3 + 0.8).astype(np.float32)
        if variant == 1:
            x = np.abs(x)
        if variant == 2:
            x = -np.abs(x) - 1
        if variant == 3:
            x[:] = 0
        q, s, zp = eg.quantize_affine(gc.to_dev(x))
        torch.cuda.synchronize()
        wq, wscale, wzp = ao.quantize(x)
        assert s.item() == wscale and zp.item() == wzp, (n, variant)
        assert np.array_equal(q.cpu().numpy(), wq), (n, variant)
    if n:                                                     # a bf16 tensor is quantised from its exact values
        xb = torch.from_numpy((rng.standard_normal(n) * 2 - 0.3).astype(np.float32)).bfloat16()
        q, s, zp = eg.quantize_affine(xb.to(gc.DEV))
        wq, wscale, wzp = ao.quantize(xb.float().numpy())
        assert s.item() == wscale and zp.item() == wzp and np.array_equal(q.cpu().numpy(), wq)


@pytest.mark.gpu
def test_quantize_affine_flags_non_finite_values():
    from paper_2201_06227_amd import binding as eg
    import tests.gpu_common as gc
    wl = si.make_fc(b=4, k=64, n=8, seed=45)
    wl.x[2, 5] = np.inf
    with pytest.raises(AssertionError):
        _gpu_affine(wl, with_taps=False)
    with pytest.raises(orc.NonFiniteInput):
        ao.ref_forward(wl)


@pytest.mark.gpu
def test_weight_code_sums():
    from paper_2201_06227_amd import binding as eg
    import tests.gpu_common as gc
    rng = np.random.default_rng(46)
    ws_ = [rng.standard_normal((37, 50)).astype(np.float32), rng.standard_normal((20, 24, 3, 3)).astype(np.float32),
           rng.standard_normal((9, 130, 1, 1)).astype(np.float32)]
    dev = [gc.to_dev(w) for w in ws_]
    cs = [eg.colsum_like(w) for w in dev]
    w_q, scales = eg.quantize_weights(dev, colsums=cs)
    torch.cuda.synchronize()
    for w, q, c in zip(ws_, w_q, cs):
        wq, _ = orc.quantize(w)
        c = c.cpu().numpy()
        if w.ndim == 2 or w.shape[2] == 1:
            assert c.shape[0] == 1 and np.array_equal(c[0], wq.reshape(w.shape[0], -1).astype(np.int64).sum(axis=1))
            continue
        for cls in range(16):
            keep = np.ones((3, 3), bool)
            if cls & 1: keep[0, :] = False
            if cls & 2: keep[2, :] = False
            if cls & 4: keep[:, 0] = False
            if cls & 8: keep[:, 2] = False
            assert np.array_equal(c[cls], (wq.astype(np.int64) * keep).sum(axis=(1, 2, 3))), cls


def _without_skip(wl):
    wl.dims["has_residual"] = 0
    return wl


AFFINE_CASES = SMALL + [("fc_ragged", lambda: si.make_fc(b=33, k=77, n=130, seed=47)),
                        ("basic_1row", lambda: si.make_basic_block(b=2, c=5, h=1, w=7, seed=48)),
                        ("basic_1col", lambda: si.make_basic_block(b=1, c=18, h=6, w=1, seed=49)),
                        ("basic_nores", lambda: _without_skip(si.make_basic_block(b=2, c=16, h=8, w=8, seed=50))),
                        ("fc_cfg1", lambda: si.make_config(1)), ("basic_cfg2", lambda: si.make_config(2)),
                        ("bottleneck_cfg3", lambda: si.make_config(3)), ("bert_cfg4", lambda: si.make_config(4))]


@pytest.mark.gpu
@pytest.mark.parametrize("name,make", AFFINE_CASES, ids=[s[0] for s in AFFINE_CASES])
def test_affine_reference_matches_oracle(name, make):
    import tests.gpu_common as gc
    wl = make()
    ot = ao.ref_forward(wl)
    a_ref, taps, ref, ws = _gpu_affine(wl)
    plain, _, _, _ = _gpu_affine(wl, with_taps=False)
    assert np.array_equal(plain, a_ref)                                  # observed and unobserved runs agree
    bert = wl.kind >= si.KIND_BERT_LAYER
    for i, t in enumerate(taps):
        tag = f"L{i // 4}.l{i % 4}." if bert else f"l{i}."
        want_q = ot[tag + "xq"]
        want_q = gc.nhwc(want_q) if want_q.ndim == 4 else want_q.reshape(-1, want_q.shape[-1])
        K = want_q.shape[1]
        got_q = (t["x_q"].astype(np.int16) + 128)
        assert np.array_equal(got_q[:, :K], want_q), (i, name)
        assert not t["x_q"][:, K:].any()
        assert t["x_scale"][0] == ot[tag + "sx"] and t["x_zp"][0] == ot[tag + "zp"], (i, name)
        want_acc, want_y = ot[tag + "acc"], ot[tag + "y"]
        if want_acc.ndim == 4:
            want_acc, want_y = gc.nhwc(want_acc), gc.nhwc(want_y)
        assert np.array_equal(t["acc"], want_acc.reshape(t["acc"].shape)), (i, name)
        if bert:
            gc.assert_within_ulp(t["y"], want_y.reshape(t["y"].shape), 1, f"{name} y{i}")
        else:
            assert np.array_equal(t["y"], want_y.reshape(t["y"].shape)), (i, name)
    want = ot["a_ref"]
    if bert:
        per = a_ref.size // len(want)
        for l, w in enumerate(want):
            gc.assert_within_ulp(a_ref[l * per:(l + 1) * per], w.reshape(-1), 1, f"{name} a_ref{l}")
    else:
        want = gc.nhwc(want) if want.ndim == 4 else want
        assert np.array_equal(a_ref, want.reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("make", [lambda: si.make_basic_block(b=2, c=20, h=9, w=11, seed=51),
                                  lambda: si.make_bottleneck(b=3, c_in=64, c_mid=32, h=8, w=8, seed=52),
                                  lambda: si.make_bottleneck(b=2, c_in=24, c_mid=13, h=6, w=5, seed=53)])
def test_affine_inner_extrema_are_this_runs(make):
    """The extrema of the inner layers come from the GEMM's epilogue: a second run in the same workspace on a smaller
    input keeps nothing of the first one's, and an infinite inner activation is flagged."""
    from paper_2201_06227_amd import binding as eg
    import tests.gpu_common as gc
    wl = make()
    first, _, ref, ws = _gpu_affine(wl, with_taps=False)
    x = wl.x
    wl.x = x * np.float32(0.03125)
    a_ref = torch.empty(first.size, dtype=torch.float32, device=gc.DEV)
    eg.ref_forward(ref, gc.to_dev(wl.x), a_ref, ws)
    want = gc.nhwc(ao.ref_forward(wl)["a_ref"]).reshape(-1)
    assert np.array_equal(a_ref.cpu().numpy(), want)
    assert eg.check(ws) == eg.OK
    eg.ref_forward(ref, gc.to_dev(np.full_like(x, 3e38)), a_ref, ws)     # finite input, sums of the first layer are not
    torch.cuda.synchronize()
    assert eg.check(ws) != eg.OK


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [1, 2, 3, 4])
def test_affine_reference_score(cfg, orc_lib=None):
    """Plasticity against the affine reference (Eq. 1): within 1e-4 of the fp64 metric on the oracle's A_R."""
    from paper_2201_06227_amd import binding as eg
    import tests.gpu_common as gc
    wl = si.make_config(cfg)
    a_ref, _, ref, ws = _gpu_affine(wl, with_taps=False)
    a_t = [a.to(gc.DEV) for a in si.train_forward(wl)]
    p = torch.zeros(len(a_t), dtype=torch.float32, device=gc.DEV)
    eg.plasticity_eval(ref, gc.to_dev(wl.x), a_t, p, ws)
    torch.cuda.synchronize()
    want_ar = ao.ref_forward(wl)["a_ref"]
    want_ar = want_ar if isinstance(want_ar, list) else [want_ar]
    for l, w in enumerate(want_ar):
        w = gc.nhwc(w) if w.ndim == 4 else w
        want = orc.sp_loss(a_t[l].float().cpu().numpy().reshape(wl.batch, -1), w.reshape(wl.batch, -1))
        assert abs(p[l].item() - want) <= 1e-4 * abs(want) + 1e-12 * 4.0 / wl.batch, (cfg, l, p[l].item(), want)


@pytest.mark.gpu
def test_affine_rejects_what_it_does_not_cover():
    from paper_2201_06227_amd import binding as eg
    import tests.gpu_common as gc
    wl = si.make_fc(b=4, k=32, n=8, seed=51)
    W, B = [gc.to_dev(w) for w in wl.weights], [None if b is None else gc.to_dev(b) for b in wl.biases]
    ws = eg.workspace(1 << 22, gc.DEV)
    a = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
    ref = eg.make_reference(wl.kind, wl.dims, W, B, act_scales=gc.to_dev(np.array([0.05], np.float32)))
    ref.desc.act_scheme = eg.ACT_AFFINE                         # static scales with affine codes
    with pytest.raises(eg.EgeriaError) as e:
        eg.ref_forward(ref, gc.to_dev(wl.x), a, ws)
    assert e.value.code == eg.ERR_UNSUPPORTED
    ref = eg.make_reference(wl.kind, wl.dims, W, B)
    ref.desc.act_scheme = eg.ACT_AFFINE                         # no weight-code sums
    with pytest.raises(eg.EgeriaError) as e:
        eg.ref_forward(ref, gc.to_dev(wl.x), a, ws)
    assert e.value.code == eg.ERR_INVALID_ARG
