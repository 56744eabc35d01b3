"""GPU parity: the HIP path, called through the C-ABI binding, against the CPU
oracle on the same seeded inputs.

Bars: int8 codes, scales and int32 accumulators bit-exact; fp32 activations of
the convolution / FC modules bit-exact too (their arithmetic is +, x, fma, max,
rint in a fixed order); plasticity within 1e-4 relative of the fp64 oracle.
"""
import math

import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eg():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2201_06227_amd import binding
    binding.lib()                      # raises if the HIP library has not been built
    return binding


@pytest.fixture(scope="module")
def gc():
    import gpu_common
    return gpu_common


@pytest.fixture(autouse=True)
def certified_attention_at_every_size(eg):
    """Unobserved Transformer runs take the certified fp32 attention kernels only above a size threshold (below
    it the fp64 kernel is faster); the tests of this module exercise those kernels on small and ragged shapes
    too.  test_attention_paths_agree covers the default choice."""
    old = eg.attention_threshold(0.0)
    yield
    eg.attention_threshold(old)


P_RTOL = 1e-4


def p_close(got, want, b):
    return abs(got - want) <= P_RTOL * abs(want) + 1e-12 * 4.0 / b


# --------------------------------------------------------------------------- quantise

@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 1000, 4099, 12305, 16380, 16383, 16384, (1 << 20) + 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_quantize_flat_bit_exact(eg, gc, orc, n, dtype):
    rng = np.random.default_rng(100 + n)
    x = (rng.standard_normal(n) * 3).astype(np.float32)
    xt = gc.to_dev(x)
    if dtype == "bf16":
        xt = xt.to(torch.bfloat16)
        x = xt.float().cpu().numpy()
    q, s = eg.quantize(xt)
    want_q, want_s = orc.quantize(x)
    assert s.cpu().numpy()[0] == want_s
    assert (q.cpu().numpy() == want_q).all()
    xh = eg.dequantize(q, s).cpu().numpy()
    assert (xh == orc.dequantize(want_q, want_s)).all()


@pytest.mark.parametrize("n", [15, 1000, 12289, 12305, 16380, 16383, 16385, 70001])
def test_quantize_flat_stays_inside_its_buffers(eg, gc, orc, n):
    """q is int8 [n] exactly: the bytes after it are not the library's to write, whatever the tail of
    the tensor looks like (the last 16-code unit of a ragged tensor is written byte by byte)."""
    import ctypes
    rng = np.random.default_rng(4000 + n)
    x = (rng.standard_normal(n) * 2).astype(np.float32)
    pad = 4096
    xbuf = torch.full((n + pad,), float("nan"), dtype=torch.float32, device=gc.DEV)   # what follows x must not matter
    xbuf[:n] = gc.to_dev(x)
    qbuf = torch.full((n + pad,), 0x55, dtype=torch.int8, device=gc.DEV)
    scale = torch.zeros(1, dtype=torch.float32, device=gc.DEV)
    ws = eg.workspace(eg.quantize_workspace_bytes())
    rc = eg.lib().egeria_quantize(ctypes.c_void_p(xbuf.data_ptr()), eg.F32, n, None, ctypes.c_void_p(qbuf.data_ptr()),
                                  ctypes.c_void_p(scale.data_ptr()), ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                                  eg._stream())
    assert rc == eg.OK
    torch.cuda.synchronize()
    want_q, want_s = orc.quantize(x)
    assert eg.check(ws) == eg.OK
    assert scale.item() == want_s
    got = qbuf.cpu().numpy()
    assert (got[:n] == want_q).all()
    assert (got[n:] == 0x55).all()


def test_quantize_special_tensors(eg, gc, orc):
    ws = eg.workspace(eg.quantize_workspace_bytes())
    for x in (np.zeros(100, np.float32), np.full(33, 1e-40, np.float32),
              np.array([127, 0.5, 1.5, 2.5, -0.5, -1.5, -2.5, 126.5], np.float32)):
        q, s = eg.quantize(gc.to_dev(x), ws=ws)
        wq, wsc = orc.quantize(x)
        assert s.item() == wsc and (q.cpu().numpy() == wq).all()
    assert eg.check(ws) == eg.OK
    # static scale saturates
    x = np.array([0.26, -3.0, 100.0, 0.24] * 5, np.float32)
    q, s = eg.quantize(gc.to_dev(x), fixed_scale=gc.to_dev(np.array([0.5], np.float32)), ws=ws)
    wq, wsc = orc.quantize(x, fixed_scale=0.5)
    assert s.item() == wsc and (q.cpu().numpy() == wq).all()
    # non-finite input raises the workspace flag, once
    for bad in (np.nan, np.inf):
        xb = np.ones(1000, np.float32)
        xb[777] = bad
        eg.quantize(gc.to_dev(xb), ws=ws)
        assert eg.check(ws) == eg.ERR_NONFINITE
        assert eg.check(ws) == eg.OK


@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (7, 16), (33, 100), (64, 768), (130, 3072)])
def test_quantize_rows_bit_exact(eg, gc, orc, shape):
    rng = np.random.default_rng(sum(shape))
    x = rng.standard_normal(shape).astype(np.float32)
    q, s = eg.quantize_rows(gc.to_dev(x))
    wq, wsc = orc.quantize(x)
    assert s.item() == wsc
    gc.assert_int8_rows(q.cpu().numpy(), wq)


@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (2, 3, 5, 7), (16, 16, 3, 3), (3, 70, 9, 9),
                                   (2, 256, 14, 14), (4, 16, 32, 32)])
def test_quantize_nchw_bit_exact(eg, gc, orc, shape):
    rng = np.random.default_rng(sum(shape))
    x = rng.standard_normal(shape).astype(np.float32)
    q, s = eg.quantize_nchw(gc.to_dev(x))
    wq, wsc = orc.quantize(x)
    assert s.item() == wsc
    gc.assert_conv_q(q.cpu().numpy().reshape(-1, q.shape[-1]), wq)


WEIGHT_SETS = {
    "small_convs": [(16, 16, 3, 3), (16, 16, 3, 3)],
    "bottleneck": [(64, 256, 1, 1), (64, 64, 3, 3), (256, 64, 1, 1)],
    "mixed_ragged": [(7, 100), (1, 1), (33, 70, 3, 3), (130, 3072), (5, 3), (2304, 768)],
    "many": [(48 + i, 17 + 3 * i) for i in range(40)],
}


@pytest.mark.parametrize("name", sorted(WEIGHT_SETS))
def test_quantize_weights_batch_bit_exact(eg, gc, orc, name):
    """One call for a whole snapshot gives the codes and scales of the per-tensor rule."""
    rng = np.random.default_rng(len(name))
    ws_np = [(rng.standard_normal(sh) * (0.02 + 0.3 * i)).astype(np.float32) for i, sh in enumerate(WEIGHT_SETS[name])]
    w_q, scales = eg.quantize_weights([gc.to_dev(w) for w in ws_np])
    for w, q, s in zip(ws_np, w_q, scales):
        wq, wsc = orc.quantize(w)
        assert s.item() == wsc
        if w.ndim == 4:
            gc.assert_conv_q(q.cpu().numpy().reshape(-1, q.shape[-1]), wq)
        else:
            gc.assert_int8_rows(q.cpu().numpy(), wq)


@pytest.mark.parametrize("shapes", [[(33, 24), (257, 768), (5, 40), (70, 1008), (300, 77)], [(130, 72, 3, 3), (64, 200), (19, 1000)],
                                    [(4101, 2048), (2050, 4104), (13, 8)]], ids=["rows", "mixed", "large"])
def test_quantize_weights_bf16_bit_exact(eg, gc, orc, shapes):
    """bf16 snapshots with one scale per tensor: whole and ragged 16-byte units, padded rows, a set large enough for the
    longer shares, and the extreme value at either end of a tensor."""
    g = torch.Generator().manual_seed(len(shapes[0]))
    ws = [(torch.randn(*sh, generator=g) * (0.02 + 0.3 * i)).to(torch.bfloat16) for i, sh in enumerate(shapes)]
    ws[0].view(-1)[-1] = -9.0
    ws[1].view(-1)[0] = 11.0
    wsp = eg.workspace(eg.quantize_weights_workspace_bytes(len(ws)))
    w_q, scales = eg.quantize_weights([w.to(gc.DEV) for w in ws], ws=wsp)
    assert eg.check(wsp) == eg.OK
    for w, q, s in zip(ws, w_q, scales):
        wq, wsc = orc.quantize(w.float().numpy())
        assert s.item() == wsc
        if w.ndim == 4:
            gc.assert_conv_q(q.cpu().numpy().reshape(-1, q.shape[-1]), wq)
        else:
            gc.assert_int8_rows(q.cpu().numpy(), wq)
    ws[-1].view(-1)[-1] = float("inf")
    eg.quantize_weights([w.to(gc.DEV) for w in ws], ws=wsp)
    assert eg.check(wsp) == eg.ERR_NONFINITE


def test_quantize_weights_batch_flags_and_empty(eg, gc, orc):
    ws = eg.workspace(eg.quantize_weights_workspace_bytes(3))
    good = np.ones((4, 20), np.float32)
    bad = np.ones((200, 300), np.float32)
    bad[150, 7] = np.inf
    w_q, scales = eg.quantize_weights([gc.to_dev(good), gc.to_dev(np.zeros((8, 8), np.float32))], ws=ws)
    assert eg.check(ws) == eg.OK
    assert scales[1].item() == 1.0 and not w_q[1].any().item()
    eg.quantize_weights([gc.to_dev(good), gc.to_dev(bad), gc.to_dev(good)], ws=ws)
    assert eg.check(ws) == eg.ERR_NONFINITE
    assert eg.check(ws) == eg.OK
    w_q, scales = eg.quantize_weights([], ws=ws)
    assert w_q == []


# --------------------------------------------------------------------------- FC / conv modules

def _check_linear_taps(gc, taps, ot, prefix, conv):
    xq, acc, y = ot[prefix + "xq"], ot[prefix + "acc"], ot[prefix + "y"]
    assert taps["x_scale"][0] == ot[prefix + "sx"]
    if conv:
        gc.assert_conv_q(taps["x_q"], xq)
        assert (taps["acc"] == gc.nhwc(acc)).all()
        assert (taps["y"] == gc.nhwc(y)).all()
    else:
        gc.assert_int8_rows(taps["x_q"], xq.reshape(-1, xq.shape[-1]))
        assert (taps["acc"] == acc).all()
        assert (taps["y"] == y).all()


FC_CASES = [dict(b=1, k=1, n=1), dict(b=5, k=100, n=7), dict(b=130, k=200, n=257),
            dict(b=64, k=3072, n=96), dict(b=32, k=512, n=512)]


@pytest.mark.parametrize("kw", FC_CASES, ids=lambda k: "b{b}_k{k}_n{n}".format(**k))
def test_fc_module_bit_exact(eg, gc, orc, kw):
    wl = si.make_fc(seed=200 + kw["k"], **kw)
    a_ref, taps, _ = gc.run_forward(wl)
    ot = orc.ref_forward(wl)
    _check_linear_taps(gc, taps[0], ot, "l0.", conv=False)
    assert (a_ref[0] == ot["a_ref"]).all()


@pytest.mark.parametrize("kw", [dict(b=1, k=16, n=8), dict(b=5, k=100, n=7), dict(b=32, k=512, n=512),
                                dict(b=64, k=96, n=700), dict(b=128, k=64, n=1024)],
                         ids=lambda k: "b{b}_k{k}_n{n}".format(**k))
def test_fc_score_equals_the_metric_on_its_activation(eg, gc, orc, kw):
    """The fused evaluation of an FC module gives the score the metric gives on the stored activation, bit for
    bit, call after call on a workspace that starts with stale bytes, and within 1e-4 of the oracle."""
    wl = si.make_fc(seed=300 + kw["n"], **kw)
    ref = gc.build_reference(wl)
    x = gc.to_dev(wl.x)
    a_t = si.train_forward(wl)[0].to(gc.DEV)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    ws.fill_(0xA5)
    a_ref = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
    eg.ref_forward(ref, x, a_ref, ws)
    sep = eg.plasticity(a_t, a_ref.reshape(wl.batch, -1))
    want = orc.sp_loss(a_t.float().cpu().numpy(), orc.ref_forward(wl)["a_ref"])
    for rep in range(3):
        p = torch.full((1,), -1.0, dtype=torch.float32, device=gc.DEV)
        eg.plasticity_eval(ref, x, [a_t], p, ws)
        torch.cuda.synchronize()
        assert p.item() == sep.item(), (rep, p.item(), sep.item())
    assert abs(p.item() - want) <= 1e-4 * abs(want) + 1e-12 * 4.0 / wl.batch


BASIC_CASES = [dict(b=1, c=1, h=1, w=1), dict(b=3, c=8, h=7, w=6), dict(b=2, c=20, h=9, w=11),
               dict(b=5, c=16, h=32, w=32), dict(b=2, c=64, h=13, w=13)]


@pytest.mark.parametrize("kw", BASIC_CASES, ids=lambda k: "b{b}_c{c}_{h}x{w}".format(**k))
def test_basic_block_bit_exact(eg, gc, orc, kw):
    wl = si.make_basic_block(seed=300 + kw["c"], **kw)
    a_ref, taps, _ = gc.run_forward(wl)
    ot = orc.ref_forward(wl)
    for i in range(2):
        _check_linear_taps(gc, taps[i], ot, f"l{i}.", conv=True)
    assert (a_ref[0].reshape(-1, kw["c"]) == gc.nhwc(ot["a_ref"])).all()


NARROW_CASES = [dict(b=1, c=1, h=1, w=1), dict(b=3, c=8, h=7, w=6), dict(b=3, c=16, h=9, w=11),
                dict(b=5, c=16, h=32, w=32), dict(b=2, c=5, h=3, w=200), dict(b=1, c=16, h=2, w=300),
                dict(b=1, c=3, h=2, w=256), dict(b=2, c=20, h=9, w=11)]


def _run_unobserved(eg, gc, wl, x_dev, act_scales=None):
    ref = gc.build_reference(wl, act_scales)
    a_ref = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    eg.ref_forward(ref, x_dev, a_ref, ws, None)
    torch.cuda.synchronize()
    return a_ref.cpu().numpy(), eg.check(ws)


@pytest.mark.parametrize("kw", NARROW_CASES, ids=lambda k: "b{b}_c{c}_{h}x{w}".format(**k))
@pytest.mark.parametrize("res", [1, 0])
@pytest.mark.parametrize("xdt", ["f32", "bf16"])
def test_basic_block_unobserved_bit_exact(eg, gc, orc, kw, res, xdt):
    """Unobserved runs of narrow basic blocks quantise their operands inside the convolutions (no int8
    tensor is stored); wide images and wider blocks take the general path.  Same A_R either way, with
    dynamic and with static scales, with and without the skip connection, fp32 and bf16 block input."""
    wl = si.make_basic_block(seed=330 + kw["c"] + kw["w"], **kw)
    wl.dims["has_residual"] = res
    if xdt == "bf16":
        wl.x = torch.from_numpy(wl.x).to(torch.bfloat16).float().numpy()
    x_dev = gc.to_dev(wl.x, torch.bfloat16 if xdt == "bf16" else None)
    ot = orc.ref_forward(wl)
    got, status = _run_unobserved(eg, gc, wl, x_dev)
    assert status == eg.OK
    assert (got.reshape(-1, kw["c"]) == gc.nhwc(ot["a_ref"])).all()
    scales = [0.7 * float(ot[f"l{i}.sx"]) for i in range(2)]              # static, a little clipping
    want = gc.nhwc(orc.ref_forward(wl, act_scales=scales)["a_ref"])
    got, status = _run_unobserved(eg, gc, wl, x_dev, scales)
    assert status == eg.OK
    assert (got.reshape(-1, kw["c"]) == want).all()


def test_basic_block_unobserved_random_shapes(eg, gc, orc):
    """Seeded random narrow blocks (1-16 channels, images of 1-40 x 1-70 pixels, 1-5 samples): the
    convolutions that quantise on load against the oracle, bit for bit."""
    rng = np.random.default_rng(20240611)
    for case in range(24):
        kw = dict(b=int(rng.integers(1, 6)), c=int(rng.integers(1, 17)), h=int(rng.integers(1, 41)),
                  w=int(rng.integers(1, 71)))
        wl = si.make_basic_block(seed=9000 + case, **kw)
        wl.dims["has_residual"] = int(rng.integers(0, 2))
        bf16 = bool(rng.integers(0, 2))
        if bf16:
            wl.x = torch.from_numpy(wl.x).to(torch.bfloat16).float().numpy()
        x_dev = gc.to_dev(wl.x, torch.bfloat16 if bf16 else None)
        ot = orc.ref_forward(wl)
        scales = None
        if rng.integers(0, 2):
            scales = [float(rng.uniform(0.5, 1.2)) * float(ot[f"l{i}.sx"]) for i in range(2)]
            ot = orc.ref_forward(wl, act_scales=scales)
        got, status = _run_unobserved(eg, gc, wl, x_dev, scales)
        assert status == eg.OK, (case, kw)
        assert (got.reshape(-1, kw["c"]) == gc.nhwc(ot["a_ref"])).all(), (case, kw, wl.dims, bf16, scales)


def test_basic_block_unobserved_reports_non_finite_input(eg, gc):
    wl = si.make_basic_block(seed=77, b=2, c=16, h=8, w=8)
    wl.x[1, 3, 2, 5] = np.inf
    _, status = _run_unobserved(eg, gc, wl, gc.to_dev(wl.x))
    assert status == eg.ERR_NONFINITE


BOTTLENECK_CASES = [dict(b=2, c_in=32, c_mid=16, h=5, w=5), dict(b=1, c_in=40, c_mid=24, h=7, w=3),
                    dict(b=3, c_in=256, c_mid=64, h=14, w=14),
                    dict(b=2, c_in=32, c_mid=16, h=5, w=5, has_residual=0)]


@pytest.mark.parametrize("kw", BOTTLENECK_CASES,
                         ids=lambda k: "b{b}_c{c_in}_{c_mid}_{h}x{w}_r{r}".format(r=k.get("has_residual", 1), **k))
def test_bottleneck_bit_exact(eg, gc, orc, kw):
    wl = si.make_bottleneck(seed=400 + kw["c_in"], **kw)
    a_ref, taps, _ = gc.run_forward(wl)
    ot = orc.ref_forward(wl)
    for i in range(3):
        _check_linear_taps(gc, taps[i], ot, f"l{i}.", conv=True)
    assert (a_ref[0].reshape(-1, kw["c_in"]) == gc.nhwc(ot["a_ref"])).all()


STATIC_CASES = [("fc", dict(b=5, k=100, n=7)), ("fc", dict(b=130, k=200, n=257)),
                ("basic", dict(b=3, c=8, h=7, w=6)), ("basic", dict(b=2, c=20, h=9, w=11)),
                ("basic", dict(b=5, c=16, h=32, w=32)), ("basic", dict(b=2, c=64, h=13, w=13)),
                ("bottleneck", dict(b=2, c_in=32, c_mid=16, h=5, w=5)),
                ("bottleneck", dict(b=1, c_in=40, c_mid=24, h=7, w=3)),
                ("bottleneck", dict(b=3, c_in=256, c_mid=64, h=14, w=14))]


def _static_workload(kind, kw):
    if kind == "fc":
        return si.make_fc(seed=700 + kw["k"], **kw), False
    if kind == "basic":
        return si.make_basic_block(seed=710 + kw["c"], **kw), True
    return si.make_bottleneck(seed=720 + kw["c_in"], **kw), True


def _check_static(gc, orc, wl, conv, scales, with_taps):
    a_ref, taps, _ = gc.run_forward(wl, with_taps=with_taps, act_scales=scales)
    ot = orc.ref_forward(wl, act_scales=scales)
    if with_taps:
        for i in range(len(taps)):
            _check_linear_taps(gc, taps[i], ot, f"l{i}.", conv=conv)
    want = gc.nhwc(ot["a_ref"]).reshape(wl.batch, -1) if conv else ot["a_ref"]
    assert (a_ref[0] == want).all()
    return want


@pytest.mark.parametrize("kind,kw", STATIC_CASES, ids=lambda v: v if isinstance(v, str) else "_".join(f"{k}{x}" for k, x in v.items()))
def test_static_scales_bit_exact(eg, gc, orc, kind, kw):
    """Static activation scales (Section 5, convolutional networks): calibrated on the batch itself they
    reproduce the dynamic forward; halved they saturate; observed and unobserved runs agree with the oracle."""
    wl, conv = _static_workload(kind, kw)
    dyn = orc.ref_forward(wl)
    n = len(wl.weights)
    scales = [float(dyn[f"l{i}.sx"]) for i in range(n)]
    want = _check_static(gc, orc, wl, conv, scales, True)
    dyn_want = gc.nhwc(dyn["a_ref"]).reshape(wl.batch, -1) if conv else dyn["a_ref"]
    assert (want == dyn_want).all()                       # same scales: same forward
    _check_static(gc, orc, wl, conv, scales, False)       # the path without fp32 round trips
    tight = [0.5 * v for v in scales]
    _check_static(gc, orc, wl, conv, tight, True)
    _check_static(gc, orc, wl, conv, tight, False)


@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_static_scales_full_size(eg, gc, orc, cfg):
    wl = si.make_config(cfg)
    conv = cfg != 1
    dyn = orc.ref_forward(wl)
    scales = [0.9 * float(dyn[f"l{i}.sx"]) for i in range(len(wl.weights))]     # a little clipping
    want = _check_static(gc, orc, wl, conv, scales, False)
    a_t = si.train_forward(wl)[0]
    p_want = orc.sp_loss(a_t.float().numpy(), want)
    ref = gc.build_reference(wl, scales)
    ws = eg.workspace(eg.workspace_bytes(ref.desc))
    p = torch.zeros(1, dtype=torch.float32, device=gc.DEV)
    eg.plasticity_eval(ref, gc.to_dev(wl.x), [a_t.to(gc.DEV)], p, ws)
    torch.cuda.synchronize()
    assert p_close(p.item(), p_want, wl.batch), (p.item(), p_want)


def test_static_scales_rejected_for_transformer_kinds(eg, gc):
    wl = si.make_bert(b=2, s=16, hidden=64, heads=4, ffn=128, n_layers=1, seed=5)
    ref = gc.build_reference(wl, [1.0, 1.0, 1.0, 1.0])
    a_ref = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    with pytest.raises(eg.EgeriaError) as e:
        eg.ref_forward(ref, gc.to_dev(wl.x), a_ref, ws, None)
    assert e.value.code == eg.ERR_UNSUPPORTED


@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_full_size_configs_bit_exact_and_scored(eg, gc, orc, cfg):
    """Configs 1-3 at full size: every observation point bit-exact, and the
    fused forward + score call within tolerance of the oracle's score."""
    wl = si.make_config(cfg)
    a_ref, taps, ref = gc.run_forward(wl)
    ot = orc.ref_forward(wl)
    conv = cfg != 1
    for i in range(len(taps)):
        _check_linear_taps(gc, taps[i], ot, f"l{i}.", conv=conv)
    want = gc.nhwc(ot["a_ref"]).reshape(wl.batch, -1) if conv else ot["a_ref"]
    assert (a_ref[0] == want).all()
    # the run without observation points is the one the benchmark times (other kernels in places)
    plain, status = _run_unobserved(eg, gc, wl, gc.to_dev(wl.x))
    assert status == eg.OK
    assert (plain.reshape(wl.batch, -1) == want).all()
    a_t = si.train_forward(wl)[0]
    p_want = orc.sp_loss(a_t.float().numpy(), want)
    ws = eg.workspace(eg.workspace_bytes(ref.desc))
    p = torch.zeros(1, dtype=torch.float32, device=gc.DEV)
    eg.plasticity_eval(ref, gc.to_dev(wl.x), [a_t.to(gc.DEV)], p, ws)
    torch.cuda.synchronize()
    assert p_close(p.item(), p_want, wl.batch), (p.item(), p_want)


# --------------------------------------------------------------------------- metric

METRIC_CASES = [(1, 7), (2, 1), (2, 3), (4, 4), (5, 129), (8, 300), (31, 1000), (32, 512), (33, 515),
                (64, 4096), (100, 2050), (128, 16384), (128, 777)]


@pytest.mark.parametrize("b,D", METRIC_CASES)
@pytest.mark.parametrize("rel", [0.3, 1e-3])
def test_plasticity_matches_oracle(eg, gc, orc, b, D, rel):
    a_t, a_r = si.noisy_pair(b, D, rel=rel, seed=500 + b + D)
    p = eg.plasticity(gc.to_dev(a_t), gc.to_dev(a_r)).item()
    want = orc.sp_loss(a_t, a_r)
    assert p_close(p, want, b), (p, want)


@pytest.mark.parametrize("b,D", [(8, 304), (32, 4096), (64, 1000)])
def test_plasticity_bf16_training_activation(eg, gc, orc, b, D):
    a_t, a_r = si.noisy_pair(b, D, rel=0.05, seed=600 + b)
    t16 = gc.to_dev(a_t).to(torch.bfloat16)
    want = orc.sp_loss(t16.float().cpu().numpy(), a_r)
    assert p_close(eg.plasticity(t16, gc.to_dev(a_r)).item(), want, b)
    r16 = gc.to_dev(a_r).to(torch.bfloat16)
    want = orc.sp_loss(t16.float().cpu().numpy(), r16.float().cpu().numpy())
    assert p_close(eg.plasticity(t16, r16).item(), want, b)


def test_plasticity_golden_and_closed_forms(eg, gc, orc):
    import os
    from test_oracle_pins import _read_sp_cases
    for c in _read_sp_cases():
        p = eg.plasticity(gc.to_dev(c["T"]), gc.to_dev(c["R"])).item()
        assert p_close(p, c["P"], c["b"]), (c["name"], p)
    for b in (2, 32, 64, 128):
        D = b + 5
        q_t = np.zeros((b, D), np.float32)
        q_t[np.arange(b), np.arange(b)] = 1 + np.arange(b) % 5
        q_r = np.tile(np.linspace(0.5, 2, D, dtype=np.float32), (b, 1))
        p = eg.plasticity(gc.to_dev(q_t), gc.to_dev(q_r)).item()
        assert p_close(p, (2.0 / b) * (1 - 1 / math.sqrt(b)), b)


def test_plasticity_invariants(eg, gc):
    a_t, a_r = si.noisy_pair(16, 1000, rel=0.1, seed=700)
    t, r = gc.to_dev(a_t), gc.to_dev(a_r)
    assert eg.plasticity(t, t.clone()).item() == 0.0
    p = eg.plasticity(t, r).item()
    assert p > 0
    assert eg.plasticity(t * 4, r * -0.125).item() == pytest.approx(p, rel=1e-5)
    perm = torch.randperm(1000, device=gc.DEV)
    assert eg.plasticity(t[:, perm].contiguous(), r).item() == pytest.approx(p, rel=1e-4)
    # a zero row and a single sample stay finite
    r0 = r.clone()
    r0[3] = 0
    assert math.isfinite(eg.plasticity(t, r0).item())
    assert eg.plasticity(t[:1].contiguous(), r[:1].contiguous()).item() == 0.0
    # same call twice: identical bits (partials are reduced in a fixed order)
    assert eg.plasticity(t, r).item() == p


@pytest.mark.parametrize("b,D,dt", [(128, 16384, "f32"), (64, 200704, "f32"), (32, 98304, "bf16"),
                                    (64, 196608, "f32")])
def test_plasticity_full_size_shapes(eg, gc, orc, b, D, dt):
    a_t, a_r = si.noisy_pair(b, D, rel=0.01, seed=800 + b, nonneg=(D == 200704))
    t = gc.to_dev(a_t)
    if dt == "bf16":
        t = t.to(torch.bfloat16)
        a_t = t.float().cpu().numpy()
    want = orc.sp_loss(a_t, a_r)
    p = eg.plasticity(t, gc.to_dev(a_r)).item()
    assert p_close(p, want, b), (p, want)


# --------------------------------------------------------------------------- Transformer modules
# Soft-max attention, layer norm and GELU sit between the int8 GEMMs.  A
# last-bit difference in any of them can move a value across a quantisation
# boundary, and an int8 code that differs is amplified by every later layer
# (measured with an fp32 evaluation of that glue: 3% relative deviation of the
# activation and up to 8% of the score after 12 layers).  Both sides therefore
# evaluate the glue in fp64 and round once to fp32, which makes the chains agree
# bit for bit on these seeded inputs: every int8 code, scale, accumulator and
# fp32 tensor is compared for equality, as for the convolution modules.

def _check_bert_layer_taps(gc, taps, ot, l):
    """The contract of the Transformer modules: every int8 code, every scale and every int32 accumulator
    equals the oracle's; so does every GEMM output that is a pure function of them (one fma).  The GELU
    output (fp64 erf on both sides, different math libraries) is compared within one fp32 ulp."""
    for i in range(4):
        t, pre = taps[4 * l + i], f"L{l}.l{i}."
        xq = ot[pre + "xq"]
        assert t["x_scale"][0] == ot[pre + "sx"], pre
        gc.assert_int8_rows(t["x_q"], xq)
        assert (t["acc"] == ot[pre + "acc"]).all(), pre
        if i == 2:
            gc.assert_within_ulp(t["y"], ot[pre + "y"], 1, pre + "y (gelu)")
        else:
            assert (t["y"] == ot[pre + "y"]).all(), pre


BERT_CASES = [dict(b=2, s=12, hidden=48, heads=4, ffn=96, n_layers=1),
              dict(b=3, s=40, hidden=128, heads=2, ffn=200, n_layers=1),
              dict(b=2, s=130, hidden=192, heads=3, ffn=320, n_layers=3),
              dict(b=1, s=1, hidden=64, heads=1, ffn=16, n_layers=2),
              dict(b=8, s=64, hidden=768, heads=12, ffn=3072, n_layers=12),
              # enough rows (12288) for the attention-output layer and its layer norm to share a launch, with
              # rows shorter than that kernel's tile
              dict(b=48, s=256, hidden=64, heads=1, ffn=16, n_layers=2)]


@pytest.mark.parametrize("kw", BERT_CASES, ids=lambda k: "b{b}_s{s}_h{hidden}_L{n_layers}".format(**k))
def test_bert_modules_bit_exact_and_scored(eg, gc, orc, kw):
    wl = si.make_bert(seed=900 + kw["s"], train_act_dtype="f32", **kw)
    a_ref, taps, ref = gc.run_forward(wl)
    ot = orc.ref_forward(wl)
    for l in range(kw["n_layers"]):
        _check_bert_layer_taps(gc, taps, ot, l)
        gc.assert_within_ulp(a_ref[l], ot["a_ref"][l].reshape(kw["b"], -1), 1, f"A_R layer {l}")
    # an unobserved run takes other kernels in places (GELU inside a quantiser, attention on the
    # fast path with certified codes): the same activations as the observed run, bit for bit
    plain, _, _ = gc.run_forward(wl, with_taps=False)
    for l in range(kw["n_layers"]):
        assert (plain[l] == a_ref[l]).all(), l
    a_t = si.train_forward(wl)
    ws = eg.workspace(eg.workspace_bytes(ref.desc))
    p = torch.zeros(kw["n_layers"], dtype=torch.float32, device=gc.DEV)
    eg.plasticity_eval(ref, gc.to_dev(wl.x), [t.to(gc.DEV) for t in a_t], p, ws)
    for l in range(kw["n_layers"]):
        want = orc.sp_loss(a_t[l].numpy(), ot["a_ref"][l])
        assert p_close(p[l].item(), want, kw["b"]), (l, p[l].item(), want)


# shapes that reach each variant of the certification kernel: keys held in LDS (all of them, or 256 at a time) or read from
# global memory (a head size that is no multiple of 4), 16 values or one value per thread
ATTENTION_SHAPES = [dict(b=3, s=77, hidden=200, heads=5, ffn=328, n_layers=2),      # keys in LDS, single values
                    dict(b=2, s=200, hidden=128, heads=2, ffn=64, n_layers=2),      # keys in LDS, 16 per thread
                    dict(b=1, s=300, hidden=96, heads=3, ffn=64, n_layers=2),       # keys in LDS in two rounds, 16 per thread
                    dict(b=1, s=129, hidden=24, heads=3, ffn=64, n_layers=2),       # heads of 8, shares of a head's tokens
                    dict(b=1, s=515, hidden=96, heads=2, ffn=64, n_layers=2),       # keys in three rounds, a token more than a share
                    dict(b=2, s=70, hidden=66, heads=3, ffn=40, n_layers=2)]        # head size 22: the fp64 kernel


@pytest.mark.parametrize("kw", ATTENTION_SHAPES, ids=lambda k: "b{b}_s{s}_h{hidden}_heads{heads}".format(**k))
def test_attention_paths_agree(eg, gc, kw):
    """The two evaluations of attention in unobserved runs (fp64 kernel below the size threshold, certified fp32
    kernels above it) and the observed run give the same A_R bit for bit."""
    wl = si.make_bert(seed=61 + kw["s"], train_act_dtype="f32", **kw)
    ref = gc.build_reference(wl)
    x = gc.to_dev(wl.x)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    outs = []
    for thr in (0.0, 5.0e9):
        eg.attention_threshold(thr)
        a = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
        eg.ref_forward(ref, x, a, ws)
        torch.cuda.synchronize()
        assert eg.check(ws) == eg.OK
        outs.append(a)
    observed, _, _ = gc.run_forward(wl)
    assert torch.equal(outs[0], outs[1])
    assert np.array_equal(outs[0].cpu().numpy().reshape(observed.shape), observed)


@pytest.mark.parametrize("kind", ["normal", "uniform x4", "2 tokens in order", "equal scores 30", "2 tokens cancelling terms"])
@pytest.mark.parametrize("S,heads,dh", [(64, 2, 16), (131, 3, 16), (200, 2, 64), (70, 3, 22)])
def test_profile_attention_writes_its_records_only(eg, gc, S, heads, dh, kind):
    """The measuring entry leaves one pair per 64 queries of a head and nothing behind them, and the error of each value is
    within the bound of its pair."""
    B, H = 2, heads * dh
    qkv = gc.to_dev(si.attention_qkv(kind, B, S, heads, dh))
    tiles = (S + 63) // 64
    n = B * heads * tiles
    rec = torch.full((2 * n + B * heads * S,), 7, dtype=torch.int32, device=gc.DEV)
    ctx = torch.empty(B, S, H, device=gc.DEV)
    assert eg.lib().egeria_profile_attention(qkv.data_ptr(), B, S, H, heads, 1, ctx.data_ptr(), rec.data_ptr(),
                                             torch.cuda.current_stream().cuda_stream) == eg.OK
    exact, _ = eg.profile_attention(qkv, heads, 0)
    torch.cuda.synchronize()
    assert bool((rec[2 * n:] == 7).all())
    pairs = rec[:2 * n].view(torch.float32).reshape(B, heads, tiles, 2).cpu()
    c, e = (t.reshape(B, S, heads, dh).permute(0, 2, 1, 3).cpu() for t in (ctx, exact))
    for t in range(tiles):
        part = c[:, :, 64 * t:64 * t + 64]
        assert torch.equal(pairs[:, :, t, 0], part.abs().amax((2, 3)))
        err = (part.double() - e[:, :, 64 * t:64 * t + 64].double()).abs() - 12 * 2.0 ** -24 * part.double().abs()
        assert bool((err.amax((2, 3)) <= pairs[:, :, t, 1].double()).all())


@pytest.mark.parametrize("kind", si.ATTENTION_KINDS)
@pytest.mark.parametrize("b,s,heads,dh", [(2, 131, 3, 64), (2, 256, 12, 64), (1, 515, 4, 48), (2, 300, 4, 8)])
def test_attention_error_is_within_its_bound(eg, gc, b, s, heads, dh, kind):
    """What the certified codes rest on: no value of the approximate context is further from the fp64 evaluation than its
    query's bound and the part that grows with the value say, on inputs whose rounding errors add up too."""
    qkv = gc.to_dev(si.attention_qkv(kind, b, s, heads, dh))
    approx, bounds = eg.profile_attention_bounds(qkv, heads)
    exact, _ = eg.profile_attention(qkv, heads, 0)
    torch.cuda.synchronize()
    split = lambda t: t.reshape(b, s, heads, dh).permute(0, 2, 1, 3).double()  # noqa: E731
    err = (split(approx) - split(exact)).abs() - 12 * 2.0 ** -24 * split(approx).abs()
    assert bool((err.amax(-1) <= bounds.double()).all()), (err.amax(-1) / bounds.double()).max().item()
    if kind == "normal":                                          # ... and is no larger than it has to be
        vmax = qkv[..., 2 * heads * dh:].abs().max().item()
        assert bounds.median().item() <= 16 * 2.0 ** -24 * vmax


@pytest.mark.parametrize("factor", [1e-3, 0.0])
@pytest.mark.parametrize("s", [20, 128, 131])
def test_attention_bound_of_zero_queries_is_a_number(eg, gc, s, factor):
    """Query rows of zeros beside small values, and nothing but zeros: the scores are zero, the bounds finite, so that the
    quantiser does not re-evaluate every value."""
    qkv = si.attention_qkv("normal", 2, s, 2, 32) * np.float32(factor)
    qkv[:, ::3, :64] = 0.0
    ctx, bounds = eg.profile_attention_bounds(gc.to_dev(qkv), 2)
    assert bool(torch.isfinite(ctx).all()) and bool(torch.isfinite(bounds).all())
    assert bounds.max().item() <= 1e-6 * factor


# what the certified kernels meet beyond ordinary activations: rows that tie for the tensor's maximum (the candidates of a
# workgroup overflow its list), nothing but zeros, whole samples twice, scores in the hundreds, values that the split's scale
# leaves few digits of (every code is re-evaluated: the list of the quantiser overflows), three tokens in uneven shares, padding
ATTENTION_INPUTS = ["equal tokens", "zeros", "equal samples", "large scores", "uneven values", "few tokens", "padding"]


@pytest.mark.parametrize("inputs", ATTENTION_INPUTS)
@pytest.mark.parametrize("kw", [dict(b=3, s=131, hidden=128, heads=2), dict(b=2, s=260, hidden=96, heads=4)],
                         ids=["s131_dh64", "s260_dh24"])
def test_attention_paths_agree_on_extreme_inputs(eg, gc, kw, inputs):
    wl = si.make_bert(seed=71, ffn=64, n_layers=1, train_act_dtype="f32", **kw)
    h = kw["hidden"]
    x, wqkv = wl.x.copy(), wl.weights[0].copy()
    per_channel = False
    if inputs == "equal tokens":
        x[:, 1:] = x[:, :1]
    elif inputs == "zeros":
        x[:] = 0.0
    elif inputs == "equal samples":
        x[1:] = x[:1]
    elif inputs == "large scores":
        wqkv[:2 * h] *= 12.0
    elif inputs == "few tokens":
        x = x[:, np.random.default_rng(5).choice(3, x.shape[1], p=[0.6, 0.3, 0.1])]
    elif inputs == "padding":
        x[:, x.shape[1] // 4:] = x[:, :1]
    else:
        per_channel = True                       # (one scale for all would round the small rows to zero)
        wqkv[2 * h:] *= np.float32(3.0e7)
    wl.x, wl.weights[0] = np.ascontiguousarray(x), np.ascontiguousarray(wqkv)
    ref = eg.make_reference(wl.kind, wl.dims, [gc.to_dev(w) for w in wl.weights], [None] * len(wl.weights), per_channel=per_channel)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    outs = []
    for thr in (0.0, 1.0e30):
        eg.attention_threshold(thr)
        a = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
        eg.ref_forward(ref, gc.to_dev(wl.x), a, ws)
        torch.cuda.synchronize()
        assert eg.check(ws) == eg.OK
        outs.append(a)
    assert torch.equal(outs[0], outs[1])


def test_equal_samples_share_the_search_for_the_maximum(eg, gc):
    """Samples that occur several times tie for the tensor's maximum; each tie is evaluated once, not by every workgroup
    that quantises (which took ten times as long as distinct samples here)."""
    b, s, h = 256, 128, 256
    wl = si.make_bert(b=b, s=s, hidden=h, heads=4, ffn=64, n_layers=1, seed=72, train_act_dtype="f32")
    ref = gc.build_reference(wl)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    x = gc.to_dev(wl.x)
    same = x[:1].expand_as(x).contiguous()
    outs, times = [], []
    for inp, thr in ((x, 0.0), (same, 0.0), (same, 1.0e30)):
        eg.attention_threshold(thr)
        a = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
        best = float("inf")
        for _ in range(5):
            start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            eg.ref_forward(ref, inp, a, ws)
            stop.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(stop))
        outs.append(a)
        times.append(best)
    assert eg.check(ws) == eg.OK
    assert torch.equal(outs[1], outs[2])
    assert times[1] <= 3.0 * times[0], times


@pytest.mark.parametrize("column", ["query", "value"])
def test_attention_reports_non_finite_values(eg, gc, column):
    """An infinite bias in the QKV layer puts non-finite values into the attention (finite inputs and weights
    do not reach that state): the approximate attention kernels must carry them into the status word, through
    the value maximum of their records (value column) or through the stored context (query column)."""
    wl = si.make_bert(b=2, s=70, hidden=64, heads=2, ffn=32, n_layers=1, seed=404, train_act_dtype="f32")
    wl.biases[0] = wl.biases[0].copy()
    wl.biases[0][(0 if column == "query" else 2 * 64) + 5] = np.inf
    ref = gc.build_reference(wl)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    a = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
    eg.ref_forward(ref, gc.to_dev(wl.x), a, ws)
    torch.cuda.synchronize()
    assert eg.check(ws) == eg.ERR_NONFINITE


def test_bert_small_preactivations(eg, gc, orc):
    """The fused GELU quantiser takes absmax = gelu(max v) as a shortcut when
    max v >= 0.5; with tiny feed-forward weights it must fall back to the exact
    absolute maximum of gelu(v) (which may then sit at a negative v)."""
    wl = si.make_bert(b=2, s=24, hidden=64, heads=2, ffn=160, n_layers=2, seed=977, train_act_dtype="f32")
    for l in range(2):
        wl.weights[4 * l + 2] = (wl.weights[4 * l + 2] * np.float32(0.02)).astype(np.float32)
    a_ref, taps, ref = gc.run_forward(wl)
    ot = orc.ref_forward(wl)
    assert float(np.abs(ot["L0.l2.acc"]).max()) > 0 and float(ot["L0.l2.y"].max()) < 0.3
    for l in range(2):
        _check_bert_layer_taps(gc, taps, ot, l)
        gc.assert_within_ulp(a_ref[l], ot["a_ref"][l].reshape(2, -1), 1, f"A_R layer {l}")
    # unobserved run: the exact maximum comes from a pass of its own
    plain, _, _ = gc.run_forward(wl, with_taps=False)
    for l in range(2):
        assert (plain[l] == a_ref[l]).all(), l


def test_bert_layer_full_size(eg, gc, orc):
    """Config 4: BERT-base layer, batch 32 x seq 128, bf16 training activations."""
    wl = si.make_config(4)
    a_ref, taps, ref = gc.run_forward(wl)
    ot = orc.ref_forward(wl)
    _check_bert_layer_taps(gc, taps, ot, 0)
    gc.assert_within_ulp(a_ref[0], ot["a_ref"][0].reshape(32, -1), 1, "A_R")
    plain, _, _ = gc.run_forward(wl, with_taps=False)
    assert (plain[0] == a_ref[0]).all()
    a_t = si.train_forward(wl)
    assert a_t[0].dtype == torch.bfloat16
    ws = eg.workspace(eg.workspace_bytes(ref.desc))
    p = torch.zeros(1, dtype=torch.float32, device=gc.DEV)
    eg.plasticity_eval(ref, gc.to_dev(wl.x), [a_t[0].to(gc.DEV)], p, ws)
    want = orc.sp_loss(a_t[0].float().numpy(), ot["a_ref"][0])
    assert p_close(p.item(), want, 32), (p.item(), want)


class _Cfg5Chain:
    """Config 5 at full size (12 layers, batch 64 x seq 256): the GPU runs once (an observed run that
    keeps the int8 input and the scale of all 48 GEMMs, an unobserved run - the one the benchmark
    times - and the fused forward + scores call); the oracle chain is advanced one layer per test."""

    def __init__(self, eg, gc, orc):
        import ctypes
        self.wl = wl = si.make_config(5)
        self.n, self.b, self.D = 12, wl.batch, 256 * 768
        n, b, D = self.n, self.b, self.D
        ref = gc.build_reference(wl)
        x = gc.to_dev(wl.x)
        ws = eg.workspace(eg.workspace_bytes(ref.desc))
        # observation points: codes and scales only (accumulators and outputs follow from them)
        shapes = gc.tap_shapes(wl)
        arr = (eg.Tap * len(shapes))()
        self.xq, self.sx = [], []
        for i, sh in enumerate(shapes):
            q = torch.zeros((sh["M"], sh["kp"]), dtype=torch.int8, device=gc.DEV)
            sc = torch.zeros(1, dtype=torch.float32, device=gc.DEV)
            arr[i].x_q, arr[i].x_scale, arr[i].acc, arr[i].y = q.data_ptr(), sc.data_ptr(), None, None
            self.xq.append(q)
            self.sx.append(sc)
        taps = eg.Taps()
        taps.n, taps.tap = len(shapes), arr
        self.a_obs = torch.empty((n, b, D), dtype=torch.float32, device=gc.DEV)
        eg.ref_forward(ref, x, self.a_obs, ws, taps)
        torch.cuda.synchronize()
        assert eg.check(ws) == eg.OK
        self.a_ref = torch.empty((n, b, D), dtype=torch.float32, device=gc.DEV)
        eg.ref_forward(ref, x, self.a_ref, ws)
        torch.cuda.synchronize()
        assert eg.check(ws) == eg.OK
        self.a_t = si.train_forward(wl, device=gc.DEV)
        self.p = torch.zeros(n, dtype=torch.float32, device=gc.DEV)
        eg.plasticity_eval(ref, x, self.a_t, self.p, ws)
        torch.cuda.synchronize()
        self.qw = orc.quantize_weights(wl.weights)
        self.cur = wl.x                     # input of the oracle's next layer
        self.next_layer = 0
        self.ulp_diffs = []


@pytest.fixture(scope="module")
def cfg5(eg, gc, orc):
    return _Cfg5Chain(eg, gc, orc)


@pytest.mark.parametrize("l", list(range(12)))
def test_bert_stack_full_size(eg, gc, orc, cfg5, l):
    """Config 5, layer l of 12 at batch 64 x seq 256, against the oracle chain run to that depth: the
    int8 input and scale of each of the layer's four GEMMs bit for bit, A_R within one fp32 ulp (the
    number of differing elements is printed), the unobserved run equal to the observed one, and the
    layer's score from the fused call within tolerance of the fp64 metric on the oracle's activations."""
    c = cfg5
    assert c.next_layer == l, "the layers of the chain are tested in order"
    d = c.wl.dims
    taps = {}
    out, _ = orc.bert_layer(c.cur, c.qw[4 * l:4 * l + 4], c.wl.biases[4 * l:4 * l + 4], d["heads"], d["ln_eps"], taps, "")
    for i in range(4):
        assert c.sx[4 * l + i].item() == taps[f"l{i}.sx"], (l, i)
        gc.assert_int8_rows(c.xq[4 * l + i].cpu().numpy(), taps[f"l{i}.xq"])
    got = c.a_obs[l].cpu().numpy()
    ndiff = gc.assert_within_ulp(got, out.reshape(c.b, -1), 1, f"A_R layer {l}")
    c.ulp_diffs.append(ndiff)
    assert torch.equal(c.a_ref[l], c.a_obs[l])
    # every token row is layer-normalised (gamma 1, beta 0)
    rows = c.a_ref[l].reshape(-1, 768)
    assert rows.mean(-1).abs().max().item() < 1e-5
    assert (rows.var(-1, unbiased=False) - 1).abs().max().item() < 1e-4
    want = orc.sp_loss(c.a_t[l].cpu().numpy(), out)
    assert p_close(c.p[l].item(), want, c.b), (l, c.p[l].item(), want)
    assert eg.plasticity(c.a_t[l], c.a_ref[l]).item() == c.p[l].item()
    c.cur = out
    c.next_layer = l + 1
    if l == 11:
        print("cfg5 A_R elements that differ from the oracle by one ulp, per layer:", c.ulp_diffs)


PER_CHANNEL_CASES = [("fc", dict(b=5, k=100, n=7)), ("fc", dict(b=130, k=200, n=257)),
                     ("basic", dict(b=2, c=20, h=9, w=11)), ("basic", dict(b=5, c=16, h=32, w=32)),
                     ("bottleneck", dict(b=1, c_in=40, c_mid=24, h=7, w=3)),
                     ("bottleneck", dict(b=3, c_in=256, c_mid=64, h=14, w=14)),
                     ("bert", dict(b=3, s=40, hidden=128, heads=4, ffn=200, n_layers=2))]


@pytest.mark.parametrize("kind,kw", PER_CHANNEL_CASES,
                         ids=lambda v: v if isinstance(v, str) else "_".join(f"{k}{x}" for k, x in v.items()))
def test_per_channel_weights_bit_exact(eg, gc, orc, kind, kw):
    """Weights quantised with one scale per output channel: the library's codes and scales, every
    observation point of the forward and the score agree with the oracle."""
    if kind == "bert":
        wl, conv = si.make_bert(seed=740, train_act_dtype="f32", **kw), False
    else:
        wl, conv = _static_workload(kind, kw)
    # channels of very different magnitude, so that one scale per tensor would not do
    rng = np.random.default_rng(9)
    wl.weights = [(w * np.exp(rng.uniform(-2, 2, size=(w.shape[0],) + (1,) * (w.ndim - 1)))).astype(np.float32)
                  for w in wl.weights]
    W = [gc.to_dev(w) for w in wl.weights]
    B = [None if b is None else gc.to_dev(b) for b in wl.biases]
    ref = eg.make_reference(wl.kind, wl.dims, W, B, None, per_channel=True)
    oqw = orc.quantize_weights(wl.weights, per_channel=True)
    for (wq, sw), q, s_ in zip(oqw, ref.w_q, ref.scales):
        assert np.array_equal(s_.cpu().numpy(), sw)
        if wq.ndim == 4:
            gc.assert_conv_q(q.cpu().numpy().reshape(-1, q.shape[-1]), wq)
        else:
            gc.assert_int8_rows(q.cpu().numpy(), wq)
    ot = orc.ref_forward(wl, oqw)
    x = gc.to_dev(wl.x)
    n_layers = wl.dims.get("n_layers", 1)
    a_ref = torch.empty(gc.a_ref_numel(wl), dtype=torch.float32, device=gc.DEV)
    ws = eg.workspace(eg.workspace_bytes(ref.desc), gc.DEV)
    taps, bufs, _keep = eg.make_taps(ref, gc.tap_shapes(wl), gc.DEV)
    eg.ref_forward(ref, x, a_ref, ws, taps)
    torch.cuda.synchronize()
    assert eg.check(ws) == eg.OK
    got = a_ref.cpu().numpy().reshape(n_layers, wl.batch, -1)
    if kind == "bert":
        for l in range(n_layers):
            assert np.array_equal(got[l], np.asarray(ot["a_ref"][l]).reshape(wl.batch, -1))
            _check_bert_layer_taps(gc, [{k: v.cpu().numpy() for k, v in b.items()} for b in bufs], ot, l)
        # unobserved run (per-column scales in the GELU-fused passes of the first feed-forward layer)
        plain = torch.empty_like(a_ref)
        eg.ref_forward(ref, x, plain, ws)
        torch.cuda.synchronize()
        assert np.array_equal(plain.cpu().numpy().reshape(n_layers, wl.batch, -1), got)
    else:
        for i in range(len(bufs)):
            _check_linear_taps(gc, {k: v.cpu().numpy() for k, v in bufs[i].items()}, ot, f"l{i}.", conv=conv)
        want = gc.nhwc(ot["a_ref"]).reshape(wl.batch, -1) if conv else ot["a_ref"]
        assert np.array_equal(got[0], want)
        # unobserved run (narrow basic blocks quantise inside the convolutions there)
        plain = torch.empty_like(a_ref)
        eg.ref_forward(ref, x, plain, ws)
        torch.cuda.synchronize()
        assert np.array_equal(plain.cpu().numpy().reshape(wl.batch, -1), want)


# --------------------------------------------------------------------------- refresh + evaluation in one call
def _refresh_workload(name):
    if name == "fc_small":
        return si.make_fc(seed=811, b=5, k=100, n=7)
    if name == "fc":
        return si.make_fc(seed=812, b=120, k=200, n=257)
    if name == "basic_narrow":
        return si.make_basic_block(seed=813, b=3, c=16, h=9, w=11)
    if name == "basic_wide":
        return si.make_basic_block(seed=814, b=2, c=20, h=9, w=11)
    if name == "bottleneck":
        return si.make_bottleneck(seed=815, b=3, c_in=256, c_mid=64, h=14, w=14)
    if name == "bottleneck_odd":
        return si.make_bottleneck(seed=817, b=2, c_in=256, c_mid=64, h=7, w=7)
    if name == "basic_wide64":
        return si.make_basic_block(seed=818, b=2, c=64, h=16, w=12)
    return si.make_bert(seed=816, b=3, s=40, hidden=128, heads=4, ffn=200, n_layers=2, train_act_dtype="f32")


@pytest.mark.parametrize("name", ["fc_small", "fc", "basic_narrow", "basic_wide", "basic_wide64", "bottleneck",
                                  "bottleneck_odd", "bert"])
@pytest.mark.parametrize("mode", ["dynamic", "static", "per_channel", "bf16_x"])
def test_refresh_eval_equals_two_calls(eg, gc, orc, name, mode):
    """egeria_refresh_eval against egeria_quantize_weights + egeria_plasticity_eval: the same codes, scales and
    scores bit for bit (the mini-batch's maximum pass rides in the snapshot's first launch), and the
    oracle's score."""
    from paper_2201_06227_amd.evaluator import PlasticityEvaluator
    if name == "bert" and mode in ("static", "bf16_x"):
        pytest.skip("the Transformer kinds take dynamic scales and an fp32 mini-batch")
    wl = _refresh_workload(name)
    if mode == "bf16_x":
        wl.x = torch.from_numpy(wl.x).to(torch.bfloat16).float().numpy()
    ot = orc.ref_forward(wl)
    scales = None
    if mode == "static":
        scales = gc.to_dev(np.asarray([float(ot[f"l{i}.sx"]) for i in range(len(wl.weights))], np.float32))
    W = [gc.to_dev(w) for w in wl.weights]
    B = [None if b is None else gc.to_dev(b) for b in wl.biases]
    ev = PlasticityEvaluator(wl.kind, wl.dims, W, B, device=gc.DEV, act_scales=scales,
                             per_channel=(mode == "per_channel"))
    x = gc.to_dev(wl.x, torch.bfloat16 if mode == "bf16_x" else None)
    a_t = [t.to(gc.DEV).contiguous() for t in si.train_forward(wl)]
    p2 = ev.step_two_calls(x, a_t).clone()
    torch.cuda.synchronize()
    q2 = [q.clone() for q in ev.w_q]
    s2 = [v.clone() for v in ev.scales]
    for t in ev.w_q + ev.scales:
        t.zero_()
    ev.p_out.zero_()
    for rep in range(2):                                   # the second call finds the workspaces used
        p1 = ev.step(x, a_t).clone()
        torch.cuda.synchronize()
        assert eg.check(ev.ws) == eg.OK and eg.check(ev.qws) == eg.OK
        assert torch.equal(p1, p2), (rep, p1, p2)
        for a, b in zip(ev.w_q + ev.scales, q2 + s2):
            assert torch.equal(a, b)
    if mode in ("dynamic", "bf16_x"):
        a_ref = ot["a_ref"]
        if wl.kind in (si.KIND_BASIC_BLOCK, si.KIND_BOTTLENECK):
            a_ref = [gc.nhwc(a_ref).reshape(wl.batch, -1)]
        elif wl.kind == si.KIND_FC_RELU:
            a_ref = [a_ref]
        for l, t in enumerate(a_t):
            want = orc.sp_loss(t.float().cpu().numpy().reshape(wl.batch, -1), np.asarray(a_ref[l]).reshape(wl.batch, -1))
            assert p_close(p1[l].item(), want, wl.batch), (l, p1[l].item(), want)

