"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle.

Integer outputs (canonical supports, coverage mask, uncovered list and count,
the first bad expert) must match bit for bit.  Float outputs must satisfy

* descriptor d:  |d - d_ref| <= 1e-5 * mean|x| over the plane;
* temperature:   |tau - tau_ref| <= 1e-5 * tau_ref;
* coefficients:  |alpha - alpha_ref| <= 1e-5 * max_i alpha_ref (per row);
* outputs y:     |y - y_ref| <= rtol * M, M = sum_i alpha_i |x_i| (the oracle's
  magnitude), rtol = 1e-5 for float32 and 1e-2 for bfloat16 outputs; bfloat16
  outputs must in addition be within one rounding of the float32 result,
  |y - y_ref| <= 2^-8 |y_ref| + 1e-5 * M.

Inputs come from the seeded workload generator; nothing the GPU computes is
ever fed to the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_23794_amd import binding as mb
from paper_2608_23794_amd import inputs
from paper_2608_23794_amd.layer import MoceLayer, to_device_x, to_host_f64

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

CASES = [("tiny", "nchw"), ("tiny", "nhwc"), ("resnet50_stage1", "nchw"), ("resnet50_stage3", "nchw"),
         ("resnet50_stage3", "nhwc"), ("resnet50_stage4", "nhwc"), ("vit_tokens", "nhwc")]
OL = {"nchw": oracle.NCHW, "nhwc": oracle.NHWC}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    mb.load()
    yield
    torch.cuda.synchronize()


_cache = {}


def workload(name, layout):
    key = (name, layout)
    if key not in _cache:
        wl = inputs.WORKLOADS[name]
        g = inputs.generate(wl, layout)
        ref = oracle.forward(g["x"], g["s"], g["w"], wl.E, OL[layout], a=g["a"], c=g["c"])
        _cache.clear()
        _cache[key] = (wl, g, ref)
    return _cache[key]


def abs_mean(x, layout):
    if x.dtype == np.uint16:
        x = x & np.uint16(0x7FFF)
    else:
        x = np.abs(x)
    return oracle.pool(x, OL[layout])


def check_d(d, d_ref, scale):
    err = np.abs(d - d_ref) / np.maximum(scale, 1e-30)
    assert err.max() <= 1e-5, f"d: max normalised error {err.max():.3e}"


def check_tau_alpha(tau, tau_ref, alpha=None, alpha_ref=None):
    e = np.abs(tau - tau_ref) / tau_ref
    assert e.max() <= 1e-5, f"tau: max relative error {e.max():.3e}"
    if alpha is not None:
        rowmax = alpha_ref.max(axis=-1, keepdims=True)
        ea = np.abs(alpha - alpha_ref) / rowmax
        assert ea.max() <= 1e-5, f"alpha: max normalised error {ea.max():.3e}"


def check_y(y, y_ref, mag, dtype):
    tiny = 1e-30
    err = np.abs(y - y_ref)
    rtol = 1e-5 if dtype == "f32" else 1e-2
    norm = err / np.maximum(mag, tiny)
    worst = np.unravel_index(np.argmax(norm), norm.shape)
    assert norm.max() <= rtol, f"y: max error/M {norm.max():.3e} at {worst}"
    if dtype == "bf16":
        bound = 2.0 ** -8 * np.abs(y_ref) + 1e-5 * mag + tiny
        assert np.all(err <= bound), f"y: {int((err > bound).sum())} outputs beyond one bf16 rounding"
    return float(norm.max())


# --------------------------------------------------------------------------- prepare

@pytest.mark.parametrize("name,layout", [CASES[i] for i in (0, 2, 3, 5, 6)])
def test_prepare_bit_exact(name, layout):
    wl, g, ref = workload(name, layout)
    layer = MoceLayer.from_workload(wl, g, layout)
    assert layer.status == 0 and layer.bad_expert == -1
    torch.cuda.synchronize()
    assert np.array_equal(layer.s_c.cpu().numpy(), ref["s"])
    assert np.array_equal(layer.w_c.cpu().numpy().view(np.uint32), ref["w"].view(np.uint32))
    assert np.array_equal(layer.covered.cpu().numpy(), ref["covered"])
    assert layer.nU == ref["nU"]
    assert np.array_equal(layer.U.cpu().numpy()[:layer.nU], ref["U"])
    assert layer.info.cpu().numpy().tolist() == [ref["nU"], -1]
    if name == "resnet50_stage3":
        assert layer.nU == 51


@pytest.mark.parametrize("C,E,k", [(64, 16, 8), (100, 7, 13), (32, 32, 32), (17, 3, 5), (64, 1, 4),
                                   (1000, 3, 1000), (5000, 9, 700)])
def test_prepare_cyclic_and_ties(C, E, k):
    rng = np.random.default_rng(C + E + k)
    R = E - 1
    s = np.array([[(e * k + j) % C for j in range(k)] for e in range(R)], np.int32).reshape(R, k)
    w = np.round(rng.standard_normal((R, k)) * 2).astype(np.float32)  # many ties
    w[:, ::7] = -0.0
    s_ref, w_ref, cov_ref, U_ref, nU_ref = oracle.prepare(C, E, s, w)
    layer = MoceLayer(C, E, k, 1, 1, "f32", "nchw", s, w, a=np.zeros((R, k)), c=np.zeros(R))
    assert layer.status == 0
    assert np.array_equal(layer.s_c.cpu().numpy(), s_ref)
    assert np.array_equal(layer.w_c.cpu().numpy().view(np.uint32), w_ref.view(np.uint32))
    assert np.array_equal(layer.covered.cpu().numpy(), cov_ref)
    assert layer.nU == nU_ref and np.array_equal(layer.U.cpu().numpy()[:nU_ref], U_ref)


@pytest.mark.parametrize("bad", ["dup", "neg", "range", "nan", "inf", "two_rows"])
def test_prepare_rejects_invalid_rows_like_the_oracle(bad):
    rng = np.random.default_rng(4)
    C, E, k = 300, 40, 24
    R = E - 1
    s = np.array([rng.choice(C, k, replace=False) for _ in range(R)], np.int32)
    w = rng.standard_normal((R, k)).astype(np.float32)
    o = 17
    if bad == "dup":
        s[o, 20] = s[o, 3]
    elif bad == "neg":
        s[o, 5] = -7
    elif bad == "range":
        s[o, 0] = C
    elif bad == "nan":
        w[o, 9] = np.nan
    elif bad == "inf":
        w[o, 9] = np.inf
    else:
        s[30, 1] = s[30, 2]
        s[o, 4] = C + 5
    with pytest.raises(oracle.SupportError) as ei:
        oracle.prepare(C, E, s, w)
    with pytest.raises(mb.MoceError):
        MoceLayer(C, E, k, 2, 2, "f32", "nchw", s, w, a=np.zeros((R, k)), c=np.zeros(R))
    layer = MoceLayer(C, E, k, 2, 2, "f32", "nchw", s, w, a=np.zeros((R, k)), c=np.zeros(R), allow_invalid=True)
    assert layer.status == -5
    assert layer.bad_expert == ei.value.expert == o
    with pytest.raises(mb.MoceError):  # an invalid layer refuses to run
        layer.forward(torch.zeros((1, C, 2, 2), dtype=torch.float32, device="cuda"))


# --------------------------------------------------------------------------- pool / gate / mix

@pytest.mark.parametrize("name,layout", CASES)
def test_pool(name, layout):
    wl, g, ref = workload(name, layout)
    layer = MoceLayer.from_workload(wl, g, layout)
    x = to_device_x(g["x"], wl.dtype)
    d = layer.pool(x).cpu().numpy().astype(np.float64)
    check_d(d, ref["d"], abs_mean(g["x"], layout))


@pytest.mark.parametrize("name", ["tiny", "resnet50_stage1", "resnet50_stage3", "resnet50_stage4", "vit_tokens"])
def test_gate_softplus_isolated(name):
    wl = inputs.WORKLOADS[name]
    g = inputs.generate(wl, with_x=False)
    d = inputs.random_descriptor(wl.B, wl.C, seed=wl.seed, signed=wl.signed)
    s_c, w_c, _, _, _ = oracle.prepare(wl.C, wl.E, g["s"], g["w"])
    tau_ref = oracle.gate_softplus(d, s_c, g["a"], g["c"])
    alpha_ref = oracle.softmax(w_c, tau_ref)
    layer = MoceLayer.from_workload(wl, g)
    tau, alpha = layer.gate_tau(torch.from_numpy(d).cuda())
    check_tau_alpha(tau.cpu().numpy(), tau_ref, alpha.cpu().numpy(), alpha_ref)


@pytest.mark.parametrize("name", ["tiny", "resnet50_stage1", "resnet50_stage3", "resnet50_stage4", "vit_tokens"])
def test_gate_mlp_isolated(name):
    wl = inputs.WORKLOADS[name]
    g = inputs.generate(wl, with_x=False)
    d = inputs.random_descriptor(wl.B, wl.C, seed=wl.seed + 100)
    s_c, w_c, _, _, _ = oracle.prepare(wl.C, wl.E, g["s"], g["w"])
    tau_ref = oracle.gate_mlp(d, s_c, g["W1"], g["b1"], g["w2"], g["b2"], g["tau_min"], g["tau_max"])
    alpha_ref = oracle.softmax(w_c, tau_ref)
    layer = MoceLayer.from_workload(wl, g, gate="mlp")
    tau, alpha = layer.gate_tau(torch.from_numpy(d).cuda())
    tau = tau.cpu().numpy()
    assert np.all(tau >= float(g["tau_min"])) and np.all(tau <= float(g["tau_max"]))
    check_tau_alpha(tau, tau_ref, alpha.cpu().numpy(), alpha_ref)


@pytest.mark.parametrize("B,C,E,k", [
    (301, 300, 257, 40),   # two 128-expert blocks, two images per workgroup, a ragged last group, k padded to 64
    (7, 160, 130, 32),     # R = 129: a block with one expert
    (3, 256, 9, 128),      # k = 128 exactly, one block of 8 experts
    (2, 300, 5, 129),      # k > 128: the per-wave kernel
    (1, 40, 2, 1),         # one routed expert, k = 1
])
def test_gate_mlp_shapes(B, C, E, k):
    """The batched MLP gate against the oracle off the workload shapes: several images per
    workgroup with a ragged last group, partial expert blocks, k padded to the next 32 and the
    fallback beyond k = 128."""
    rng = np.random.default_rng(B * 1000 + k)
    R = E - 1
    s = np.array([rng.choice(C, k, replace=False) for _ in range(R)], np.int32).reshape(R, k)
    w = rng.standard_normal((R, k)).astype(np.float32)
    W1 = (rng.standard_normal((k, k)) * k ** -0.5).astype(np.float32)
    b1 = (rng.standard_normal(k) * 0.1).astype(np.float32)
    w2 = (rng.standard_normal(k) * k ** -0.5).astype(np.float32)
    b2, tmin, tmax = np.float32(0.25), np.float32(0.2), np.float32(6.0)
    d = inputs.random_descriptor(B, C, seed=k + 11)
    s_c, w_c, _, _, _ = oracle.prepare(C, E, s, w)
    tau_ref = oracle.gate_mlp(d, s_c, W1, b1, w2, b2, tmin, tmax)
    alpha_ref = oracle.softmax(w_c, tau_ref)
    layer = MoceLayer(C, E, k, 1, 1, "f32", "nchw", s, w, gate="mlp", W1=W1, b1=b1, w2=w2, b2=float(b2),
                      tau_min=float(tmin), tau_max=float(tmax))
    tau, alpha = layer.gate_tau(torch.from_numpy(d).cuda())
    check_tau_alpha(tau.cpu().numpy(), tau_ref, alpha.cpu().numpy(), alpha_ref)


@pytest.mark.parametrize("name,layout", CASES)
def test_mix_with_given_coefficients(name, layout):
    wl, g, ref = workload(name, layout)
    alpha32 = ref["alpha"].astype(np.float32)
    y_ref, mag = oracle.mix(g["x"], ref["s"], alpha32.astype(np.float64), ref["U"], wl.E, OL[layout])
    layer = MoceLayer.from_workload(wl, g, layout)
    y = layer.mix(to_device_x(g["x"], wl.dtype), torch.from_numpy(alpha32).cuda())
    check_y(to_host_f64(y), y_ref, mag, wl.dtype)


@pytest.mark.parametrize("name,layout", CASES)
def test_forward(name, layout):
    wl, g, ref = workload(name, layout)
    layer = MoceLayer.from_workload(wl, g, layout)
    x = to_device_x(g["x"], wl.dtype)
    y = layer.forward(x)
    e = check_y(to_host_f64(y), ref["y"], ref["mag"], wl.dtype)
    print(f"{name}/{layout}: max |y - y_ref| / M = {e:.3e}")


@pytest.mark.parametrize("name,layout", [("tiny", "nchw"), ("resnet50_stage3", "nchw"), ("resnet50_stage3", "nhwc"),
                                         ("resnet50_stage4", "nhwc"), ("vit_tokens", "nhwc")])
def test_forward_mlp_gate(name, layout):
    wl = inputs.WORKLOADS[name]
    g = inputs.generate(wl, layout)
    ref = oracle.forward(g["x"], g["s"], g["w"], wl.E, OL[layout], gate="mlp", W1=g["W1"], b1=g["b1"],
                         w2=g["w2"], b2=g["b2"], tau_min=g["tau_min"], tau_max=g["tau_max"])
    layer = MoceLayer.from_workload(wl, g, layout, gate="mlp")
    y = layer.forward(to_device_x(g["x"], wl.dtype))
    check_y(to_host_f64(y), ref["y"], ref["mag"], wl.dtype)


def test_forward_mlp_gate_mfma_path():
    """The MLP gate on the stage-1 shape: plane-wise pooling, the gate kernel, then the MFMA mix."""
    wl = inputs.WORKLOADS["resnet50_stage1"]
    g = inputs.generate(wl, batch=5)
    ref = oracle.forward(g["x"], g["s"], g["w"], wl.E, oracle.NCHW, gate="mlp", W1=g["W1"], b1=g["b1"],
                         w2=g["w2"], b2=g["b2"], tau_min=g["tau_min"], tau_max=g["tau_max"])
    layer = MoceLayer.from_workload(wl, g, gate="mlp")
    assert mb.moce_forward_path(layer.desc(5), mb.MOCE_GATE_MLP_SIGMOID) == mb.PATH_MFMA
    y = layer.forward(to_device_x(g["x"], wl.dtype))
    check_y(to_host_f64(y), ref["y"], ref["mag"], wl.dtype)


# --------------------------------------------------------------------------- edge cases

def _custom(B, C, E, k, H, W, dtype, layout, seed, signed=False, cyclic=False, s=None, w=None):
    rng = np.random.default_rng(seed)
    R = E - 1
    if s is None:
        if cyclic:
            s = np.array([[(e * k + j) % C for j in range(k)] for e in range(R)], np.int32).reshape(R, k)
        else:
            s = np.array([rng.choice(C, k, replace=False) for _ in range(R)], np.int32).reshape(R, k)
    if w is None:
        w = rng.standard_normal((R, k)).astype(np.float32)
    a = (rng.standard_normal((R, k)) * k ** -0.5).astype(np.float32)
    c = rng.standard_normal(R).astype(np.float32) * np.float32(0.5)
    shape = (B, C, H, W) if layout == "nchw" else (B, H, W, C)
    x = rng.standard_normal(shape).astype(np.float32)
    if not signed:
        x = np.maximum(x, 0)
    if dtype == "bf16":
        x = inputs.f32_to_bf16_bits(x)
    return x, s, w, a, c


EDGE = [
    # B, C, E, k, H, W, dtype, layout, extra
    (3, 64, 1, 4, 5, 9, "f32", "nchw", {}),            # no routed expert: y = mean over all channels
    (2, 96, 13, 8, 7, 7, "bf16", "nchw", dict(cyclic=True)),  # |U| = 0 exactly, ragged 2-byte rows
    (2, 40, 9, 1, 3, 11, "bf16", "nchw", {}),          # k = 1
    (1, 24, 24, 24, 13, 5, "f32", "nchw", {}),         # E = C = k
    (5, 200, 30, 17, 10, 10, "bf16", "nchw", dict(signed=True)),  # 8-byte rows, tail tile
    (2, 50, 11, 7, 1, 1, "bf16", "nchw", {}),          # one position
    (2, 700, 40, 20, 6, 6, "f32", "nchw", {}),         # tile beyond LDS: global-memory path
    (3, 60, 10, 6, 5, 7, "bf16", "nhwc", {}),          # C*2 not a multiple of 16: scalar pooling
    (2, 6000, 30, 40, 3, 3, "bf16", "nhwc", {}),        # tile beyond LDS: global-memory path
    (2, 3000, 30, 40, 3, 3, "bf16", "nhwc", {}),        # 16-position tile beyond LDS: 8 positions
    (2, 512, 8, 200, 4, 4, "bf16", "nhwc", {}),         # gate with 128 < k <= 256: four positions per lane
    (1, 600, 4, 300, 2, 2, "f32", "nchw", {}),          # gate with k > 256: the looping kernel
    (4, 72, 9, 9, 9, 1, "f32", "nhwc", dict(signed=True)),
    (1, 2048, 512, 128, 1, 1, "bf16", "nhwc", {}),      # single token
]


@pytest.mark.parametrize("B,C,E,k,H,W,dtype,layout,extra", EDGE)
def test_forward_edge_cases(B, C, E, k, H, W, dtype, layout, extra):
    x, s, w, a, c = _custom(B, C, E, k, H, W, dtype, layout, seed=B * 1000 + C + E + k, **extra)
    ref = oracle.forward(x, s, w, E, OL[layout], a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, dtype, layout, s, w, a=a, c=c)
    assert layer.nU == ref["nU"]
    y = to_host_f64(layer.forward(to_device_x(x, dtype)))
    check_y(y, ref["y"], ref["mag"], dtype)
    res = y[:, E - 1] if layout == "nchw" else y[..., E - 1]
    if ref["nU"] == 0:
        assert np.all(res == 0.0)
    if k == 1:  # a single channel per expert is copied exactly, even in bf16
        routed = y[:, :E - 1] if layout == "nchw" else y[..., :E - 1]
        rr = ref["y"][:, :E - 1] if layout == "nchw" else ref["y"][..., :E - 1]
        assert np.array_equal(routed, rr)


@pytest.mark.parametrize("dtype,layout", [("bf16", "nchw"), ("f32", "nchw"), ("bf16", "nhwc"), ("f32", "nhwc")])
def test_one_hot_limit_is_an_exact_copy(dtype, layout):
    """tau at its floor (c = -1e4) with a clear top logit: every routed output is an exact copy of its
    top channel, in every layout and element type (the coefficients are exactly 1 and 0)."""
    B, C, E, k, H, W = 2, 80, 12, 6, 8, 8
    x, s, w, a, c = _custom(B, C, E, k, H, W, dtype, layout, seed=77, signed=True)
    w[:, 0] = w.max(axis=1) + 1.0       # a clear top logit
    a[:] = 0.0
    c[:] = -1e4                          # tau = 1e-3
    ref = oracle.forward(x, s, w, E, OL[layout], a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, dtype, layout, s, w, a=a, c=c)
    y = to_host_f64(layer.forward(to_device_x(x, dtype)))
    routed = (lambda t: t[:, :E - 1]) if layout == "nchw" else (lambda t: t[..., :E - 1])
    assert np.array_equal(routed(y), routed(ref["y"]))


@pytest.mark.parametrize("dtype,layout", [("f32", "nhwc"), ("bf16", "nhwc"), ("f32", "nchw")])
def test_forward_low_temperature_mlp_gate(dtype, layout):
    """The paper's gate with a low temperature floor (tau_min = 0.01, g pushed negative): the
    coefficients are near one-hot, where rebuilding them from the softmax statistics must not lose
    precision against the oracle."""
    B, C, E, k, H, W = 3, 96, 20, 12, 6, 6
    x, s, w, a, c = _custom(B, C, E, k, H, W, dtype, layout, seed=5, signed=True)
    rng = np.random.default_rng(6)
    W1 = (rng.standard_normal((k, k)) * k ** -0.5).astype(np.float32)
    b1 = (rng.standard_normal(k) * 0.1).astype(np.float32)
    w2 = (rng.standard_normal(k) * k ** -0.5).astype(np.float32)
    b2 = np.float32(-12.0)
    ref = oracle.forward(x, s, w, E, OL[layout], gate="mlp", W1=W1, b1=b1, w2=w2, b2=b2, tau_min=0.01,
                         tau_max=6.0)
    assert ref["tau"].max() < 0.02
    layer = MoceLayer(C, E, k, H, W, dtype, layout, s, w, gate="mlp", W1=W1, b1=b1, w2=w2, b2=b2,
                      tau_min=0.01, tau_max=6.0)
    xd = to_device_x(x, dtype)
    tau, alpha = layer.gate_tau(layer.pool(xd))
    check_tau_alpha(tau.cpu().numpy(), ref["tau"], alpha.cpu().numpy(), ref["alpha"])
    check_y(to_host_f64(layer.forward(xd)), ref["y"], ref["mag"], dtype)


GENERIC_STAGES = [
    # B, C, E, k, H, W, dtype, layout: the generic kernels, where the forward rebuilds the
    # coefficients from the softmax statistics instead of reading them
    (4, 96, 20, 20, 6, 6, "bf16", "nhwc"),
    (2, 64, 16, 8, 8, 8, "f32", "nchw"),
    (3, 64, 16, 8, 8, 8, "f32", "nhwc"),
    (2, 300, 40, 70, 5, 5, "bf16", "nhwc"),
]


@pytest.mark.parametrize("B,C,E,k,H,W,dtype,layout", GENERIC_STAGES)
def test_generic_forward_equals_stages(B, C, E, k, H, W, dtype, layout):
    """The forward's rebuilt coefficients equal those moce_gate writes, bit for bit, so the forward
    and pool + gate + mix agree bit for bit."""
    x, s, w, a, c = _custom(B, C, E, k, H, W, dtype, layout, seed=B * 7 + k, signed=True)
    layer = MoceLayer(C, E, k, H, W, dtype, layout, s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == mb.PATH_GENERIC
    xd = to_device_x(x, dtype)
    y = layer.forward(xd)
    _, alpha = layer.gate_tau(layer.pool(xd))
    y_st = layer.mix(xd, alpha)
    torch.cuda.synchronize()
    iv = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(y.view(iv), y_st.view(iv))


@pytest.mark.parametrize("k", [1, 3, 4, 15, 16, 17, 23, 37])
@pytest.mark.parametrize("dtype,layout", [("f32", "nchw"), ("f32", "nhwc"), ("bf16", "nchw")])
def test_generic_mix_entry_rounds(dtype, layout, k):
    """Supports of one entry up to past two rounds of sixteen and their remainders."""
    B, C, E, H, W = 2, 76, 19, 5, 7
    x, s, w, a, c = _custom(B, C, E, k, H, W, dtype, layout, seed=k, signed=True)
    layer = MoceLayer(C, E, k, H, W, dtype, layout, s, w, a=a, c=c)
    ref = oracle.forward(x, s, w, E, OL[layout], a=a, c=c)
    check_y(to_host_f64(layer.forward(to_device_x(x, dtype))), ref["y"], ref["mag"], dtype)


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_forward_deterministic_and_fully_written(layout):
    wl = inputs.WORKLOADS["resnet50_stage3"]
    g = inputs.generate(wl, layout, batch=8)
    layer = MoceLayer.from_workload(wl, g, layout)
    x = to_device_x(g["x"], wl.dtype)
    shape = layer.y_shape(8)
    n = int(np.prod(shape))
    guard = 4096
    buf = torch.full((n + 2 * guard,), float("nan"), dtype=torch.bfloat16, device="cuda")
    y = buf[guard:guard + n].view(shape)
    layer.forward(x, y)
    torch.cuda.synchronize()
    first = y.clone()
    assert not torch.isnan(first).any(), "some outputs were not written"
    assert torch.isnan(buf[:guard]).all() and torch.isnan(buf[guard + n:]).all(), "write outside y"
    layer.forward(x, y)
    assert torch.equal(first.view(torch.int16), y.view(torch.int16)), "forward is not deterministic"


def test_batch_prefix_consistency():
    """Images are independent: the first images of a batch do not depend on the rest."""
    wl = inputs.WORKLOADS["resnet50_stage1"]
    g = inputs.generate(wl, batch=6)
    layer = MoceLayer.from_workload(wl, g)
    x = to_device_x(g["x"], wl.dtype)
    full = layer.forward(x)
    part = layer.forward(x[:2].contiguous())
    assert torch.equal(full[:2].view(torch.int16), part.view(torch.int16))


# --------------------------------------------------------------------------- MFMA mix (NCHW bf16)
MFMA = [
    # B, C, E, k, H, W: shapes served by the dense matrix-core mix
    (3, 256, 64, 32, 56, 56),    # a few images
    (24, 256, 64, 32, 56, 56),   # several images per workgroup range (rebuilds of A_b mid-range)
    (8, 128, 32, 16, 10, 20),    # 200 positions: four tiles, the last ragged (8 positions); E = 32
    (5, 64, 64, 64, 16, 24),     # E = C = k
    (4, 96, 24, 12, 28, 30),     # three load rounds, ragged last tile, half the expert waves idle
    (2, 256, 8, 256, 16, 16),    # k = C
    (2, 64, 16, 8, 128, 128),    # 256 tiles per image
    (2, 64, 2, 5, 8, 8),         # one routed expert, k not a multiple of 4
    (3, 256, 64, 64, 8, 8),      # R k = 4032 coefficients: more than the register prefetch holds
    (2, 32, 32, 3, 4, 6),        # C = 32 (one load round), fewer tiles than CUs
    (2, 64, 40, 3, 4, 6),        # E above 32: the second expert half partly filled
    (1, 160, 40, 20, 2, 4),      # eight positions in a single partial tile
    (2, 192, 48, 9, 7, 8),
    (3, 224, 20, 30, 6, 12),
    (600, 64, 16, 2, 8, 8),      # one tile per image: a rebuild of A_b at every tile of a range
    (300, 32, 32, 1, 4, 16),     # k = 1
]


@pytest.mark.parametrize("B,C,E,k,H,W", MFMA)
def test_mfma_forward_shapes(B, C, E, k, H, W):
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nchw", seed=B + C + E + k + H, signed=(C % 64 == 32))
    ref = oracle.forward(x, s, w, E, oracle.NCHW, a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, "bf16", "nchw", s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == _mfma_path(k)
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    check_y(y, ref["y"], ref["mag"], "bf16")
    res = y[:, E - 1]
    if ref["nU"] == 0:
        assert np.all(res == 0.0)


def test_mfma_residual_only_uncovered():
    """Cyclic supports that leave exactly the top channels uncovered: the residual row is their mean."""
    B, C, E, k, H, W = 2, 64, 9, 6, 8, 8
    s = np.array([[(e * k + j) % 48 for j in range(k)] for e in range(E - 1)], np.int32)
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nchw", seed=5, s=s)
    ref = oracle.forward(x, s, w, E, oracle.NCHW, a=a, c=c)
    assert ref["nU"] == 16
    layer = MoceLayer(C, E, k, H, W, "bf16", "nchw", s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == mb.PATH_MFMA
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    check_y(y, ref["y"], ref["mag"], "bf16")


def test_mfma_exact_copies():
    """k = 1 and the one-hot limit give coefficients of exactly 1: the routed outputs are copies of
    channels, bit for bit, through the split-coefficient products."""
    B, C, E, H, W = 2, 64, 12, 8, 8
    x, s, w, a, c = _custom(B, C, E, 1, H, W, "bf16", "nchw", seed=91, signed=True)
    ref = oracle.forward(x, s, w, E, oracle.NCHW, a=a, c=c)
    layer = MoceLayer(C, E, 1, H, W, "bf16", "nchw", s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == mb.PATH_MFMA
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    assert np.array_equal(y[:, :E - 1], ref["y"][:, :E - 1])
    k = 6
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nchw", seed=77, signed=True)
    w[:, 0] = w.max(axis=1) + 1.0
    a[:] = 0.0
    c[:] = -1e4
    ref = oracle.forward(x, s, w, E, oracle.NCHW, a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, "bf16", "nchw", s, w, a=a, c=c)
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    assert np.array_equal(y[:, :E - 1], ref["y"][:, :E - 1])


# --------------------------------------------------------------------------- tile kernel (NCHW bf16)
TILED = [
    # B, C, E, k, H, W: shapes served by the tile gather kernel (C not a multiple of 32 or E > 64)
    (3, 200, 200, 4, 8, 8),      # E = C: 199 routed experts, seven passes, one tile per image
    (3, 240, 64, 32, 56, 56),    # stage-1 sized, C not a multiple of 32
    (8, 120, 32, 16, 10, 20),    # 200 positions: four tiles, the last ragged (8 positions)
    (5, 80, 80, 64, 16, 24),     # E = C, two expert passes
    (4, 88, 24, 12, 28, 30),     # ragged last tile
    (2, 256, 96, 16, 16, 16),    # E above the MFMA path's 64
    (2, 48, 2, 5, 8, 8),         # one routed expert, k not a multiple of 4
    (3, 200, 20, 40, 8, 16),     # 33 <= k <= 48: three register rows per expert, one expert pass
    (2, 200, 40, 45, 8, 8),      # three register rows, two expert passes
    (2, 168, 30, 56, 12, 12),    # 49 <= k <= 64: four register rows, one pass
    (2, 200, 50, 60, 8, 8),      # four register rows, two passes
]


@pytest.mark.parametrize("B,C,E,k,H,W", TILED)
def test_tile_forward_shapes(B, C, E, k, H, W):
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nchw", seed=B + C + E + k + H)
    ref = oracle.forward(x, s, w, E, oracle.NCHW, a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, "bf16", "nchw", s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == mb.PATH_TILE
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    check_y(y, ref["y"], ref["mag"], "bf16")


def test_forward_path_choice():
    """The MFMA mix where its limits allow, then the tile kernel, then the generic kernels."""
    def path(B, C, E, k, H, W, dtype="bf16", layout="nchw", gate=mb.MOCE_GATE_SOFTPLUS_LINEAR):
        d = mb.make_desc(B, C, H, W, E, k, mb.MOCE_BF16 if dtype == "bf16" else mb.MOCE_F32,
                         mb.MOCE_NCHW if layout == "nchw" else mb.MOCE_NHWC)
        return mb.moce_forward_path(d, gate)
    assert path(64, 256, 64, 32, 56, 56) == mb.PATH_MFMA_GATE     # k = 32: the gate inside the mix
    assert path(64, 256, 64, 32, 56, 56, gate=mb.MOCE_GATE_MLP_SIGMOID) == mb.PATH_MFMA
    assert path(5, 128, 24, 64, 12, 16) == mb.PATH_MFMA
    assert path(4, 240, 64, 32, 16, 16) == mb.PATH_TILE          # C not a multiple of 32
    assert path(4, 256, 65, 32, 16, 16) == mb.PATH_TILE          # E > 64
    assert path(2, 64, 16, 8, 8, 8, dtype="f32") == mb.PATH_GENERIC
    assert path(64, 1024, 256, 64, 14, 14, layout="nhwc") == mb.PATH_SCHEDULED
    assert path(128, 2048, 512, 128, 7, 7, layout="nhwc") == mb.PATH_SCHEDULED
    assert path(4, 96, 24, 20, 7, 7, layout="nhwc") == mb.PATH_GENERIC     # C not a multiple of 64
    assert path(4, 128, 20, 20, 7, 7, layout="nhwc") == mb.PATH_GENERIC    # E not a multiple of 8
    assert path(4, 128, 24, 8, 7, 7, dtype="f32", layout="nhwc") == mb.PATH_GENERIC
    assert path(512, 2048, 512, 8, 7, 7, layout="nhwc") == mb.PATH_GATHER   # k <= 16: the gather
    assert path(4, 96, 20, 16, 7, 7, layout="nhwc") == mb.PATH_GATHER       # C a multiple of 8
    assert path(4, 4096, 1025, 1, 1, 1, layout="nhwc") == mb.PATH_GATHER    # its size limits
    assert path(4, 4104, 24, 8, 7, 7, layout="nhwc") == mb.PATH_GENERIC     # C > 4096
    assert path(4, 2048, 1032, 8, 7, 7, layout="nhwc") == mb.PATH_SCHEDULED  # E - 1 > 1024
    assert path(4, 2048, 520, 12, 7, 7, layout="nhwc") == mb.PATH_SCHEDULED  # E - 1 > 512 with k > 8
    assert path(4, 2048, 513, 12, 7, 7, layout="nhwc") == mb.PATH_GATHER
    assert path(4, 100, 24, 8, 7, 7, layout="nhwc") == mb.PATH_GENERIC      # C not a multiple of 8
    assert path(4, 512, 64, 32, 16, 16) == mb.PATH_SCHEDULED     # C > 256: the scheduled product
    assert path(64, 1024, 256, 64, 14, 14) == mb.PATH_SCHEDULED  # the stage-3 layer, channels-first
    assert path(4, 512, 64, 32, 15, 15) == mb.PATH_GENERIC       # H W not a multiple of 4
    assert path(4, 520, 64, 32, 16, 16) == mb.PATH_GENERIC       # C not a multiple of 64
    assert path(4, 96, 24, 12, 30, 30) == mb.PATH_GENERIC        # H*W not a multiple of 8
    assert path(4, 64, 1, 8, 8, 8) == mb.PATH_GENERIC            # no routed expert


def test_forward_reused_workspace_sees_new_inputs():
    """Descriptors and coefficients of one call never leak into the next."""
    wl = inputs.WORKLOADS["resnet50_stage1"]
    g = inputs.generate(wl, batch=16)
    layer = MoceLayer.from_workload(wl, g)
    ws = layer.new_workspace(16)
    xs = [g["x"], np.ascontiguousarray(g["x"][::-1]), inputs.f32_to_bf16_bits(
        inputs.bf16_bits_to_f32(g["x"]) * np.float32(3.0))]
    y = None
    for x in xs + xs[:1]:
        ref = oracle.forward(x, g["s"], g["w"], wl.E, oracle.NCHW, a=g["a"], c=g["c"])
        y = layer.forward(to_device_x(x, wl.dtype), y, ws)
        check_y(to_host_f64(y), ref["y"], ref["mag"], wl.dtype)


def _mfma_path(k):
    """The forward's path code on the MFMA mix with the softplus-linear gate."""
    return mb.PATH_MFMA_GATE if k == 32 else mb.PATH_MFMA


MFMA_STAGES = [
    # B, C, E, k, H, W: moce_forward against moce_pool + moce_gate + moce_mix on the MFMA path
    (64, 256, 64, 32, 56, 56),   # the ResNet-50 stage-1 layer
    (24, 256, 64, 32, 56, 56),   # workgroup ranges that straddle images (a rebuild mid-range)
    (600, 64, 16, 2, 8, 8),      # ranges over three images
    (5, 128, 24, 64, 12, 16),    # k = 64: the gate kernel's 64-lane segments
    (9, 32, 8, 3, 8, 8),         # C = 32, one partial expert group, k not a power of two
    (3, 96, 40, 20, 6, 12),      # three expert groups, the last partial; ragged last tile (72 positions)
    (2, 64, 17, 8, 4, 4),        # the residual row alone in the second group
    # k = 32: the forward evaluates the gate inside the mix kernel
    (120, 64, 9, 32, 12, 16),    # ranges that straddle images (the gate again mid-range), one partial group
    (7, 64, 33, 32, 28, 28),     # the residual row alone in the third group; ragged last tile (16 positions)
]


@pytest.mark.parametrize("B,C,E,k,H,W", MFMA_STAGES)
def test_mfma_forward_equals_stages(B, C, E, k, H, W):
    """The whole-layer entry point gives the same bits as the three stage entry points in a row."""
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nchw", seed=11 * B + k, signed=(E % 2 == 1))
    layer = MoceLayer(C, E, k, H, W, "bf16", "nchw", s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == _mfma_path(k)
    xd = to_device_x(x, "bf16")
    y = layer.forward(xd)
    d = layer.pool(xd)
    _, alpha = layer.gate_tau(d)
    y_st = layer.mix(xd, alpha)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y_st.view(torch.int16))
    if k == 32:
        # the one-kernel gate and mix entry point, twice (the second output
        # buffer starts from other contents)
        for fill in (0, -1):
            y_gm = torch.full_like(y, fill)
            layer.gate_mix(xd, d, y_gm)
            torch.cuda.synchronize()
            assert torch.equal(y_gm.view(torch.int16), y_st.view(torch.int16))
    ref = oracle.forward(x, s, w, E, oracle.NCHW, a=a, c=c)
    check_y(to_host_f64(y), ref["y"], ref["mag"], "bf16")


# --------------------------------------------------------------------------- scheduled matrix-core mix (NHWC bf16)
SCHEDULED = [
    # B, C, E, k, H, W, extra: shapes served by the channels-last matrix-core mix
    (3, 1024, 256, 64, 14, 14, {}),            # stage-3 layer, a few images
    (2, 2048, 512, 128, 7, 7, {}),             # stage-4 layer
    (3, 768, 192, 48, 197, 1, dict(signed=True)),  # ViT token layer
    (2, 64, 8, 17, 5, 5, {}),                  # one 64-channel chunk; experts past E in the range
    (2, 128, 40, 17, 3, 11, dict(signed=True)),  # residual row in a partial group; 33 positions
    (1, 256, 24, 256, 2, 9, {}),               # k = C: 256 entries per group and step (overflow path)
    (2, 192, 96, 17, 10, 10, {}),              # 6 steps: the prefetch ring's tail
    (2, 256, 8, 17, 4, 4, dict(cyclic=True)),  # cyclic supports: U = channels 119..255
    (2, 256, 24, 17, 4, 4, dict(cyclic=True)),  # cyclic supports wrapping past C: U empty
    (1, 64, 64, 64, 113, 1, {}),               # E = C = k, positions over two 112-row tiles
]


@pytest.mark.parametrize("B,C,E,k,H,W,extra", SCHEDULED)
def test_scheduled_forward_shapes(B, C, E, k, H, W, extra):
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nhwc", seed=B * 31 + C + E + k, **extra)
    ref = oracle.forward(x, s, w, E, oracle.NHWC, a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, "bf16", "nhwc", s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == mb.PATH_SCHEDULED
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    check_y(y, ref["y"], ref["mag"], "bf16")
    if ref["nU"] == 0:
        assert np.all(y[..., E - 1] == 0.0)


SCHEDULED_NCHW = [
    # B, C, E, k, H, W, extra: channels-first shapes served by the scheduled product
    (3, 1024, 256, 64, 14, 14, {}),            # stage-3 layer: 196 positions over two 112-row tiles
    (2, 2048, 512, 128, 7, 8, {}),             # 32 steps, four expert ranges
    (2, 512, 64, 32, 16, 16, dict(signed=True)),
    (2, 320, 40, 17, 6, 10, {}),               # 5 steps; residual row in a partial group; 60 positions
    (1, 64, 64, 64, 1, 4, {}),                 # one step, E = C = k, 4 positions (off the tile paths)
    (2, 512, 24, 17, 3, 12, dict(cyclic=True)),  # cyclic supports: U = channels 391..511
    (2, 384, 56, 8, 4, 4, dict(cyclic=True)),  # cyclic supports wrapping past C: U empty
    (3, 768, 192, 48, 8, 25, dict(signed=True)),  # 200 positions: ragged last tile
    (4, 512, 40, 1, 6, 6, {}),                 # k = 1: exact copies
    (1, 4096, 16, 20, 2, 2, {}),               # C = 4096: 64 steps
    (2, 320, 48, 12, 20, 20, {}),              # 400 positions: planes pooled by 32 lanes
    (2, 512, 64, 16, 28, 28, dict(signed=True)),  # 784 positions: planes pooled by 64 lanes
]


@pytest.mark.parametrize("B,C,E,k,H,W,extra", SCHEDULED_NCHW)
def test_scheduled_nchw_forward_shapes(B, C, E, k, H, W, extra):
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nchw", seed=B * 37 + C + E + k, **extra)
    ref = oracle.forward(x, s, w, E, oracle.NCHW, a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, "bf16", "nchw", s, w, a=a, c=c)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_SOFTPLUS_LINEAR) == mb.PATH_SCHEDULED
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    check_y(y, ref["y"], ref["mag"], "bf16")
    if ref["nU"] == 0:
        assert np.all(y[:, E - 1] == 0.0)
    if k == 1:
        assert np.array_equal(y[:, :E - 1], ref["y"][:, :E - 1])


def test_scheduled_forward_mlp_gate_and_one_hot():
    """The paper's gate on the scheduled path, and the one-hot limit as exact copies there."""
    B, C, E, k, H, W = 2, 512, 64, 24, 6, 6
    x, s, w, a, c = _custom(B, C, E, k, H, W, "bf16", "nhwc", seed=17, signed=True)
    rng = np.random.default_rng(18)
    W1 = (rng.standard_normal((k, k)) * k ** -0.5).astype(np.float32)
    b1 = (rng.standard_normal(k) * 0.1).astype(np.float32)
    w2 = (rng.standard_normal(k) * k ** -0.5).astype(np.float32)
    ref = oracle.forward(x, s, w, E, oracle.NHWC, gate="mlp", W1=W1, b1=b1, w2=w2, b2=0.0)
    layer = MoceLayer(C, E, k, H, W, "bf16", "nhwc", s, w, gate="mlp", W1=W1, b1=b1, w2=w2, b2=0.0)
    assert mb.moce_forward_path(layer.desc(B), mb.MOCE_GATE_MLP_SIGMOID) == mb.PATH_SCHEDULED
    check_y(to_host_f64(layer.forward(to_device_x(x, "bf16"))), ref["y"], ref["mag"], "bf16")
    w[:, 0] = w.max(axis=1) + 1.0
    a[:] = 0.0
    c[:] = -1e4
    ref = oracle.forward(x, s, w, E, oracle.NHWC, a=a, c=c)
    layer = MoceLayer(C, E, k, H, W, "bf16", "nhwc", s, w, a=a, c=c)
    y = to_host_f64(layer.forward(to_device_x(x, "bf16")))
    assert np.array_equal(y[..., :E - 1], ref["y"][..., :E - 1])


@pytest.mark.parametrize("B,C,E,k,dtype,layout", [
    (4_300_000, 5, 2, 1, "f32", "nchw"),     # the generic mixes: 1024 threads an image
    (4_300_000, 5, 2, 1, "f32", "nhwc"),
    (8_400_000, 8, 8, 1, "bf16", "nhwc"),    # pooling of 16-byte rows: 512 threads an image
    (4_900_000, 64, 8, 17, "bf16", "nhwc"),  # the scheduled mix: a workgroup an image
    (1_100_000, 65, 65, 3, "f32", "nhwc"),   # 70 million (image, expert) rows of the gate
])
def test_forward_of_more_images_than_one_launch(B, C, E, k, dtype, layout):
    """Images of one position, more than the 2^32 threads of a launch hold (the excess is dropped without an
    error): the ends and the middle of the batch against those images alone."""
    _, s, w, a, c = _custom(1, C, E, k, 1, 1, dtype, layout, seed=C, signed=True)
    layer = MoceLayer(C, E, k, 1, 1, dtype, layout, s, w, a=a, c=c)
    td = layer.torch_dtype
    x = torch.randn((B, C, 1, 1) if layout == "nchw" else (B, 1, 1, C), device="cuda").to(td)
    ws = layer.new_workspace(B).fill_(255)        # NaN: what a launch leaves out shows
    y = layer.forward(x, torch.full(layer.y_shape(B), float("nan"), dtype=td, device="cuda"), ws)
    assert not torch.isnan(y).any()
    for b0 in (0, B // 2, B - 520):
        ref = layer.forward(x[b0:b0 + 520].clone())
        torch.testing.assert_close(y[b0:b0 + 520], ref, rtol=2.0 ** -7 if dtype == "bf16" else 1e-5, atol=1e-5)
