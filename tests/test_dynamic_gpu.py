"""GPU parity of the input-conditioned (dynamic) support path (Sec. 4.5 Eq. 11) against the oracle.

The selection is an integer decision taken from floating-point logits: the device forms the
example's logits in float32 from its own pooled descriptor, the oracle in float64 from the exact one.
The test therefore checks that the device's supports are a valid top k of the oracle's logits up to
a margin (every selected logit at least, every other logit at most, the oracle's k-th largest within
``EPS``; the order canonical within ``EPS``), and that they agree with the oracle's own selection
wherever the k-th and (k+1)-th largest logits are further apart than ``2 EPS``.  The outputs are then
compared with the oracle's layer evaluated at the device's supports (the oracle's logits there), to the
static layer's tolerances.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_23794_amd import inputs
from paper_2608_23794_amd.layer import DynamicMoceLayer, to_device_x, to_host_f64

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

OL = {"nchw": oracle.NCHW, "nhwc": oracle.NHWC}
EPS = 1e-4

CASES = [("tiny", "nchw"), ("tiny", "nhwc"), ("resnet50_stage1", "nchw"), ("resnet50_stage3", "nchw"),
         ("resnet50_stage3", "nhwc"), ("resnet50_stage4", "nhwc"), ("vit_tokens", "nhwc")]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    yield
    torch.cuda.synchronize()


def check_y(y, y_ref, mag, dtype):
    err = np.abs(y - y_ref)
    rtol = 1e-5 if dtype == "f32" else 1e-2
    e = (err / np.maximum(mag, 1e-30)).max()
    assert e <= rtol, f"y: max |y - y_ref| / M = {e:.3e}"
    if dtype == "bf16":
        assert np.all(err <= 2.0 ** -8 * np.abs(y_ref) + 1e-5 * mag), "y: beyond one bf16 rounding"


def check_selection(S, Lx, k):
    """S [n, R, k] device supports, Lx [n, R, C] oracle logits (float64)."""
    n, R, C = Lx.shape
    agree = 0
    for b in range(n):
        for e in range(R):
            vals, sel = Lx[b, e], S[b, e]
            assert np.unique(sel).size == k and sel.min() >= 0 and sel.max() < C
            srt = np.sort(vals)[::-1]
            kth = srt[k - 1]
            mask = np.zeros(C, bool)
            mask[sel] = True
            assert vals[mask].min() >= kth - EPS, (b, e)
            if k < C:
                assert vals[~mask].max() <= kth + EPS, (b, e)
            assert np.all(vals[sel][:-1] >= vals[sel][1:] - EPS), (b, e)
            if k == C or srt[k - 1] - srt[k] > 2 * EPS:
                ref = np.lexsort((np.arange(C), -vals))[:k]
                np.testing.assert_array_equal(np.sort(sel), np.sort(ref))
                agree += 1
    return agree


def run_case(wl, layout, B=None, images=None, gate="softplus"):
    g = inputs.generate(wl, layout, batch=B)
    rt = inputs.router_params(wl)
    layer = DynamicMoceLayer.from_workload(wl, g, rt, layout, gate=gate)
    x = to_device_x(g["x"], wl.dtype)
    Bn = x.shape[0]
    S = torch.empty((Bn, wl.E - 1, wl.k), dtype=torch.int32, device="cuda")
    y = to_host_f64(layer.forward(x, S_out=S))
    S = S.cpu().numpy()
    imgs = list(range(Bn)) if images is None else images
    xs = g["x"][imgs]
    d = oracle.pool(xs, OL[layout])
    Lx = oracle.dynamic_logits(oracle.router(d, rt["Wh"], rt["bh"]), rt["L"], rt["q"], rt["v"])
    agree = check_selection(S[imgs], Lx, wl.k)
    W = np.take_along_axis(Lx, S[imgs].astype(np.int64), axis=2)
    kw = dict(a=g["a"], c=g["c"]) if gate == "softplus" else dict(
        W1=g["W1"], b1=g["b1"], w2=g["w2"], b2=g["b2"], tau_min=g["tau_min"], tau_max=g["tau_max"])
    ref = oracle.dynamic_forward(xs, rt["L"], rt["Wh"], rt["bh"], rt["v"], rt["q"], wl.k, wl.E, OL[layout],
                                 gate=gate, S=S[imgs], W=W, **kw)
    check_y(y[imgs], ref["y"], ref["mag"], wl.dtype)
    return S, agree


@pytest.mark.parametrize("name,layout", CASES)
def test_dynamic_forward(name, layout):
    """The full batch runs on the device; the oracle checks the first two images and the last."""
    wl = inputs.WORKLOADS[name]
    imgs = sorted({0, 1, wl.B - 1}) if wl.B > 3 else None
    S, agree = run_case(wl, layout, images=imgs)
    assert agree > 0
    # the supports do depend on the example
    assert any(not np.array_equal(S[0], S[b]) for b in range(1, S.shape[0])) or wl.B == 1


@pytest.mark.parametrize("name,layout", [("tiny", "nchw"), ("resnet50_stage3", "nhwc")])
def test_dynamic_forward_mlp_gate(name, layout):
    wl = inputs.WORKLOADS[name]
    run_case(wl, layout, B=4, gate="mlp")


@pytest.mark.parametrize("B,C,E,k,d,H,W,dtype,layout", [
    (3, 40, 5, 40, 3, 2, 3, "f32", "nchw"),      # k = C: every channel in every support, U(X) empty
    (2, 96, 33, 1, 1, 3, 3, "bf16", "nhwc"),     # k = 1, d = 1
    (2, 300, 20, 200, 64, 1, 5, "f32", "nhwc"),  # k past a power of two, the widest router
    (1, 70, 2, 9, 5, 1, 1, "bf16", "nchw"),      # one routed expert, one position
    (2, 4096, 9, 512, 16, 1, 2, "f32", "nhwc"),  # the size limits: C = 4096, k = 512
    # bfloat16 NCHW with C <= 256 and H W a multiple of 8 takes the tile mix, which reloads the
    # supports when the image changes: one tile per image, a ragged last tile, and a coefficient
    # table too large to prefetch in registers
    (6, 64, 17, 8, 4, 4, 6, "bf16", "nchw"),
    (3, 256, 64, 16, 8, 12, 12, "bf16", "nchw"),
    (2, 200, 200, 12, 8, 8, 8, "bf16", "nchw"),
])
def test_dynamic_forward_edges(B, C, E, k, d, H, W, dtype, layout, gate="softplus"):
    rng = np.random.default_rng(B * 7919 + C)
    R = E - 1
    shape = (B, C, H, W) if layout == "nchw" else (B, H, W, C)
    x = np.maximum(rng.standard_normal(shape), 0).astype(np.float32)
    if dtype == "bf16":
        x = inputs.f32_to_bf16_bits(x)
    L = rng.standard_normal((R, C)).astype(np.float32)
    L[0, :8] = 0.5                                   # exact ties in the static logits
    Wh = (rng.standard_normal((d, C)) * 2 / np.sqrt(C)).astype(np.float32)
    bh = (rng.standard_normal(d) * 0.1).astype(np.float32)
    v = rng.standard_normal((C, d)).astype(np.float32)
    q = (rng.standard_normal((R, d)) / np.sqrt(d)).astype(np.float32)
    a = (rng.standard_normal((R, k)) / np.sqrt(k)).astype(np.float32)
    c = np.zeros(R, np.float32)
    p = dict(a=a, c=c) if gate == "softplus" else dict(
        W1=(rng.standard_normal((k, k)) / np.sqrt(k)).astype(np.float32), b1=np.zeros(k, np.float32),
        w2=(rng.standard_normal(k) / np.sqrt(k)).astype(np.float32), b2=0.1, tau_min=0.2, tau_max=6.0)
    layer = DynamicMoceLayer(C, E, k, H, W, dtype, layout, L, Wh, bh, v, q, gate=gate, **p)
    xd = to_device_x(x, dtype)
    S = torch.empty((B, R, k), dtype=torch.int32, device="cuda")
    y = to_host_f64(layer.forward(xd, S_out=S))
    S = S.cpu().numpy()
    d_ref = oracle.pool(x, OL[layout])
    Lx = oracle.dynamic_logits(oracle.router(d_ref, Wh, bh), L, q, v)
    check_selection(S, Lx, k)
    Wsel = np.take_along_axis(Lx, S.astype(np.int64), axis=2)
    ref = oracle.dynamic_forward(x, L, Wh, bh, v, q, k, E, OL[layout], gate=gate, S=S, W=Wsel, **p)
    check_y(y, ref["y"], ref["mag"], dtype)


def test_dynamic_forward_without_offset_matches_static_supports():
    """q = 0: the device's supports are the top k of the static logits for every example, ties to the
    lower channel, bit for bit (the logits are then the given float32 values on both sides)."""
    wl = inputs.WORKLOADS["resnet50_stage3"]
    g = inputs.generate(wl, "nhwc", batch=3)
    rt = dict(inputs.router_params(wl))
    rt["q"] = np.zeros_like(rt["q"])
    rt["L"] = np.round(rt["L"] * 4) / 4          # many exact ties
    layer = DynamicMoceLayer.from_workload(wl, g, rt, "nhwc")
    S = torch.empty((3, wl.E - 1, wl.k), dtype=torch.int32, device="cuda")
    layer.forward(to_device_x(g["x"], wl.dtype), S_out=S)
    S = S.cpu().numpy()
    ref = np.stack([np.lexsort((np.arange(wl.C), -row))[:wl.k] for row in rt["L"].astype(np.float64)])
    for b in range(3):
        np.testing.assert_array_equal(S[b], ref)


# the one-pass selection's limits: row lengths of 256 to 2048 keys filled and ragged, 16-byte and
# single reads of L, lists of 64, 128 and 240 entries, one expert more than a block of 16
ONE_PASS = [(4, 3, 2, 32), (65, 17, 32, 32), (256, 33, 33, 32), (300, 18, 64, 32), (512, 16, 65, 32), (1022, 17, 8, 31),
            (1024, 40, 128, 32), (1500, 9, 160, 32), (2048, 34, 1, 32), (2048, 34, 128, 32), (2048, 18, 160, 7)]


@pytest.mark.parametrize("C,E,k,d", ONE_PASS)
def test_dynamic_one_pass_selection_edges(C, E, k, d):
    """Logits against the oracle, to the margins of the other shapes."""
    test_dynamic_forward_edges(2, C, E, k, d, 2, 3, "f32", "nhwc")


@pytest.mark.parametrize("C,E,k,d", ONE_PASS)
@pytest.mark.parametrize("rows", ["ties", "outliers", "equal"])
def test_dynamic_one_pass_selection_is_exact(C, E, k, d, rows):
    """q = 0 (the given logits on both sides): supports equal the stable sort bit for bit, where thresholds
    fall among many equal keys, among infinities and signed zeros, and where every key is the same."""
    rng = np.random.default_rng(C * 31 + k)
    R = E - 1
    L = rng.standard_normal((R, C)).astype(np.float32)
    if rows == "ties":
        L = (np.round(L * 2) / 2).astype(np.float32)            # -0.0 among them
    elif rows == "outliers":
        L = (L * np.float32(10.0) ** rng.integers(-30, 30, (R, C))).astype(np.float32)
        L[:, ::7] = -np.inf
        L[:, 3::max(4, C // 3)] = np.inf
    else:
        L[:] = -1.5
    z = np.zeros
    layer = DynamicMoceLayer(C, E, k, 1, 2, "f32", "nhwc", L, z((d, C)), z(d), rng.standard_normal((C, d)), z((R, d)),
                             a=z((R, k)), c=z(R))
    x = torch.from_numpy(rng.standard_normal((3, 1, 2, C)).astype(np.float32)).cuda()
    S = torch.empty((3, R, k), dtype=torch.int32, device="cuda")
    layer.forward(x, S_out=S)
    ref = np.stack([np.lexsort((np.arange(C), -row))[:k] for row in L.astype(np.float64)])
    np.testing.assert_array_equal(S.cpu().numpy(), np.broadcast_to(ref, (3, R, k)))


@pytest.mark.parametrize("B,C,E,k,d,H,W,dtype,layout", [
    (256, 40, 6, 33, 4, 5, 5, "bf16", "nhwc"),    # four 8-position units, four lanes an expert, a ragged last read
    (256, 41, 6, 36, 4, 5, 5, "bf16", "nhwc"),    # odd C: x by elements
    (128, 264, 5, 64, 4, 4, 8, "bf16", "nchw"),   # whole 16-byte pieces of planes, two units
    (256, 40, 40, 7, 3, 3, 3, "bf16", "nchw"),    # planes by elements, a lane an expert
    (256, 24, 5, 8, 2, 4, 5, "f32", "nchw"),      # four 4-position units, a ragged last tile
    (86, 44, 9, 32, 2, 3, 5, "f32", "nhwc"),      # one unit
])
def test_dynamic_gather_edges(B, C, E, k, d, H, W, dtype, layout):
    """The gather's tiles, readers of x and lanes an expert at the ends of their ranges."""
    test_dynamic_forward_edges(B, C, E, k, d, H, W, dtype, layout)


def test_dynamic_forward_of_more_positions_than_one_launch_of_full_workgroups():
    """67.2 million positions: 1024 threads for every 16 of them would pass the 2^32 threads of a launch, whose
    excess is dropped without an error.  k = 1, so that the routed output is the selected channel itself and the
    residual the other one, both bit for bit."""
    B, HW = 64, 1_050_000
    z = np.zeros
    L = np.array([[0.25, 1.0]], np.float32)
    layer = DynamicMoceLayer(2, 2, 1, 1, HW, "f32", "nchw", L, z((1, 2)), z(1), z((2, 1)), z((1, 1)), a=z((1, 1)), c=z(1))
    x = torch.randn((B, 2, 1, HW), device="cuda")
    y = torch.full((B, 2, 1, HW), float("nan"), device="cuda")
    layer.forward(x, y)
    assert torch.equal(y, x.flip(1))


@pytest.mark.parametrize("B,C,E,k,d,H,W,dtype,layout", [
    (300, 40, 3, 7, 4, 5, 5, "bf16", "nhwc"),      # workgroups of 128: two experts and the residual's wave
    (300, 40, 30, 35, 4, 5, 5, "f32", "nchw"),     # 256: 29 experts by four lanes
    (300, 420, 4, 7, 4, 4, 9, "f32", "nhwc"),      # 512 by the LDS share
    (90, 300, 130, 7, 4, 3, 5, "f32", "nchw"),     # 1024 for one workgroup a CU
    (260, 300, 260, 40, 4, 1, 1, "bf16", "nhwc"),  # more lanes than threads; one position, one unit
    (260, 40, 5, 8, 4, 1, 17, "bf16", "nhwc"),     # three units: four a workgroup, one past the image
])
def test_dynamic_gather_workgroups(B, C, E, k, d, H, W, dtype, layout):
    """The gather's workgroup sizes and units a tile."""
    test_dynamic_forward_edges(B, C, E, k, d, H, W, dtype, layout)


# past the one-pass selection's limits, a launch for each step: blocks of eight, four and two rows, lists that fill a
# power of two and lists that do not, both router widths that the kernels are built for
STEPS = [(512, 18, 200, 32), (3, 3, 2, 5), (1100, 10, 161, 1), (2304, 10, 16, 32), (2049, 6, 1, 32), (4096, 4, 256, 32),
         (600, 11, 40, 33), (4096, 4, 512, 64)]


@pytest.mark.parametrize("C,E,k,d,gate", [s + ("softplus",) for s in STEPS] + [s + ("mlp",) for s in STEPS if s[2] <= 256])
def test_dynamic_selection_step_by_step(C, E, k, d, gate):
    test_dynamic_forward_edges(2, C, E, k, d, 2, 3, "f32", "nhwc", gate=gate)


@pytest.mark.parametrize("C,E,k,d", STEPS)
@pytest.mark.parametrize("rows", ["ties", "outliers", "equal"])
def test_dynamic_selection_step_by_step_is_exact(C, E, k, d, rows):
    test_dynamic_one_pass_selection_is_exact(C, E, k, d, rows)


@pytest.mark.parametrize("k,gate", [(2, "softplus"), (2, "mlp")])
def test_dynamic_forward_of_more_images_than_one_launch(k, gate):
    """2.2 million images: a wave for each of 32 router units passes the 2^32 threads of a launch.  The ends of the
    batch against those images alone."""
    B, C, E, d = 2_200_000, 4, 3, 32
    rng = np.random.default_rng(0)
    f = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    p = dict(a=f(E - 1, k), c=f(E - 1)) if gate == "softplus" else dict(W1=f(k, k), b1=f(k), w2=f(k))
    layer = DynamicMoceLayer(C, E, k, 1, 1, "f32", "nhwc", f(E - 1, C), f(d, C), f(d), f(C, d), f(E - 1, d), gate=gate, **p)
    x = torch.randn((B, 1, 1, C), device="cuda")
    S = torch.full((B, E - 1, k), -1, dtype=torch.int32, device="cuda")
    y = layer.forward(x, torch.full((B, 1, 1, E), float("nan"), device="cuda"), layer.new_workspace(B).fill_(255), S_out=S)
    assert not torch.isnan(y).any()
    for b0 in (0, B // 2, B - 520):
        Sr = torch.empty((520, E - 1, k), dtype=torch.int32, device="cuda")
        ref = layer.forward(x[b0:b0 + 520].clone(), S_out=Sr)
        assert torch.equal(S[b0:b0 + 520], Sr)
        torch.testing.assert_close(y[b0:b0 + 520], ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("B,C,E,k,d,H,W,dtype,layout", [
    (1, 600, 600, 3, 32, 1, 2, "f32", "nhwc"),     # more runs of experts than U has room for their bitmaps
    (1, 600, 600, 1, 32, 1, 2, "f32", "nhwc"),     # 599 words of room, 600 in U
    (2, 640, 513, 40, 32, 3, 3, "bf16", "nchw"),   # sixteen workgroups a tile, four lanes an expert
    (1, 300, 130, 7, 32, 1, 9, "f32", "nchw"),     # one expert past a workgroup's share: no second one
    (1, 300, 257, 7, 32, 1, 9, "bf16", "nhwc"),    # two workgroups a tile, an expert each lane
    (3, 2304, 300, 30, 4, 1, 5, "bf16", "nhwc"),   # the same after the selection step by step
    (3, 300, 9, 33, 4, 3, 8, "bf16", "nchw"),      # whole planes, pieces of two, eight and four positions
    (3, 300, 9, 7, 4, 3, 8, "bf16", "nchw"),
    (3, 300, 9, 7, 4, 3, 4, "f32", "nchw"),
])
@pytest.mark.parametrize("gate", ["softplus", "mlp"])
def test_dynamic_forward_of_few_tiles(B, C, E, k, d, H, W, dtype, layout, gate):
    """Few images and positions under many experts: the gather's tiles and the selection's runs shared out."""
    test_dynamic_forward_edges(B, C, E, k, d, H, W, dtype, layout, gate=gate)
