"""GPU parity of the layer's backward (moce_backward) and of the routing-logit gradient with the coverage
loss (moce_logit_backward) against the oracle's float64 gradients, on the same seeded inputs.

Tolerances, from the arithmetic: every gradient is a float32 sum (over positions, support entries and
images) of products of float32 or bfloat16 values, so its error is a few float32 roundings of the
largest partial sums, well below 2e-5 of the tensor's largest entry at these sizes.  dx in bfloat16 is
rounded once more on its way out (half an ulp, 2^-9 of the value), so it may differ by 2^-8 of the
value on top.  The comparison scale of a parameter gradient is its largest entry over the tensor,
since single entries can cancel to near zero.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import backward as ob
from paper_2608_23794_amd import inputs
from paper_2608_23794_amd import binding as mb
from paper_2608_23794_amd.layer import MoceLayer, to_device_x, to_host_f64

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

OL = {"nchw": oracle.NCHW, "nhwc": oracle.NHWC}
RTOL_F32 = 2e-5


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    yield
    torch.cuda.synchronize()


def close(name, dev, ref, bf16=False, rtol=RTOL_F32):
    dev = np.asarray(dev, np.float64)
    ref = np.asarray(ref, np.float64)
    assert dev.shape == ref.shape, (name, dev.shape, ref.shape)
    scale = max(np.abs(ref).max(), 1e-30)
    bound = rtol * scale + (2.0 ** -8 * np.abs(ref) if bf16 else 0.0)
    err = np.abs(dev - ref)
    worst = np.unravel_index(np.argmax(err - bound), err.shape)
    assert np.all(err <= bound), f"{name}: |dev - ref| = {err[worst]:.3e} at {worst}, bound {np.asarray(bound).max():.3e}"


def make_dy(shape, dtype, seed):
    g = np.random.default_rng(seed).standard_normal(shape).astype(np.float32)
    if dtype == "bf16":
        bits = inputs.f32_to_bf16_bits(g)
        return bits, inputs.bf16_bits_to_f32(bits).astype(np.float64)
    return g, g.astype(np.float64)


def oracle_grads(layer, x, dy64, gate, params, images=None):
    """Oracle gradients over the canonical rows (so dw comes in the device's order), summed over chunks
    of images; dx only for `images` (all when None)."""
    s_c = layer.s_c.cpu().numpy()
    w_c = layer.w_c.cpu().numpy()
    kw = dict(a=params["a"], c=params["c"]) if gate == "softplus" else dict(
        W1=params["W1"], b1=params["b1"], w2=params["w2"], b2=params["b2"], tau_min=params["tau_min"],
        tau_max=params["tau_max"])
    B = x.shape[0]
    acc = {}
    dx = {}
    step = max(1, int(4e6 // max(1, layer.R * layer.k * layer.H * layer.W)))
    for b0 in range(0, B, step):
        sl = slice(b0, min(B, b0 + step))
        g = ob.layer_backward(x[sl], s_c, w_c, layer.E, dy64[sl], layout=OL[layer.layout], gate=gate, **kw)
        for n in ("dw", "da", "dc", "dW1", "db1", "dw2", "db2"):
            if n in g:
                acc[n] = acc.get(n, 0.0) + np.asarray(g[n])
        for j, b in enumerate(range(sl.start, sl.stop)):
            if images is None or b in images:
                dx[b] = g["dx"][j]
    return acc, dx


def run(layer, x_host, dtype, gate, params, seed=0, images=None):
    B = x_host.shape[0]
    x = to_device_x(x_host, dtype)
    dyh, dy64 = make_dy(layer.y_shape(B), dtype, seed)
    dy = to_device_x(dyh, dtype)
    out = layer.backward(x, dy)
    torch.cuda.synchronize()
    ref, rdx = oracle_grads(layer, x_host, dy64, gate, params, images)
    dx = to_host_f64(out["dx"])
    for b, v in rdx.items():
        close(f"dx[{b}]", dx[b], v, bf16=dtype == "bf16")
    if layer.R > 0:
        close("dw", out["dw"].cpu().numpy(), ref["dw"])
        if gate == "softplus":
            close("da", out["da"].cpu().numpy(), ref["da"])
            close("dc", out["dc"].cpu().numpy()[:layer.R], ref["dc"])
        else:
            close("dW1", out["dW1"].cpu().numpy(), ref["dW1"])
            close("db1", out["db1"].cpu().numpy(), ref["db1"])
            close("dw2", out["dw2"].cpu().numpy(), ref["dw2"])
            close("db2", out["db2"].cpu().numpy()[0], ref["db2"])
    return out


CASES = [("tiny", "nchw", None), ("resnet50_stage1", "nchw", 2), ("resnet50_stage3", "nchw", 3),
         ("resnet50_stage3", "nhwc", 3), ("resnet50_stage4", "nhwc", 2), ("vit_tokens", "nhwc", 2)]


@pytest.mark.parametrize("name,layout,B", CASES)
def test_backward_matches_oracle(name, layout, B):
    wl = inputs.WORKLOADS[name]
    g = inputs.generate(wl, layout, batch=B)
    layer = MoceLayer.from_workload(wl, g, layout)
    run(layer, g["x"], wl.dtype, "softplus", g, seed=wl.seed)


@pytest.mark.parametrize("name,layout,B", [("tiny", "nchw", None), ("resnet50_stage3", "nhwc", 2),
                                           ("resnet50_stage1", "nchw", 2)])
def test_backward_mlp_gate_matches_oracle(name, layout, B):
    wl = inputs.WORKLOADS[name]
    g = inputs.generate(wl, layout, batch=B)
    layer = MoceLayer.from_workload(wl, g, layout, gate="mlp")
    run(layer, g["x"], wl.dtype, "mlp", g, seed=wl.seed + 1)


def test_backward_full_batch_stage3_nhwc():
    """The whole batch of 64 images on the device; the parameter gradients against the oracle summed
    over every image, dx on the first, a middle and the last image."""
    wl = inputs.WORKLOADS["resnet50_stage3"]
    g = inputs.generate(wl, "nhwc")
    layer = MoceLayer.from_workload(wl, g, "nhwc")
    run(layer, g["x"], wl.dtype, "softplus", g, seed=5, images={0, 31, wl.B - 1})


def rand_layer(seed, B, C, E, k, H, W, dtype, layout, gate="softplus", a_scale=0.7):
    rng = np.random.default_rng(seed)
    R = E - 1
    s = np.array([rng.choice(C, size=k, replace=False) for _ in range(R)], np.int32).reshape(R, k)
    w = (rng.standard_normal((R, k)) * 1.5).astype(np.float32)
    shape = (B, C, H, W) if layout == "nchw" else (B, H, W, C)
    x = (rng.standard_normal(shape) + 0.3).astype(np.float32)
    if dtype == "bf16":
        x = inputs.f32_to_bf16_bits(x)
    p = dict(a=(rng.standard_normal((R, k)) * a_scale).astype(np.float32),
             c=(rng.standard_normal(R) * 0.5).astype(np.float32),
             W1=(rng.standard_normal((k, k)) / np.sqrt(k)).astype(np.float32),
             b1=(rng.standard_normal(k) * 0.2).astype(np.float32),
             w2=(rng.standard_normal(k) / np.sqrt(k)).astype(np.float32), b2=np.float32(0.1), tau_min=0.2,
             tau_max=6.0)
    layer = MoceLayer(C, E, k, H, W, dtype, layout, s, w, gate=gate, **p)
    return layer, x, p


@pytest.mark.parametrize("B,C,E,k,H,W,dtype,layout", [
    (2, 40, 1, 5, 3, 3, "f32", "nchw"),        # no routed expert: every channel is in U
    (2, 40, 6, 1, 2, 3, "bf16", "nhwc"),       # k = 1: alpha = 1, no gradient reaches the gate
    (2, 24, 4, 24, 2, 2, "f32", "nhwc"),       # k = C: U empty
    (3, 37, 9, 7, 3, 5, "bf16", "nchw"),       # C not a multiple of 8, odd plane
    (2, 130, 17, 70, 1, 1, "bf16", "nhwc"),    # one position, k past 64
    (1, 300, 33, 200, 2, 7, "f32", "nhwc"),    # k past 128
    (2, 264, 72, 9, 5, 8, "bf16", "nhwc"),     # matrix-core dalpha: ragged channel and expert blocks
    (2, 72, 16, 7, 9, 8, "bf16", "nchw"),      # matrix-core dalpha, NCHW: 72 positions, a ragged last stage
    (1, 48, 24, 6, 5, 4, "bf16", "nchw"),      # NCHW with 4-position loads
    (2, 512, 9, 255, 2, 3, "bf16", "nhwc"),    # rows of 16 lanes by 16 entries, the last one empty
    (2, 512, 9, 256, 2, 3, "bf16", "nhwc"),    # the same, full
    (1, 264, 136, 9, 7, 10, "bf16", "nhwc"),   # matrix-core dx: 3 channel blocks, 3 expert chunks, 2 position tiles
    (1, 300, 136, 5, 6, 6, "bf16", "nchw"),    # the same, NCHW with 4-position loads
])
def test_backward_edge_shapes(B, C, E, k, H, W, dtype, layout):
    layer, x, p = rand_layer(B * 1000 + C, B, C, E, k, H, W, dtype, layout)
    run(layer, x, dtype, "softplus", p, seed=C)


@pytest.mark.parametrize("B,C,E,k,H,W,dtype,layout", [
    (2, 37, 9, 7, 3, 5, "bf16", "nchw"),
    (2, 300, 33, 128, 1, 3, "f32", "nhwc"),    # the MLP backward's limit k = 128
])
def test_backward_mlp_edge_shapes(B, C, E, k, H, W, dtype, layout):
    layer, x, p = rand_layer(B * 77 + C, B, C, E, k, H, W, dtype, layout, gate="mlp")
    run(layer, x, dtype, "mlp", p, seed=C + 1)


def test_backward_residual_only_upstream_is_exact_mean():
    """dy zero on the routed outputs: dx is dy_res / |U| on U and 0 elsewhere, and nothing reaches w or
    the gate (exact zeros on both sides)."""
    layer, x, p = rand_layer(3, 2, 48, 5, 4, 3, 3, "f32", "nchw")
    xd = to_device_x(x, "f32")
    dy = torch.zeros(layer.y_shape(2), dtype=torch.float32, device="cuda")
    dy[:, 4] = torch.randn(2, 3, 3, device="cuda")
    out = layer.backward(xd, dy)
    torch.cuda.synchronize()
    U = layer.U.cpu().numpy()[:layer.nU]
    ref = np.zeros(x.shape)
    ref[:, U] = (dy[:, 4:5].cpu().numpy() / np.float32(layer.nU)).astype(np.float32)
    np.testing.assert_array_equal(out["dx"].cpu().numpy(), ref.astype(np.float32))
    assert torch.all(out["dw"] == 0) and torch.all(out["da"] == 0) and torch.all(out["dc"][:4] == 0)


@pytest.mark.parametrize("R,C,k,eps,lam", [(63, 256, 32, 1e-8, 5e-4), (255, 1024, 64, 1e-8, 0.05),
                                           (7, 100, 9, 0.3, 1.0), (3, 32768, 5, 1e-8, 2.0)])
def test_logit_backward_matches_oracle(R, C, k, eps, lam):
    rng = np.random.default_rng(R + C)
    L = (rng.standard_normal((R, C)) * 0.5).astype(np.float32)
    s = np.argsort(-L, axis=1, kind="stable")[:, :k].astype(np.int32)
    w = np.take_along_axis(L, s, axis=1)
    layer = MoceLayer(C, R + 1, k, 1, 1, "f32", "nchw", s, w, a=np.zeros((R, k), np.float32),
                      c=np.zeros(R, np.float32))
    s_c = layer.s_c.cpu().numpy()
    dw = rng.standard_normal((R, k)).astype(np.float32)
    Ld = torch.from_numpy(L).cuda()
    loss, dL = layer.logit_backward(Ld, torch.from_numpy(dw).cuda(), eps, lam)
    loss0, dL0 = layer.logit_backward(Ld, None, eps, lam)
    torch.cuda.synchronize()
    ref_loss = ob.coverage_loss(L, eps)
    G = lam * ob.coverage_grad(L, eps)
    assert float(loss.cpu()[0]) == pytest.approx(ref_loss, rel=1e-4, abs=1e-7)
    assert float(loss0.cpu()[0]) == float(loss.cpu()[0])
    close("dL (coverage only)", dL0.cpu().numpy(), G, rtol=1e-4)
    full = G.copy()
    np.put_along_axis(full, s_c.astype(np.int64), np.take_along_axis(full, s_c.astype(np.int64), 1) + dw, 1)
    close("dL", dL.cpu().numpy(), full, rtol=1e-4)


# rows of W1 padded to 32, 64 and 128, ragged blocks of 64 (image, expert) rows, and more blocks than
# workgroups (17 010 rows: 266 blocks, 256 partials)
@pytest.mark.parametrize("B,C,E,k", [(3, 40, 9, 1), (2, 70, 34, 31), (3, 64, 22, 32), (5, 66, 14, 33), (2, 130, 65, 64),
                                     (3, 100, 20, 65), (2, 200, 40, 128), (70, 260, 244, 4)])
def test_backward_mlp_row_blocks(B, C, E, k):
    layer, x, p = rand_layer(B * 1009 + k, B, C, E, k, 1, 3, "f32", "nhwc", gate="mlp")
    run(layer, x, "f32", "mlp", p, seed=3)


@pytest.mark.parametrize("R,C,k", [(1, 33, 5), (30, 31, 31), (33, 65, 1), (100, 257, 8)])
def test_logit_backward_ragged_sizes(R, C, k):
    """Rows and channels around the 32 of a column block, channels around the 256 threads of a row."""
    test_logit_backward_matches_oracle(R, C, k, 0.3, 0.05)


@pytest.mark.parametrize("B,C,E,k,H,W,layout", [
    (2, 136, 72, 9, 7, 7, "nhwc"),        # one position stage, two channel and expert blocks, 16-byte loads
    (2, 132, 68, 100, 9, 20, "nhwc"),     # stages of dy in LDS, 8-byte loads
    (2, 130, 70, 129, 7, 7, "nhwc"),      # single loads in dx, k past 128; the vector dalpha
    (3, 140, 66, 20, 5, 5, "nchw"),       # planes by elements in dx; the vector dalpha
    (2, 72, 9, 8, 11, 17, "nchw"),        # planes by elements in both
    (520, 16, 8, 3, 20, 15, "nhwc"),      # images enough not to split 300 positions: dy staged
    (520, 13, 5, 3, 20, 15, "nhwc"),      # single elements, few rows: the vector kernels
    (520, 12, 5, 3, 15, 20, "nchw"),
    (520, 9, 4, 2, 7, 43, "nchw"),        # the vector kernels
    (2, 136, 127, 9, 9, 9, "nhwc"),       # one expert past the last of a chunk's pieces
    (1, 8, 2, 1, 1, 1, "nchw"),           # one position
    (1, 4100, 1091, 1, 1, 1, "nhwc"),     # one position and few entries: the vector kernels
    (1, 2304, 2180, 1, 1, 3, "nhwc"),     # the same
    (1, 4200, 4200, 1, 1, 1, "nhwc"),     # more chunks than dx and the product of dd keep ranges of in LDS
])
def test_backward_position_stages_and_alignments(B, C, E, k, H, W, layout):
    """The matrix-core dalpha's stages, readers and row writers; dx of the same shapes."""
    layer, x, p = rand_layer(B * 31 + C, B, C, E, k, H, W, "bf16", layout)
    run(layer, x, "bf16", "softplus", p, seed=C, images={0, B - 1})


@pytest.mark.parametrize("B,C,E,k,H,W,dtype,layout", [
    (35, 130, 70, 9, 5, 5, "f32", "nchw"),     # two chunks, groups of images, the product's zeros
    (3, 130, 70, 9, 5, 5, "bf16", "nchw"),     # rows by single elements
    (3, 150, 68, 20, 9, 9, "bf16", "nhwc"),    # 8-byte rows, two position blocks
    (3, 150, 67, 20, 9, 9, "bf16", "nhwc"),
])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_backward_keeps_what_is_not_finite_to_its_channels(B, C, E, k, H, W, dtype, layout, value):
    """One element of dy that is not finite reaches dx of its image on its expert's
    channels alone; all other elements are those of the same dy with a zero there, to
    the rounding of sums in another order (and of bfloat16)."""
    layer, x, p = rand_layer(B * 7 + C, B, C, E, k, H, W, dtype, layout)
    dyh, _ = make_dy(layer.y_shape(B), dtype, 5)
    xd, dy = to_device_x(x, dtype), to_device_x(dyh, dtype)
    b, e, h, w = B - 1, E // 2, H - 1, W // 2
    at = (b, e, h, w) if layout == "nchw" else (b, h, w, e)
    dy[at] = 0.0
    ref = to_host_f64(layer.backward(xd, dy)["dx"])
    dy[at] = value
    got = to_host_f64(layer.backward(xd, dy)["dx"])
    if layout == "nhwc":
        ref, got = np.moveaxis(ref, -1, 1), np.moveaxis(got, -1, 1)
    on = np.zeros(C, bool)
    on[layer.s_c.cpu().numpy()[e]] = True
    assert not np.isfinite(got[b][on]).any()
    # the expert's gate gradient, and with it dd of its channels, is lost for that image
    mask = np.ones(got.shape, bool)
    mask[b, on] = False
    assert np.isfinite(got[mask]).all()
    close("dx", got[mask], ref[mask], bf16=dtype == "bf16")


@pytest.mark.parametrize("C,HW,layout", [(3, 1, "nchw"), (5, 4, "nchw"), (9, 1, "nhwc")])
def test_backward_of_more_images_than_one_launch_of_tiles(C, HW, layout):
    """2^24 + 8 small images: a 256-thread workgroup each would pass the 2^32 threads of a launch, whose excess is
    dropped without an error.  k = 1: alpha = 1 and no gradient reaches the gate, so dx is dy on the routed channel
    and dy of the residual over |U| elsewhere, exact in bfloat16 where |U| is a power of two."""
    B = (1 << 24) + 8
    z = np.zeros
    layer = MoceLayer(C, 2, 1, HW, 1, "bf16", layout, z((1, 1)), z((1, 1)), a=z((1, 1)), c=z(1))
    shape = lambda n: (B, n, HW, 1) if layout == "nchw" else (B, HW, 1, n)
    x = torch.randn(shape(C), device="cuda").bfloat16()
    dy = torch.randn(shape(2), device="cuda").bfloat16()
    ws = layer.new_backward_workspace(B).fill_(255)      # NaN: what a launch leaves out shows
    dx = layer.backward(x, dy, torch.full_like(x, float("nan")), ws)["dx"]
    ax = 1 if layout == "nchw" else 3
    dx, dy = dx.movedim(ax, 0), dy.movedim(ax, 0)
    assert torch.equal(dx[0], dy[0])
    assert torch.equal(dx[1:], (dy[1:] / (C - 1)).expand(dx[1:].shape))



@pytest.mark.parametrize("B", [1, 5, 8, 11])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_backward_units_over_the_dies(B, layout):
    """Batches that are fewer than, as many as and no multiple of the eight dies, several blocks an image: every unit
    is taken once."""
    layer, x, p = rand_layer(B + 50, B, 264, 136, 9, 8, 9, "bf16", layout)
    run(layer, x, "bf16", "softplus", p, seed=B)


@pytest.mark.parametrize("B,C,E,k", [(1030, 9, 3, 2), (2600, 7, 2, 5), (700, 300, 4, 270)])
def test_backward_many_image_groups(B, C, E, k):
    """Few experts over many images: one to three images a group, up to 1024 groups, and lanes of a whole wave a row."""
    layer, x, p = rand_layer(B + k, B, C, E, k, 1, 2, "f32", "nhwc")
    run(layer, x, "f32", "softplus", p, seed=B, images={0, B // 2, B - 1})


@pytest.mark.parametrize("B,C,E,k,H,W,layout,gate", [
    (900, 130, 67, 2, 1, 1, "nhwc", "softplus"),   # few entries at one position: both vector kernels
    (900, 130, 67, 2, 1, 1, "nchw", "mlp"),
    (900, 13, 5, 3, 1, 1, "nchw", "softplus"),
    (1, 4100, 1091, 1, 1, 1, "nhwc", "softplus"),  # the same, one image
    (60, 300, 67, 30, 3, 3, "nhwc", "softplus"),   # the matrix-core dx, the vector dalpha
    (520, 6, 3, 6, 9, 11, "nchw", "softplus"),     # few waves over many positions: both vector kernels, by a little
    (520, 6, 3, 6, 9, 11, "nhwc", "softplus"),     # the matrix-core dalpha, the vector dx
    (30, 260, 130, 60, 7, 7, "nchw", "softplus"),  # both matrix-core kernels
    (30, 260, 130, 60, 7, 7, "nhwc", "softplus"),
    (1, 4100, 1091, 9, 7, 7, "nhwc", "softplus"),  # the matrix-core dalpha over many channel blocks, the vector dx
    (1, 2304, 2180, 8, 7, 9, "nhwc", "softplus"),  # the same, 8-byte rows
    (2, 1300, 302, 60, 7, 7, "nhwc", "softplus"),  # both matrix-core kernels: many channel blocks, single elements
    (2, 2304, 2181, 60, 9, 7, "nhwc", "softplus"),  # the same, more chunks than bucket ranges kept in LDS
    (520, 13, 13, 3, 10, 10, "nhwc", "softplus"),  # the matrix-core dalpha: two stages of dy in LDS, single elements
    (520, 9, 9, 2, 9, 11, "nchw", "softplus"),
    (520, 12, 12, 3, 10, 10, "nhwc", "softplus"),  # the same, 8-byte rows
    (520, 13, 13, 3, 20, 15, "nhwc", "softplus"),  # the same, dy staged again and again
    (520, 9, 9, 2, 7, 43, "nchw", "softplus"),
    (520, 12, 12, 3, 20, 15, "nhwc", "softplus"),
    (3, 37, 1, 5, 3, 3, "nchw", "softplus"),       # no routed expert
    (3, 37, 1, 5, 3, 3, "nhwc", "mlp"),
])
def test_backward_ragged_rows(B, C, E, k, H, W, layout, gate):
    """bfloat16 rows without wide loads, on either side of the lines between the vector and the matrix-core kernels.
    (The MLP gate at few (image, expert) rows: among B (E-1) k = 2e5 units one lies within float32 rounding of its
    ReLU's kink, 5e-9, and takes either derivative.)"""
    layer, x, p = rand_layer(B * 13 + C, B, C, E, k, H, W, "bf16", layout, gate=gate)
    run(layer, x, "bf16", gate, p, seed=C, images={0, B - 1})


@pytest.mark.parametrize("B,C,E,k,H,dtype,layout", [
    (2, 300, 280, 5, 2, "f32", "nhwc"),      # few images, several chunks of experts: dd from the channel lists
    (2, 300, 280, 1, 2, "f32", "nchw"),      # the same, channels with no entry
    (3, 1030, 700, 40, 1, "bf16", "nchw"),   # the same under the bfloat16 vector dx
    (70, 70, 60, 40, 2, "f32", "nhwc"),      # one chunk, many entries: the product, beside the lists
])
def test_backward_dd_beside_the_vector_dx(B, C, E, k, H, dtype, layout):
    layer, x, p = rand_layer(B + C + k, B, C, E, k, H, 1, dtype, layout)
    run(layer, x, dtype, "softplus", p, seed=C)


@pytest.mark.parametrize("C,dtype", [(524_289, "f32"), (600_000, "bf16"), (1_048_640, "f32")])
def test_backward_bucket_windows(C, dtype):
    """More blocks of 64 channels than bucket counters are in LDS at a time: two and three windows."""
    layer, x, p = rand_layer(C, 2, C, 4, 50, 1, 1, dtype, "nhwc")
    run(layer, x, dtype, "softplus", p, seed=3)


def test_backward_vector_dx_of_more_elements_than_one_launch():
    """dx of 4.3e9 elements (2^32 and a slice's rest) through the kernel with a thread per element.  k = 1: dx is dy
    on the routed channel and dy of the residual over |U| = 64 elsewhere, exact in bfloat16."""
    B, C, HW = 3_900_000, 65, 17
    z = np.zeros
    layer = MoceLayer(C, 2, 1, HW, 1, "bf16", "nchw", z((1, 1)), z((1, 1)), a=z((1, 1)), c=z(1))
    x = torch.zeros((B, C, HW, 1), dtype=torch.bfloat16, device="cuda")
    dy = torch.randn((B, 2, HW, 1), device="cuda").bfloat16()
    dx = layer.backward(x, dy, torch.full_like(x, float("nan")))["dx"]
    for part in (slice(0, 1000), slice(B // 2, B // 2 + 1000), slice(B - 20_000, B)):
        assert torch.equal(dx[part, :1], dy[part, :1])
        assert torch.equal(dx[part, 1:], (dy[part, 1:] / 64).expand(dx[part, 1:].shape))
    assert not torch.isnan(dx.view(-1)[::257].float().sum())


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_backward_vector_dalpha_of_more_rows_than_one_launch(layout):
    """70 million (image, expert) rows, a wave each, over one position: more than a launch holds.  The parameter
    gradients are sums over the images, so those of the batch are those of its halves added; float32 sums of 1.1
    million images in other groups (5e-7 of the largest entry) and a wide margin."""
    B, C, E = 1_100_000, 65, 65
    layer, _, _ = rand_layer(3, 1, C, E, 2, 1, 1, "bf16", layout)
    x = torch.randn((B, C, 1, 1) if layout == "nchw" else (B, 1, 1, C), device="cuda").bfloat16()
    dy = torch.randn(layer.y_shape(B), device="cuda").bfloat16()
    nan = lambda n: layer.new_backward_workspace(n).fill_(255)
    whole = layer.backward(x, dy, None, nan(B))
    h = B // 2
    parts = [layer.backward(x[p], dy[p], None, nan(h)) for p in (slice(0, h), slice(h, B))]
    assert torch.equal(whole["dx"], torch.cat([q["dx"] for q in parts]))
    for n in ("dw", "da", "dc"):
        ref = (parts[0][n].double() + parts[1][n].double()).cpu().numpy()
        close(n, whole[n].double().cpu().numpy(), ref)


@pytest.mark.parametrize("C,E,k,gate", [
    (72, 66, 70, "softplus"),       # one expert past a chunk, lists of nearly every expert
    (320, 300, 300, "softplus"),    # lists of 280 entries
    (600, 590, 128, "mlp"),
    (4300, 4098, 9, "softplus"),    # one chunk past what is marked at a time
    (4400, 4400, 270, "softplus"),  # the same, 270 entries a channel
])
def test_backward_long_channel_lists(C, E, k, gate):
    """Slopes of k^-0.5, so that g stays within a few units whatever k: with 0.7 a row of 300 entries meets
    temperatures of 1e-3, and logits over them of 4e3, whose float32 rounding (2.4e-4 of a coefficient) alone is ten
    times the tolerance."""
    layer, x, p = rand_layer(C + k, 2, C, E, k, 1, 1, "f32", "nchw", gate=gate, a_scale=k ** -0.5)
    run(layer, x, "f32", gate, p, seed=C)
