"""GPU parity of the learned depth prefilter (BF16 matrix-core kernels with
fp32 accumulation) against the oracle.

Per layer, the oracle recomputes the GPU's result from the GPU's own bf16
activations and upstream gradients with the definition's operators -- 3x3
convolution with the bf16-rounded taps, after nearest 2x upsampling for the
decoder layers -- in float64, so the only differences are accumulation order
and the final bf16 rounding: outputs within 1 bf16 ulp-scale (0.8% relative
plus a small absolute floor), weight gradients within 1e-3 relative.  The
forward pass also meets the plain float64 oracle (fp32 master weights, no
bf16 rounding anywhere) within 2e-2 per layer.  End to end against the
float64 oracle on bf16-rounded weights and input: per-layer gradient cosine
>= 0.999.  Adam matches the oracle's update; a zero head is the identity
exactly.  The end-to-end comparison runs the oracle with bf16 rounding of
everything the kernels store in bf16, so both sides take their relu
decisions on the same values; without it, decisions at near-zero sums differ
and compound.

Sizes: 2 x 32x48 and 2 x 40x56 (the deepest source is 5x7: odd sizes and
ragged column runs in the parity-split kernels) and 1 x 256x256, where the
weight-gradient reductions leave their small-size regime: e1 runs 128 chunks
of 512 pixels (8 staging rounds each), e2 and d1 64 chunks of 256 pixels (4
rounds), as the full-size training shapes do with more chunks."""
import numpy as np
import pytest

from oracle import denoise as D

pytestmark = pytest.mark.gpu

N, H, W = 2, 32, 48


def _log(*a):
    print(*a, flush=True)


def _setup(seed=0, shape=(N, H, W)):
    nb, h, w = shape
    import torch
    import paper_1708_00783_amd as T
    rng = np.random.default_rng(seed)
    P = D.init_params(seed, np.float64)
    for k in P:
        if k.endswith(".b"):
            P[k] = rng.standard_normal(P[k].shape) * 0.05
    P["head.w"] = rng.standard_normal(P["head.w"].shape) * 0.05
    P = {k: v.astype(np.float32).astype(np.float64) for k, v in P.items()}
    # a smooth surface with depth-sensor-like noise and holes (realistic input scale)
    yy, xx = np.mgrid[0:h, 0:w]
    depth = np.stack([1.2 + 1.5 * n + 0.3 * np.sin(xx / (7.0 + n)) + 0.2 * np.cos(yy / 5.0) for n in range(nb)])
    depth = (depth + rng.normal(0, 0.004, depth.shape)).astype(np.float32)
    depth[0, 5:9, 10:20] = 0.0
    if nb > 1:
        depth[1, :, :3] = 0.0
    target = (depth + rng.normal(0, 0.02, depth.shape)).astype(np.float32)
    target[0, 20:24] = 0.0
    net = T.Denoiser(nb, h, w, training=True)
    net.set_params(T.nn_flatten(P))
    d_depth = torch.from_numpy(depth).cuda()
    out = net.forward(d_depth)
    return T, net, P, depth, target, out


def _bf(net, name):
    import paper_1708_00783_amd as T
    return T.bf16_bits_to_float(net.tensor(name)).astype(np.float64)


def _close(gpu, ref, tag, rel=8e-3, floor=None):
    floor = floor if floor is not None else 1e-3 * max(1e-6, np.abs(ref).max())
    err = np.abs(gpu - ref)
    bad = err > rel * np.abs(ref) + floor
    assert not bad.any(), f"{tag}: {bad.sum()} of {bad.size} off, max err {err.max():.3g} (ref max {np.abs(ref).max():.3g})"


def _rb(w):
    return D.to_bf16(w.astype(np.float32)).astype(np.float64)


LAYER_IO = {"e1": ("input", 1, False, None), "e2": ("e1", 2, False, None), "e3": ("e2", 2, False, None),
            "e4": ("e3", 2, False, None), "d3": ("e4", 1, True, "e3"), "d2": ("d3", 1, True, "e2"),
            "d1": ("d2", 1, True, "e1")}


# 40 x 56: the deepest source is 5 x 7, so the folded decoder kernels and the
# stride-2 parity split meet odd sizes and ragged column runs; 256 x 256: the
# weight-gradient reductions run 128 chunks (e1) and several 64-pixel staging
# rounds per chunk (e1, e2, d1)
SHAPES = [(N, H, W), (2, 40, 56), (1, 256, 256)]


@pytest.mark.parametrize("shape", SHAPES)
def test_forward_layers_match_oracle(shape):
    T, net, P, depth, target, out = _setup(1, shape)
    x = _bf(net, "input")
    assert np.array_equal(x[..., 0], D.to_bf16(depth * 0.25)) and np.array_equal(x[..., 1], (depth > 0) * 1.0)
    hp = D.make_input(depth.astype(np.float64))[..., 2]
    assert np.allclose(x[..., 2], hp, rtol=8e-3, atol=1e-4)
    assert not x[..., 3:].any()
    for name, (src, stride, up, skip) in LAYER_IO.items():
        a = _bf(net, src)
        if name == "e1":
            a = a[..., :3]
        ref = D.conv(D.up2(a) if up else a, _rb(P[name + ".w"]), P[name + ".b"], stride)
        if skip:
            ref = ref + _bf(net, skip)
        ref = np.maximum(ref, 0)
        _close(_bf(net, name), ref, name)
        _log(f"{name}: ok, {ref.shape}, max {ref.max():.3g}")
    d1 = _bf(net, "d1")
    delta = D.conv(d1, P["head.w"], P["head.b"])[..., 0]
    ref = np.where(depth > 0, depth + D.CORRECTION_SCALE * delta, 0.0)
    got = out.cpu().numpy()
    assert np.abs(got - ref).max() < 1e-5
    assert np.all(got[depth == 0] == 0)


@pytest.mark.parametrize("shape", SHAPES)
def test_backward_layers_match_oracle(shape):
    import torch
    T, net, P, depth, target, out = _setup(2, shape)
    loss = net.backward(torch.from_numpy(target).cuda()).cpu().numpy()
    o = out.cpu().numpy().astype(np.float64)
    l_ref, g_ref, n_ref = D.loss_and_grad_out(o, depth, target)
    assert int(loss[1]) == n_ref and abs(loss[0] - l_ref) < 1e-5 * max(1.0, l_ref)
    dd = net.tensor("ddelta").cpu().numpy().astype(np.float64).reshape(shape)
    assert np.allclose(dd, np.where(depth > 0, D.CORRECTION_SCALE * g_ref, 0), rtol=1e-6, atol=1e-12)
    grads = T.nn_unflatten(net.tensor("grads").cpu().numpy().reshape(-1))
    # head: gradient at d1 and head parameters
    d1 = _bf(net, "d1")
    dd1, dwh, dbh = D.conv_backward(d1, P["head.w"], dd[..., None])
    _close(_bf(net, "grad_d1"), dd1 * (d1 > 0), "grad_d1")
    assert np.allclose(grads["head.w"], dwh, rtol=1e-3, atol=1e-6 * np.abs(dwh).max())
    assert np.allclose(grads["head.b"], dbh, rtol=1e-4, atol=1e-9)
    # conv layers, from the GPU's own upstream gradients
    skip_to = {"e1": "d1", "e2": "d2", "e3": "d3"}
    for name, (src, stride, up, _) in reversed(list(LAYER_IO.items())):
        g = _bf(net, "grad_" + name)
        a = _bf(net, src)
        if name == "e1":
            a = a[..., :3]
        a_in = D.up2(a) if up else a
        wb = _rb(P[name + ".w"])
        dx, dw, db = D.conv_backward(a_in, wb, g, stride)
        cos = float(np.sum(grads[name + ".w"] * dw) / (np.linalg.norm(grads[name + ".w"]) * np.linalg.norm(dw)))
        rel = float(np.linalg.norm(grads[name + ".w"] - dw) / np.linalg.norm(dw))
        assert rel < 1e-3, (name, rel)
        assert np.allclose(grads[name + ".b"], db, rtol=1e-3, atol=1e-6 * max(1e-9, np.abs(db).max()))
        _log(f"{name}: dW rel {rel:.2e} cos {cos:.6f}")
        if name == "e1":
            continue
        if up:
            dx = D.up2_backward(dx)
        if src in skip_to:
            dx = dx + _bf(net, "grad_" + skip_to[src])
        _close(_bf(net, "grad_" + src), dx * (a > 0), "grad_" + src)


@pytest.mark.parametrize("shape", [(1, 8, 8), (3, 24, 136), (1, 136, 72)])
def test_tiles_and_blocks_at_their_edges(shape):
    """Activations, gradients at the conv inputs and weight gradients where the
    kernels' tiles and blocks end: the smallest image (sources of 1 x 1, less
    than a tile in both directions), and widths and heights one past 1, 2 and 4
    tiles of 16 columns, of blocks of 32 columns and of 2 or 4 rows, with 3
    images (the tiles are not a multiple of the 8 they are dealt in).  The
    bounds are those of the tests of whole layers."""
    import torch
    T, net, P, depth, target, out = _setup(11, shape)
    net.backward(torch.from_numpy(target).cuda())
    grads = T.nn_unflatten(net.tensor("grads").cpu().numpy().reshape(-1))
    skip_to = {"e1": "d1", "e2": "d2", "e3": "d3"}
    for name, (src, stride, up, skip) in reversed(list(LAYER_IO.items())):
        a = _bf(net, src)
        if name == "e1":
            a = a[..., :3]
        y = D.conv(D.up2(a) if up else a, _rb(P[name + ".w"]), P[name + ".b"], stride)
        _close(_bf(net, name), np.maximum(y + _bf(net, skip) if skip else y, 0), f"{shape} {name}")
        dx, dw, db = D.conv_backward(D.up2(a) if up else a, _rb(P[name + ".w"]), _bf(net, "grad_" + name), stride)
        assert np.linalg.norm(grads[name + ".w"] - dw) < 1e-3 * np.linalg.norm(dw), (shape, name)
        assert np.allclose(grads[name + ".b"], db, rtol=1e-3, atol=1e-6 * max(1e-9, np.abs(db).max())), (shape, name)
        if name == "e1":
            continue
        if up:
            dx = D.up2_backward(dx)
        if src in skip_to:
            dx = dx + _bf(net, "grad_" + skip_to[src])
        _close(_bf(net, "grad_" + src), dx * (a > 0), f"{shape} grad_{src}")
    d1, dd = _bf(net, "d1"), net.tensor("ddelta").cpu().numpy().astype(np.float64).reshape(shape)
    dx, dw, db = D.conv_backward(d1, P["head.w"], dd[..., None])
    _close(_bf(net, "grad_d1"), dx * (d1 > 0), f"{shape} grad_d1")
    assert np.allclose(grads["head.w"], dw, rtol=1e-3, atol=1e-6 * np.abs(dw).max()), shape
    assert np.allclose(grads["head.b"], db, rtol=1e-4, atol=1e-9), shape


@pytest.mark.parametrize("name", ["e1", "e2", "e3", "e4", "d3", "d2", "d1", "head"])
def test_a_non_finite_activation_spoils_only_its_own_taps(name):
    """An infinity in the last pixel of a layer's input and a NaN in the first:
    of the layer's weight gradients, those of their channels and of the taps
    that lead to them from an output inside the image are not finite, all
    others are as before (24 x 40: blocks and tiles reach past every border,
    where zeros stand for the outputs)."""
    import torch
    T, net, P, depth, target, out = _setup(13, (1, 24, 40))
    t = torch.from_numpy(target).cuda()
    src, stride, up, _ = LAYER_IO.get(name, ("d1", 1, False, None))

    def weight_grads():
        net.backward(t)
        return T.nn_unflatten(net.tensor("grads").cpu().numpy().reshape(-1))[name + ".w"].copy()

    before = weight_grads()
    x = net.tensor(src)
    mark = np.zeros(x.shape)
    for pixel, channel, bits in ((-1, 1, 0x7f80), (0, 2, 0x7fc0)):
        x[0, pixel, pixel, channel] = bits
        mark[0, pixel, pixel, channel] = 1.0
    after = weight_grads()
    if name == "e1":
        mark = mark[..., :3]
    mark = D.up2(mark) if up else mark
    g = np.ones((1, *[-(-n // stride) for n in mark.shape[1:3]], before.shape[0]))
    spoilt = D.conv_backward(mark, np.zeros_like(before, dtype=np.float64), g, stride)[1] > 0
    assert np.isfinite(before).all() and spoilt.any() and not spoilt.all()
    _log(f"{name}: {int(spoilt.sum())} of {spoilt.size} weights read the two pixels")
    assert np.array_equal(~np.isfinite(after), spoilt)
    assert np.array_equal(after[~spoilt], before[~spoilt])


def test_end_to_end_gradient_cosine():
    import torch
    T, net, P, depth, target, out = _setup(3)
    net.backward(torch.from_numpy(target).cuda())
    torch.cuda.synchronize()
    grads = T.nn_unflatten(net.tensor("grads").cpu().numpy().reshape(-1))
    Pb = {k: (_rb(v) if k.endswith(".w") and not k.startswith("head") else v) for k, v in P.items()}
    # the oracle at the kernels' storage precision: bf16 input, activations and gradients
    o, c = D.forward(Pb, depth.astype(np.float64), q=lambda a: D.to_bf16(a).astype(np.float64))
    _, g, _ = D.loss_and_grad_out(o, depth, target)
    G = D.backward(Pb, c, g)
    for k in G:
        a, b = grads[k].reshape(-1).astype(np.float64), G[k].reshape(-1)
        cos = float(a @ b / (np.linalg.norm(a) * np.linalg.norm(b) + 1e-30))
        _log(f"{k}: cosine {cos:.6f}")
        assert cos >= 0.999, (k, cos)


@pytest.mark.parametrize("shape", [(N, H, W), (1, 256, 256)])
def test_forward_against_plain_float64_oracle(shape):
    """The GPU's activations against the plain float64 oracle (fp32 master
    weights, no bf16 rounding of anything): per layer within 2e-2 of the
    layer's largest value, and within 2e-2 in norm; the output depth's
    correction likewise.  (bf16 storage alone moves a layer by <= 1%.)"""
    T, net, P, depth, target, out = _setup(7, shape)
    o, c = D.forward(P, depth.astype(np.float64))
    for name in LAYER_IO:
        got, ref = _bf(net, name), c[name]
        scale = np.abs(ref).max()
        err = np.abs(got - ref)
        rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
        _log(f"{name}: max err {err.max() / scale:.2e} of the layer max, norm {rel:.2e}")
        assert err.max() <= 2e-2 * scale, (name, float(err.max() / scale))
        assert rel <= 2e-2, (name, rel)
    got = out.cpu().numpy().astype(np.float64)
    corr = np.abs(o - depth).max()
    assert corr > 1e-4
    assert np.abs(got - o).max() <= 2e-2 * corr, float(np.abs(got - o).max() / corr)


def test_adam_matches_oracle():
    import torch
    T, net, P, depth, target, out = _setup(4)
    net.backward(torch.from_numpy(target).cuda())
    torch.cuda.synchronize()
    g = net.tensor("grads").cpu().numpy().reshape(-1).astype(np.float64)
    p0 = net.get_params().cpu().numpy().astype(np.float64)
    net.adam_step(1e-3, 0.9, 0.999, 1e-8)
    p1 = net.get_params().cpu().numpy().astype(np.float64)
    Po, st = {"p": p0.copy()}, {}
    D.adam_step(Po, {"p": g}, st, 1, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8)
    assert np.abs(p1 - Po["p"]).max() < 1e-6
    # the forward pass uses the updated weights
    net.forward(torch.from_numpy(depth).cuda())
    assert not np.array_equal(net.tensor("out").cpu().numpy(), out.cpu().numpy())


def test_zero_head_is_identity_and_fuses_like_raw_depth():
    import torch
    import paper_1708_00783_amd as T
    from synth import configs
    d, p, K, _ = configs.c1_frames(3)
    net = T.Denoiser(1, K.height, K.width)
    net.set_params(T.nn_flatten(D.init_params(0)))
    raw = T.Volume(configs.C1_VOLUME, K.width, K.height)
    den = T.Volume(configs.C1_VOLUME, K.width, K.height)
    for k in range(3):
        dk = torch.from_numpy(d[k]).cuda()
        o = net.forward(dk[None])[0]
        assert torch.equal(o, torch.where(dk > 0, dk, torch.zeros_like(dk)))
        raw.frame(dk, K, p[k])
        den.frame(o.contiguous(), K, p[k])
    a, b = raw.voxels_by_position(), den.voxels_by_position()
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


def test_training_reduces_loss():
    """Adam on one fixed batch (noisy planes -> clean planes): the loss falls."""
    import torch
    import paper_1708_00783_amd as T
    rng = np.random.default_rng(5)
    net = T.Denoiser(4, 64, 64, training=True)
    net.set_params(T.nn_flatten(D.init_params(5)))
    yy, xx = np.mgrid[0:64, 0:64]
    base = np.stack([1.0 + 0.01 * (xx * rng.uniform(-1, 1) + yy * rng.uniform(-1, 1)) + rng.uniform(0, 1)
                     for _ in range(4)]).astype(np.float32)
    noisy = torch.from_numpy((base + rng.normal(0, 0.01, base.shape)).astype(np.float32)).cuda()
    clean = torch.from_numpy(base).cuda()
    losses = []
    for it in range(150):
        net.forward(noisy)
        loss = net.backward(clean)
        net.adam_step(2e-4)
        losses.append(float(loss[0].item()))
    _log("loss", losses[:3], losses[-3:])
    assert np.isfinite(losses).all()
    # the untrained prefilter is the identity: its loss is the raw noise; training lowers it
    assert np.mean(losses[-10:]) < 0.9 * losses[0]


def test_training_is_deterministic():
    """Every reduction on the training path sums in a fixed order (no atomics),
    so the same steps from the same parameters give bit-identical weights and
    losses."""
    import torch
    T, net, P, depth, target, out = _setup(6, (2, 40, 56))
    x = torch.from_numpy(depth).cuda()
    t = torch.from_numpy(target).cuda()
    flat = T.nn_flatten(P)

    def run():
        net.set_params(flat)
        losses = []
        for _ in range(5):
            net.forward(x)
            losses.append(net.backward(t).cpu().numpy().copy())
            net.adam_step(1e-3)
        torch.cuda.synchronize()
        return net.get_params().cpu().numpy().copy(), np.stack(losses)

    p1, l1 = run()
    p2, l2 = run()
    assert not np.array_equal(p1, flat.astype(np.float32))   # the steps did change the weights
    assert np.array_equal(p1.view(np.uint32), p2.view(np.uint32))
    assert np.array_equal(l1.view(np.uint32), l2.view(np.uint32))
