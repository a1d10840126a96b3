"""Steps of networks small enough for one stream, whose last launches are shared between layers: losses, gradients and updated
state of the MLP and of a small LeNet over sizes on both sides of the limits that decide what shares a launch."""
import pytest

import test_gpu_kernels as tk

pytestmark = pytest.mark.gpu
gpu = tk.gpu

CASES = [
    # n, batch, hidden
    (3, 128, 128),   # the small workload
    (1, 1, 1),
    (1, 17, 37),     # rows of no whole vectors
    (2, 100, 256),   # 256 features in the one-kernel head
    (6, 64, 260),
    (1, 300, 40),    # more rows than a group's small tiles take
    (2, 257, 64),
    (6, 128, 512),   # the widest that the one-kernel head takes; more tiles than two per compute unit
    (1, 64, 520),    # beyond: the loss with the softmax, both weight gradients and the update in one launch without it
    (1, 33, 517),    # ... rows of no whole vectors
    (3, 100, 600),   # ... the first layer's weight gradient by itself
]


def _config(pb, n, batch, model, arch, **kw):
    return pb.make_config(model=model, n_replicas=n, batch=batch, in_h=28, in_w=28, in_c=1, n_classes=10, arch=arch, eta_inner=0.05,
                          eta_outer=0.1, momentum=0.9, alpha=0.75, gamma0=0.3, rho0=1.0, weight_decay=1e-3, **kw)


def _run(torch, pb, cfg, n, batch):
    from paper_1707_00424_amd import synth
    gen = torch.Generator(device="cuda").manual_seed(7 * n + batch)
    row = torch.as_tensor(synth.init_params(pb.parle_query_layout(cfg), 3, "uniform")).cuda()
    x0 = row + 0.02 * torch.randn((n, row.numel()), generator=gen, device="cuda") * row.std()
    P = pb.Parle(cfg, x0.contiguous())
    images = torch.randn((n, batch, 28, 28, 1), generator=gen, device="cuda")
    labels = torch.randint(0, 10, (n, batch), generator=gen, device="cuda").int()
    return P, images, labels


def _segments(pb, cfg, row):
    return {s["name"]: row[s["offset"]:s["offset"] + s["size"]].reshape(s["shape"]) for s in pb.parle_query_layout(cfg)}


def _check_update(P, cfg, before, after, N):
    """The state after a step from the state before it and the step's gradient, in 64 bits."""
    y, x, v, z = (before[k][:, :N].double() for k in ("y", "x", "vy", "z"))
    d = P.grad[:, :N].double() + cfg.weight_decay * y + cfg.gamma0 * (y - x)
    vn = cfg.momentum * v + d
    yn = y - cfg.eta_inner * (d + cfg.momentum * vn)
    zn = cfg.alpha * z + (1 - cfg.alpha) * yn
    for name, want in (("vy", vn), ("y", yn), ("z", zn)):
        # a handful of roundings of values no larger than those that enter
        bound = 8 * 2.0 ** -24 * (want.abs() + y.abs() + d.abs() + v.abs() + z.abs())
        assert ((after[name][:, :N].double() - want).abs() <= bound).all(), name


@pytest.mark.parametrize("case", CASES)
def test_mlp_steps(gpu, case):
    torch, pb = gpu
    n, batch, hidden = case
    cfg = _config(pb, n, batch, pb.MODEL_MLP, (hidden, 0, 0, 0))
    P, images, labels = _run(torch, pb, cfg, n, batch)
    N = P.sizes.n_params
    loss = torch.full((n,), float("nan"), device="cuda")
    for _ in range(2):
        before = {k: getattr(P, k).clone() for k in ("x", "y", "vy", "z")}
        P.grad[:, :N].fill_(float("nan"))
        P.parle_inner_step(images, labels, loss)
        after = {k: getattr(P, k) for k in ("y", "vy", "z")}
        for a in range(n):
            seg = {k: t.double().requires_grad_(True) for k, t in _segments(pb, cfg, before["y"][a]).items()}
            h = (images[a].double().reshape(batch, -1) @ seg["fc1.w"].reshape(hidden, -1).t() + seg["fc1.b"]).relu()
            logits = h @ seg["fc2.w"].reshape(10, -1).t() + seg["fc2.b"]
            ref = torch.nn.functional.cross_entropy(logits, labels[a].long())
            assert abs(loss[a].item() - ref.item()) <= 1e-5 * max(1.0, ref.item())
            grads = torch.autograd.grad(ref, list(seg.values()))
            got = _segments(pb, cfg, P.grad[a])
            for (name, _), g in zip(seg.items(), grads):
                # sums of up to 784 fp32 products, and the same again behind them
                assert ((got[name].double() - g).norm() <= 1e-5 * g.norm() + 1e-9), (name, a)
        _check_update(P, cfg, before, after, N)


@pytest.mark.parametrize("model,arch", [("mlp", (64, 0, 0, 0)), ("lenet", (12, 16, 5, 64))])
def test_recorded_block_equals_single_steps(gpu, model, arch):
    torch, pb = gpu
    n, batch, steps = 2, 24, 3
    kind = pb.MODEL_MLP if model == "mlp" else pb.MODEL_LENET
    cfgs = [_config(pb, n, batch, kind, arch, graph_block=g) for g in (0, 1)]
    runs = [_run(torch, pb, c, n, batch) for c in cfgs]
    images = torch.stack([runs[0][1] * (1 + 0.1 * s) for s in range(steps)]).contiguous()
    labels = torch.stack([runs[0][2]] * steps).contiguous()
    losses = [torch.full((steps, n), float("nan"), device="cuda") for _ in cfgs]
    for _ in range(4):
        for s in range(steps):
            runs[0][0].parle_inner_step(images[s], labels[s], losses[0][s])
        runs[1][0].parle_inner_block(images, labels, losses[1])
        torch.cuda.synchronize()
        assert torch.equal(losses[0], losses[1])
        N = runs[0][0].sizes.n_params
        for name in ("y", "vy", "z", "grad"):
            assert torch.equal(getattr(runs[0][0], name)[:, :N], getattr(runs[1][0], name)[:, :N]), name
        for P, _, _ in runs:
            P.parle_outer_step()


@pytest.mark.parametrize("case", [
    # n, batch, image side, channels, first layer's outputs, window: 24 x 24, ragged tiles of windows, odd sides, whole and partial vectors
    (2, 5, 28, 1, 20, 5), (1, 3, 15, 1, 12, 4), (3, 2, 17, 3, 32, 3), (1, 1, 14, 2, 4, 3), (2, 400, 17, 1, 16, 5), (1, 33, 32, 3, 28, 3),
    # several workgroups per image: eleven for the forward pass of 23 x 23 windows and three for their gradient, ragged shares; 18 and five
    (1, 2, 48, 1, 8, 3), (2, 3, 64, 1, 4, 5)])
def test_first_layer_with_its_pool(gpu, case):
    """Loss and every gradient of a LeNet whose first layer runs as one operation with its pool."""
    torch, pb = gpu
    n, batch, side, ch, c1, k = case
    gen = torch.Generator(device="cuda").manual_seed(sum(case))
    cfg = pb.make_config(model=pb.MODEL_LENET, n_replicas=n, batch=batch, in_h=side, in_w=side, in_c=ch, n_classes=10, arch=(c1, 12, k, 24),
                         eta_inner=0.05, eta_outer=0.1, gamma0=0.3, rho0=1.0)
    layout = pb.parle_query_layout(cfg)
    from paper_1707_00424_amd import synth
    x0 = torch.stack([torch.as_tensor(synth.init_params(layout, 3 + a, "uniform")) for a in range(n)]).cuda()
    x0 += 0.05 * torch.randn(x0.shape, generator=gen, device="cuda")
    P = pb.Parle(cfg, x0.contiguous())
    images = torch.randn((n, batch, side, side, ch), generator=gen, device="cuda")
    labels = torch.randint(0, 10, (n, batch), generator=gen, device="cuda").int()
    loss = torch.full((n,), float("nan"), device="cuda")
    P.parle_inner_step(images, labels, loss)
    eval_loss, _, _ = P.parle_eval(-1, images.reshape(-1, side, side, ch), labels.reshape(-1))

    def logits_of(seg, x):
        x = x.double().permute(0, 3, 1, 2)
        for name in ("conv1", "conv2"):
            x = torch.nn.functional.conv2d(x.cpu(), seg[name + ".w"].permute(0, 3, 1, 2).cpu(), seg[name + ".b"].cpu()).relu()
            x = torch.nn.functional.max_pool2d(x, 2)
        h = x.permute(0, 2, 3, 1).reshape(x.shape[0], -1).cuda()
        h = (h @ seg["fc1.w"].reshape(seg["fc1.b"].numel(), -1).t() + seg["fc1.b"]).relu()
        return h @ seg["fc2.w"].reshape(10, -1).t() + seg["fc2.b"]

    for a in range(n):
        seg = {key: t.double().requires_grad_(True) for key, t in _segments(pb, cfg, x0[a]).items()}
        ref = torch.nn.functional.cross_entropy(logits_of(seg, images[a]), labels[a].long())
        assert abs(loss[a].item() - ref.item()) <= 1e-5 * max(1.0, ref.item())
        got = _segments(pb, cfg, P.grad[a])
        for name, g in zip(seg, torch.autograd.grad(ref, list(seg.values()))):
            # fp32 sums; an input within rounding of a ReLU's or a pool's decision would show as 1e-3 and more: none at these seeds
            assert (got[name].double() - g).norm() <= 2e-5 * g.norm() + 1e-9, (name, a, ((got[name].double() - g).norm() / g.norm()).item())
    with torch.no_grad():
        mean = {key: t.double() for key, t in _segments(pb, cfg, x0.double().mean(0).float()).items()}
        ref = torch.nn.functional.cross_entropy(logits_of(mean, images.reshape(-1, side, side, ch)), labels.reshape(-1).long())
    assert abs(eval_loss - ref.item()) <= 1e-5 * max(1.0, ref.item())


@pytest.mark.parametrize("case", [
    # n, batch, image side, channels, first layer's outputs, window: LeNet's own, windows of 9, 16 and 27 values
    (6, 128, 28, 1, 20, 5), (3, 100, 17, 1, 16, 3), (2, 150, 21, 1, 12, 4), (2, 120, 16, 3, 32, 3)])
def test_first_layer_takes_the_largest_output_of_the_convolution_alone(gpu, case):
    """Images that repeat themselves after a window's side, and every second output channel with equal weights: the four outputs of
    such a channel under a pool window are sums of the same products in four orders, and rounding decides which one is the largest.
    The layer by itself (convolution, bias and ReLU) says which one gets the gradient, in the network as well."""
    torch, pb = gpu
    from paper_1707_00424_amd import synth
    n, batch, side, ch, c1, k = case
    gen = torch.Generator(device="cuda").manual_seed(sum(case))
    cfg = pb.make_config(model=pb.MODEL_LENET, n_replicas=n, batch=batch, in_h=side, in_w=side, in_c=ch, n_classes=10, arch=(c1, 12, k, 24),
                         eta_inner=0.05, eta_outer=0.1, gamma0=0.3, rho0=1.0)
    layout = pb.parle_query_layout(cfg)
    x0 = torch.stack([torch.as_tensor(synth.init_params(layout, 3 + a, "uniform")) for a in range(n)]).cuda()
    for a in range(n):
        _segments(pb, cfg, x0[a])["conv1.w"].reshape(c1, -1)[::2] = torch.rand((c1 // 2, 1), generator=gen, device="cuda") * 0.1 + 0.05
    P = pb.Parle(cfg, x0.contiguous())
    reps = side // k + 1
    images = torch.rand((n, batch, k, k, ch), generator=gen, device="cuda").repeat(1, 1, reps, reps, 1)[:, :, :side, :side].contiguous()
    labels = torch.randint(0, 10, (n, batch), generator=gen, device="cuda").int()
    P.parle_inner_step(images, labels, torch.empty(n, device="cuda"))

    out = side - k + 1
    w, bias = (torch.stack([_segments(pb, cfg, x0[a])[name] for a in range(n)]).contiguous() for name in ("conv1.w", "conv1.b"))
    y = torch.empty((n, batch, out, out, c1), device="cuda")
    pb.parle_k_conv_forward(pb.parle_conv_desc(0, n, batch, side, side, ch, c1, k, 1, 0), images, w, bias, None, 1, y)
    half = out // 2
    win = y[:, :, :2 * half, :2 * half].reshape(n, batch, half, 2, half, 2, c1).permute(0, 1, 2, 4, 6, 3, 5).reshape(n, batch, half, half, c1, 4)
    pooled = win.amax(-1)
    assert ((win - pooled[..., None]).abs() < 1e-5).sum(-1)[..., ::2].min() == 4 and (win != pooled[..., None]).any()
    at = (win == pooled[..., None]).int().argmax(-1)  # the first of equals
    for a in range(n):
        seg = {key: t.double() for key, t in _segments(pb, cfg, x0[a]).items()}
        p = pooled[a].double().requires_grad_(True)
        x = torch.nn.functional.conv2d(p.permute(0, 3, 1, 2).cpu(), seg["conv2.w"].permute(0, 3, 1, 2).cpu(), seg["conv2.b"].cpu()).relu()
        h = torch.nn.functional.max_pool2d(x, 2).permute(0, 2, 3, 1).reshape(batch, -1).cuda()
        h = (h @ seg["fc1.w"].reshape(seg["fc1.b"].numel(), -1).t() + seg["fc1.b"]).relu()
        loss = torch.nn.functional.cross_entropy(h @ seg["fc2.w"].reshape(10, -1).t() + seg["fc2.b"], labels[a].long())
        dp = torch.autograd.grad(loss, p)[0] * (pooled[a] > 0)
        dy = torch.zeros(win[a].shape, dtype=torch.float64, device="cuda").scatter_(-1, at[a][..., None], dp[..., None])
        dy = dy.reshape(batch, half, half, c1, 2, 2).permute(0, 1, 4, 2, 5, 3).reshape(-1, c1)
        xd = images[a].double()
        cols = torch.stack([xd[:, r:r + 2 * half, c:c + 2 * half] for r in range(k) for c in range(k)], 3).reshape(dy.shape[0], -1)
        ref, got = dy.t() @ cols, _segments(pb, cfg, P.grad[a])["conv1.w"].reshape(c1, -1)
        # fp32 sums; one window's gradient given to another output shows as 1e-4 and more of its channel's
        assert ((got.double() - ref).norm(dim=1) <= 2e-5 * ref.norm(dim=1) + 1e-9).all().item(), a
