"""The training kernels at the batch sizes where their tiling changes or leaves remainders:
one sample, the edges of a 32-sample tile, the last batch of one 32-sample tile per workgroup
and the first of 64-sample tiles, and workgroups that take several tiles.

The gradient of a batch is compared with the sum of the gradients of pieces of at most 24
samples (one partial tile each; the same kernels at a fixed batch are held against the
oracle elsewhere).  The targets are so far away (2^40) that dL/dY does not depend on the
network's output, and are scaled with the batch so that it does not depend on the batch
either: every bfloat16 value is then the same in both, and only FP32 sums differ.  At most
about 1000 dependent additions (tiles of one workgroup, then workgroups) of rounding 2^-24
each: 2^-13 of an entry and of its tensor's rms.  The train step must equal the gradient
followed by Adam bit for bit (the same sums, the same update)."""
import numpy as np
import pytest
import torch

from oracle import lite_oracle as L
from oracle import mlp_oracle as M
from paper_2606_15622_amd import inputs as I

pytestmark = pytest.mark.gpu
LR, FAR, PIECE = 1e-3, 2.0 ** 40, 24
SIZES = [1, 31, 32, 33, 8192, 8193, 16 * 1024 + 65]


def fp():
    from paper_2606_15622_amd import fpgpu
    fpgpu.load()
    return fpgpu


def dev(a, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dtype).cuda()


def flat_params(shapes, n_out, seed):
    rng = np.random.default_rng(seed)
    parts = []
    for name, shp in shapes:
        if name[0] == "W":
            p = rng.standard_normal(shp) * np.sqrt(2.0 / shp[1])
        elif name[0] == "b" or name == "x_mean":
            p = rng.standard_normal(shp) * 0.1
        elif name == "x_std":
            p = rng.uniform(0.5, 1.5, shp)
        else:
            p = np.zeros(shp) if name == "y_mean" else np.ones(shp)
        if shp[0] == 16 and name[0] in "Wb":
            p[n_out:] = 0.0
        parts.append(p.ravel())
    return np.concatenate(parts).astype(np.float32)


def check_sum(B, shapes, total, grad_of):
    """grad_of(i0, i1): gradient of samples i0 .. i1 as a batch of their own."""
    g = total.double().cpu().numpy()
    ref = torch.zeros(total.shape, dtype=torch.float64, device="cuda")
    for i in range(0, B, PIECE):
        ref += grad_of(i, min(i + PIECE, B)).double()
    ref = ref.cpu().numpy()
    o = 0
    for name, shp in shapes:
        n = int(np.prod(shp))
        a, b = g[o:o + n], ref[o:o + n]
        rms = float(np.sqrt((b ** 2).mean()))
        assert rms > 0.0, name
        assert np.all(np.abs(a - b) <= 2.0 ** -13 * (np.abs(b) + rms)), (name, float(np.abs(a - b).max() / rms))
        o += n
    assert np.all(g[o:] == 0)


def check_step(net, adam, pd, args, grad, loss):
    """One train step on copies of pd against the gradient and Adam of the same batch."""
    p1, p2 = pd.clone(), pd.clone()
    m1, v1, m2, v2 = (torch.zeros_like(pd) for _ in range(4))
    l1 = torch.zeros_like(loss)
    net.train_step(p1, m1, v1, 1, LR, *args, l1)
    adam(p2, grad, m2, v2, 1, LR)
    torch.cuda.synchronize()
    for a, b in ((p1, p2), (m1, m2), (v1, v2), (l1, loss)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B", SIZES)
@pytest.mark.parametrize("loss_kind", [0, 1])
def test_network_gradient(B, loss_kind):
    F = fp()
    rng = np.random.default_rng(B + loss_kind)
    feats = dev(rng.standard_normal((B, 32)))
    t = np.zeros((B, 16))
    t[:, :9] = rng.integers(1, 8, (B, 9)) * FAR
    A = rng.integers(-2, 3, (B, 81)).astype(np.float64)
    ctx = F.Context(I.couette(ncell=1), 1)
    net = F.Network(ctx, B)
    pd = dev(flat_params(M.SHAPES, 9, B))
    loss = torch.zeros(1, device="cuda")

    def args(i0, i1):
        n = i1 - i0
        sys = np.concatenate([A[i0:i1], -n * t[i0:i1, :9]], 1)
        return feats[i0:i1].contiguous(), dev(n * t[i0:i1]), dev(sys, torch.float64), n, loss_kind

    def grad_of(i0, i1):
        g = torch.zeros(M.N_PARAMS, device="cuda")
        net.grad(pd, *args(i0, i1), g, loss)
        return g

    total = grad_of(0, B)
    full = loss.clone()
    check_sum(B, M.SHAPES[:8], total, grad_of)
    check_step(net, ctx.nn_adam, pd, args(0, B), total, full)


@pytest.mark.parametrize("B", SIZES)
def test_lite_gradient(B):
    F = fp()
    rng = np.random.default_rng(B)
    feats = dev(2.0 * rng.standard_normal((B, 16)))
    t = np.zeros((B, 16))
    t[:, :9] = rng.integers(1, 8, (B, 9)) * FAR
    ctx = F.Context(I.couette(ncell=1), 1)
    net = F.LiteNetwork(ctx, B)
    pd = dev(flat_params(L.SHAPES, 9, B))
    loss = torch.zeros(1, device="cuda")

    def args(i0, i1):
        return feats[i0:i1].contiguous(), dev((i1 - i0) * t[i0:i1]), i1 - i0

    def grad_of(i0, i1):
        g = torch.zeros(F.LITE_PARAMS, device="cuda")
        net.grad(pd, *args(i0, i1), g, loss)
        return g

    total = grad_of(0, B)
    full = loss.clone()
    check_sum(B, L.SHAPES[:10], total, grad_of)
    check_step(net, ctx.lite_adam, pd, args(0, B), total, full)
