"""The seed network's kernels at the sizes where their work is split: inference
in groups of 64 samples over a fixed grid, the gradient's tiles of 16 over one
to 256 blocks of four waves and its two-step reduction, and the features' key
window, against the oracle. Bounds: an FP32 sum of k terms is off by at most
k 2^-24 times the sum of their sizes; the bf16 errors entering the gradient's
products bound it to 1e-3 of its norm per tensor."""
import numpy as np
import pytest

import oracle
from paper_2602_19873_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2602_19873_amd as sf
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    torch.cuda.set_device(0)
    ctx = sf.Context(0)
    yield sf, ctx, torch
    ctx.close()


def _inputs(env, n, seed):
    sf, ctx, torch = env
    rng = np.random.default_rng(seed)
    feat = torch.from_numpy(rng.uniform(-2, 2, (n, 8)).astype(np.float32)).cuda().to(torch.bfloat16)
    p = sf.mlp_init(ctx, seed)
    p += 0.05 * torch.randn(p.shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")
    t = torch.from_numpy(rng.uniform(-1, 1, n).astype(np.float32)).cuda()
    return feat, p, t


@pytest.mark.parametrize("n", [1, 15, 16, 63, 64, 65, 257, 131072 + 3])
def test_inference_sizes(env, n):
    sf, ctx, torch = env
    feat, p, _ = _inputs(env, n, n)
    out = torch.full((n + 64,), 7.0, dtype=torch.float32, device="cuda")
    sf.mlp_infer(ctx, p, feat.view(torch.int16), out=out)
    x = feat.float().double().cpu().numpy()
    y, _ = oracle.mlp_forward(p.cpu().numpy().astype(np.float64), x, quant=True)
    got = out[:n].double().cpu().numpy()
    # a hidden activation on a bf16 rounding boundary may round the other way: 2^-8 of it times a weight, a few of them
    assert np.abs(got - y).max() <= 2e-2 * (1.0 + np.abs(y).max())
    assert np.median(np.abs(got - y)) <= 2e-5 * (1.0 + np.median(np.abs(y)))
    assert bool((out[n:] == 7.0).all())  # nothing past the end


@pytest.mark.parametrize("batch", [1, 16, 17, 64, 65, 4096, 16384, 20000])
def test_gradient_batches(env, batch):
    sf, ctx, torch = env
    n = 20011
    feat, p, t = _inputs(env, n, batch)
    mul = 7919
    grad, loss, _ = sf.mlp_grad(ctx, p, feat.view(torch.int16), t, batch, start=3, mul=mul, add=11)
    again, loss2, _ = sf.mlp_grad(ctx, p, feat.view(torch.int16), t, batch, start=3, mul=mul, add=11)
    assert torch.equal(grad, again) and torch.equal(loss, loss2)  # one order of summation
    at = ((np.arange(batch) + 3) * mul + 11) % n
    x, tt = feat.float().double().cpu().numpy()[at], t.double().cpu().numpy()[at]
    ref_loss, ref = oracle.mlp_loss_grad(p.cpu().numpy().astype(np.float64), x, tt, quant=True)
    assert abs(float(loss) - ref_loss) <= 1e-3 * abs(ref_loss) + 1e-6
    a, b = oracle.mlp_unpack(grad.double().cpu().numpy()), oracle.mlp_unpack(np.asarray(ref))
    for k in a:
        d = np.linalg.norm(a[k].ravel() - b[k].ravel())
        assert d <= 5e-3 * np.linalg.norm(b[k].ravel()) + 1e-6, k


@pytest.mark.parametrize("n,factor", [(1, 1.0), (255, 1.0), (257, 4.0), (5000, 0.3), (5000, 8.0), (60000, 8.0)])
def test_feature_windows(env, n, factor):
    """Radii from small (cells of single particles) to large (cells reaching far beyond the staged keys)."""
    sf, ctx, torch = env
    s = workloads.uniform_varied(n, 5 + n, target=60.0)
    f = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (s.x, s.y, s.z, (factor * s.h).astype(np.float32))]
    keys, perm = sf.sfc_sort(ctx, f[0], f[1], f[2], s.box)
    x, y, z, h = sf.sfc_gather(ctx, perm, f)
    feat = sf.hseed_features(ctx, keys, x, y, z, h, None, 1.0, 60).view(torch.bfloat16).double().cpu().numpy()[:n]
    xa, ya, za, ha = (t.cpu().numpy() for t in (x, y, z, h))
    ref = oracle.hseed_features(keys.cpu().numpy().view(np.uint64), ha, None, oracle.cluster_bboxes(xa, ya, za, ha, 8),
                                1.0, 60)
    # bf16 of a float32 value: half an ulp (2^-9) and its rounding; the level columns may jump where log2 is a tie
    bad = np.abs(feat - ref) > 2.0 ** -8 * (np.abs(ref) + 2.0 ** -8)
    assert bad.any(1).mean() <= 1e-3
