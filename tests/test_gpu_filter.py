"""The traversal's matrix-core filter at the places where it can go wrong:
coordinates and squares that are ties between two halves, squared distances
equal to or one rounding from a squared radius, frames scaled far up and down,
offset far from the origin, radii of very different sizes, and super-clusters
it does not serve (periodic boxes a few radii wide). Lists bit for bit and
counts exactly as the oracle's."""
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


def _dyadic(n, seed, bits, spread=0.0):
    """Positions on multiples of 2^-bits in [0, 1), radii whose squares are sums of three squares of that grid (so
    pairs at exactly the radius occur), times e^U(-spread, spread) when given."""
    rng = np.random.default_rng(seed)
    p = rng.integers(0, 1 << bits, (3, n)) / float(1 << bits)
    r = workloads.radius_for_neighbours(n, 50.0)
    k = np.maximum(1, np.rint(r * (1 << bits) * rng.uniform(0.7, 1.2, (3, n)) / np.sqrt(3.0)))
    h = np.sqrt((k * k).sum(0)) / (1 << bits) * np.exp(rng.uniform(-spread, spread, n))
    return p, h


def _check(env, p, h, box, cs, half, period=None):
    sf, ctx, torch = env
    print("filter case n=%d cs=%d half=%d period=%s box=%s" % (p.shape[1], cs, half, period, box), flush=True)
    f = [np.ascontiguousarray(v.astype(np.float32)) for v in (p[0], p[1], p[2], h)]
    t = [torch.from_numpy(v).cuda() for v in f]
    pipe = sf.Pipeline(ctx, p.shape[1], box, cluster_size=cs, half=half, period=period)
    nl = pipe.step(*t)
    torch.cuda.synchronize()
    order = pipe.perm.cpu().numpy()
    xo, yo, zo, ho = (v[order] for v in f)
    offs, jj, mm = oracle.cluster_list(xo, yo, zo, ho, cs, "grid", half=half, period=period)
    info, pool = oracle.encode_all(offs, jj, mm, cs, True)
    np.testing.assert_array_equal(nl.sc_info.cpu().numpy().view(np.uint32), info)
    np.testing.assert_array_equal(nl.pool.cpu().numpy().view(np.uint32)[:nl.used_bytes // 4], pool)
    _, cnt = oracle.density(xo, yo, zo, ho, None, "grid", period=period)
    np.testing.assert_array_equal(pipe.nnb.cpu().numpy(), cnt)


@pytest.mark.parametrize("cs", [4, 8, 16])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("bits", [6, 10])
def test_ties(env, cs, half, bits):
    p, h = _dyadic(20011, 3 + bits, bits)
    _check(env, p, h, workloads.UNIT_BOX, cs, half)


@pytest.mark.parametrize("scale", [2.0 ** -30, 2.0 ** 30])
@pytest.mark.parametrize("offset", [0.0, 1000.0])
def test_scale_and_offset(env, scale, offset):
    p, h = _dyadic(8009, 17, 10)
    b = (offset * scale, (offset + 1.0) * scale)
    _check(env, (p + offset) * scale, h * scale, b * 3, 8, True)


@pytest.mark.parametrize("cs", [4, 8, 16])
def test_radii_of_many_sizes(env, cs):
    p, h = _dyadic(8009, 23, 12, spread=2.5)
    _check(env, p, h, workloads.UNIT_BOX, cs, False)


@pytest.mark.parametrize("n", [700, 20011])
@pytest.mark.parametrize("half", [False, True])
def test_periodic_ties(env, n, half):
    p, h = _dyadic(n, 29, 9)
    _check(env, p, np.minimum(h, 0.49), workloads.UNIT_BOX, 8, half, (1.0, 1.0, 1.0))


@pytest.mark.parametrize("cs", [4, 8, 16])
def test_counting_lists(env, cs):
    """The restricted rounds of the h-iteration (recount 1: lists of the moved particles)."""
    sf, ctx, torch = env
    p, h = _dyadic(20011, 31, 9)
    f = [torch.from_numpy(np.ascontiguousarray(v.astype(np.float32))).cuda() for v in (p[0], p[1], p[2], 1.7 * h)]
    keys, perm = sf.sfc_sort(ctx, f[0], f[1], f[2], workloads.UNIT_BOX)
    xs, ys, zs, hs = sf.sfc_gather(ctx, perm, f)
    h0 = hs.clone()
    # (ties make single counts jump, so not every radius need converge: each round's counts are compared)
    res = sf.h_iterate(ctx, keys, xs, ys, zs, hs, target=50, tol=1, max_iters=6, cluster_size=cs, recount=1)
    walk = h0.clone()
    other = sf.h_iterate(ctx, keys, xs, ys, zs, walk, target=50, tol=1, max_iters=6, cluster_size=cs, recount=2)
    print("cs=%d unconverged %d" % (cs, res.unconverged), flush=True)
    np.testing.assert_array_equal(res.nnb.cpu().numpy(), other.nnb.cpu().numpy())
    np.testing.assert_array_equal(hs.cpu().numpy(), walk.cpu().numpy())
    x, y, z = (t.cpu().numpy() for t in (xs, ys, zs))
    conv = np.abs(res.nnb.cpu().numpy() - 50) <= 1
    _, cnt = oracle.density(x, y, z, hs.cpu().numpy(), None, "grid")
    np.testing.assert_array_equal(cnt[conv], res.nnb.cpu().numpy()[conv])


@pytest.mark.parametrize("cs", [4, 8, 16])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("n,period", [(20011, None), (20011, (1.0, 1.0, 1.0)), (2500, (0.0, 1.0, 0.0))])
def test_condensed_with_outskirts(env, cs, half, n, period):
    """A dense core inside a thin halo: super-clusters whose boxes hold the core and whose spheres do not reach it (the
    particle by particle tests), halo radii both far from and into the core."""
    rng = np.random.default_rng(n + cs)
    core = rng.random(n) < 0.9
    p = np.where(core, 0.47 + 0.01 * rng.standard_normal((3, n)), rng.random((3, n)))
    r = np.sqrt(((p - 0.47) ** 2).sum(0))
    h = np.where(core, 0.002 + 0.1 * np.abs(r), rng.uniform(0.3, 1.05, n) * np.maximum(r, 0.02))
    _check(env, p, np.minimum(h, 0.45), (0.0, 1.0, 0.0, 1.0, 0.0, 1.0), cs, half, period)
