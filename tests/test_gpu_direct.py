"""Lists of small systems, built without an octree by 8 or 4 wavefronts a
super-cluster, and of the sizes just above, which walk one: bit for bit the
oracle's, for every cluster size, open and periodic, uniform and condensed."""
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


def _check(env, f, cs, half, period=None):
    sf, ctx, torch = env
    n = len(f[0])
    print("direct n=%d cs=%d half=%d period=%s" % (n, cs, half, period), flush=True)
    f = [np.ascontiguousarray(v.astype(np.float32)) for v in f]
    pipe = sf.Pipeline(ctx, n, workloads.UNIT_BOX, cluster_size=cs, half=half, period=period)
    nl = pipe.step(*(torch.from_numpy(v).cuda() for v in f))
    host = [v.cpu().numpy() for v in pipe.sorted[:4]]
    offs, jj, mm = oracle.cluster_list(*host, cs, "grid", half=half, period=period)
    info, pool = oracle.encode_all(offs, jj, mm, cs, True)
    np.testing.assert_array_equal(nl.sc_info.cpu().numpy().view(np.uint32), info)
    np.testing.assert_array_equal(nl.pool.cpu().numpy().view(np.uint32)[:nl.used_bytes // 4], pool)
    _, cnt = oracle.density(*host, None, "grid", period=period)
    np.testing.assert_array_equal(pipe.nnb.cpu().numpy()[:n], cnt)


def _uniform(n, seed, target):
    rng = np.random.default_rng(seed)
    h = workloads.radius_for_neighbours(n, target) * rng.uniform(0.6, 1.3, n)
    return [*rng.random((3, n)), h]


def _condensed(n, seed):
    rng = np.random.default_rng(seed)
    core = rng.random(n) >= min(0.1, 1500.0 / n)
    p = np.where(core, 0.47 + 0.01 * rng.standard_normal((3, n)), rng.random((3, n)))
    r = np.sqrt(((p - 0.47) ** 2).sum(0))
    s = (20000.0 / n) ** (1.0 / 3.0)
    h = np.where(core, s * (0.002 + 0.1 * np.abs(r)), rng.uniform(0.3, 1.02, n) * np.maximum(r, 0.02))
    return [*p, np.minimum(h, 0.45)]


@pytest.mark.parametrize("period", [None, (1.0, 1.0, 1.0), (0.0, 1.0, 0.0)])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("cs", [4, 8, 16])
@pytest.mark.parametrize("n", [3, 64, 65, 129, 511, 1000, 4099])
def test_smallest(env, n, cs, half, period):
    f = _uniform(n, n + cs, min(20.0, 0.3 * n))
    f[3] = np.minimum(f[3], 0.45)
    _check(env, f, cs, half, period)


@pytest.mark.parametrize("period", [None, (1.0, 1.0, 1.0)])
@pytest.mark.parametrize("cs,n", [(8, 32768), (8, 32769), (4, 32769), (16, 32768), (4, 65536), (4, 65537), (8, 131072),
                                  (8, 131073), (16, 131073), (16, 196608), (16, 196609)])
def test_edges(env, cs, n, period):
    _check(env, _uniform(n, n + cs, 12.0), cs, (n + cs) % 2 == 0, period)


# (above 65,536 particles with clusters of 4 and above 131,072 with 8: the octree walk's particle by particle tests)
@pytest.mark.parametrize("cs,half,n,period", [(cs, half, n, None) for cs in (4, 8, 16) for half in (False, True)
                                              for n in (6001, 20011)] +
                         [(4, False, 70001, None), (4, True, 70001, (1.0, 1.0, 1.0)), (8, True, 140001, None)])
def test_condensed(env, cs, half, n, period):
    _check(env, _condensed(n, n + cs), cs, half, period)
