"""Lists of systems of small clumps, where a super-cluster spans gaps much wider
than the radii and the matrix-core filter leaves most tiles open for the exact
tests: bit for bit the oracle's for every cluster size and list form, open and
periodic, in batches (whose padding is NaN) and through counting lists."""
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


def _clumps(n, per, target, seed):
    """n particles in clumps of about `per`, radii for about `target` neighbours in a clump's core."""
    rng = np.random.default_rng(seed)
    k = max(2, n // per)
    sigma = 0.25 * k ** (-1.0 / 3.0) / 6.0
    p = (rng.random((3, k))[:, rng.integers(0, k, n)] + sigma * rng.standard_normal((3, n))) % 1.0
    h = 2.5 * sigma * (3.0 * target / (4.0 * np.pi * per)) ** (1.0 / 3.0) * rng.uniform(0.7, 1.3, n)
    return [np.minimum(a, np.float32(1.0 - 2.0 ** -24)).astype(np.float32) for a in (*p, np.minimum(h, 0.4))]


@pytest.mark.parametrize("period", [None, (1.0, 1.0, 1.0)])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("cs", [4, 8, 16])
@pytest.mark.parametrize("n,per,target", [(133, 5, 3.0), (20011, 47, 30.0), (70001, 20, 6.0), (200003, 50, 10.0)])
def test_lists(env, n, per, target, cs, half, period):
    sf, ctx, torch = env
    print("open tiles n=%d per=%d T=%g cs=%d half=%d period=%s" % (n, per, target, cs, half, period), flush=True)
    f = _clumps(n, per, target, n + per)
    pipe = sf.Pipeline(ctx, n, workloads.UNIT_BOX, cluster_size=cs, half=half, period=period)
    nl = pipe.step(*(torch.from_numpy(v).cuda() for v in f))
    host = [v.cpu().numpy() for v in pipe.sorted[:4]]
    offs, jj, mm = oracle.cluster_list(*host, cs, "grid", half=half, period=period)
    info, pool = oracle.encode_all(offs, jj, mm, cs, True)
    np.testing.assert_array_equal(nl.sc_info.cpu().numpy().view(np.uint32), info)
    np.testing.assert_array_equal(nl.pool.cpu().numpy().view(np.uint32)[:nl.used_bytes // 4], pool)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("cs", [4, 8, 16])
def test_batch_and_counting_lists(env, cs, half):
    sf, ctx, torch = env
    print("open tiles in batches cs=%d half=%d" % (cs, half), flush=True)
    systems = [_clumps(n, 30, 12.0, n) for n in (3001, 70, 9013)]
    counts = [len(s[0]) for s in systems]
    b = sf.Batch(ctx, counts, [workloads.UNIT_BOX] * 3)
    f = [torch.from_numpy(np.concatenate([s[k] for s in systems])).cuda() for k in range(4)]
    keys, perm = sf.batch_sort(ctx, b, *f[:3])
    xs, ys, zs, h0 = sf.batch_gather(ctx, b, perm, f)
    bbox = sf.batch_build_clusters(ctx, b, xs, ys, zs, h0, cluster_size=cs)
    nl = sf.batch_build_nlist(ctx, b, keys, xs, ys, zs, h0, bbox, cluster_size=cs, half=half)
    info, pool = nl.sc_info.cpu().numpy().view(np.uint32), nl.pool.cpu().numpy().view(np.uint32)
    for s, c in enumerate(counts):
        lo, (s0, s1) = int(b.pbase[s]), b.sc_range(s)
        host = [v.cpu().numpy()[lo:lo + c] for v in (xs, ys, zs, h0)]
        offs, jj, mm = oracle.cluster_list(*host, cs, "grid", half=half)
        winfo, wpool = oracle.encode_all(offs, jj, mm, cs, True)
        np.testing.assert_array_equal(info[s0:s1, 1], winfo[:, 1])
        got = np.concatenate([pool[info[s0, 0]:info[s1, 0] if s1 < len(info) else nl.used_bytes // 4]])
        np.testing.assert_array_equal(got, wpool)
    out = {}
    for recount in (1, 2):
        h = h0.clone()
        r = sf.batch_h_iterate(ctx, b, keys, xs, ys, zs, h, target=9, tol=1, cluster_size=cs, half=half, recount=recount)
        real = torch.cat([torch.arange(int(b.pbase[s]), int(b.pbase[s]) + c) for s, c in enumerate(counts)]).cuda()
        out[recount] = (h[real].cpu().numpy(), r.nnb[real].cpu().numpy(), r.sys_rounds.tolist(), r.moved, r.unconverged)
    for k in range(2):
        np.testing.assert_array_equal(out[1][k], out[2][k])
    assert out[1][2:] == out[2][2:]
