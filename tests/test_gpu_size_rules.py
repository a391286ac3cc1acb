"""Sizes at which the build changes its launches: blocks of node counts and
lists that add up their own offsets or take prefix sums, leaf levels in blocks
of one or four groups, node ends by 16 or 2 lanes, and short scans. Lists bit
for bit and counts exactly as the oracle's; h-iterations against its counts."""
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


@pytest.mark.parametrize("bucket", [8, 128, 256])
@pytest.mark.parametrize("n", [1, 256, 257, 65536, 65537, 262144, 262145])
def test_lists_at_size_rules(env, n, bucket):
    sf, ctx, torch = env
    print("size rules n=%d bucket=%d" % (n, bucket), flush=True)
    s = workloads.uniform_varied(n, 40 + bucket, target=min(8.0, 0.5 * n)) if n > 1 else workloads.uniform_varied(1, 1, target=0.5)
    pipe = sf.Pipeline(ctx, n, s.box, leaf_bucket=bucket, half=True)
    nl = pipe.step(*(torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (s.x, s.y, s.z, s.h)))
    host = [t.cpu().numpy() for t in pipe.sorted[:4]]
    offs, jj, mm = oracle.cluster_list(*host, 8, "grid", half=True)
    info, pool = oracle.encode_all(offs, jj, mm, 8, True)
    np.testing.assert_array_equal(nl.sc_info.cpu().numpy().view(np.uint32), info)
    assert nl.used_bytes == 4 * len(pool)
    np.testing.assert_array_equal(nl.pool.cpu().numpy().view(np.uint32)[:len(pool)], pool)
    _, cnt = oracle.density(*host)
    np.testing.assert_array_equal(pipe.nnb.cpu().numpy()[:n], cnt)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("n", [65537, 262144, 262145])
def test_iteration_at_size_rules(env, n, half):
    # radii of every round and the closing list (new boxes on the first round's nodes)
    sf, ctx, torch = env
    print("size rules iteration n=%d half=%d" % (n, half), flush=True)
    s = workloads.uniform_global(n, 50, target=25.0)
    f = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (s.x, s.y, s.z, s.h)]
    keys, perm = sf.sfc_sort(ctx, *f[:3], s.box)
    xs, ys, zs, h0 = sf.sfc_gather(ctx, perm, f)
    out = []
    for recount in (0, 1):
        h = h0.clone()
        r = sf.h_iterate(ctx, keys, xs, ys, zs, h, target=16, tol=1, half=half, recount=recount)
        assert r.converged
        out.append((h.cpu().numpy(), r.nnb.cpu().numpy()[:n], r.iters, r.moved, r.nl.sc_info.cpu().numpy(),
                    r.nl.pool.cpu().numpy()[:r.nl.used_bytes // 4]))
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    host = [v.cpu().numpy() for v in (xs, ys, zs)]
    _, cnt = oracle.density(*host, out[0][0])
    np.testing.assert_array_equal(out[0][1], cnt)
    offs, jj, mm = oracle.cluster_list(*host, out[0][0], 8, "grid", half=half)
    info, pool = oracle.encode_all(offs, jj, mm, 8, True)
    np.testing.assert_array_equal(out[0][4].view(np.uint32), info)
    np.testing.assert_array_equal(out[0][5].view(np.uint32), pool)


@pytest.mark.parametrize("kind", ["uniform", "equal", "ties"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 3071, 3072, 3073, 4095, 4096, 4097, 20479, 49151, 49152, 49153])
def test_small_sort(env, n, kind):
    # one launch up to 3072 particles, ordered tiles up to 49152, the radix passes above; equal keys keep their order
    sf, ctx, torch = env
    rng = np.random.default_rng(n)
    p = rng.random((3, n))
    if kind == "equal":
        p[:] = 0.3
    elif kind == "ties":
        p = np.floor(p * 4.0) / 4.0 + rng.random((3, n)) * 1e-9
    p = p.astype(np.float32)
    print("small sort n=%d %s" % (n, kind), flush=True)
    keys, perm = sf.sfc_sort(ctx, *(torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in p), workloads.UNIT_BOX)
    ref = oracle.hilbert_keys(*p, workloads.UNIT_BOX)
    order = np.argsort(ref, kind="stable")
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64)[:n], ref[order])
    np.testing.assert_array_equal(perm.cpu().numpy().view(np.uint32)[:n], order)


@pytest.mark.parametrize("nf", [1, 4, 5, 8])
@pytest.mark.parametrize("n", [1, 262144, 262145])
def test_gather_at_size_rules(env, n, nf):
    sf, ctx, torch = env
    g = torch.Generator(device="cuda").manual_seed(n + nf)
    perm = torch.randperm(n, generator=g, device="cuda")
    f = [torch.rand(n, generator=g, device="cuda") for _ in range(nf)]
    ws = torch.empty(sf.sfc_gather_workspace(n), dtype=torch.uint8, device="cuda")
    out = sf.sfc_gather(ctx, perm.to(torch.int32), f, ws=ws)
    for a, b in zip(out, f):
        assert torch.equal(a[:n], b[perm])
    # in place, four fields at a time
    ref = [v.clone() for v in f[:4]]
    if nf > 1:
        sf.sfc_gather(ctx, perm.to(torch.int32), f[:4], outs=f[:4], ws=ws)
        for a, b in zip(f, ref):
            assert torch.equal(a, b[perm])
