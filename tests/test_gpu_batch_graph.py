"""Batched iterations with lists in every round (recount 1), whose rounds are
replayed four to a graph launch (one where fewer are left): with and without
graphs, and against the particles' own rounds (recount 2), the same radii,
counts, rounds and totals, also where a round limit cuts through a replay and
where counts far above the target are left short."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("max_iters", [3, 5, 6, 7, 64])
def test_replayed_rounds(env, max_iters, half):
    sf, ctx, torch = env
    print("graph rounds max_iters=%d half=%d" % (max_iters, half), flush=True)
    target = 60
    systems = [workloads.plummer(6000, 1, target=target), workloads.uniform_global(300, 2, target=target),
               workloads.uniform_varied(9001, 3, target=4.0 * target), workloads.plummer(3000, 4, target=target)]
    b = sf.Batch(ctx, [t.n for t in systems], [t.box for t in systems])
    f = [torch.from_numpy(np.concatenate([getattr(t, c) for t in systems])).cuda() for c in "xyzh"]
    keys, perm = sf.batch_sort(ctx, b, *f[:3])
    xs, ys, zs, h0 = sf.batch_gather(ctx, b, perm, f)
    out = {}
    for graph, recount in ((True, 1), (False, 1), (True, 2)):
        h = h0.clone()
        r = sf.batch_h_iterate(ctx, b, keys, xs, ys, zs, h, target=target, tol=1, max_iters=max_iters, half=half,
                               use_graph=graph, recount=recount, max_j_per_sc=2048)
        out[graph, recount] = (h.cpu().numpy(), r.nnb.cpu().numpy(), r.sys_rounds.tolist(),
                               (r.iters, r.moved, r.unconverged, r.converged))
    a = out[True, 1]
    assert a[3][3] == (max_iters == 64) and a[3][0] == (max_iters if max_iters < 64 else a[3][0])
    real = np.concatenate([np.arange(int(b.pbase[k]), int(b.pbase[k]) + t.n) for k, t in enumerate(systems)])
    for other in ((False, 1), (True, 2)):
        c = out[other]
        np.testing.assert_array_equal(a[0][real], c[0][real])
        np.testing.assert_array_equal(a[1][real], c[1][real])
        assert a[2:] == c[2:]
