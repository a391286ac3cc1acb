"""Where the automatic recount of an h-iteration leaves the rounds of lists for
the particles' own rounds: right after the first round for small systems whose
target's pairs a wavefront can keep, later for larger targets. Read from the
number of list builds; radii, counts and rounds as with lists in every round."""
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


@pytest.mark.parametrize("n,target,own", [(20000, 100, True), (20000, 450, True), (40000, 400, True),
                                          (40000, 410, False), (70000, 600, False), (262145, 20, False)])
def test_builds(env, n, target, own):
    sf, ctx, torch = env
    print("finish limit n=%d T=%d" % (n, target), flush=True)
    s = workloads.uniform_global(n, 5, target=0.3 * target)  # (every particle moves in the first round)
    f = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (s.x, s.y, s.z, s.h)]
    keys, perm = sf.sfc_sort(ctx, *f[:3], s.box)
    xs, ys, zs, h0 = sf.sfc_gather(ctx, perm, f)
    out = {}
    for recount in (0, 1):
        h = h0.clone()
        kw = dict(target=target, tol=2, recount=recount, max_j_per_sc=2048,
                  pool=torch.empty(24 * n, dtype=torch.int32, device="cuda"))
        ctx.profile_begin(256)
        r = sf.h_iterate(ctx, keys, xs, ys, zs, h, **kw)
        builds = ctx.profile_end()["traverse"][1]
        assert r.converged
        out[recount] = (h.cpu().numpy(), r.nnb.cpu().numpy()[:n], r.iters, r.moved)
        if recount == 0:  # the first round's lists and the closing ones, or more
            assert builds == 2 if own else builds > 2
    for k in range(2):
        np.testing.assert_array_equal(out[0][k], out[1][k])
    assert out[0][2:] == out[1][2:]
