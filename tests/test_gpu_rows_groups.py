"""The 1x1 rows where their groups of 1, 4 or 8 particles can go wrong: sizes
around a group's edge, rows of many segments (longer than the words staged),
every cluster size and encoding, and a pool that ends inside a group. Headers
and words bit for bit and counts exactly as the oracle's, densities within 1e-5."""
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


def _list(env, n, seed, target, cs):
    sf, ctx, torch = env
    s = workloads.uniform_varied(n, seed, target=target)
    pipe = sf.Pipeline(ctx, n, s.box, cluster_size=cs, half=False, leaf_bucket=64)
    nl = pipe.step(*(torch.from_numpy(a).cuda() for a in (s.x, s.y, s.z, s.h)), density=False)
    return nl, pipe.sorted[:4], [t.cpu().numpy() for t in pipe.sorted[:4]]


@pytest.mark.parametrize("cs", [4, 8, 16])
@pytest.mark.parametrize("comp", [True, False])
@pytest.mark.parametrize("n,target", [(7, 5.0), (8, 5.0), (9, 5.0), (72, 30.0), (79, 30.0), (3001, 1500.0),
                                      (12001, 20.0), (127999, 8.0), (128003, 8.0)])
def test_groups(env, cs, comp, n, target):
    sf, ctx, torch = env
    print("rows groups n=%d cs=%d comp=%d" % (n, cs, comp), flush=True)
    nl, arrays, host = _list(env, n, 7 + n, target, cs)
    m = torch.from_numpy(np.random.default_rng(n).uniform(0.5, 2.0, n).astype(np.float32)).cuda()
    rl = sf.build_rows(ctx, nl, *arrays, compress=comp)
    rho, nnb = sf.rows_pass(ctx, rl, *arrays, m=m)
    info, pool = oracle.row_list(*host, comp)
    np.testing.assert_array_equal(rl.row_info.cpu().numpy().view(np.uint32), info)
    np.testing.assert_array_equal(rl.pool.cpu().numpy().view(np.uint32)[:rl.used_bytes // 4], pool)
    r, c = oracle.density(*host, m.cpu().numpy())
    np.testing.assert_array_equal(nnb.cpu().numpy(), c)
    assert (np.abs(rho.cpu().numpy().astype(np.float64) - r) / r).max() <= 1e-5


@pytest.mark.parametrize("n", [500, 12001, 128003])
def test_pool_ends_inside_a_group(env, n):
    sf, ctx, torch = env
    nl, arrays, host = _list(env, n, 3, 20.0, 8)
    info, pool = oracle.row_list(*host, True)
    cut = int(info[243, 0]) + 1  # row 243 (the fourth of its group of 4 or 8) does not fit any more
    short = torch.full((cut + 64,), -7, dtype=torch.int32, device="cuda")
    got = torch.empty((n, 2), dtype=torch.int32, device="cuda")
    with pytest.raises(sf.SfcnlError) as e:
        sf.build_rows(ctx, nl, *arrays, pool=short[:cut], row_info=got, grow=False)
    assert e.value.code == -3
    g = got.cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(g[:, 0], info[:, 0])
    np.testing.assert_array_equal(g[:243, 1], info[:243, 1])
    assert not g[243:, 1].any()
    w = short.cpu().numpy()
    np.testing.assert_array_equal(w.view(np.uint32)[:cut - 1], pool[:cut - 1])
    assert (w[cut - 1:] == -7).all()  # nothing of the rows that did not fit
