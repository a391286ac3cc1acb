"""The rows' pass over rows that did not all fit their pool: build_rows reports
the overflow and records the rows that did not fit as empty, so a pass over them
gives every particle whose row fitted its density and count and the others the
density of a particle alone. The pool is the front of a larger allocation."""
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


@pytest.mark.parametrize("comp", [True, False])
@pytest.mark.parametrize("n,row", [(500, 243), (500, 0), (12001, 11990), (12001, 700)])
def test_pass_over_rows_that_did_not_fit(env, n, row, comp):
    sf, ctx, torch = env
    print("short rows n=%d row=%d comp=%d" % (n, row, comp), flush=True)
    s = workloads.uniform_varied(n, 3, target=20.0)
    pipe = sf.Pipeline(ctx, n, s.box, half=False, leaf_bucket=64)
    nl = pipe.step(*(torch.from_numpy(a).cuda() for a in (s.x, s.y, s.z, s.h)), density=False)
    arrays, host = pipe.sorted[:4], [t.cpu().numpy() for t in pipe.sorted[:4]]
    info, pool = oracle.row_list(*host, comp)
    cut = int(info[row, 0]) + 1  # the pool ends inside this row
    room = torch.full((len(pool) + 4096,), -7, dtype=torch.int32, device="cuda")
    got = torch.empty((n, 2), dtype=torch.int32, device="cuda")
    with pytest.raises(sf.SfcnlError) as e:
        sf.build_rows(ctx, nl, *arrays, compress=comp, pool=room[:cut], row_info=got, grow=False)
    assert e.value.code == -3
    rl = sf.RowList(n, comp, got, room[:cut], 0)
    m = torch.from_numpy(np.random.default_rng(n).uniform(0.5, 2.0, n).astype(np.float32)).cuda()
    rho, nnb = sf.rows_pass(ctx, rl, *arrays, m=m)
    mh, h = m.cpu().numpy(), host[3].astype(np.float64)
    ref, cnt = oracle.density(*host, mh)
    fits = np.append(info[1:, 0], len(pool)) <= cut
    assert fits.any() != fits.all() or row == 0
    alone = mh * 8.0 / (np.pi * h ** 3)
    np.testing.assert_array_equal(nnb.cpu().numpy(), np.where(fits, cnt, 0))
    want = np.where(fits, ref, alone)
    assert (np.abs(rho.cpu().numpy().astype(np.float64) - want) / want).max() <= 1e-5
