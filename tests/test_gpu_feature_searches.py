"""The seed's cell occupancies where a cell's run of keys ends in the staged
window on neither, one or both sides: condensed systems, a dense corner and
particles at one position, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2602_19873_amd import hseed, workloads

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


def _system(kind, n):
    if kind == "plummer":
        return workloads.plummer(n, 3, target=60.0)
    s = workloads.uniform_varied(n, 5, target=60.0)
    for a in (s.x, s.y, s.z):
        if kind == "corner":
            a[: n // 2] *= np.float32(0.02)
        if kind == "point":
            a[:] = np.float32(0.25)
    return s


def _check(feat, keys, x, y, z, h, edge):
    lev = np.clip(np.rint(np.log2(np.float32(edge) / h)), 2, 20).astype(np.int64)
    ref = oracle.hseed_features(keys, h, None, oracle.cluster_bboxes(x, y, z, h, 8), edge, 60, level=lev)
    # bf16 of a float32 logarithm: half an ulp (2^-9) and its rounding; radii whose level is a tie may take the other
    bad = np.abs(feat - ref)[:, 3:6] > 2.0 ** -8 * (np.abs(ref[:, 3:6]) + 2.0 ** -8)
    assert bad.any(1).mean() <= 1e-3


@pytest.mark.parametrize("kind,n", [("plummer", 2000), ("plummer", 30011), ("plummer", 300007), ("corner", 30011),
                                    ("corner", 5003), ("point", 3001), ("point", 900)])
def test_occupancies(env, kind, n):
    sf, ctx, torch = env
    print("features %s n=%d" % (kind, n), flush=True)
    s = _system(kind, n)
    f = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (s.x, s.y, s.z, s.h)]
    keys, perm = sf.sfc_sort(ctx, *f[:3], s.box)
    a = sf.sfc_gather(ctx, perm, f)
    edge = hseed.box_edge(s.box)
    feat = sf.hseed_features(ctx, keys, *a, None, edge, 60).view(torch.bfloat16).double().cpu().numpy()[:n]
    _check(feat, keys.cpu().numpy().view(np.uint64), *(t.cpu().numpy() for t in a), edge)
