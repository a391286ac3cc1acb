"""Passes whose super-clusters are shared by 8, 4, 2 or 1 wavefronts, at the
sizes where the number of parts changes: counts exactly and densities within
1e-5 of the oracle's, forces within 1e-5 of the summed pair magnitudes, and a
full list's sums the same bits alone and inside a batch with other parts."""
import numpy as np
import pytest

import oracle
from paper_2602_19873_amd import workloads

pytestmark = pytest.mark.gpu

# (cluster size, half, last size of a rule: super-clusters of 64)
EDGES = [(8, False, 512), (8, False, 1600), (4, False, 1600), (16, False, 1600), (8, True, 800), (8, True, 4096),
         (8, True, 16384), (4, True, 1600), (16, True, 1600), (4, True, 16384)]


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


@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("cs,half,nsc", EDGES)
def test_density_at_edges(env, cs, half, nsc, more):
    sf, ctx, torch = env
    n = 64 * nsc + more
    print("pass split n=%d cs=%d half=%d" % (n, cs, half), flush=True)
    s = workloads.uniform_varied(n, 11 + nsc, target=60.0 if n < 300000 else 8.0)
    m = np.random.default_rng(n).uniform(0.5, 2.0, n).astype(np.float32)
    pipe = sf.Pipeline(ctx, n, s.box, cluster_size=cs, half=half, with_mass=True)
    pipe.step(*(torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (s.x, s.y, s.z, s.h, m)))
    ref, cnt = oracle.density(*(v.cpu().numpy() for v in pipe.sorted))
    np.testing.assert_array_equal(pipe.nnb.cpu().numpy()[:n], cnt)
    assert (np.abs(pipe.rho.cpu().numpy()[:n].astype(np.float64) - ref) / ref).max() <= 1e-5


def _wrapped(x, y, z, q, eps, sigma, coulomb, r_cut, rows):
    """Forces in a periodic unit box from the pair formula's float32 minimum-image components (their rounding next to
    the box's faces is the formula's, not the sum's), all else in float64."""
    out = {k: np.zeros((len(rows), 3) if k == "f" else len(rows)) for k in ("f", "e", "scale", "escale")}
    rc2 = np.float32(r_cut) * np.float32(r_cut)
    for k, i in enumerate(rows):
        d = [v - v[i] for v in (x, y, z)]
        d = [v - np.rint(v) for v in d]
        d2 = sum(v.astype(np.float64) ** 2 for v in d)
        j = np.nonzero((d2 < float(rc2)) & (np.arange(len(x)) != i))[0]
        dx, r2 = np.stack([v[j].astype(np.float64) for v in d], 1), d2[j]
        s6 = (sigma * sigma / r2) ** 3
        kqq = coulomb * float(q[i]) * q[j].astype(np.float64)
        fr = 24 * eps / r2 * s6 * (2 * s6 - 1) + kqq / r2 ** 1.5
        u = 4 * eps * s6 * (s6 - 1) + kqq / np.sqrt(r2)
        out["f"][k] = -(fr[:, None] * dx).sum(0)
        out["scale"][k] = (np.abs(fr) * np.sqrt(r2)).sum()
        out["e"][k], out["escale"][k] = 0.5 * u.sum(), 0.5 * np.abs(u).sum()
    return out


@pytest.mark.parametrize("period", [False, True])
@pytest.mark.parametrize("cs,half,nsc", [e for e in EDGES if e[2] <= 1600])
def test_forces_at_edges(env, cs, half, nsc, period):
    sf, ctx, torch = env
    side = int(np.ceil((64 * nsc + 1) ** (1.0 / 3.0)))
    s = workloads.lj_lattice(side, 5)
    mt = s.meta
    per = (1.0, 1.0, 1.0) if period else None
    for n in (64 * nsc, 64 * nsc + 1):
        print("pass split lj n=%d cs=%d half=%d period=%s" % (n, cs, half, per), flush=True)
        rng = np.random.default_rng(n)
        keep = np.sort(rng.choice(s.n, n, replace=False))
        x, y, z, h, q = (np.ascontiguousarray(v[keep]) for v in (s.x, s.y, s.z, s.h, s.q))
        pipe = sf.Pipeline(ctx, n, s.box, cluster_size=cs, half=half, with_mass=True, period=per)
        nl = pipe.step(*(torch.from_numpy(v).cuda() for v in (x, y, z, h, q)), density=False)
        xs, ys, zs, _, qs = pipe.sorted
        f, e = sf.nlist_pass_lj(ctx, nl, xs, ys, zs, qs, mt["eps"], mt["sigma"], mt["coulomb"], mt["r_cut"],
                                energy=True)
        rows = rng.choice(n, 1000, replace=False)
        host = [v.cpu().numpy() for v in (xs, ys, zs, qs)]
        par = (mt["eps"], mt["sigma"], mt["coulomb"], mt["r_cut"])
        ref = _wrapped(*host, *par, rows) if period else oracle.lj(*host, *par, idx=rows)
        g = f.cpu().numpy().T.astype(np.float64)[rows]
        assert (np.abs(g - ref["f"]).max(axis=1) / np.maximum(ref["scale"], 1e-300)).max() <= 1e-5
        ge = e.cpu().numpy().astype(np.float64)[rows]
        assert (np.abs(ge - ref["e"]) / np.maximum(ref["escale"], 1e-300)).max() <= 1e-5


def test_full_sums_do_not_depend_on_the_split(env):
    # 30000 particles alone (8 parts), and the first of batches with 4 parts and with one
    sf, ctx, torch = env
    sys_ = [workloads.uniform_varied(30000, 3 + k, target=60.0) for k in range(4)]
    pipe = sf.Pipeline(ctx, 30000, sys_[0].box, half=False)
    pipe.step(*(torch.from_numpy(getattr(sys_[0], c)).cuda() for c in "xyzh"))
    alone = pipe.rho.cpu().numpy()[:30000]
    for k in (3, 4):
        print("pass split batch of %d" % k, flush=True)
        b = sf.Batch(ctx, [30000] * k, [t.box for t in sys_[:k]])
        f = [torch.from_numpy(np.concatenate([getattr(t, c) for t in sys_[:k]])).cuda() for c in "xyzh"]
        keys, perm = sf.batch_sort(ctx, b, *f[:3])
        srt = sf.batch_gather(ctx, b, perm, f)
        bbox = sf.batch_build_clusters(ctx, b, *srt)
        nl = sf.batch_build_nlist(ctx, b, keys, *srt, bbox)
        rho, _ = sf.batch_pass(ctx, b, nl, *srt)
        np.testing.assert_array_equal(rho.cpu().numpy()[:30000], alone)
