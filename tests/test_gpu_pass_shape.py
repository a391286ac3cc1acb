"""The launch shape of the density passes: with sfcnl_set_pass_waves at 2 or 4 a
workgroup has that many super-clusters at every size, with 1 several wavefronts
share a small system's super-clusters. Read from the kernel node of a captured
pass; the results are those of the oracle for every shape."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2602_19873_amd import workloads

pytestmark = pytest.mark.gpu


class Dim3(C.Structure):
    _fields_ = [("x", C.c_uint), ("y", C.c_uint), ("z", C.c_uint)]


class KernelParams(C.Structure):  # hipKernelNodeParams
    _fields_ = [("block", Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", Dim3), ("args", C.c_void_p),
                ("shared", C.c_uint)]


def _hip():
    """The HIP runtime that the process has loaded."""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return C.CDLL(path)


def _shape(hip, stream, call):
    """(blocks, threads a block) of the one kernel that `call` launches."""
    s, g = C.c_void_p(stream.cuda_stream), C.c_void_p()
    assert hip.hipStreamBeginCapture(s, 1) == 0  # thread-local
    call()
    assert hip.hipStreamEndCapture(s, C.byref(g)) == 0
    try:
        k = C.c_size_t()
        assert hip.hipGraphGetNodes(g, None, C.byref(k)) == 0 and k.value == 1
        node, p = (C.c_void_p * 1)(), KernelParams()
        assert hip.hipGraphGetNodes(g, node, C.byref(k)) == 0
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node[0]), C.byref(p)) == 0
        return p.grid.x, p.block.x
    finally:
        hip.hipGraphDestroy(g)


@pytest.mark.parametrize("cs,n", [(8, 1000), (8, 20011), (8, 70001), (4, 20011), (16, 3000)])
def test_shape(cs, n):
    import torch
    import paper_2602_19873_amd as sf
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    torch.cuda.set_device(0)
    print("pass shape cs=%d n=%d" % (cs, n), flush=True)
    hip, stream = _hip(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = sf.Context(0)
        s = workloads.uniform_varied(n, n, target=20.0)
        pipe = sf.Pipeline(ctx, n, s.box, cluster_size=cs, half=False)
        nl = pipe.step(*(torch.from_numpy(a).cuda() for a in (s.x, s.y, s.z, s.h)))
        ref, cnt = oracle.density(*(t.cpu().numpy() for t in pipe.sorted[:4]))
        nsc = (n + 63) // 64
        for waves in (1, 2, 4):
            ctx.set_pass_waves(waves)
            run = lambda: sf.nlist_pass(ctx, nl, *pipe.sorted[:4], rho=pipe.rho, nnb=pipe.nnb)  # noqa: E731
            blocks, threads = _shape(hip, stream, run)
            if waves == 1:
                assert blocks == nsc and threads in (64, 256, 512)
            else:
                assert (blocks, threads) == ((nsc + waves - 1) // waves, 64 * waves)
            run()
            stream.synchronize()
            np.testing.assert_array_equal(pipe.nnb.cpu().numpy()[:n], cnt)
            assert (np.abs(pipe.rho.cpu().numpy()[:n].astype(np.float64) - ref) / ref).max() <= 1e-5
        ctx.close()
