"""Ordered products at the edges of every form they run in -- outputs side by side in a
wave, a wave per output in groups of 8 or 32 rows, a workgroup per output, chunks whose
products are multiplied by a second kernel -- against the oracle, bit for bit."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2309_01906_amd as hp
import workloads
from gpu_util import say

pytestmark = pytest.mark.gpu

KINDS = {"affine": (hp.AFFINE64, workloads.AFFINE, 2), "mat2": (hp.MAT2X2_64, workloads.MAT2, 4)}
BLOCKS = [1, 2, 3, 5, 16, 31, 32, 33, 63, 64, 65, 127, 129, 511, 512, 513, 1025, 2047, 2048, 2049, 4097, 8191, 8192,
          8193, 20011]


def device(x, shift=0):
    """The input on the device, `shift` bytes into an allocation."""
    import torch
    buf = torch.empty(x.size + 8, dtype=torch.int64, device="cuda")
    d = buf[shift // 8:shift // 8 + x.size]
    d.copy_(torch.from_numpy(np.ascontiguousarray(x).view(np.int64).reshape(-1)))
    return d


def check(kind, ext, seed, shift=0):
    import torch
    dt, ok, w = KINDS[kind]
    x = workloads.monoid_input(seed, ext, ok)
    ref = oracle.prod(x, ext, (oracle.NONE, oracle.PROD), ok, threads=8)
    d = device(x, shift).view(*ext, w)
    with hp.Plan(ext, ("NONE", "PROD"), dt) as p:
        out = p.run(d)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint64).reshape(ref.shape), ref, err_msg=f"{kind} {ext}")
        stat = torch.zeros_like(out)
        nest = hp.make_nest(ext, ("NONE", "PROD"), dt)
        hp.check(hp.lib().hp_reduce_static(ctypes.byref(nest), None, 0, d.data_ptr(), stat.data_ptr(),
                                           torch.cuda.current_stream().cuda_stream))
        assert torch.equal(out, stat), (kind, ext)


@pytest.mark.parametrize("kind", ["affine", "mat2"])
@pytest.mark.parametrize("n", [1, 3, 67, 4100])
def test_blocks_of_every_form(kind, n):
    for k, block in enumerate(BLOCKS):
        if n * block < 1 << 21:
            say("case ordered rows", kind, n, block)
            check(kind, (n, block), 400 + k, shift=16 * (k % 4))


@pytest.mark.parametrize("kind", ["affine", "mat2"])
@pytest.mark.parametrize("ext", [(1, 1 << 20), (1, 2097153), (2, 700001), (9, 100003), (1000, 1500), (2000, 700),
                                 (70000, 5), (4096, 300)])
def test_chunks_and_many_outputs(kind, ext):
    say("case ordered rows", kind, ext)
    check(kind, ext, 450, shift=48)


@pytest.mark.parametrize("kind,ext", [
    ("affine", (16, 6144)), ("affine", (16, 6145)), ("affine", (17, 5120)), ("affine", (17, 5121)), ("affine", (1024, 2048)),
    ("affine", (1023, 2048)), ("affine", (1024, 2049)), ("mat2", (64, 3072)), ("mat2", (64, 3073)), ("mat2", (65, 2048)),
    ("mat2", (65, 2049)), ("mat2", (300, 256)), ("mat2", (300, 257)), ("mat2", (1537, 513)), ("mat2", (1537, 768)),
    ("mat2", (1537, 769)), ("mat2", (1536, 600))])
def test_edges_of_the_forms(kind, ext):
    say("case ordered edges", kind, ext)
    check(kind, ext, 455, shift=32)


def test_graph_replays():
    import torch
    for kind, ext in [("affine", (30, 40001)), ("mat2", (3, 5000)), ("affine", (500, 50))]:
        dt, ok, w = KINDS[kind]
        d = device(workloads.monoid_input(460, ext, ok)).view(*ext, w)
        with hp.Plan(ext, ("NONE", "PROD"), dt) as p:
            a, b = p.empty_out("cuda"), p.empty_out("cuda")
            p.run(d, a)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                p.run(d, b)
            for k in range(3):
                d.mul_(3 + 2 * k)
                g.replay()
                p.run(d, a)
                torch.cuda.synchronize()
                assert torch.equal(a, b)
