"""Row kernels: automatic plans with one reduction per output over a contiguous block.
Blocks at the edges of every shape the route picks -- shorter than a vector, one to four
vectors per lane, one wave to eight, split over workgroups -- starting at any element,
against the oracle and against the plan's own kernels (integers bit for bit)."""
import numpy as np
import pytest

import paper_2309_01906_amd as hp
import workloads
from gpu_util import assert_match, gpu_reduce, say, to_device

pytestmark = pytest.mark.gpu

F32_BLOCKS = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 101, 127, 128, 129, 255, 256, 257, 509, 512, 513,
              767, 769, 1021, 1024, 1025, 1027, 4096, 4099, 16384, 16387, 65536, 65539, 70001]
BF16_BLOCKS = [1, 7, 8, 9, 15, 16, 17, 33, 65, 129, 511, 512, 513, 1024, 1025, 1537, 2047, 2048, 2049, 2063, 8200, 40001]


def data(dtype, shape, seed):
    if dtype == hp.F32:
        return workloads.normal_f32(seed, shape)
    if dtype == hp.BF16:
        return workloads.normal_bf16_bits(seed, shape)
    return workloads.uniform_i32(seed, shape, -4, 4)  # many ties


@pytest.mark.parametrize("dtype,op,blocks", [(hp.F32, "SUM", F32_BLOCKS), (hp.BF16, "SUM", BF16_BLOCKS)] +
                         [(hp.I32, op, F32_BLOCKS) for op in ("SUM", "MIN", "MAX", "ARGMIN", "ARGMAX")])
def test_blocks_of_every_shape(dtype, op, blocks):
    for b in blocks:
        for n in (1, 3, 130) if b < 20000 else (1, 5):
            say("case rows", dtype, op, n, b)
            x = data(dtype, (n, b), 200 + b % 7)
            dev = to_device(x)
            got, _ = gpu_reduce(x, x.shape, ("NONE", op), dev=dev)
            assert_match(got, x, x.shape, ("NONE", op), what=f"rows {op} {x.shape}")
            want, _ = gpu_reduce(x, x.shape, ("NONE", op), flags=hp.FLAG_NO_XCD, dev=dev)  # the plan's kernels
            if dtype == hp.I32:
                np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("n,b", [(40000, 3), (100003, 16), (70001, 33), (9001, 300), (5003, 700), (300, 1 << 16), (2, 1 << 21)])
@pytest.mark.parametrize("dtype,op", [(hp.F32, "SUM"), (hp.BF16, "SUM"), (hp.I32, "SUM"), (hp.I32, "ARGMAX")])
def test_many_outputs_and_split_blocks(dtype, op, n, b):
    """More steps than one pass of the grid takes, and blocks split over workgroups."""
    say("case rows many", dtype, op, n, b)
    x = data(dtype, (n, b), 220)
    got, _ = gpu_reduce(x, x.shape, ("NONE", op))
    assert_match(got, x, x.shape, ("NONE", op), what=f"rows {op} {x.shape}")


def test_extremes_and_non_finite_values():
    """MIN / MAX / ARG rows made only of the value an empty carrier holds, and float rows
    with infinities and NaNs (a NaN result, as the compensated oracle gives)."""
    for fill, op in [(np.iinfo(np.int32).max, "MIN"), (np.iinfo(np.int32).min, "MAX")]:
        for b in (3, 5, 67, 1001, 5000, 70001):
            x = np.full((9, b), fill, np.int32)
            for o in (op, "ARG" + op):
                got, _ = gpu_reduce(x, x.shape, ("NONE", o))
                assert_match(got, x, x.shape, ("NONE", o), what=f"extremes {o} {b}")
    for b in (3, 40, 900, 5000, 300000):
        x = np.ones((5, b), np.float32)
        x[1, b - 1], x[2, 0], x[3, b // 2] = np.inf, -np.inf, np.nan
        for flags in (0, hp.FLAG_NO_XCD):
            got, _ = gpu_reduce(x, x.shape, ("NONE", "SUM"), flags=flags)
            np.testing.assert_array_equal(got, [b, np.nan, np.nan, np.nan, b])


@pytest.mark.parametrize("dtype,op", [(hp.F32, "SUM"), (hp.BF16, "SUM"), (hp.I32, "ARGMIN")])
def test_lanes_and_waves_at_their_edges(dtype, op):
    """Blocks where the lanes per row (16, 32 and 64, one to four vectors each) and the
    waves per block change, in bytes, an element less and more, with many and few outputs."""
    es = 2 if dtype == hp.BF16 else 4
    for nbytes in [256, 512, 528, 768, 784, 1024, 1536, 1552, 3072, 4096]:
        for d in (-1, 0, 1):
            check_rows(dtype, op, 2100, nbytes // es + d)
    for nbytes in [12 << 10, 16 << 10, 24 << 10, 32 << 10, 64 << 10, 192 << 10]:
        for n, d in [(1024, 0), (1031, 1), (1023, -1), (130, 3), (3, 0)]:
            if n * nbytes < 80 << 20:
                check_rows(dtype, op, n, nbytes // es + d)


def check_rows(dtype, op, n, b):
    say("case rows", dtype, op, n, b)
    x = data(dtype, (n, b), 230 + b % 5)
    got, _ = gpu_reduce(x, x.shape, ("NONE", op))
    assert_match(got, x, x.shape, ("NONE", op), what=f"rows {op} {x.shape}")
