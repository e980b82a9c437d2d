"""Segment kernels: automatic int32 plans of two or three reducing segments.  Rows and
middle levels at the edges of every shape the route picks -- rows shorter than a vector,
one to four vectors per lane, longer rows reduced by the row kernels; several pairs side
by side in a wave, a run of pairs per wave, waves sharing a pair, parts and the tail --
against the oracle, bit for bit."""
import numpy as np
import pytest

import paper_2309_01906_amd as hp
import workloads
from gpu_util import assert_match, gpu_reduce, say, to_device

pytestmark = pytest.mark.gpu

TWO = [("SUM", "MAX"), ("ARGMAX", "SUM"), ("MIN", "SUM"), ("SUM", "ARGMIN"), ("ARGMIN", "ARGMAX"), ("MAX", "MIN")]
THREE = [("SUM", "MAX", "ARGMIN"), ("ARGMAX", "SUM", "MIN"), ("MIN", "ARGMIN", "SUM"), ("ARGMIN", "MAX", "ARGMAX")]


def check(ext, ops, lo, hi, seed):
    say("case segs", ext, ops)
    x = workloads.uniform_i32(seed, ext, lo, hi)
    got, _ = gpu_reduce(x, ext, ops)
    assert_match(got, x, ext, ops, what=f"segs {ext} {ops}")


@pytest.mark.parametrize("ops", TWO)
@pytest.mark.parametrize("rows", [1, 2, 3, 4, 5, 7, 16, 33, 63, 64, 65, 255, 256, 257, 500, 513, 769, 1023, 1024, 1025, 4100])
def test_two_segments(ops, rows):
    for m, n in [(1, 5), (2, 70), (3, 300), (17, 33), (64, 9), (65, 3), (1000, 1)]:
        check((n, m, rows), ("NONE",) + ops, -(1 << 31), (1 << 31) - 1, 300 + rows)  # sums beyond 32 bits
        check((n, m, rows), ("NONE",) + ops, -2, 2, 301 + rows)                       # ties


@pytest.mark.parametrize("ops", THREE)
@pytest.mark.parametrize("rows", [1, 3, 4, 9, 64, 100, 1000, 1030])
def test_three_segments(ops, rows):
    for q, m, n in [(2, 2, 40), (3, 7, 5000), (70, 3, 2), (9, 33, 11), (1500, 2, 1), (5, 300, 3)]:
        if n * q * m * rows < 1 << 23:
            check((n, q, m, rows), ("NONE",) + ops, -3, 3, 310 + rows)


@pytest.mark.parametrize("ext,ops", [
    ((1, 2, 1 << 21), ("SUM", "MAX")), ((1, 3, 700001), ("ARGMAX", "SUM")),     # rows split over workgroups
    ((1, 200001, 2), ("MAX", "SUM")), ((2, 50001, 33), ("ARGMIN", "MAX")),      # M split into parts
    ((9000, 3, 5), ("SUM", "MIN")), ((20011, 9, 40), ("ARGMAX", "SUM")),        # runs of pairs
    ((6000, 4, 5, 6), ("SUM", "MAX", "SUM")), ((40, 900, 65, 7), ("MIN", "SUM", "ARGMAX"))])
def test_many_pairs_and_parts(ext, ops):
    check(ext, ("NONE",) + ops, -1000, 1000, 320)


def test_levels_that_merge_and_single_iterations():
    """Adjacent levels of one operator are one segment, levels of one iteration pass
    their value on, and an ARG level of one iteration gives 0."""
    for ext, ops in [((7, 3, 1, 5, 6), ("NONE", "SUM", "MIN", "MAX", "MAX")), ((64, 1, 2, 100), ("NONE", "ARGMAX", "ARGMIN", "MIN")),
                     ((5, 4, 3, 2, 30), ("NONE", "SUM", "SUM", "MAX", "MAX")), ((8, 9, 1, 40), ("NONE", "MAX", "ARGMIN", "SUM")),
                     ((6, 50, 1), ("NONE", "MIN", "ARGMAX")), ((4, 6, 5, 1), ("NONE", "ARGMAX", "MIN", "SUM"))]:
        check(ext, ops, -50, 50, 330)


@pytest.mark.parametrize("fill,mm", [(np.iinfo(np.int32).max, "MIN"), (np.iinfo(np.int32).min, "MAX")])
def test_extreme_rows(fill, mm):
    for ext in [(5, 7, 3), (5, 40, 67), (2, 9, 2000)]:
        x = np.full(ext, fill, np.int32)
        for ops in [("NONE", "ARG" + mm, mm), ("NONE", mm, "ARG" + mm), ("NONE", "SUM", "ARG" + mm), ("NONE", mm, "SUM")]:
            got, _ = gpu_reduce(x, ext, ops)
            assert_match(got, x, ext, ops, what=f"extremes {ext} {ops}")


def test_static_entry_and_graph_replay():
    """The allocation-free entry point gives the same bits, and a captured run replays on
    new values."""
    import torch
    for ext, ops in [((9, 40, 33, 21), ("NONE", "SUM", "MAX", "ARGMIN")), ((3, 5, 5000), ("NONE", "ARGMAX", "SUM"))]:
        x = to_device(workloads.uniform_i32(340, ext, -1000, 1000))
        with hp.Plan(ext, ops, hp.I32) as p:
            a, b = p.empty_out("cuda"), p.empty_out("cuda")
            p.run(x, a)
            hp.reduce_static(x, b, ext, ops)
            assert torch.equal(a, b)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                p.run(x, b)
            for k in range(3):
                x.add_(k + 1)
                x[0] *= -1
                g.replay()
                p.run(x, a)
                torch.cuda.synchronize()
                assert torch.equal(a, b)


@pytest.mark.parametrize("ops", [("MAX", "ARGMIN"), ("ARGMIN", "SUM"), ("SUM", "MAX", "SUM"), ("ARGMAX", "SUM", "MIN")])
def test_waves_per_pair_and_runs_at_their_edges(ops):
    """Pairs around the sizes where a wave's run, four or eight waves of a pair and parts
    take over, with steps that do not fill the last round."""
    q = (3,) if len(ops) == 3 else ()
    for ext in [(700, 48, 64), (700, 47, 65), (700, 49, 63), (200, 127, 64), (200, 129, 64), (90, 260, 128), (2, 3000, 67),
                (5000, 5, 17), (9001, 9, 13), (20011, 2, 5), (12289, 1, 9), (4097, 4, 1024), (4099, 4, 1021), (30, 70, 300),
                (8200, 33, 2), (600, 500, 3), (5, 20000, 1), (40, 3, 3)]:
        check(ext[:1] + q + ext[1:], ("NONE",) + ops, -4, 4, 350)


def test_arg_of_extreme_sums():
    """Keys of an ARG level over int64 sums at the ends of their range, with ties."""
    lo, hi = np.iinfo(np.int32).min, np.iinfo(np.int32).max
    for ext in [(4, 7, 3), (4, 5, 1000), (3, 3000, 64), (2, 1, 33), (2, 64, 1), (2, 65, 4)]:
        for fill, other in [(lo, hi), (hi, lo), (lo, lo), (hi, hi)]:
            x = np.full(ext, fill, np.int32)
            x[1:, ext[1] // 2, ext[2] // 2:] = other
            for op in ["ARGMIN", "ARGMAX"]:
                got, _ = gpu_reduce(x, ext, ("NONE", op, "SUM"))
                assert_match(got, x, ext, ("NONE", op, "SUM"), what=f"sums {ext} {op}")


@pytest.mark.parametrize("fill,mm", [(np.iinfo(np.int32).max, "MIN"), (np.iinfo(np.int32).min, "MAX")])
def test_extreme_rows_beside_waves_without_steps(fill, mm):
    """A part with fewer steps than its workgroup has waves leaves waves without a row: their
    empty carrier ties with rows that hold the extreme value, and must not win."""
    for ext in [(1, 16388, 64), (1, 177, 1000), (3, 177, 1000), (1, 3355, 64), (1, 4001, 1000), (2, 10, 1000), (1, 2, 3355, 64),
                (2, 3, 177, 1000), (3, 2, 40001, 3)]:
        x = np.full(ext, fill, np.int32)
        for arg in ["ARG" + mm, mm]:
            for child in ["MIN", "MAX", "ARGMIN"]:
                for outer in [("SUM",), ("ARGMIN",), ("MIN",)] if len(ext) == 4 else [()]:
                    ops = ("NONE",) + outer + (arg, child)
                    got, _ = gpu_reduce(x, ext, ops)
                    assert_match(got, x, ext, ops, what=f"extremes {ext} {ops}")


@pytest.mark.parametrize("ext,ops", [
    ((1, 40000, 3, 5), ("ARGMIN", "MAX", "SUM")), ((3, 20011, 2, 8), ("SUM", "ARGMAX", "MIN")),      # a lane per iteration of Q
    ((1, 100, 5000, 64), ("ARGMAX", "MIN", "SUM")), ((2, 512, 10, 1257), ("ARGMIN", "MAX", "ARGMIN")),  # a wave per iteration
    ((1, 5000, 2, 1030), ("MAX", "ARGMIN", "SUM")), ((1, 20000, 1030), ("ARGMAX", "MIN")), ((2, 17001, 1030), ("MIN", "SUM")),
    ((70, 9001, 1, 7), ("ARGMAX", "ARGMIN", "MAX"))])
def test_tail_in_parts(ext, ops):
    """Outermost levels that several workgroups of the tail share: ties across the parts,
    and the extreme value everywhere."""
    check(ext, ("NONE",) + ops, -2, 2, 360)
    check(ext, ("NONE",) + ops, -(1 << 31), (1 << 31) - 1, 361)
    fill = np.iinfo(np.int32).max if "MIN" in ops[0] else np.iinfo(np.int32).min
    x = np.full(ext, fill, np.int32)
    got, _ = gpu_reduce(x, ext, ("NONE",) + ops)
    assert_match(got, x, ext, ("NONE",) + ops, what=f"extremes {ext} {ops}")


@pytest.mark.parametrize("ops", THREE)
def test_short_even_chains(ops):
    """Even nests on both sides of the line between the chain kernel and the segment kernels."""
    for ext in [(512, 8, 4, 8), (16, 4, 16, 4), (265, 128, 2, 16), (6516, 32, 4, 4), (3183, 64, 2, 4), (1, 32, 2, 16),
                (102, 4, 2, 256), (512, 512, 8, 4), (9000, 2, 8, 8), (1030, 8, 4, 64)]:
        check(ext, ("NONE",) + ops, -3, 3, 370)


@pytest.mark.parametrize("ext", [(4096, 21, 1, 4), (4096, 8, 2, 5), (4097, 9, 3, 5), (11300, 8, 2, 3), (12600, 9, 1, 7), (12599, 9, 1, 7)])
def test_tails_of_many_outputs(ext):
    """Tails by a lane and by a workgroup per output, on both sides of the line."""
    for ops in THREE:
        check(ext, ("NONE",) + ops, -2, 2, 380)
