"""Which kernels automatic plans and batched nests take, and with what partition: the
planner's route functions, compiled for the host."""
import math
import os
import subprocess

import pytest

import paper_2309_01906_amd as hp

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2309_01906_amd", "csrc")


@pytest.fixture(scope="session")
def probe(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "route_probe")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(HERE, "route_probe.cpp"), os.path.join(CSRC, "hp_plan.cpp"),
                    os.path.join(CSRC, "hp_units.cpp"), "-o", exe], check=True)

    def routes(nests, dtype=hp.I32):
        text = nests if isinstance(nests, str) else "".join(f"{len(e)} " + " ".join(f"{x}:{hp._op(o)}" for x, o in zip(e, ("NONE",) + ops)) + f" {dtype}\n"
                       for e, ops in nests)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == (nests.count("\n") if text is nests else len(nests))
        return [dict(zip(w[::2], map(int, w[1::2]))) for w in map(str.split, out)]
    return routes


LONG_TAILS = [((1, 131072, 8, 64), ("SUM", "MAX", "ARGMIN")), ((1, 1048576, 4, 8), ("SUM", "MAX", "SUM")),
              ((16, 131072, 4, 8), ("SUM", "MAX", "SUM")), ((2, 100000, 16, 20), ("MAX", "SUM", "ARGMIN")),
              ((1, 1000, 10, 1100), ("MAX", "SUM", "MIN")), ((2, 512, 10, 1257), ("MIN", "MAX", "ARGMIN")),
              ((1, 1000000, 1100), ("MAX", "SUM")), ((3, 40000, 2, 8), ("SUM", "MIN", "MAX")),
              ((1, 100, 5000, 64), ("ARGMAX", "MIN", "SUM"))]


def test_no_workgroup_ends_a_long_outermost_level_alone(probe):
    """Few outputs with a long outermost level: the tail's work is shared, so that no
    workgroup of it goes through more than a few rounds of memory latency."""
    for (ext, ops), r in zip(LONG_TAILS, probe(LONG_TAILS)):
        assert r["seg_kind"], ext
        q, n = (ext[1], ext[2] if r["seg_kind"] == 2 else r["seg_parts"]) if len(ops) == 3 else (0, ext[1])
        per = r["tail_per"] if r["tail_parts"] > 1 else (q or n)
        rounds = math.ceil(per / 4096) if not q else math.ceil(per / 1024) * n if n <= 8 else math.ceil(per / 16) * math.ceil(n / 256)
        assert rounds <= 16, (ext, r)
        if r["tail_parts"] > 1:
            assert (r["tail_parts"] - 1) * per < (q or n) <= r["tail_parts"] * per, (ext, r)
            assert r["tail_off"] + ext[0] * r["tail_parts"] * 16 == r["seg_ws"]
            carriers = ext[0] * q * n * 16 if r["seg_kind"] == 1 else math.prod(ext[:-1]) * 8
            assert r["tail_off"] >= carriers and r["tail_off"] % 256 == 0


def test_short_even_chains_stay_with_the_chain_kernel(probe):
    """Even nests of three segments whose pairs are short and whose outputs a workgroup ends
    in a strip or two take one launch; longer pairs, uneven levels and split outputs take the
    segment kernels."""
    chain = [(512, 8, 4, 8), (16, 4, 16, 4), (265, 128, 2, 16), (997, 16, 4, 16), (2251, 16, 4, 16), (1, 32, 2, 16),
             (6516, 32, 4, 4), (199, 128, 4, 16), (3183, 64, 2, 4)]
    segs = [(64, 128, 64, 64), (61, 125, 67, 59), (128, 2, 220, 256), (512, 512, 8, 4), (102, 4, 2, 256), (32, 48, 16, 16),
            (16, 4, 15, 4), (1, 131072, 8, 64), (3, 5, 6, 16)]
    ops = ("MIN", "ARGMAX", "MAX")
    for ext, r in zip(chain + segs, probe([(e, ops) for e in chain + segs])):
        assert (r["seg_kind"] == 0) == (ext in chain), (ext, r)
        assert r["kernel"] == 7 or ext in segs, ext


def test_ordered_blocks_leave_the_workgroup_in_time():
    """A workgroup multiplies a block alone only while that is short: beyond, and with many
    blocks, chunks or waves of their own."""
    for dt, ext, joined in [(hp.AFFINE64, (16, 6144), True), (hp.AFFINE64, (17, 6144), False), (hp.AFFINE64, (17, 5120), True),
                            (hp.AFFINE64, (62, 8052), False), (hp.AFFINE64, (129, 4096), False), (hp.MAT2X2_64, (64, 3072), True),
                            (hp.MAT2X2_64, (65, 3072), False), (hp.MAT2X2_64, (6, 5742), False), (hp.MAT2X2_64, (107, 7465), False),
                            (hp.MAT2X2_64, (128, 2048), True)]:
        i = hp.inspect(ext, ("NONE", "PROD"), dt)
        assert (i["waves"] == 16) == joined and (i["gsplit"] == 1) == joined, (ext, i)
    assert hp.inspect((2018, 2048), ("NONE", "PROD"), hp.AFFINE64)["gsplit"] == 1
    assert hp.inspect((1000, 2048), ("NONE", "PROD"), hp.AFFINE64)["gsplit"] == 4
    assert hp.inspect((5941, 99), ("NONE", "PROD"), hp.MAT2X2_64)["kernel_name"] == "hp::k_ordered<4, 256, false>"


def test_tall_stencils_of_one_or_two_strips_keep_their_tiles(probe):
    """Two to four sweeps over a tall array of one or two strips of 248 columns, all of which
    hold an edge, run in LDS tiles; shorter and wider arrays in registers."""
    tiles = [(2516, 484, 2), (5091, 432, 2), (1024, 482, 2), (6675, 230, 2), (4096, 380, 3), (1315, 243, 3), (2048, 256, 4),
             (8192, 8192, 1)]
    regs = [(600, 484, 2), (1000, 230, 2), (2516, 700, 2), (1500, 380, 3), (1000, 243, 3), (2964, 286, 3), (1024, 500, 4), (4096, 398, 4), (8192, 8192, 4),
            (1500, 1500, 8), (8192, 8192, 8)]
    got = probe("".join(f"0 {r} {c} {t}\n" for r, c, t in tiles + regs))
    assert [g["reg"] for g in got] == [0] * len(tiles) + [1] * len(regs)


def test_no_fold_of_a_batched_nest_is_long(probe):
    """What unit tasks leave of an output takes its fold a few dozen rounds of memory latency
    at most; where it would take more the nest runs as its plan's tasks."""
    nests = LONG_TAILS + [((4, 64, 16, 1024), ("SUM", "ARGMIN", "ARGMAX")), ((1, 345, 131072), ("MIN", "ARGMIN")),
                          ((1, 89012, 480), ("ARGMAX", "ARGMIN")), ((16, 65536, 2, 128), ("ARGMAX", "ARGMIN", "ARGMAX")),
                          ((1, 1 << 28), ("SUM",)), ((3, 5, 20, 70), ("SUM", "MAX", "SUM"))]
    on = 0
    for (ext, ops), r in zip(nests, probe(nests)):
        if not r["unit_on"] or not r["folds"]:
            continue
        on += 1
        waves, q = r["fold_waves"], ext[1] if len(ops) == 3 else 1
        assert waves in (1, 16) and r["folds"] == ext[0]
        cut = r["lparts"] > 1
        rows, parts = (ext[-2] if cut and len(ops) > 1 else 1), (r["lparts"] if cut else r["mparts"])
        up, some, lanes = lambda a, b: -(-a // b), -(-parts // 4), 64 * waves
        if len(ops) == 3:
            rounds = [up(q, lanes) * rows * some, up(q, waves) * up(rows, 64) * some, up(q, waves) * rows * up(parts, 256)]
        else:
            rounds = [1 << 60, up(rows, lanes) * some, up(rows, waves) * up(parts, 256) if rows > 1 else up(parts, 4 * lanes)]
        assert rounds[r["fold_form"]] == min(rounds) <= (1 if ext[-1] % 4 == 0 else 4) * (40 if waves > 1 else 4 if ext[0] <= 256 else 32), (ext, r)
    assert 5 <= on < len(nests)


def test_a_launch_of_tasks_stays_below_the_grid_limit(probe):
    """Lists of tasks go out in launches of fewer than 2^32 threads, whole workgroups each."""
    r = probe([((2, 3), ("SUM",))])[0]
    assert r["launch_wave"] * 64 < 1 << 32 and r["launch_wave"] % 4 == 0
    assert r["launch_group"] * 1024 < 1 << 32


def test_batched_nests_keep_little_memory(probe):
    """Unit tasks keep at most a sixteenth of a nest's input on the device beside it, or 64
    MiB, or what the plan's tasks would keep."""
    nests = [((1048576, 64, 4, 2), ("SUM", "MAX", "SUM")), ((67108864, 2, 2, 4), ("SUM", "MAX", "SUM")),
             ((1048576, 64, 8, 32), ("MIN", "SUM", "ARGMAX")), ((1000000, 3, 40, 7), ("SUM", "MAX", "SUM")),
             ((4096, 256, 16, 16), ("SUM", "MAX", "SUM")), ((1 << 22, 4, 2, 8), ("SUM", "MAX", "SUM"))]
    on = []
    for (ext, ops), r in zip(nests, probe(nests)):
        kept = r["unit_ws"] + 8 * r["folds"]
        assert not r["unit_on"] or kept <= max(64 << 20, math.prod(ext) * 4 // 16, r["plan_ws"]), (ext, r)
        on.append(r["unit_on"])
    assert on == [0, 0, 1, 1, 1, 0]  # the third keeps 1 GiB beside 64


def test_chains_beyond_the_last_level_cache_stay_with_the_chain_kernel(probe):
    """Even nests of 256 MiB and more in a few pairs, or of 128 MiB and more in short pairs of
    whole lines; smaller ones, other rows and many pairs take the segment kernels.  Pairs of
    64 KiB that fill a quarter of the chip are not cut in two."""
    two, three = ("MIN", "SUM"), ("MIN", "ARGMAX", "MAX")
    cases = [((4, 65536, 256), two, 0), ((512, 1024, 128), two, 0), ((4, 32768, 256), two, 1), ((4, 65536, 255), two, 1),
             ((1 << 16, 8, 128), two, 1), ((4096, 256, 2, 64), three, 0), ((8, 32768, 4, 64), three, 0),
             ((64, 8192, 4, 32), three, 1), ((64, 1024, 4, 64), three, 1)]
    for (ext, ops, kind), r in zip(cases, probe([c[:2] for c in cases])):
        assert r["seg_kind"] == kind, (ext, r)
    for r in probe([((512, 128, 128), two), ((300, 100, 163), two)]):
        assert r["seg_parts"] == 1 and r["seg_tail"] == 0
