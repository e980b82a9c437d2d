"""Unit tasks of batches.  Nests at the edges of what the partition picks -- rows below a
vector, up to eight vectors per lane, parts of a row, parts of the middle level, pairs side
by side and runs of them, one to three segments -- in one batch per element type against
the oracle, bit for bit equal to one launch per nest and, for int32, to a plan of each."""
import numpy as np
import pytest

import paper_2309_01906_amd as hp
import workloads
from gpu_util import assert_match, say, to_device

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROWS = [1, 2, 3, 4, 5, 7, 8, 9, 31, 63, 64, 65, 127, 255, 257, 511, 513, 1023, 1025, 2047, 2049, 3001, 4097, 8191]
LONG = [40000, 65537, 262145, 1000003]
FLAT_OPS = ["SUM", "MAX", "MIN", "ARGMAX", "ARGMIN"]
TWO = [("SUM", "MAX"), ("ARGMAX", "SUM"), ("MIN", "SUM"), ("SUM", "ARGMIN"), ("ARGMIN", "ARGMAX"), ("MAX", "MIN")]
THREE = [("SUM", "MAX", "ARGMIN"), ("ARGMAX", "SUM", "MIN"), ("MIN", "ARGMIN", "SUM"), ("ARGMIN", "MAX", "ARGMAX")]


def flat(ops):
    for k, rows in enumerate(ROWS):
        for n in (1, 3, 67, 1001):
            if n * rows < 1 << 20:
                yield (n, rows), ("NONE", ops[k % len(ops)])
    for k, rows in enumerate(LONG):
        yield (1 + k % 2, rows), ("NONE", ops[k % len(ops)])


def nested():
    for k, rows in enumerate(ROWS[:18]):
        for j, (m, n) in enumerate([(1, 5), (2, 70), (17, 33), (65, 3), (1000, 1)]):
            yield (n, m, rows), ("NONE",) + TWO[(k + j) % 6]
    for k, (q, m, n, rows) in enumerate([(2, 2, 40, 1), (3, 7, 500, 3), (70, 3, 2, 9), (9, 33, 11, 64), (1500, 2, 1, 100),
                                         (5, 300, 3, 17), (4, 3, 2, 30001), (3, 2000, 2, 40), (600, 3, 2, 5)]):
        for ops in THREE:
            yield (n, q, m, rows), ("NONE",) + ops
    yield (2, 3, 70001), ("NONE", "ARGMAX", "SUM")  # parts of a row under a middle level
    yield (3, 20001, 5), ("NONE", "ARGMIN", "SUM")  # parts of the middle level, wide keys
    yield (2, 1, 90000), ("NONE", "ARGMAX", "MIN")  # an ARG level of one iteration
    yield (4, 1, 33), ("NONE", "SUM", "MAX")
    yield (4, 1, 1), ("NONE", "SUM", "MAX")
    yield (6, 5, 1), ("NONE", "MAX", "SUM")


def run(nests, hosts, flags=0):
    """Outputs of the batch, of three replays of its graph, and of one launch per nest."""
    devs = [to_device(h) for h in hosts]
    with hp.Batch(nests, flags) as b:
        outs = [torch.zeros(b.info(i)["n_out"], dtype=hp.torch_out_dtype(b.info(i)["out_dtype"]), device="cuda")
                for i in range(len(nests))]
        b.set_io(devs, outs)
        got = []
        for _ in range(3 if flags & hp.BATCH_GRAPH else 1):
            for t in outs:
                t.fill_(77)
            torch.cuda.synchronize()
            b.run()
            torch.cuda.synchronize()
            got.append([t.cpu().numpy() for t in outs])
            torch.sum(outs[0].double()).item()  # eager work between replays
        for t in outs:
            t.fill_(77)
        b.run_each()
        torch.cuda.synchronize()
        each = [t.cpu().numpy() for t in outs]
    for g in got:
        for i, (e, o, _) in enumerate(nests):
            np.testing.assert_array_equal(g[i], each[i], err_msg=f"nest {i} {e} {o}")
    return each


@pytest.mark.parametrize("flags", [0, hp.BATCH_GRAPH])
@pytest.mark.parametrize("lo,hi", [(-(1 << 31), (1 << 31) - 1), (-2, 2)])  # sums beyond 32 bits; ties
def test_int32_units(lo, hi, flags):
    shapes = list(flat(FLAT_OPS)) + list(nested())
    nests = [(e, o, hp.I32) for e, o in shapes]
    hosts = [workloads.uniform_i32(700 + i, e, lo, hi) for i, (e, _) in enumerate(shapes)]
    say("case units int32", len(nests), lo, hi, flags)
    outs = run(nests, hosts, flags)
    for i, (e, o) in enumerate(shapes):
        assert_match(outs[i], hosts[i], e, o, what=f"{e} {o}")
        if not flags:
            with hp.Plan(e, o, hp.I32) as p:
                np.testing.assert_array_equal(p.run(to_device(hosts[i])).cpu().numpy(), outs[i], err_msg=f"{e} {o}")


@pytest.mark.parametrize("flags", [0, hp.BATCH_GRAPH, hp.FLAG_OUT_F32])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_float_units(dtype, flags):
    shapes = list(flat(["SUM"])) + [((3, 5, 77), ("NONE", "SUM", "SUM")), ((4, 1, 9000), ("NONE", "SUM", "SUM"))]
    draw, code = (workloads.normal_f32, hp.F32) if dtype == "f32" else (workloads.normal_bf16_bits, hp.BF16)
    nests = [(e, o, code) for e, o in shapes]
    hosts = [draw(800 + i, e) for i, (e, _) in enumerate(shapes)]
    say("case units", dtype, len(nests), flags)
    outs = run(nests, hosts, flags)
    for i, (e, o) in enumerate(shapes):
        assert_match(outs[i], hosts[i], e, o, rel=2.0 ** -23 if flags & hp.FLAG_OUT_F32 else 1e-13, what=f"{e} {o}")


def test_extremes_and_non_finite_values():
    nests, hosts = [], []
    for fill, mm in [(np.iinfo(np.int32).max, "MIN"), (np.iinfo(np.int32).min, "MAX")]:
        for ext in [(5, 3), (5, 67), (2, 9000), (1, 70000), (5, 7, 3), (2, 9, 2000)]:
            for op in [mm, "ARG" + mm]:
                nests.append((ext, ("NONE", op) if len(ext) == 2 else ("NONE", op, mm), hp.I32))
                hosts.append(np.full(ext, fill, np.int32))
    for (e, o, _), x, got in zip(nests, hosts, run(nests, hosts)):
        assert_match(got, x, e, o, what=f"extremes {e} {o}")
    exts = [(3, 2), (3, 5), (3, 700), (2, 9001), (1, 300000)]
    x = [workloads.normal_f32(900 + i, e) for i, e in enumerate(exts)]
    for v, bad in zip(x, [np.inf, np.nan, -np.inf, np.inf, np.nan]):
        v[0, v.shape[1] // 2] = bad
    for e, v, got in zip(exts, x, run([(e, ("NONE", "SUM"), hp.F32) for e in exts], x)):
        assert np.isnan(got[0]) and np.isfinite(got[1:]).all(), e


@pytest.mark.parametrize("slot_bytes", [8 << 10, 64 << 10, 64 << 20])
def test_served_units_and_plan_tasks(slot_bytes):
    """Requests on unit tasks and on plan tasks (four reducing segments), with folds of
    both kinds, in one server: the same bits as a batch of them where the slot lets the
    request run alike, and the oracle's values in slots too small for some unit tasks."""
    shapes = [(e, ("NONE", "SUM"), hp.F32) for e in [(5, 3), (67, 33), (2, 9000), (1, 1000003)]]
    shapes += [(e, o, hp.I32) for e, o in [((40, 50, 3, 30), ("NONE", "ARGMAX", "SUM", "MIN")), ((2, 3, 70001), ("NONE", "ARGMAX", "SUM")),
                                          ((300, 77), ("NONE", "ARGMIN")), ((2, 3, 4, 5, 6), ("NONE", "SUM", "MAX", "SUM", "MIN")),
                                          ((1, 3, 4, 5, 6000), ("NONE", "SUM", "MAX", "SUM", "MIN")), ((9,), ("NONE",))]]
    hosts = [workloads.normal_f32(950 + i, e) if d == hp.F32 else workloads.uniform_i32(950 + i, e, -9, 9)
             for i, (e, _, d) in enumerate(shapes)]
    want = run(shapes, hosts)
    devs = [to_device(h) for h in hosts]
    say("case served units", slot_bytes)
    with hp.Server(slot_bytes=slot_bytes, streams=2, max_batch=32, window_us=200) as s:
        for _ in range(3):
            tickets, outs = [], []
            for k in range(4 * len(shapes)):
                i = k % len(shapes)
                e, o, d = shapes[i]
                outs.append(torch.full(want[i].shape, 77, dtype=torch.from_numpy(want[i]).dtype, device="cuda"))
                torch.cuda.synchronize()
                try:
                    tickets.append(s.submit(e, o, d, devs[i].data_ptr(), outs[-1].data_ptr()))
                except hp.HPError as err:
                    assert err.status_name == "HP_ETOOBIG" and slot_bytes == 8 << 10
                    tickets.append(None)
            for k, t in enumerate(tickets):
                if t is None:
                    continue
                assert s.wait(t)["status"] == 0
                i = k % len(shapes)
                e, o, _ = shapes[i]
                got = outs[k].cpu().numpy()
                assert_match(got, hosts[i], e, o, rel=1e-13, what=f"served {e} {o}")
                if slot_bytes == 64 << 20:
                    np.testing.assert_array_equal(got, want[i])


@pytest.mark.parametrize("flags", [0, hp.BATCH_GRAPH])
def test_folds_that_a_workgroup_shares(flags):
    """Outputs of many carriers beside ones of few: every form of the fold, at several waves
    and at one, with ties and with the extreme value everywhere."""
    shapes = [((2, 3000, 8, 64), ("ARGMIN", "MAX", "SUM")), ((1, 40000, 4, 8), ("SUM", "MAX", "SUM")),
              ((3, 700, 40, 90), ("ARGMAX", "ARGMIN", "MAX")), ((1, 700000, 64), ("ARGMAX", "MIN")),
              ((2, 90, 40000), ("SUM", "ARGMAX")), ((1, 4, 60, 30000), ("ARGMIN", "MIN", "MAX")),
              ((1, 3, 5, 900000), ("MAX", "ARGMAX", "MIN")), ((1, 1 << 24), ("ARGMIN",)), ((5, 100, 4, 8), ("MIN", "SUM", "MAX")),
              ((4, 33), ("SUM",)), ((1, 2, 300000), ("ARGMIN", "SUM"))]
    nests = [(e, ("NONE",) + o, hp.I32) for e, o in shapes]
    for fill in [None, np.iinfo(np.int32).max, np.iinfo(np.int32).min]:
        hosts = [workloads.uniform_i32(900 + i, e, -2, 2) if fill is None else np.full(e, fill, np.int32)
                 for i, (e, _) in enumerate(shapes)]
        say("case shared folds", fill, flags)
        for (e, o, _), x, got in zip(nests, hosts, run(nests, hosts, flags)):
            assert_match(got, x, e, o, what=f"shared folds {e} {o}")
    x = workloads.normal_f32(950, (1, 1 << 25))
    nests = [((1, 1 << 25), ("NONE", "SUM"), hp.F32), ((2, 1 << 24), ("NONE", "SUM"), hp.F32), ((7, 9), ("NONE", "SUM"), hp.F32)]
    hosts = [x, x.reshape(2, -1), x[0, :63].reshape(7, 9).copy()]
    for (e, o, _), h, got in zip(nests, hosts, run(nests, hosts, flags)):
        assert_match(got, h, e, o, rel=1e-13, what=f"shared folds {e}")


def test_served_folds_that_a_workgroup_shares():
    """Requests whose outputs a workgroup or a wave folds, and plan tasks, in the same batches of a server."""
    shapes = [((2, 3000, 8, 64), ("ARGMIN", "MAX", "SUM")), ((5, 100, 4, 8), ("MIN", "SUM", "MAX")), ((4, 33), ("SUM",)),
              ((1, 40000, 4, 8), ("SUM", "MAX", "SUM")), ((3, 700, 40, 90), ("ARGMAX", "ARGMIN", "MAX")),
              ((2, 3, 2, 5, 7), ("SUM", "MAX", "SUM", "MIN")), ((2, 90, 40000), ("SUM", "ARGMAX"))]
    nests = [(e, ("NONE",) + o, hp.I32) for e, o in shapes]
    hosts = [workloads.uniform_i32(970 + i, e, -2, 2) for i, (e, _) in enumerate(shapes)]
    devs = [to_device(h) for h in hosts]
    say("case served folds", len(nests))
    with hp.Server(slot_bytes=64 << 20, streams=2, max_batch=32) as s:
        for _ in range(3):
            outs = []
            for e, o, d in nests:
                inf = hp.inspect(e, o, d)
                outs.append(torch.full((inf["n_out"],), 77, dtype=hp.torch_out_dtype(inf["out_dtype"]), device="cuda"))
            torch.cuda.synchronize()
            tickets = s.replay(nests, [t.data_ptr() for t in devs], [t.data_ptr() for t in outs], [0.0] * len(nests))
            assert all(s.wait(t)["status"] == 0 for t in tickets)
            torch.cuda.synchronize()
            for (e, o, _), x, got in zip(nests, hosts, outs):
                assert_match(got.cpu().numpy(), x, e, o, what=f"served folds {e} {o}")
