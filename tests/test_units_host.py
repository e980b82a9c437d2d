"""Host side of the unit tasks: what a server accepts does not depend on how a request runs."""
import pytest

import paper_2309_01906_amd as hp


@pytest.mark.parametrize("nest", [
    ((40, 500, 3, 30), ("NONE", "ARGMAX", "SUM", "MIN"), hp.I32),   # a carrier per pair: a larger workspace than the plan's
    ((2, 3, 70001), ("NONE", "ARGMAX", "SUM"), hp.I32), ((1, 1 << 22), ("NONE", "SUM"), hp.F32),
    ((3000, 7), ("NONE", "SUM"), hp.BF16), ((9,), ("NONE",), hp.I32)])
def test_a_slot_that_fits_the_plan_is_enough(nest):
    """From the smallest slot that takes the request to far larger ones, every request of
    a burst completes (its unit tasks run only where they fit the slot too)."""
    def served(slot):
        with hp.Server(flags=hp.SERVER_FAKE_DEVICE, slot_bytes=slot, streams=2, max_batch=16, window_us=50) as s:
            infos = [s.wait(t) for t in [s.submit(*nest, 0, 0) for _ in range(20)]]
        return all(i["status"] == 0 for i in infos)
    slot = 4096
    while True:
        try:
            ok = served(slot)
            break
        except hp.HPError as e:
            assert e.status_name == "HP_ETOOBIG"
            slot += 256
    assert ok
    for k in (slot + 256, slot + 4096, 2 * slot, 3 * slot + 256, 1 << 20, 64 << 20):
        assert served(k), k


def test_nests_pack_as_their_fields():
    """Packed nests hold what field by field stores give, also for values that are not
    plain whole numbers."""
    np = pytest.importorskip("numpy")
    for ext, ops, dt in [((4, 5), ("NONE", "sum"), hp.F32), ([3, 2, 7], [0, "ARGMAX", hp.OP_NAMES["MIN"]], 0),
                         ((np.int64(6), np.int32(9)), ("NONE", "MAX"), np.int32(hp.I32)), ((3.0, True), (0, 1.0), 1.0),
                         ((1,) * 8, ("SUM",) * 8, 2), ((-1, 1 << 62), ("NONE", "SUM"), 0)]:
        n = hp.make_nest(ext, ops, dt)
        assert (n.depth, n.dtype) == (len(ext), int(dt))
        assert list(n.extent) == [int(e) for e in ext] + [0] * (8 - len(ext))
        assert list(n.op) == [hp._op(o) for o in ops] + [0] * (8 - len(ext))
    with pytest.raises(ValueError):
        hp.make_nest((1, 2), ("NONE",), 0)
    with pytest.raises(KeyError):
        hp.make_nest((1,), ("AVERAGE",), 0)
