"""A lone entry of a collective in fold steps takes a short way through the fetch: its context goes straight into its LDS
slot, its SQ slot is freed when a later poll is back, its completion writes nothing back.  Checked where that can go
wrong: the smallest SQ (every entry reuses a slot that has just been freed), ids whose contexts share one LDS slot, waits
that are given up at once (the last one of a lone collective: after 256 polls) or never, collectives that need the connectors in between, the three CQ variants, and many
invocations of one id (the counters that run on).  Bit-exact against the oracle."""
import numpy as np
import pytest

import workload_inputs as wi
from oracle import ring_data as rd

pytestmark = pytest.mark.gpu


def _slot(cid):
    return ((cid * 2654435769) & 0xffffffff) >> 26


def _ids_of_one_slot(n, limit=2048):
    return [i for i in range(limit) if _slot(i) == _slot(1)][:n]


@pytest.mark.parametrize("knobs", [dict(), dict(scan_min=0, spin_init=1, spin_min=1, spin_max=1, spin_boost=1), dict(preempt=0), dict(cq_mode=1), dict(cq_mode=2),
                                   dict(order_policy=1), dict(sq_in_device=0)], ids=["defaults", "give_up_at_once", "never_give_up", "cq1", "cq2", "priority", "sq_on_host"])
def test_lone_entries_reuse_everything(knobs):
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    R = 4
    ids = _ids_of_one_slot(3)
    # two in fold steps of one channel, and (largest buffer above fold_max_bytes) two of several channels through the connectors
    colls = [wi.CollSpec(ids[0], wi.AR, wi.F32, 1000), wi.CollSpec(ids[1], wi.BC, wi.BF16, 4099, 2), wi.CollSpec(ids[2], wi.RS, wi.I32, 20000),
             wi.CollSpec(7, wi.AR, wi.F16, 70001)]
    w = wi.Workload("lone", R, colls, [list(range(4))] * R, seed=5, cfg=92)
    dw = gh.DeviceWorkload(w)
    ctx = dfx.Context(R, gh.make_config(max_channels=4, chan_spread=0, sq_depth=2, cq_slots=2, fold_max_bytes=131072, **knobs))
    try:
        gh.prepare_all(ctx, w)
        for it in range(40):
            for ci in ((0, 1, 2, 3), (3, 0, 0, 1), (2, 2, 1, 0))[it % 3]:
                gh.submit_round_robin(ctx, dw, orders=[[ci]] * R)      # one after the other: every entry is a lone one
                assert ctx.wait_all(20.0) == dfx.OK
        assert ctx.stop() == dfx.OK
        for ci, c in enumerate(colls):
            want, got = rd.run_closed_form(c.kind, dw.send_host[ci], c.dtype, c.root, c.op), dw.results(ci)
            for r in range(R):
                assert np.array_equal(got[r].view(np.uint8), want[r].view(np.uint8)), (knobs, ci, r)
        dw.check_untouched()
    finally:
        assert ctx.finalize() == dfx.OK


@pytest.mark.parametrize("how", ["all_at_once", "rank_by_rank"])
def test_the_last_wait_outlasts_its_polls(how):
    """A collective that is alone in its queue is not given up at its threshold, but after so many polls it is, and taken up again by
    the next pass: one channel, whose job takes far longer than the polls do."""
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    R = 4
    w = wi.Workload("lone_long", R, [wi.CollSpec(0, wi.AR, wi.I32, (6 << 20) + 5)], [[0]] * R, seed=8, cfg=104)
    dw = gh.DeviceWorkload(w)
    ctx = dfx.Context(R, gh.make_config(max_channels=1))
    try:
        gh.prepare_all(ctx, w)
        assert ctx.coll_info(0)["rounds"] == 1
        p = ctx.make_all([t.data_ptr() for t in dw.send[0]], [t.data_ptr() for t in dw.recv[0]])
        for _ in range(5):
            if how == "all_at_once":
                assert ctx.submit_all(0, p) == dfx.OK
            else:
                gh.submit_round_robin(ctx, dw)
            assert ctx.wait_all(20.0) == dfx.OK
        assert ctx.stop() == dfx.OK
        assert sum(ctx.stats(r)["preemptions"] for r in range(R)) >= 5 * R
    finally:
        assert ctx.finalize() == dfx.OK
    want, got = rd.run_closed_form(wi.AR, dw.send_host[0], wi.I32, 0, wi.SUM), dw.results(0)
    for r in range(R):
        assert np.array_equal(got[r], want[r]), r
    dw.check_untouched()
