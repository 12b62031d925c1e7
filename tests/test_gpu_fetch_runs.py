"""Runs of more entries than a fetch has lanes: 64 of them a round trip, each workgroup reading its own in full and the others' only as far
as says whose they are.  Runs that end at, before and behind a multiple of 64, SQs shorter and longer than the run, a task queue that
fills up on the way, an exit entry inside the run, rings (whose fetch drops caches) among fold steps, priorities, a limit on entries
in a row, the SQ in host memory; three passes on the same context, the last one begun by a daemon that finds everything in the SQ, each
compared by itself; and what the daemon counts says that fetches went on behind their first 64 entries, and did not where they must not.
Bit-exact against the oracle (same order of combination, one rounding per hop: no tolerance)."""
import numpy as np
import pytest

import workload_inputs as wi
from oracle import ring_data as rd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,channels,n,knobs", [
    (8, 4, 129, {}), (8, 4, 128, dict(sq_depth=128)), (8, 2, 127, dict(sq_depth=64)), (4, 8, 320, {}), (2, 1, 200, dict(max_colls=200)),
    (4, 2, 193, dict(order_policy=1)), (4, 4, 150, dict(fetch_batch=70)), (4, 4, 150, dict(sq_in_device=0)), (4, 2, 140, dict(fold_max_bytes=0)),
    (3, 4, 260, dict(sq_depth=256, cq_mode=2)), (8, 8, 300, dict(chan_spread=0))])
def test_runs_of_entries(R, channels, n, knobs):
    from paper_2303_06324_amd import harness as gh
    import paper_2303_06324_amd as dfx
    g = np.random.default_rng(R * 1000 + n)
    colls = []
    for i in range(n):
        kind, dtype = (wi.AR, wi.RS, wi.AG, wi.BC, wi.RD)[i % 5], (wi.I32, wi.F32, wi.BF16, wi.F16)[i // 5 % 4]
        count = int(g.integers(1, 700)) if i % 9 else 30000      # (now and then several channels; odd all-gathers are rings)
        colls.append(wi.CollSpec(i, kind, dtype, count, int(g.integers(R)) if kind in (wi.BC, wi.RD) else 0, wi.SUM))
    w = wi.Workload(f"runs_{R}_{n}", R, colls, [list(map(int, g.permutation(n))) for _ in range(R)], seed=n, cfg=130)
    dw = gh.DeviceWorkload(w)
    want = [rd.run_closed_form(c.kind, dw.send_host[ci], c.dtype, c.root, c.op) for ci, c in enumerate(w.colls)]

    def check(it):
        for ci, c in enumerate(w.colls):
            got = dw.results(ci)
            for r in range(R):
                if c.kind == wi.RD and r != c.root:
                    assert np.all(got[r].view(np.uint8) == 0xA5), (it, ci, r)
                else:
                    assert np.array_equal(got[r].view(np.uint8), want[ci][r].view(np.uint8)), (it, ci, c, r)
        dw.check_untouched()

    ctx = dfx.Context(R, gh.make_config(max_channels=channels, **knobs))
    try:
        gh.prepare_all(ctx, w, priorities=[(i * 5) % 7 - 3 for i in range(n)] if knobs.get("order_policy") else None)
        for it in range(3):
            dw.reset_recv()
            if it == 2 and knobs.get("sq_depth", 1024) > n + 1:
                # an exit entry behind the run of all ranks but one; the last rank's run and the rest are another daemon's
                for r in range(R - 1):
                    burst = ctx.make_burst(w.orders[r], [dw.send[ci][r].data_ptr() for ci in w.orders[r]], [dw.recv[ci][r].data_ptr() for ci in w.orders[r]])
                    assert ctx.submit_burst(r, burst) == n
                assert ctx.stop() == dfx.OK
                r = R - 1
                burst = ctx.make_burst(w.orders[r], [dw.send[ci][r].data_ptr() for ci in w.orders[r]], [dw.recv[ci][r].data_ptr() for ci in w.orders[r]])
                assert ctx.submit_burst(r, burst) == n
            else:
                gh.submit_threads(ctx, dw) if it else gh.submit_bursts(ctx, dw)
            assert ctx.wait_all(30.0) == dfx.OK
            check(it)
        assert ctx.stop() == dfx.OK
        st, ways = [ctx.stats(r) for r in range(R)], [ctx.counters(r) for r in range(R)]
    finally:
        ctx.finalize()
    assert all(s["cqe_posted"] == 3 * n for s in st)
    assert all(s["sqe_fetched"] >= 3 * n * channels for s in st)
    went_on = sum(k["run_on"] for k in ways)
    if "fetch_batch" in knobs or knobs.get("sq_depth", 1024) <= 64:
        assert went_on == 0, ways
    else:
        assert went_on > 0, ways


def test_an_sq_that_32_bit_offsets_do_not_reach():
    """2^25 slots, 4 GiB: the part of the fetch that addresses slots by 32-bit offsets is left out, and no entry is lost."""
    import torch
    from paper_2303_06324_amd import harness as gh
    import paper_2303_06324_amd as dfx
    n = 300
    try:
        ctx = dfx.Context(1, gh.make_config(max_channels=1, max_colls=n, sq_depth=1 << 25, pool_bytes=64 << 20))
    except dfx.DfxError as e:
        pytest.skip(f"no memory for such a ring: {e}")
    try:
        send = torch.arange(64 * n, dtype=torch.int32, device="cuda").view(n, 64)
        recv = torch.full((n, 64), -1, dtype=torch.int32, device="cuda")
        for i in range(n):
            ctx.prepare(i, dfx.ALLREDUCE, 64, dfx.I32)
        for _ in range(3):
            recv.fill_(-1)
            torch.cuda.synchronize()
            assert ctx.submit_many(0, list(range(n)), [t.data_ptr() for t in send], [t.data_ptr() for t in recv]) == n
            assert ctx.wait_all(10.0) == dfx.OK
            assert ctx.stop() == dfx.OK
            assert torch.equal(send, recv)
    finally:
        ctx.finalize()
