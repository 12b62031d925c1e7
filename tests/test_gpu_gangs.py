"""Bursts of short collectives in fold steps, which a readiness scan hands to the movers several at a time and whose completions it
posts itself: every kind, element type and reducing function at the edges of rows and of the longest share that goes with others,
collectives of one and of several channels and a long one between them, every rank in an order of its own, in queues of one, two
and four channels (more and fewer entries than a scan holds), with and without priorities, with the ring-buffer completion queue,
three passes on the same context and one that begins with a stop half way, each compared by itself; and what the daemon counts says that
gangs were formed, and none where they are switched off.
Bit-exact against the oracle (same order of combination, one rounding per hop: no tolerance)."""
import numpy as np
import pytest

import workload_inputs as wi
from oracle import ring_data as rd

pytestmark = pytest.mark.gpu


def _workload(R, n, seed):
    g = np.random.default_rng(seed)
    colls = []
    for i in range(n):
        kind, dtype = (wi.AR, wi.AG, wi.RS, wi.BC, wi.RD)[i % 5], (wi.F32, wi.BF16, wi.F16, wi.I32)[i // 5 % 4]
        eb, op = wi.ELEM_BYTES[dtype], (wi.SUM, wi.MAX, wi.PROD, wi.MIN)[i % 4] if kind in (wi.AR, wi.RS, wi.RD) else wi.SUM
        part = (16, 2032, 2048, 4112, 8192, 16368, 16384, 16400, 40000, 70000)[i * 7 % 10]         # bytes of a rank's region, about
        count = part // 16 * 16 // eb if kind in (wi.AG, wi.RS) else max(1, R * part // eb - (0, 1, 3)[i % 3])
        colls.append(wi.CollSpec(i, kind, dtype, count, int(g.integers(R)) if kind in (wi.BC, wi.RD) else 0, op))
    colls[n // 2] = wi.CollSpec(n // 2, wi.AR, wi.BF16, (1 << 20) + 5)
    return wi.Workload(f"gangs_{R}", R, colls, [list(map(int, g.permutation(n))) for _ in range(R)], seed=seed, cfg=110)


@pytest.mark.parametrize("R,channels,n,knobs", [
    (2, 1, 60, {}), (3, 2, 80, {}), (4, 4, 120, {}), (8, 2, 60, {}), (8, 4, 200, {}), (16, 1, 40, {}), (33, 1, 20, {}),
    (8, 1, 90, {}),                                  # a queue longer than a scan's lanes
    (4, 2, 60, dict(order_policy=1)), (8, 1, 90, dict(order_policy=1)), (8, 2, 60, dict(cq_mode=1)), (8, 2, 60, dict(spin_min=2)),
    (8, 2, 60, dict(focus_bytes=0)), (5, 2, 60, dict(quit_idle_us=30))])
def test_short_collectives_together(R, channels, n, knobs):
    from paper_2303_06324_amd import harness as gh
    import paper_2303_06324_amd as dfx
    w = _workload(R, n, seed=R * 100 + n)
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
        for it in range(4):
            dw.reset_recv()
            if it == 3:                              # the daemon leaves with some ranks' entries in its queues, and comes back
                for r in range(R - 1):
                    for ci in w.orders[r]:
                        assert ctx.submit(r, ci, dw.send[ci][r].data_ptr(), dw.recv[ci][r].data_ptr()) == dfx.OK
                assert ctx.stop() == dfx.OK
                gh.submit_round_robin(ctx, dw, orders=[[]] * (R - 1) + [w.orders[R - 1]])
            else:
                gh.submit_bursts(ctx, dw)
            assert ctx.wait_all(30.0) == dfx.OK
            check(it)
        assert ctx.stop() == dfx.OK
        st, ways = [ctx.stats(r) for r in range(R)], [ctx.counters(r) for r in range(R)]
    finally:
        ctx.finalize()
    assert all(s["cqe_posted"] == 4 * n for s in st)
    assert all(s["preemptions"] == s["ctx_saves"] + s["lazy_skips"] for s in st)
    gangs, ganged, unpolled = (sum(k[name] for k in ways) for name in ("gangs", "ganged", "unpolled"))
    if R > 32 or "focus_bytes" in knobs or "spin_min" in knobs:      # controls: nothing goes in gangs
        assert gangs == ganged == 0, ways
    else:
        assert gangs > 0 and ganged >= 2 * gangs, ways
    assert (unpolled > 0) == ("spin_min" not in knobs) and all(k["unpolled"] <= s["preemptions"] for k, s in zip(ways, st)), ways


@pytest.mark.parametrize("R,knobs,budget", [(8, dict(order_policy=1), 32 << 10), (4, dict(order_policy=1), 32 << 10), (2, dict(order_policy=1, focus_bytes=20000), 20000),
                                            (8, dict(focus_bytes=20000), 40000), (4, dict(), 256 << 10)])
def test_a_gang_holds_to_the_bytes_of_a_pass(R, knobs, budget):
    """Shares of up to 16 KiB, as many of them queued as would fill the largest gangs: one job takes no more than a pass may hand the movers
    before it looks at the SQ and the queue again (32 KiB at most under priority ordering; under FIFO ordering twice focus_bytes)."""
    from paper_2303_06324_amd import harness as gh
    import paper_2303_06324_amd as dfx
    n, channels = 60, 4
    colls = [wi.CollSpec(i, (wi.AR, wi.RS, wi.BC)[i % 3], wi.F32, (R if i % 3 != 1 else 1) * ((16 << 10) * channels - 64 * (i % 5)) // 4) for i in range(n)]
    w = wi.Workload(f"gang_bytes_{R}", R, colls, [list(range(n))] * R, seed=R, cfg=112)
    dw = gh.DeviceWorkload(w)
    ctx = dfx.Context(R, gh.make_config(max_channels=channels, **knobs))
    try:
        gh.prepare_all(ctx, w)
        for _ in range(4):
            dw.reset_recv()
            gh.submit_bursts(ctx, dw)
            assert ctx.wait_all(30.0) == dfx.OK
        assert ctx.stop() == dfx.OK
        went = [ctx.counters(r) for r in range(R)]
    finally:
        ctx.finalize()
    assert sum(k["gangs"] for k in went) > 0 or budget < 32 << 10, went
    assert all(k["ganged"] >= 2 * k["gangs"] and k["gang_max_bytes"] <= budget for k in went), went
    for ci, c in enumerate(w.colls):
        want, got = rd.run_closed_form(c.kind, dw.send_host[ci], c.dtype, c.root, c.op), dw.results(ci)
        assert all(np.array_equal(got[r].view(np.uint8), want[r].view(np.uint8)) for r in range(R)), (ci, c)
    dw.check_untouched()


@pytest.mark.parametrize("R,nbytes,knobs", [(8, 128 << 10, dict(chan_spread=0)), (4, 64 << 10, dict(max_channels=1)), (2, 32 << 10, dict(chan_spread=0, max_channels=4))])
def test_a_long_one_has_its_turn_in_steady_traffic(R, nbytes, knobs, tmp_path):
    """Forty short collectives on one channel, each submitted again as soon as it is complete, and a long one among them: it is
    complete long before the traffic ends (int32: exact)."""
    import ctypes as C
    import os
    import subprocess
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    here = os.path.dirname(os.path.abspath(__file__))
    so, lib = str(tmp_path / "stream.so"), os.path.dirname(dfx.LIB_PATH)
    subprocess.run(["gcc", "-O2", "-Wall", "-shared", "-fPIC", "-I" + os.path.join(here, "..", "include"), os.path.join(here, "c_abi", "stream.c"), "-o", so,
                    "-L" + lib, "-ldfx", "-Wl,-rpath," + lib], check=True)
    turn = C.CDLL(so).stream_turn
    turn.argtypes, turn.restype = [C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_long, C.c_long], C.c_long
    n, sizes = 40, [nbytes // 4] * 40 + [(8 << 20) // 4 + 3]
    g = torch.Generator(device="cuda").manual_seed(R)
    send = [[torch.randint(-1000, 1000, (m,), generator=g, device="cuda", dtype=torch.int32) for _ in range(R)] for m in sizes]
    recv = [[torch.full((m,), -7, device="cuda", dtype=torch.int32) for _ in range(R)] for m in sizes]
    torch.cuda.synchronize()
    s = (C.c_void_p * ((n + 1) * R))(*[t.data_ptr() for row in send for t in row])
    d = (C.c_void_p * ((n + 1) * R))(*[t.data_ptr() for row in recv for t in row])
    ctx = dfx.Context(R, gh.make_config(quit_idle_us=20000, **knobs))
    try:
        for i, m in enumerate(sizes):
            ctx.prepare(i, dfx.ALLREDUCE, m, dfx.I32)
        assert ctx.coll_info(0)["nchan"] == 1 and ctx.coll_info(0)["slot_bytes"] == 16 << 10
        went = [turn(ctx._h, R, n, C.cast(s, C.c_void_p), C.cast(d, C.c_void_p), 400, 6000) for _ in range(5)]
        assert ctx.stop() == dfx.OK
        gangs = sum(ctx.counters(r)["gangs"] for r in range(R))
    finally:
        assert ctx.finalize() == dfx.OK
    assert all(0 < k <= 1500 for k in went), went
    assert gangs > 0
    for row, out in zip(send, recv):
        total = torch.stack(row).sum(0).to(torch.int32)
        assert all(torch.equal(t, total) for t in out)
