"""Send buffers rewritten by kernels while the daemon stays resident.  A collective in fold steps drops no cache at its fetch
and writes none back at its completion: its loads and stores go past the L2s.  So between two invocations inside ONE daemon launch
other kernels rewrite every send buffer, read every send and recv buffer (old lines come to lie in the L2s of all XCDs) and
keep what the invocation before left in the recv buffers; nothing in between waits for the daemon to leave (no copies to
the host, no device-wide synchronization, a stream that is seen to run beside the daemon).  The same buffers also go through
a ring, whose fetch and completion do work on the caches.  int32 sums and copies: exact."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

R, ITERATIONS, ROOT = 8, 12, 3


def _done(ev, seconds):
    t0 = time.perf_counter()
    while not ev.query():
        if time.perf_counter() - t0 > seconds:
            return False
    return True


def _stream_beside_the_daemon(torch, x):
    """Streams share a few hardware queues; work on the daemon's own one would wait for it to leave."""
    for _ in range(8):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            x.add_(1)
            ev = torch.cuda.Event()
            ev.record(st)
        if _done(ev, 0.2):
            return st
    pytest.fail("no stream ran beside the daemon")


@pytest.mark.parametrize("n", [256, 4096, 1 << 18])
@pytest.mark.parametrize("kind", ["allreduce", "allgather", "reducescatter", "broadcast", "reduce"])
def test_send_buffers_rewritten_under_a_resident_daemon(kind, n):
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    k = dict(allreduce=dfx.ALLREDUCE, allgather=dfx.ALLGATHER, reducescatter=dfx.REDUCESCATTER, broadcast=dfx.BROADCAST, reduce=dfx.REDUCE)[kind]
    ns, nr = (n * R if k == dfx.REDUCESCATTER else n), (n * R if k == dfx.ALLGATHER else n)
    base = [(np.arange(ns, dtype=np.int64) * 3 + 1000003 * r).astype(np.int32) for r in range(R)]
    send = [torch.from_numpy(b).cuda() for b in base]
    recv = [torch.full((nr,), -1, dtype=torch.int32, device="cuda") for _ in range(R)]
    ring = [torch.full((R * n,), -1, dtype=torch.int32, device="cuda") for _ in range(R)]        # an all-gather of odd blocks
    kept = torch.zeros((ITERATIONS, R, nr), dtype=torch.int32, device="cuda")
    kept_ring = torch.zeros((ITERATIONS, R, (n - 1) * R), dtype=torch.int32, device="cuda")
    scratch, reads = torch.zeros(64, device="cuda"), torch.zeros(R, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    # four channels per rank leave the other kernels most of the compute units; a second without work before the daemon leaves
    ctx = dfx.Context(R, gh.make_config(max_channels=4, quit_idle_us=1_000_000, pool_bytes=256 << 20))
    try:
        ctx.prepare(0, k, n, dfx.I32, dfx.SUM, ROOT if k in (dfx.BROADCAST, dfx.REDUCE) else 0)
        ctx.prepare(1, dfx.ALLGATHER, n - 1, dfx.I32)
        assert ctx.coll_info(0)["nprim"] == 2 and ctx.coll_info(1)["nprim"] == R                 # fold steps; the ring through slots
        p0 = ctx.make_all([t.data_ptr() for t in send], [t.data_ptr() for t in recv])
        p1 = ctx.make_all([t.data_ptr() for t in send], [t.data_ptr() for t in ring])
        assert ctx.start() == dfx.OK
        st = _stream_beside_the_daemon(torch, scratch)
        for i in range(ITERATIONS):
            with torch.cuda.stream(st):
                for r in range(R):
                    reads[r] = send[r].sum() + recv[r].sum()
                    send[r].add_(r * 7 + i + 1)
                ev = torch.cuda.Event()
                ev.record(st)
            assert _done(ev, 10.0)
            for cid, ptrs in ((0, p0), (1, p1)) if i % 2 == 0 else ((1, p1), (0, p0)):
                assert ctx.submit_all(cid, ptrs) == dfx.OK and ctx.wait_all(10.0) == dfx.OK
            with torch.cuda.stream(st):
                for r in range(R):
                    torch.add(recv[r], 0, out=kept[i, r])
                    torch.add(ring[r][:(n - 1) * R], 0, out=kept_ring[i, r])
                ev = torch.cuda.Event()
                ev.record(st)
            assert _done(ev, 10.0)
            if i == 0: launches = ctx.stats(0)["launches"]
        assert ctx.stats(0)["launches"] == launches          # one daemon through all iterations but the first
        assert ctx.stop() == dfx.OK
    finally:
        ctx.finalize()
    torch.cuda.synchronize()
    kept, kept_ring = kept.cpu().numpy(), kept_ring.cpu().numpy()
    for i in range(ITERATIONS):
        now = [(b.astype(np.int64) + sum(r * 7 + j + 1 for j in range(i + 1))).astype(np.int32) for r, b in enumerate(base)]
        total = np.sum([x.astype(np.int64) for x in now], axis=0).astype(np.int32)
        for r in range(R):
            want = {dfx.ALLREDUCE: total, dfx.ALLGATHER: np.concatenate(now), dfx.REDUCESCATTER: total[r * n:(r + 1) * n],
                    dfx.BROADCAST: now[ROOT], dfx.REDUCE: total}[k]
            if k == dfx.REDUCE and r != ROOT:
                want = np.full(nr, -1, np.int32)
            assert np.array_equal(kept[i, r], want), (kind, n, i, r)
            assert np.array_equal(kept_ring[i, r], np.concatenate([x[:n - 1] for x in now])), (kind, n, i, r)


@pytest.mark.parametrize("kind", ["allreduce", "allgather", "reducescatter", "broadcast", "reduce"])
def test_swept_messages_rewritten_under_a_resident_daemon(kind):
    """The same for a message that all ranks sweep together: its loads carry the non-temporal hint."""
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    k = dict(allreduce=dfx.ALLREDUCE, allgather=dfx.ALLGATHER, reducescatter=dfx.REDUCESCATTER, broadcast=dfx.BROADCAST, reduce=dfx.REDUCE)[kind]
    whole = (32 if k in (dfx.ALLGATHER, dfx.BROADCAST) else 16) << 18               # elements of the largest per-rank buffer
    n = whole // R if k in (dfx.ALLGATHER, dfx.REDUCESCATTER) else whole
    ns, nr = (n * R if k == dfx.REDUCESCATTER else n), (n * R if k == dfx.ALLGATHER else n)
    send = [torch.arange(ns, dtype=torch.int32, device="cuda") * 3 + 1000003 * r for r in range(R)]
    recv = [torch.full((nr,), -1, dtype=torch.int32, device="cuda") for _ in range(R)]
    wrong = torch.zeros((ITERATIONS, R), dtype=torch.int64, device="cuda")
    scratch, reads = torch.zeros(64, device="cuda"), torch.zeros(R, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    cfg = gh.make_config(max_channels=4, quit_idle_us=1_000_000, pool_bytes=256 << 20)
    root = ROOT if k in (dfx.BROADCAST, dfx.REDUCE) else 0
    assert "sweep" in dfx.plan_route(R, k, n, dfx.I32, root, cfg)
    ctx = dfx.Context(R, cfg)
    try:
        ctx.prepare(0, k, n, dfx.I32, dfx.SUM, root)
        p = ctx.make_all([t.data_ptr() for t in send], [t.data_ptr() for t in recv])
        assert ctx.start() == dfx.OK
        st = _stream_beside_the_daemon(torch, scratch)
        for i in range(ITERATIONS):
            with torch.cuda.stream(st):
                for r in range(R):
                    reads[r] = send[r].sum() + recv[r].sum()
                    send[r].add_(r * 7 + i + 1)
                ev = torch.cuda.Event()
                ev.record(st)
            assert _done(ev, 10.0)
            assert ctx.submit_all(0, p) == dfx.OK and ctx.wait_all(10.0) == dfx.OK
            with torch.cuda.stream(st):
                total = sum(send[1:], send[0])
                for r in range(R):
                    want = {dfx.ALLREDUCE: total, dfx.REDUCESCATTER: total[r * n:(r + 1) * n], dfx.REDUCE: total, dfx.BROADCAST: send[ROOT]}.get(k)
                    if k == dfx.ALLGATHER:
                        wrong[i, r] = sum((recv[r][q * n:(q + 1) * n] != send[q]).sum() for q in range(R))
                    elif k == dfx.REDUCE and r != ROOT:
                        wrong[i, r] = (recv[r] != -1).sum()
                    else:
                        wrong[i, r] = (recv[r] != want).sum()
                ev = torch.cuda.Event()
                ev.record(st)
            assert _done(ev, 10.0)
            if i == 0: launches = ctx.stats(0)["launches"]
        assert ctx.stats(0)["launches"] == launches          # one daemon through all iterations but the first
        assert ctx.stop() == dfx.OK
    finally:
        ctx.finalize()
    torch.cuda.synchronize()
    assert int(wrong.sum()) == 0, wrong.cpu()
