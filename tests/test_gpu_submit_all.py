"""Submissions on every rank at once: the entries come with all ranks' buffers, and a rank that finds one alone in its queue starts
without having seen the others.  Checked where that can go wrong: buffers that change from call to call under the same ids (the
tables of a reused SQ slot), calls that overtake one another (two or more entries in a queue, a table replaced while its collective
still waits), single submissions and rings in between, several jobs, priority ordering, rank counts with and without a data mover
of their own, an SQ of two entries, a table that outlives its invocation.  int32, sums and copies: exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,knobs", [(8, dict()), (8, dict(sq_depth=2, chan_spread=0)), (3, dict(order_policy=1)), (4, dict(scan_min=0, spin_init=1, spin_min=1, spin_max=1, spin_boost=1)),
                                     (16, dict(max_channels=4)), (32, dict(max_channels=3)), (8, dict(fold_max_bytes=1 << 16, direct_min_bytes=0, max_channels=2)), (2, dict(sq_in_device=0))],
                         ids=["defaults", "two_entries", "priority", "give_up_at_once", "sixteen", "thirty_two", "several_jobs", "sq_on_host"])
def test_buffers_change_from_call_to_call(R, knobs):
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    kinds = [dfx.ALLREDUCE, dfx.ALLGATHER, dfx.REDUCESCATTER, dfx.BROADCAST, dfx.REDUCE, dfx.ALLREDUCE, dfx.ALLGATHER]
    counts = [1001, 4096, 2052, 70003, 33333, 200004, 255]                   # (the last one: a ring of odd blocks)
    roots = [0, 0, 0, R - 1, R // 2, 0, 0]
    g = torch.Generator(device="cuda").manual_seed(R)
    sets, want = [], []
    for s in range(3):
        rows = []
        for k, n, root in zip(kinds, counts, roots):
            ns, nr = n * (R if k == dfx.REDUCESCATTER else 1), n * (R if k == dfx.ALLGATHER else 1)
            send = [torch.randint(-1000, 1000, (ns,), generator=g, device="cuda", dtype=torch.int32) for _ in range(R)]
            recv = [torch.full((nr,), -7, device="cuda", dtype=torch.int32) for _ in range(R)]
            total = torch.stack(send).sum(0).to(torch.int32)
            out = [torch.cat(send) if k == dfx.ALLGATHER else total[r * n:(r + 1) * n] if k == dfx.REDUCESCATTER else send[root] if k == dfx.BROADCAST
                   else total if k == dfx.ALLREDUCE or r == root else recv[r].clone() for r in range(R)]
            rows.append((send, recv))
            want.append((recv, out))
        sets.append(rows)
    torch.cuda.synchronize()
    ctx = dfx.Context(R, gh.make_config(**{**dict(max_channels=min(8, 256 // R)), **knobs}))
    try:
        for i, (k, n, root) in enumerate(zip(kinds, counts, roots)):
            ctx.prepare(i, k, n, dfx.I32, dfx.SUM, root, priority=i % 3)
        ptrs = [[ctx.make_all([t.data_ptr() for t in send], [t.data_ptr() for t in recv]) for send, recv in rows] for rows in sets]
        rng = np.random.default_rng(R)
        for it in range(60):
            s = int(rng.integers(3))
            ids = [int(i) for i in rng.permutation(len(kinds))[:int(rng.integers(1, 5))]]
            for i in ids:
                if rng.random() < 0.25:                                    # rank by rank, in another order
                    send, recv = sets[s][i]
                    for r in rng.permutation(R):
                        while ctx.submit(int(r), i, send[r].data_ptr(), recv[r].data_ptr()) == dfx.ERR_SQ_FULL:
                            pass
                else:
                    assert ctx.submit_all(i, ptrs[s][i]) == dfx.OK
            assert ctx.wait_all(20.0) == dfx.OK, (it, ids)
        for s in range(3):                                                 # every set once more, one call at a time
            for i in range(len(kinds)):
                for t in sets[s][i][1]:
                    t.fill_(-7)
        torch.cuda.synchronize()
        for s in range(3):
            for i in range(len(kinds)):
                assert ctx.submit_all(i, ptrs[s][i]) == dfx.OK and ctx.wait_all(20.0) == dfx.OK
        assert ctx.stop() == dfx.OK
    finally:
        assert ctx.finalize() == dfx.OK
    for n, (recv, out) in enumerate(want):
        for r in range(R):
            assert torch.equal(recv[r], out[r]), (n // len(kinds), n % len(kinds), r)


@pytest.mark.parametrize("max_channels,count", [(63, 70000), (64, 70000), (65, 70000), (128, 150001)])
def test_more_channels_than_a_wave_has_lanes(max_channels, count):
    """The last wait looks at a counter per channel, a lane each, and at the SQ where a lane is left for it: below, at and beyond 64 channels."""
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    R = 2
    g = torch.Generator(device="cuda").manual_seed(max_channels)
    send = [torch.randint(-1000, 1000, (count,), generator=g, device="cuda", dtype=torch.int32) for _ in range(R)]
    recv = [torch.full((count,), -7, device="cuda", dtype=torch.int32) for _ in range(R)]
    torch.cuda.synchronize()
    ctx = dfx.Context(R, gh.make_config(max_channels=max_channels, chan_min_bytes=1024))
    try:
        ctx.prepare(0, dfx.ALLREDUCE, count, dfx.I32)
        assert ctx.coll_info(0)["nchan"] == max_channels
        ptrs = ctx.make_all([t.data_ptr() for t in send], [t.data_ptr() for t in recv])
        for it in range(30):
            if it % 3 == 2:
                for r in range(R):
                    assert ctx.submit(r, 0, send[r].data_ptr(), recv[r].data_ptr()) == dfx.OK
            else:
                assert ctx.submit_all(0, ptrs) == dfx.OK
            assert ctx.wait_all(20.0) == dfx.OK
        assert ctx.stop() == dfx.OK
    finally:
        assert ctx.finalize() == dfx.OK
    want = send[0] + send[1]
    for r in range(R):
        assert torch.equal(recv[r], want), r


@pytest.mark.parametrize("R,n", [(2, 700), (8, 300)])
def test_a_table_is_for_its_own_invocation(R, n):
    """A collective of several channels, submitted on all ranks at once ahead of a run of others that a daemon finds in the SQ when it
    comes: its one job goes to the movers at the head of the fetch.  It is submitted anew, with other buffers, as soon as it is
    complete, while workgroups may still fetch the run that its table came with (int32: exact)."""
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    count, small = 8 * 4 * 512 + 5, 260
    g = torch.Generator(device="cuda").manual_seed(R)
    def sends(m):
        return [torch.randint(-1000, 1000, (m,), generator=g, device="cuda", dtype=torch.int32) for _ in range(R)]
    def recvs(m):
        return [torch.full((m,), -7, device="cuda", dtype=torch.int32) for _ in range(R)]
    sets = [(sends(count), recvs(count)) for _ in range(4)]
    others = (sends(small), [torch.full((n, small), -7, device="cuda", dtype=torch.int32) for _ in range(R)])
    torch.cuda.synchronize()
    ctx = dfx.Context(R, gh.make_config(max_channels=4, chan_spread=0, chan_min_bytes=1024))
    try:
        ctx.prepare(0, dfx.ALLREDUCE, count, dfx.I32)
        assert ctx.coll_info(0) == dict(ctx.coll_info(0), nchan=4, rounds=1, nprim=2)
        for i in range(n):
            ctx.prepare(1 + i, dfx.ALLREDUCE, small, dfx.I32)
        ptrs = [ctx.make_all([t.data_ptr() for t in s], [t.data_ptr() for t in d]) for s, d in sets]
        bursts = [ctx.make_burst(list(range(1, n + 1)), [others[0][r].data_ptr()] * n, [others[1][r][i].data_ptr() for i in range(n)]) for r in range(R)]
        for it in range(6):
            for s, d in sets:
                for t in d:
                    t.fill_(-7)
            torch.cuda.synchronize()
            assert ctx.submit_all(0, ptrs[0]) == dfx.OK
            for r in range(R):
                assert ctx.submit_burst(r, bursts[r]) == n
            for k in range(1, 4):
                for r in range(R):
                    assert ctx.wait(r, 0, 20.0) == dfx.OK
                assert ctx.submit_all(0, ptrs[k]) == dfx.OK
            assert ctx.wait_all(20.0) == dfx.OK
            assert ctx.stop() == dfx.OK                              # (the next run is found by a daemon that comes)
            for k, (s, d) in enumerate(sets):
                total = torch.stack(s).sum(0).to(torch.int32)
                assert all(torch.equal(t, total) for t in d), (it, k)
    finally:
        assert ctx.finalize() == dfx.OK
    total = torch.stack(others[0]).sum(0).to(torch.int32)
    for r in range(R):
        assert bool((others[1][r] == total).all()), r
