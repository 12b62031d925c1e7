"""A collective that runs again and again while another one, which not all ranks have submitted, stays in the queue with it: two entries, a
pass without a readiness scan.  The stuck one is given up in every pass (nothing of it has progressed: no save); the last wait of the
other, behind the job that it has just posted, has nothing left to be given up for and goes on within its threshold, so that its context is
saved in hardly any invocation.  int32: exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,count,how", [(8, 2048, "at_once"), (8, 2048, "rank_by_rank"), (4, 262147, "at_once"), (2, 4096, "rank_by_rank")])
def test_the_last_wait_beside_a_stuck_one(R, count, how):
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    g = torch.Generator(device="cuda").manual_seed(R)
    send = [torch.randint(-1000, 1000, (count,), generator=g, device="cuda", dtype=torch.int32) for _ in range(R)]
    recv = [[torch.full((count,), -7, device="cuda", dtype=torch.int32) for _ in range(R)] for _ in range(2)]
    torch.cuda.synchronize()
    n = 200
    ctx = dfx.Context(R, gh.make_config(max_channels=4, chan_spread=0, spin_init=256, spin_max=1024, quit_idle_us=20000))
    try:
        for i in range(2):
            ctx.prepare(i, dfx.ALLREDUCE, count, dfx.I32)
        p = ctx.make_all([t.data_ptr() for t in send], [t.data_ptr() for t in recv[0]])
        for r in range(R - 1):                               # stuck: the last rank's is not there
            assert ctx.submit(r, 1, send[r].data_ptr(), recv[1][r].data_ptr()) == dfx.OK
        for _ in range(n):
            if how == "at_once":
                assert ctx.submit_all(0, p) == dfx.OK
            else:
                for r in range(R):
                    assert ctx.submit(r, 0, send[r].data_ptr(), recv[0][r].data_ptr()) == dfx.OK
            for r in range(R):
                assert ctx.wait(r, 0, 10.0) == dfx.OK
        assert ctx.submit(R - 1, 1, send[R - 1].data_ptr(), recv[1][R - 1].data_ptr()) == dfx.OK
        assert ctx.wait_all(10.0) == dfx.OK
        assert ctx.stop() == dfx.OK
        st = [ctx.stats(r) for r in range(R)]
    finally:
        ctx.finalize()
    saves = [s["ctx_saves"] for s in st[:R - 1]]             # (of the ranks whose queues hold the stuck one)
    assert all(k <= n // 4 for k in saves), saves
    total = torch.stack(send).sum(0).to(torch.int32)
    for row in recv:
        assert all(torch.equal(t, total) for t in row)
