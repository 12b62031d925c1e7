"""The kernel behind the entry point that allocates nothing, for collectives in fold steps: one launch, a workgroup per stretch of
rows.  Regions that end 16 bytes before, at and behind a row, a workgroup's rows and two workgroups' rows, elements behind the
last whole 16 bytes, ranks without a chunk, nothing at all; for every kind and rank counts with movers of their own (2, 4, 8) and
without (3, 16); one message of each kind long enough for a sweep; and a captured call replayed with eager work in between.
Bit-exact against the oracle (same order of combination, one rounding per hop: no tolerance), guard zones around the recv buffers."""
import numpy as np
import pytest

import workload_inputs as wi
from oracle import ring_data as rd

pytestmark = pytest.mark.gpu

ROW, MIB = 2048, 1 << 20


def _check(w, dw, ci=0):
    c = w.colls[ci]
    want, got = rd.run_closed_form(c.kind, dw.send_host[ci], c.dtype, c.root, c.op), dw.results(ci)
    for r in range(w.R):
        if c.kind == wi.RD and r != c.root:
            assert np.all(got[r].view(np.uint8) == 0xA5), (c, r)
        else:
            assert np.array_equal(got[r].view(np.uint8), want[r].view(np.uint8)), (c, r)


def _call(dw, w, ci, status, stream=None):
    import paper_2303_06324_amd as dfx
    c = w.colls[ci]
    rc = dfx.collective_noalloc(w.R, c.kind, c.count, c.dtype, c.op, c.root, [t.data_ptr() for t in dw.send[ci]],
                                [t.data_ptr() for t in dw.recv[ci]], status.data_ptr() if status is not None else 0, stream)
    assert rc == dfx.OK, dfx.strerror(rc)


@pytest.mark.parametrize("R", [2, 3, 4, 8, 16])
@pytest.mark.parametrize("kind", [wi.AR, wi.AG, wi.RS, wi.BC, wi.RD])
def test_regions_at_the_edges_of_rows_and_workgroups(kind, R):
    import torch
    from paper_2303_06324_amd import harness as gh
    spans = [0, 16, ROW - 16, ROW + 16, 4 * ROW, 8 * ROW - 16, 8 * ROW + 16, 16 * ROW + 48, 67 * ROW + 32, 300 * ROW + 16]
    colls = []
    for i, nbytes in enumerate(spans):
        dtype = (wi.F32, wi.BF16, wi.F16, wi.I32)[i % 4]
        eb = wi.ELEM_BYTES[dtype]
        op = (wi.SUM, wi.MAX, wi.SUM, wi.MIN)[i % 4] if kind in (wi.AR, wi.RS, wi.RD) else wi.SUM
        n = nbytes // eb
        counts = [n] if kind in (wi.AG, wi.RS) else [max(R * n - d, 0) for d in (0, 3)] + [n // R + 1]
        colls += [wi.CollSpec(len(colls) + k, kind, dtype, c, R - 1 if kind in (wi.BC, wi.RD) else 0, op) for k, c in enumerate(counts)]
    w = wi.Workload(f"once_{kind}_{R}", R, colls, [list(range(len(colls)))] * R, seed=kind * 10 + R, cfg=99)
    dw = gh.DeviceWorkload(w)
    status = torch.full((len(colls),), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for _ in range(2):
        for ci in range(len(colls)):
            _call(dw, w, ci, status[ci:])
    torch.cuda.synchronize()
    assert torch.all(status == 0)
    for ci in range(len(colls)):
        _check(w, dw, ci)
    dw.check_untouched()


@pytest.mark.parametrize("kind,R", [(k, R) for R in (4, 8, 16) for k in (wi.AR, wi.AG, wi.RS, wi.BC, wi.RD)] + [(wi.AR, 32), (wi.RS, 32)])
def test_messages_that_are_swept(kind, R):
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    n = max((256 if kind in (wi.AG, wi.BC) else 128) * MIB // R, 16 * MIB if R > 16 else 0) // 2
    n = n // R + 56 if kind in (wi.AG, wi.RS) else n + 1027
    w = wi.Workload(f"once_sweep_{kind}_{R}", R, [wi.CollSpec(0, kind, wi.BF16, n, R - 2 if kind in (wi.BC, wi.RD) else 0)], [[0]] * R, seed=R, cfg=100)
    route = dfx.plan_route(R, kind, n, wi.BF16, w.colls[0].root, gh.make_config(max_channels=min(32, 256 // R)))
    assert ("sweep_noalloc" in route) == (R <= 8 or kind not in (wi.AG, wi.BC)), route
    dw = gh.DeviceWorkload(w)
    torch.cuda.synchronize()
    _call(dw, w, 0, None)
    torch.cuda.synchronize()
    _check(w, dw)
    dw.check_untouched()


def test_captured_and_replayed():
    """Two kernel nodes, the collective's and the outcome's: every replay reports one."""
    import torch
    from paper_2303_06324_amd import harness as gh
    R, n = 8, 40008
    w = wi.Workload("once_graph", R, [wi.CollSpec(0, wi.AR, wi.I32, n)], [[0]] * R, seed=1, cfg=101)
    dw = gh.DeviceWorkload(w)
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    _call(dw, w, 0, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _call(dw, w, 0, status, torch.cuda.current_stream().cuda_stream)
    send = [t.clone() for t in dw.send[0]]
    for it in range(5):
        status.fill_(-1)
        for r in range(R):
            dw.send[0][r].copy_(send[r])
            dw.send[0][r].view(torch.int32).add_(it)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert int(status.item()) == 0, it
        want = torch.stack([t.view(torch.int32) for t in dw.send[0]]).sum(0).to(torch.int32)
        for r in range(R):
            got = torch.from_numpy(dw.results(0)[r].view(np.int32).copy())
            assert torch.equal(got[:n], want.cpu()[:n]), (it, r)
    for r in range(R):
        dw.send[0][r].copy_(send[r])
    dw.check_untouched()


def test_calls_that_overlapped_leave_the_next_ones_their_outcome():
    """Calls of different sizes on two streams at once (buffers and status words of their own), then one at a time, more of them than
    there are counters: every one of these reports its outcome and nobody else's."""
    import torch
    from paper_2303_06324_amd import harness as gh
    R = 8
    counts = [2051, MIB + 9, 300007, 4 * MIB + 3]
    w = wi.Workload("once_overlap", R, [wi.CollSpec(i, wi.AR, wi.I32, c) for i, c in enumerate(counts)], [list(range(4))] * R, seed=7, cfg=102)
    dw = gh.DeviceWorkload(w)
    streams = [torch.cuda.Stream() for _ in range(2)]
    status = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for it in range(60):
        for k, st in enumerate(streams):                     # stream 0: the first and third, stream 1: the others
            ci = k + 2 * (it % 2)
            _call(dw, w, ci, status[ci:], st.cuda_stream)
    torch.cuda.synchronize()
    dw.reset_recv()
    for it in range(1100):
        ci = it // 50 % 2 if it % 50 == 49 else 2 * (it % 2)
        status.fill_(-1)
        _call(dw, w, ci, status[ci:])
        assert status.tolist() == [0 if i == ci else -1 for i in range(4)], (it, ci)
    for ci in range(3):
        _check(w, dw, ci)
    dw.check_untouched()
