"""All-gathers and reduce-scatters whose blocks are no 16-byte multiples, in fold steps: blocks begin anywhere, rows on 16 bytes (long
ones on lines) of the recv buffers, and the loads are what is not aligned.  Blocks of one element, around a row, around the length
from which rows begin on lines, with drawn rows, in several jobs and swept; every element type; rank counts with movers of their own
(2, 4, 8) and without (3, 16); submitted on all ranks at once, in disordered bursts (where short ones go in gangs) and without a context.
Bit-exact against the oracle (same order of combination, one rounding per hop: no tolerance), guard zones around the recv buffers."""
import numpy as np
import pytest

import workload_inputs as wi
from oracle import ring_data as rd

pytestmark = pytest.mark.gpu

ROW, KIB, MIB = 2048, 1 << 10, 1 << 20
DTYPES = (wi.F32, wi.BF16, wi.F16, wi.I32)


def _colls(kind, R, spans, first=0):
    out = []
    for i, nbytes in enumerate(spans):
        dtype = DTYPES[(i + first) % 4]
        eb = wi.ELEM_BYTES[dtype]
        op = (wi.SUM, wi.MAX, wi.PROD, wi.MIN, wi.SUM)[i % 5] if kind == wi.RS else wi.SUM
        n = nbytes // eb
        if n * eb % 16 == 0:
            n += 1 + i % (16 // eb - 1)
        out.append(wi.CollSpec(len(out), kind, dtype, n, 0, op))
    return out


def _check(w, dw):
    for ci, c in enumerate(w.colls):
        want, got = rd.run_closed_form(c.kind, dw.send_host[ci], c.dtype, c.root, c.op), dw.results(ci)
        for r in range(w.R):
            assert np.array_equal(got[r].view(np.uint8), want[r].view(np.uint8)), (c, r)


def _all_ways(w, **knobs):
    import torch
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    n = len(w.colls)
    dw = gh.DeviceWorkload(w)
    status = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for ci, c in enumerate(w.colls):
        rc = dfx.collective_noalloc(w.R, c.kind, c.count, c.dtype, c.op, 0, [t.data_ptr() for t in dw.send[ci]], [t.data_ptr() for t in dw.recv[ci]],
                                    status[ci:].data_ptr())
        assert rc == dfx.OK, (c, dfx.strerror(rc))
    torch.cuda.synchronize()
    assert torch.all(status == 0)
    _check(w, dw)
    dw.reset_recv()
    ctx = dfx.Context(w.R, gh.make_config(**{**dict(max_channels=min(32, 256 // w.R)), **knobs}))
    try:
        gh.prepare_all(ctx, w)
        assert all(ctx.coll_info(ci)["nprim"] == 2 for ci in range(n))
        for ci in range(n):
            assert ctx.submit_all(ci, ctx.make_all([t.data_ptr() for t in dw.send[ci]], [t.data_ptr() for t in dw.recv[ci]])) == dfx.OK
            assert ctx.wait_all(20.0) == dfx.OK, w.colls[ci]
        assert ctx.stop() == dfx.OK
        _check(w, dw)
        dw.reset_recv()
        gh.submit_bursts(ctx, dw)
        assert ctx.wait_all(20.0) == dfx.OK
        assert ctx.stop() == dfx.OK
    finally:
        ctx.finalize()
    _check(w, dw)
    dw.check_untouched()


def _workload(name, R, colls, seed):
    g = np.random.default_rng(seed)
    return wi.Workload(name, R, colls, [list(map(int, g.permutation(len(colls)))) for _ in range(R)], seed=seed, cfg=120)


@pytest.mark.parametrize("R", [2, 3, 4, 8, 16])
def test_reducescatter(R):
    spans = [2, 14, 18, ROW - 6, ROW + 2, 5 * ROW + 10, 8 * ROW - 2, 16 * KIB + 6, 31 * KIB + 4, 33 * KIB + 2, 70 * KIB + 12, 300 * ROW + 2, MIB + 14]
    for first in range(2):
        _all_ways(_workload(f"odd_rs_{R}", R, _colls(wi.RS, R, spans, 2 * first + 1), seed=R + first), **(dict(max_channels=3) if first else {}))


@pytest.mark.parametrize("R", [2, 3, 4, 8, 16])
def test_allgather(R):
    _all_ways(_workload(f"odd_ag_{R}", R, _colls(wi.AG, R, [MIB, MIB + 34, MIB + 130, MIB + ROW * 3 + 6], R), seed=20 + R))


@pytest.mark.parametrize("kind,R,dtype", [(wi.RS, 8, wi.BF16), (wi.RS, 4, wi.F32), (wi.AG, 8, wi.F16), (wi.AG, 4, wi.I32), (wi.RS, 16, wi.F16)])
def test_swept(kind, R, dtype):
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    n = (256 if kind == wi.AG else 128) * MIB // R // R // wi.ELEM_BYTES[dtype] + 3
    assert "sweep" in dfx.plan_route(R, kind, n, dtype, 0, gh.make_config(max_channels=min(32, 256 // R)))
    _all_ways(_workload(f"odd_sweep_{kind}_{R}", R, [wi.CollSpec(0, kind, dtype, n)], seed=40 + R))


@pytest.mark.parametrize("kind", [wi.AG, wi.RS])
def test_several_jobs(kind):
    """Above fold_max_bytes: jobs of at most so many rows, each with the bytes before and behind its rows."""
    _all_ways(_workload(f"odd_jobs_{kind}", 5, _colls(kind, 5, [MIB + 2, 2 * MIB + 6, 3 * MIB + 14], 1), seed=60 + kind), fold_max_bytes=1 << 16, direct_min_bytes=0, max_channels=2)
