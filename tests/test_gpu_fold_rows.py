"""Steps with data of collectives in fold steps at the edges of their rows: regions that end 16 bytes before, at and
behind a row, all waves' first rows and the length from which rows are drawn instead of dealt, regions with elements behind the
last whole 16 bytes, ranks without a chunk, for every kind and for rank counts with a data mover of their own (2, 4, 8) and
without (3, 5); twice each, so that the row counters of both parities are used, and the first parity's again.
Bit-exact against the oracle (same order of combination, one rounding per hop: no tolerance); nothing outside the recv
buffers is written (guard zones)."""
import pytest

import workload_inputs as wi
from oracle import ring_data as rd

pytestmark = pytest.mark.gpu

ROW = 2048                      # bytes a mover wave takes at a time (R = 2, 4 and copies: a multiple of it)


@pytest.mark.parametrize("R", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("kind", [wi.AR, wi.AG, wi.RS, wi.BC, wi.RD])
def test_regions_at_the_edges_of_rows(kind, R):
    from paper_2303_06324_amd import harness as gh
    import numpy as np
    spans = [16, ROW - 16, ROW, ROW + 16, 4 * ROW + 16, 12 * ROW, 48 * ROW - 16, 48 * ROW, 97 * ROW + 48, 192 * ROW - 16, 192 * ROW + 16, 301 * ROW + 32]
    colls = []
    for i, nbytes in enumerate(spans):
        dtype = (wi.F32, wi.BF16, wi.F16, wi.I32)[i % 4]
        eb = wi.ELEM_BYTES[dtype]
        op = (wi.SUM, wi.MAX, wi.SUM)[i % 3] if kind in (wi.AR, wi.RS, wi.RD) else wi.SUM
        if kind in (wi.AG, wi.RS):
            counts = [nbytes // eb]                                        # blocks are 16-byte multiples
        elif kind == wi.BC:
            counts = [R * nbytes // eb, R * nbytes // eb - 1]              # one stretch, the r-th part of it
        else:
            counts = [R * nbytes // eb, R * nbytes // eb - 3, nbytes // eb + 1]   # whole chunks; a ragged last one; ranks without any
        colls += [wi.CollSpec(len(colls) + k, kind, dtype, max(c, 1), R - 1 if kind in (wi.BC, wi.RD) else 0, op) for k, c in enumerate(counts)]
    order = list(range(len(colls)))
    w = wi.Workload(f"rows_{kind}_{R}", R, colls, [order] * R, seed=kind * 10 + R, cfg=91)
    import paper_2303_06324_amd as dfx
    dw = gh.DeviceWorkload(w)
    ctx = dfx.Context(R, gh.make_config(max_channels=3))
    try:
        gh.prepare_all(ctx, w)
        for _ in range(3):
            dw.reset_recv()
            gh.submit_round_robin(ctx, dw)
            assert ctx.wait_all(30.0) == dfx.OK
        assert ctx.stop() == dfx.OK
        dw.check_untouched()
    finally:
        ctx.finalize()
    for ci, c in enumerate(colls):
        want, got = rd.run_closed_form(c.kind, dw.send_host[ci], c.dtype, c.root, c.op), dw.results(ci)
        for r in range(R):
            if kind == wi.RD and r != c.root:
                assert np.all(got[r].view(np.uint8) == 0xA5), (ci, r)
            else:
                assert np.array_equal(got[r].view(np.uint8), want[r].view(np.uint8)), (ci, c, r)
