"""Collectives in fold steps that all ranks sweep together (messages from 128 MiB of inputs, or 256 MiB of outputs, on): a rank
moves rows of every region, each in that region's own order of combination.  Just above the limit and ragged -- regions that end
inside a row and inside 16 bytes, a last region shorter than the others -- for every kind and the rank
counts that sweep (4 and 8 with movers of their own; 16, 32 and 64 without, which sweep where they combine), with one job per share and with several, with dealt rows
(priority ordering), few channels, and the daemon stopped between jobs.  Bit-exact against the oracle (same order of
combination, one rounding per hop: no tolerance), guard zones around the recv buffers."""
import numpy as np
import pytest

import workload_inputs as wi
from oracle import ring_data as rd

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _specs(kind, R):
    """Two collectives: the shortest that sweeps, and one with a ragged end (all-reduce: in its last region, which is shorter than the others)."""
    least = max((256 if kind in (wi.AG, wi.BC) else 128) * MIB // R, R * (128 if kind == wi.RS else 40) << 10)      # (regions of so much)
    dtypes = (wi.BF16, wi.F32) if kind != wi.RD else (wi.I32, wi.F16)
    out = []
    for i, dtype in enumerate(dtypes):
        eb = wi.ELEM_BYTES[dtype]
        n = least // eb
        if kind in (wi.AG, wi.RS):
            n = n // R + i * (2048 + 3 * 16) // eb                     # blocks are 16-byte multiples
        elif i:
            n = R * (n // R + (2048 + 32) // eb) - 32 // eb - 3 if kind == wi.AR else n + 2048 // eb + 5
        op = (wi.SUM, wi.MAX)[i] if kind in (wi.AR, wi.RS, wi.RD) else wi.SUM
        out.append(wi.CollSpec(i, kind, dtype, n, R - 2 if kind in (wi.BC, wi.RD) else 0, op))
    return out


def _run(w, knobs, stop_between=False, passes=2):
    from paper_2303_06324_amd import harness as gh
    import paper_2303_06324_amd as dfx
    dw = gh.DeviceWorkload(w)
    cfg = gh.make_config(**{**dict(max_channels=min(32, 256 // w.R)), **knobs})
    for c in w.colls:
        swept = w.R <= 8 or c.kind not in (wi.AG, wi.BC)
        assert ("sweep" in dfx.plan_route(w.R, c.kind, c.count, c.dtype, c.root, cfg)) == swept, c
    ctx = dfx.Context(w.R, cfg)
    try:
        gh.prepare_all(ctx, w)
        for ci in range(len(w.colls)):
            assert ctx.coll_info(ci)["nprim"] == 2, ctx.coll_info(ci)
        for _ in range(passes):                          # row counters of both parities
            dw.reset_recv()
            gh.submit_round_robin(ctx, dw)
            if stop_between:
                assert ctx.stop() == dfx.OK
            assert ctx.wait_all(30.0) == dfx.OK
        assert ctx.stop() == dfx.OK
    finally:
        ctx.finalize()
    for ci, c in enumerate(w.colls):
        want, got = rd.run_closed_form(c.kind, dw.send_host[ci], c.dtype, c.root, c.op), dw.results(ci)
        for r in range(w.R):
            if c.kind == wi.RD and r != c.root:
                assert np.all(got[r].view(np.uint8) == 0xA5), (ci, r)
            else:
                assert np.array_equal(got[r].view(np.uint8), want[r].view(np.uint8)), (ci, c, r)
    dw.check_untouched()


@pytest.mark.parametrize("kind,R", [(k, R) for R in (4, 8, 16) for k in (wi.AR, wi.AG, wi.RS, wi.BC, wi.RD)] + [(k, 32) for k in (wi.AR, wi.RS, wi.RD)] +
                         [(wi.AR, 64), (wi.RS, 64)])
def test_sweeps_at_the_edges(kind, R):
    specs = _specs(kind, R)
    if kind == wi.AG and R != 8:
        specs = specs[:1]                                # (R results of 256 MiB in all: one is enough)
    _run(wi.Workload(f"sweep_{kind}_{R}", R, specs, [list(range(len(specs)))] * R, seed=kind * 10 + R, cfg=95), {})


@pytest.mark.parametrize("knobs", [dict(fold_max_bytes=1 << 20), dict(order_policy=1, fold_max_bytes=1 << 20), dict(max_channels=3),
                                   dict(scan_min=0, spin_init=1, spin_min=1, spin_max=1, spin_boost=1, fold_max_bytes=1 << 20)],
                         ids=["several_jobs", "dealt_rows", "few_channels", "give_up_at_once"])
@pytest.mark.parametrize("kind", [wi.AR, wi.RS, wi.BC])
def test_sweeps_in_jobs(kind, knobs):
    _run(wi.Workload(f"sweep_jobs_{kind}", 8, _specs(kind, 8), [[0, 1], [1, 0]] * 4, seed=kind, cfg=96), knobs)


def test_daemon_stopped_between_jobs_of_a_sweep():
    _run(wi.Workload("sweep_stop", 8, _specs(wi.AR, 8), [[0, 1]] * 8, seed=3, cfg=97), dict(max_channels=1, fold_max_bytes=1 << 20), stop_between=True)


def test_sweep_in_place():
    """recvbuf == sendbuf: every byte is read by the wave that then overwrites it, and by no other."""
    from paper_2303_06324_amd import harness as gh
    import paper_2303_06324_amd as dfx
    import torch
    R, c = 8, _specs(wi.AR, 8)[1]
    w = wi.Workload("sweep_in_place", R, [c], [[0]] * R, seed=9, cfg=98)
    host = wi.all_sends(w, 0)
    want = rd.run_closed_form(wi.AR, host, c.dtype, 0, c.op)[0]
    ctx = dfx.Context(R, gh.make_config())
    try:
        ctx.prepare(0, wi.AR, c.count, c.dtype, c.op)
        buf = [torch.from_numpy(h.view(np.uint8).copy()).cuda() for h in host]
        torch.cuda.synchronize()
        p = [t.data_ptr() for t in buf]
        assert ctx.submit_all(0, ctx.make_all(p, p)) == dfx.OK and ctx.wait_all(20.0) == dfx.OK
        for r in range(R):
            assert np.array_equal(buf[r].cpu().numpy(), want.view(np.uint8)), r
    finally:
        ctx.finalize()
