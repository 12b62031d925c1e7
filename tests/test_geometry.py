"""The kernel's index arithmetic, walked on the CPU (dfx_check_geometry compiles the same functions as the
kernel: workgroup -> (rank, channel), connector addresses, primitive sequences, slice geometry, the order of
slices and primitives).  No GPU: for every workgroup of the grid, every address the kernel would form is
checked against the buffers and the connector block, the writes to each recv buffer must tile it exactly,
and both ends of every connector must agree.

It covers the workload of the run that once ended in a GPU memory fault (every kind at 256 MiB and
all-reduces of 8 KiB - 64 MiB, under a third workgroup labelling that has since been taken out of the
kernel): that labelling, wg_map 2 here, is checked along with the two the kernel offers."""
import itertools

import pytest

import paper_2303_06324_amd as dfx

KINDS = [dfx.ALLREDUCE, dfx.ALLGATHER, dfx.REDUCESCATTER, dfx.BROADCAST, dfx.REDUCE]


def _cfg(**kw):
    cfg = dfx.config_default()
    for k, v in kw.items():
        setattr(cfg, k, v)
    return cfg


@pytest.mark.parametrize("wg_map", [0, 1, 2])
def test_workload_of_the_faulting_run_under_every_map(wg_map):
    R, n = 8, (256 << 20) // 4
    cases = [(dfx.ALLREDUCE, n), (dfx.ALLGATHER, n // R), (dfx.REDUCESCATTER, n // R), (dfx.BROADCAST, n), (dfx.REDUCE, n),
             (dfx.ALLREDUCE, 2048), (dfx.ALLREDUCE, 1 << 18), (dfx.ALLREDUCE, 1 << 21), (dfx.ALLREDUCE, 1 << 24),
             (dfx.BROADCAST, 1 << 21)]
    for i, (kind, count) in enumerate(cases):                       # coll ids 0 .. 9 as in that run
        assert dfx.check_geometry(R, kind, count, dfx.F32, root=3, coll_id=i, wg_map=wg_map) == "", (kind, count)
        assert dfx.check_geometry(R, kind, count, dfx.F32, root=3, coll_id=i, wg_map=wg_map, cfg=_cfg(fold_max_bytes=0)) == "", (kind, count)
    for p in range(13, 27):                                         # the all-reduce size sweep
        assert dfx.check_geometry(R, dfx.ALLREDUCE, (1 << p) // 4, dfx.F32, wg_map=wg_map) == ""
    n3 = 25 * (1 << 20) // 2                                        # the sixteen bf16 buckets
    for i in range(16):
        assert dfx.check_geometry(R, dfx.ALLREDUCE, n3, dfx.BF16, coll_id=i, wg_map=wg_map) == ""


@pytest.mark.parametrize("kind", KINDS)
def test_ragged_counts_rank_counts_and_dtypes(kind):
    for R, count, dtype in itertools.product([1, 2, 3, 5, 8, 16], [0, 1, 7, 4099, 100003, (1 << 20) + 24], [dfx.F32, dfx.BF16]):
        cfg = _cfg(max_channels=min(32, 256 // R))
        for root in {0, R - 1}:
            for wg_map in (0, 1):
                msg = dfx.check_geometry(R, kind, count, dtype, root=root, coll_id=count % 7, wg_map=wg_map, cfg=cfg)
                assert msg == "", (kind, R, count, dtype, root, wg_map, msg)


@pytest.mark.parametrize("knobs", [dict(direct=0), dict(direct_min_bytes=0), dict(window=1), dict(window=4, nslots=8), dict(nslots=2),
                                   dict(slot_bytes=4096, max_channels=4), dict(chan_spread=0), dict(chan_min_bytes=1 << 20),
                                   dict(direct_min_bytes=0, slot_bytes=16 << 10, max_channels=2, window=1),
                                   dict(fold_slice_bytes=4096), dict(fold_slice_bytes=48, max_channels=2), dict(order_policy=1, fold_slice_bytes=32 << 10),
                                   dict(fold_slice_bytes=1 << 16, fold_max_bytes=1 << 30)])
def test_scheduler_knobs(knobs):
    cfg = _cfg(**knobs)
    for kind in KINDS:
        for count in (8, 30008, (3 << 20) + 8, 1 << 24):
            for cid in (0, 5, 1023):
                msg = dfx.check_geometry(8, kind, count, dfx.F16, op=dfx.MAX, root=5, coll_id=cid, cfg=cfg)
                assert msg == "", (knobs, kind, count, cid, msg)


@pytest.mark.parametrize("R", [2, 3, 4, 5, 8, 16])
@pytest.mark.parametrize("kind", KINDS)
def test_drawn_rows_are_taken_once_in_bounded_jobs(kind, R):
    """From the shortest region whose rows are drawn to shares of several jobs, with edges in between: the check lets the
    waves of a rank get on in three orders and holds every job to twice an equal part."""
    for C, long in itertools.product([1, 3, 256 // R if R > 8 else 32], [False, True]):
        cfg = _cfg(max_channels=C, **(dict(fold_max_bytes=4096, direct_min_bytes=0) if long else {}))
        for rows in (16, 17, 31, 64, 65, 100, 301):                         # per wave and channel, rows of 2 KiB
            for extra in (0, 16, 2048, 2064):
                region = rows * 2048 * 4 * C // 4 + extra
                n = region // 4 if kind in (dfx.ALLGATHER, dfx.REDUCESCATTER) else R * region // 4 - 3
                msg = dfx.check_geometry(R, kind, n, dfx.F32, root=R - 1, cfg=cfg)
                assert msg == "", (kind, R, C, long, rows, extra, msg)
    for mib in (32, 63, 64, 256, 1024):                                     # the defaults
        n = (mib << 20) // 4 // (R if kind in (dfx.ALLGATHER, dfx.REDUCESCATTER) else 1) // 4 * 4
        msg = dfx.check_geometry(R, kind, n, dfx.F32, root=1, cfg=_cfg(max_channels=min(32, 256 // R)))
        assert msg == "", (kind, R, mib, msg)


SWEEP_LEAST = {dfx.ALLREDUCE: 128 << 20, dfx.REDUCESCATTER: 128 << 20, dfx.REDUCE: 128 << 20, dfx.ALLGATHER: 256 << 20, dfx.BROADCAST: 256 << 20}   # all ranks' inputs (outputs)


@pytest.mark.parametrize("R", [2, 3, 4, 5, 6, 8, 12, 16, 24, 32, 40, 48, 56, 63, 64])
@pytest.mark.parametrize("kind", KINDS)
def test_which_messages_are_swept(kind, R):
    """Both sides of every line of the rule: powers of two from four ranks on (copies: up to eight), from so many bytes in all on, with
    regions of 40 KiB (results for one rank: 128 KiB) at least; in the allocation-free call on more than 16 ranks from 16 MiB per rank on."""
    blocks, one = kind in (dfx.ALLGATHER, dfx.REDUCESCATTER), kind in (dfx.REDUCESCATTER, dfx.REDUCE)
    cfg = _cfg(max_channels=min(32, 256 // R))
    ranks_ok = R in ((4, 8) if kind in (dfx.ALLGATHER, dfx.BROADCAST) else (4, 8, 16, 32, 64)) and not (kind == dfx.REDUCE and R > 63)
    for total in (SWEEP_LEAST[kind] * 3 // 4, SWEEP_LEAST[kind], 3 << 27, 1 << 30, 3 << 30):
        n = -(-total // R // 4 // (R if blocks else 1) // 4) * 4              # elements, at least `total` bytes over all ranks
        nbytes = n * 4 * (R if blocks else 1)
        region = n * 4 if blocks or kind in (dfx.REDUCE, dfx.BROADCAST) else -(-n // R // 4) * 16
        want = ranks_ok and R * nbytes >= SWEEP_LEAST[kind] and region >= ((128 if one else 40) << 10)
        route = dfx.plan_route(R, kind, n, dfx.F32, root=R - 1, cfg=cfg)
        assert ("sweep" in route) == want, (kind, R, total, route)
        assert ("sweep_noalloc" in route) == (want and (R <= 16 or nbytes >= 16 << 20)), (kind, R, total, route)
        assert dfx.check_geometry(R, kind, n, dfx.F32, root=R - 1, cfg=cfg) == "", (kind, R, total)
        assert dfx.check_geometry(R, kind, n + 4, dfx.BF16, root=0, cfg=_cfg(max_channels=min(32, 256 // R), order_policy=1, fold_max_bytes=1 << 20)) == "", (kind, R, total)


@pytest.mark.parametrize("knobs", [dict(), dict(fold_max_bytes=0), dict(direct=0)], ids=["defaults", "ring_with_direct_steps", "through_slots"])
def test_a_large_offset_case(knobs):
    """5 GiB + a ragged tail per rank on two ranks: byte offsets beyond 2^32, hundreds of slices per channel."""
    assert dfx.check_geometry(2, dfx.ALLREDUCE, (5 << 30) // 4 + 12345, dfx.I32, cfg=_cfg(**knobs)) == ""


def test_more_jobs_than_the_walk_counts():
    """128 GiB on two ranks with one channel: 2^32 slices of 16 bytes do not fit the walk's 32-bit count, so it stays a ring."""
    cfg = _cfg(max_channels=1, fold_slice_bytes=16, slot_bytes=1 << 30)
    assert dfx.check_geometry(2, dfx.ALLREDUCE, (128 << 30) // 4, dfx.F32, cfg=cfg) == ""


def test_it_refuses_what_it_cannot_check():
    assert dfx.check_geometry(8, dfx.BROADCAST, 1024, dfx.F32, root=9) != ""
    assert dfx.check_geometry(8, dfx.ALLREDUCE, 1024, dfx.F32, wg_map=3) != ""


@pytest.mark.parametrize("R", [2, 3, 4, 8, 16, 33, 64])
@pytest.mark.parametrize("kind", [dfx.ALLGATHER, dfx.REDUCESCATTER])
def test_blocks_that_are_no_16_byte_multiples(kind, R):
    """Which of them run in fold steps (reduce-scatters; all-gathers from 1 MiB per block on), and that their rows and the bytes before
    and behind them tile the recv buffers, one channel to many, one job to several, dealt, drawn and swept."""
    cmax = min(32, 256 // R)
    for knobs in (dict(), dict(max_channels=1), dict(max_channels=3, fold_max_bytes=1 << 16, direct_min_bytes=0), dict(order_policy=1), dict(fold_slice_bytes=4096)):
        cfg = _cfg(**{**dict(max_channels=cmax), **knobs})
        for dtype, eb in ((dfx.F32, 4), (dfx.F16, 2)):
            for nbytes in (eb, 16 + eb, 2048 - eb, 2048 + eb, 32768 - eb, 33000, 100002, 524286, (1 << 20) - eb, (1 << 20) + eb, (5 << 20) + 3 * eb):
                n = nbytes // eb
                if n * eb % 16 == 0:
                    n += 1
                route = dfx.plan_route(R, kind, n, dtype, 0, cfg)
                assert ("fold" in route) == (kind == dfx.REDUCESCATTER or n * eb >= 1 << 20), (knobs, n, route)
                assert dfx.check_geometry(R, kind, n, dtype, op=dfx.MAX if kind == dfx.REDUCESCATTER else dfx.SUM, cfg=cfg) == "", (knobs, dtype, n)
    assert "fold" not in dfx.plan_route(R, kind, (1 << 20) + 1, dfx.F32, 0, _cfg(fold_max_bytes=0, max_channels=cmax))
