"""Collectives in fold steps whose share takes several jobs: what they hold of the connector pool."""
import pytest

pytestmark = pytest.mark.gpu


def test_long_collectives_hold_no_slots():
    """With the default pool of 4 GiB: a slot-based all-reduce of 256 MiB holds 256 MiB of it, one in fold steps its flag
    lines (36 KiB), however many are prepared."""
    import paper_2303_06324_amd as dfx
    from paper_2303_06324_amd import harness as gh
    R, n = 8, (256 << 20) // 4
    ctx = dfx.Context(R, gh.make_config())
    try:
        for i in range(60):
            kind = (dfx.ALLREDUCE, dfx.ALLGATHER, dfx.REDUCESCATTER, dfx.REDUCE)[i % 4] if i >= 40 else dfx.ALLREDUCE
            ctx.prepare(i, kind, n // R if kind in (dfx.ALLGATHER, dfx.REDUCESCATTER) else n, dfx.F32)
            assert ctx.coll_info(i)["nprim"] == 2
    finally:
        assert ctx.finalize() == dfx.OK
    ctx = dfx.Context(R, gh.make_config(pool_bytes=1 << 20))           # 28 blocks of 36 864 bytes in 1 MiB
    try:
        with pytest.raises(dfx.DfxError) as e:
            for i in range(30):
                ctx.prepare(i, dfx.ALLREDUCE, n, dfx.F32)
        assert e.value.status == dfx.ERR_NO_RESOURCES and i == 28
    finally:
        assert ctx.finalize() == dfx.OK
