"""What a program has this library do, as cases that can be timed and checked.

A case is one pass through the public entry points of the Python binding:

  call "one"      one collective on every virtual rank: Context.submit_all, then Context.wait_all, inside a daemon that
                  stays resident from pass to pass (the library's defaults: it leaves after 2 ms without work)
  call "burst"    many collectives, every rank in an order of its own: one Context.submit_burst per rank, then wait_all
  call "noalloc"  one collective through collective_noalloc, which only enqueues work on the current stream

kind, dtype and op are the library's own numbers; count is dfx_prepare's: elements per rank (all-reduce, broadcast,
reduce), each rank's contribution (all-gather) or result (reduce-scatter).

Every result is the fold of the ranks' inputs in the order that the library documents, with one rounding per hop, or a
copy: the outputs of two correct builds are the same bits, so the tolerance is "exact" everywhere.
"""
import math
import random
import weakref

import torch

import paper_2303_06324_amd as dfx

KIB, MIB = 1 << 10, 1 << 20
AR, AG, RS, BC, RD = dfx.ALLREDUCE, dfx.ALLGATHER, dfx.REDUCESCATTER, dfx.BROADCAST, dfx.REDUCE
F32, BF16, F16, I32 = dfx.F32, dfx.BF16, dfx.F16, dfx.I32
SUM, PROD, MAX, MIN = dfx.SUM, dfx.PROD, dfx.MAX, dfx.MIN
TORCH = {F32: torch.float32, BF16: torch.bfloat16, F16: torch.float16, I32: torch.int32}
EB = {F32: 4, BF16: 2, F16: 2, I32: 4}
PAD = 256      # bytes that every collective's place in a flat buffer is aligned to


def _one(name, kind, dtype, count, ranks=8, op=SUM, root=0, call="one"):
    c = {"call": call, "kind": kind, "dtype": dtype, "op": op, "root": root, "ranks": ranks, "count": count}
    return dict(c, name=name) if name else c


def _burst(name, what, n, lo, hi, dtype, ranks=8, priority=False, spec=0):
    """n collectives of lo .. hi bytes (largest per-rank buffer, sizes spread over their logarithm); what: "allreduce" (all
    of one element type) or "mixed" (all-reduce, all-gather, reduce-scatter and broadcast of fp32, fp16 and int32);
    spec: the seed of their sizes and of the ranks' orders, which belong to the program and not to its data."""
    c = {"call": "burst", "what": what, "n": n, "lo": lo, "hi": hi, "dtype": dtype, "ranks": ranks, "priority": priority,
         "spec": spec}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest all-reduce of the size sweep: nothing but latency, from the call to the completion
        _one("allreduce 8 KiB fp32", AR, F32, 2 * KIB),
        # activations or a small gradient of odd length
        _one("allreduce 1 MiB bf16 odd", AR, BF16, 524309),
        # one gradient bucket of the usual 25 MiB
        _one("allreduce 25 MiB bf16", AR, BF16, 25 * MIB // 2),
        # the benchmark's headline: the largest message of the sweep, a ring through the connectors by default
        _one("allreduce 256 MiB fp32", AR, F32, 64 * MIB),
        # sharded weights gathered before a layer
        _one("allgather 32 MiB bf16", AG, BF16, 2 * MIB),
        # sharded gradients; the block is no power of two
        _one("reducescatter 128 MiB fp32", RS, F32, 4 * MIB + 12),
        # initial weights handed out
        _one("broadcast 100 MiB bf16", BC, BF16, 50 * MIB, root=5),
        # a metric or a norm's largest value collected on one of four ranks
        _one("reduce 4 MiB fp32 max", RD, F32, MIB, ranks=4, op=MAX, root=3),
        # sixteen gradient buckets, every rank in its own order
        _burst("16 buckets 25 MiB bf16", "allreduce", 16, 25 * MIB, 25 * MIB, BF16, spec=3),
        # a thousand small all-reduces, every rank in its own order
        _burst("1024 small fp32", "allreduce", 1024, 4 * KIB, 64 * KIB, F32, spec=5),
        # mixed kinds, element types and sizes, every rank in its own order
        _burst("64 mixed", "mixed", 64, 4 * KIB, 64 * MIB, F32, spec=4),
        # one collective inside a captured or allocation-free serving loop
        _one("noalloc allreduce 64 KiB fp32", AR, F32, 16 * KIB, call="noalloc"),
    ]


def _spread(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    if rng.random() < 0.25:
        ranks = rng.choice((2, 4, 8, 8))
        if rng.random() < 0.5:
            n, lo, hi, what = _spread(rng, 64, 1024), 4 * KIB, 64 * KIB, "allreduce"
        elif rng.random() < 0.5:
            n, what = rng.randint(4, 16), "allreduce"
            lo = hi = _spread(rng, MIB, 25 * MIB)
        else:
            n, lo, hi, what = rng.randint(16, 64), 4 * KIB, 32 * MIB, "mixed"
        return _burst("", what, n, lo, hi, rng.choice((F32, BF16)), ranks=ranks, priority=rng.random() < 0.2,
                      spec=rng.randrange(1 << 20))
    call = "one" if rng.random() < 0.8 else "noalloc"
    kind = rng.choice((AR, AR, AR, AG, RS, BC, RD))
    dtype = rng.choice((F32, F32, BF16, BF16, F16, I32))
    op = rng.choice((SUM, SUM, SUM, PROD, MAX, MIN)) if kind in (AR, RS, RD) else SUM
    ranks = rng.choice((2, 4, 8, 8, 8, 8, 16))
    nbytes = _spread(rng, 4 * KIB, 256 * MIB if call == "one" else 64 * MIB)
    if ranks > 8:
        nbytes //= 2
    count = max(1, nbytes // EB[dtype] // (ranks if kind in (AG, RS) else 1))
    how = rng.random()      # whole multiples of 16 elements, as model dimensions give them, or any number
    if how < 0.5:
        count = max(16, count // 16 * 16)
    root = rng.randrange(ranks) if kind in (BC, RD) else 0
    return _one("", kind, dtype, count, ranks=ranks, op=op, root=root, call=call)


# --------------------------------------------------------------------------------------------
# what a pass consists of: collectives with places in one flat send and one flat recv buffer per rank and element type
# --------------------------------------------------------------------------------------------
def _specs(case):
    """[(kind, dtype, op, root, count)] of the case, in id order."""
    if case["call"] != "burst":
        return [(case["kind"], case["dtype"], case["op"], case["root"], case["count"])]
    rng, R, out = random.Random(case["spec"]), case["ranks"], []
    for _ in range(case["n"]):
        nbytes = case["lo"] if case["lo"] == case["hi"] else max(R * 16, _spread(rng, case["lo"], case["hi"]) // (R * 16) * (R * 16))
        kind, dtype, root = AR, case["dtype"], 0
        if case["what"] == "mixed":
            kind, dtype = rng.choice((AR, AG, RS, BC)), rng.choice((F32, F16, I32))
            root = rng.randrange(R) if kind == BC else 0
        count = nbytes // EB[dtype] // (R if kind in (AG, RS) else 1)
        out.append((kind, dtype, SUM, root, count))
    return out


def _orders(case):
    out = []
    for r in range(case["ranks"]):
        o = list(range(case["n"]))
        random.Random(case["spec"] * 1000 + r + 1).shuffle(o)
        out.append(o)
    return out


def _places(case):
    """Per collective: its spec, and where its send and its recv buffer begin (elements of the flat buffers) and how long
    they are; and the length of the flat buffers per element type."""
    R, out, total = case["ranks"], [], {}
    for kind, dtype, op, root, count in _specs(case):
        t = total.setdefault(dtype, [0, 0])
        ns, nr = count * (R if kind == RS else 1), count * (R if kind == AG else 1)
        out.append((kind, dtype, op, root, count, t[0], ns, t[1], nr))
        step = PAD // EB[dtype]
        t[0] += -(-ns // step) * step
        t[1] += -(-nr // step) * step
    return out, total


def _values(case, seed, total):
    """{dtype: the ranks' flat send buffers}: N(0, 1) (16-bit types in a burst or a sum: gradients, sigma 1e-2), whole
    numbers up to 2^20 for int32."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    out = {}
    for dtype, (n, _) in sorted(total.items()):
        rows = []
        for _ in range(case["ranks"]):
            if dtype == I32:
                t = torch.randint(-(1 << 20), (1 << 20) + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
            else:
                t = torch.randn(n, generator=g, device="cuda")
                if dtype == BF16 and case.get("op", SUM) == SUM:
                    t.mul_(1e-2)
                t = t.to(TORCH[dtype])
            rows.append(t)
        out[dtype] = rows
    return out


class _Program:
    """The context of one case with its collectives prepared: what a program sets up once and keeps while it has buffers
    to work on."""

    def __init__(self, case, places):
        cfg = dfx.config_default()
        cfg.max_channels = min(32, 256 // case["ranks"])      # the grid has to be resident at once: one workgroup per CU
        cfg.order_policy = 1 if case.get("priority") else 0
        self.ctx = dfx.Context(case["ranks"], cfg)
        for i, (kind, dtype, op, root, count, *_) in enumerate(places):
            self.ctx.prepare(i, kind, count, dtype, op, root, priority=i if case.get("priority") else 0)


_programs = weakref.WeakValueDictionary()      # one program per case: all of its states submit to the same context


def _key(case):
    return tuple(sorted((k, v) for k, v in case.items() if k != "name"))


def prepare(case, seed):
    places, total = _places(case)
    R = case["ranks"]
    send = _values(case, seed, total)
    recv = {d: [torch.zeros(n, dtype=TORCH[d], device="cuda") for _ in range(R)] for d, (_, n) in sorted(total.items())}
    if case["call"] == "burst":
        out = recv
    else:
        kind, dtype, _, root, _, _, _, _, nr = places[0]
        out = [recv[dtype][r][:nr] for r in range(R) if kind != RD or r == root]      # a reduce writes the root's buffer only
    s = {"case": dict(case), "send": send, "recv": recv, "out": out}
    if case["call"] == "noalloc":
        kind, dtype, *_ = places[0]
        s["status"] = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        s["ptrs"] = [t.data_ptr() for t in send[dtype]], [t.data_ptr() for t in recv[dtype]]
        torch.cuda.synchronize()
        return s
    program = _programs.get(_key(case))
    if program is None:
        program = _programs[_key(case)] = _Program(case, places)
    s["program"] = program
    if case["call"] == "one":
        dtype = places[0][1]
        s["ptrs"] = program.ctx.make_all([t.data_ptr() for t in send[dtype]], [t.data_ptr() for t in recv[dtype]])
    else:
        s["bursts"] = []
        for r, order in enumerate(_orders(case)):
            sp = [send[places[i][1]][r].data_ptr() + places[i][5] * EB[places[i][1]] for i in order]
            rp = [recv[places[i][1]][r].data_ptr() + places[i][7] * EB[places[i][1]] for i in order]
            s["bursts"].append(program.ctx.make_burst(order, sp, rp))
    torch.cuda.synchronize()      # the daemon is on a stream of its own: the inputs are there before anything is submitted
    return s


def run(state):
    case = state["case"]
    if case["call"] == "noalloc":
        rc = dfx.collective_noalloc(case["ranks"], case["kind"], case["count"], case["dtype"], case["op"], case["root"],
                                    *state["ptrs"], state["status"].data_ptr(), torch.cuda.current_stream().cuda_stream)
        if rc != dfx.OK:
            raise dfx.DfxError(rc, "collective_noalloc")
        return state["out"], state["status"]
    ctx = state["program"].ctx
    if case["call"] == "one":
        rc = ctx.submit_all(0, state["ptrs"])
        if rc != dfx.OK:
            raise dfx.DfxError(rc, "submit_all")
    else:
        for r, burst in enumerate(state["bursts"]):
            n = ctx.submit_burst(r, burst)
            if n != burst[0]:
                raise dfx.DfxError(n if n < 0 else dfx.ERR_TIMEOUT, "submit_burst")
    rc = ctx.wait_all(30.0)
    if rc != dfx.OK:
        raise dfx.DfxError(rc, "wait_all")
    return state["out"]


def work(case):
    """Every send buffer read once (a broadcast: the root's), every recv buffer written once (a reduce: the root's); one
    operation per element and hop."""
    R, nbytes, flops = case["ranks"], 0, 0
    for kind, dtype, op, root, count, _, ns, _, nr in _places(case)[0]:
        nbytes += (ns * (1 if kind == BC else R) + nr * (1 if kind == RD else R)) * EB[dtype]
        flops += 0 if kind in (AG, BC) else (R - 1) * ns
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    return "exact"


def exact(case, seed):
    places, total = _places(case)
    send, R = _values(case, seed, total), case["ranks"]
    wide = {d: torch.int64 if d == I32 else torch.float64 for d in total}
    fold = {SUM: torch.add, PROD: torch.mul, MAX: torch.maximum, MIN: torch.minimum}
    out = {d: [torch.zeros(n, dtype=wide[d], device="cuda") for _ in range(R)] for d, (_, n) in total.items()}
    for kind, dtype, op, root, count, s0, ns, r0, nr in places:
        x = [t[s0:s0 + ns].to(wide[dtype]) for t in send[dtype]]
        if kind == AG:
            y = torch.cat(x)
        elif kind == BC:
            y = x[root]
        else:
            y = x[0].clone()
            for t in x[1:]:
                fold[op](y, t, out=y)
        for r in range(R):
            out[dtype][r][r0:r0 + nr] = y[r * count:(r + 1) * count] if kind == RS else y
    if case["call"] == "burst":
        return out
    kind, dtype, _, root, _, _, _, _, nr = places[0]
    got = [out[dtype][r][:nr] for r in range(R) if kind != RD or r == root]
    return (got, None) if case["call"] == "noalloc" else got
