// Index arithmetic of the daemon kernel: which workgroup serves which (rank, channel), the primitive
// sequence of every collective kind, the connector addresses of an invocation, where a slice lies in
// the buffers, and the order in which a workgroup walks through slices and primitives.
//
// Pure functions of their arguments, compiled for the device (the kernel) and for the host (the
// library's geometry self-check, which walks the same arithmetic without a GPU).
#ifndef DFX_GEOMETRY_H
#define DFX_GEOMETRY_H

#include <stddef.h>
#include <stdint.h>

#include "dfx_internal.h"

#if defined(__HIPCC__)
#define DFX_HD __host__ __device__ __forceinline__
#else
#define DFX_HD inline
#endif

constexpr int KIND_AR = 0, KIND_AG = 1, KIND_RS = 2, KIND_BC = 3, KIND_RD = 4;
constexpr int DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2, DT_I32 = 3;

// Workgroup -> (rank, channel).  Workgroups go to the XCDs round-robin (workgroup w runs on XCD w mod 8).
//   map 0: workgroup = channel * R + rank: with R = 8 a vrank per XCD
//   map 1: workgroup = rank * cmax + channel: a channel's whole ring per XCD
struct WgPlace { uint32_t rank, ch; };
DFX_HD WgPlace wg_place(uint32_t wg_map, uint32_t wg, uint32_t R, uint32_t cmax) {
  WgPlace w;
  if (wg_map == 0) { w.rank = wg % R; w.ch = wg / R; }
  else { w.rank = wg / cmax; w.ch = wg % cmax; }
  return w;
}

// Channel of collective coll_id that the workgroup on channel `ch` of its rank serves (>= nchan: none).
// A collective with fewer channels than the grid has per rank starts at workgroup (coll_id * nchan) mod
// cmax, so that many small collectives spread over the rank's workgroups instead of queueing on the
// first ones; every rank derives the same start from the id, which keeps both ends of a connector on
// the same channel.
// The start is worked out where the collective is planned and travels in its entries (DfxStatic::start): a workgroup
// that reads an entry only subtracts.
DFX_HD uint32_t start_channel(bool spread, uint32_t cmax, uint32_t coll_id, uint32_t nchan) {
  return spread && nchan < cmax ? (coll_id * nchan) % cmax : 0u;
}
DFX_HD uint32_t serving_channel(uint32_t ch, uint32_t cmax, uint32_t start) { return ch >= start ? ch - start : ch + cmax - start; }

// primitive descriptor for (kind, position p in the sequence); the ring-chunk index travels in
// the dynamic context and is stepped by next_cidx, so nothing here divides
struct Prim {
  bool recv, send;         // uses recv / send connector (send: waits for a free slot and fills it)
  bool from_send, to_recv; // touches the send buffer / recv buffer
  // Direct gather steps of an all-reduce: every rank's buffers lie in the same HBM, so the copy
  // steps need no second copy through a FIFO slot.  notify: the result goes to the own recv buffer
  // with device-coherent stores and the send connector's counter is raised without a slot being
  // filled; din: the input is read from the previous rank's recv buffer instead of a slot;
  // drain: no data, the wait ends when the next rank has consumed everything notified so far
  // (the recv buffer is the caller's again once the completion is posted).
  bool notify, din, drain;
  bool din_send;   // the input is the previous rank's SEND buffer (first reduce step of a direct all-reduce / reduce-scatter)
  // Fold steps (see make_fold_prim): fold = 1 the step with data, 3 the last wait, which moves nothing; 0 = neither.
  // fwait: the channel's shared counter that says whether the step can run (0 published, 1 done).
  uint8_t fold, fwait;
};

// Collectives in fold steps.  Every rank's buffers lie in the same HBM, so the dependent hops of a ring or
// a chain (a few microseconds each, whatever the size) can be replaced by steps that wait on all ranks at once:
//   step with data: when every rank has published this invocation's buffers, a rank does its part of the work
//                reading other ranks' send buffers where they lie and writing the result straight into the recv
//                buffers it belongs to; reductions combine in the ring's (the chain's) own order -- the same
//                association as the hops would give, hence the same bits;
//   last wait:   no data; when every rank has done its part, every byte of the own recv buffer has arrived, nobody
//                reads this rank's send buffer any more, and the completion may be posted.  One workgroup per rank, channel
//                0's, waits for all channels; the others are through when their last job is posted.
// What rank r reads and writes in its step with data:
//   all-reduce:      chunk r out of all R send buffers, x[r+1] (op) ... (op) x[r]     -> chunk r of all R recv buffers
//   reduce-scatter:  block r out of all R send buffers, in the same order             -> the own recv buffer
//   reduce:          chunk r out of all R send buffers, x[root+1] (op) ... (op) x[root] -> chunk r of the root's recv buffer
//   all-gather:      the own send buffer, once                                        -> block r of all R recv buffers
//   broadcast:       the r-th of R parts of the root's send buffer                    -> the same of all R recv buffers
// So every input is read once and every output written once, whatever the kind.  (All-gather and broadcast hand
// their data out instead of every rank fetching all of it: one read per byte instead of R.)
// Each step is a bounded wait followed by the data, like any primitive: nothing is touched before the wait has
// succeeded, so a collective stuck in either of them is preempted like any other.
constexpr uint32_t DFX_FOLD_NPRIM = 2u;
DFX_HD Prim make_fold_prim(uint32_t p) {
  Prim q;
  q.recv = q.send = q.notify = q.din = q.drain = q.din_send = q.from_send = q.to_recv = false;   // (no connectors, no pointers of its own)
  q.fold = p == 0 ? 1 : 3;
  q.fwait = p == 0 ? 0 : 1;
  return q;
}

// The tables of a step with data.  Entry k is about rank fold_peer(.., k); the entries begin behind this rank (behind
// the root: reduce, broadcast), which makes their order the order of combination and the last entry, R - 1, this rank
// (the root).  A kind that combines reads every entry's send buffer, a kind that copies only the last entry's;
// a kind with results for everybody writes every entry's recv buffer, the others only the last entry's.
DFX_HD uint32_t fold_peer(int kind, uint32_t R, uint32_t rank, uint32_t root, uint32_t k) {
  const uint32_t r = ((kind == KIND_RD || kind == KIND_BC) ? root : rank) + 1u + k;
  return r >= R ? r - R : r;
}
DFX_HD bool fold_copies(int kind) { return kind == KIND_AG || kind == KIND_BC; }
DFX_HD bool fold_to_all(int kind) { return kind != KIND_RS && kind != KIND_RD; }

// The part of a rank -- its region: a chunk, a block, its R-th of a broadcast -- is worked through in rows: a mover wave
// takes 64 lanes x 16 bytes x as many vectors as keep about sixteen loads in flight per lane, out of every source, and
// goes on to another row.  Row t begins at fold_head + t * fold_row_bytes.  The first rows go to the waves of the region's
// workgroups in turn (workgroup by workgroup, so that a short region spreads over them).
//   dealt rows: the next ones in turn as well;
//   drawn rows: whoever is through draws the next from a counter.
// Either way the waves advance side by side and sweep one compact stretch of every buffer: with one contiguous part per
// workgroup (256 x 16 streams megabytes apart) the same loop took 85-87 us for 24 MiB per rank and 22.5 us for 8 MiB,
// side by side 78 and 20 us (fp32, R = 8).  Drawing them pays where a wave has several rows: the memory system
// does not serve workgroups alike, and the workgroups of one rank were through with equal parts after 15 to 50 us
// (all-gather of 32 MiB); drawn, after 46 to 53.  Host to host: 25 MiB bf16 bucket 107 -> 101 us, sixteen of them 1405 -> 1315,
// all-reduce of 256 MiB 876 -> 857.
// A job is a span of the region with its rows dealt (a slice; all of it where there is one slice), or at most so and so
// many drawn rows per wave.  The limit holds for every job, so that a workgroup that is alone at a region -- the others of
// its rank are still at another collective -- moves no more than twice its equal part before it looks at its queue again;
// all jobs together may take more rows than there are, so that whoever is through early can go on.
constexpr uint32_t DFX_FOLD_WAVES = DFX_MOVERS / 64 / DFX_MOVER_GROUPS;      // mover waves that share a job
DFX_HD uint32_t fold_row_bytes(bool copies, uint32_t R) { return 1024u * (R == 2 ? 8u : copies || R == 4 ? 4u : 2u); }

// A rank's region in elements: where it begins in the message and how long it is.  chunk: what one rank has, in elements.
DFX_HD uint64_t fold_chunk_elems(int kind, uint64_t count, uint64_t block, uint32_t R, uint32_t eb) {
  if (kind == KIND_AR || (kind == KIND_RD && block != count)) return block;      // (planned as chunks)
  if (kind == KIND_RD || kind == KIND_BC) return ((count + R - 1) / R + 16 / eb - 1) / (16 / eb) * (16 / eb);
  return count;                                                                 // (a block per rank)
}

// Bytes at the front of a span that come before its first row: rows begin on 128-byte lines of the recv
// buffers.  A region begins at any multiple of 16 bytes (the chunk of an all-reduce, the block of an all-gather), and rows
// counted from there end inside a line, of which two waves then write a part each, straight to memory.  us per call, fp32,
// regions at odd multiples of 16 bytes, rows from the region's start -> from the line (= regions on lines): all-gather of 64 MiB
// 192 -> 132 (R = 8), 158 -> 96 (R = 6), all-reduce of 25 MiB 98 -> 92, broadcast of 110 MiB 306 -> 205 (R = 8).
// Short spans keep their rows at the front: the round trip for the bytes before would cost what whole lines gain (64 KiB,
// R = 8: 0.4 us; a wave has four rows from 32 KiB per workgroup on).  Blocks that are no 16-byte multiples begin anywhere; their rows
// begin on 16 bytes of the recv buffers all the same, so that it is the loads that are not aligned and never the stores.
DFX_HD uint32_t fold_head(uint64_t dst, uint32_t bytes, uint32_t nchan) {
  const uint32_t head = (uint32_t)(0u - dst) & (bytes >= nchan << 15 ? 127u : 15u);
  return head < bytes ? head : bytes;
}

// Sweeps.  Long messages leave the caches behind, and then it matters that few places of the memory are open at once: with a
// region per rank the ranks move along R x 2R stretches of the buffers.  In a sweep all ranks go through the regions one
// after the other, 2R stretches in all: the rows of all regions are numbered through, and of every R x W of them (W: mover
// waves of a rank) a rank takes W in a row, so that a rank's workgroups -- an XCD's, or those of a few whole ones -- stay side
// by side.  Which rank moves a row has nothing to do with whose region it lies in; every region keeps its order of combination.
// The rows' loads carry the non-temporal hint: nothing of a long message is read again.  The hint alone gave 804 -> 772 us
// for an all-reduce of 256 MiB fp32 (R = 8), the sweep with it 746; reduce-scatter of 128 MiB 268 -> 262 and 221 (blocks on lines).
// Row t of the message is row t mod n of region t / n, where n = ceil(longest region / row).
DFX_HD uint32_t sweep_row_bytes(bool copies, uint32_t R) { return 1024u * (copies || R == 4 ? 4u : 2u); }
// Regions: a chunk or block per rank (all-reduce, reduce-scatter, all-gather); a broadcast or reduce, whose parts are all
// combined or copied alike, is one.
DFX_HD uint32_t sweep_regions(int kind, uint32_t R) { return kind == KIND_RD || kind == KIND_BC ? 1u : R; }
struct FoldRegion { uint64_t src, dst; uint32_t len, head, end; };   // offsets in the buffers, length; its rows lie in [head, end)
DFX_HD FoldRegion sweep_region(int kind, uint64_t longest, uint64_t total, uint32_t c) {
  FoldRegion o;
  const uint64_t at = (uint64_t)c * longest;
  o.len = (uint32_t)(at >= total ? 0u : total - at < longest ? total - at : longest);
  o.src = kind == KIND_AG ? 0u : at;
  o.dst = kind == KIND_RS ? 0u : at;
  o.head = fold_head(o.dst, o.len, o.len >= 128u ? 0u : 1u);      // (rows on lines of the recv buffers; of the shortest, on 16 bytes)
  o.end = o.head + ((o.len - o.head) & ~15u);
  return o;
}
// Entry of a rank's tables (fold_peer) at which region c's order of combination begins; a region with one destination goes to
// the last one from there.
DFX_HD uint32_t sweep_first(uint32_t nreg, uint32_t c, uint32_t rank, uint32_t R) { return nreg == 1 ? 0u : c >= rank ? c - rank : c + R - rank; }
// The n-th row of a rank, counted over all regions (base: rank x W; skip: W x (R - 1)).
DFX_HD uint32_t sweep_row(uint32_t n, uint32_t waves, uint32_t base, uint32_t skip) { return base + n + n / waves * skip; }

// As a plain kernel (DfxFoldOnce) a rank has `groups` workgroups, and a workgroup's rows lie together: its waves take them in turn.
constexpr uint32_t DFX_ONCE_WAVES = DFX_ONCE_THREADS / 64;
struct OnceWave { uint32_t row; bool head, tail; };   // first row (the next ones DFX_ONCE_WAVES apart); takes the bytes before or behind the region's rows
DFX_HD OnceWave once_wave(uint32_t group, uint32_t groups, uint32_t rows_per_wave, uint32_t wave) {
  OnceWave w;
  w.row = group * rows_per_wave * DFX_ONCE_WAVES + wave;
  w.head = group + 1 == groups && wave + 1 == DFX_ONCE_WAVES;
  w.tail = group == 0 && wave == 0;
  return w;
}

// The entry (SQE) of a collective in fold steps for one rank, from its plan in elements: everything about the rank's
// part that does not depend on the channel, in bytes, so that the workgroups that read the entry multiply nothing.
//   count       length of the rank's region
//   block_elems where the region begins in the send buffers it is read from
//   part_elems  where it begins in the recv buffers it is written to
//   slice_elems span of one slice, all channels together (at most 1 GiB); rows are drawn: the longest region, all of it
//   slot_bytes  rows are drawn: rows per wave and job at most (0: rows are dealt)
//   share       one channel's part of a slice or job
// and where all ranks sweep the message together (sweep_region):
//   count       the longest region
//   block_elems the whole message: what a region beyond it is clipped to
//   slice_elems rows per wave and job; slot_bytes the same where rows are drawn, else 0
DFX_HD void fold_entry(DfxStatic& e, uint32_t R, uint32_t rank) {
  const int kind = e.kind;
  const uint32_t eb = (e.dtype == DT_F32 || e.dtype == DT_I32) ? 4u : 2u;
  const uint64_t count = e.count, chunk = fold_chunk_elems(kind, count, e.block_elems, R, eb);
  e.share = e.slice_elems * eb;
  if (e.flags & DFX_SQE_SWEEP) {
    e.slice_elems = e.slot_bytes;
    if (!(e.flags & DFX_SQE_DRAWN)) e.slot_bytes = 0;
    e.count = (sweep_regions(kind, R) == 1 ? count : chunk) * eb;
    e.block_elems = (kind == KIND_AG || kind == KIND_RS ? R * count : count) * eb;
    e.part_elems = 0;
    return;
  }
  uint64_t start = 0, len = count;
  if (kind == KIND_AR || kind == KIND_RD || kind == KIND_BC) {
    start = (uint64_t)rank * chunk;
    len = start >= count ? 0 : (count - start < chunk ? count - start : chunk);
  }
  e.count = len * eb;
  e.block_elems = (start + (kind == KIND_RS ? (uint64_t)rank * count : 0u)) * eb;
  e.part_elems = (start + (kind == KIND_AG ? (uint64_t)rank * count : 0u)) * eb;
  if (e.flags & DFX_SQE_DRAWN) e.slice_elems = (uint32_t)(chunk * eb);      // (slot_bytes: the plan's row limit)
  else {
    e.slice_elems = (uint32_t)(e.nchan * (uint64_t)e.share);
    e.slot_bytes = 0;
  }
}

struct FoldGeom { uint64_t src, dst; uint32_t bytes; };   // byte offsets of the job's span in the buffers, its length
DFX_HD FoldGeom fold_geometry(uint64_t len, uint64_t src, uint64_t dst, uint32_t span, bool drawn, uint32_t g) {
  FoldGeom o;
  const uint64_t at = drawn ? 0u : (uint64_t)g * span, lo = at < len ? at : len, n = len - lo;
  o.src = src + lo; o.dst = dst + lo;
  o.bytes = n < span ? (uint32_t)n : span;
  return o;
}
DFX_HD FoldGeom fold_geometry(const DfxCooked& S, uint32_t g) {
  return fold_geometry(S.count, S.block_elems, S.part_elems, S.slice_elems, (S.bc_pos & DFX_CTX_DRAWN) != 0, g);
}

// Where a fold collective's lines are, from a workgroup's own line: the line of rank r on the same channel,
// and the channel's shared line.
DFX_HD uint64_t fold_line(uint64_t own_line, uint32_t rank, uint32_t r, uint32_t nchan) {
  return own_line + ((uint64_t)r - (uint64_t)rank) * nchan * DFX_FLAG_STRIDE;
}
// the row counter of the region of `rank`, for invocation seq, from the channel's line of rank 0
DFX_HD uint64_t fold_draw_word(uint64_t line0, uint32_t rank, uint32_t vch, uint32_t nchan, uint32_t seq) {
  return line0 + (uint64_t)rank * nchan * DFX_FLAG_STRIDE - (uint64_t)vch * DFX_FLAG_STRIDE + DFX_FOLD_DRAW + 8u * (seq & 1u);
}
DFX_HD uint64_t fold_shared_line(uint64_t own_line, uint32_t rank, uint32_t R, uint32_t nchan) {
  return own_line + ((uint64_t)R - (uint64_t)rank) * nchan * DFX_FLAG_STRIDE;
}

DFX_HD Prim make_prim(int kind, uint32_t R, uint32_t bc_pos, uint32_t p, bool direct) {
  Prim q;
  q.notify = q.din = q.drain = q.din_send = false;
  q.fold = q.fwait = 0;
  if (R == 1) { q.recv = q.send = false; q.from_send = q.to_recv = true; return q; }   // copy
  if (kind == KIND_AR && direct) {
    const uint32_t last_reduce = R - 1;
    q.recv = p > 0; q.send = p < last_reduce; q.from_send = p <= last_reduce; q.to_recv = p >= last_reduce;
    // The opening send moves nothing either: the rank only notifies, and the next rank's first
    // reduce step reads the chunk out of this rank's send buffer (which the caller leaves alone
    // until the completion, and the drain keeps the completion behind that read).
    if (p == 0) { q.send = false; q.from_send = false; q.notify = true; }             // notify only
    else if (p == 1) q.din_send = true;                                               // recv-reduce-send / -copy from the neighbour's send buffer
    if (p == last_reduce) q.notify = true;                                            // recv-reduce-copy, notify
    else if (p > last_reduce && p < 2u * R - 2) { q.din = true; q.notify = true; }    // direct recv-copy, notify
    else if (p == 2u * R - 2) q.din = true;                                           // direct recv-copy
    else if (p == 2u * R - 1) { q.recv = false; q.to_recv = false; q.drain = true; }  // drain
    return q;
  }
  if (kind == KIND_RS && direct) {
    // the reduce phase of the direct all-reduce: notify only, then the first reduce step reads the
    // neighbour's send buffer; the drain keeps the completion behind that read
    q.recv = p > 0 && p < R; q.send = p > 0 && p + 1 < R; q.from_send = q.recv; q.to_recv = p == R - 1;
    if (p == 0) q.notify = true;
    else if (p == 1) q.din_send = true;
    else if (p == R) q.drain = true;
    return q;
  }
  if (kind == KIND_AR || kind == KIND_RS) {
    const uint32_t last_reduce = R - 1;
    if (p == 0) { q.recv = false; q.send = true; q.from_send = true; q.to_recv = false; }                         // send
    else if (p < last_reduce) { q.recv = true; q.send = true; q.from_send = true; q.to_recv = false; }           // recv-reduce-send
    else if (p == last_reduce) { q.recv = true; q.send = (kind == KIND_AR); q.from_send = true; q.to_recv = true; }  // recv-reduce-copy(-send)
    else if (p < 2u * R - 2) { q.recv = true; q.send = true; q.from_send = false; q.to_recv = true; }            // recv-copy-send
    else { q.recv = true; q.send = false; q.from_send = false; q.to_recv = true; }                               // recv-copy
  } else if (kind == KIND_AG && direct) {
    // every block is written once: the own one by a copy that notifies, the others by direct copies
    q.send = false;
    if (p == 0) { q.recv = false; q.from_send = true; q.to_recv = true; q.notify = true; }                        // copy, notify
    else if (p < R) { q.recv = true; q.from_send = false; q.to_recv = true; q.din = true; q.notify = p < R - 1; } // direct recv-copy (, notify)
    else { q.recv = false; q.from_send = false; q.to_recv = false; q.drain = true; }                              // drain
  } else if (kind == KIND_AG) {
    if (p == 0) { q.recv = false; q.send = true; q.from_send = true; q.to_recv = true; }                          // copy-send
    else if (p < R - 1) { q.recv = true; q.send = true; q.from_send = false; q.to_recv = true; }
    else { q.recv = true; q.send = false; q.from_send = false; q.to_recv = true; }
  } else if (kind == KIND_RD) {  // reduce chain root+1 -> root+2 -> ... -> root (bc_pos: 0 first, 1 middle, 2 the root, 3 second)
    if (bc_pos == 0) { q.recv = false; q.send = true; q.from_send = true; q.to_recv = false; }                    // send
    else if (bc_pos == 2) { q.recv = true; q.send = false; q.from_send = true; q.to_recv = true; }               // recv-reduce-copy
    else { q.recv = true; q.send = true; q.from_send = true; q.to_recv = false; }                                 // recv-reduce-send
    if (direct) {
      // the first rank only notifies and the second one reads the slice out of its send buffer
      if (bc_pos == 0) { q.send = false; q.from_send = false; q.notify = true; }
      else if (bc_pos == 3 || R == 2) q.din_send = true;
    }
  } else if (direct) {  // broadcast chain with direct steps: every rank writes its recv buffer only
    q.send = false; q.to_recv = true;
    q.recv = bc_pos != 0; q.din = bc_pos != 0; q.from_send = bc_pos == 0; q.notify = bc_pos != 2;
  } else {  // broadcast chain root -> root+1 -> ... -> root-1
    if (bc_pos == 0) { q.recv = false; q.send = true; q.from_send = true; q.to_recv = true; }
    else if (bc_pos == 2) { q.recv = true; q.send = false; q.from_send = false; q.to_recv = true; }
    else { q.recv = true; q.send = true; q.from_send = false; q.to_recv = true; }
  }
  return q;
}

// A chain (broadcast, reduce) has one primitive per slice, so its drain cannot be a step of the
// per-slice sequence: with direct steps it counts one round more than it has slices, and that
// round is the drain (nothing to move; the last rank of the chain has sent nothing and passes at once).
DFX_HD Prim chain_drain_round(Prim q, int kind, bool direct, uint32_t g, uint32_t rounds) {
  if (direct && (kind == KIND_BC || kind == KIND_RD) && g + 1 == rounds) {
    q.recv = q.send = q.from_send = q.to_recv = q.notify = q.din = false;
    q.drain = true;
  }
  return q;
}

// Ring chunk that the first primitive of a sequence works on (see DfxDyn.cidx): an all-gather
// starts with the rank's own block, the chains (broadcast, reduce) have one block, all-reduce and
// reduce-scatter start with the chunk of the rank before.
DFX_HD uint32_t first_chunk(int kind, uint32_t rank, uint32_t R) {
  if (kind == KIND_AG) return rank;
  if (kind == KIND_BC || kind == KIND_RD || R == 1) return 0u;
  return (rank + R - 1) % R;
}

// The SQE of an invocation "cooked" for one workgroup: every address a primitive needs resolved
// once, so that a context load is a plain copy (Sec. 4.2 (4)).  vch: channel of the collective
// that this workgroup serves.
DFX_HD DfxCooked cook_sqe(const DfxStatic& q, uint8_t* pool, uint32_t rank, uint32_t R, uint32_t vch) {
  DfxCooked k;
  k.sendbuf = q.sendbuf; k.recvbuf = q.recvbuf; k.count = q.count;
  k.block_elems = q.block_elems; k.part_elems = q.part_elems;
  uint8_t* conn = pool + q.conn_off;   // flags first, then slots
  const uint32_t e_out = rank, e_in = (rank + R - 1) % R;
  const size_t fo = (size_t)e_out * q.nchan + vch, fi = (size_t)e_in * q.nchan + vch;
  uint8_t* slots = conn + (size_t)R * q.nchan * DFX_FLAG_STRIDE;
  k.flags_out = (uint64_t)(conn + fo * DFX_FLAG_STRIDE);
  k.flags_in = (uint64_t)(conn + fi * DFX_FLAG_STRIDE);
  k.fifo_out = (uint64_t)(slots + fo * q.nslots * q.slot_bytes);
  k.fifo_in = (uint64_t)(slots + fi * q.nslots * q.slot_bytes);
  // a direct broadcast has no slots (no step of it fills or reads one)
  if (q.kind == KIND_BC && (q.flags & DFX_SQE_DIRECT)) k.fifo_out = k.fifo_in = 0;
  if (q.flags & DFX_SQE_FOLD) {
    // fold steps have no connectors: the words carry the channel's shared counters, the channel's first line (rank 0's;
    // the others follow nchan lines apart) and what the counter of finished steps shows at the end of this invocation
    k.fifo_in = fold_line(k.flags_out, rank, 0, q.nchan);
    k.flags_in = fold_shared_line(k.flags_out, rank, R, q.nchan);
    k.fifo_out = ((uint64_t)q.seq + 1u) * (R * q.rounds);
    // the buffers' addresses travel through the lines: the words carry the jobs' row limit and a channel's part of a slice
    k.sendbuf = q.slot_bytes;
    k.recvbuf = q.share & ~DFX_SHARE_PEERS;
  }
  k.slice_elems = q.slice_elems; k.rounds = q.rounds; k.seq = q.seq;
  k.nprim = (uint16_t)q.nprim; k.nchan = q.nchan;
  k.nslots = (uint8_t)((q.flags & DFX_SQE_FOLD) ? q.root : q.nslots);   // (no slots in fold steps: the byte carries the root)
  k.kind = q.kind; k.dtype = (uint8_t)(q.dtype | (q.op << 4));
  // place in the chain: broadcast starts at the root, reduce at the rank after it
  const uint32_t bpos = (rank + 2 * R - q.root - (q.kind == KIND_RD ? 1u : 0u)) % R;
  k.bc_pos = bpos == 0 ? 0 : (bpos == R - 1 ? 2 : 1);
  if (q.kind == KIND_RD && (q.flags & DFX_SQE_DIRECT) && bpos == 1 && R > 2) k.bc_pos = 3;   // reads the first rank's send buffer
  if (q.flags & DFX_SQE_DIRECT) k.bc_pos |= DFX_CTX_DIRECT;   // a collective with direct steps
  if (q.flags & DFX_SQE_FOLD) k.bc_pos |= DFX_CTX_FOLD;       // a collective in fold steps
  if (q.flags & DFX_SQE_DRAWN) k.bc_pos |= DFX_CTX_DRAWN;     // ... whose rows are drawn
  if (q.flags & DFX_SQE_SWEEP) k.bc_pos |= DFX_CTX_SWEEP;     // ... that all ranks sweep together
  k.priority = q.priority; k.vch = (uint16_t)vch;
  return k;
}

// Where slice g of ring chunk cidx lies for the workgroup that holds context S: element offsets
// in the send and the recv buffer and the slice's length in bytes (clipped to the chunk's and the
// channel's true length: the last ones may be short or empty).
struct SliceGeom { uint64_t soff, doff; uint32_t bytes, eb; };
DFX_HD SliceGeom slice_geometry(const DfxCooked& S, uint32_t R, uint32_t g, uint32_t cidx) {
  const int kind = S.kind, dt = S.dtype & 15;
  SliceGeom o;
  o.eb = (dt == DT_F32 || dt == DT_I32) ? 4u : 2u;
  const uint32_t slice_elems = S.slice_elems, vch = S.vch;
  const uint64_t count = S.count, block_elems = S.block_elems, part_elems = S.part_elems;
  const bool ring_chunks = R > 1 && kind == KIND_AR;
  uint64_t blen = count;
  if (ring_chunks) {
    const uint64_t start = (uint64_t)cidx * block_elems;
    blen = start >= count ? 0 : (count - start < block_elems ? count - start : block_elems);
  }
  uint64_t lo = (uint64_t)vch * part_elems + (uint64_t)g * slice_elems;
  uint64_t hi = lo + slice_elems;
  const uint64_t pend = (uint64_t)(vch + 1) * part_elems;
  if (hi > pend) hi = pend;
  if (lo > pend) lo = pend;     // (the drain round of a chain lies behind the channel's last slice: empty, not negative)
  if (lo > blen) lo = blen;
  if (hi > blen) hi = blen;
  o.bytes = (uint32_t)(hi - lo) * o.eb;
  o.soff = lo; o.doff = lo;
  if (ring_chunks) { o.soff += (uint64_t)cidx * block_elems; o.doff = o.soff; }
  else if (kind == KIND_RS) o.soff += (uint64_t)cidx * count;
  else if (kind == KIND_AG) o.doff += (uint64_t)cidx * count;
  return o;
}


// The position after a primitive.  Slices are taken in windows of W: primitive p of every slice of the
// window, then primitive p+1 of every slice, ...  The neighbour does the same, so when this rank comes
// to (slice, p+1) the neighbour finished (slice, p) one job ago instead of at this very moment, and the
// hop latency hides behind the other slice's data.  The chunk index steps down the ring with p; a new
// window starts the sequence over.  g >= rounds afterwards: that was the last primitive of the share.
struct SeqPos { uint32_t g, p, cidx; };
DFX_HD SeqPos next_position(int kind, uint32_t R, uint32_t rank, uint32_t W, uint32_t rounds, uint32_t nprim,
                            uint32_t g, uint32_t p, uint32_t cidx) {
  SeqPos n;
  n.g = g; n.p = p; n.cidx = cidx;
  if (((g + 1) & (W - 1)) != 0 && g + 1 < rounds) ++n.g;
  else {
    n.g &= ~(W - 1);
    n.cidx = (cidx == 0) ? R - 1 : cidx - 1;
    if (++n.p == nprim) {
      n.p = 0; n.g += W;
      n.cidx = first_chunk(kind, rank, R);
    }
    if (kind == KIND_BC || kind == KIND_RD) n.cidx = 0;
  }
  return n;
}

// The walk of a collective in fold steps: the step with data (p = 0) for every slice of the share, then, on channel 0, the last
// wait (p = 1) once, which is for all channels.  g >= rounds afterwards: that was it.
DFX_HD SeqPos next_fold_position(uint32_t rounds, uint32_t vch, uint32_t g, uint32_t p, uint32_t cidx) {
  SeqPos n;
  n.cidx = cidx; n.p = 0;
  if (p == 0 && g + 1 < rounds) n.g = g + 1;
  else if (p == 0 && vch == 0) { n.g = g; n.p = 1; }
  else n.g = rounds;
  return n;
}

#endif
