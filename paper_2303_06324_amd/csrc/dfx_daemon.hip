// The daemon kernel: one persistent grid that executes, preempts and schedules ring
// collectives for R virtual ranks on one MI355X (gfx950).
//
// Workgroup = (virtual rank, channel).  Every workgroup runs the scheduling loop of the
// paper's Alg. 1 (Sec. 4.3) on its own: fetch SQEs into an LDS task queue, walk the queue,
// load a collective's context into an LDS slot, execute its primitives in two-phase blocking
// fashion (bounded spin on the connector flags, then the slice's data movement), raise the
// spin threshold after a success, and on a timed-out wait save the dynamic context (lazily)
// and switch to the next collective.  Completion is counted per collective; the last channel
// posts the CQE.  Connectors are FIFOs of K slots in HBM guarded by monotone tail/head
// counters; a primitive touches nothing before both its conditions hold (Sec. 4.1, 4.5).
// Every rank's buffers lie in the same HBM, so most collectives run in fold steps, which need no connectors: every rank
// does its part straight from send buffers to recv buffers when all have submitted, and its workgroup on channel 0 posts the
// completion when all are through (see make_fold_prim; dfx_config.fold_max_bytes says which do).
// Rings and chains, where they run, take direct steps from direct_min_bytes on: in
// the copy steps (gather phase of an all-reduce, all-gather, broadcast) the result goes to the
// rank's recv buffer only (through the coherent path described below), the counter is raised
// all the same, and the next rank reads the chunk from that recv buffer; the opening send of
// a reduce phase (all-reduce, reduce-scatter, reduce chain) moves nothing, the next rank reads
// the chunk from this rank's send buffer; a last step waits until the neighbour has read
// everything (see Prim::notify / din / din_send / drain).
//
// Memory-model rules used here (AMDGPU, one agent with one L2 per XCD), two connector modes:
//   device-coherent accesses (fifo_coherent = 1, the default)
//     connector slots are only ever touched by sc1 (device-scope) buffer loads/stores, which
//     do not linger in the per-XCD caches; every mover wave drains its stores (vmcnt(0)) and
//     counts itself done in LDS; the wave that completes the count raises the connector
//     counter with a device-scope atomic; the consumer's scheduler wave polls the counter with
//     sc1 loads and its movers read the slot with sc1 loads.  No bulk L2 write-back or
//     invalidate per slice.  User buffers stay ordinary cached memory: the send buffer is made
//     visible by the system-scope acquire at SQE fetch, the recv buffer is flushed by the
//     system-scope release before the completion counter.
//   fenced (fifo_coherent = 0, kept for comparison)
//     connector slots are ordinary cached memory; the publishing wave issues an agent-scope
//     release fence (L2 write-back) before it raises the counter, and every mover wave an
//     agent-scope acquire fence (invalidate) before its loads of a slot.
//   fold steps
//     device-coherent accesses throughout: the send buffers are read and the recv buffers written with sc1, which
//     bypasses the L2s, so neither the fetch of such a collective invalidates a cache nor its completion writes one
//     back (an L2 write-back or invalidate costs 0.6 - 1 us on an idle device, and an XCD's 32 workgroups queue for it).
//   SQ / CQ / host control words are host-visible and use system scope.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfx_internal.h"
#include "dfx_geometry.h"
#include "dfx_movers.h"
#include "dfx_rules.h"

namespace {


constexpr int NT = DFX_WG_THREADS;
#ifndef DFX_UNROLL
#define DFX_UNROLL 8
#endif
constexpr int UNROLL = DFX_UNROLL;   // independent 16-byte vectors in flight per source and thread
constexpr int DT_COPY = -1;   // a primitive without a reducing side moves bytes, whatever the element type

enum { W_OK = 0, W_TIMEOUT = 1, W_STOP = 2 };
enum { STOP_NONE = 0, STOP_ABORT = 1, STOP_QUIT = 2, STOP_EXIT = 3 };

template <class T>
__device__ __forceinline__ T* known_global(T* p) {
  __builtin_assume(!__builtin_amdgcn_is_shared((const __attribute__((address_space(0))) void*)p) &&
                   !__builtin_amdgcn_is_private((const __attribute__((address_space(0))) void*)p));
  return p;
}

__device__ __forceinline__ u64 ld_agent64(const u64* p) { return __hip_atomic_load(global_ptr(p), __ATOMIC_RELAXED, SCOPE_AGENT); }
__device__ __forceinline__ uint32_t ld_agent32(const uint32_t* p) { return __hip_atomic_load(global_ptr(p), __ATOMIC_RELAXED, SCOPE_AGENT); }
__device__ __forceinline__ u64 ld_sys64(const u64* p) { return __hip_atomic_load(global_ptr(p), __ATOMIC_RELAXED, SCOPE_SYSTEM); }
__device__ __forceinline__ uint32_t ld_sys32(const uint32_t* p) { return __hip_atomic_load(global_ptr(p), __ATOMIC_RELAXED, SCOPE_SYSTEM); }

// Release fences end with an explicit wait: the L2 write-back they issue must have completed
// before the flag store that follows.  The compiler's own wait is dropped when it believes no
// memory operation is pending (the wave's own stores were drained earlier), and the write-back
// itself is not on its scoreboard.
__device__ __forceinline__ void fence_acquire_agent() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }
__device__ __forceinline__ void fence_release_agent() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent"); __builtin_amdgcn_s_waitcnt(0); }
__device__ __forceinline__ void fence_acquire_system() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, ""); }
__device__ __forceinline__ void fence_release_system() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, ""); __builtin_amdgcn_s_waitcnt(0); }

// ------------------------------------------------------------------------------------------
// slice mover: value = [fifo_in[i]] (+) [sendbuf[i]];  recvbuf[i] = value;  fifo_out[i] = value
// (each side present or not, as the primitive says).  128-bit coalesced accesses, four
// independent vectors in flight per source and thread.
//
// Connector slots are accessed through buffer instructions.  COH = 1 marks those accesses
// device-coherent (sc1: they bypass the non-coherent levels and write through), so that
// connector traffic needs no bulk L2 write-back / invalidate around every slice; COH = 0 uses
// ordinary cached accesses and relies on the agent-scope fences of the caller.
// User buffers are plain pointers, accessed with 16-byte vectors whatever their alignment; only
// the sub-vector tail of a slice is moved element by element.
// ------------------------------------------------------------------------------------------
// User-buffer accesses of the main loop are marked non-temporal: each byte is touched once, and
// keeping it out of the way leaves the memory-side cache to the connector slots (+3 % measured).
// They are 16-byte accesses through a type that promises only element alignment (2 bytes): the
// blocks of an all-gather / reduce-scatter of odd length start anywhere, and the hardware does
// under-aligned vector accesses at full width (element by element the same blocks ran ten times
// slower).
typedef v4u v4u_user __attribute__((aligned(2)));
__device__ __forceinline__ uint4 ld_user(const v4u_user* p) {
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const GLOBAL_AS v4u_user*)p));
}
__device__ __forceinline__ void st_user(v4u_user* p, uint4 v) {
  __builtin_nontemporal_store(__builtin_bit_cast(v4u, v), (GLOBAL_AS v4u_user*)p);
}

template <int AUX>
struct Slot {   // one connector slot seen through a buffer resource
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ Slot(const void* base, uint32_t bytes) {
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
  }
  __device__ __forceinline__ uint4 ld16(uint32_t off) const {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, AUX));
  }
  __device__ __forceinline__ void st16(uint32_t off, uint4 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), rsrc, (int)off, 0, AUX);
  }
  __device__ __forceinline__ uint32_t ld4(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off, 0, AUX); }
  __device__ __forceinline__ void st4(uint32_t off, uint32_t v) const { __builtin_amdgcn_raw_buffer_store_b32(v, rsrc, (int)off, 0, AUX); }
  __device__ __forceinline__ uint16_t ld2(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)off, 0, AUX); }
  __device__ __forceinline__ void st2(uint32_t off, uint16_t v) const { __builtin_amdgcn_raw_buffer_store_b16(v, rsrc, (int)off, 0, AUX); }
};

// GEN = false: the sum only (the common case keeps its own instantiation); GEN = true: `op` picks
// the reducing function at run time (a wave-uniform branch per vector).
template <int DT, bool GEN, int AIN, int AOUT, bool FIN, bool SB, bool RB, bool FOUT, int NTH>
__device__ __forceinline__ void move_slice(const void* fin_p, const char* __restrict__ sb, char* __restrict__ rb,
                                           void* fout_p, uint32_t bytes, uint32_t tid, int op) {
  constexpr int NT = NTH;   // threads that share the slice: the mover waves
  static_assert(FIN || SB, "a primitive has a source");
  static_assert(RB || FOUT, "a primitive has a destination");
  const Slot<AIN> fin(fin_p, FIN ? bytes : 0);
  const Slot<AOUT> fout(fout_p, FOUT ? bytes : 0);
  uint32_t done = 0;
  {
    const v4u_user* __restrict__ S = (const v4u_user*)sb;
    v4u_user* __restrict__ D = (v4u_user*)rb;
    const uint32_t nvec = bytes >> 4;
    uint32_t i = tid;
    for (; i + (UNROLL - 1) * NT < nvec; i += UNROLL * NT) {
      uint4 v[UNROLL];
      if (FIN) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = fin.ld16((i + u * NT) << 4);
      }
      if (SB) {
        uint4 w[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) w[u] = ld_user(&S[i + u * NT]);
        if (FIN && GEN) op_batch<DT, UNROLL>(v, w, op);
        else {
#pragma unroll
          for (int u = 0; u < UNROLL; ++u) v[u] = FIN ? add_vec<DT>(v[u], w[u]) : w[u];
        }
      }
      if (FOUT) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) fout.st16((i + u * NT) << 4, v[u]);
      }
      if (RB) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) st_user(&D[i + u * NT], v[u]);
      }
    }
    if (i < nvec) {
      // remainder: the same unrolled shape with per-vector predicates, so that all loads of the
      // tail are in flight together (a short slice is one such block: one memory round trip)
      uint4 v[UNROLL];
      if (FIN) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = fin.ld16((i + u * NT) << 4);   // out of range reads return 0
      }
      if (SB) {
        uint4 w[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) w[u] = (i + u * NT < nvec) ? ld_user(&S[i + u * NT]) : uint4{0, 0, 0, 0};
        if (FIN && GEN) op_batch<DT, UNROLL>(v, w, op);
        else {
#pragma unroll
          for (int u = 0; u < UNROLL; ++u) v[u] = FIN ? add_vec<DT>(v[u], w[u]) : w[u];
        }
      }
      if (FOUT) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) if (i + u * NT < nvec) fout.st16((i + u * NT) << 4, v[u]);
      }
      if (RB) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) if (i + u * NT < nvec) st_user(&D[i + u * NT], v[u]);
      }
    }
    done = nvec << 4;
  }
  // element-wise remainder: the sub-vector tail of a slice
  if (done < bytes) {
    if (DT == DT_F32 || DT == DT_I32) {
      const uint32_t* S = (const uint32_t*)sb;
      uint32_t* D = (uint32_t*)rb;
      for (uint32_t o = done + (tid << 2); o < bytes; o += NT << 2) {
        uint32_t v = 0;
        if (FIN) v = fin.ld4(o);
        if (SB) { uint32_t w = S[o >> 2]; v = FIN ? (GEN ? op_word<DT>(v, w, op) : add_word<DT>(v, w)) : w; }
        if (FOUT) fout.st4(o, v);
        if (RB) D[o >> 2] = v;
      }
    } else {   // 16-bit elements; pure copies also come here (every dtype is a multiple of 2 bytes)
      const uint16_t* S = (const uint16_t*)sb;
      uint16_t* D = (uint16_t*)rb;
      for (uint32_t o = done + (tid << 1); o < bytes; o += NT << 1) {
        uint16_t v = 0;
        if (FIN) v = fin.ld2(o);
        if (SB) { uint16_t w = S[o >> 1]; v = FIN ? (GEN ? op_half<DT>(v, w, op) : add_half<DT>(v, w)) : w; }
        if (FOUT) fout.st2(o, v);
        if (RB) D[o >> 1] = v;
      }
    }
  }
}

// `dtype` carries the element type in its low four bits and the reducing function above them.
template <int AIN, int AOUT, bool FIN, bool SB, bool RB, bool FOUT, int NTH>
__device__ __forceinline__ void move_dispatch(int dtype, const void* fin, const char* sb, char* rb, void* fout, uint32_t bytes, uint32_t tid) {
  if (!(FIN && SB)) { move_slice<DT_COPY, false, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, 0); return; }
  const int dt = dtype & 15, op = dtype >> 4;
  if (op == OP_SUM) {
    switch (dt) {
      case DT_F32: move_slice<DT_F32, false, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, 0); break;
      case DT_BF16: move_slice<DT_BF16, false, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, 0); break;
      case DT_F16: move_slice<DT_F16, false, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, 0); break;
      default: move_slice<DT_I32, false, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, 0); break;
    }
  } else {
    switch (dt) {
      case DT_F32: move_slice<DT_F32, true, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, op); break;
      case DT_BF16: move_slice<DT_BF16, true, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, op); break;
      case DT_F16: move_slice<DT_F16, true, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, op); break;
      default: move_slice<DT_I32, true, AIN, AOUT, FIN, SB, RB, FOUT, NTH>(fin, sb, rb, fout, bytes, tid, op); break;
    }
  }
}

#ifndef DFX_LDS_STAGE
#define DFX_LDS_STAGE 0
#endif
#if DFX_LDS_STAGE
// Experiment build (-DDFX_LDS_STAGE=1): the recv-reduce-send step with both inputs staged through LDS.
// Each mover wave brings the vectors of the connector slot and of the send buffer in with gfx950's
// 16-byte global -> LDS loads (no registers held while they travel), STAGE_D - 1 batches of STAGE_U
// vectors per lane and source ahead of the batch being reduced, reads them back with ds_read_b128, adds,
// and stores to the outgoing slot.  Per lane 2 x STAGE_U x (STAGE_D - 1) = 24 loads are in flight all the
// time, instead of 16 that are issued together and waited for together.
// The waits are counted by hand: the compiler would put vmcnt(0) in front of every LDS read that follows
// an LDS-writing load, which would undo the prefetch.  Vector memory operations of a wave complete in the
// order they were issued, so "at most N outstanding" means that everything older than the youngest N is
// done; that is also why both inputs go through LDS: a wait for a register load would wait for every
// LDS-writing load issued before it.
constexpr uint32_t STAGE_U = 4;                              // vectors per lane, source and batch
constexpr uint32_t STAGE_D = 4;                              // batches in LDS per wave (STAGE_D - 1 ahead of the one in use)
constexpr uint32_t STAGE_BATCH_BYTES = 2 * STAGE_U * 1024;   // two sources x U vectors x 64 lanes x 16 bytes
constexpr uint32_t STAGE_WAVE_BYTES = STAGE_D * STAGE_BATCH_BYTES;
typedef __attribute__((address_space(3))) unsigned char lds_byte;

template <int N>
__device__ __forceinline__ void stage_read(uint32_t lds_addr, v4u (&v)[8]) {
  asm volatile(
      "s_waitcnt vmcnt(%9)\n\t"
      "ds_read_b128 %0, %8\n\t"
      "ds_read_b128 %1, %8 offset:1024\n\t"
      "ds_read_b128 %2, %8 offset:2048\n\t"
      "ds_read_b128 %3, %8 offset:3072\n\t"
      "ds_read_b128 %4, %8 offset:4096\n\t"
      "ds_read_b128 %5, %8 offset:5120\n\t"
      "ds_read_b128 %6, %8 offset:6144\n\t"
      "ds_read_b128 %7, %8 offset:7168\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(lds_addr), "n"(N)
      : "memory");
}

// bytes: a multiple of STAGE_U x NTH x 16; fin_p and sb 16-byte aligned; stage: this workgroup's staging
// area (NTH / 64 waves x STAGE_WAVE_BYTES)
template <int DT, int NTH>
__device__ __forceinline__ void move_rrs_staged(const void* fin_p, const char* __restrict__ sb, void* fout_p, uint32_t bytes,
                                                uint32_t tid, lds_byte* stage) {
  static_assert(STAGE_U == 4, "stage_read reads 2 x 4 vectors");
  const Slot<AUX_DEVICE> fout(fout_p, bytes);
  const uint32_t wave = tid >> 6, lane = tid & 63u;
  lds_byte* mine = stage + wave * STAGE_WAVE_BYTES;
  const uint32_t lds0 = (uint32_t)(uintptr_t)mine + lane * 16u;
  const uint4* F = (const uint4*)fin_p;
  const uint4* S = (const uint4*)sb;
  const uint32_t nvec = bytes >> 4, per_batch = STAGE_U * NTH, nbatch = nvec / per_batch;
  auto bring = [&](uint32_t k) {       // batch k -> its place in LDS: 2 x STAGE_U instructions
    lds_byte* dst = mine + (k % STAGE_D) * STAGE_BATCH_BYTES;
    const uint32_t i = tid + k * per_batch;
#pragma unroll
    for (uint32_t u = 0; u < STAGE_U; ++u)
      __builtin_amdgcn_global_load_lds((const void*)&F[i + u * NTH], (__attribute__((address_space(3))) void*)(dst + u * 1024), 16, 0, AUX_DEVICE);
#pragma unroll
    for (uint32_t u = 0; u < STAGE_U; ++u)
      __builtin_amdgcn_global_load_lds((const void*)&S[i + u * NTH], (__attribute__((address_space(3))) void*)(dst + (STAGE_U + u) * 1024), 16, 0, 2 /* nt */);
  };
  for (uint32_t k = 0; k + 1 < STAGE_D && k < nbatch; ++k) bring(k);
  for (uint32_t b = 0; b < nbatch; ++b) {
    if (b + STAGE_D - 1 < nbatch) bring(b + STAGE_D - 1);
    asm volatile("" ::: "memory");
    // Issued after batch b's loads: the loads of the batches ahead (2U each) and, in the steady state, the
    // stores of the STAGE_D - 1 iterations in between (U each).  Towards the ends the stores are left out of
    // the count: a smaller count only waits for more.
    const uint32_t ahead = (nbatch - 1 - b) < (STAGE_D - 1) ? (nbatch - 1 - b) : (STAGE_D - 1);
    v4u v[8];
    const uint32_t at = lds0 + (b % STAGE_D) * STAGE_BATCH_BYTES;
    if (ahead == STAGE_D - 1 && b >= STAGE_D - 1) stage_read<(STAGE_D - 1) * 3 * STAGE_U>(at, v);
    else if (ahead == 3) stage_read<3 * 2 * STAGE_U>(at, v);
    else if (ahead == 2) stage_read<2 * 2 * STAGE_U>(at, v);
    else if (ahead == 1) stage_read<1 * 2 * STAGE_U>(at, v);
    else stage_read<0>(at, v);
    const uint32_t i = tid + b * per_batch;
#pragma unroll
    for (uint32_t u = 0; u < STAGE_U; ++u)
      fout.st16((i + u * NTH) << 4, add_vec<DT>(__builtin_bit_cast(uint4, v[u]), __builtin_bit_cast(uint4, v[STAGE_U + u])));
  }
}
#endif

// fin / sb / rb / fout are null when the primitive does not use that side.
// AUX: how connector slots are accessed (AUX_DEVICE, or AUX_CACHED in the fenced mode).
template <int AUX, int NTH>
__device__ __forceinline__ void run_prim(int dtype, const void* fin, const char* sb, char* rb, void* fout, uint32_t bytes, uint32_t tid) {
  if (fin) {
    if (sb) {
      if (rb) { if (fout) move_dispatch<AUX, AUX, true, true, true, true, NTH>(dtype, fin, sb, rb, fout, bytes, tid);    // recv-reduce-copy-send
                else move_dispatch<AUX, AUX, true, true, true, false, NTH>(dtype, fin, sb, rb, fout, bytes, tid); }      // recv-reduce-copy
      else move_dispatch<AUX, AUX, true, true, false, true, NTH>(dtype, fin, sb, rb, fout, bytes, tid);                  // recv-reduce-send
    } else {
      if (!rb) move_dispatch<AUX, AUX, true, false, false, true, NTH>(dtype, fin, sb, rb, fout, bytes, tid);             // direct recv-copy (coherent destination)
      else if (fout) move_dispatch<AUX, AUX, true, false, true, true, NTH>(dtype, fin, sb, rb, fout, bytes, tid);        // recv-copy-send
      else move_dispatch<AUX, AUX, true, false, true, false, NTH>(dtype, fin, sb, rb, fout, bytes, tid);                 // recv-copy
    }
  } else {
    if (rb) { if (fout) move_dispatch<AUX, AUX, false, true, true, true, NTH>(dtype, fin, sb, rb, fout, bytes, tid);     // copy-send
              else move_dispatch<AUX, AUX, false, true, true, false, NTH>(dtype, fin, sb, rb, fout, bytes, tid); }       // copy
    else move_dispatch<AUX, AUX, false, true, false, true, NTH>(dtype, fin, sb, rb, fout, bytes, tid);                   // send
  }
}

// ------------------------------------------------------------------------------------------
// LDS state of one workgroup
// ------------------------------------------------------------------------------------------
struct Job {                         // what the scheduler wave hands to the mover waves for one slice
  const void* fin; const char* sb; char* rb; void* fout;
  uint32_t bytes; int dtype;
  uint32_t coll, prim;               // for the timeline trace only
  uint32_t nsrc, ndst;               // not 0: step with data of a collective in fold steps (that many sources and destinations in the job's tables)
  uint32_t index, sharers;           // ... which of the region's workgroups this is, and how many there are
  uint32_t head;                     // ... bytes before the first row (fold_head)
  uint32_t limit, fresh;             // ... drawn rows per wave at most (0 = rows are dealt); first job of the share
  uint32_t gang;                     // not 0 (and nsrc 0): so many short collectives, which the waves take in turn (GangEntry)
  u64 draw;                          // ... the region's row counter (0 = rows are dealt)
};
constexpr uint32_t FRESH_SWEEP = 2u;   // (fresh: all ranks sweep the message together, SweepJob says more)
struct SweepJob { uint32_t kind, R, rank, longest, at, pad; u64 total; };   // at: rows of this wave's that earlier jobs have taken, times the rank's waves (dealt)

// Short collectives in fold steps that a readiness scan finds runnable together go to the movers as one job, a gang.  What bounds them
// is no bandwidth but the chain of each -- lines polled, job posted, a row or a few loaded, folded and stored, the last wait polled --,
// and one after the other that took 5.3 us of which the movers worked 2.5.  Together they share the poll (a lane per collective and
// rank) and run side by side, a mover wave each.  1024 all-reduces of 4 - 64 KiB, every rank in its own order: R = 8 531 -> 378 us,
// R = 4 415 -> 215, R = 2 480 -> 195 (R = 8 since then 266, of which the data takes 75); 256 of them 145 -> 107, 114 -> 68, 145 -> 67; 64 of them 57 -> 48, 45 -> 37, 42 -> 32.
// GangRun is what the scan leaves of a runnable one (its lane has the context in registers), GangEntry what a mover wave needs of it.
struct alignas(16) GangRun {
  u64 line0, counters, src, dst;     // the channel's line of rank 0, its shared counters; offsets of the region in the buffers
  uint32_t bytes, seq, nchan_vch, what;   // length of the region; invocation; channels | channel << 16; kind | type and function << 8 | root << 16
  uint32_t coll, pos, share, pad;    // ... its place in the queue; a channel's part of the region
};
struct alignas(16) GangEntry { u64 add_one; uint32_t bytes, index, sharers, dtype, nsrc, ndst; };
constexpr uint32_t GANG_MAX = 16u;           // collectives of a gang at most; 64 lanes hold all of their buffers
constexpr uint32_t GANG_SHARE = 16u << 10;   // bytes of a share at most: what one channel has up to 512 KiB per region, one wave's work for 10 us

// What publishing and retiring a posted job needs.  Written by the scheduler when it posts the
// job; read by the mover wave that finishes the job last (counter updates) and by the scheduler
// when it retires the job (statistics, completion).
struct Flight {
  u64* tail_out; u64* head_in;       // counters to raise (null = that side is not used)
  u64 sent_new, recvd_new;           // their new values
  uint32_t last;                     // the primitive ends this workgroup's share of the invocation
  uint32_t coll, seq, nchan;
  u64* add_one;                      // fold steps: shared counter to add 1 to (null = none)
};

struct Shared {
  DfxDaemonArgs args;
  DfxCtxEntry slot[DFX_CTX_SLOTS];   // active context slots (Sec. 5, direct-mapped)
  uint32_t slot_tag[DFX_CTX_SLOTS];
  uint32_t slot_claim[DFX_CTX_SLOTS];  // readiness scan: which entry of the scan gets to fill a slot (scan step << 8 | lane)
  Job job[2];                        // posted jobs, indexed by job number & 1
  Flight fl[2];
  SweepJob sweep[2];                 // ... of a sweep
  u64 tab_src[2][64];                // fold steps: source addresses of the job, in the order of combination
  u64 tab_dst[2][64];                // ... and where the result goes
  GangRun run[64];                   // the runnable short collectives of the last scan, in the order of the pass
  GangEntry gang[2][GANG_MAX];       // the collectives of a posted gang; their addresses in tab_src and tab_dst, so many lanes apart as hold a rank each
  u64 gone;                          // queue positions that gangs of the pass are through with
  uint4 peer[64];                    // table of buffers that came with the lone entry in hand (DfxPeer)
  uint32_t peers_seq;                // ... of which invocation
  uint32_t behind;                   // passes in a row that left others unvisited behind short ones (turn_due)
  uint32_t nothers;                  // runnable entries of the pass behind short ones
  uint32_t turn, turns;              // one of these has its turn in the pass: 1 + its place in the list (0: none has); turns there have been
  uint32_t job_seq;                  // jobs posted so far (scheduler -> movers)
  uint32_t wave_done[2];             // mover waves that have finished job k, at index k & 1
  uint32_t jobs_done;                // jobs finished and published (movers -> scheduler)
  uint32_t leave;                    // scheduler -> movers: no more jobs
  uint32_t trace_n;                  // trace samples written (monotone)
  uint32_t qlen_out;                 // queue length handed to all waves when leaving
  u64 stat[DFX_NSTAT];               // counters (LDS atomics without return: one instruction, no wait)
  uint16_t rlist[DFX_MAX_COLLS];     // queue positions the readiness scan found runnable, ascending
  uint16_t taskq[DFX_MAX_COLLS];     // task queue (Sec. 4.2 (1))
#if DFX_LDS_STAGE
  __attribute__((aligned(16))) unsigned char stage[(DFX_MOVERS / 64) * STAGE_WAVE_BYTES];   // experiment build: staging area of the mover waves
#endif
};

__device__ __forceinline__ void raise_error(const DfxDaemonArgs& a, uint32_t code, uint32_t wg) {
  uint32_t expected = 0;
  if (__hip_atomic_compare_exchange_strong(&a.dev_ctl[DC_ERR], &expected, code, __ATOMIC_RELAXED, __ATOMIC_RELAXED, SCOPE_AGENT))
  {
    __hip_atomic_store(&a.dev_ctl[DC_ERR_WG], wg, __ATOMIC_RELAXED, SCOPE_AGENT);
    if (a.status) __hip_atomic_store(a.status, 0x100u | code, __ATOMIC_RELAXED, SCOPE_AGENT);
  }
  __hip_atomic_store(&a.dev_ctl[DC_ABORT], 1u, __ATOMIC_RELEASE, SCOPE_AGENT);
}

__device__ __forceinline__ void bump(u64* stat, int i, u64 v) {
  (void)__hip_atomic_fetch_add(&stat[i], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// saved contexts in memory, in 16-byte words
__device__ __forceinline__ uint4 ld_ctx(const uint4* p) { return __builtin_bit_cast(uint4, *(const GLOBAL_AS v4u*)p); }
__device__ __forceinline__ void st_ctx(uint4* p, uint4 v) { *(GLOBAL_AS v4u*)p = __builtin_bit_cast(v4u, v); }
template <class T>
__device__ __forceinline__ void st_ctx(T* p, const T& v) {
  struct Words { uint4 w[sizeof(T) / 16]; };
  const Words x = __builtin_bit_cast(Words, v);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 16); ++i) st_ctx((uint4*)p + i, x.w[i]);
}


// LDS slot of a collective's context: a multiplicative hash, because the ids that share a workgroup's
// queue are far from random (with single-channel collectives spread over the channels they are all
// congruent modulo the channel count)
static_assert(DFX_CTX_SLOTS == 64, "ctx_slot takes the top six bits");
__device__ __forceinline__ uint32_t ctx_slot(uint32_t coll) { return (coll * 2654435769u) >> 26; }

// A gang's collectives lie 1 << gang_shift(R) lanes apart.
__device__ __forceinline__ uint32_t gang_shift(uint32_t R) { return R < 2u ? 0u : 32u - (uint32_t)__builtin_clz(R - 1u); }

// What a mover wave does for collective `c` of a gang: all rows of the workgroup's share, and the elements before and behind them where
// they are its (rows of a short span begin on 16 bytes of the recv buffers: fold_head).
__device__ __forceinline__ void gang_move(const GangEntry& c, const u64* src_tab, const u64* dst_tab, uint32_t R, uint32_t lane) {
  const uint32_t bytes = bcast0(c.bytes), index = bcast0(c.index), sharers = bcast0(c.sharers);
  const uint32_t off = (0u - bcast0((uint32_t)dst_tab[0])) & 15u, head = off < bytes ? off : bytes, end = head + ((bytes - head) & ~15u);
  const uint32_t dtype = bcast0(c.dtype), nsrc = bcast0(c.nsrc), ndst = bcast0(c.ndst);
  const int op = (int)(dtype >> 4), dt = nsrc == 1u ? DT_F16 : (int)(dtype & 15u);     // (copies: every element type is a multiple of 2 bytes)
  const uint32_t row = fold_row_bytes(nsrc == 1u, R);
  for (uint32_t at = head + index * row; at < end; at += sharers * row) {
    if (nsrc == 1u) fold_row<DT_F16>(src_tab, 1u, dst_tab, ndst, at, row, end, lane, OP_SUM);
    else if (dt == DT_F32) fold_row<DT_F32>(src_tab, nsrc, dst_tab, ndst, at, row, end, lane, op);
    else if (dt == DT_BF16) fold_row<DT_BF16>(src_tab, nsrc, dst_tab, ndst, at, row, end, lane, op);
    else if (dt == DT_F16) fold_row<DT_F16>(src_tab, nsrc, dst_tab, ndst, at, row, end, lane, op);
    else fold_row<DT_I32>(src_tab, nsrc, dst_tab, ndst, at, row, end, lane, op);
  }
  for (uint32_t behind = 0; behind < 2u; ++behind) {
    const uint32_t at = behind ? end : 0u, stop = behind ? bytes : head;
    if (at >= stop || index != (behind ? 0u : sharers - 1u)) continue;
    if (dt == DT_F32) fold_ends<DT_F32>(src_tab, nsrc, dst_tab, ndst, at, stop, lane, op);
    else if (dt == DT_BF16) fold_ends<DT_BF16>(src_tab, nsrc, dst_tab, ndst, at, stop, lane, op);
    else if (dt == DT_F16) fold_ends<DT_F16>(src_tab, nsrc, dst_tab, ndst, at, stop, lane, op);
    else fold_ends<DT_I32>(src_tab, nsrc, dst_tab, ndst, at, stop, lane, op);
  }
}

// The sum of v over this lane and those before it (all 64 active): within rows of sixteen lanes, then across them.
__device__ __forceinline__ uint32_t wave_sum_upto(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);      // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);      // row_bcast:15, into rows 1 and 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);      // row_bcast:31, into rows 2 and 3
  return v;
}

// The buffers that a rank has published in its line (DFX_DIRECT_OFF), every lane the line of its own pointer.
__device__ __forceinline__ void ld_published(const void* line, v4u& recv, v4u& send) {
  static_assert(DFX_DIRECT_OFF == 16, "offsets of the two loads");
  asm volatile("global_load_dwordx4 %0, %2, off offset:16 sc1\n\t"
               "global_load_dwordx4 %1, %2, off offset:32 sc1\n\t"
               "s_waitcnt vmcnt(0)"
               : "=&v"(recv), "=&v"(send) : "v"(line) : "memory");
}

// LDS words shared between the scheduler and the mover waves
__device__ __forceinline__ uint32_t lds_ld(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void lds_st(uint32_t* p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP); }

// Raise a connector counter.  A maximum instead of a store: the waves that publish two
// consecutive jobs are different ones, and their updates may reach memory in either order.
__device__ __forceinline__ void raise_counter(u64* p, u64 v) {
  (void)__hip_atomic_fetch_max(global_ptr(p), v, __ATOMIC_RELAXED, SCOPE_AGENT);
}

// one trace sample; the index comes from an LDS counter that both kinds of wave use
__device__ __forceinline__ void trace_put(u64* trace, uint32_t* trace_n, u64 v) {
  const uint32_t i = __hip_atomic_fetch_add(trace_n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  trace[i % DFX_TRACE_N] = v;
}

__device__ __forceinline__ u64 timeline_sample(u64 t0, u64 t1, uint32_t coll, uint32_t prim) {
  u64 dur = t1 - t0;
  if (dur > 0xffffu) dur = 0xffffu;
  return (t0 & 0xffffffffull) | (dur << 32) | ((u64)(coll & 0xfffu) << 48) | ((u64)(prim & 0xfu) << 60);
}

}  // namespace

// Structure of a workgroup: wave 0 is the SCHEDULER, waves 1..4 are the MOVERS.
//
// The scheduler wave runs Alg. 1 on its own -- control checks, SQE fetch, queue walk, context
// load, bounded polling, preemption, lazy save, completion -- with its state in its registers
// and the task queue and context slots in LDS.  When a primitive's wait phase has succeeded it
// claims the connector slots (its private counters advance), posts the slice as a job in LDS and
// goes straight on to the wait phase of whatever comes next, while the movers carry the data.
// Up to two jobs are posted at a time, so the movers run from one slice into the next without
// waiting for the scheduler, and everything the scheduler does -- polling flags that live in
// HBM, scanning the queue, switching contexts -- overlaps with data movement.
//
// A mover wave takes the jobs in order; after its part of a slice it drains its stores and
// counts itself done in LDS.  The wave that completes the count raises the connector counters
// of that job (the data of all waves is then in memory) and reports the job finished; the
// scheduler retires finished jobs in order (statistics; for the last primitive of an invocation
// the completion counter and the CQE).  No workgroup barrier is used after start-up.
extern "C" __global__ void __launch_bounds__(DFX_WG_THREADS) dfx_daemon_kernel(DfxDaemonArgs kargs) {
  __shared__ Shared sh;
  // The arguments are read from an LDS copy: kept in scalar registers for the whole kernel they
  // overflow the scalar register file, and the spill reloads at every loop head cost more than
  // the LDS reads.
  if (threadIdx.x == 0) sh.args = kargs;
  __syncthreads();
  const DfxDaemonArgs& a = sh.args;
  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u;
  const bool sched = tid < 64;       // the scheduler wave
  const uint32_t wg = blockIdx.x;
  const WgPlace place = wg_place(a.wg_map, wg, a.R, a.cmax);
  const uint32_t rank = place.rank, ch = place.ch;
  const uint32_t D = a.sq_depth;
  const bool coh = a.fifo_coherent != 0;

  DfxWgState* ws = known_global(&a.wgstate[wg]);
  DfxCtxEntry* myctx = known_global(a.ctxbuf + (size_t)wg * a.max_colls);
  uint16_t* qstore = known_global(a.taskq_store + (size_t)wg * a.max_colls);
  DfxSqSlot* sqbase = known_global(a.sq + (size_t)rank * D);
  u64* cqbase = known_global(a.cq + (size_t)rank * a.cq_slots);
  u64* trace = a.trace ? known_global(a.trace + (size_t)wg * DFX_TRACE_N) : nullptr;

  // ---- restore the workgroup state left by the previous launch (Sec. 4.5)
  u64 ri = ws->read_index;
  uint32_t qlen = ws->qlen;
  for (uint32_t i = tid; i < qlen; i += NT) sh.taskq[i] = qstore[i];
  if (tid < DFX_CTX_SLOTS) sh.slot_tag[tid] = 0xffffffffu;
  if (tid < DFX_NSTAT) sh.stat[tid] = ws->stat[tid];
  if (tid == 0) {
    sh.behind = 0; sh.nothers = 0; sh.turn = 0; sh.turns = 0;
    sh.job_seq = 0; sh.wave_done[0] = 0; sh.wave_done[1] = 0; sh.jobs_done = 0; sh.leave = 0;
    sh.trace_n = ws->trace_n;
  }
  __syncthreads();

  uint32_t stop = STOP_NONE;

  if (!sched) {
    // =====================================================================================
    // mover waves
    // =====================================================================================
    // The mover waves work in DFX_MOVER_GROUPS groups; group k takes the jobs k, k + GROUPS, ...: with two
    // groups the drain of one job's stores and the first loads of the next overlap in time.
    constexpr uint32_t GROUPS = DFX_MOVER_GROUPS, GTHREADS = DFX_MOVERS / GROUPS;
    const uint32_t mtid = (tid - 64) % GTHREADS;
    const uint32_t group = (tid - 64) / GTHREADS;
    const bool first_wave = mtid < 64;
    uint32_t seen = group;
    for (;;) {
      // the leave flag is looked at only when no job is waiting: every posted job is executed
      bool go = true;
      while ((int32_t)(lds_ld(&sh.job_seq) - seen) <= 0) {
        if (lds_ld(&sh.leave)) { go = false; break; }
        __builtin_amdgcn_s_sleep(1);
      }
      if (!go) break;
      const Job j = sh.job[seen & 1];
      u64 t0 = 0;
      if (a.trace_on > 1 && first_wave) t0 = wall_clock64();
      // fenced mode: every wave invalidates before its own loads of the slot (the poll was the scheduler's)
      if (!coh && j.fin && j.bytes) fence_acquire_agent();
#if DFX_LDS_STAGE
      if (coh && GROUPS == 1 && j.fin && j.sb && !j.rb && j.fout && (j.dtype >> 4) == OP_SUM && j.bytes &&
          j.bytes % (STAGE_U * GTHREADS * 16u) == 0 && (((uintptr_t)j.sb | (uintptr_t)j.fin) & 15u) == 0) {
        lds_byte* st = (lds_byte*)sh.stage;
        switch (j.dtype & 15) {
          case DT_F32: move_rrs_staged<DT_F32, GTHREADS>(j.fin, j.sb, j.fout, j.bytes, mtid, st); break;
          case DT_BF16: move_rrs_staged<DT_BF16, GTHREADS>(j.fin, j.sb, j.fout, j.bytes, mtid, st); break;
          case DT_F16: move_rrs_staged<DT_F16, GTHREADS>(j.fin, j.sb, j.fout, j.bytes, mtid, st); break;
          default: move_rrs_staged<DT_I32, GTHREADS>(j.fin, j.sb, j.fout, j.bytes, mtid, st); break;
        }
      } else
#endif
      if (j.nsrc && __builtin_expect(bcast0(j.fresh) >= FRESH_SWEEP, 0)) {
        const SweepJob sj = sh.sweep[seen & 1];
        const uint32_t wave = bcast0(mtid >> 6), sharers = bcast0(j.sharers), index = bcast0(j.index);
        const bool fresh = (bcast0(j.fresh) & 1u) != 0;
        Sweep w;
        w.kind = bcast0(sj.kind); w.R = bcast0(sj.R); w.rank = bcast0(sj.rank); w.longest = bcast0(sj.longest);
        w.total = bcast64((uint32_t)sj.total, (uint32_t)(sj.total >> 32));
        w.nreg = sweep_regions((int)w.kind, w.R);
        const uint32_t row = sweep_row_bytes(fold_copies((int)w.kind), w.R), mine = index * DFX_FOLD_WAVES + wave;
        w.rows = (w.longest + row - 1u) / row; w.all = w.rows * w.nreg;
        w.waves = sharers * DFX_FOLD_WAVES; w.base = w.rank * w.waves; w.skip = w.waves * (w.R - 1u);
        w.lo = w.hi = 0;
        Rows rows;
        rows.ctr = (GLOBAL_AS uint32_t*)(uint32_t*)bcast64((uint32_t)j.draw, (uint32_t)(j.draw >> 32));
        rows.waves = w.waves;
        rows.left = bcast0(j.limit);
        rows.drawn = 0;
        if (rows.ctr) rows.begin(fresh, mine);
        else rows.row = mine + bcast0(sj.at);
        w.ends = 0;
        if (fresh && w.rank < w.nreg) {
          const FoldRegion own = sweep_region((int)w.kind, w.longest, w.total, w.rank);
          const bool front = mine + 1 == w.waves, tail = mine == 0 && own.end < own.len;
          w.own_src = own.src; w.own_dst = own.dst;
          w.ends_at = front ? 0u : own.end;
          w.ends = front ? own.head : tail ? own.len : 0u;
        }
        sweep_dispatch((int)bcast0((uint32_t)j.dtype), sh.tab_src[seen & 1], sh.tab_dst[seen & 1], w, rows, lane);
      }
      else if (j.nsrc) {
        const uint32_t wave = bcast0(mtid >> 6), sharers = bcast0(j.sharers), index = bcast0(j.index), limit = bcast0(j.limit), jbytes = bcast0(j.bytes);
        const bool fresh = bcast0(j.fresh) != 0;
        Rows rows;
        rows.ctr = (GLOBAL_AS uint32_t*)(uint32_t*)bcast64((uint32_t)j.draw, (uint32_t)(j.draw >> 32));
        rows.waves = sharers * DFX_FOLD_WAVES;
        rows.left = limit ? limit : 0xffffffffu;
        rows.drawn = 0;
        rows.begin(fresh, wave * sharers + index);
        Span sp;
        sp.head = bcast0(j.head); sp.end = sp.head + ((jbytes - sp.head) & ~15u);
        const bool front = fresh && index + 1 == sharers && wave + 1 == DFX_FOLD_WAVES, tail = sp.end < jbytes && fresh && index == 0 && wave == 0;
        sp.ends_at = front ? 0u : sp.end;
        sp.ends = front ? sp.head : tail ? jbytes : 0u;
        fold_dispatch((int)bcast0((uint32_t)j.dtype), sh.tab_src[seen & 1], bcast0(j.nsrc), sh.tab_dst[seen & 1], bcast0(j.ndst), sp, rows, lane);
      }
      else if (__builtin_expect(bcast0(j.gang) != 0, 0)) {
        // the waves take a gang's collectives in turn, and count the steps finished one by one
        const uint32_t gang = bcast0(j.gang), R = bcast0(a.R), sh_r = gang_shift(R);
        for (uint32_t e = bcast0(mtid >> 6); e < gang; e += DFX_FOLD_WAVES) {
          const GangEntry& c = sh.gang[seen & 1][e];
          gang_move(c, sh.tab_src[seen & 1] + (e << sh_r), sh.tab_dst[seen & 1] + (e << sh_r), R, lane);
          __builtin_amdgcn_s_waitcnt(0);
          if (lane == 0) (void)__hip_atomic_fetch_add(global_ptr((u64*)c.add_one), 1ull, __ATOMIC_RELAXED, SCOPE_AGENT);
        }
      }
      else if (coh) run_prim<AUX_DEVICE, GTHREADS>(j.dtype, j.fin, j.sb, j.rb, j.fout, j.bytes, mtid);
      else run_prim<AUX_CACHED, GTHREADS>(j.dtype, j.fin, j.sb, j.rb, j.fout, j.bytes, mtid);
      // this wave's stores (and loads) have been performed before it counts itself done
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_s_waitcnt(0);
      u64 t1 = 0;
      if (a.trace_on > 1) t1 = wall_clock64();
      uint32_t last = 0;
      if (lane == 0) {
        const uint32_t old = __hip_atomic_fetch_add(&sh.wave_done[seen & 1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
        last = (old + 1 == GTHREADS / 64) ? 1u : 0u;
        if (first_wave && a.trace_on > 1) {
          bump(sh.stat, ST_T_DATA, t1 - t0);
          if (a.trace_on == 3 && trace && j.prim != 0xffu) trace_put(trace, &sh.trace_n, timeline_sample(t0, t1, j.coll, j.prim));   // not the drain step
        }
      }
      if (bcast0(last)) {
        // all waves of the group have drained job `seen`: its data is in memory
        if (lane == 0) {
          const Flight f = sh.fl[seen & 1];
          // Jobs are published in order: a counter raised for job k tells the neighbour that every slice
          // up to k is there, so the job before must have been published (with one group every wave has
          // finished it by now and its publisher is a few instructions away; with two it may still run).
          while (lds_ld(&sh.jobs_done) != seen) __builtin_amdgcn_s_sleep(0);
          if (!coh) fence_release_agent();
          if (f.tail_out) raise_counter(f.tail_out, f.sent_new);
          if (f.head_in) raise_counter(f.head_in, f.recvd_new);
          if (f.add_one) (void)__hip_atomic_fetch_add(global_ptr(f.add_one), 1ull, __ATOMIC_RELAXED, SCOPE_AGENT);
          __hip_atomic_store(&sh.wave_done[seen & 1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (a.trace_on > 1) bump(sh.stat, ST_T_PUB, wall_clock64() - t1);
          lds_st(&sh.jobs_done, seen + 1);
        }
      }
      seen += GROUPS;
    }
  } else {
    // =====================================================================================
    // scheduler wave
    // =====================================================================================
    // What the scheduler reads all the time is made scalar once: a read of the LDS copy is a round trip of a hundred
    // cycles in a chain of dependent instructions, a scalar that has overflowed into a vector register's lanes one instruction.
    const uint32_t R = bcast0(a.R);
    const struct { uint32_t cmax, max_colls, sq_shift, cq_slots, spin_init, spin_min, spin_max, spin_boost, preempt, order_policy, trace_on, fetch_batch, cq_mode, sq_eager, window, sq_local, focus_bytes, scan_min, oneshot, nwg, epoch; u64 watchdog_ticks, quit_ticks; } hot = {
      bcast0(a.cmax), bcast0(a.max_colls), bcast0(a.sq_shift), bcast0(a.cq_slots), bcast0(a.spin_init), bcast0(a.spin_min), bcast0(a.spin_max), bcast0(a.spin_boost), bcast0(a.preempt), bcast0(a.order_policy), bcast0(a.trace_on), bcast0(a.fetch_batch), bcast0(a.cq_mode), bcast0(a.sq_eager), bcast0(a.window), bcast0(a.sq_local), bcast0(a.focus_bytes), bcast0(a.scan_min), bcast0(a.oneshot), bcast0(a.nwg), bcast0(a.epoch),
      bcast64((uint32_t)a.watchdog_ticks, (uint32_t)(a.watchdog_ticks >> 32)), bcast64((uint32_t)a.quit_ticks, (uint32_t)(a.quit_ticks >> 32))};
    u64 last_act = wall_clock64();
    if (hot.trace_on && hot.trace_on < 3) {
      // what one clock read costs (the switch samples contain two of them, the split samples five): 16 in a row
      u64 tc = last_act;
#pragma unroll
      for (int k = 0; k < 16; ++k) tc = wall_clock64();
      if (lane == 0) { bump(sh.stat, ST_T_STAMP, tc - last_act); bump(sh.stat, ST_N_STAMP, 16); }
      last_act = tc;
    }
    bool acted = true, voted = false;
    uint32_t iter = 0, idle = 0, burst = 0;
    bool in_pass = false, pass_progress = false, scanned = false;
    uint32_t nready = 0, rk = 0, pass_bytes = 0;   // readiness list of the pass: length, cursor; bytes posted in the pass
    // Gangs: so many collectives, and bytes of a share, at most.  A threshold of one poll
    // says that a wait nobody can expect to succeed yet may be left unpolled.
    const bool give_way = hot.preempt && hot.spin_min <= 1u;
    const uint32_t gang_sh = gang_shift(R), gang_n = (64u >> gang_sh) < GANG_MAX ? 64u >> gang_sh : GANG_MAX;
    const uint32_t gang_share = !give_way || R < 2u || R > 32u ? 0u : GANG_SHARE;
    bool focus = false;                            // the pass visits the list furthest-along first, up to a byte budget
    uint32_t pos = 0;
    // context-switch sample in flight: t0 = abort decision, ts = after the save, lb/le = load
    u64 sw_t0 = 0, sw_ts = 0, sw_lb = 0, sw_le = 0;
    bool sw_pending = false;
    // The collective in hand.  Its static context stays in the LDS slot and is read where it is
    // needed (few values live across a wait); the dynamic part is in registers.  sent / recvd
    // count the slots this workgroup has CLAIMED (posted to the movers), which may run ahead
    // of the counters in memory by the jobs in flight.
    bool have = false;
    uint32_t coll = 0, sl = 0;
    uint32_t g = 0, p = 0, cidx = 0;
    u64 sent = 0, recvd = 0, thr = 0;
    bool progressed = false;
    u64 prev_recv = 0, prev_send = 0;   // the previous rank's recv / send buffer (direct steps), 0 = not read yet
    uint32_t posted = 0, retired = 0;   // jobs handed to the movers / jobs whose bookkeeping is done

    // ---- completion of this workgroup's share of an invocation (Sec. 5): completion counter,
    // and the last channel posts the CQE.  Lane 0 only.
    // in_memory: every byte of the result went to memory with sc1 stores that have been acknowledged (fold steps):
    // there is nothing to write back before the counter and the CQE.  On one channel that is 1 us less; with 32 workgroups
    // of an XCD writing back the same L2, the completion and the fetch without write-backs and invalidates took sixteen
    // disordered 25 MiB buckets from 1794 to 1422 us and one 8 KiB all-reduce from 25 to 20.7 us.
    auto complete = [&](uint32_t c_coll, uint32_t c_seq, uint32_t c_nchan, bool in_memory) {
      if (!in_memory) fence_release_system();   // results in the recv buffer are visible to host and later kernels
      GLOBAL_AS uint32_t* dc = global_ptr(&a.done_cnt[(size_t)rank * hot.max_colls + c_coll]);
      // (one channel, or channel 0 for all of them in fold steps: nobody to count with, no round trip for the counter)
      uint32_t old = 0;
      if (c_nchan > 1) old = __hip_atomic_fetch_add(dc, 1u, __ATOMIC_ACQ_REL, SCOPE_AGENT);
      // (the counter runs on from invocation to invocation, modulo 2^32: no reset that the next one's counts could overtake)
      if (c_nchan == 1 || old + 1 == (c_seq + 1u) * c_nchan) {
        const u64 tq0 = wall_clock64();
        if (hot.cq_mode == 0) {
          // optimized CQ (Sec. 5: the id in one atomic write, no ring semantics): id and invocation in one posted 8-byte
          // write into the id's own slot.  At most one invocation of an id is outstanding on a rank, and the host has taken
          // the one before when it submits the next, so the slot is free and belongs to this workgroup: nothing to find, to
          // wait for or to write back.  (Relaxed: what the entry vouches for is in memory, by the fence above or to begin with.)
          // The CAS into a slot that was looked for was a round trip to host memory each, 17.6 of them per us over all
          // workgroups at most, and 1024 small all-reduces on eight ranks took 668 -> 537 us by it, one of 8 KiB 17.5 -> 16.9.
          const u64 v = (1ull << 63) | ((u64)(c_seq & 0x7fffffffu) << 32) | c_coll;
          __hip_atomic_store(global_ptr(&cqbase[c_coll]), v, __ATOMIC_RELAXED, SCOPE_SYSTEM);
        } else {
          // The two ring-buffer CQs that Sec. 5 compares the optimized one with.  Both reserve a
          // position with an atomic in host memory and read the consumer's head to see whether
          // the ring has room.
          u64* ctl = a.cq_ctl + (size_t)rank * DFX_CQ_CTL_WORDS;
          const u64 t = __hip_atomic_fetch_add(&ctl[0], 1ull, __ATOMIC_RELAXED, SCOPE_SYSTEM);
          bool give_up = false;
          uint32_t k = 0;
          while (t - __hip_atomic_load(&ctl[16], __ATOMIC_RELAXED, SCOPE_SYSTEM) >= (u64)hot.cq_slots) {
            if ((++k & 63u) == 0 && (ld_agent32(&a.dev_ctl[DC_ABORT]) || ld_sys32(&a.host_ctl[HC_ABORT]))) { give_up = true; break; }
            __builtin_amdgcn_s_sleep(20);
          }
          if (!give_up && hot.cq_mode == 1) {
            // vanilla ring: entry, fence, then the shared tail, which moves in position order
            const u64 v = ((u64)(c_seq & 0x7fffffffu) << 32) | c_coll;
            __hip_atomic_store(&cqbase[t % hot.cq_slots], v, __ATOMIC_RELAXED, SCOPE_SYSTEM);
            fence_release_system();
            while (__hip_atomic_load(&ctl[8], __ATOMIC_RELAXED, SCOPE_SYSTEM) != t) {
              if ((++k & 63u) == 0 && (ld_agent32(&a.dev_ctl[DC_ABORT]) || ld_sys32(&a.host_ctl[HC_ABORT]))) { give_up = true; break; }
              __builtin_amdgcn_s_sleep(2);
            }
            if (!give_up) __hip_atomic_store(&ctl[8], t + 1, __ATOMIC_RELEASE, SCOPE_SYSTEM);
          } else if (!give_up) {
            // optimized ring: id and position travel in one 64-bit atomic write, no tail, no fence;
            // the poller accepts the entry at its head when the position in it says head + 1
            const u64 v = (((t + 1) & 0xffffffffull) << 32) | ((u64)(c_seq & 0xffffu) << 16) | (c_coll & 0xffffu);
            __hip_atomic_store(&cqbase[t % hot.cq_slots], v, __ATOMIC_RELEASE, SCOPE_SYSTEM);
          }
        }
        bump(sh.stat, ST_T_CQE, wall_clock64() - tq0);
        bump(sh.stat, ST_CQE, 1);
      }
    };

    // ---- retire the jobs the movers have finished (their counters are already raised)
    auto retire_finished = [&]() {
      while (retired != posted && lds_ld(&sh.jobs_done) != retired) {
        if (lane == 0) {
          const Flight f = sh.fl[retired & 1];
          bump(sh.stat, ST_PRIMS, 1);
          if (f.last) complete(f.coll, f.seq, f.nchan, false);
        }
        ++retired;
        acted = true;
      }
    };

    // ---- the last of a rank's workgroups to read an SQ slot frees it (Sec. 5) by writing the entry's generation where
    // the submitter looks for it, in host memory.  The answer of a lone entry's reader counter is looked at when the
    // next wait's first poll is back (it is then there already), not waited for before the entry is worked on.
    uint32_t rd_old = 0;       // lane 0: readers of the slot before this workgroup
    u64 rd_idx = 0;            // the entry
    bool rd_open = false;
    uint32_t peers_of = 0;     // the collective (id + 1) whose buffers are in sh.peer
    bool ctx_open = false;     // the stores of a lone collective's context may still be under way
    auto free_slot = [&](uint32_t readers_before, u64 idx) {
      // (the counter runs on from generation to generation, modulo 2^32: no reset to wait for before the slot is used again)
      const uint32_t gen = (uint32_t)(idx >> hot.sq_shift) + 1u;
      if (readers_before + 1 == gen * hot.cmax)
        __hip_atomic_store(global_ptr(&a.sq_freed[(size_t)rank * D + (idx & (D - 1))]), gen, __ATOMIC_RELAXED, SCOPE_SYSTEM);
    };
    auto settle_slot = [&]() {
      if (rd_open) { if (lane == 0) free_slot(rd_old, rd_idx); rd_open = false; }
      if (ctx_open) { __builtin_amdgcn_s_waitcnt(0); ctx_open = false; }
    };

    // ---- FetchSQE, the parts of it: is the entry there, its words (system scope throughout: nothing of an SQ slot is ever taken
    // from a cache); an entry of this workgroup's taken into its contexts; where it goes in the queue
    auto entry_there = [&](u64 idx) -> bool { return ld_sys32(&sqbase[idx & (D - 1)].e.ready) == (uint32_t)(idx >> hot.sq_shift) + 1u; };
    auto load_entry = [&](u64 idx) -> DfxStatic {
      struct { u64 w[sizeof(DfxStatic) / 8]; } qw;
      const u64* const src = (const u64*)&sqbase[idx & (D - 1)].e;
#pragma unroll
      for (int i = 0; i < (int)(sizeof(DfxStatic) / 8); ++i) qw.w[i] = ld_sys64(src + i);
      return __builtin_bit_cast(DfxStatic, qw);
    };
    auto take_entry = [&](const DfxStatic& q, uint32_t vch, uint32_t round, uint32_t prim, bool lone) {
      // cook the static context of this invocation into the context buffer (addresses
      // resolved once, here); restart the sequence, keep the monotone connector counters
      const DfxCooked k = cook_sqe(q, a.pool, rank, R, vch);
      // direct and fold steps: other ranks read this rank's send buffer and read or write its recv buffer; their
      // addresses and the invocation they belong to go into the rank's line (two 16-byte device-coherent
      // stores, each with its tag; complete before any job of an invocation with direct steps is posted)
      if (q.flags & DFX_SQE_DIRECT)
      {
        const Slot<AUX_DEVICE> line((const void*)k.flags_out, DFX_FLAG_STRIDE);
        line.st16(DFX_DIRECT_OFF, uint4{(uint32_t)q.recvbuf, (uint32_t)(q.recvbuf >> 32), q.seq + 1u, 0u});
        line.st16(DFX_DIRECT_OFF + 16, uint4{(uint32_t)q.sendbuf, (uint32_t)(q.sendbuf >> 32), q.seq + 1u, 0u});
      }
      // rows to be drawn: the counter of the next invocation starts over (nobody draws from it: every rank has
      // finished the invocation before this one, or this rank would not have been given this one)
      if ((q.flags & DFX_SQE_DRAWN) && vch == 0)
        __hip_atomic_store(global_ptr((uint32_t*)(k.flags_out + DFX_FOLD_DRAW + 8u * ((q.seq + 1u) & 1u))), 0u, __ATOMIC_RELAXED, SCOPE_AGENT);
      // fold steps: the channel's count of published invocations, a hint for the readiness scans
      if (q.flags & DFX_SQE_FOLD) (void)__hip_atomic_fetch_add(global_ptr((u64*)(k.flags_in + DFX_FOLD_PUB)), 1ull, __ATOMIC_RELAXED, SCOPE_AGENT);
      const uint32_t c_id = q.coll_id, csl = ctx_slot(c_id);
      if (lone) {
        DfxDyn d; d.round = round; d.prim = prim; d.sent = 0; d.recvd = 0; d.preempted = 0; d.cidx = 0;   // (no connectors: nothing to keep)
        sh.slot[csl].st = k; sh.slot[csl].dyn = d;
        sh.slot_tag[csl] = c_id;
      } else if (sh.slot_tag[csl] == c_id) sh.slot_tag[csl] = 0xffffffffu;
      st_ctx(&myctx[c_id].st, k);
      GLOBAL_AS DfxDyn* dy = global_ptr(&myctx[c_id].dyn);
      dy->round = round; dy->prim = prim; dy->preempted = 0;
      dy->cidx = first_chunk(q.kind, rank, R);
    };
    // The entries of `m`, each in its lane, join the task queue in SQ order.
    auto join_queue = [&](u64 m, uint32_t id_new, int pr) {
      const bool mine = (m >> lane & 1u) != 0;
      if (__builtin_expect(hot.order_policy == 1, 0)) {
        // Priority ordering: the queue stays sorted, an entry behind those of higher or equal priority (64 at once: one by one, a
        // fetch each, 1024 entries took 3.4 ms, longer than the collectives they described).  From the back of the queue on, 64
        // entries at a time, every queued one moves up by the number of new ones that go before it.
        uint32_t at = 0;                 // (of a new one: queued entries and new ones before it)
        for (u64 t = m; t; t &= t - 1) {
          const uint32_t b = (uint32_t)__builtin_ctzll(t);
          const int pb = __builtin_amdgcn_readlane(pr, b);
          at += (pb > pr || (pb == pr && b < lane)) ? 1u : 0u;
        }
        for (uint32_t base = (qlen + 63u) & ~63u; m && base; ) {
          base -= 64u;
          const uint32_t i = base + lane;
          const bool old = i < qlen;
          uint16_t id = 0;
          int po = 0;
          if (old) { id = sh.taskq[i]; po = *(const GLOBAL_AS int16_t*)&myctx[id].st.priority; }
          uint32_t up = 0;
          for (u64 t = m; t; t &= t - 1) {
            const uint32_t b = (uint32_t)__builtin_ctzll(t);
            const int pb = __builtin_amdgcn_readlane(pr, b);
            const uint32_t before = (uint32_t)__builtin_popcountll(__ballot(old && po >= pb));
            if (lane == b) at += before;
            up += pb > po ? 1u : 0u;
          }
          __builtin_amdgcn_wave_barrier();
          if (old) sh.taskq[i + up] = id;
          __builtin_amdgcn_wave_barrier();
        }
        if (mine) sh.taskq[at] = (uint16_t)id_new;
      } else if (mine) sh.taskq[qlen + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull))] = (uint16_t)id_new;
    };

    // ---- a step with data of a collective in fold steps goes to the movers; lane k holds the buffers of entry k's rank
    struct FoldStep { int kind, dtype; uint32_t coll, seq, nchan, vch, limit, fresh; u64 line0, counters; bool drawn, sweep; uint32_t g, longest; u64 total; };
    auto post_fold = [&](const FoldStep& st, const FoldGeom& fg, u64 sendbuf, u64 recvbuf) {
      const bool copies = fold_copies(st.kind), to_all = fold_to_all(st.kind);
      const uint32_t fs = posted & 1;
      if (__builtin_expect(st.sweep, 0)) {      // whole buffers, every rank's
        if (lane < R) { sh.tab_src[fs][lane] = sendbuf; sh.tab_dst[fs][lane] = recvbuf; }
        if (lane == 0) {
          SweepJob sj;
          sj.kind = (uint32_t)st.kind; sj.R = R; sj.rank = rank; sj.longest = st.longest; sj.pad = 0;
          sj.at = st.g * st.limit * st.nchan * DFX_FOLD_WAVES;
          sj.total = st.total;
          sh.sweep[fs] = sj;
        }
      } else if (lane < R) {
        const u64 src = sendbuf + fg.src, dst = recvbuf + fg.dst;
        if (!copies) sh.tab_src[fs][lane] = src;
        else if (lane + 1 == R) sh.tab_src[fs][0] = src;
        if (to_all) sh.tab_dst[fs][lane] = dst;
        else if (lane + 1 == R) sh.tab_dst[fs][0] = dst;
      }
      __builtin_amdgcn_wave_barrier();
      if (lane == 0) {
        Job j;
        j.fin = nullptr; j.fout = nullptr; j.sb = nullptr; j.rb = nullptr;
        j.bytes = fg.bytes; j.head = fold_head(fg.dst, fg.bytes, st.nchan); j.index = st.vch; j.sharers = st.nchan;
        j.limit = st.limit;
        j.fresh = st.fresh; j.gang = 0;
        j.draw = st.drawn ? fold_draw_word(st.line0, rank, st.vch, st.nchan, st.seq) : 0;
        j.nsrc = copies ? 1u : R; j.ndst = to_all ? R : 1u;
        j.dtype = st.dtype; j.coll = st.coll; j.prim = 0;
        sh.job[fs] = j;
        Flight f;
        f.tail_out = nullptr; f.head_in = nullptr; f.sent_new = 0; f.recvd_new = 0;
        f.last = 0; f.coll = st.coll; f.seq = st.seq; f.nchan = st.nchan;
        f.add_one = (u64*)st.counters + DFX_FOLD_RED / 8;
        sh.fl[fs] = f;
        lds_st(&sh.job_seq, posted + 1);
      }
      ++posted;
    };

    // The movers wait for nothing but their own memory operations, so the loops below that wait
    // for them end on their own; they still look at the abort words now and then, so that the
    // host can always get the grid back.
    uint32_t spins = 0;
    auto abort_seen = [&]() -> bool {
      uint32_t s = 0;
      if (lane == 0) s = (ld_agent32(&a.dev_ctl[DC_ABORT]) || ld_sys32(&a.host_ctl[HC_ABORT])) ? 1u : 0u;
      return bcast0(s) != 0;
    };
    // a flight slot: at most two jobs are posted and not yet retired
    auto flight_free = [&](uint32_t depth) -> bool {
      while (posted - retired >= depth) {
        retire_finished();
        if (posted - retired >= depth) {
          if ((++spins & 0xffffu) == 0 && abort_seen()) return false;
          __builtin_amdgcn_s_sleep(1);
        }
      }
      return true;
    };

    for (;;) {
      retire_finished();
      if (stop != STOP_NONE) {
        settle_slot();
        // leaving: the posted jobs run to their end first (their slots are claimed in the saved contexts)
        if (retired == posted) break;
        if ((++spins & 0xffffu) == 0 && abort_seen()) break;
        __builtin_amdgcn_s_sleep(1);
        continue;
      }

      // ================= no collective in hand: control check, fetch, next queue entry =================
      if (!have) {
        if (!in_pass) {
          settle_slot();
          ++iter;
          uint32_t s = STOP_NONE, got = 0;
          // The SQ is probed before every pass.  (Sec. 4.3 has FIFO ordering fetch only when the queue
          // is empty or stuck and priority ordering before every pass.  Here the probe rides along
          // with the control words and costs nothing, new entries join the queue's tail either way,
          // and a workgroup that kept working without reading the SQ held back its rank's SQ slots
          // -- every workgroup must read every SQE -- and with them the submitter and the rest of
          // the grid.)  A fetch is followed by further fetches, up to fetch_batch in a row.
          const bool want = (hot.sq_eager && burst < hot.fetch_batch) || (qlen == 0) || !pass_progress || hot.order_policy == 1 || (burst > 0 && burst < hot.fetch_batch);
          const bool probe = want && qlen < hot.max_colls;
          const bool slow = ((iter & 31u) == 0) || qlen == 0 || !pass_progress;
          const bool host_look = ((iter & 31u) == 0) || qlen == 0;
          // the three control words live in different memories; three lanes fetch them at once
          uint32_t w0 = 0, w1 = 0;
          if (lane == 0) {
            const u64 c2 = ld_agent64((const u64*)&a.dev_ctl[DC_ABORT]);   // abort | quit
            w0 = (uint32_t)c2; w1 = (uint32_t)(c2 >> 32);
          } else if (lane == 1) {
            if (probe) {
              const u64 sr = ld_sys64((const u64*)&sqbase[ri & (D - 1)].e.share);        // share | generation
              w0 = (uint32_t)(sr >> 32); w1 = (uint32_t)sr;
            }
          } else if (lane == 2) {
            if (host_look) w0 = ld_sys32(&a.host_ctl[HC_ABORT]);
          }
          const uint32_t c_abort = __builtin_amdgcn_readlane(w0, 0), c_quit = __builtin_amdgcn_readlane(w1, 0);
          const uint32_t c_ready = __builtin_amdgcn_readlane(w0, 1), c_habort = __builtin_amdgcn_readlane(w0, 2);
          const bool with_table = (__builtin_amdgcn_readlane(w1, 1) & DFX_SHARE_PEERS) != 0;      // (of an entry that is there)
          if (c_abort || c_habort) s = STOP_ABORT;
          else if (c_quit) s = STOP_QUIT;
          if (lane == 0) {
            if (!s && slow) {
              const u64 now = wall_clock64();
              if (acted) { last_act = now; acted = false; }
              if (hot.watchdog_ticks && qlen > 0 && now - last_act > hot.watchdog_ticks) {
                ws->dbg[0] = ((u64)sh.taskq[0] << 32) | qlen; ws->dbg[1] = ri; ws->dbg[2] = now - last_act;
                raise_error(a, 1u, wg);
                s = STOP_ABORT;
              } else if (hot.oneshot) {
                // A launch that brings all of its work with it: this workgroup is through when it has read every
                // entry of its rank's SQ, its queue is empty and its jobs are retired (completions posted).  Nobody waits
                // for it any more, so it leaves on its own; the last one to count itself out knows that everybody is
                // through and writes the outcome (an error has been written by the workgroup that raised it, which
                // does not count itself out).
                if (qlen == 0 && ri >= (u64)hot.oneshot && retired == posted) {
                  __builtin_amdgcn_s_waitcnt(0);      // (its completion is in the CQ before it counts itself out)
                  if (__hip_atomic_fetch_add(&a.dev_ctl[DC_VOTES], 1u, __ATOMIC_RELAXED, SCOPE_AGENT) + 1 == hot.nwg && a.status) {
                    uint32_t n = 0;
                    for (uint32_t i = 0; i < R * hot.cq_slots; ++i) n += (uint32_t)(ld_sys64(&a.cq[i]) >> 63);
                    __hip_atomic_store(a.status, n == R ? 0u : 0x200u, __ATOMIC_RELAXED, SCOPE_AGENT);
                  }
                  s = STOP_EXIT;
                }
              } else if (hot.quit_ticks) {
                // Voluntary quit (Sec. 4.4).  Every workgroup has duties towards the others (each
                // must read every SQE of its rank before the slot is reusable), so the grid leaves
                // as a whole: a workgroup that has been idle or stuck for the quit period casts a
                // vote and keeps running; it withdraws the vote when it becomes active again; the
                // vote that completes the set raises the quit flag, which everybody obeys.
                const bool tired = now - last_act > hot.quit_ticks;
                if (tired && !voted) {
                  voted = true;
                  if (__hip_atomic_fetch_add(&a.dev_ctl[DC_VOTES], 1u, __ATOMIC_ACQ_REL, SCOPE_AGENT) + 1 == hot.nwg) {
                    __hip_atomic_store(&a.dev_ctl[DC_QUIT], 1u, __ATOMIC_RELEASE, SCOPE_AGENT);
                    s = STOP_QUIT;
                  }
                } else if (!tired && voted) {
                  voted = false;
                  __hip_atomic_fetch_sub(&a.dev_ctl[DC_VOTES], 1u, __ATOMIC_ACQ_REL, SCOPE_AGENT);
                }
              }
            }
            if (!s && probe) {
              const uint32_t gen = (uint32_t)(ri >> hot.sq_shift) + 1u;
              if (c_ready == gen) got = 1;
            }
          }
          s = bcast0(s);
          got = bcast0(got);
          if (s) { stop = s; continue; }

          // ---- FetchSQE (Alg. 1 line 2), up to 64 entries at a time: one per lane.
          // Every workgroup of a rank reads every SQE of the rank (Sec. 5), so a burst of a thousand
          // submissions is a thousand entries for each of them, most of them for other channels;
          // taken one by one (a fence, six loads, an atomic with its answer) they cost more than
          // the collectives they describe.
          if (got) {
            const u64 tf0 = wall_clock64();
            // how many consecutive entries from the read index on are there?
            uint32_t room = hot.max_colls - qlen;
            if (room > 64) room = 64;
            const uint32_t left = burst < hot.fetch_batch ? hot.fetch_batch - burst : 1u;
            if (left < room) room = left;
            // Lane 0's entry has been seen by the control check: its words are loaded while the lanes behind it look
            // whether theirs are there.  System scope throughout: nothing of an SQ slot is ever taken from a cache.
            bool here = lane == 0;
            DfxStatic q = {};
            // (the table of buffers that lane 0's entry may come with, lane k its entry k)
            uint4 peer = uint4{0, 0, 0, 0};
            if (with_table && lane < R) {
              const u64* const t = (const u64*)(known_global(a.sq_peers) + ((size_t)rank * D + (ri & (D - 1))) * R + lane);
              const u64 t0 = ld_sys64(t), t1 = ld_sys64(t + 1);
              peer = uint4{(uint32_t)t0, (uint32_t)(t0 >> 32), (uint32_t)t1, (uint32_t)(t1 >> 32)};
            }
            if (lane == 0) q = load_entry(ri);
            else if (lane < room) here = entry_there(ri + lane);
            const u64 here_mask = __ballot(here);
            uint32_t n = (here_mask == ~0ull) ? 64u : (uint32_t)__builtin_ctzll(~here_mask);   // length of the run that starts at lane 0
            if (lane != 0 && lane < n) q = load_entry(ri + lane);
            // (a full look: the run may go on, see below)
            const bool chain = n == 64u && hot.fetch_batch == 0xffffffffu && run_goes_on(D, (uint32_t)sizeof(DfxSqSlot));
            bool more = chain && entry_there(ri + 64u + lane);
            __builtin_amdgcn_s_waitcnt(0);        // (the entries have been read before they count as read below)
            bool is_exit_sqe = false, is_exit = false;
            if (lane < n) {
              // an exit SQE ends the launch it was posted for; one left over from an earlier launch
              // (some workgroups had already gone when it arrived) is consumed and ignored
              is_exit_sqe = (q.flags & DFX_SQE_EXIT) != 0;
              is_exit = is_exit_sqe && q.seq == hot.epoch;
            }
            u64 exit_mask = __ballot(is_exit);
            if (exit_mask) n = (uint32_t)__builtin_ctzll(exit_mask) + 1;   // nothing behind an exit SQE is touched
            bool mine = false;
            uint32_t c_id = 0, my_vch = 0;
            if (lane < n) {
              c_id = q.coll_id;
              my_vch = is_exit_sqe ? ch : serving_channel(ch, hot.cmax, q.start);
              mine = !is_exit_sqe && my_vch < q.nchan && c_id < hot.max_colls;
            }
            const bool q_fold = (q.flags & DFX_SQE_FOLD) != 0;
            // the submitter wrote the send buffers before the SQEs: drop what this CU / XCD cached (fold steps read
            // them with loads that bypass the caches)
            if (__ballot(mine && !q_fold)) fence_acquire_system();
            const u64 mine_mask = __ballot(mine);
            // A lone collective in fold steps is what a latency-bound caller waits for: its context goes straight into
            // its LDS slot as well, and nothing waits for the copy in memory.
            const bool lone = mine_mask != 0 && (mine_mask & (mine_mask - 1)) == 0 && __ballot(mine && q_fold) != 0;
            // Such an entry with all ranks' buffers, and nothing else to do: its first step with data goes to the movers at once, straight
            // from the entry; the context and what the other ranks may want to see follow while the data moves.  (By way of the
            // context, the pass over the queue and the other ranks' lines the job was posted 3.4 us later: all-reduce of 8 KiB 16.9 ->
            // 15.0, 1 MiB bf16 22.1 -> 19.6, 25 MiB bf16 97.8 -> 93.8, reduce of 4 MiB on four ranks 19.4 -> 16.6.)  The table serves the invocation's further jobs until another fetch.
            peers_of = 0;
            uint32_t first_round = 0, first_prim = 0;      // where the invocation's walk goes on
            bool through = false;                          // ... nowhere: it needs no place in the queue
            if (lone && with_table && mine_mask == 1ull) {
              peers_of = bcast0(c_id) + 1u;
              if (lane == 0) sh.peers_seq = q.seq;
              if (qlen == 0 && posted == retired) {
                const uint32_t e_rounds = bcast0(q.rounds), e_flags = bcast0(q.flags), e_nchan = bcast0(q.nchan), e_vch = bcast0(my_vch);
                const bool e_drawn = (e_flags & DFX_SQE_DRAWN) != 0;
                const FoldGeom fg = fold_geometry(bcast64((uint32_t)q.count, (uint32_t)(q.count >> 32)), bcast64((uint32_t)q.block_elems, (uint32_t)(q.block_elems >> 32)),
                                                  bcast64((uint32_t)q.part_elems, (uint32_t)(q.part_elems >> 32)), bcast0(q.slice_elems), e_drawn, 0);
                const u64 line0 = (u64)(uintptr_t)a.pool + bcast64((uint32_t)q.conn_off, (uint32_t)(q.conn_off >> 32)) + (u64)e_vch * DFX_FLAG_STRIDE;
                const bool e_sweep = (e_flags & DFX_SQE_SWEEP) != 0;
                const FoldStep st = {(int)bcast0(q.kind), (int)bcast0((uint32_t)q.dtype | ((uint32_t)q.op << 4)), peers_of - 1u, bcast0(q.seq), e_nchan, e_vch,
                                     e_sweep ? bcast0(q.slice_elems) : bcast0(q.slot_bytes), e_sweep ? FRESH_SWEEP | 1u : 1u, line0, fold_line(line0, 0, R, e_nchan), e_drawn,
                                     e_sweep, 0, bcast0((uint32_t)q.count), bcast64((uint32_t)q.block_elems, (uint32_t)(q.block_elems >> 32))};
                post_fold(st, fg, ((u64)peer.y << 32) | peer.x, ((u64)peer.w << 32) | peer.z);
                const SeqPos nx = next_fold_position(e_rounds, e_vch, 0, 0, 0);
                through = nx.g >= e_rounds;
                first_round = nx.g; first_prim = nx.p;
              }
              sh.peer[lane] = peer;
            }
            if (mine) {
              take_entry(q, my_vch, first_round, first_prim, lone);
            }
            // every workgroup of the rank reads every SQE; the last reader frees the slot (relaxed: the entries have been
            // read, and nothing else hangs on the counter)
            if (lane < n) {
              const uint32_t old = __hip_atomic_fetch_add(global_ptr(&a.sq_readers[(size_t)rank * D + ((ri + lane) & (D - 1))]), 1u, __ATOMIC_RELAXED, SCOPE_AGENT);
              if (n == 1) rd_old = old;
              else free_slot(old, ri + lane);
            }
            if (n == 1) { rd_open = true; rd_idx = ri; }
            // (contexts and published buffer addresses are in memory before anything is built on them)
            if (lone) ctx_open = true;
            else __builtin_amdgcn_s_waitcnt(0);
            // the entries that are this workgroup's join the task queue in SQ order
            if (!through) join_queue(mine_mask, c_id, q.priority);
            if (!through) qlen += (uint32_t)__builtin_popcountll(mine_mask);
            uint32_t taken = n;
            // ---- The run goes on: 64 entries a round trip.  Every workgroup reads every entry of its rank, most of them for others: those
            // are read only as far as says whose they are (the second half; whole, 64 entries were 4 us of traffic past the caches that 32
            // workgroups of an XCD shared).  While a batch's own entries travel, so do the halves of the next and the
            // generation words of the one behind it; the reader counters' answers are looked at a batch later.  1024 entries: 66 us, now 29.
            if (chain && !exit_mask) {
              const __amdgpu_buffer_rsrc_t ring = __builtin_amdgcn_make_buffer_rsrc(sqbase, 0, (int)(D * (uint32_t)sizeof(DfxSqSlot)), 0x00020000);
              auto half = [&](u64 idx, uint32_t at) -> uint4 {
                return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ring, (int)(((uint32_t)idx & (D - 1)) * (uint32_t)sizeof(DfxSqSlot) + at), 0, AUX_SYSTEM));
              };
              auto run_length = [&](bool there) -> uint32_t {
                const u64 m = __ballot(there);
                return m == ~0ull ? 64u : (uint32_t)__builtin_ctzll(~m);
              };
              u64 at = ri + 64u;                  // the batch in hand
              uint32_t m = run_length(more), old = 0, old_n = 0;
              uint4 h0 = uint4{0, 0, 0, 0}, h1 = h0;
              asm volatile("" ::: "memory");      // (nothing of an entry is read before its generation word has been)
              if (lane < m) { h0 = half(at + lane, 64u); h1 = half(at + lane, 80u); }
              more = m == 64u && entry_there(at + 64u + lane);
              // (after 16 of them, 30 us, the control words are looked at again)
              for (uint32_t batch = 0; batch < 16u && m && hot.max_colls - qlen >= 64u && !exit_mask; ++batch) {
                struct { uint4 w[6]; } w = {};
                w.w[4] = h0; w.w[5] = h1;
                DfxStatic e = __builtin_bit_cast(DfxStatic, w);
                const uint32_t e_vch = serving_channel(ch, hot.cmax, e.start);
                const bool e_exit = lane < m && (e.flags & DFX_SQE_EXIT) != 0;
                const bool wanted = lane < m && (e_exit || e_vch < e.nchan);
                const uint32_t mn = run_length(more);
                asm volatile("" ::: "memory");
                if (wanted) {
#pragma unroll
                  for (uint32_t i = 0; i < 4u; ++i) w.w[i] = half(at + lane, i * 16u);
                }
                if (lane < mn) { h0 = half(at + 64u + lane, 64u); h1 = half(at + 64u + lane, 80u); }
                more = mn == 64u && entry_there(at + 128u + lane);
                __builtin_amdgcn_s_waitcnt(0);        // (as above; all of these travel together)
                if (wanted) e = __builtin_bit_cast(DfxStatic, w);
                exit_mask = __ballot(e_exit && e.seq == hot.epoch);
                if (exit_mask) m = (uint32_t)__builtin_ctzll(exit_mask) + 1u;
                const bool own = lane < m && wanted && !e_exit && e.coll_id < hot.max_colls;
                const u64 own_mask = __ballot(own);
                if (__ballot(own && !(e.flags & DFX_SQE_FOLD))) fence_acquire_system();
                if (own) take_entry(e, e_vch, 0u, 0u, false);
                if (lane < old_n) free_slot(old, at - 64u + lane);
                old_n = m;
                if (lane < m) old = __hip_atomic_fetch_add(global_ptr(&a.sq_readers[(size_t)rank * D + ((at + lane) & (D - 1))]), 1u, __ATOMIC_RELAXED, SCOPE_AGENT);
                if (hot.order_policy == 1) __builtin_amdgcn_s_waitcnt(0);      // (the queue's order is read from the contexts)
                join_queue(own_mask, e.coll_id, e.priority);
                qlen += (uint32_t)__builtin_popcountll(own_mask);
                taken += m;
                at += m;
                m = exit_mask ? 0u : mn;
                retire_finished();
              }
              if (lane < old_n) free_slot(old, at - old_n + lane);
              __builtin_amdgcn_s_waitcnt(0);
            }
            if (lane == 0) {
              bump(sh.stat, ST_SQE, taken);
              if (taken != n) bump(sh.stat, ST_RUN_ON, taken - n);
              bump(sh.stat, ST_T_SQE, wall_clock64() - tf0);
              __hip_atomic_fetch_max(&sh.stat[ST_MAXQ], (u64)qlen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __builtin_amdgcn_wave_barrier();
            acted = true;
            sw_pending = false;
            ri += taken;
            if (exit_mask) {
              // the whole grid leaves (every workgroup has reader duties towards its rank's SQ)
              if (lane == 0) __hip_atomic_store(&a.dev_ctl[DC_QUIT], 1u, __ATOMIC_RELEASE, SCOPE_AGENT);
              stop = STOP_EXIT;
              continue;
            }
            burst += taken;
            idle = 0;
            if (n == room) continue;   // the run may go on: probe the SQ again before walking the queue
            // (fewer entries than lanes looked: the SQ is empty behind them, go on to the pass)
          }
          burst = 0;
          if (qlen == 0) {
            // idle: back off the SQ probe (an SQ in host memory is probed across PCIe: back off further)
            ++idle;
            if (idle < 64) __builtin_amdgcn_s_sleep(8);
            else if (hot.sq_local || idle < 4096) __builtin_amdgcn_s_sleep(32);
            else __builtin_amdgcn_s_sleep(127);
            continue;
          }
          idle = 0;
          // ---- start one pass over the task queue (Alg. 1 lines 4-19)
          in_pass = true;
          pass_progress = false;
          pos = 0;
          if (lane == 0) bump(sh.stat, ST_PASSES, 1);
          // ---- readiness scan: 64 queue entries per step, one per lane.  Each lane reads the
          // saved context of its entry, works out which connector sides its next primitive
          // needs, loads those counters and votes; the runnable positions are compacted into a
          // list (ballot + popcount) and the pass visits only those.  The conditions are
          // monotone: only this workgroup consumes its recv side and fills its send side, so
          // "ready" stays true until it acts.  A queue of a thousand stuck collectives costs
          // sixteen memory round trips instead of a thousand context loads and bounded spins.
          scanned = hot.scan_min && qlen >= hot.scan_min;
          if (scanned) {
            settle_slot();     // (the scan reads the contexts in memory)
            nready = 0; rk = 0; pass_bytes = 0;
            uint32_t kept = 0, nshort = 0;       // entries that stay in the queue; runnable short ones
            focus = hot.focus_bytes != 0 && qlen <= 64u;
            if (lane < DFX_CTX_SLOTS) sh.slot_claim[lane] = 0xffffffffu;
            for (uint32_t base = 0; base < qlen; base += 64) {
              const uint32_t i = base + lane;
              bool rdy = false, short_one = false, over = false;
              uint32_t key = 0;     // 0 = not runnable; else (priority under priority ordering,) primitives done so far, then queue position
              uint32_t cid = 0;
              uint4 e0 = uint4{0, 0, 0, 0}, e1 = e0, e4 = e0, e2c = e0, e3c = e0, e5c = e0, e6c = e0, e7c = e0;
              if (i < qlen) {
                cid = sh.taskq[i];
                const uint4* e = (const uint4*)&myctx[cid];
                e0 = ld_ctx(e); e1 = ld_ctx(e + 1); e4 = ld_ctx(e + 4);   // not needed for the vote, but for the deposit below
                const uint4 fl = ld_ctx(e + 2);    // bytes 32..47: part_elems | flags_out
                const uint4 fi = ld_ctx(e + 3);    // bytes 48..63: flags_in | fifo_out
                const uint4 ge = ld_ctx(e + 5);    // bytes 80..95: seq | nprim,nchan | nslots,kind,dtype,bc_pos | priority,vch
                const uint4 d0 = ld_ctx(e + 6);    // dyn: round | prim | sent
                const uint4 d1 = ld_ctx(e + 7);    // dyn: recvd | preempted | cidx
                e2c = fl; e3c = fi; e5c = ge; e6c = d0; e7c = d1;
                const bool e_fold = ((ge.z >> 24) & DFX_CTX_FOLD) != 0;
                Prim pq = e_fold ? make_fold_prim(d0.y)
                                 : make_prim((int)((ge.z >> 8) & 0xffu), R, (ge.z >> 24) & 3u, d0.y, ((ge.z >> 24) & DFX_CTX_DIRECT) != 0);
                if (!e_fold && ((ge.z >> 24) & DFX_CTX_DIRECT))
                  pq = chain_drain_round(pq, (int)((ge.z >> 8) & 0xffu), true, d0.x, e4.w);   // bytes 64..79: fifo_in | slice_elems | rounds
                const u64 f_out = ((u64)fl.w << 32) | fl.z, f_in = ((u64)fi.y << 32) | fi.x;
                const u64 e_sent = ((u64)d0.w << 32) | d0.z, e_recvd = ((u64)d1.y << 32) | d1.x;
                bool okr = true, oks = true;
                // Fold steps: every rank of the channel has got as far as this step needs (bytes 48..63: shared counters, count at the end).
                // The last wait is for all channels; its own stands for them here: a visit too early is a poll and a switch, 2 % of
                // the visits among 64 mixed collectives, none among 1024 small ones.  All channels' counters looked at here: 64
                // mixed 959 us, then 972, 1024 small 535, then 547.
                if (pq.fold)
                  okr = ld_agent64((const u64*)f_in + pq.fwait) >= (pq.fwait ? ((u64)fi.w << 32) | fi.z : ((u64)ge.x + 1u) * R);
                if (pq.recv) okr = ld_agent64((const u64*)f_in) > e_recvd;
                if (pq.send) oks = (e_sent - ld_agent64((const u64*)f_out + 8)) < (u64)(ge.z & 0xffu);
                else if (pq.drain) oks = e_sent == ld_agent64((const u64*)f_out + 8);
                rdy = okr && oks;
                // A last wait on one channel that the counter has ended: nothing is left but the completion, which the lane posts below.
                over = rdy && pq.fold == 3 && (ge.y >> 16) == 1u && hot.cq_mode == 0;
                if (over) rdy = false;
                // a short collective's one step with data: it may go with others
                short_one = focus && rdy && pq.fold == 1 && e4.w == 1u && !((ge.z >> 24) & (DFX_CTX_DRAWN | DFX_CTX_SWEEP)) && e0.z <= gang_share;
                if (rdy) {
                  // primitives done so far, in the order of the walk: a ring takes its slices in windows (next_position),
                  // so primitive p of the window's second slice comes right behind primitive p of its first
                  const uint32_t wmask = e_fold ? 0u : hot.window - 1u;
                  u64 done = (u64)(d0.x & ~wmask) * (ge.y & 0xffffu) + (u64)d0.y * (wmask + 1u) + (d0.x & wmask);
                  if (hot.order_policy == 1) {
                    // priority ordering (Sec. 4.3): the user's priority decides first, progress and
                    // queue position only among equals
                    if (done > 0xffu) done = 0xffu;
                    const uint32_t pr = (uint32_t)((int)(int16_t)(ge.w & 0xffffu) + 32768);
                    key = ((pr << 14) | ((uint32_t)done << 6) | (63u - lane)) + 1u;
                  } else {
                    key = pass_key(short_one, done, lane);
                  }
                }
              }
              // The contexts of the runnable entries are in registers now: they go into their LDS
              // slots (direct-mapped; of several entries of the scan that share a slot the first one
              // gets it), so that the pass finds them there instead of loading them from HBM again.
              if (rdy) (void)__hip_atomic_fetch_min(&sh.slot_claim[ctx_slot(cid)], ((base >> 6) << 8) | lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
              __builtin_amdgcn_wave_barrier();
              if (rdy && sh.slot_claim[ctx_slot(cid)] == (((base >> 6) << 8) | lane)) {
                uint4* dstc = (uint4*)&sh.slot[ctx_slot(cid)];
                dstc[0] = e0; dstc[1] = e1; dstc[2] = e2c; dstc[3] = e3c; dstc[4] = e4; dstc[5] = e5c; dstc[6] = e6c; dstc[7] = e7c;
                sh.slot_tag[ctx_slot(cid)] = cid;
              }
              const u64 mask = __ballot(rdy), over_mask = __ballot(over);
              // Completions, a lane each: visited one by one, each cost the look-up of its context, a poll and a move of the queue, 3 - 4 us
              // behind the last job of a burst.  The entries left over move together.
              uint32_t now_at = i;
              if (over_mask | (u64)(kept != base)) {
                if (over) {
                  const u64 tq0 = wall_clock64();
                  const u64 v = (1ull << 63) | ((u64)(e5c.x & 0x7fffffffu) << 32) | cid;
                  __hip_atomic_store(global_ptr(&cqbase[cid]), v, __ATOMIC_RELAXED, SCOPE_SYSTEM);
                  if (lane == (uint32_t)__builtin_ctzll(over_mask)) {
                    bump(sh.stat, ST_CQE, __builtin_popcountll(over_mask));
                    bump(sh.stat, ST_PRIMS, __builtin_popcountll(over_mask));
                    bump(sh.stat, ST_T_CQE, wall_clock64() - tq0);
                  }
                }
                const u64 stay = __ballot(i < qlen && !over);
                now_at = kept + (uint32_t)__builtin_popcountll(stay & ((1ull << lane) - 1ull));
                if (i < qlen && !over) sh.taskq[now_at] = (uint16_t)cid;
                kept += (uint32_t)__builtin_popcountll(stay);
              } else kept += qlen - base < 64u ? qlen - base : 64u;
              if (focus) {
                // One step holds the whole queue.  The runnable entries are visited furthest-along
                // first (ties: queue order): every rank ranks them alike, so the ranks settle on
                // the same few collectives and carry those through, instead of moving all of
                // them forward side by side with all of their FIFO slots in use at once.
                uint32_t rank_in_pass = 0;
                const uint32_t nq = qlen < 64u ? qlen : 64u;
                for (uint32_t j = 0; j < nq; ++j)
                  rank_in_pass += ((uint32_t)__builtin_amdgcn_readlane((int)key, (int)j) > key) ? 1u : 0u;
                if (rdy) sh.rlist[rank_in_pass] = (uint16_t)now_at;
                // the short ones: first in the pass; under priority ordering as many as nothing else goes before
                nshort = (uint32_t)__builtin_popcountll(__ballot(short_one));
                if (lane == 0) {
                  const uint32_t others = nshort ? (uint32_t)__builtin_popcountll(mask) - nshort : 0u;      // (among themselves they have their order)
                  sh.nothers = others;
                  sh.turn = 0;
                  if (__builtin_expect(others && hot.order_policy != 1 && turn_due(sh.behind), 0)) sh.turn = nshort + turn_of(sh.turns++, others) + 1u;
                }
                if (hot.order_policy == 1 && nshort) {
                  nshort = 0;
                  for (; __ballot(short_one && rank_in_pass == nshort); ) ++nshort;
                }
                if (short_one) {
                  const FoldGeom fg = fold_geometry(((u64)e1.y << 32) | e1.x, ((u64)e1.w << 32) | e1.z, ((u64)e2c.y << 32) | e2c.x, e4.z, false, 0);
                  GangRun r;
                  r.line0 = ((u64)e4.y << 32) | e4.x; r.counters = ((u64)e3c.y << 32) | e3c.x;
                  r.src = fg.src; r.dst = fg.dst; r.bytes = fg.bytes; r.seq = e5c.x;
                  r.nchan_vch = (e5c.y >> 16) | (e5c.w & 0xffff0000u);
                  r.what = (e5c.z >> 8 & 0xffffu) | (e5c.z & 0xffu) << 16;
                  r.coll = cid; r.pos = now_at; r.share = e0.z; r.pad = 0;
                  sh.run[rank_in_pass] = r;
                }
              } else if (rdy) sh.rlist[nready + (uint32_t)__builtin_popcountll(mask & ((1ull << lane) - 1ull))] = (uint16_t)now_at;
              nready += (uint32_t)__builtin_popcountll(mask);
            }
            __builtin_amdgcn_wave_barrier();
            const bool ended = kept != qlen;
            if (lane == 0) { bump(sh.stat, ST_POLLS, (qlen + 63) / 64); bump(sh.stat, ST_SCAN_SKIPS, kept - nready); }
            qlen = kept;
            if (ended) { acted = true; pass_progress = true; }
            if (nready == 0) {           // nothing can run: the pass is over before it began
              in_pass = false;
              if (!ended) __builtin_amdgcn_s_sleep(4);
              continue;
            }
            // ---- gangs: so many short collectives at a time as their ranks fill the lanes, lane (e, k) the line of entry k's rank of
            // collective e.  One load for all of them says which every rank has published; those go to the movers as one job.
            if (__builtin_expect(nshort >= 2u, 0)) {
              bool ok_all = true;
              if (lane == 0) sh.gone = 0;
              const uint32_t e = lane >> gang_sh, k = lane & ((1u << gang_sh) - 1u);
              while (rk < nshort && pass_bytes < hot.focus_bytes) {
                const uint32_t n = nshort - rk < gang_n ? nshort - rk : gang_n;
                const GangRun g_ = sh.run[rk + (e < n ? e : 0u)];
                // (the first lane of collective e; not known to the compiler to be the same in every pass: it kept three masks made of it, across
                // everything the scheduler does, in scratch memory, where each was a wait of its own)
                uint32_t first = e << gang_sh;
                asm volatile("" : "+v"(first));
                const uint32_t nch = g_.nchan_vch & 0xffffu, vch = g_.nchan_vch >> 16, dt = g_.what >> 8 & 0xffu;
                const int kd = (int)(g_.what & 0xffu);
                v4u ln_recv, ln_send;
                ld_published((const void*)(g_.line0 + (u64)(k < R ? fold_peer(kd, R, rank, g_.what >> 16, k) : 0u) * nch * DFX_FLAG_STRIDE), ln_recv, ln_send);
                const u64 all_lanes = (gang_sh == 6u ? ~0ull : (1ull << (1u << gang_sh)) - 1ull) << first;
                bool there = e < n && (__ballot(e < n && ln_recv.z == g_.seq + 1u && ln_send.z == g_.seq + 1u) & all_lanes) == all_lanes;
                // as many of them as the pass's bytes go for, a bit for the first lane of each: nothing overtakes a job.  (With the budget looked
                // at before a gang only, an urgent 8 KiB all-reduce behind sixty of 4 MiB took 372 us under priority ordering, now 113 (R = 8); behind sixty of 2 MiB
                // 190, now 50 (R = 4), while all sixty take 628 instead of 497.)
                // The shares are summed over the lanes: one after the other sixteen of them cost 0.3 us a gang.
                const bool head = there && k == 0;
                const uint32_t share = head ? g_.share : 0u, upto = wave_sum_upto(share);
                const u64 heads_all = __ballot(head), heads = __ballot(head && gang_takes(pass_bytes + upto - share, share, gang_budget(hot.focus_bytes, hot.order_policy == 1)));
                const uint32_t bytes_of = heads ? (uint32_t)__builtin_amdgcn_readlane((int)upto, 63 - (int)__builtin_clzll(heads)) : 0u;
                const bool full = heads != heads_all;
                there = (heads >> first & 1u) != 0;
                const uint32_t cnt = (uint32_t)__builtin_popcountll(heads);
                rk += n;
                pass_bytes += bytes_of;
                if (full && pass_bytes < hot.focus_bytes) pass_bytes = hot.focus_bytes;      // (the pass ends: the others go with the next one)
                if (!cnt) continue;
                if (!flight_free(hot.order_policy == 1 ? 1u : 2u)) { ok_all = false; break; }
                const uint32_t fs = posted & 1, idx = (uint32_t)__builtin_popcountll(heads & ((1ull << first) - 1ull));
                if (there) {
                  const bool cp = fold_copies(kd), to_all = fold_to_all(kd);
                  if (k < R) {
                    u64* const ts = sh.tab_src[fs] + (idx << gang_sh);
                    u64* const td = sh.tab_dst[fs] + (idx << gang_sh);
                    const u64 src = (((u64)ln_send.y << 32) | ln_send.x) + g_.src, dst = (((u64)ln_recv.y << 32) | ln_recv.x) + g_.dst;
                    if (!cp) ts[k] = src;
                    else if (k + 1 == R) ts[0] = src;
                    if (to_all) td[k] = dst;
                    else if (k + 1 == R) td[0] = dst;
                  }
                  if (k == 0) {
                    const uint32_t nsrc = cp ? 1u : R, ndst = to_all ? R : 1u;
                    u64* const add = (u64*)g_.counters + DFX_FOLD_RED / 8;
                    GangEntry ge;
                    ge.add_one = (u64)add; ge.bytes = g_.bytes; ge.index = vch; ge.sharers = nch; ge.dtype = dt; ge.nsrc = nsrc; ge.ndst = ndst;
                    sh.gang[fs][idx] = ge;
                    if (idx == 0) {            // (a gang of one is an ordinary job)
                      Job j;
                      j.fin = nullptr; j.fout = nullptr; j.sb = nullptr; j.rb = nullptr;
                      j.bytes = g_.bytes; j.head = fold_head(g_.dst, g_.bytes, nch); j.index = vch; j.sharers = nch; j.limit = 0; j.fresh = 1; j.draw = 0;
                      j.nsrc = cnt > 1u ? 0u : nsrc; j.ndst = ndst; j.dtype = (int)dt; j.coll = g_.coll; j.prim = 0;
                      j.gang = cnt > 1u ? cnt : 0u;
                      sh.job[fs] = j;
                      Flight f;
                      f.tail_out = nullptr; f.head_in = nullptr; f.sent_new = 0; f.recvd_new = 0;
                      f.last = 0; f.coll = g_.coll; f.seq = g_.seq; f.nchan = nch;
                      f.add_one = cnt > 1u ? nullptr : add;
                      sh.fl[fs] = f;
                      bump(sh.stat, ST_PRIMS, cnt - 1u);       // (one is counted when the job is retired)
                    }
                    // where its walk goes on: at the last wait (channel 0), or nowhere
                    if (vch == 0) {
                      DfxDyn d; d.round = 0; d.prim = 1; d.sent = 0; d.recvd = 0; d.preempted = 1; d.cidx = 0;
                      const uint32_t gsl = ctx_slot(g_.coll);
                      if (sh.slot_tag[gsl] == g_.coll) sh.slot[gsl].dyn = d;
                      st_ctx(&myctx[g_.coll].dyn, d);
                      bump(sh.stat, ST_PREEMPT, 1); bump(sh.stat, ST_SAVE, 1); bump(sh.stat, ST_UNPOLLED, 1);
                    } else (void)__hip_atomic_fetch_or(&sh.gone, 1ull << g_.pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    bump(sh.stat, ST_HIT, 1);
                  }
                }
                __builtin_amdgcn_wave_barrier();
                if (lane == 0) lds_st(&sh.job_seq, posted + 1);
                ++posted;
                if (lane == 0 && cnt > 1u) {
                  bump(sh.stat, ST_GANGS, 1);
                  bump(sh.stat, ST_GANGED, cnt);
                  __hip_atomic_fetch_max(&sh.stat[ST_GANG_MAX], (u64)bytes_of, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                pass_progress = true;
                acted = true;
              }
              if (!ok_all) { stop = STOP_ABORT; continue; }
              __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
              __builtin_amdgcn_wave_barrier();
              const u64 gone_l = sh.gone;
              const u64 gone = bcast64((uint32_t)gone_l, (uint32_t)(gone_l >> 32));
              if (gone) {
                // (the whole queue is 64 entries at most: the ones left over move together, and so do the places in the list)
                uint16_t id = 0, at = 0;
                if (lane < qlen) id = sh.taskq[lane];
                if (lane < nready) at = sh.rlist[lane];
                __builtin_amdgcn_wave_barrier();
                if (lane < qlen && !(gone >> lane & 1u)) sh.taskq[__builtin_popcountll(~gone & ((1ull << lane) - 1ull))] = id;
                if (lane < nready) sh.rlist[lane] = (uint16_t)__builtin_popcountll(~gone & ((1ull << at) - 1ull));
                qlen -= (uint32_t)__builtin_popcountll(gone);
                __builtin_amdgcn_wave_barrier();
              }
            }
          }
        }
        if (scanned) {
          // (a pass that ends is not a switch between two collectives: the latency sample is dropped)
          // A focused pass also ends once it has handed the movers its share of bytes: the next scan
          // looks again at which collectives are furthest along.
          bool ended = rk >= nready;
          if (!ended && focus && pass_bytes >= hot.focus_bytes) {
            const uint32_t turn = bcast0(sh.turn);
            ended = turn == 0 || rk >= turn || turn > nready;      // (none has, it has been visited, there is none)
            if (!ended) {
              rk = turn - 1u;
              if (lane == 0) sh.turn = 0;
            }
          }
          if (ended) {
            if (focus && lane == 0) sh.behind = passes_over(sh.behind, sh.nothers, rk < nready ? nready - rk : 0u);
            in_pass = false; sw_pending = false;
            continue;
          }
          pos = bcast0((uint32_t)sh.rlist[rk]);
        } else if (pos >= qlen) { in_pass = false; sw_pending = false; continue; }

        // ---- LoadCollectiveContext: HBM context buffer -> LDS slot, 8 lanes x 16 bytes
        coll = bcast0(sh.taskq[pos]);
        sl = ctx_slot(coll);
        if (sw_pending && hot.trace_on > 1) sw_lb = wall_clock64();
        if (sh.slot_tag[sl] != coll) {
          if (lane < 8) ((uint4*)&sh.slot[sl])[lane] = ld_ctx((const uint4*)&myctx[coll] + lane);
          if (lane == 0) { sh.slot_tag[sl] = coll; bump(sh.stat, ST_LOAD, 1); }
          __builtin_amdgcn_wave_barrier();
        } else if (lane == 0) bump(sh.stat, ST_HIT, 1);
        if (sw_pending && hot.trace_on > 1) sw_le = wall_clock64();
        {
          // (every lane reads the same words: into scalar registers, so that what follows branches and counts there)
          const uint4* const y = (const uint4*)&sh.slot[sl].dyn;
          const uint4 y0 = y[0], y1 = y[1];   // round | prim | sent, recvd | preempted | cidx
          g = bcast0(y0.x); p = bcast0(y0.y); sent = bcast64(y0.z, y0.w); recvd = bcast64(y1.x, y1.y); cidx = bcast0(y1.w);
        }
        // SetInitialSpinThreshold (Alg. 1 line 3): largest at the front, halving per position.
        // In a scanned pass every entry visited was seen runnable, and the rest of the list is
        // known work: waiting on one collective would only keep the movers idle, so the
        // threshold stays at its minimum there.
        thr = hot.spin_init >> (pos < 31 ? pos : 31);
        if (thr < hot.spin_min || scanned) thr = hot.spin_min;
        progressed = false;
        prev_recv = 0;
        have = true;
      }

      // ================= next primitive of the collective in hand =================
      // The static context stays in the LDS slot; the words that every step needs are read at once and made scalar.
      const DfxCooked& S = sh.slot[sl].st;
      const uint4* const sv = (const uint4*)&S;
      const uint4 v3 = sv[3], v4 = sv[4], v5 = sv[5];   // flags_in | fifo_out, fifo_in | slice_elems | rounds, seq | nprim,nchan | nslots,kind,dtype,bc_pos | ..
      const u64 s_in = bcast64(v3.x, v3.y), s_fout = bcast64(v3.z, v3.w), s_fin = bcast64(v4.x, v4.y);
      const uint32_t s_slice = bcast0(v4.z), s_rounds = bcast0(v4.w), inv_seq = bcast0(v5.x);
      const uint32_t s_n = bcast0(v5.y), s_k = bcast0(v5.z), inv_nchan = s_n >> 16, K = s_k & 0xffu, bcp = s_k >> 24;   // (K: the root in fold steps)
      const int kind = (int)(s_k >> 8 & 0xffu), dtype = (int)(s_k >> 16 & 0xffu);   // dtype: element type | reducing function << 4
      const bool fold = (bcp & DFX_CTX_FOLD) != 0;

      if (sw_pending) {   // the first poll of the next collective ends the context switch
        const u64 t1 = wall_clock64();
        if (trace && hot.trace_on < 3 && lane == 0) {
          // total | save | queue advance (save done -> context load begins) | load | set-up of the primitive (load done -> here)
          u64 tot = t1 - sw_t0, sv = sw_ts - sw_t0, adv = sw_lb - sw_ts, ldt = sw_le - sw_lb, su = t1 - sw_le;
          if (hot.trace_on < 2) { sv = 0; adv = 0; ldt = 0; su = 0; }
          if (tot > 0xffffu) tot = 0xffffu;
          if (sv > 0xfffu) sv = 0xfffu;
          if (adv > 0xfffu) adv = 0xfffu;
          if (ldt > 0xfffu) ldt = 0xfffu;
          if (su > 0xfffu) su = 0xfffu;
          trace_put(trace, &sh.trace_n, tot | (sv << 16) | (adv << 28) | (ldt << 40) | (su << 52));
        }
        sw_pending = false;
      }
      u64 tm0 = 0;
      if (hot.trace_on > 1) tm0 = wall_clock64();

      // While the first poll travels: which entry would the pass visit next, and is its context in its LDS slot?
      // If not, its load from the context buffer sets off now.  Should this wait be given up, the switch finds
      // the answer in registers (nothing below changes the queue, the list, another collective's slot or its
      // saved context before then).
      bool nx_ok = false, nx_hit = false;
      uint32_t nx_pos = 0, nx_coll = 0, nx_sl = 0;
      DfxDyn nx_dyn = {};
      uint4 nx_ctx = uint4{0, 0, 0, 0};
      auto look_ahead = [&]() {
        const uint32_t ni = scanned ? rk + 1u : pos + 1u;
        if (scanned ? (ni < nready && !(focus && pass_bytes >= hot.focus_bytes)) : (ni < qlen)) {
          nx_pos = scanned ? (uint32_t)sh.rlist[ni] : ni;
          nx_coll = sh.taskq[nx_pos];
          nx_sl = ctx_slot(nx_coll);
          nx_ok = true;
          nx_hit = sh.slot_tag[nx_sl] == nx_coll;
          if (nx_hit) nx_dyn = sh.slot[nx_sl].dyn;
          else if (lane < 8) nx_ctx = ld_ctx((const uint4*)&myctx[nx_coll] + lane);
        }
      };
      // The wait phase (Sec. 4.2 (3)), with the first poll on its way already: ready() looks at what poll() has brought.
      // The movers may be busy with earlier slices meanwhile; finished ones are retired between polls.
      // lone: the wait may go on past its threshold while nothing else is there to do (at most LONE_POLLS times).
      constexpr u64 LONE_POLLS = 256;
      auto wait_until = [&](auto&& poll, auto&& ready, auto&& lone) -> uint32_t {
        u64 n = 0;
        uint32_t r = W_OK;
        for (;;) {
          const bool ok = ready();
          ++n;
          if (__ballot(!ok) == 0) break;
          settle_slot();
          retire_finished();
          if (hot.preempt && n >= thr && !(n < LONE_POLLS && lone())) { r = W_TIMEOUT; break; }
          if ((n & 255u) == 0) {
            uint32_t s = 0;
            if (lane == 0) {
              if (ld_agent32(&a.dev_ctl[DC_ABORT]) || ld_sys32(&a.host_ctl[HC_ABORT])) s = 1;
              else if (hot.watchdog_ticks) {
                const u64 now = wall_clock64();
                if (acted) { last_act = now; acted = false; }
                if (now - last_act > hot.watchdog_ticks) {
                  ws->dbg[0] = ((u64)coll << 32) | qlen; ws->dbg[1] = ((u64)g << 32) | p; ws->dbg[2] = sent; ws->dbg[3] = recvd;
                  ws->dbg[4] = ld_agent64((const u64*)s_in); ws->dbg[5] = ld_agent64((const u64*)S.flags_out + 8); ws->dbg[6] = ri; ws->dbg[7] = now - last_act;
                  raise_error(a, 2u, wg);
                  s = 1;
                }
              }
            }
            if (bcast0(s)) { r = W_STOP; break; }
          }
          __builtin_amdgcn_s_sleep(1);
          poll();
        }
        if (lane == 0) bump(sh.stat, ST_POLLS, n);
        return r;
      };
      auto wait_traced = [&]() {
        if (hot.trace_on > 1) { const u64 tm1 = wall_clock64(); if (lane == 0) bump(sh.stat, ST_T_WAIT, tm1 - tm0); }
      };

      uint32_t res = W_OK, bytes = 0;
      SeqPos nx;
      bool last;
      if (fold) {
        // ================= fold steps =================
        nx = next_fold_position(s_rounds, bcast0(v5.w) >> 16, g, p, cidx);
        last = nx.g >= s_rounds;
        if (p == 0) {
          const uint4 v0 = sv[0], v1 = sv[1], v2 = sv[2];   // row limit | share, length | source offset, destination offset
          const bool drawn = (bcp & DFX_CTX_DRAWN) != 0;
          const uint32_t row_limit = bcast0(v0.x), vch = bcast0(v5.w) >> 16;
          const FoldGeom fg = fold_geometry(bcast64(v1.x, v1.y), bcast64(v1.z, v1.w), bcast64(v2.x, v2.y), s_slice, drawn, g);
          bytes = bcast0(v0.z);
          const bool sweep = (bcp & DFX_CTX_SWEEP) != 0;
          const FoldStep st = {kind, dtype, coll, inv_seq, inv_nchan, vch, sweep ? s_slice : row_limit, sweep ? FRESH_SWEEP | (g == 0) : !drawn || g == 0,
                               s_fin, s_in, drawn, sweep, g, bcast0(v1.x), bcast64(v1.z, v1.w)};
          if (peers_of == coll + 1u && table_serves(peers_of, bcast0(sh.peers_seq), coll, inv_seq)) {
            // The entry came with every rank's buffers, so every rank has submitted: there is nothing to wait for.  Without the
            // others' lines (a store and its way to memory, a load or two) a 25 MiB all-reduce takes 96.5 us instead of 97.8.
            if (!flight_free(hot.order_policy == 1 ? 1u : 2u)) { stop = STOP_ABORT; have = false; continue; }
            const uint4 pe = sh.peer[lane];
            post_fold(st, fg, ((u64)pe.y << 32) | pe.x, ((u64)pe.w << 32) | pe.z);
          } else {
            // The step with data waits until every rank's line carries this invocation's tag, lane k looking at the line of
            // entry k's rank, so that the poll that succeeds has brought the addresses along.  (Lanes without an entry
            // look at the first line: no branch around the loads, and none of their registers meets another path's.)
            const uint32_t line_off = lane < R ? fold_peer(kind, R, rank, K, lane) * inv_nchan * DFX_FLAG_STRIDE : 0u;
            const __amdgpu_buffer_rsrc_t lines = __builtin_amdgcn_make_buffer_rsrc((void*)s_fin, 0, (int)(R * inv_nchan * DFX_FLAG_STRIDE), 0x00020000);
            uint4 ln_recv, ln_send;
            auto poll = [&]() {
              asm volatile("" ::: "memory");     // (these loads are made anew at every poll)
              ln_recv = rs_ld16(lines, line_off + DFX_DIRECT_OFF);
              ln_send = rs_ld16(lines, line_off + DFX_DIRECT_OFF + 16);
            };
            poll();
            look_ahead();
            res = wait_until(poll, [&]() { return lane >= R || (ln_recv.z == inv_seq + 1u && ln_send.z == inv_seq + 1u); }, [] { return false; });
            if (res == W_OK) {
              wait_traced();
              // (under priority ordering a step with data, which is one long job, waits until the movers have nothing
              // else: what is posted cannot be overtaken by a more urgent collective that arrives)
              if (!flight_free(hot.order_policy == 1 ? 1u : 2u)) { stop = STOP_ABORT; have = false; continue; }
              post_fold(st, fg, ((u64)ln_send.y << 32) | ln_send.x, ((u64)ln_recv.y << 32) | ln_recv.x);
            }
          }
        } else {
          // The last wait moves nothing.  Lane v looks at channel v's counter (they lie a line apart, this workgroup's first), and what
          // they show together says that every rank's data steps of all channels are in memory: the completion is posted here
          // and now.  With every channel's workgroup waiting for its own counter and adding to one of the rank's, the
          // last of them posting, a reduce of 4 MiB on four ranks took 16.8 us, now 16.1, an all-gather of 32 MiB 66.9, now 66.0, and
          // 64 mixed collectives in disorder 993, now 962.
          // A collective that is alone in the queue has nothing to be given up for until another entry arrives: lane 63 looks for
          // that one in the same poll (an SQ in device memory; behind PCIe it would hold the poll up).  Given up after its
          // threshold and taken up again by the next pass, the wait saw the counter up to 3 us late: a 25 MiB bf16 all-reduce
          // took 98.6 us, now 97.8, an all-gather of 32 MiB 76.7, now 73.6.
          const bool alone = qlen == 1 && hot.sq_local && inv_nchan < 64u;
          const bool sq_lane = alone && lane == 63u;
          const u64* const counter = (const u64*)(s_in + (u64)(lane < inv_nchan ? lane : 0u) * DFX_FLAG_STRIDE) + DFX_FOLD_RED / 8;
          const u64* const word = sq_lane ? (const u64*)&sqbase[ri & (D - 1)].e.share : counter;
          u64 seen_cnt;
          auto poll = [&]() {
            seen_cnt = ld_sys64(word);
            for (uint32_t v = lane + 64u; v < inv_nchan; v += 64u) {      // (more channels than lanes)
              const u64 c = ld_sys64((const u64*)(s_in + (u64)v * DFX_FLAG_STRIDE) + DFX_FOLD_RED / 8);
              seen_cnt = c < seen_cnt ? c : seen_cnt;
            }
          };
          poll();
          look_ahead();
          res = wait_until(poll, [&]() { return sq_lane || seen_cnt >= s_fout; },
                           [&]() { return alone && (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(seen_cnt >> 32), 63) != (uint32_t)(ri >> hot.sq_shift) + 1u; });
          if (res == W_OK) {
            wait_traced();
            if (lane == 0) { bump(sh.stat, ST_PRIMS, 1); complete(coll, inv_seq, 1u, true); }
          }
        }
      } else {
        // ================= rings and chains =================
        const Prim q = chain_drain_round(make_prim(kind, R, bcp & 3u, p, (bcp & DFX_CTX_DIRECT) != 0), kind, (bcp & DFX_CTX_DIRECT) != 0, g, s_rounds);
        u64* const tail_out = (u64*)S.flags_out;
        u64* const tail_in = (u64*)s_in;
        // Lane 0 polls the recv side, lane 1 the send side.  The first poll is sent off before the slice's geometry is
        // worked out, which depends only on the sequence position: the arithmetic runs while the counters travel, and
        // a poll that succeeds is followed by the job at once.
        u64 seen_cnt = 0;
        auto poll = [&]() {
          if (lane == 0 && q.recv) seen_cnt = ld_agent64(tail_in);
          if (lane == 1 && (q.send || q.drain)) seen_cnt = ld_agent64(tail_out + 8);
        };
        poll();

        // ---- slice geometry and the job's four pointers, and the position after this primitive
        const SliceGeom geo = slice_geometry(S, R, g, cidx);
        const uint32_t eb = geo.eb;
        const u64 soff = geo.soff, doff = geo.doff;
        bytes = geo.bytes;
        const size_t slot_bytes = (size_t)s_slice * eb;
        const void* jfin = q.recv ? (const void*)((const uint8_t*)s_fin + (size_t)(recvd & (K - 1)) * slot_bytes) : nullptr;
        void* jfout = q.send ? (void*)((uint8_t*)s_fout + (size_t)(sent & (K - 1)) * slot_bytes) : nullptr;
        const char* jsb = q.from_send ? (const char*)S.sendbuf + soff * eb : nullptr;
        char* jrb = q.to_recv ? (char*)S.recvbuf + doff * eb : nullptr;
        // a notified result goes to the recv buffer through the coherent path of a slot
        if (q.notify) { jfout = jrb; jrb = nullptr; }
        // (slices in windows, the chunk index stepping down the ring)
        nx = next_position(kind, R, rank, hot.window, s_rounds, s_n & 0xffffu, g, p, cidx);
        last = nx.g >= s_rounds;
        if (q.recv || q.send || q.drain) {
          look_ahead();
          res = wait_until(poll, [&]() {
            bool ok = true;
            if (lane == 0 && q.recv) ok = seen_cnt > recvd;
            if (lane == 1 && q.send) ok = (sent - seen_cnt) < (u64)K;
            if (lane == 1 && q.drain) ok = sent == seen_cnt;
            return ok;
          }, [] { return false; });
        }
        if (res == W_OK) {
          wait_traced();
          if (!flight_free(2u)) { stop = STOP_ABORT; have = false; continue; }
          if (q.din || q.din_send) {
            // The previous rank published its buffers for this invocation before it notified anything
            // (the counter just seen).  Read once per stay of the collective in hand.
            if (prev_recv == 0) {
              const Slot<AUX_DEVICE> line((const void*)tail_in, DFX_FLAG_STRIDE);
              uint4 w = uint4{0, 0, 0, 0}, w2 = w;
              for (uint32_t tries = 0; tries < 1024u; ++tries) {
                w = line.ld16(DFX_DIRECT_OFF);
                w2 = line.ld16(DFX_DIRECT_OFF + 16);
                if (w.z == inv_seq + 1u && w2.z == inv_seq + 1u) break;
                __builtin_amdgcn_s_sleep(2);
              }
              if (w.z != inv_seq + 1u || w2.z != inv_seq + 1u) { raise_error(a, 3u, wg); stop = STOP_ABORT; have = false; continue; }
              prev_recv = ((u64)w.y << 32) | w.x;
              prev_send = ((u64)w2.y << 32) | w2.x;
            }
            jfin = q.din_send ? (const void*)((const char*)prev_send + soff * eb) : (const void*)((const char*)prev_recv + doff * eb);
          }
          // ---- post the slice (an empty one is only a handshake: the movers just raise the counters);
          // this claims the slots: the data follows, the counters after it
          if (q.send || q.notify) ++sent;
          if (q.recv) ++recvd;
          if (lane == 0) {
            Job j;
            j.fin = jfin; j.fout = jfout; j.sb = jsb; j.rb = jrb;
            j.bytes = (q.drain || (!q.recv && !q.from_send)) ? 0u : bytes;   // drain and notify-only steps move nothing
            j.nsrc = 0; j.ndst = 0; j.index = j.sharers = j.head = j.limit = j.fresh = j.gang = 0; j.draw = 0;
            j.dtype = dtype; j.coll = coll; j.prim = q.drain ? 0xffu : p;   // (prim: for the timeline only)
            sh.job[posted & 1] = j;
            Flight f;
            f.tail_out = (q.send || q.notify) ? tail_out : nullptr; f.head_in = q.recv ? tail_in + 8 : nullptr;
            f.sent_new = sent; f.recvd_new = recvd;
            f.last = last ? 1u : 0u; f.coll = coll; f.seq = inv_seq; f.nchan = inv_nchan;
            f.add_one = nullptr;
            sh.fl[posted & 1] = f;
            lds_st(&sh.job_seq, posted + 1);
          }
          ++posted;
        }
      }

      if (res == W_OK) {
        g = nx.g; p = nx.p; cidx = nx.cidx;
        pass_bytes += bytes;
        progressed = true;
        pass_progress = true;
        acted = true;
        // AdaptivelyAdjustSpinThreshold (Alg. 1 line 9)
        if (!scanned) {
          thr *= hot.spin_boost;
          if (thr > hot.spin_max) thr = hot.spin_max;
        }
        if (last) {
          // ---- CollectiveSuccess: the entry leaves the queue now; the completion counter and the
          // CQE follow at retirement, when the data is in memory
          if (lane == 0) {
            DfxDyn d; d.round = 0; d.prim = 0; d.sent = sent; d.recvd = recvd; d.preempted = 0; d.cidx = 0;
            sh.slot[sl].dyn = d;
            st_ctx(&myctx[coll].dyn, d);
          }
          // later entries move up, the position stays (Sec. 4.3)
          --qlen;
          for (uint32_t base = pos; base < qlen; base += 64) {
            const uint32_t i = base + lane;
            uint16_t v = 0;
            if (i < qlen) v = sh.taskq[i + 1];
            __builtin_amdgcn_wave_barrier();
            if (i < qlen) sh.taskq[i] = v;
            __builtin_amdgcn_wave_barrier();
          }
          have = false;
          sw_pending = false;
          if (scanned) {
            // the entries behind the one that left have moved up by one: so do their positions in the list
            ++rk;
            for (uint32_t base = rk; base < nready; base += 64) {
              const uint32_t k = base + lane;
              if (k < nready && (uint32_t)sh.rlist[k] > pos) sh.rlist[k] = (uint16_t)(sh.rlist[k] - 1u);
            }
            __builtin_amdgcn_wave_barrier();
          }
        } else if (__builtin_expect(fold && p == 1u && qlen > 1u, 0)) {
          // The last wait cannot be over while the job just posted is not, and there is other work.  In a scanned pass, whose threshold
          // is one poll, it is left unpolled (polled, it was given up in 9011 of 9011 passes over 1024 small all-reduces, 1.4 us each);
          // elsewhere it gets the smallest threshold where the pass still has entries to visit.  (Those in front have just been given
          // up: gone back to before this wait, beside a stuck one, an all-reduce of 8 KiB took 34.5 us, now 26.4.)
          if (scanned && give_way) {
            if (lane == 0) {
              DfxDyn d; d.round = g; d.prim = p; d.sent = sent; d.recvd = recvd;
              d.preempted = sh.slot[sl].dyn.preempted + 1; d.cidx = cidx;
              sh.slot[sl].dyn = d;
              st_ctx(&myctx[coll].dyn, d);
              bump(sh.stat, ST_PREEMPT, 1); bump(sh.stat, ST_SAVE, 1); bump(sh.stat, ST_UNPOLLED, 1);
            }
            have = false;
            sw_pending = false;
            ++rk;
          } else if (!scanned && pos + 1u < qlen) thr = hot.spin_min;
        }
      } else {
        // ---- PreemptCollective + SaveCollectiveContext (lazy: only if it progressed)
        if (hot.trace_on == 3 && trace && lane == 0)   // timeline sample of a wait that ended without the primitive: index 15
          trace_put(trace, &sh.trace_n, timeline_sample(tm0, wall_clock64(), coll, 15));
        const bool tr = hot.trace_on && res == W_TIMEOUT && pos + 1 < qlen;
        if (tr) sw_t0 = wall_clock64();
        if (lane == 0) {
          if (res == W_TIMEOUT) bump(sh.stat, ST_PREEMPT, 1);
          if (progressed) {
            DfxDyn d; d.round = g; d.prim = p; d.sent = sent; d.recvd = recvd;
            d.preempted = sh.slot[sl].dyn.preempted + 1; d.cidx = cidx;
            sh.slot[sl].dyn = d;
            st_ctx(&myctx[coll].dyn, d);
            bump(sh.stat, ST_SAVE, 1);
          } else if (res == W_TIMEOUT) bump(sh.stat, ST_LAZY, 1);
        }
        if (tr) { if (hot.trace_on > 1) sw_ts = wall_clock64(); sw_pending = true; }
        have = false;
        if (res == W_STOP) { stop = STOP_ABORT; continue; }
        if (scanned) ++rk; else ++pos;
        if (nx_ok && res == W_TIMEOUT) {
          // LoadCollectiveContext of the entry looked up during the wait (the same steps as at the head of the
          // loop): its context is in its slot and the dynamic part in registers, or the load is under way and
          // goes into the slot now
          pos = bcast0(nx_pos); coll = bcast0(nx_coll); sl = bcast0(nx_sl);
          if (nx_hit) {
            if (lane == 0) bump(sh.stat, ST_HIT, 1);
          } else {
            if (lane < 8) ((uint4*)&sh.slot[sl])[lane] = nx_ctx;
            if (lane == 0) { sh.slot_tag[sl] = coll; bump(sh.stat, ST_LOAD, 1); }
            __builtin_amdgcn_wave_barrier();
            nx_dyn = sh.slot[sl].dyn;
          }
          g = bcast0(nx_dyn.round); p = bcast0(nx_dyn.prim); cidx = bcast0(nx_dyn.cidx);
          sent = bcast64((uint32_t)nx_dyn.sent, (uint32_t)(nx_dyn.sent >> 32)); recvd = bcast64((uint32_t)nx_dyn.recvd, (uint32_t)(nx_dyn.recvd >> 32));
          thr = hot.spin_init >> (pos < 31 ? pos : 31);
          if (thr < hot.spin_min || scanned) thr = hot.spin_min;
          progressed = false;
          prev_recv = 0;
          have = true;
          if (sw_pending && hot.trace_on > 1) { sw_lb = wall_clock64(); sw_le = sw_lb; }
        }
      }
    }

    // every posted job has been retired and no collective is in hand: the movers may go
    if (lane == 0) {
      if (stop == STOP_QUIT) bump(sh.stat, ST_QUITS, 1);
      ws->read_index = ri;
      ws->qlen = qlen;
      sh.qlen_out = qlen;
      lds_st(&sh.leave, 1u);
    }
  }

  // ================= leave: persist what the next launch needs =================
  __syncthreads();
  if (tid == 0) {
    ws->trace_n = sh.trace_n;
    for (int i = 0; i < DFX_NSTAT; ++i) ws->stat[i] = sh.stat[i];
  }
  const uint32_t qn = sh.qlen_out;
  for (uint32_t i = tid; i < qn; i += NT) qstore[i] = sh.taskq[i];
}

// Plain copy kernel of known traffic: calibrates the HBM byte counters of the profiler and shows
// what a streaming copy reaches.  Four independent 16-byte vectors in flight per thread.
extern "C" __global__ void __launch_bounds__(256) dfx_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t nvec) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + 3 * stride < nvec; i += 4 * stride) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = ld_user((const v4u_user*)&src[i + u * stride]);
#pragma unroll
    for (int u = 0; u < 4; ++u) st_user((v4u_user*)&dst[i + u * stride], v[u]);
  }
  for (; i < nvec; i += stride) dst[i] = src[i];
}

// ------------------------------------------------------------------------------------------
// launch helpers for the host library (kept in this translation unit with the kernels)
// ------------------------------------------------------------------------------------------
hipError_t dfx_daemon_occupancy(int* blocks_per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, dfx_daemon_kernel, DFX_WG_THREADS, 0);
}

hipError_t dfx_daemon_launch(uint32_t nwg, hipStream_t stream, const DfxDaemonArgs& a) {
  hipLaunchKernelGGL(dfx_daemon_kernel, dim3(nwg), dim3(DFX_WG_THREADS), 0, stream, a);
  return hipGetLastError();
}

hipError_t dfx_copy_launch(const void* src, void* dst, size_t bytes, hipStream_t stream) {
  hipLaunchKernelGGL(dfx_copy_kernel, dim3(4096), dim3(256), 0, stream, (const uint4*)src, (uint4*)dst, bytes >> 4);
  return hipGetLastError();
}
