// The data movers of collectives in fold steps (make_fold_prim): rows of up to 64 buffers read, combined and written, and what they
// share with the connectors' slice movers -- the reducing functions, address spaces, cache policies.
#ifndef DFX_MOVERS_H
#define DFX_MOVERS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfx_internal.h"
#include "dfx_geometry.h"

namespace {

typedef uint64_t u64;

#define SCOPE_AGENT __HIP_MEMORY_SCOPE_AGENT
#define SCOPE_SYSTEM __HIP_MEMORY_SCOPE_SYSTEM

// A pointer that is known to be one to device or host memory, never to LDS: what is accessed through it takes global
// instructions instead of flat ones (pointers that came out of LDS or were put together from integers look like
// either to the compiler, and a flat access is waited for on both counters).
#define GLOBAL_AS __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ GLOBAL_AS T* global_ptr(T* p) { return (GLOBAL_AS T*)p; }

__device__ __forceinline__ uint32_t bcast0(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
// two words that every lane holds alike -> one scalar
__device__ __forceinline__ u64 bcast64(uint32_t lo, uint32_t hi) { return ((u64)bcast0(hi) << 32) | (u64)bcast0(lo); }

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// cache-policy operand of the buffer instructions (gfx940+): bit 0 = sc0, bit 4 = sc1
constexpr int AUX_CACHED = 0;    // ordinary cached access (per-CU cache, write-back in this XCD's L2)
constexpr int AUX_DEVICE = 16;   // sc1: device scope, coherent across the XCDs' L2s
constexpr int AUX_SYSTEM = 17;   // sc0 | sc1: system scope, nothing of it is taken from a cache
constexpr int AUX_STREAM = 18;   // sc1 | nt: the same for what is read once: the caches on the way need not keep it

// ------------------------------------------------------------------------------------------
// reduce: one hop a (+) b in the storage dtype (one rounding per hop)
// ------------------------------------------------------------------------------------------
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// two fp32 values -> packed bf16, round to nearest even: one conversion instruction on gfx950
__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  f32x2_t s;
  s[0] = lo; s[1] = hi;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(s, bf16x2_t));
}

__device__ __forceinline__ uint32_t bf16x2_add(uint32_t a, uint32_t b) {
  // widen (exact), add in fp32, round to nearest even back to bf16
  return pack_bf16_rne(__uint_as_float(a << 16) + __uint_as_float(b << 16),
                       __uint_as_float(a & 0xffff0000u) + __uint_as_float(b & 0xffff0000u));
}

template <int DT>
__device__ __forceinline__ uint32_t add_word(uint32_t a, uint32_t b) {
  if (DT == DT_F32) return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
  if (DT == DT_I32) return a + b;
  if (DT == DT_F16) {
    half2_t x = __builtin_bit_cast(half2_t, a), y = __builtin_bit_cast(half2_t, b);
    return __builtin_bit_cast(uint32_t, x + y);
  }
  return bf16x2_add(a, b);
}

template <int DT>
__device__ __forceinline__ uint4 add_vec(uint4 a, uint4 b) {
  uint4 r;
  r.x = add_word<DT>(a.x, b.x);
  r.y = add_word<DT>(a.y, b.y);
  r.z = add_word<DT>(a.z, b.z);
  r.w = add_word<DT>(a.w, b.w);
  return r;
}

template <int DT>
__device__ __forceinline__ uint16_t add_half(uint16_t a, uint16_t b) {
  if (DT == DT_F16) {
    _Float16 x = __builtin_bit_cast(_Float16, a), y = __builtin_bit_cast(_Float16, b);
    return __builtin_bit_cast(uint16_t, (_Float16)(x + y));
  }
  return (uint16_t)(bf16x2_add(a, b) & 0xffffu);
}

// The other reducing functions (Sec. 4.1: "a specified reducing function"), evaluated as
// partial (op) own with the partial that arrived from the left first.  Product rounds once per
// hop like the sum; maximum / minimum pass one operand on unchanged: the partial if it is
// strictly greater (smaller), else the own value -- plain compare-and-select, so that equal
// values (+0 / -0 included) behave the same everywhere.
enum { OP_SUM = 0, OP_PROD = 1, OP_MAX = 2, OP_MIN = 3 };

template <int OP>
__device__ __forceinline__ uint32_t bf16x2_op(uint32_t a, uint32_t b) {
  const float al = __uint_as_float(a << 16), bl = __uint_as_float(b << 16);
  const float ah = __uint_as_float(a & 0xffff0000u), bh = __uint_as_float(b & 0xffff0000u);
  if (OP == OP_PROD) return pack_bf16_rne(al * bl, ah * bh);
  const bool tl = (OP == OP_MAX) ? (al > bl) : (al < bl);
  const bool th = (OP == OP_MAX) ? (ah > bh) : (ah < bh);
  return ((tl ? a : b) & 0xffffu) | ((th ? a : b) & 0xffff0000u);
}

// one 32-bit word (one fp32 / int32 element or two 16-bit ones), reducing function fixed at compile time
template <int DT, int OP>
__device__ __forceinline__ uint32_t op_word_t(uint32_t a, uint32_t b) {
  if (OP == OP_SUM) return add_word<DT>(a, b);
  if (DT == DT_F32) {
    const float x = __uint_as_float(a), y = __uint_as_float(b);
    if (OP == OP_PROD) return __float_as_uint(x * y);
    return ((OP == OP_MAX) ? (x > y) : (x < y)) ? a : b;
  }
  if (DT == DT_I32) {
    if (OP == OP_PROD) return a * b;
    const int x = (int)a, y = (int)b;
    return ((OP == OP_MAX) ? (x > y) : (x < y)) ? a : b;
  }
  if (DT == DT_F16) {
    const half2_t x = __builtin_bit_cast(half2_t, a), y = __builtin_bit_cast(half2_t, b);
    if (OP == OP_PROD) return __builtin_bit_cast(uint32_t, x * y);
    const bool tl = (OP == OP_MAX) ? (x[0] > y[0]) : (x[0] < y[0]);
    const bool th = (OP == OP_MAX) ? (x[1] > y[1]) : (x[1] < y[1]);
    return ((tl ? a : b) & 0xffffu) | ((th ? a : b) & 0xffff0000u);
  }
  return bf16x2_op<OP>(a, b);
}

// the same with the reducing function picked at run time (element-wise tails)
template <int DT>
__device__ __forceinline__ uint32_t op_word(uint32_t a, uint32_t b, int op) {
  switch (op) {
    case OP_PROD: return op_word_t<DT, OP_PROD>(a, b);
    case OP_MAX: return op_word_t<DT, OP_MAX>(a, b);
    case OP_MIN: return op_word_t<DT, OP_MIN>(a, b);
    default: return add_word<DT>(a, b);
  }
}

template <int DT, int OP>
__device__ __forceinline__ uint4 op_vec_t(uint4 a, uint4 b) {
  uint4 r;
  r.x = op_word_t<DT, OP>(a.x, b.x);
  r.y = op_word_t<DT, OP>(a.y, b.y);
  r.z = op_word_t<DT, OP>(a.z, b.z);
  r.w = op_word_t<DT, OP>(a.w, b.w);
  return r;
}

// A whole batch of vectors under one (wave-uniform) branch on the reducing function: the branch
// stays out of the unrolled loads and stores around it.
template <int DT, int N>
__device__ __forceinline__ void op_batch(uint4 (&v)[N], const uint4 (&w)[N], int op) {
  switch (op) {
    case OP_PROD:
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = op_vec_t<DT, OP_PROD>(v[u], w[u]);
      break;
    case OP_MAX:
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = op_vec_t<DT, OP_MAX>(v[u], w[u]);
      break;
    case OP_MIN:
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = op_vec_t<DT, OP_MIN>(v[u], w[u]);
      break;
    default:
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = add_vec<DT>(v[u], w[u]);
      break;
  }
}

template <int DT>
__device__ __forceinline__ uint16_t op_half(uint16_t a, uint16_t b, int op) {
  if (op == OP_SUM) return add_half<DT>(a, b);
  return (uint16_t)(op_word<DT>(a, b, op) & 0xffffu);   // the upper half combines zeros and is dropped
}

// ------------------------------------------------------------------------------------------
// Fold steps (make_fold_prim): the data movers
// ------------------------------------------------------------------------------------------
// a buffer resource over memory whose address every lane holds alike (it came out of LDS)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(u64 addr, uint32_t bytes) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)addr), hi = __builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)(((u64)hi << 32) | lo), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 rs_ld16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, AUX_DEVICE));   // out of range reads return 0
}
__device__ __forceinline__ uint4 rs_ld16_stream(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, AUX_STREAM));
}
__device__ __forceinline__ void rs_st16(__amdgpu_buffer_rsrc_t r, uint32_t off, uint4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, (int)off, 0, AUX_DEVICE);        // out of range stores are dropped
}

// The rows of a job that one mover wave takes (see fold_row_bytes): dealt (ctr null) or drawn.
struct Rows {
  GLOBAL_AS uint32_t* ctr;   // the region's row counter
  uint32_t waves;            // mover waves of all the region's workgroups
  uint32_t row;              // the row in hand
  uint32_t left;             // rows this wave may still take in the job, the one in hand included (0xffffffff = no limit: dealt)
  uint32_t drawn;            // lane 0: the answer to the last draw
  // Begin: the first job of a share starts with the wave's own row, later ones draw theirs.
  __device__ __forceinline__ void begin(bool fresh, uint32_t wave_index) {
    if (fresh) row = wave_index;
    else { draw(); row = waves + (uint32_t)__builtin_amdgcn_readfirstlane(drawn); }
  }
  __device__ __forceinline__ void draw() {
    if ((threadIdx.x & 63u) == 0) drawn = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, SCOPE_AGENT);
  }
  // Ahead of the row's loads: the next draw sets off (its answer arrives before the data does).
  __device__ __forceinline__ void prefetch() { if (ctr && left > 1) draw(); }
  // Behind the row: on to the next; false = the job is over for this wave.
  __device__ __forceinline__ bool next() {
    if (left == 1) return false;
    if (left != 0xffffffffu) --left;
    row = ctr ? waves + (uint32_t)__builtin_amdgcn_readfirstlane(drawn) : row + waves;
    return true;
  }
};

// dst[d][i] = src[0][i] (op) src[1][i] (op) ... (op) src[nsrc-1][i], left to right, for every destination d: the
// source table lists the ranks in the ring's order of combination.  Sources are other ranks' send buffers:
// device-coherent loads; the destinations are recv buffers of this and of other ranks, whose workgroups post the
// completion: device-coherent stores, which are in memory when the step counts itself done.
//
// What bounds it is HBM (2R streams, every byte once).  About sixteen 16-byte loads are in flight per thread whatever
// the number of sources; with 2, 4 or 8 of them (and as many destinations, or one) all buffer resources stay in
// scalar registers over the whole job (looked up for every round they cost 0.4 us per round and side: the one job of
// an 8 KiB all-reduce took 3.4 us, now 1.8; a 25 MiB bf16 bucket, with the rows, 92 -> 75 us).  A buffer's
// resource ends with the last row's last whole 16 bytes: loads behind it return 0 and stores behind it are dropped, so
// the last row needs no predicates.
// Next round's loads before this round's combine, 512 movers or plain cached accesses measured the same (838-845 us for 256 MiB per
// rank, fp32, R = 8, before rows).  The non-temporal hint is for sweeps: below the size of the memory-side cache it costs
// (8 MiB: 25 against 20.5 us).
template <int DT, int NS, bool ALL>
__device__ __forceinline__ void fold_fixed(const u64* src_tab, const u64* dst_tab, uint32_t from, uint32_t end, Rows& rows, uint32_t lane, int op) {
  constexpr int U = 16 / NS, ND = ALL ? NS : 1;      // (fold_row_bytes)
  __amdgpu_buffer_rsrc_t S[NS], D[ND];
#pragma unroll
  for (int k = 0; k < NS; ++k) S[k] = uniform_rsrc(src_tab[k], end);
#pragma unroll
  for (int k = 0; k < ND; ++k) D[k] = uniform_rsrc(dst_tab[k], end);
  for (;;) {
    const uint32_t at = from + rows.row * (U * 1024u);
    if (at >= end) break;
    rows.prefetch();
    const uint32_t o = at + lane * 16u;
    uint4 w[NS][U];
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) w[k][u] = rs_ld16(S[k], o + u * 1024u);
#pragma unroll
    for (int k = 1; k < NS; ++k) op_batch<DT, U>(w[0], w[k], op);
#pragma unroll
    for (int k = 0; k < ND; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) rs_st16(D[k], o + u * 1024u, w[0][u]);
    if (!rows.next()) break;
  }
}

// A table of up to 64 addresses in one register pair, entry k in lane k: a wave that works with any number of buffers picks the
// next one with two lane reads.  (Out of LDS, with a wait for each, three ranks took 482 us for a reduce-scatter of 200 MiB
// with drawn rows and 406 with dealt ones, 416 as the ring it once was.)
struct LaneTable {
  uint32_t lo, hi;
  __device__ __forceinline__ LaneTable(const u64* tab, uint32_t n, uint32_t lane, u64 off = 0, uint32_t first = 0) {
    uint32_t e = lane < n ? first + lane : 0u;       // (entry k: the one `first` + k of n, all of them `off` bytes on)
    if (e >= n) e -= n;
    const u64 a = tab[e] + off;
    lo = (uint32_t)a; hi = (uint32_t)(a >> 32);
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(uint32_t k, uint32_t bytes) const {
    const uint32_t l = __builtin_amdgcn_readlane(lo, k), h = __builtin_amdgcn_readlane(hi, k);
    return __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)(((u64)h << 32) | l), 0, (int)bytes, 0x00020000);
  }
};

// the same for any number of sources and destinations
template <int DT>
__device__ __forceinline__ void fold_any(const u64* src_tab, uint32_t nsrc, const u64* dst_tab, uint32_t ndst, uint32_t from, uint32_t end,
                                         Rows& rows, uint32_t lane, int op) {
  constexpr int U = 2, NS = 8;      // vectors per source (fold_row_bytes) and sources in flight
  const LaneTable S(src_tab, nsrc, lane), D(dst_tab, ndst, lane);
  for (;;) {
    const uint32_t at = from + rows.row * (U * 1024u);
    if (at >= end) break;
    rows.prefetch();
    const uint32_t o = at + lane * 16u;
    uint4 acc[U];
    for (uint32_t base = 0; base < nsrc; base += NS) {
      uint4 w[NS][U];
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (base + k < nsrc) {
          const __amdgpu_buffer_rsrc_t r = S.rsrc(base + k, end);
#pragma unroll
          for (int u = 0; u < U; ++u) w[k][u] = rs_ld16(r, o + u * 1024u);
        }
      }
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (base + k < nsrc) {
          if (base + k == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = w[0][u];
          } else op_batch<DT, U>(acc, w[k], op);
        }
      }
    }
    for (uint32_t d = 0; d < ndst; ++d) {
      const __amdgpu_buffer_rsrc_t r = D.rsrc(d, end);
#pragma unroll
      for (int u = 0; u < U; ++u) rs_st16(r, o + u * 1024u, acc[u]);
    }
    if (!rows.next()) break;
  }
}

// One row, [at, at + row) up to `end`, of any number of sources and destinations: 2 KiB at a time of eight sources, 16 loads in flight
// per lane; the buffers out of lanes, so one form serves all rank counts.  Of a gang, whose waves are at different collectives and
// whose rows are few.
template <int DT>
__device__ __forceinline__ void fold_row(const u64* src_tab, uint32_t nsrc, const u64* dst_tab, uint32_t ndst, uint32_t at, uint32_t row, uint32_t end,
                                         uint32_t lane, int op) {
  constexpr int U = 2, NS = 8;
  const LaneTable S(src_tab, nsrc, lane), D(dst_tab, ndst, lane);
  const uint32_t stop = at + row < end ? at + row : end;
  for (; at < stop; at += U * 1024u) {
    const uint32_t o = at + lane * 16u;
    uint4 acc[U];
    for (uint32_t base = 0; base < nsrc; base += NS) {
      uint4 w[NS][U];
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (base + k < nsrc) {
          const __amdgpu_buffer_rsrc_t r = S.rsrc(base + k, stop);
#pragma unroll
          for (int u = 0; u < U; ++u) w[k][u] = rs_ld16(r, o + u * 1024u);
        }
      }
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (base + k < nsrc) {
          if (base + k == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = w[0][u];
          } else op_batch<DT, U>(acc, w[k], op);
        }
      }
    }
    for (uint32_t d = 0; d < ndst; ++d) {
      const __amdgpu_buffer_rsrc_t r = D.rsrc(d, stop);
#pragma unroll
      for (int u = 0; u < U; ++u) rs_st16(r, o + u * 1024u, acc[u]);
    }
  }
}

// One source handed out to every destination (all-gather, broadcast): ND destinations, or any number (ND = 0).
// What bounds it is the writes (R per byte read).  Reading once instead of every rank reading everything (R reads and R
// writes per byte): host to host, bf16, R = 8, broadcast of 100 MiB 270 -> 208 us, all-gather of 32 MiB 104 -> 80 us.
// Two ranks have 64 workgroups in all and take twice the vectors per row: broadcast of 32 MiB 62 -> 38.5 us,
// all-gather of 128 MiB 233 -> 171.
template <int ND, int U>
__device__ __forceinline__ void fold_copy(const u64* src_tab, const u64* dst_tab, uint32_t ndst, uint32_t from, uint32_t end, Rows& rows, uint32_t lane) {
  // (U: fold_row_bytes)
  const __amdgpu_buffer_rsrc_t S = uniform_rsrc(src_tab[0], end);
  __amdgpu_buffer_rsrc_t D[ND ? ND : 1];
#pragma unroll
  for (int k = 0; k < ND; ++k) D[k] = uniform_rsrc(dst_tab[k], end);
  const LaneTable T(dst_tab, ndst, lane);      // (any number of them)
  for (;;) {
    const uint32_t at = from + rows.row * (U * 1024u);
    if (at >= end) break;
    rows.prefetch();
    const uint32_t o = at + lane * 16u;
    uint4 w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = rs_ld16(S, o + u * 1024u);
    if (ND) {
#pragma unroll
      for (int k = 0; k < ND; ++k)
#pragma unroll
        for (int u = 0; u < U; ++u) rs_st16(D[k], o + u * 1024u, w[u]);
    } else {
      for (uint32_t d = 0; d < ndst; ++d) {
        const __amdgpu_buffer_rsrc_t r = T.rsrc(d, end);
#pragma unroll
        for (int u = 0; u < U; ++u) rs_st16(r, o + u * 1024u, w[u]);
      }
    }
    if (!rows.next()) break;
  }
}

// The bytes [at, end) of a span, at most 64 elements, element by element (fold or copy), eight sources in flight: one after the
// other they took as long as a short span's rows (all-reduce of 1 MiB bf16 with an odd end 23.6 us, now 22.8).
template <int DT>
__device__ __forceinline__ void fold_ends(const u64* src_tab, uint32_t nsrc, const u64* dst_tab, uint32_t ndst, uint32_t at, uint32_t end,
                                          uint32_t lane, int op, u64 src_off = 0, u64 dst_off = 0) {
  constexpr uint32_t EB = (DT == DT_F32 || DT == DT_I32) ? 4u : 2u;
  constexpr int NS = 8;
  const LaneTable S(src_tab, nsrc, lane, src_off), D(dst_tab, ndst, lane, dst_off);
  const uint32_t o = at + lane * EB;       // (elements behind the end: loads return 0, stores are dropped)
  uint32_t v = 0;
  for (uint32_t base = 0; base < nsrc; base += NS) {
    uint32_t x[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (base + k < nsrc) {
        const __amdgpu_buffer_rsrc_t r = S.rsrc(base + k, end);
        x[k] = EB == 4 ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)o, 0, AUX_DEVICE)
                       : (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)o, 0, AUX_DEVICE);
      }
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (base + k < nsrc) v = base + k == 0 ? x[0] : (EB == 4 ? op_word<DT>(v, x[k], op) : (uint32_t)op_half<DT>((uint16_t)v, (uint16_t)x[k], op));
    }
  }
  for (uint32_t d = 0; d < ndst; ++d) {
    const __amdgpu_buffer_rsrc_t r = D.rsrc(d, end);
    if (EB == 4) __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)o, 0, AUX_DEVICE);
    else __builtin_amdgcn_raw_buffer_store_b16((uint16_t)v, r, (int)o, 0, AUX_DEVICE);
  }
}

// A span: `head` bytes (fold_head), rows, and the bytes behind the last whole 16.  ends_at < ends: this wave takes these bytes
// before or behind the rows (exactly one of the region's waves each, once; never the same one).
struct Span { uint32_t head, end, ends_at, ends; };
static_assert(DFX_FOLD_WAVES >= 2, "the first and the last mover wave of a region are two");

// A reduction has one source per rank and one destination, or as many destinations as sources.
template <int DT>
__device__ __forceinline__ void fold_reduce(const u64* src_tab, uint32_t nsrc, const u64* dst_tab, uint32_t ndst, const Span& sp,
                                            Rows& rows, uint32_t lane, int op) {
  const uint32_t from = sp.head, end = sp.end;
  const bool all = ndst > 1;
  if (nsrc == 8 && all) fold_fixed<DT, 8, true>(src_tab, dst_tab, from, end, rows, lane, op);
  else if (nsrc == 8) fold_fixed<DT, 8, false>(src_tab, dst_tab, from, end, rows, lane, op);
  else if (nsrc == 4 && all) fold_fixed<DT, 4, true>(src_tab, dst_tab, from, end, rows, lane, op);
  else if (nsrc == 4) fold_fixed<DT, 4, false>(src_tab, dst_tab, from, end, rows, lane, op);
  else if (nsrc == 2 && all) fold_fixed<DT, 2, true>(src_tab, dst_tab, from, end, rows, lane, op);
  else if (nsrc == 2) fold_fixed<DT, 2, false>(src_tab, dst_tab, from, end, rows, lane, op);
  else fold_any<DT>(src_tab, nsrc, dst_tab, ndst, from, end, rows, lane, op);
  if (sp.ends) fold_ends<DT>(src_tab, nsrc, dst_tab, ndst, sp.ends_at, sp.ends, lane, op);
}

__device__ __forceinline__ void fold_dispatch(int dtype, const u64* src_tab, uint32_t nsrc, const u64* dst_tab, uint32_t ndst, const Span& sp,
                                              Rows& rows, uint32_t lane) {
  if (nsrc == 1) {
    const uint32_t from = sp.head, end = sp.end;
    if (ndst == 8) fold_copy<8, 4>(src_tab, dst_tab, ndst, from, end, rows, lane);
    else if (ndst == 4) fold_copy<4, 4>(src_tab, dst_tab, ndst, from, end, rows, lane);
    else if (ndst == 2) fold_copy<2, 8>(src_tab, dst_tab, ndst, from, end, rows, lane);
    else fold_copy<0, 4>(src_tab, dst_tab, ndst, from, end, rows, lane);
    // (every element type is a multiple of 2 bytes)
    if (sp.ends) fold_ends<DT_F16>(src_tab, 1, dst_tab, ndst, sp.ends_at, sp.ends, lane, OP_SUM);
    return;
  }
  const int op = dtype >> 4;
  switch (dtype & 15) {
    case DT_F32: fold_reduce<DT_F32>(src_tab, nsrc, dst_tab, ndst, sp, rows, lane, op); break;
    case DT_BF16: fold_reduce<DT_BF16>(src_tab, nsrc, dst_tab, ndst, sp, rows, lane, op); break;
    case DT_F16: fold_reduce<DT_F16>(src_tab, nsrc, dst_tab, ndst, sp, rows, lane, op); break;
    default: fold_reduce<DT_I32>(src_tab, nsrc, dst_tab, ndst, sp, rows, lane, op); break;
  }
}

// ---- sweeps (sweep_region): the same movers over all regions of the message.  Their tables hold whole buffers, every rank's.
// What bounds them is HBM: reads alone go at 6.7 - 7 TB/s, writes alone at 5.5, which one after the other is 710 us for the all-reduce of
// 256 MiB per rank (R = 8); it takes 723 - 746 on different boxes.  The pace of the loads counts: in a kernel of its own the same loop (dealt
// rows) takes 750 - 765, and so it does here with its resources in scalar registers (750 - 760).  As it stands the compiler has
// them in vector registers -- the movers' branch to it is a divergent one -- and takes every access in a loop over readfirstlane,
// which spaces them; scalar with s_sleep(1) behind every load measured 734 - 736.  Deeper pipelines (next row's loads ahead, 32 in flight per
// lane), 512 or 1024 movers and non-temporal stores measured the same.
struct Sweep {
  uint32_t kind, R, rank, nreg;
  uint32_t rows, all;                      // rows of a region, of the message
  uint32_t waves, base, skip;              // sweep_row
  uint32_t longest;
  u64 total;
  uint32_t lo, hi;                         // rows of the region in hand
  uint32_t first;                          // ... where its order of combination begins in the tables
  FoldRegion f;
  u64 own_src, own_dst;                    // the rank's own region
  uint32_t ends_at, ends;                  // ... bytes before or behind its rows that this wave takes
  __device__ __forceinline__ void enter(uint32_t t) {
    const uint32_t c = t / rows;
    lo = c * rows; hi = lo + rows;
    f = sweep_region((int)kind, longest, total, c);
    first = sweep_first(nreg, c, rank, R);
  }
  // Bytes at which the row in hand begins; the region's address tables are to be looked up where `moved` says so.  False: no row left.
  __device__ __forceinline__ bool row(uint32_t n, uint32_t row_bytes, uint32_t& at, bool& moved) {
    const uint32_t t = bcast0(sweep_row(n, waves, base, skip));
    if (t >= all) return false;
    moved = t >= hi;
    if (moved) enter(t);
    at = f.head + (t - lo) * row_bytes;
    return true;
  }
};

template <int DT, int NS, bool ALL>
__device__ __forceinline__ void sweep_fixed(const u64* src_tab, const u64* dst_tab, Sweep& w, Rows& rows, uint32_t lane, int op) {
  constexpr int U = 16 / NS, ND = ALL ? NS : 1;      // (sweep_row_bytes)
  __amdgpu_buffer_rsrc_t S[NS], D[ND];
  uint32_t at;
  bool moved;
  while (w.row(rows.row, U * 1024u, at, moved)) {
    if (moved) {
      const LaneTable a(src_tab, NS, lane, w.f.src, w.first), b(dst_tab, NS, lane, w.f.dst, w.first);
#pragma unroll
      for (int k = 0; k < NS; ++k) S[k] = a.rsrc(k, w.f.end);
#pragma unroll
      for (int k = 0; k < ND; ++k) D[k] = b.rsrc(ALL ? k : NS - 1, w.f.end);
    }
    rows.prefetch();
    if (at < w.f.end) {      // (a short last region has rows without bytes)
      const uint32_t o = at + lane * 16u;
      uint4 v[NS][U];
#pragma unroll
      for (int k = 0; k < NS; ++k)
#pragma unroll
        for (int u = 0; u < U; ++u) v[k][u] = rs_ld16_stream(S[k], o + u * 1024u);
#pragma unroll
      for (int k = 1; k < NS; ++k) op_batch<DT, U>(v[0], v[k], op);
#pragma unroll
      for (int k = 0; k < ND; ++k)
#pragma unroll
        for (int u = 0; u < U; ++u) rs_st16(D[k], o + u * 1024u, v[0][u]);
    }
    if (!rows.next()) break;
  }
}

template <int DT>
__device__ __forceinline__ void sweep_any(const u64* src_tab, const u64* dst_tab, bool to_all, Sweep& w, Rows& rows, uint32_t lane, int op) {
  constexpr int U = 2, NS = 8;      // vectors per source (sweep_row_bytes) and sources in flight
  const uint32_t R = w.R;
  LaneTable S(src_tab, R, lane), D(dst_tab, R, lane);
  uint32_t at;
  bool moved;
  while (w.row(rows.row, U * 1024u, at, moved)) {
    if (moved) {
      S = LaneTable(src_tab, R, lane, w.f.src, w.first);
      D = LaneTable(dst_tab, R, lane, w.f.dst, w.first);
    }
    rows.prefetch();
    if (at < w.f.end) {
      const uint32_t o = at + lane * 16u;
      uint4 acc[U];
      for (uint32_t k0 = 0; k0 < R; k0 += NS) {
        uint4 v[NS][U];
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          if (k0 + k < R) {
            const __amdgpu_buffer_rsrc_t r = S.rsrc(k0 + k, w.f.end);
#pragma unroll
            for (int u = 0; u < U; ++u) v[k][u] = rs_ld16_stream(r, o + u * 1024u);
          }
        }
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          if (k0 + k < R) {
            if (k0 + k == 0) {
#pragma unroll
              for (int u = 0; u < U; ++u) acc[u] = v[0][u];
            } else op_batch<DT, U>(acc, v[k], op);
          }
        }
      }
      for (uint32_t d = to_all ? 0u : R - 1u; d < R; ++d) {
        const __amdgpu_buffer_rsrc_t r = D.rsrc(d, w.f.end);
#pragma unroll
        for (int u = 0; u < U; ++u) rs_st16(r, o + u * 1024u, acc[u]);
      }
    }
    if (!rows.next()) break;
  }
}

// Copies store half a row at a time to every destination (R = 8; sixteen stores): 2415 MB from one buffer to eight in 420 us, a row of
// 4 KiB at a time in 457.
template <int ND>
__device__ __forceinline__ void sweep_copy(const u64* src_tab, const u64* dst_tab, Sweep& w, Rows& rows, uint32_t lane) {
  constexpr int U = 16 / ND, B = 4 / U;      // (sweep_row_bytes)
  __amdgpu_buffer_rsrc_t S, D[ND];
  uint32_t at;
  bool moved;
  while (w.row(rows.row, B * U * 1024u, at, moved)) {
    if (moved) {
      const LaneTable a(src_tab, ND, lane, w.f.src, w.first), b(dst_tab, ND, lane, w.f.dst, w.first);
      S = a.rsrc(ND - 1, w.f.end);
#pragma unroll
      for (int k = 0; k < ND; ++k) D[k] = b.rsrc(k, w.f.end);
    }
    rows.prefetch();
    const uint32_t o = at + lane * 16u;
    uint4 v[B * U];
#pragma unroll
    for (int u = 0; u < B * U; ++u) v[u] = rs_ld16_stream(S, o + u * 1024u);
#pragma unroll
    for (int h = 0; h < B * U; h += U)
#pragma unroll
      for (int k = 0; k < ND; ++k)
#pragma unroll
        for (int u = h; u < h + U; ++u) rs_st16(D[k], o + u * 1024u, v[u]);
    if (!rows.next()) break;
  }
}

template <int DT>
__device__ __forceinline__ void sweep_reduce(const u64* src_tab, const u64* dst_tab, bool to_all, Sweep& w, Rows& rows, uint32_t lane, int op) {
  if (w.R == 8 && to_all) sweep_fixed<DT, 8, true>(src_tab, dst_tab, w, rows, lane, op);
  else if (w.R == 8) sweep_fixed<DT, 8, false>(src_tab, dst_tab, w, rows, lane, op);
  else if (w.R == 4 && to_all) sweep_fixed<DT, 4, true>(src_tab, dst_tab, w, rows, lane, op);
  else if (w.R == 4) sweep_fixed<DT, 4, false>(src_tab, dst_tab, w, rows, lane, op);
  else sweep_any<DT>(src_tab, dst_tab, to_all, w, rows, lane, op);
  if (w.ends) fold_ends<DT>(src_tab, w.R, dst_tab + (to_all ? 0u : w.R - 1u), to_all ? w.R : 1u, w.ends_at, w.ends, lane, op, w.own_src, w.own_dst);
}

__device__ __forceinline__ void sweep_dispatch(int dtype, const u64* src_tab, const u64* dst_tab, Sweep& w, Rows& rows, uint32_t lane) {
  if (fold_copies((int)w.kind)) {      // (on four or eight ranks)
    if (w.R == 8) sweep_copy<8>(src_tab, dst_tab, w, rows, lane);
    else sweep_copy<4>(src_tab, dst_tab, w, rows, lane);
    if (w.ends) fold_ends<DT_F16>(src_tab + (w.R - 1u), 1, dst_tab, w.R, w.ends_at, w.ends, lane, OP_SUM, w.own_src, w.own_dst);
    return;
  }
  const int op = dtype >> 4;
  const bool to_all = fold_to_all((int)w.kind);
  switch (dtype & 15) {
    case DT_F32: sweep_reduce<DT_F32>(src_tab, dst_tab, to_all, w, rows, lane, op); break;
    case DT_BF16: sweep_reduce<DT_BF16>(src_tab, dst_tab, to_all, w, rows, lane, op); break;
    case DT_F16: sweep_reduce<DT_F16>(src_tab, dst_tab, to_all, w, rows, lane, op); break;
    default: sweep_reduce<DT_I32>(src_tab, dst_tab, to_all, w, rows, lane, op); break;
  }
}

}  // namespace

#endif
