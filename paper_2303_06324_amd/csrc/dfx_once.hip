// One collective in fold steps as one plain kernel.  Everything a rank does lies in its one step with data, and where all ranks
// have "submitted" because the call brings every buffer along, nothing is left to wait for: the launch is the wait, its end the
// completion.  No queues, no flags, no grid that has to be resident at once.
//
// What bounds a short one is the launch; a long one HBM, as in the daemon.  A workgroup takes a stretch of rows and ends, so the
// dispatcher hands the rows out: whoever is through gets the next workgroup, in the order of the rows.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfx_internal.h"
#include "dfx_geometry.h"
#include "dfx_movers.h"

// Four mover waves; three workgroups fit a compute unit without a vector register spilled (four, with spills, measured the same).
extern "C" __global__ void __launch_bounds__(DFX_ONCE_THREADS, 2) dfx_fold_once_kernel(DfxFoldOnce a) {
  __shared__ u64 tab_src[DFX_ONCE_MAX_RANKS], tab_dst[DFX_ONCE_MAX_RANKS];
  const uint32_t R = a.R, rank = blockIdx.x % R, group = blockIdx.x / R;      // (R = 8: a rank per XCD)
  const uint32_t lane = threadIdx.x & 63u, wave = bcast0(threadIdx.x >> 6);
  DfxStatic e = a.e;
  fold_entry(e, R, rank);
  const int kind = e.kind, dtype = e.dtype | (e.op << 4);
  const bool sweep = (e.flags & DFX_SQE_SWEEP) != 0, copies = fold_copies(kind), to_all = fold_to_all(kind);
  const FoldGeom fg = fold_geometry(e.count, e.block_elems, e.part_elems, 1u << 30, true, 0);
  if (threadIdx.x < R) {
    const uint32_t k = threadIdx.x, p = fold_peer(kind, R, rank, e.root, k);
    const u64 src = a.sendbuf[p] + (sweep ? 0u : fg.src), dst = a.recvbuf[p] + (sweep ? 0u : fg.dst);
    if (sweep || !copies) tab_src[k] = src;
    else if (k + 1 == R) tab_src[0] = src;
    if (sweep || to_all) tab_dst[k] = dst;
    else if (k + 1 == R) tab_dst[0] = dst;
  }
  __syncthreads();

  const OnceWave ow = once_wave(group, a.groups, a.rows_per_wave, wave);
  Rows rows;
  rows.ctr = nullptr; rows.drawn = 0;
  rows.waves = DFX_ONCE_WAVES; rows.left = a.rows_per_wave; rows.row = ow.row;
  if (sweep) {
    Sweep w;
    w.kind = (uint32_t)kind; w.R = R; w.rank = rank; w.longest = (uint32_t)e.count; w.total = e.block_elems;
    w.nreg = sweep_regions(kind, R);
    const uint32_t row = sweep_row_bytes(copies, R);
    w.rows = (w.longest + row - 1u) / row; w.all = w.rows * w.nreg;
    w.waves = DFX_ONCE_STRETCH; w.base = rank * DFX_ONCE_STRETCH; w.skip = DFX_ONCE_STRETCH * (R - 1u);
    w.lo = w.hi = 0;
    w.ends = 0;
    if (rank < w.nreg) {
      const FoldRegion own = sweep_region(kind, w.longest, w.total, rank);
      w.own_src = own.src; w.own_dst = own.dst;
      w.ends_at = ow.head ? 0u : own.end;
      w.ends = ow.head ? own.head : ow.tail && own.end < own.len ? own.len : 0u;
    }
    sweep_dispatch(dtype, tab_src, tab_dst, w, rows, lane);
  } else {
    Span sp;
    sp.head = fold_head(fg.dst, fg.bytes, e.nchan);
    sp.end = sp.head + ((fg.bytes - sp.head) & ~15u);
    sp.ends_at = ow.head ? 0u : sp.end;
    sp.ends = ow.head ? sp.head : ow.tail && sp.end < fg.bytes ? fg.bytes : 0u;
    fold_dispatch(dtype, tab_src, copies ? 1u : R, tab_dst, to_all ? R : 1u, sp, rows, lane);
  }
  // the outcome, behind everybody's stores: the last workgroup writes it
  if (a.count) {
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(global_ptr(a.clear), 0u, __ATOMIC_RELAXED, SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(a.count, 1u) + 1u == gridDim.x) {
      __hip_atomic_store(global_ptr(a.count), 0u, __ATOMIC_RELAXED, SCOPE_AGENT);
      __hip_atomic_store(global_ptr(a.status), 0u, __ATOMIC_RELAXED, SCOPE_AGENT);
    }
  }
}

__global__ void dfx_once_outcome_kernel(uint32_t* status) { *status = 0u; }

hipError_t dfx_fold_once_launch(const DfxFoldOnce& a, hipStream_t stream) {
  hipLaunchKernelGGL(dfx_fold_once_kernel, dim3(a.R * a.groups), dim3(DFX_ONCE_THREADS), 0, stream, a);
  if (a.status && !a.count) hipLaunchKernelGGL(dfx_once_outcome_kernel, dim3(1), dim3(1), 0, stream, a.status);
  return hipGetLastError();
}
