// The schedule's geometry and the plan, shared by the table builder (which
// stores the schedule images and the plan with the routing tables) and the
// kernels that run them.
#pragma once

#include "common.h"
#include "kernels.h"

namespace moe {

// XCD-aware tile queues.  A tile's weight slab is its GEMM0 column tile, or
// its GEMM1 (column tile, split) pair; the tiles of one slab share the slab's
// weights, so they are queued for one XCD (slab class = slab mod NXCD) and
// read them from that XCD's L2.  Stage = (chunk, phase) in DAG order; each
// stage has one queue per class, the row tile fastest within a slab.
__device__ __forceinline__ int class_slabs(int ns, int x) { return ns > x ? (ns - x + NXCD - 1) / NXCD : 0; }

// Readiness levels order the row tiles of a stage by when their inputs can be
// complete.  Shared-expert rows are read straight from x: level 0, ready at
// launch.  With every worker copying rows at the start, the routed row tiles
// all complete at nearly the same time, and one routed level (NLVL = 1)
// measures fastest: it keeps the row tiles of one expert and weight slab
// together, so the tiles running on an XCD share that slab in its L2 (levels
// by the fraction of a segment that must be written spread the first claims
// over every expert and slab and fetch the weights several times over).

// Queue order of the stages (chunk, phase) of a K-chunk schedule, skewed by
// one chunk: (0,G0), (1,G0), (0,G1), (2,G0), (1,G1), ..., (K-1,G0), (K-2,G1),
// (K-1,G1).  Workers reach chunk q's GEMM1 tiles only after claiming chunk
// q+1's GEMM0 tiles, which depend on dispatch alone, so chunk q's last GEMM0
// tiles finish while those run instead of holding up a worker at every chunk
// boundary.  Returns chunk << 1 | phase.
__device__ __forceinline__ int stage_qph(int s, int K) {
  if (s == 0) return 0;
  if (s >= 2 * K - 1) return ((K - 1) << 1) | 1;
  const int j = (s + 1) >> 1;
  return (s & 1) ? (j << 1) : (((j - 1) << 1) | 1);
}

// Wavefront argmin of (t, i) (lanes with i < 0 hold no point): the smallest
// t, the lowest i among equal ones, with n carried along; lane 0 ends with
// the result.  DPP exchanges within each row of 16 lanes (xor 1, xor 2, then
// the half-row and row mirrors, each pairing the lanes of two disjoint halves),
// then the four rows' results through readlane.  The order of the minimum
// with its index tie-break is total, so the pairing order does not matter.
__device__ __forceinline__ void argmin_take(double& t, int& i, int& n, double t2, int i2, int n2) {
  if (i2 >= 0 && (i < 0 || t2 < t || (t2 == t && i2 < i))) {
    t = t2;
    i = i2;
    n = n2;
  }
}
template <int CTRL>
__device__ __forceinline__ void argmin_dpp_step(double& t, int& i, int& n) {
  const uint64_t b = (uint64_t)__builtin_bit_cast(uint64_t, t);
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
  const int i2 = __builtin_amdgcn_mov_dpp(i, CTRL, 0xF, 0xF, false);
  const int n2 = __builtin_amdgcn_mov_dpp(n, CTRL, 0xF, 0xF, false);
  const double t2 = __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
  argmin_take(t, i, n, t2, i2, n2);
}
__device__ __forceinline__ void wave_argmin(double& t, int& i, int& n) {
  argmin_dpp_step<0xB1>(t, i, n);   // quad_perm [1, 0, 3, 2]
  argmin_dpp_step<0x4E>(t, i, n);   // quad_perm [2, 3, 0, 1]
  argmin_dpp_step<0x141>(t, i, n);  // row_half_mirror
  argmin_dpp_step<0x140>(t, i, n);  // row_mirror
  const uint64_t b = (uint64_t)__builtin_bit_cast(uint64_t, t);
#pragma unroll
  for (int r = 1; r < 4; ++r) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, 16 * r);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 16 * r);
    const int i2 = __builtin_amdgcn_readlane(i, 16 * r);
    const int n2 = __builtin_amdgcn_readlane(n, 16 * r);
    argmin_take(t, i, n, __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo), i2, n2);
  }
}

// The cost model's plan on one wavefront (all 64 lanes call; lane 0 ends with
// it in p): Eq 15 at every grid point, one point per lane, with its steal
// count (Eq 11-14) alongside; Eq 16 by a wavefront argmin in the host model's
// order (c ascending, then K): the smallest T_total, the lowest grid index
// among equal ones, which is the first strict minimum of the host's scan.
// cal, st: the calibration table and the routing stats (LDS).
__device__ __forceinline__ void model_plan(const DevCalib& cal, const int* st, int H, int F, int shared_rows, int N,
                                           moe_plan& p) {
  const int lane = threadIdx.x & (WAVE - 1);
  double wc, wd, wb;
  cm_volumes(st, H, F, shared_rows, cal.literal, &wc, &wd, &wb);
  const int nk = cal.n_k, npt = cal.n_c * nk;
  double best = 0.0;
  int bi = -1;
  for (int i = lane; i < npt; i += WAVE) {
    const double t = cm_t_total(cal, i / nk, i - (i / nk) * nk, wc, wd, wb);
    if (bi < 0 || t < best) { best = t; bi = i; }
  }
  int ns = 0;
  if (bi >= 0) {
    long long nt_by_k[MOE_CALIB_MAX_K];
    for (int j = 0; j < nk; ++j) nt_by_k[j] = st[ST_NTK + kopt_index(cal.kk[j])];
    moe_plan q;
    cm_finish(cal, N, wc, wd, wb, nt_by_k, bi / nk, bi - (bi / nk) * nk, best, &q);
    ns = q.n_steal;
  }
  wave_argmin(best, bi, ns);
  if (lane == 0) {
    p.c = cal.c[bi / nk];
    p.K = cal.kk[bi - (bi / nk) * nk];
    p.n_steal = ns;
    p.final_all = 1;
    p.t_pred_s = best;
  }
}

}  // namespace moe
