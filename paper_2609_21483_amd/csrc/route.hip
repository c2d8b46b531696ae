// The routing tables of this GPU's share (section 3.1 descriptors X_local,
// X_in, X_in^uniq; the dispatch permutation and its deduplication, section 4;
// the chunk offsets of section 3.2.1) and the weight packing.
//
// Everything here is deterministic: slots come from block histograms, an
// ordered scan and lane masks, never from atomic slot claiming.
#include "common.h"
#include "gemm.h"
#include "kernels.h"
#include "sched.h"

namespace moe {

// ---------------------------------------------------------------------------
// Routing tables.  A pair (g, j) is local when id = topk_idx[g,j] is in
// [0, E), not repeated earlier in row g, and le = id - e0 is in [0, E_l).
// ---------------------------------------------------------------------------
constexpr int TB = NTH;  // tokens per count block of tab_count_kernel

// local expert of entry j < k of a token's ids, or -1; straight-line, as every
// entry's evaluation is in the same few instructions
__device__ __forceinline__ int local_expert(const TableArgs& a, const int* ids, int j, bool valid, bool& bad) {
  const int id = ids[j];
  bool wrong = (unsigned)id >= (unsigned)a.E;
#pragma unroll
  for (int jj = 0; jj < j; ++jj) wrong |= ids[jj] == id;
  const bool in = valid & (j < a.k);
  bad |= in & wrong;
  const int le = id - a.e0;
  return (in & !wrong & ((unsigned)le < (unsigned)a.El)) ? le : -1;
}

__device__ __forceinline__ void count_block(const TableArgs& a, const int* ids, bool valid) {
  __shared__ int hist[MAX_SEG];
  __shared__ int nbad;
  const int tid = threadIdx.x;
  for (int i = tid; i < a.El; i += NTH) hist[i] = 0;
  if (tid == 0) nbad = 0;
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int j = 0; j < MAX_TOPK; ++j) {
    const int le = local_expert(a, ids, j, valid, bad);
    if (le >= 0) atomicAdd(&hist[le], 1);
  }
  if (bad) {
    atomicAdd(&nbad, 1);
    atomicOr(a.err, ERR_ROUTING);
  }
  __syncthreads();
  for (int i = tid; i < a.El; i += NTH) a.blk_cnt[(size_t)blockIdx.x * a.El + i] = hist[i];
  if (tid == 0) a.blk_bad[blockIdx.x] = nbad;
}

// the ids of token g (clamped to the last token), every load in flight at once
__device__ __forceinline__ void load_ids(const TableArgs& a, int g, int* ids) {
  const int32_t* src = a.topk_idx + (size_t)min(g, a.T - 1) * a.k;
#pragma unroll
  for (int j = 0; j < MAX_TOPK; ++j) ids[j] = j < a.k ? src[j] : -1;
}

__global__ void __launch_bounds__(NTH) tab_count_kernel(TableArgs a) {
  const int g = blockIdx.x * TB + threadIdx.x;
  const bool valid = g < a.T;
  int ids[MAX_TOPK];
  load_ids(a, g, ids);
  count_block(a, ids, valid);
}

// Expert offsets and each count block's offset within every expert, where
// the count words are too many for every table block to sum them itself
// (TAB_SUM_MAX): one wavefront per expert scans the counts 64 at a time.
__global__ void __launch_bounds__(TAB_SCAN_THREADS) tab_scan_kernel(TableArgs a) {
  constexpr int NW = TAB_SCAN_THREADS / WAVE;
  __shared__ int tot[MAX_EL];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  for (int le = wave; le < a.El; le += NW) {
    int carry = 0;
    for (int b0 = 0; b0 < a.nblk; b0 += WAVE) {
      const int b = b0 + lane;
      const int c = b < a.nblk ? a.blk_cnt[(size_t)b * a.El + le] : 0;
      int x = c;
#pragma unroll
      for (int d = 1; d < WAVE; d <<= 1) {
        const int y = __shfl_up(x, d, WAVE);
        if (lane >= d) x += y;
      }
      if (b < a.nblk) a.blk_off[(size_t)b * a.El + le] = carry + x - c;
      carry += __shfl(x, WAVE - 1, WAVE);
    }
    if (lane == 0) tot[le] = carry;
  }
  __syncthreads();
  if (tid == 0) {
    int s = 0;
    for (int le = 0; le < a.El; ++le) { a.off[le] = s; s += tot[le]; }
    a.off[a.El] = s;
  }
}

__device__ __forceinline__ int wave_incl_scan(int x, int lane) {
#pragma unroll
  for (int d = 1; d < WAVE; d <<= 1) {
    const int y = __shfl_up(x, d, WAVE);
    if (lane >= d) x += y;
  }
  return x;
}

// barrier for LDS traffic only (__syncthreads also waits for every global
// store of the wavefront)
__device__ __forceinline__ void lds_sync() { gemm::lds_barrier(); }
// LDS writes of this wavefront, before its own lanes read them
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// first token of chunk q of K = 2^ki: ceil(q T / K) (T <= 2^22, q <= 8)
__device__ __forceinline__ int chunk_bnd(int T, int ki, int q) { return (q * T + (1 << ki) - 1) >> ki; }

// Rows of segment seg (local experts, then shared experts) in chunk q of
// the K-chunk option ki; so: the sub_off tables.  A shared expert takes rank
// 0's tokens of the chunk.
__device__ __forceinline__ int seg_chunk_rows(const TableArgs& a, const int* so, int ki, int seg, int q) {
  if (seg < a.El) {
    const int* e = so + (ki * a.El + seg) * SUBW;
    return e[q + 1] - e[q];
  }
  return max(0, min(chunk_bnd(a.T, ki, q + 1), a.Tr) - chunk_bnd(a.T, ki, q));
}

// The tables of one GPU's share in one launch: every workgroup ranks the
// slots of its TBN tokens, and the last one to finish completes what needs
// all of them (row maps, stats, schedule images, the plan).
//   - Ranks: a 64-bit mask per (wavefront, local expert) of the lanes that
//     selected it, set by LDS atomics; a slot is the expert's offset, plus the
//     selections of earlier workgroups (summed from the count blocks, or from
//     tab_scan_kernel's result) and wavefronts, plus the lower lanes of its
//     own mask.  Slots order by expert, then token, whatever the schedule.
//   - The first slot of every expert at or after each rank boundary and each
//     inner chunk boundary in the workgroup's tokens, and the unique-token
//     counts, go to the last workgroup through agent-coherent stores and
//     atomics, drained before its arrival is counted; the slots are written
//     while that count's round trip is out.
//   - The last workgroup gives each chunk option two wavefronts (row map;
//     schedule image) and the plan one of its own: the cost model's dependent
//     fp64 divisions take 2 us.
// The steps are short and depend on each other, so they are bound by the
// latency of memory, instruction fetch and launches, not by their work.  As
// separate kernels (scan, slots, row map, schedules; 3 to 20 us each) they
// took 35 us for 32 tokens, 41 us for 1332 and 56 us for 32768 (32 local
// experts of 128, k = 8); in one they take 10, 16 and 18 us, 2 us of it the
// plan.
template <int TBN, bool ONE>
__global__ void __launch_bounds__(TBN + WAVE) tab_build_kernel(TableArgs a) {
  constexpr int NW = TBN / WAVE;  // wavefronts with tokens; one more has none
  constexpr int NT = TBN + WAVE;
  static_assert(NW >= 2 * KOPT, "two wavefronts per chunk option");
  __shared__ uint64_t mk[NW][MAX_EL];
  __shared__ int wp[NW][MAX_EL];  // first slot of each (wavefront, expert)
  __shared__ int pre[MAX_EL], tot[MAX_EL], offs[MAX_EL + 1];
  __shared__ int uq[MAX_R];
  __shared__ int nbad, last, xl;
  __shared__ int ntk[KOPT];
  __shared__ int so[KOPT * MAX_EL * SUBW];   // the chunk offsets
  __shared__ int rb[(MAX_R - 1) * MAX_EL];   // the rank boundaries' first slots (ONE)
  __shared__ int base[KOPT][MAX_K + 1];      // row tiles before each chunk
  __shared__ DevCalib cal;
  __shared__ int st[ST_WORDS];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const int El = a.El, R = a.R, T = a.T, nrb = R - 1;
  const int t0 = blockIdx.x * TBN, g = t0 + tid;
  const bool valid = tid < TBN && g < T;

  int ids[MAX_TOPK], le_j[MAX_TOPK];
  load_ids(a, g, ids);
  constexpr int NCW = (int)(sizeof(DevCalib) / 4);
  static_assert(NCW <= NT, "one calibration word per thread");
  const uint32_t cw = tid < NCW ? reinterpret_cast<const uint32_t*>(a.calib)[tid] : 0u;
  for (int i = tid; i < NW * MAX_EL; i += NT) mk[i / MAX_EL][i % MAX_EL] = 0;
  if (tid < MAX_EL) { pre[tid] = 0; tot[tid] = 0; }
  if (tid < R) uq[tid] = 0;
  if (tid == 0) { nbad = 0; xl = 0; }
  __syncthreads();
  bool bad = false, any = false;
#pragma unroll
  for (int j = 0; j < MAX_TOPK; ++j) {
    le_j[j] = local_expert(a, ids, j, valid, bad);
    any |= le_j[j] >= 0;
    if (le_j[j] >= 0) atomicOr((unsigned long long*)&mk[wave][le_j[j]], 1ull << lane);
  }
  if (any) atomicAdd(&uq[g / a.Tr], 1);
  if (tid < NCW) reinterpret_cast<uint32_t*>(&cal)[tid] = cw;
  if constexpr (ONE) {
    if (bad) {
      atomicAdd(&nbad, 1);
      atomicOr(a.err, ERR_ROUTING);
    }
  } else if (a.scanned) {
    if (tid < El) {
      pre[tid] = a.blk_off[(size_t)(t0 / a.cb) * El + tid];
      tot[tid] = a.off[tid + 1] - a.off[tid];
    }
  } else if (tid < TBN) {
    // thread (slice, le) sums every (TBN / elp)-th count block of expert le
    const int b0 = t0 / a.cb, sh = El <= 1 ? 0 : 32 - __builtin_clz((unsigned)(El - 1));
    const int le = tid & ((1 << sh) - 1), ns = TBN >> sh;
    if (le < El) {
      int p = 0, s = 0;
      constexpr int U = 8;
#pragma unroll 1
      for (int b = tid >> sh; b < a.nblk; b += U * ns) {
        int c[U];
#pragma unroll
        for (int i = 0; i < U; ++i) c[i] = a.blk_cnt[(size_t)min(b + i * ns, a.nblk - 1) * El + le];
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const int bb = b + i * ns;
          s += bb < a.nblk ? c[i] : 0;
          p += bb < b0 ? c[i] : 0;
        }
      }
      atomicAdd(&pre[le], p);
      atomicAdd(&tot[le], s);
    }
  }
  __syncthreads();
  // wave 0, lane le: the expert's offset, then the first slot of every
  // wavefront's selections
  if (wave == 0) {
    int n[NW], c = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      n[w] = c;
      c += lane < El ? __popcll(mk[w][lane]) : 0;
    }
    const int t = ONE ? c : (lane < El ? tot[lane] : 0);
    const int x = wave_incl_scan(t, lane);
    if (lane < El) {
      offs[lane + 1] = x;
      const int b = x - t + (ONE ? 0 : pre[lane]);
#pragma unroll
      for (int w = 0; w < NW; ++w) wp[w][lane] = b + n[w];
    }
    if (lane == 0) offs[0] = 0;
  }
  __syncthreads();
  // boundaries: rank r*Tr (0 < r < R), then the inner chunk boundaries
  // ceil(q*T/K) (0 < q < K) of K = 2, 4, 8; chunk(g) = floor(g*K/T) >= q
  // exactly when g >= ceil(q*T/K).  Boundary bi of them; ki, q: the chunk
  // option and chunk of an inner one.
  auto boundary = [&](int bi, int& ki, int& q) {
    if (bi < nrb) return (bi + 1) * a.Tr;
    const int c = bi - nrb;  // 0: K = 2, q = 1; 1..3: K = 4, q = 1..3; 4..10: K = 8, q = 1..7
    ki = c < 1 ? 1 : (c < 4 ? 2 : 3);
    q = c - (ki == 1 ? 0 : ki == 2 ? 1 : 4) + 1;
    return chunk_bnd(T, ki, q);
  };
  {
    const int t1 = min(T, t0 + TBN), nbnd = nrb + 1 + 3 + 7;
#pragma unroll 1
    for (int v = tid; v < nbnd * El; v += NT) {
      const int bi = v / El, le = v - bi * El;
      int ki = 0, q = 0;
      const int b = boundary(bi, ki, q);
      if (b < t0 || b >= t1) continue;
      const int p = b - t0, pw = p / WAVE, pl = p % WAVE;
      const int cnt = wp[pw][le] + __popcll(mk[pw][le] & ((1ull << pl) - 1));
      if constexpr (ONE) {
        if (bi < nrb) rb[bi * El + le] = cnt;
        else so[(ki * El + le) * SUBW + q] = cnt;
      } else {
        if (bi < nrb) st_relaxed(&a.rbnd[le * (R + 1) + bi + 1], cnt);
        else st_relaxed(&a.sub_off[(ki * El + le) * SUBW + q], cnt);
      }
    }
  }
  if constexpr (!ONE) {
    if (tid < R && uq[tid]) fetch_add_relaxed(&a.uniq_acc[tid], uq[tid]);
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's boundary stores and counts are at the coherence point
    __syncthreads();
    if (tid == 0) last = fetch_add_relaxed(a.done, 1) == (int)gridDim.x - 1;
  }
  if (valid) {
    int first = -1, first_le = MAX_SEG;
    int32_t* slot = a.slot + (size_t)g * a.k;
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) {
      const int le = le_j[j], lc = max(le, 0);
      const int s = le < 0 ? -1 : wp[wave][lc] + (int)__popcll(mk[wave][lc] & ((1ull << lane) - 1));
      if (s >= 0) a.inv[s] = g * a.k + j;
      if (s >= 0 && le < first_le) { first_le = le; first = s; }
      if (j < a.k) slot[j] = s;
    }
    a.first_slot[g] = first;
  }
  lds_sync();
  if constexpr (!ONE) {
    if (!last) return;
  }

  // ---- the last workgroup: everything that needs every token ----
  if constexpr (!ONE) {
    if (tid == 0) st_relaxed(a.done, 0);
    int nb = 0;
    for (int b = tid; b < a.nblk; b += NT) nb += a.blk_bad[b];
    if (nb) atomicAdd(&nbad, nb);
    if (tid < R) {
      uq[tid] = ld_relaxed(&a.uniq_acc[tid]);
      st_relaxed(&a.uniq_acc[tid], 0);
    }
#pragma unroll 2
    for (int v = tid; v < 11 * El; v += NT) {
      int ki = 0, q = 0;
      const int c = v / El, le = v - c * El;
      const int b = boundary(nrb + c, ki, q), at = (ki * El + le) * SUBW + q;
      // a boundary at T (fewer tokens than chunks) is in no workgroup: every
      // slot of the expert lies before it
      so[at] = b < T ? ld_relaxed(&a.sub_off[at]) : offs[le + 1];
    }
  } else {
#pragma unroll 1
    for (int v = tid; v < 11 * El; v += NT) {
      int ki = 0, q = 0;
      const int c = v / El, le = v - c * El;
      if (boundary(nrb + c, ki, q) >= T) so[(ki * El + le) * SUBW + q] = offs[le + 1];
    }
  }
#pragma unroll 1
  for (int v = tid; v < KOPT * El * SUBW; v += NT) {
    const int kl = v / SUBW, q = v - kl * SUBW, ki = kl / El, le = kl - ki * El, K = kopt_value(ki);
    if (q == 0 || q >= K) so[v] = q == 0 ? offs[le] : q == K ? offs[le + 1] : 0;
  }
#pragma unroll 1
  for (int v = tid; v < El * R; v += NT) {
    const int le = v / R, r = v - le * R;
    int hi = offs[le + 1], lo = offs[le];
    if (r + 1 < R) hi = ONE ? rb[r * El + le] : ld_relaxed(&a.rbnd[le * (R + 1) + r + 1]);
    if (r > 0) lo = ONE ? rb[(r - 1) * El + le] : ld_relaxed(&a.rbnd[le * (R + 1) + r]);
    a.cnt_rank[v] = hi - lo;
    if (r == 0) atomicAdd(&xl, hi - lo);
  }
  if (tid <= El) a.off[tid] = offs[tid];
  if (tid < R) a.uniq[tid] = uq[tid];
  lds_sync();
  for (int v = tid; v < KOPT * El * SUBW; v += NT) a.sub_off[v] = so[v];
  // row tiles of the layer at each chunk option (the cost model's tile
  // counts, Eq 14)
  const int nseg = El + a.S;
  if (wave < KOPT) {
    const int ki = wave, n = nseg << ki;
    int tiles = 0;
#pragma unroll 1
    for (int v = lane; v < n; v += WAVE) tiles += (seg_chunk_rows(a, so, ki, v >> ki, v & ((1 << ki) - 1)) + BM - 1) / BM;
    tiles = wave_incl_scan(tiles, lane);
    if (lane == WAVE - 1) ntk[ki] = tiles * (a.wide0 + a.wide1);
  }
  lds_sync();
  if (wave == NW) {
    // stats (word 8, ST_CANDS, belongs to the gate), then the cost model's
    // plan of these tables under the current calibration (every workgroup of
    // a launch would evaluate the same; a prologue whose calibration
    // generation differs evaluates it again)
    int uin = 0;
    for (int r = 1; r < R; ++r) uin += uq[r];
    if (lane < ST_WORDS && lane != ST_CANDS) {
      const int X = offs[El];
      int v = 0;
      if (lane == ST_X) v = X;
      else if (lane == ST_XLOCAL) v = xl;
      else if (lane == ST_XIN) v = X - xl;
      else if (lane == ST_ULOCAL) v = uq[0];
      else if (lane == ST_UIN) v = uin;
      else if (lane == ST_BADIDS) v = nbad;
      else if (lane >= ST_NTK && lane < ST_NTK + KOPT) v = ntk[lane - ST_NTK];
      st[lane] = v;
      a.stats[lane] = v;
    }
    wave_lds_sync();
    moe_plan p;
    model_plan(cal, st, a.H, a.F, a.S * a.Tr, a.N, p);
    if (lane == 0) {
      StoredPlan* sp = reinterpret_cast<StoredPlan*>(a.sched + (size_t)KOPT * SCHED_WORDS);
      sp->p = p;
      sp->gen = a.calib_gen;
    }
  } else if (wave < KOPT) {
    // the row map (common.h): the (segment, chunk) pairs in segment-major
    // order, each taking its rows rounded up to a 32-row group; entries
    // q >= K are zero
    const int ki = wave, K = kopt_value(ki), n = nseg << ki;
    Sched* img = reinterpret_cast<Sched*>(a.sched + (size_t)ki * SCHED_WORDS);
    int carry = 0;
#pragma unroll 1
    for (int b = 0; b < n; b += WAVE) {
      const int v = b + lane, seg = v >> ki, q = v & (K - 1);
      const int sz = v < n ? align_rows(seg_chunk_rows(a, so, ki, seg, q)) : 0;
      const int x = wave_incl_scan(sz, lane), row0 = carry + x - sz;
      if (v < n) {
        a.row_off[(ki * nseg + seg) * SUBW + q] = row0;
        img->row0[q * nseg + seg] = row0;
        img->arow0[q * nseg + seg] = seg < El ? row0 : chunk_bnd(T, ki, q);
      }
      carry += __builtin_amdgcn_readlane(x, WAVE - 1);
    }
    const int nz = SUBW - K;
#pragma unroll 1
    for (int v = lane; v < nseg * nz; v += WAVE) a.row_off[(ki * nseg + v / nz) * SUBW + K + v % nz] = 0;
  } else if (wave < 2 * KOPT) {
    // the rest of the schedule image
    const int ki = wave - KOPT, K = kopt_value(ki), n = nseg << ki;
    Sched* img = reinterpret_cast<Sched*>(a.sched + (size_t)ki * SCHED_WORDS);
    int carry = 0;
#pragma unroll 1
    for (int b = 0; b < n; b += WAVE) {
      const int v = b + lane, q = v / nseg, seg = v - q * nseg;
      const int rows = v < n ? seg_chunk_rows(a, so, ki, seg, q) : 0;
      const int m = (rows + BM - 1) / BM;
      const int x = wave_incl_scan(m, lane), mb = carry + x - m;
      if (v < n) {
        img->rows[v] = rows;
        img->sbase[v] = seg < El ? so[(ki * El + seg) * SUBW + q] : chunk_bnd(T, ki, q);
        img->mb[v] = mb;
        if (seg == 0) base[ki][q] = mb;
      }
      carry += __builtin_amdgcn_readlane(x, WAVE - 1);
    }
    if (lane == 0) base[ki][K] = carry;
    wave_lds_sync();
    static_assert(NLVL == 1, "shared row tiles (level 0), then the routed ones");
    // A layer of few rows takes the time of streaming its experts' weights.
    // Whole-slab tiles stream 25 to 29 GB/s each (224 of them together 5.7
    // TB/s, 144 of them 4.2), so with few of them HBM idles, and narrow tiles
    // do better, although one streams 17 to 21 GB/s only, if the phase is deep
    // enough for their fixed cost.  Narrow against whole slabs on 256 workers,
    // weights from HBM, time of the layer over 900 random shapes and routings
    // (geometric means) by the number m of narrow tiles:
    //   GEMM0: H to 512 0.97 to 1.24; to 1024 1.08 up to m = 16, then 0.92 to 0.96 up
    //   to 256, 1.02 to 1.17 above; to 1536 1.03 (0.82 for m = 14 to 16), 0.86 to
    //   0.92, 0.98 to 1.08; past 1536 0.69 to 0.99 up to m = 512, 1.01 to 1.09 above.
    //   GEMM1 by the depth of a split: to 128 0.96 to 1.00 up to m = 128, 1.00 to
    //   1.17 above; to 512 0.92 to 1.01 up to 256, 1.02 to 1.17 above; past 512 0.72
    //   to 1.00 up to 512, 0.98 to 1.13 above.
    const int m0 = carry * ceil_div(2 * a.F, THIN_N), m1 = carry * ceil_div(a.H, THIN_N) * a.nsplit, d1 = a.F / a.nsplit;
    const bool thin0 = a.few && (a.H > 1536 ? m0 <= 2 * a.N : a.H > 512 && m0 > a.N / (a.H > 1024 ? 32 : 16) && m0 <= a.N);
    const bool thin1 = a.few && m1 <= (d1 > 512 ? 2 * a.N : d1 > 128 ? a.N : a.N / 2);
    const int nt0 = thin0 ? ceil_div(2 * a.F, THIN_N) : a.wide0;
    const int nt1 = thin1 ? ceil_div(a.H, THIN_N) : ceil_div(a.H, BN);
#pragma unroll 1
    for (int v = lane; v < 2 * K * NXCD; v += WAVE) {
      const int stage = v / NXCD, x = v % NXCD, qp = stage_qph(stage, K), q = qp >> 1;
      img->ncls[stage][x] = class_slabs(qp & 1 ? nt1 * a.nsplit : nt0, x) * (base[ki][q + 1] - base[ki][q]);
    }
    if (lane < K) {
      img->lvl[lane][0] = a.S ? a.S * ((seg_chunk_rows(a, so, ki, El, lane) + BM - 1) / BM) : 0;
      img->lvl[lane][1] = base[ki][lane + 1] - base[ki][lane];
    }
    if (lane <= K) img->bnd[lane] = chunk_bnd(T, ki, lane);
    if (lane == 0) {
      img->nt[0] = nt0;
      img->nt[1] = nt1;
      img->bn[0] = thin0 ? THIN_N : BN;
      img->bn[1] = thin1 ? THIN_N : BN;
      img->K = K;
      img->nseg = nseg;
      img->n_disp = ceil_div(T, a.dt);
      img->n_comb = ceil_div(T, a.ct);
    }
  }
}

template __global__ void tab_build_kernel<TAB_TB, true>(TableArgs);
template __global__ void tab_build_kernel<TAB_ONE_T, true>(TableArgs);
template __global__ void tab_build_kernel<TAB_TB, false>(TableArgs);

__global__ void zero_i32_kernel(int* p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// ---------------------------------------------------------------------------
// Weight packing (one-off, not part of the layer): transposes each expert's
// [H][F] / [F][H] matrix into the slab-tiled GEMM B layout (common.h).
// W1/W3 go to [2F][H] with 32-column groups interleaved (gate f..f+31, then
// up f..f+31), so one 64-column slice of GEMM0 holds matching gate and up
// columns; W2 goes to [H][F].  pack_pad_kernel zeroes the slab padding.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(NTH) pack_transpose_kernel(PackArgs a) {
  __shared__ uint16_t tile[32][33];
  const int seg = blockIdx.z;
  const uint16_t* src = a.src + (size_t)seg * a.rows * a.cols;
  uint16_t* dst = a.dst + (size_t)seg * a.seg_stride;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int i = ty; i < 32; i += 8) {
    int r = r0 + i, c = c0 + tx;
    if (r < a.rows && c < a.cols) tile[i][tx] = src[(size_t)r * a.cols + c];
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    int c = c0 + i, r = r0 + tx;  // dst row index is the source column
    if (r < a.rows && c < a.cols) {
      int drow = a.interleave ? (c / 32) * 64 + a.which * 32 + (c % 32) : c;
      dst[slab_index(drow, r, a.rows)] = tile[tx][i];
    }
  }
}

__global__ void __launch_bounds__(NTH) pack_pad_kernel(PadArgs a) {
  const int pad = (int)(slab_rows(a.R) - a.R);
  const long long per_seg = (long long)pad * a.K;
  for (long long v = (long long)blockIdx.x * NTH + threadIdx.x; v < per_seg * a.nseg; v += (long long)gridDim.x * NTH) {
    const int seg = (int)(v / per_seg);
    const long long e = v - seg * per_seg;
    const int n = a.R + (int)(e / a.K), k = (int)(e % a.K);
    a.dst[seg * a.seg_stride + slab_index(n, k, a.K)] = 0;
  }
}

}  // namespace moe
