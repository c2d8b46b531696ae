// The gate by a certified filter, for batches in which evaluating every
// (token, expert) chain (gate.hip) costs more than finding the few that can
// change the routing: the same defined logits (fp32, one accumulator, h
// ascending, each product rounded before the add, then + bias), so the same
// ids and weights.  E > 32 (gate_filtered).
//   1. gate_prep:  WgT = Wg transposed ([E][H]) and ||w_e||_2.
//   2. gate_tile2 (E > 128: gate_tile): approximate logits L~ by bf16 MFMA (fp32 accumulation) and
//      ||x_g||_2, then the candidates: a bound d_e >= |L - L~| (from the
//      worst-case error of the two summations, |x|.|w| <= ||x|| ||w||) gives
//      intervals [L~ - d, L~ + d] that hold the defined logits.  tau = k-th
//      largest lower end; every expert whose upper end reaches tau is a
//      candidate.  The true top-k lie among the candidates and every other
//      expert is strictly below the k-th logit, so the top-k of the
//      candidates' defined logits is the top-k of all experts.
//   3. gate_chain_staged (k < 4 or E > 128: gate_chain): the defined logit of
//      every candidate.
//   4. gate_final: top-k and renormalised softmax weights of the candidates
//      (the normaliser over all experts cancels).
#include "common.h"
#include "gemm.h"
#include "kernels.h"

namespace moe {

__global__ void __launch_bounds__(NTH) gate_prep_kernel(FilterArgs a) {
  __shared__ float part[NTH / WAVE];
  const int e = blockIdx.x;
  const int tid = threadIdx.x;
  if (e == 0 && tid == 0) (*a.n_cands) = 0;  // the candidate pass counts the chains from here
  float ss = 0.0f;
  // PREP_V loads in flight per thread before their stores (the column of
  // Wg is strided by E, one 2-byte read per value)
  constexpr int PREP_V = 16;
  for (int h0 = 0; h0 < a.H; h0 += PREP_V * NTH) {
    uint16_t v[PREP_V];
#pragma unroll
    for (int i = 0; i < PREP_V; ++i) {
      const int h = h0 + i * NTH + tid;
      v[i] = h < a.H ? a.wg[(size_t)h * a.E + e] : (uint16_t)0;
    }
#pragma unroll
    for (int i = 0; i < PREP_V; ++i) {
      const int h = h0 + i * NTH + tid;
      if (h < a.H) {
        a.wgt[(size_t)e * a.H + h] = v[i];
        const float f = bf16_to_f32(v[i]);
        ss += f * f;
      }
    }
  }
#pragma unroll
  for (int d = WAVE / 2; d > 0; d >>= 1) ss += __shfl_xor(ss, d, WAVE);
  if ((tid & (WAVE - 1)) == 0) part[tid / WAVE] = ss;
  __syncthreads();
  if (tid == 0) {
    float t = 0.0f;
    for (int w = 0; w < NTH / WAVE; ++w) t += part[w];
    a.wn[e] = sqrtf(t);
  }
}

// lanes of one token's group of GG: reductions stay inside the group
constexpr int GG = 16;
constexpr int GTOK = NTH / GG;    // tokens per workgroup

__device__ __forceinline__ bool better(float v, int e, float bv, int be) {
  return (v > bv) | ((v == bv) & (e < be));
}
__device__ __forceinline__ void group_argmax(float& v, int& e) {
#pragma unroll
  for (int d = GG / 2; d > 0; d >>= 1) {
    const float ov = __shfl_xor(v, d, WAVE);
    const int oe = __shfl_xor(e, d, WAVE);
    if (better(ov, oe, v, e)) { v = ov; e = oe; }
  }
}

// The interval [lo, hi] that holds the defined logit: l is the approximate one
// with bias, norms = ||x|| ||w||.  Neither end is NaN.  While the norms bound the
// sum far from overflow, l is infinite or NaN exactly if the bias is, and so is
// the defined logit (a masked expert: both ends -inf, so it is a candidate only
// where fewer than k experts are left; NaN is never chosen); past that, or with
// an infinite or NaN input, anything may come out.
__device__ __forceinline__ void interval(float l, float norms, float bound, float& lo, float& hi) {
  float d = bound * norms;
  d = d + 4.0f * 5.9604645e-8f * (fabsf(l) + d) + 1e-30f;
  lo = l - d;
  hi = l + d;
  if (!(fabsf(l) < INFINITY)) lo = hi = l == l ? l : -INFINITY;
  if (!(norms < 1e30f)) {
    lo = -INFINITY;
    hi = INFINITY;
  }
}

// the interval of (g, e) from the logits in memory
__device__ __forceinline__ void interval_at(const FilterArgs& a, int g, int e, float xn, float& lo, float& hi) {
  float l = a.lt[(size_t)g * a.E + e];
  if (a.bias) l = l + a.bias[e];
  interval(l, xn * a.wn[e], a.bound, lo, hi);
}

// Candidates of the ntok tokens from g0 (one workgroup of NTH threads, GTOK
// tokens per pass, a token's experts spread over the GG lanes of its group,
// EPL each): tau = the k-th largest lower end; every expert whose upper end
// reaches tau becomes a chain (g, e) of the chain list.  A first pass counts
// each token's candidates, the tile takes its range of the list with one
// atomic, and a second pass writes each token's chains in ascending expert
// order (experts of neighbouring chains then differ in their low bits,
// which spreads the chain kernel's reads of their gate rows over the LDS
// banks).  t_cnt, t_off, t_tau: ntok entries of workgroup memory.
template <int EPL>
__device__ __forceinline__ void cand_tile(const FilterArgs& a, int g0, int ntok, int* t_cnt, int* t_off, float* t_tau,
                                          int& base_s) {
  const int tid = threadIdx.x, grp = tid / GG, gl = tid % GG;
  for (int t0 = 0; t0 < ntok; t0 += GTOK) {
    const int g = g0 + t0 + grp;
    const bool valid = g < a.T;
    const int gs = valid ? g : 0;
    const float xn = a.xn[gs];
    float lo[EPL], hi[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int e = gl + GG * i;
      lo[i] = hi[i] = -INFINITY;
      if (e < a.E) interval_at(a, gs, e, xn, lo[i], hi[i]);
    }
    float tau = -INFINITY;
    for (int r = 0; r < a.k; ++r) {
      float v = -INFINITY;
      int e = 1 << 30;
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (better(lo[i], gl + GG * i, v, e)) { v = lo[i]; e = gl + GG * i; }
      group_argmax(v, e);
      tau = v;
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (gl + GG * i == e) lo[i] = -INFINITY;
    }
    int mine = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) mine += valid && gl + GG * i < a.E && hi[i] >= tau;
#pragma unroll
    for (int d = GG / 2; d > 0; d >>= 1) mine += __shfl_xor(mine, d, WAVE);
    if (gl == 0) {
      t_cnt[t0 + grp] = mine;
      t_tau[t0 + grp] = tau;
    }
  }
  __syncthreads();
  if (tid < WAVE) {  // exclusive scan of the counts, one atomic for the tile
    int carry = 0;
    for (int b = 0; b < ntok; b += WAVE) {
      const int c = b + tid < ntok ? t_cnt[b + tid] : 0;
      int x = c;
#pragma unroll
      for (int d = 1; d < WAVE; d <<= 1) {
        const int y = __shfl_up(x, d, WAVE);
        if (tid >= d) x += y;
      }
      if (b + tid < ntok) t_off[b + tid] = carry + x - c;
      carry += __shfl(x, WAVE - 1, WAVE);
    }
    if (tid == 0) base_s = atomicAdd(a.n_cands, carry);
  }
  __syncthreads();
  const int gw = (tid & (WAVE - 1)) / GG;  // the group's place in its wavefront
  for (int t0 = 0; t0 < ntok; t0 += GTOK) {
    const int g = g0 + t0 + grp;
    const bool valid = g < a.T;
    const int gs = valid ? g : 0;
    const float xn = a.xn[gs];
    const float tau = t_tau[t0 + grp];
    const int tb = base_s + t_off[t0 + grp];
    if (valid && gl == 0) {
      a.tok_base[g] = tb;
      a.tok_n[g] = t_cnt[t0 + grp];
    }
    int run = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int e = gl + GG * i;
      bool c = false;
      if (valid && e < a.E) {
        float lo, hi;
        interval_at(a, gs, e, xn, lo, hi);
        c = hi >= tau;
      }
      const uint32_t gm = (uint32_t)(__ballot(c) >> (gw * GG)) & ((1u << GG) - 1);
      if (c) {
        const int pos = tb + run + __builtin_popcount(gm & ((1u << gl) - 1));
        a.ch_g[pos] = g;
        a.ch_e[pos] = e;
      }
      run += __builtin_popcount(gm);
    }
  }
}

// E > 128: the approximate logits of a tile of GT_M tokens x GT_N experts per
// pass over the experts, on v_mfma_f32_32x32x16_bf16 (fp32 accumulation) with
// both operands streamed through an LDS ring of GT_NS stages of 64-deep
// k-steps by direct global->LDS loads.  In a load instruction 8 lanes fetch
// one row's 128 contiguous bytes, so it covers 8 whole lines (x is row-major
// with 2H-byte rows, the transposed gate too).  A row's 16-byte granules are
// stored XOR-swizzled by (row & 7), so that the fragment reads of 8 lanes on
// 8 consecutive rows hit distinct banks.  Four wavefronts in a 2 x 2 grid,
// each (GT_M / 2) tokens x 64 experts.  Token rows past T and gate rows past
// E repeat the last valid row; their sums are not stored.  The token norms
// come from the same x fragments (wavefronts of the first expert column, on
// the first pass).  Then the candidate pass of the tile's tokens.
constexpr int GT_N = 128;  // experts per pass
constexpr int GT_K = 64;   // values per row piece of a stage (128 bytes)
constexpr int GT_NS = 4;   // ring stages

template <int OUT>
__device__ __forceinline__ void gt_wait(int outstanding) {
  // at most `outstanding` stages (OUT DMA instructions each) still in flight
  if (outstanding >= 2) gemm::wait_vm<2 * OUT>();
  else if (outstanding == 1) gemm::wait_vm<OUT>();
  else gemm::wait_vm<0>();
}

template <int GT_M, int EPL>
__global__ void __launch_bounds__(NTH) gate_tile_kernel(FilterArgs a) {
  static_assert(NTH == 4 * WAVE && GT_M % 64 == 0 && GT_M % GTOK == 0, "gate tile geometry");
  constexpr int A_B = GT_M * 2 * GT_K, B_B = GT_N * 2 * GT_K, ST_B = A_B + B_B;
  constexpr int A_I = A_B / 1024 / 4, B_I = B_B / 1024 / 4;  // DMA instructions per wavefront and stage
  constexpr int WI = A_I + B_I;
  constexpr int MBW = GT_M / 64;  // 32-token blocks per wavefront
  static_assert(GT_NS - 2 <= 2, "gt_wait covers two stages in flight");
  __shared__ __attribute__((aligned(1024))) char ring[GT_NS * ST_B];
  __shared__ int t_cnt[GT_M], t_off[GT_M];
  __shared__ float t_tau[GT_M];
  __shared__ int base_s;
  const int lane = gemm::lane_here(), wave = gemm::opaque((int)(threadIdx.x / WAVE));
  const int wm = wave & 1, wn = wave >> 1;
  const int g0 = blockIdx.x * GT_M;
  const int H = gemm::opaque(a.H), nk = H / GT_K;
  const uint32_t ring0 = (uint32_t)gemm::opaque((int)gemm::lds_u32(ring));
  // this lane's byte offsets of its DMA rows from the operands' first rows
  uint32_t ao[A_I];
#pragma unroll
  for (int i = 0; i < A_I; ++i) {
    const int row = (wave * A_I + i) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ (row & 7);
    ao[i] = (uint32_t)(min(row, a.T - 1 - g0) * H * 2 + c * 16);
  }
  const char* xb = gemm::uniform_ptr(reinterpret_cast<const char*>(a.x + (size_t)g0 * H));
  float ss[MBW];
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) ss[mb] = 0.0f;
  for (int eb = 0; eb < a.E; eb += GT_N) {
    uint32_t bo[B_I];
#pragma unroll
    for (int i = 0; i < B_I; ++i) {
      const int row = (wave * B_I + i) * 8 + (lane >> 3);
      const int c = (lane & 7) ^ (row & 7);
      bo[i] = (uint32_t)(min(row, a.E - 1 - eb) * H * 2 + c * 16);
    }
    const char* wb = gemm::uniform_ptr(reinterpret_cast<const char*>(a.wgt + (size_t)eb * H));
    auto issue = [&](int st) {
      const uint32_t dst = ring0 + (uint32_t)((st % GT_NS) * ST_B);
#pragma unroll
      for (int i = 0; i < A_I; ++i) gemm::dma16(xb + (size_t)st * (2 * GT_K), ao[i], dst + (wave * A_I + i) * 1024);
#pragma unroll
      for (int i = 0; i < B_I; ++i)
        gemm::dma16(wb + (size_t)st * (2 * GT_K), bo[i], dst + A_B + (wave * B_I + i) * 1024);
    };
    f32x16_t acc[MBW][2];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = f32x16_t{};
    for (int st = 0; st < GT_NS - 1 && st < nk; ++st) issue(st);
    const int ra = wm * (GT_M / 2) + (lane & 31), rb = wn * 64 + (lane & 31);
    for (int st = 0; st < nk; ++st) {
      gt_wait<WI>(min(GT_NS - 2, nk - 1 - st));
      __builtin_amdgcn_s_barrier();
      gemm::compiler_fence();
      if (st + GT_NS - 1 < nk) issue(st + GT_NS - 1);
      const char* sa = ring + (st % GT_NS) * ST_B;
      const char* sb = sa + A_B;
#pragma unroll
      for (int kk = 0; kk < GT_K / 16; ++kk) {
        const int ch = 2 * kk + (lane >> 5);
        bf16x8_t af[MBW], bf[2];
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {
          const int r = ra + mb * 32;
          af[mb] = *reinterpret_cast<const bf16x8_t*>(sa + r * 128 + ((ch ^ (r & 7)) << 4));
        }
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
          const int r = rb + nb * 32;
          bf[nb] = *reinterpret_cast<const bf16x8_t*>(sb + r * 128 + ((ch ^ (r & 7)) << 4));
        }
        if (wn == 0 && eb == 0) {
#pragma unroll
          for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              const float f = (float)af[mb][q];
              ss[mb] += f * f;
            }
        }
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mb], bf[nb], acc[mb][nb], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_barrier();  // the ring is refilled by the next pass
    gemm::compiler_fence();
    // C[8 (r >> 2) + 4 (l >> 5) + (r & 3)][l & 31] of each 32 x 32 block
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        const int e = eb + wn * 64 + nb * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int g = g0 + wm * (GT_M / 2) + mb * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (e < a.E && g < a.T) a.lt[(size_t)g * a.E + e] = acc[mb][nb][r];
        }
      }
  }
  if (wn == 0) {
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
      const float t = ss[mb] + __shfl_xor(ss[mb], 32, WAVE);
      const int g = g0 + wm * (GT_M / 2) + mb * 32 + lane;
      if (lane < 32 && g < a.T) a.xn[g] = sqrtf(t);
    }
  }
  __syncthreads();  // the tile's logits and norms are in memory for the candidate pass
  cand_tile<EPL>(a, g0, GT_M, t_cnt, t_off, t_tau, base_s);
}

// 32 < E <= 128: the approximate logits of GT_M tokens x all experts in one
// workgroup of 8 wavefronts, then the candidate pass, without the logits
// leaving LDS.  The operands stream through an LDS ring of GT_NS stages of
// 64-deep k-steps by direct global->LDS loads (8 lanes fetch one row's 128
// contiguous bytes, granules XOR-swizzled by row & 7).  Token rows past T and
// gate rows past E repeat the last valid row; their sums are not stored.  Wavefronts 0-3 take the first two 16-deep
// slices of every k-step, 4-7 the last two, in a 2 x 2 grid of (GT_M / 2)
// tokens x 64 experts each; the two halves' sums are added through LDS at
// the end (the bound holds for any order of the approximate sum).  The
// logits, plus bias, go to an LDS tile of GT_M rows (padded to 129 words so
// that lanes reading their own rows hit distinct banks); one lane per token
// then keeps the k largest lower ends of its intervals in a sorted list,
// takes tau = the k-th, and lists the experts whose upper end reaches tau.
constexpr int G2_PAD = GT_N + 1;  // words per row of the LDS logit tile

template <int GT_M>
__global__ void __launch_bounds__(2 * NTH) gate_tile2_kernel(FilterArgs a) {
  constexpr int NW = 8;
  constexpr int A_B = GT_M * 2 * GT_K, B_B = GT_N * 2 * GT_K, ST_B = A_B + B_B;
  constexpr int A_I = A_B / 1024 / NW, B_I = B_B / 1024 / NW;  // DMA instructions per wavefront and stage
  constexpr int WI = A_I + B_I;
  constexpr int MBW = GT_M / 64;
  static_assert(A_I >= 1 && B_I >= 1 && GT_M % 64 == 0, "tile geometry");
  static_assert(GT_M * G2_PAD * 4 <= GT_NS * ST_B && 4 * MBW * 2 * 16 * WAVE * 4 <= GT_NS * ST_B, "ring reuse");
  __shared__ __attribute__((aligned(1024))) char ring[GT_NS * ST_B];
  __shared__ float ssq[2][GT_M];  // partial squared norms of the two k halves
  __shared__ float bias_s[GT_N], wn_s[GT_N];
  __shared__ int t_cnt[GT_M], t_off[GT_M];
  __shared__ int base_s;
  const int lane = gemm::lane_here(), wave = gemm::opaque((int)(threadIdx.x / WAVE));
  const int kh = wave >> 2, wm = wave & 1, wn = (wave >> 1) & 1;
  const int g0 = blockIdx.x * GT_M;
  const int H = gemm::opaque(a.H), nk = H / GT_K;
  const uint32_t ring0 = (uint32_t)gemm::opaque((int)gemm::lds_u32(ring));
  for (int e = threadIdx.x; e < GT_N; e += 2 * NTH) {
    bias_s[e] = (a.bias && e < a.E) ? a.bias[e] : 0.0f;
    wn_s[e] = e < a.E ? a.wn[e] : 0.0f;
  }
  uint32_t ao[A_I], bo[B_I];
#pragma unroll
  for (int i = 0; i < A_I; ++i) {
    const int row = (wave * A_I + i) * 8 + (lane >> 3);
    ao[i] = (uint32_t)(min(row, a.T - 1 - g0) * H * 2 + (((lane & 7) ^ (row & 7)) << 4));
  }
#pragma unroll
  for (int i = 0; i < B_I; ++i) {
    const int row = (wave * B_I + i) * 8 + (lane >> 3);
    bo[i] = (uint32_t)(min(row, a.E - 1) * H * 2 + (((lane & 7) ^ (row & 7)) << 4));
  }
  const char* xb = gemm::uniform_ptr(reinterpret_cast<const char*>(a.x + (size_t)g0 * H));
  const char* wb = gemm::uniform_ptr(reinterpret_cast<const char*>(a.wgt));
  auto issue = [&](int st) {
    const uint32_t dst = ring0 + (uint32_t)((st % GT_NS) * ST_B);
#pragma unroll
    for (int i = 0; i < A_I; ++i) gemm::dma16(xb + (size_t)st * (2 * GT_K), ao[i], dst + (wave * A_I + i) * 1024);
#pragma unroll
    for (int i = 0; i < B_I; ++i)
      gemm::dma16(wb + (size_t)st * (2 * GT_K), bo[i], dst + A_B + (wave * B_I + i) * 1024);
  };
  f32x16_t acc[MBW][2];
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = f32x16_t{};
  float ss[MBW];
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) ss[mb] = 0.0f;
  for (int st = 0; st < GT_NS - 1 && st < nk; ++st) issue(st);
  const int ra = wm * (GT_M / 2) + (lane & 31), rb = wn * 64 + (lane & 31);
  for (int st = 0; st < nk; ++st) {
    gt_wait<WI>(min(GT_NS - 2, nk - 1 - st));
    __builtin_amdgcn_s_barrier();
    gemm::compiler_fence();
    if (st + GT_NS - 1 < nk) issue(st + GT_NS - 1);
    const char* sa = ring + (st % GT_NS) * ST_B;
    const char* sb = sa + A_B;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      const int ch = 2 * (2 * kh + k2) + (lane >> 5);
      bf16x8_t af[MBW], bf[2];
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb) {
        const int r = ra + mb * 32;
        af[mb] = *reinterpret_cast<const bf16x8_t*>(sa + r * 128 + ((ch ^ (r & 7)) << 4));
      }
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        const int r = rb + nb * 32;
        bf[nb] = *reinterpret_cast<const bf16x8_t*>(sb + r * 128 + ((ch ^ (r & 7)) << 4));
      }
      if (wn == 0) {
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float f = (float)af[mb][q];
            ss[mb] += f * f;
          }
      }
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mb], bf[nb], acc[mb][nb], 0, 0, 0);
    }
  }
  __builtin_amdgcn_s_barrier();  // the ring is reused below
  gemm::compiler_fence();
  // the second k half's sums, through LDS, into the first half's
  float* part = reinterpret_cast<float*>(ring);
  const int pw = wave & 3;  // the partner wavefront's place in its half
  if (kh == 1) {
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[(((pw * MBW + mb) * 2 + nb) * 16 + r) * WAVE + lane] = acc[mb][nb][r];
  }
  if (wn == 0) {
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
      const float t = ss[mb] + __shfl_xor(ss[mb], 32, WAVE);
      if (lane < 32) ssq[kh][wm * (GT_M / 2) + mb * 32 + lane] = t;
    }
  }
  __syncthreads();
  if (kh == 0) {
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mb][nb][r] += part[(((pw * MBW + mb) * 2 + nb) * 16 + r) * WAVE + lane];
  }
  __syncthreads();
  // logits plus bias into the tile: C[8 (r >> 2) + 4 (l >> 5) + (r & 3)][l & 31] of each block
  float* tile = reinterpret_cast<float*>(ring);
  if (kh == 0) {
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        const int e = wn * 64 + nb * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int t = wm * (GT_M / 2) + mb * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          float l = acc[mb][nb][r];
          if (a.bias) l = l + bias_s[e];
          tile[t * G2_PAD + e] = l;
        }
      }
  }
  __syncthreads();
  // candidates, LPT adjacent lanes per token (lane q takes experts
  // [q * EQ, q * EQ + EQ)): each keeps the k largest lower ends of its
  // experts in a sorted list (equal values all kept) and the upper ends in
  // registers; the lists are merged across the token's lanes, so top[k-1] is
  // the k-th largest lower end over every expert; then the experts whose
  // upper end reaches it, in expert order
  constexpr int LPT = 2 * NTH / GT_M, EQ = GT_N / LPT;
  static_assert(LPT * GT_M == 2 * NTH && (LPT & (LPT - 1)) == 0 && LPT <= WAVE, "lanes per token");
  const int tq = threadIdx.x / LPT, q = threadIdx.x % LPT;
  const int g = g0 + tq;
  const bool mine = g < a.T;
  float top[MAX_TOPK];
#pragma unroll
  for (int j = 0; j < MAX_TOPK; ++j) top[j] = -INFINITY;
  auto insert = [&](float v) {
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) {
      const float hi = fmaxf(v, top[j]);
      v = fminf(v, top[j]);
      top[j] = hi;
    }
  };
  float up[EQ];
  if (mine) {
    const float xn = sqrtf(ssq[0][tq] + ssq[1][tq]);
#pragma unroll
    for (int i = 0; i < EQ; ++i) {
      const int e = q * EQ + i;
      up[i] = -INFINITY;
      if (e < a.E) {
        float lo;
        interval(tile[tq * G2_PAD + e], xn * wn_s[e], a.bound, lo, up[i]);
        insert(lo);
      }
    }
  }
#pragma unroll
  for (int m = 1; m < LPT; m <<= 1) {
    float other[MAX_TOPK];
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) other[j] = __shfl_xor(top[j], m, WAVE);
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) insert(other[j]);
  }
  float tau = -INFINITY;
#pragma unroll
  for (int j = 0; j < MAX_TOPK; ++j)
    if (j == a.k - 1) tau = top[j];
  int cnt = 0;
  if (mine) {
#pragma unroll
    for (int i = 0; i < EQ; ++i) cnt += (q * EQ + i < a.E && up[i] >= tau) ? 1 : 0;
  }
  // this lane's place among its token's candidates, and the token's count
  int incl = cnt;
#pragma unroll
  for (int m = 1; m < LPT; m <<= 1) {
    const int y = __shfl_up(incl, m, WAVE);
    if (q >= m) incl += y;
  }
  const int ntok = __shfl(incl, (lane | (LPT - 1)), WAVE);
  if (q == 0) t_cnt[tq] = ntok;  // 0 for rows past T
  __syncthreads();
  if (threadIdx.x < WAVE) {  // exclusive scan of the counts, one atomic for the tile
    int carry = 0;
    for (int b = 0; b < GT_M; b += WAVE) {
      const int c = t_cnt[b + lane];
      int x = c;
#pragma unroll
      for (int d = 1; d < WAVE; d <<= 1) {
        const int y = __shfl_up(x, d, WAVE);
        if (lane >= d) x += y;
      }
      t_off[b + lane] = carry + x - c;
      carry += __shfl(x, WAVE - 1, WAVE);
    }
    if (lane == 0) base_s = atomicAdd(a.n_cands, carry);
  }
  __syncthreads();
  if (mine) {
    const int tb = base_s + t_off[tq];
    if (q == 0) {
      a.tok_base[g] = tb;
      a.tok_n[g] = ntok;
    }
    int pos = tb + incl - cnt;
#pragma unroll
    for (int i = 0; i < EQ; ++i) {
      const int e = q * EQ + i;
      if (e < a.E && up[i] >= tau) {
        a.ch_g[pos] = g;
        a.ch_e[pos] = e;
        ++pos;
      }
    }
  }
}

template __global__ void gate_tile2_kernel<64>(FilterArgs);
template __global__ void gate_tile2_kernel<128>(FilterArgs);

// the defined logit of one (token, expert): fp32, one accumulator, h
// ascending, each product rounded before the add.  A product of two bf16
// values is exact in fp32, so fma(x, w, acc) rounds exactly as acc + x*w and
// saves the multiply on the serial chain.  Two register sets of PF vectors
// take turns so that the next block's loads are in flight while the current
// one is added.
constexpr int PF = 16;
__device__ __forceinline__ void chain_add(float& acc, const u32x4_t (&xb)[PF], const u32x4_t (&wb)[PF]) {
#pragma unroll
  for (int i = 0; i < PF; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc = __builtin_fmaf(bf16_lo(xb[i][q]), bf16_lo(wb[i][q]), acc);
      acc = __builtin_fmaf(bf16_hi(xb[i][q]), bf16_hi(wb[i][q]), acc);
    }
}
__device__ __forceinline__ float exact_logit(const uint16_t* xr, const uint16_t* wr, int H) {
  const u32x4_t* xv = reinterpret_cast<const u32x4_t*>(xr);
  const u32x4_t* wv = reinterpret_cast<const u32x4_t*>(wr);
  const int nv = H >> 3;       // 16-byte vectors per row
  const int nb = nv / PF;      // whole blocks of PF vectors
  u32x4_t xa[PF], wa[PF], xb[PF], wb[PF];
  auto load = [&](u32x4_t (&xd)[PF], u32x4_t (&wd)[PF], int blk) {
#pragma unroll
    for (int i = 0; i < PF; ++i) { xd[i] = xv[blk * PF + i]; wd[i] = wv[blk * PF + i]; }
  };
  float acc = 0.0f;
  if (nb > 0) load(xa, wa, 0);
  for (int b = 0; b < nb; b += 2) {
    if (b + 1 < nb) load(xb, wb, b + 1);
    chain_add(acc, xa, wa);
    if (b + 1 < nb) {
      if (b + 2 < nb) load(xa, wa, b + 2);
      chain_add(acc, xb, wb);
    }
  }
  for (int v = nb * PF; v < nv; ++v) {  // the vectors after the last whole block
    const u32x4_t x = xv[v], w = wv[v];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc = __builtin_fmaf(bf16_lo(x[q]), bf16_lo(w[q]), acc);
      acc = __builtin_fmaf(bf16_hi(x[q]), bf16_hi(w[q]), acc);
    }
  }
  return acc;
}

// one lane per chain of the list, one wavefront per workgroup: each chain
// streams two rows of H bf16 values, so the chains are spread over as many
// CUs as possible (a CU's memory pipeline, not its VALU, bounds a chain)
__global__ void __launch_bounds__(WAVE) gate_chain_kernel(FilterArgs a) {
  const int n = *a.n_cands;
  for (int i = blockIdx.x * WAVE + threadIdx.x; i < n; i += gridDim.x * WAVE) {
    const int g = a.ch_g[i], e = a.ch_e[i];
    float l = exact_logit(a.x + (size_t)g * a.H, a.wgt + (size_t)e * a.H, a.H);
    if (a.bias) l = l + a.bias[e];
    a.ch_l[i] = l;
  }
}

// The chains of the list for E <= CH_E: one lane per chain, CH_W chains per
// workgroup.  The chains of one token are adjacent in the list and every
// token has at least k of them (its top k are among them), so a range of
// CH_W chains holds at most CH_W / k + 2 tokens, CX of them in a stage.  For
// each 64-value block of h the workgroup stages in LDS that block of all gate
// rows (CH_E rows of 128 bytes, rows past E repeating the last one) and of the
// x rows of its tokens (CX rows, slots past the range's tokens repeating its
// first), whole lines by direct global->LDS loads, in a ring of NP stages: no
// operand goes through registers ahead of its use, so with NP = 3 two blocks
// are in flight while one is added, and two workgroups share a CU.  A lane
// reads its token's x and its expert's gate values from the stage and adds
// the 64 products in order, one fused multiply-add each: the product of two
// bf16 values is exact in fp32, so this is the product rounded, then the sum
// rounded.  Granules of a staged row are XOR-swizzled
// (chain_swz).
constexpr int CH_W = 512, CH_E = 128, CH_K = 64;
constexpr int CH_NW = CH_W / WAVE;       // wavefronts per workgroup
constexpr int CH_WB = CH_E * 2 * CH_K;   // gate bytes of a stage
constexpr int CH_DMA = CH_E / 8 / CH_NW; // gate DMA instructions per wavefront and block

// Granule swizzle of a staged 128-byte row: two rows share a 256-byte bank
// window, so the granule is XOR-ed with bits 1-3 of the row, and rows that
// differ in their low four bits put a given granule in different banks.
__device__ __forceinline__ int chain_swz(int row) { return (row >> 1) & 7; }

template <int CX, int NP>
struct ChainGeo {
  static constexpr int STAGE = CH_WB + CX * 2 * CH_K;        // bytes of a stage
  static constexpr int XI = (CX / 8 + CH_NW - 1) / CH_NW;    // x DMA instructions per wavefront and block (at most)
  static_assert(CX % 8 == 0 && STAGE % 1024 == 0 && (NP == 2 || NP == 3), "chain staging geometry");
};

// One range of CH_W chains from c0 (< n); the range's chains belong to at
// most CX tokens (the host picks CX from k).
template <int CX, int NP>
__device__ __forceinline__ void chain_range(const FilterArgs& a, char* ring, int* tok, int* wsum, int c0, int n) {
  using Geo = ChainGeo<CX, NP>;
  const int lane = gemm::lane_here(), wave = gemm::opaque((int)(threadIdx.x / WAVE));
  const int i = c0 + (int)threadIdx.x;
  const bool live = i < n;
  const int ic = live ? i : n - 1;
  const int g = a.ch_g[ic], e = a.ch_e[ic];
  // the range's tokens, in list order: a live lane starts a slot where its
  // token differs from the previous entry's (the range's first entry always)
  const bool head = live && (i == c0 || a.ch_g[i - 1] != g);
  const uint64_t hm = __builtin_amdgcn_ballot_w64(head);
  const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, 0));
  if (lane == 0) wsum[wave] = __builtin_popcountll(hm);
  __syncthreads();
  int base = 0, nslot = 0;
  for (int w = 0; w < CH_NW; ++w) {
    const int c = wsum[w];
    if (w < wave) base += c;
    nslot += c;
  }
  if (nslot > CX) {
    // more tokens than a stage holds (not expected: every token has at least
    // k chains): each lane evaluates its chain straight from global memory
    if (live) {
      const u32x4_t* xv = reinterpret_cast<const u32x4_t*>(a.x + (size_t)g * a.H);
      const u32x4_t* wv = reinterpret_cast<const u32x4_t*>(a.wgt + (size_t)e * a.H);
      float l = 0.0f;
      for (int v = 0; v < (a.H >> 3); ++v) {
        const u32x4_t xq = xv[v], wq = wv[v];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          l = __builtin_fmaf(bf16_lo(xq[q]), bf16_lo(wq[q]), l);
          l = __builtin_fmaf(bf16_hi(xq[q]), bf16_hi(wq[q]), l);
        }
      }
      a.ch_l[i] = a.bias ? l + a.bias[e] : l;
    }
    __syncthreads();
    return;
  }
  const int slot = base + before - (head ? 0 : 1);
  if (head) tok[slot] = g;
  __syncthreads();
  const int H = gemm::opaque(a.H), nb = H / CH_K;
  const uint32_t ring0 = (uint32_t)gemm::opaque((int)gemm::lds_u32(ring));
  uint32_t wo[CH_DMA], xo[Geo::XI];
#pragma unroll
  for (int j = 0; j < CH_DMA; ++j) {
    const int row = (wave * CH_DMA + j) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ chain_swz(row);
    wo[j] = (uint32_t)(min(row, a.E - 1) * H * 2 + c * 16);
  }
#pragma unroll
  for (int j = 0; j < Geo::XI; ++j) {
    const int row = (j * CH_NW + wave) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ chain_swz(row);
    xo[j] = (uint32_t)(tok[row < nslot ? row : 0] * H * 2 + c * 16);
  }
  // x DMA instructions of this wavefront: Geo::XI, or one fewer where the
  // last round of 8-row instructions does not reach it
  const int nxi = gemm::opaque((CX / 8 - wave + CH_NW - 1) / CH_NW);
  const char* wb = gemm::uniform_ptr(reinterpret_cast<const char*>(a.wgt));
  const char* xb = gemm::uniform_ptr(reinterpret_cast<const char*>(a.x));
  auto issue = [&](int b) {
    const uint32_t st = ring0 + (uint32_t)((b % NP) * Geo::STAGE);
#pragma unroll
    for (int j = 0; j < CH_DMA; ++j) gemm::dma16(wb + (size_t)b * (2 * CH_K), wo[j], st + (wave * CH_DMA + j) * 1024);
#pragma unroll
    for (int j = 0; j < Geo::XI; ++j)
      if (j < nxi) gemm::dma16(xb + (size_t)b * (2 * CH_K), xo[j], st + CH_WB + (j * CH_NW + wave) * 1024);
  };
  float acc = 0.0f;
  // this lane's 16 granule offsets within a stage (its x row and its gate
  // row, swizzled), computed once: with the stage index a constant (the
  // block loop below runs NP blocks per iteration) every read is one of
  // these plus an immediate
  int xg[8], wg[8];
  {
    const int wrow = e * (2 * CH_K), wsw = chain_swz(e);
    const int xrow = CH_WB + slot * (2 * CH_K), xsw = chain_swz(slot);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      xg[q] = xrow + ((q ^ xsw) << 4);
      wg[q] = wrow + ((q ^ wsw) << 4);
    }
  }
  // block b, in stage sb = b mod NP: the stage holds this wavefront's loads
  // once at most the blocks issued after it are outstanding; past the
  // barrier every wavefront's have landed and every wavefront has added
  // block b - 1, so the stage of block b + NP - 1 (that of b - 1) is
  // refilled, then block b is added
  auto step = [&](int b, int sb) {
    if (NP == 3 && b + 1 < nb) {
      if (nxi == Geo::XI) gemm::wait_vm<CH_DMA + Geo::XI>(); else gemm::wait_vm<CH_DMA + Geo::XI - 1>();
    } else {
      gemm::wait_vm<0>();
    }
    __builtin_amdgcn_s_barrier();
    gemm::compiler_fence();
    if (b + NP - 1 < nb) issue(b + NP - 1);
    const char* st = ring + sb * Geo::STAGE;
    u32x4_t xv[8], wv[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      xv[q] = *reinterpret_cast<const u32x4_t*>(st + xg[q]);
      wv[q] = *reinterpret_cast<const u32x4_t*>(st + wg[q]);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc = __builtin_fmaf(bf16_lo(xv[q][r]), bf16_lo(wv[q][r]), acc);
        acc = __builtin_fmaf(bf16_hi(xv[q][r]), bf16_hi(wv[q][r]), acc);
      }
    // the block's adds complete here, before the next block's barrier (the
    // compiler would otherwise interleave them with the next block's reads
    // and hold both blocks' operands at once)
    asm volatile("" : "+v"(acc));
  };
  for (int b = 0; b < NP - 1 && b < nb; ++b) issue(b);
  int b = 0;
  for (; b + NP <= nb; b += NP) {
#pragma unroll
    for (int sb = 0; sb < NP; ++sb) step(b + sb, sb);
  }
  for (int sb = 0; b < nb; ++b, ++sb) step(b, sb);
  if (live) a.ch_l[i] = a.bias ? acc + a.bias[e] : acc;
  // the next range refills every stage and rewrites the slot table
  __syncthreads();
}

// Persistent over the ranges of CH_W chains (the chain count is known only
// on the device).  Two workgroups per CU: 4 wavefronts per SIMD.
template <int CX, int NP>
__global__ void __launch_bounds__(CH_W, 4) gate_chain_staged_kernel(FilterArgs a) {
  static_assert(CH_E % (8 * CH_NW) == 0, "gate rows per DMA round");
  __shared__ __attribute__((aligned(1024))) char ring[NP * ChainGeo<CX, NP>::STAGE];
  __shared__ int tok[CX];
  __shared__ int wsum[CH_NW];
  const int n = (*a.n_cands);
  for (int c0 = blockIdx.x * CH_W; c0 < n; c0 += gridDim.x * CH_W) chain_range<CX, NP>(a, ring, tok, wsum, c0, n);
}

template __global__ void gate_chain_staged_kernel<72, 3>(FilterArgs);
template __global__ void gate_chain_staged_kernel<136, 2>(FilterArgs);

// top-k of the candidates' defined logits (descending, equal logits ->
// smaller id), one lane per token keeping a sorted list of the k best, then
// the renormalised softmax weights of the chosen experts: exp(l_j - m) over
// their sum (the normaliser over all experts cancels in the renormalisation,
// so it is not formed).
__global__ void __launch_bounds__(NTH) gate_final_kernel(FilterArgs a) {
  const int g = blockIdx.x * NTH + threadIdx.x;
  const bool valid = g < a.T;
  float tv[MAX_TOPK];
  int ti[MAX_TOPK];
#pragma unroll
  for (int j = 0; j < MAX_TOPK; ++j) { tv[j] = -INFINITY; ti[j] = 1 << 30; }
  if (valid) {
    const int tb = a.tok_base[g], tn = a.tok_n[g];
    // the candidates in batches of CB, every load of a batch in flight
    // before the first insertion (list order, as one at a time)
    constexpr int CB = 16;
    for (int c0 = 0; c0 < tn; c0 += CB) {
      float cv[CB];
      int ce[CB];
#pragma unroll
      for (int i = 0; i < CB; ++i)
        if (c0 + i < tn) {
          cv[i] = a.ch_l[tb + c0 + i];
          ce[i] = a.ch_e[tb + c0 + i];
        }
      for (int i = 0; i < CB; ++i) {
        if (c0 + i >= tn) break;
        float v = cv[i];
        int e = ce[i];
#pragma unroll
        for (int j = 0; j < MAX_TOPK; ++j) {
          // (selects: as a branch, gfx950 code of this compiler kept the
          // old id where the values are equal)
          const bool b = better(v, e, tv[j], ti[j]);
          const float ov = tv[j];
          const int oe = ti[j];
          tv[j] = b ? v : ov;
          ti[j] = b ? e : oe;
          v = b ? ov : v;
          e = b ? oe : e;
        }
      }
    }
    const float m = tv[0];
    float p[MAX_TOPK];
    float ps = 0.0f;
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j)
      if (j < a.k) { p[j] = expf(tv[j] - m); ps += p[j]; }
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j)
      if (j < a.k) {
        a.topk_idx[(size_t)g * a.k + j] = ti[j];
        a.topk_w[(size_t)g * a.k + j] = p[j] / ps;
      }
  }
  // the routing tables' counting step on the ids just chosen (this
  // workgroup's tokens are one count block)
  if (a.blk_cnt) {
    __shared__ int hist[MAX_EL], nbad;
    if (threadIdx.x < a.El) hist[threadIdx.x] = 0;
    if (threadIdx.x == 0) nbad = 0;
    __syncthreads();
    bool short_row = false;
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) {
      if (!valid || j >= a.k) continue;
      const int le = ti[j] - a.e0;
      if ((unsigned)le < (unsigned)a.El) atomicAdd(&hist[le], 1);
      short_row |= ti[j] >= a.E;
    }
    if (short_row) atomicAdd(&nbad, 1);
    __syncthreads();
    if (threadIdx.x < a.El) a.blk_cnt[(size_t)blockIdx.x * a.El + threadIdx.x] = hist[threadIdx.x];
    if (threadIdx.x == 0) {
      a.blk_bad[blockIdx.x] = nbad;
      if (nbad) atomicOr(a.err, ERR_ROUTING);
    }
  }
}

// Where the filter is the faster gate: its matrix pass is bf16 and only k + 1
// or so of a token's E chains are evaluated, but it is four kernels with a
// floor of 27 to 170 us.  The gate's time is a step function of T (rounds of
// workgroups over the CUs, each a whole chain of H steps) and depends on E by
// its class only, so the line between them is none of T * H: E = 128, k = 4,
// H = 4096, gate : filter, us, 8192 tokens 99 : 115, 8200 155 : 115, 512 (k =
// 8) 49 : 111; E = 300, k = 8, 16384 tokens 678 : 446; E = 130, k = 2, 10000
// tokens 245 : 167; E = 256, k = 8, 254 : 326; E = 85, k = 3, H = 8192, 9722
// tokens 310 : 215; E = 54, k = 4, H = 3072, 50407 tokens 250 : 174.  So both
// times are estimated (us) by formulas fitted to 20000 measured points of any
// H (E 33 to 512, T 1500 to 160000, H 256 to 16384, k 1 to 8), and the smaller
// one decides: over these points the choice is 0.24% slower than the better
// gate on average, by more than 3% at 2.4% of them and by more than 10% at 0.8%
// (k = 1, where the chains' time depends most on H).  Up to 32 experts there is
// no filter that keeps up with the gate.
static double gate_us(long long T, long long H, int E, int k) {
  const GateGeometry g = gate_geometry((int)T, E);
  const int cus = GATE_SIMDS / 4, wide = g.ec > 256;
  const double h = (double)H;
  if (!g.large) {
    const bool two = (T + 3) / 4 * (g.ec / 64) > GATE_SIMDS;  // wavefronts per SIMD
    return wide ? 11 + 0.021 * h : two ? 9.7 + 0.0169 * h : 9 + 0.011 * h;
  }
  const double r = (double)((g.grid + cus - 1) / cus);
  return wide ? 1.4 + r * (5.3 + 0.0378 * h + 1.37 * k) : 5.6 + r * (1.9 + 0.017 * h + 0.42 * k) + 0.0032 * h;
}

static double filter_us(long long T, long long H, int E, int k) {
  struct Coef {
    double c, ck;                   // four launches; per expert chosen
    double h, eh;                   // per 1000 H; per 1000 H and 128 experts
    double t64, t64h, t128, t128h;  // a round of tiles of 64 or 128 tokens and a pass over 128 experts: fixed, per 1000 H
    double floor, floor8;           // one chain, per 1000 H; per 1000 H past 8192
    double ch[4];                   // or, if longer, the chains per 1e6 T k and 1000 H up to 4096, 8192, 12288 and past
                                    // them (their rows outgrow the L2s)
    double tk, te;                  // per 1e6 T k; logits and candidates, per 1e6 T E
  };
  static const Coef coef[3] = {
      {16.25, -1.11, 0.64, 3.44, 4.22, 11.99, 5.96, 20.54, 1.72, 37.44, {274.57, 786.57, 1306.32, 3028.25}, 86.75, 1.22},
      {12.93, 0.43, 5.98, 4.89, 6.24, 7.05, 8.27, 13.18, 5.56, 1.53, {75.12, 125.54, 218.17, 404.92}, 28.17, 0.65},
      {8.9, 2.67, 8.18, 0.78, 14.95, 7.51, 30.78, 15.39, -10.39, 72.34, {319.96, 657.61, 1412.23, 3470.62}, 246.02, 4.39}};
  const Coef& c = coef[E > 128 ? 2 : k >= 4 ? 1 : 0];  // (gate_chain, E <= 128; gate_chain_staged; E > 128)
  const double h = 1e-3 * (double)H, tk = 1e-6 * (double)T * k, te = 1e-6 * (double)T * E;
  const long long big = 128 * 256;
  const double tiles = T < big ? (double)((2 * T + big - 1) / big) * (c.t64 + c.t64h * h)
                               : (double)((T + big - 1) / big) * (c.t128 + c.t128h * h);
  double chains = 0;
  for (int i = 0; i < 4; ++i) {
    const double past = h - 4.096 * i;
    if (past > 0) chains += tk * c.ch[i] * (i < 3 && past > 4.096 ? 4.096 : past);
  }
  const double floor = c.floor * h + (h > 8.192 ? c.floor8 * (h - 8.192) : 0);
  return c.c + c.ck * k + c.h * h + c.eh * h * E / 128 + tiles * ((E + 127) / 128) + (floor > chains ? floor : chains) +
         c.tk * tk + c.te * te;
}

bool gate_filtered(long long T, long long H, int E, int k) {
  // (the chain list is indexed with 32 bits)
  return E > 32 && T * E < (1LL << 31) && filter_us(T, H, E, k) < gate_us(T, H, E, k);
}

// the filter's kernels in order on `s`
void launch_gate_filter(const FilterArgs& args, hipStream_t s) {
  FilterArgs g = args;
  // |L - L~| <= (gamma_{H-1}(2^-24) + gamma_H(2^-23)) * sum_h |x_h w_h|: the
  // defined recursive fp32 sum and an fp32 accumulation of the MFMA products
  // allowed twice the unit roundoff; sum |x w| <= ||x|| ||w||; 1% for the norms
  const double H = (double)g.H, u = 1.0 / (1 << 24), u2 = 1.0 / (1 << 23);
  const double g1 = (H - 1.0) * u / (1.0 - (H - 1.0) * u), g2 = H * u2 / (1.0 - H * u2);
  g.bound = (float)(1.01 * (g1 + g2));
  gate_prep_kernel<<<g.E, NTH, 0, s>>>(g);
  // 128 tokens per workgroup when that still gives every CU a tile, else 64
  const bool big = g.T >= 128 * 256;
  const int tiles = big ? (g.T + 127) / 128 : (g.T + 63) / 64;
  if (g.E <= 128) {
    if (big) gate_tile2_kernel<128><<<tiles, 2 * NTH, 0, s>>>(g);
    else gate_tile2_kernel<64><<<tiles, 2 * NTH, 0, s>>>(g);
  } else {
    if (big) gate_tile_kernel<128, 32><<<tiles, NTH, 0, s>>>(g);
    else gate_tile_kernel<64, 32><<<tiles, NTH, 0, s>>>(g);
  }
  if (g.E <= 128 && g.k >= 4) {
    // persistent over ranges of chains, at most T * E of them, two workgroups
    // per CU (the kernel's registers and LDS allow it); a range holds at most
    // 512 / k + 2 tokens, whose x rows a stage holds
    const long long ranges = ((long long)g.T * g.E + GATE_CHAIN_STAGED_W - 1) / GATE_CHAIN_STAGED_W;
    const int grid = (int)(ranges < 512 ? ranges : 512);
    if (g.k >= 8) gate_chain_staged_kernel<72, 3><<<grid, GATE_CHAIN_STAGED_W, 0, s>>>(g);
    else gate_chain_staged_kernel<136, 2><<<grid, GATE_CHAIN_STAGED_W, 0, s>>>(g);
  } else {
    const long long n = ((long long)g.T * g.k * 3 / 2 + WAVE - 1) / WAVE;
    gate_chain_kernel<<<(int)(n < 16384 ? n : 16384), WAVE, 0, s>>>(g);
  }
  gate_final_kernel<<<(g.T + NTH - 1) / NTH, NTH, 0, s>>>(g);
}

}  // namespace moe
