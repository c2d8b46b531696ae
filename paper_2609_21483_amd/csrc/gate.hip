// The gate: logits -> top-k (on logits, ties -> smaller id) -> renormalised
// softmax weights, the routing that precedes the MoE layer (paper section 4
// takes its result as input), in one kernel.
//
// The logit of (token g, expert e) is defined in fp32 with one accumulator,
// hidden index ascending, each product rounded to fp32 before it is added,
// then + bias[e].  A product of two bf16 values is exact in fp32, so that sum
// is a chain of H dependent fused multiply-adds, and the fp32 matrix
// instructions of depth 1 (v_mfma_f32_4x4x1_16b_f32, v_mfma_f32_16x16x1_4b_f32)
// evaluate 256 or 1024 such chains one step at a time: each output element
// takes one fused multiply-add per instruction, with the bits of fmaf for
// every operand (subnormals, infinities and NaN included), so every logit of
// the layer is evaluated as defined and nothing has to be filtered.
//
// What bounds it: a step takes 13.3 cycles for 256 chains (latency of the
// dependent 4x4x1) or 32 for 1024 (rate of the 16x16x1), and the fp32 matrix
// instructions run on the vector ALU's own pipe, so every other vector
// instruction of a SIMD takes its turn from them: one between two of them
// costs 9 to 11 cycles, one of a row of eight 5 to 6.  So the operands are
// widened in rows, and as few of them as the instruction's broadcasts allow:
// a register holds several steps' token values (one per block, picked by
// cbsz / abid) and, for E <= 32, several steps' gate values (one per lane
// group, picked by blgp).  18.8 cycles a step remain for the small shape and
// 38.4 for the large one at 64 experts per wavefront, stages aside: with their
// barriers and one wavefront per SIMD the large one takes 29 to 32 ns a step
// (8192 tokens x 128 experts, H = 2048: 59 to 65 us).
#include <type_traits>
#include <utility>

#include "common.h"
#include "gemm.h"
#include "kernels.h"

namespace moe {

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// Geometry of an expert class: at most EC experts, in EW wavefronts of NE
// experts side by side; TW of them, of TPW tokens each, in the tokens (the
// blocks of the matrix instruction that the experts leave take more tokens).
// A stage of the LDS ring holds HK values of h: XI DMA instructions (1 KiB
// each) of token rows, RPI rows each, then WI of the gate's rows; every
// wavefront issues DPW of them (the last one repeated).
// Registers: a lane holds one token's values of every XP-th run of RX steps,
// and one expert's of every WP-th quad.  The top-k takes LPT lanes per token,
// EQ experts each.
template <int EC, bool LM, int TWV>
struct GateGeo {
  static constexpr int NE = EC <= 16 ? 16 : EC < 64 ? EC : 64, EW = (EC + NE - 1) / NE, TW = TWV, NW = EW * TW;
  static constexpr int TPW = (LM ? 1024 : 256) / NE, TT = TW * TPW;
  static constexpr int HK = (LM || EC > 128) ? 32 : 64;
  static constexpr int RPI = 1024 / (2 * HK);
  static constexpr int XI = (TT + RPI - 1) / RPI, WI = (HK * EC * 2 + 1023) / 1024;
  static constexpr int DPW = (XI + WI + NW - 1) / NW;
  static constexpr int STAGE = (XI + WI) * 1024;
  // a workgroup by itself on its CU takes a deep ring; else two share one
  static constexpr int RING0 = EC > 256 || (!LM && TW == 1) ? 150 << 10 : 76 << 10;
  static constexpr int NST0 = RING0 / STAGE, NST = NST0 > 8 ? 8 : NST0, RING = NST * STAGE;
  static constexpr int XP = NE / (LM ? 16 : 4), WP = 64 / NE;
  static constexpr int RX = HK / XP < 8 ? HK / XP : 8, NX = HK / (XP * RX);  // run length, runs per lane and stage
  static constexpr int NWQ = HK / (4 * WP);                                  // gate quads per lane and stage
  static constexpr int GS = 16;                                              // steps per row of widenings
  static constexpr int CBSZ = XP == 16 ? 4 : XP == 8 ? 3 : XP == 4 ? 2 : XP == 2 ? 1 : 0;
  static constexpr int LPT = NW * WAVE / TT >= 16 && EC > 8 ? 16 : 8, EQ = EC / LPT;
  static constexpr int LGB = TT * (EC + 1) * 4;  // bytes of the logits, in the ring's place
  static constexpr int LDS = RING > LGB ? RING : LGB;
  static_assert(NST >= 4 && (NST - 2) * DPW < 64, "ring");
  static_assert(RX >= 2 && HK % GS == 0 && NWQ % (GS / (4 * WP)) == 0, "rows of widenings");
};

__device__ __forceinline__ bool better(float v, int e, float bv, int be) { return v > bv || (v == bv && e < be); }

// best (v, e) of the LPT adjacent lanes of a token, known to all of them: DPP
// exchanges (xor 1, xor 2, half-row mirror, row mirror: each pairs the lanes
// of two disjoint halves that agree within themselves)
template <int CTRL>
__device__ __forceinline__ void argmax_step(float& v, int& e) {
  const float ov = __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
  const int oe = __builtin_amdgcn_mov_dpp(e, CTRL, 0xF, 0xF, false);
  if (better(ov, oe, v, e)) { v = ov; e = oe; }
}

template <bool LM, int CBSZ, int ABID, int BLGP, typename Acc>
__device__ __forceinline__ void gate_mfma(Acc& acc, float x, float w) {
  if constexpr (LM) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(x, w, acc, CBSZ, ABID, BLGP);
  else acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, w, acc, CBSZ, ABID, BLGP);
}

// One workgroup of TW x EW wavefronts.  The token rows and the gate's rows
// (natural layout [H][E]: a stage is one contiguous piece) stream through an
// LDS ring by direct global->LDS loads; a stage's operands are read into
// registers one stage ahead of their use, each row of them behind its
// widening.  Token rows past T repeat the last one; their results are not
// stored.  The gate's values are read with the transposing LDS read, four h
// of one expert per lane, which takes rows of a multiple of 4 values (a.ldw;
// gate_pad_kernel).
template <int EC, bool LM, int TWV>
__global__ void __launch_bounds__((GateGeo<EC, LM, TWV>::NW * WAVE)) gate_kernel(GateArgs a) {
  using G = GateGeo<EC, LM, TWV>;
  constexpr int NE = G::NE, TPW = G::TPW, TT = G::TT, HK = G::HK, RPI = G::RPI, NW = G::NW, XI = G::XI, DPW = G::DPW;
  constexpr int NST = G::NST, XP = G::XP, WP = G::WP, RX = G::RX, NX = G::NX, NWQ = G::NWQ, GS = G::GS;
  __shared__ __attribute__((aligned(1024))) char lds[G::LDS];
  __shared__ int hist[MAX_EL], nbad;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int E = a.E, ldw = a.ldw, nk = a.H / HK, chunk = HK * ldw * 2;
  const int g0 = blockIdx.x * TT;
  const int wt = wave / G::EW, eb = (wave % G::EW) * 64;  // this wavefront's token block and first expert

  // DMA slot i of this wavefront is instruction wave + i * NW of the stage
  uint32_t off[DPW], dst[DPW];
  const char* src[DPW];
  int stp[DPW];
#pragma unroll
  for (int i = 0; i < DPW; ++i) {
    const int id = min(wave + i * NW, XI + G::WI - 1);
    const bool x = id < XI;
    constexpr int LPR = HK / 8;  // lanes per token row
    dst[i] = (uint32_t)id * 1024u;
    off[i] = x ? (uint32_t)(min(id * RPI + lane / LPR, a.T - 1 - g0) * a.H * 2 + lane % LPR * 16)
               : (uint32_t)min((id - XI) * 1024 + lane * 16, chunk - 16);
    src[i] = gemm::uniform_ptr(reinterpret_cast<const char*>(x ? a.x + (size_t)g0 * a.H : a.wg));
    stp[i] = x ? HK * 2 : chunk;
  }
  const uint32_t ring0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)gemm::lds_u32(lds));
  uint32_t islot = ring0;  // ring slot of the next stage to issue
  auto issue = [&] {
#pragma unroll
    for (int i = 0; i < DPW; ++i) {
      gemm::dma16(src[i], off[i], islot + dst[i]);
      src[i] += stp[i];
    }
    islot = islot == ring0 + (NST - 1) * G::STAGE ? ring0 : islot + G::STAGE;
  };

  // this lane's operands: A a token and its phase among the blocks that share
  // the set's tokens, B an expert and its phase among the lane groups
  constexpr int BR = LM ? 16 : 4;  // tokens per block
  const int blk = lane / BR, tok = wt * TPW + blk / XP * BR + lane % BR;
  const int xo = tok * (HK * 2) + blk % XP * (RX * 2);
  // lane j of 16 reads 4 experts of row j / 4 and receives 4 rows of expert j
  const int grp = lane >> 4, l16 = lane & 15;
  const int wo = XI * 1024 + ((grp / (NE / 16) * 4 + (l16 >> 2)) * ldw + min(eb + grp % (NE / 16) * 16 + 4 * (l16 & 3), ldw - 4)) * 2;
  typedef uint32_t Run __attribute__((ext_vector_type(RX / 2 == 1 ? 2 : RX / 2)));
  Run xr[NX];
  u32x2_t wr[NWQ];
  int rslot = 0;  // ring offset of the stage being read
  auto read_x = [&] {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const char* p = lds + rslot + xo + i * (XP * RX * 2);
      if constexpr (RX == 2) xr[i][0] = *reinterpret_cast<const uint32_t*>(p);
      else xr[i] = *reinterpret_cast<const Run*>(p);
    }
  };
  auto read_w = [&](int i) {
    typedef __attribute__((address_space(3))) i16x4_t* lds_p;
    wr[i] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(lds + (rslot + wo + i * (4 * WP) * 2 * ldw))));
  };
  auto next_slot = [&] { rslot = rslot == (NST - 1) * G::STAGE ? 0 : rslot + G::STAGE; };
  typedef float Acc __attribute__((ext_vector_type(LM ? 16 : 4)));
  Acc acc = {};
  // stage s is in registers: its HK steps in rows of GS; each row's registers
  // are refilled from stage s + 1 once they are widened (READ)
  auto compute = [&](auto read_next) {
    constexpr bool READ = decltype(read_next)::value;
    float xf[NX * RX];
#pragma unroll
    for (int i = 0; i < NX * RX; ++i) xf[i] = i & 1 ? bf16_hi(xr[i / RX][i % RX / 2]) : bf16_lo(xr[i / RX][i % RX / 2]);
    if constexpr (READ) read_x();
    constexpr int QG = GS / (4 * WP);  // gate quads per row of widenings
    auto row = [&](auto rc) {
      constexpr int r = decltype(rc)::value;
      float wf[QG * 4];
#pragma unroll
      for (int i = 0; i < QG * 4; ++i) {
        const uint32_t d = wr[r * QG + i / 4][i % 4 / 2];
        wf[i] = i & 1 ? bf16_hi(d) : bf16_lo(d);
      }
      if constexpr (READ) {
#pragma unroll
        for (int i = 0; i < QG; ++i) read_w(r * QG + i);
      }
      // the scheduler would move the widenings between the matrix instructions
      __builtin_amdgcn_sched_barrier(0);
      auto steps = [&]<int... J>(std::integer_sequence<int, J...>) {
        (gate_mfma<LM, G::CBSZ, (r * GS + J) % (XP * RX) / RX, WP == 1 ? 0 : (WP == 2 ? 1 : 4) + J % (4 * WP) / 4>(
             acc, xf[(r * GS + J) / (XP * RX) * RX + (r * GS + J) % RX], wf[J / (4 * WP) * 4 + J % 4]),
         ...);
      };
      steps(std::make_integer_sequence<int, GS>{});
      __builtin_amdgcn_sched_barrier(0);
    };
    auto rows = [&]<int... R>(std::integer_sequence<int, R...>) { (row(std::integral_constant<int, R>{}), ...); };
    rows(std::make_integer_sequence<int, HK / GS>{});
  };
  for (int s = 0; s < NST - 1 && s < nk; ++s) issue();
  // at most the DMA of the stages after the one waited for stays in flight
  if (nk >= NST - 1) gemm::wait_vm<(NST - 2) * DPW>(); else gemm::wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  gemm::compiler_fence();
  read_x();
#pragma unroll
  for (int i = 0; i < NWQ; ++i) read_w(i);
  int s = 0;
  // steady state: stage s + 1 has landed in every wavefront past the barrier;
  // every wavefront is done with stage s - 1, whose slot is refilled
#pragma unroll 1
  for (; s + NST - 1 < nk; ++s) {
    gemm::wait_vm<(NST - 3) * DPW>();
    __builtin_amdgcn_s_barrier();
    gemm::compiler_fence();
    issue();
    next_slot();
    compute(std::true_type{});
  }
#pragma unroll 1
  for (; s + 1 < nk; ++s) {
    gemm::wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    gemm::compiler_fence();
    next_slot();
    compute(std::true_type{});
  }
  compute(std::false_type{});
  if (tid < a.El) hist[tid] = 0;
  if (tid == 0) nbad = 0;
  __syncthreads();  // every wavefront has read the last stage: the ring is free

  // logits plus bias into LDS, one row per token
  float* lg = reinterpret_cast<float*>(lds);
  const int ls = E + 1;
  if constexpr (LM) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int t = wt * TPW + (v >> 2) / XP * 16 + 4 * (lane >> 4) + (v & 3);
      const int e = eb + (v >> 2) % XP * 16 + (lane & 15);
      if (e < E) lg[t * ls + e] = a.bias ? acc[v] + a.bias[e] : acc[v];
    }
  } else {
    const int e = eb + lane % NE;
    const float b = a.bias && e < E ? a.bias[e] : 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int t = wt * TPW + blk / XP * 4 + v;
      if (e < E) lg[t * ls + e] = a.bias ? acc[v] + b : acc[v];
    }
  }
  __syncthreads();

  // top-k: LPT adjacent lanes per token, lane q holding experts q, q + LPT,
  // ...; k rounds of the best one left (descending, equal logits -> smaller
  // id), lane q keeping round q's; the weights are exp(l_j - m) over their sum
  // (the softmax normaliser over all experts cancels in the renormalisation).
  // Rolled: unrolled over the rounds, the instruction fetch of code that runs
  // once took 9 us.
  constexpr int LPT = G::LPT, EQ = G::EQ;
  static_assert(LPT >= MAX_TOPK, "one lane per chosen expert");
  const int q = tid % LPT;
#pragma unroll 1
  for (int t = tid / LPT; t < TT; t += G::NW * WAVE / LPT) {
    const int g = g0 + t;
    // a lane's experts; one that is chosen, past E or NaN becomes (-inf, no
    // expert), which loses to every other
    constexpr int NOEXP = 1 << 30;
    float v[EQ];
    int ev[EQ];
#pragma unroll
    for (int i = 0; i < EQ; ++i) {
      const int e = q + LPT * i;
      const float l = lg[t * ls + min(e, E - 1)];
      const bool ok = e < E && l == l;
      v[i] = ok ? l : -INFINITY;
      ev[i] = ok ? e : NOEXP;
    }
    float mv = -INFINITY, m = 0.0f;
    int id = NOEXP;
    bool short_row = false;
#pragma unroll 1
    for (int j = 0; j < a.k; ++j) {
      float tv[EQ];
      int te[EQ];
#pragma unroll
      for (int i = 0; i < EQ; ++i) { tv[i] = v[i]; te[i] = ev[i]; }
#pragma unroll
      for (int d = 1; d < EQ; d <<= 1)
#pragma unroll
        for (int i = 0; i + d < EQ; i += 2 * d)
          if (better(tv[i + d], te[i + d], tv[i], te[i])) { tv[i] = tv[i + d]; te[i] = te[i + d]; }
      float bv = tv[0];
      int be = te[0];
      argmax_step<0xB1>(bv, be);
      argmax_step<0x4E>(bv, be);
      argmax_step<0x141>(bv, be);
      if constexpr (LPT == 16) argmax_step<0x140>(bv, be);
#pragma unroll
      for (int i = 0; i < EQ; ++i) {
        const bool chosen = ev[i] == be;
        v[i] = chosen ? -INFINITY : v[i];
        ev[i] = chosen ? NOEXP : ev[i];
      }
      if (j == 0) m = bv;
      if (q == j) { mv = bv; id = be; }
      short_row |= be >= E;  // fewer than k logits that compare (NaN rows): no valid id
    }
    const float p = expf(mv - m);
    float ps = 0.0f;
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) {
      const float pj = __shfl(p, (lane & ~(LPT - 1)) + j, WAVE);
      if (j < a.k) ps += pj;
    }
    if (g < a.T && q < a.k) {
      a.topk_idx[(size_t)g * a.k + q] = id;
      a.topk_w[(size_t)g * a.k + q] = p / ps;
      if (a.blk_cnt) {
        const int le = id - a.e0;
        if ((unsigned)le < (unsigned)a.El) atomicAdd(&hist[le], 1);
        if (q == 0 && short_row) atomicAdd(&nbad, 1);
      }
    }
  }
  if (blockIdx.x == 0 && tid == 0 && a.cands) *a.cands = a.T * a.k;
  // the routing tables' counting step on the ids just chosen (this
  // workgroup's tokens are one count block)
  if (a.blk_cnt) {
    __syncthreads();
    if (tid < a.El) a.blk_cnt[(size_t)blockIdx.x * a.El + tid] = hist[tid];
    if (tid == 0) {
      a.blk_bad[blockIdx.x] = nbad;
      if (nbad) atomicOr(a.err, ERR_ROUTING);
    }
  }
}

// A copy of the gate [H][E] with rows of E4 values (E rounded up to a multiple
// of 4), aligned.  In front of the gate it takes 3 to 5 us; reading unpadded rows value
// by value instead made the gate 40% slower (E = 127 against 128, H = 4096).
__global__ void __launch_bounds__(NTH) gate_pad_kernel(const uint16_t* wg, uint16_t* out, int H, int E, int E4) {
  const int n = H * E4;
  for (int i = blockIdx.x * NTH + threadIdx.x; i < n; i += gridDim.x * NTH) {
    const int h = i / E4, e = i - h * E4;
    out[i] = e < E ? wg[(size_t)h * E + e] : (uint16_t)0;
  }
}

// A copy of token rows at an aligned address, where the caller's is not (a view
// into a larger buffer): value by value.
__global__ void __launch_bounds__(NTH) copy_rows_kernel(const uint16_t* src, uint16_t* dst, long long n) {
  for (long long i = (long long)blockIdx.x * NTH + threadIdx.x; i < n; i += (long long)gridDim.x * NTH) dst[i] = src[i];
}

void launch_copy_rows(const uint16_t* src, uint16_t* dst, long long n, hipStream_t s) {
  const long long grid = (n + 4 * NTH - 1) / (4 * NTH);
  copy_rows_kernel<<<(int)(grid < 16384 ? grid : 16384), NTH, 0, s>>>(src, dst, n);
}

// Every (expert class, shape, token wavefronts) with a kernel; the most token
// wavefronts of a class last.  More of them share the gate's rows in LDS
// (less L2 traffic), fewer spread few tokens over more CUs.
#define MOE_GATE_CLASSES(X)                                                                            \
  X(8, false, 1) X(8, false, 4) X(16, false, 1) X(16, false, 4) X(32, false, 1) X(32, false, 4)        \
  X(64, false, 1) X(64, false, 4) X(128, false, 1) X(128, false, 2) X(256, false, 1) X(256, false, 2)  \
  X(512, false, 1)                                                                                     \
  X(8, true, 2) X(16, true, 2) X(32, true, 4) X(64, true, 4) X(128, true, 2) X(256, true, 1) X(512, true, 1)

// Wavefronts of the small shape: one per 256 / NE tokens and 64 experts.  Up
// to two per SIMD the small shape is faster (18.8 cycles a step alone, 25 to
// 28 for two, against 38.4 of the large shape, whose wavefronts are then too
// few); beyond, wavefronts queue for the matrix pipe, which one of the large
// shape fills alone.  Several token wavefronts share a workgroup (and its
// gate rows) where one each would give more workgroups than CUs.
GateGeometry gate_geometry(int T, int E) {
  GateGeometry g{};
  g.ec = E <= 8 ? 8 : E <= 16 ? 16 : E <= 32 ? 32 : E <= 64 ? 64 : E <= 128 ? 128 : E <= 256 ? 256 : 512;
  const int ne = g.ec <= 16 ? 16 : g.ec < 64 ? g.ec : 64;
  const long long small_waves = (long long)((T + 256 / ne - 1) / (256 / ne)) * ((g.ec + ne - 1) / ne);
  g.large = small_waves > 2 * GATE_SIMDS;
  const int cus = GATE_SIMDS / 4;
#define MOE_GATE_PICK(EC, LM, TW)                                                        \
  if (g.ec == EC && (g.large != 0) == LM) {                                              \
    using G = GateGeo<EC, LM, TW>;                                                       \
    if (!g.tw || (T + G::TPW - 1) / G::TPW > cus) {                                      \
      g.tw = TW;                                                                         \
      g.tt = G::TT;                                                                      \
    }                                                                                    \
  }
  MOE_GATE_CLASSES(MOE_GATE_PICK)
#undef MOE_GATE_PICK
  g.grid = (T + g.tt - 1) / g.tt;
  return g;
}

void launch_gate(const GateArgs& args, const GateGeometry& g, uint16_t* pad, hipStream_t s) {
  GateArgs a = args;
  a.ldw = gate_ldw(a.E);
  if (gate_padded(a.wg, a.E)) {
    const int n = a.H * a.ldw, grid = (n + 4 * NTH - 1) / (4 * NTH);
    gate_pad_kernel<<<grid, NTH, 0, s>>>(a.wg, pad, a.H, a.E, a.ldw);
    a.wg = pad;
  }
#define MOE_GATE_RUN(EC, LM, TW)                                                                       \
  if (g.ec == EC && (g.large != 0) == LM && g.tw == TW) {                                              \
    gate_kernel<EC, LM, TW><<<g.grid, GateGeo<EC, LM, TW>::NW * WAVE, 0, s>>>(a);                      \
    return;                                                                                            \
  }
  MOE_GATE_CLASSES(MOE_GATE_RUN)
#undef MOE_GATE_RUN
}

}  // namespace moe
