// Prefill attention of fp32 plans: the same mask and online softmax as the
// bf16 kernel, on the fp32 matrix cores (32x32x2 MFMA).
//
// What bounds it: an fp32 product takes 64 cycles for 2,048 multiply-adds, a
// sixteenth of the bf16 rate (152 TFLOP/s in a large library product), so a
// wave's operands can come straight from memory in the registers' layout,
// without LDS, barriers or transposition: the loads of one product pass hide
// behind the other one.  Every wave is on its own: 32 (or 64) query rows of one
// (sequence, query head) against 32-key tiles, of which it visits only those
// that meet the sink prefix or the band of its own rows.  8 heads of 1,501
// tokens, head_dim 64: 13 -> 34 TFLOP/s; 8 x 16 heads of 2,048: 83 -> 98;
// 64 heads of 2,048, head_dim 128: 61 -> 91.  (The kernel further down shares
// 64-key tiles of 128 rows through LDS, V transposed by 4-byte writes with bank
// conflicts, and has 96 work-groups for 256 compute units in the first case; it
// is the better one for long prompts of head_dim 64.)
//
//   S^T = K Q^T  : lane (row l % 32, half l / 32) holds, of its key row and of
//                  its query row, the 16-byte chunks 2c + half.  The reduction
//                  order is permuted alike on both operands.
//   O^T += V^T P^T : P^T straight from the score registers, V^T by 4-byte
//                  loads of 32 consecutive elements of a row.
// K(t + 1) is loaded behind S(t), into the registers that S(t) has read, and
// V(t) before S(t); the fences keep the loads there.
//
// KG waves of a work-group share one block of 32 rows where a launch has too
// few rows for the chip: wave kg takes every KG-th tile, and the states meet in
// LDS at the end.
#include "moa_device.h"
#include "prefill_rule.h"

namespace moa {

namespace {

constexpr int NW = 4;                   // waves per work-group
constexpr int BR = 32;                  // query rows per wave
constexpr int BK = 32;                  // keys per tile
constexpr int kPairsPerDie = 4;         // (KV head, sequence) pairs per die from which each keeps to one
constexpr float kRescaleSlack = 8.0f;   // log2 headroom before the offset is raised

__device__ __forceinline__ f32x16 mma(float a, float b, const f32x16& c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
#else
  (void)a;
  (void)b;
  return c;
#endif
}

// x * y - z with the product rounded on its own (never fused): a row's maximal
// score then gives exactly 2^0, so a window of one key returns v bit-exactly.
__device__ __forceinline__ float mul_then_sub(float x, float y, float z) {
#pragma clang fp contract(off)
  return x * y - z;
}

template <int D, int KG, int RW>
__global__ void __launch_bounds__(NW * 64, D == 64 ? 2 : 1) prefill_f32_kernel(PrefillArgs a) {
  constexpr int KR = D / 2;             // K (or Q) registers per lane
  constexpr int DT = D / 32;            // 32-row output tiles of O^T
  constexpr int RB = NW / KG;           // waves with rows of their own
  constexpr int WR = RW * BR;           // query rows per wave
  constexpr int kRegs = RW * (D / 2 + 2);      // state values per lane
  __shared__ float s_state[KG > 1 ? (NW - RB) * kRegs * 64 : 1];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lrow = lane & 31;
  const int half = lane >> 5;
  const int rb = wave % RB, kg = wave / RB;

  // Work item: latest rows (most keys) first, then widest window; the query
  // heads of a (KV head, sequence) pair run side by side.  With enough pairs
  // each stays on one accelerator die (work-group i runs on die i % kNumXcd),
  // whose L2 then holds its keys and values; the pairs are dealt in alternating
  // direction, so that every die gets wide and narrow windows.
  const int pairs = a.hkv * a.batch;
  int i_block, pair, head;
  if (pairs >= kPairsPerDie * kNumXcd) {
    const int xcd = static_cast<int>(blockIdx.x % kNumXcd), local = static_cast<int>(blockIdx.x / kNumXcd);
    const int deals = (pairs + kNumXcd - 1) / kNumXcd;
    i_block = local / (deals * a.group);
    const int deal = local / a.group - i_block * deals;
    pair = deal * kNumXcd + (deal & 1 ? kNumXcd - 1 - xcd : xcd);
    head = local % a.group;
    if (pair >= pairs) return;
  } else {
    const int per_rows = pairs * a.group;
    i_block = static_cast<int>(blockIdx.x) / per_rows;
    const int item = static_cast<int>(blockIdx.x) - i_block * per_rows;
    pair = item / a.group;
    head = item % a.group;
  }
  const int b = pair % a.batch;
  const int g = a.kv_order[pair / a.batch];
  const int h = g * a.group + head;
  const int n = static_cast<int>(a.n);
  const int n_blocks = (n + WR * RB - 1) / (WR * RB);
  const int iw0 = ((n_blocks - 1 - i_block) * RB + rb) * WR;
  const int iw1 = min(n, iw0 + WR);
  const bool active = iw0 < n;
  const int my_row = iw0 + lrow;          // of the first block; BR further on of the second

  const int wband = a.window[g];
  const int bsh = a.band_shift;
  auto band_start = [&](int i) { return ((i >> bsh) - wband + 1) * (1 << bsh); };
  const int s = a.num_sink;
  const float c2 = a.scale_log2;

  // Tiles to visit: sink tiles [0, ta), then band tiles [tb, tl].
  const int tl = active ? (iw1 - 1) / BK : -1;
  const int ta = active ? (min(s, iw1) + BK - 1) / BK : 0;
  const int tb = max(ta, max(0, band_start(iw0)) / BK);
  const int ntiles = ta + max(0, tl - tb + 1);
  auto tile_j0 = [&](int t) { return (t < ta ? t : tb + (t - ta)) * BK; };

  const int64_t kv_row = int64_t(a.hkv) * D;            // elements between consecutive tokens
  const int64_t q_row = int64_t(a.hq) * D;
  const float* qg = static_cast<const float*>(a.q) + (int64_t(b) * n * a.hq + h) * D;
  const float* kg_base = static_cast<const float*>(a.k) + (int64_t(b) * n * a.hkv + g) * D;
  const float* vg_base = static_cast<const float*>(a.v) + (int64_t(b) * n * a.hkv + g) * D;

  // A whole tile's addresses are a uniform base and a lane offset of 32 bits.
  // Keys past the end re-read the last key (always masked by causality).
  float kf[KR], vf[DT][16], qf[RW][KR];
  const uint32_t k_lane = uint32_t(lrow) * uint32_t(kv_row) + 4u * half;
  const uint32_t v_lane = 4u * half * uint32_t(kv_row) + lrow;
  auto load_k = [&](int t) {
    const int j0 = tile_j0(t);
    const float* base = kg_base + j0 * kv_row;
    const uint32_t at = j0 + BK <= n ? k_lane : uint32_t(min(lrow, n - 1 - j0)) * uint32_t(kv_row) + 4u * half;
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(base + 8 * c + at);
#pragma unroll
      for (int e = 0; e < 4; ++e) kf[4 * c + e] = x[e];
    }
  };
  // Score register r of a tile holds key (r / 4) * 8 + half * 4 + r % 4.
  auto load_v = [&](int t) {
    const int j0 = tile_j0(t);
    const float* base = vg_base + j0 * kv_row;
    if (j0 + BK <= n) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) vf[dt][r] = (base + ((r >> 2) * 8 + (r & 3)) * kv_row + dt * 32)[v_lane];
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t at = uint32_t(min((r >> 2) * 8 + half * 4 + (r & 3), n - 1 - j0)) * uint32_t(kv_row) + lrow;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) vf[dt][r] = (base + dt * 32)[at];
      }
    }
  };

  f32x16 oacc[RW][DT];
  float m_run[RW], l_run[RW];
#pragma unroll
  for (int w = 0; w < RW; ++w) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[w][dt] = f32x16{};
    m_run[w] = kNegBig;
    l_run[w] = 0.0f;
  }

  if (kg < ntiles) {
    load_k(kg);
#pragma unroll
    for (int w = 0; w < RW; ++w) {
      const float* row = qg + min(my_row + w * BR, n - 1) * q_row + 4 * half;
#pragma unroll
      for (int c = 0; c < D / 8; ++c) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(row + 8 * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) qf[w][4 * c + e] = x[e];
      }
    }
  }
  for (int t = kg; t < ntiles; t += KG) {
    const int j0 = tile_j0(t);
    load_v(t);
    sched_fence();
    f32x16 sacc[RW];
#pragma unroll
    for (int w = 0; w < RW; ++w) sacc[w] = f32x16{};
#pragma unroll
    for (int kk = 0; kk < KR; ++kk)
#pragma unroll
      for (int w = 0; w < RW; ++w) sacc[w] = mma(kf[kk], qf[w][kk], sacc[w]);
    sched_fence();
    load_k(min(t + KG, ntiles - 1));          // past the last tile: unused
    sched_fence();

#pragma unroll
    for (int w = 0; w < RW; ++w) {
      const int r0 = iw0 + w * BR, r1 = min(iw1, r0 + BR);
      // Mask (edge tiles only) and the tile's raw row maximum.
      const bool all_vis = (j0 + BK - 1 <= r0) && (r1 - r0 == BR) && ((j0 + BK <= s) || band_start(r1 - 1) <= j0);
      if (!all_vis) {
        const int jl = j0 + half * 4;                   // key of register 0 of this lane
        const int row = r0 + lrow;
        const int hi = row < r1 ? row - jl : -1;        // causal: key offset <= hi
        const int band = band_start(row) - jl;          // band: key offset >= band
        const int sink = s - jl;                        // sink: key offset < sink
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dj = (r >> 2) * 8 + (r & 3);
          const bool vis = (dj <= hi) & ((dj < sink) | (dj >= band));
          sacc[w][r] = vis ? sacc[w][r] : -INFINITY;
        }
      }
      float tmax = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sacc[w][r]);
      tmax *= c2;
      // The exponent offset is raised only when some row of the wave needs it.
      // Only then do the two lanes of a row meet; their sums meet at the end.
      if (__any(tmax > m_run[w] + kRescaleSlack)) {
        const float m_new = fmaxf(m_run[w], max_xor<32>(tmax));
        const float alpha = fast_exp2(m_run[w] - m_new);
        m_run[w] = m_new;
        l_run[w] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) oacc[w][dt] *= alpha;
      }
      float psum = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sacc[w][r] = fast_exp2(mul_then_sub(sacc[w][r], c2, m_run[w]));
        psum += sacc[w][r];
      }
      l_run[w] += psum;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int w = 0; w < RW; ++w) oacc[w][dt] = mma(vf[dt][r], sacc[w][r], oacc[w][dt]);
    sched_fence();
  }

#pragma unroll
  for (int w = 0; w < RW; ++w) l_run[w] = sum_xor<32>(l_run[w]);
  if constexpr (KG > 1) {
    // The states of the same rows sit in the same lanes of waves rb + RB * kg.
    constexpr int kBlock = kRegs / RW;                   // values of one block of 32 rows
    float* const st = s_state + lane;
    if (kg > 0) {
#pragma unroll
      for (int w = 0; w < RW; ++w) {
        float* p = st + ((wave - RB) * kRegs + w * kBlock) * 64;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) p[(dt * 16 + r) * 64] = oacc[w][dt][r];
        p[(kBlock - 2) * 64] = m_run[w];
        p[(kBlock - 1) * 64] = l_run[w];
      }
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll 1
    for (int v = 0; v < KG - 1; ++v) {
#pragma unroll
      for (int w = 0; w < RW; ++w) {
        const float* p = st + ((v * RB + rb) * kRegs + w * kBlock) * 64;
        const float m2 = p[(kBlock - 2) * 64];
        const float m_new = fmaxf(m_run[w], m2);
        const float f1 = fast_exp2(m_run[w] - m_new), f2 = fast_exp2(m2 - m_new);
        m_run[w] = m_new;
        l_run[w] = l_run[w] * f1 + p[(kBlock - 1) * 64] * f2;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[w][dt][r] = oacc[w][dt][r] * f1 + p[(dt * 16 + r) * 64] * f2;
      }
    }
  }

#pragma unroll
  for (int w = 0; w < RW; ++w) {
    const int row = my_row + w * BR;
    if (row >= iw1) continue;
    const float inv_l = 1.0f / l_run[w];
    float* orow = static_cast<float*>(a.o) + (int64_t(b) * n * a.hq + h) * D + int64_t(row) * q_row;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int grp = 0; grp < 4; ++grp) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = oacc[w][dt][grp * 4 + e] * inv_l;
        *reinterpret_cast<f32x4*>(orow + dt * 32 + grp * 8 + half * 4) = x;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Long prompts at head_dim 64: 4 waves share 64-key tiles through LDS, so that a
// byte of K or V is loaded once per 128 query rows (by the kernel above once per
// 64, in 4-byte loads for V).  64 query and 8 KV heads x 8,192 tokens: 121 TFLOP/s,
// the kernel above 103, with any number of waves per block and of rows per wave
// and with its pairs kept on one die or not.  Shorter prompts lose more to the
// barriers and to V's transposition by 4-byte LDS writes (prefill_rule.h).
// K fragments are read two steps ahead (one step: 0 - 4 % slower at 8,192 tokens,
// up to 4 % faster at 4,096).
// Dispatch, visited tiles and band rotation are those of the bf16 kernel.
// ---------------------------------------------------------------------------
template <int D>
struct SharedTiles {
  static constexpr int BM = 128;                    // query rows per work-group
  static constexpr int BN = 64;                     // keys per tile
  static constexpr int RB = D * 4;                  // bytes per K/V row
  static constexpr int CPR = RB / 16;               // 16-byte chunks per row
  static constexpr int K_BYTES = BN * RB;           // a K tile, rows unpadded
  static constexpr int DPW = K_BYTES / 1024 / NW;   // 1 KB direct-to-LDS loads per wave
  static constexpr int VT_LD = BN + 4;              // V^T row stride (elements)
  static constexpr int VT_BYTES = D * VT_LD * 4;
  static constexpr int VREG = BN * CPR / (NW * 64); // V chunks staged per thread
  // Chunk c of K row r sits at chunk position c ^ swz(r).
  __device__ __forceinline__ static int swz(int r) { return CPR >= 16 ? (r & 15) : ((r >> 1) & 7); }
};

template <int D>
__global__ void __launch_bounds__(NW * 64, 2) prefill_f32_shared_kernel(PrefillArgs a) {
  using TL = SharedTiles<D>;
  constexpr int BM = TL::BM, BN = TL::BN, RB = TL::RB, CPR = TL::CPR, DPW = TL::DPW;
  constexpr int KS = D / 2;                         // MFMA steps over the head dimension
  __shared__ __attribute__((aligned(1024))) char sK[2][TL::K_BYTES];
  __shared__ __attribute__((aligned(1024))) char sV[2][TL::VT_BYTES];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lrow = lane & 31;
  const int half = lane >> 5;

  const int xcd = static_cast<int>(blockIdx.x % kNumXcd);
  const int local = static_cast<int>(blockIdx.x / kNumXcd);
  const int per_unit = a.group * a.qchunk;
  const int round = local / per_unit;
  const int unit = round * kNumXcd + ((round & 1) ? kNumXcd - 1 - xcd : xcd);
  if (unit >= a.n_units) return;                    // padding unit
  const int within = local % per_unit;
  const int hb = a.hkv * a.batch;
  const int cd = unit / hb;                         // chunk rank, heaviest first
  const int g = a.kv_order[(unit % hb) / a.batch];
  const int b = unit % a.batch;
  const int qt = (a.n_chunks - 1 - cd) * a.qchunk + (a.qchunk - 1 - within / a.group);
  if (qt >= a.n_qtiles) return;                     // past the last query tile
  const int h = g * a.group + within % a.group;
  const int64_t n = a.n;
  const int wband = a.window[g];
  const int bsh = a.band_shift;
  auto band_start = [&](int i) { return ((i >> bsh) - wband + 1) * (1 << bsh); };
  const int s = a.num_sink;
  const float c2 = a.scale_log2;

  const int i0 = qt * BM;
  const int i1 = static_cast<int>(min(n, int64_t(i0 + BM)));    // exclusive
  const int iw0 = i0 + wave * 32;                                 // this wave's rows
  const int iw1 = min(i1, iw0 + 32);
  const bool wave_active = iw0 < i1;
  const int my_row = iw0 + lrow;

  // Tiles to visit: sink tiles [0, ta), then band tiles [tb, tl], from tr up to tl
  // and from tb up to tr - 1.
  const int ta = (min(s, i1) + BN - 1) / BN;
  const int tl = (i1 - 1) / BN;
  const int tb = max(ta, max(0, band_start(i0)) / BN);
  const int ntiles = ta + max(0, tl - tb + 1);
  const int qt_top = min(a.n_qtiles - 1, (a.n_chunks - 1 - cd) * a.qchunk + a.qchunk - 1);
  const int tr = a.rotate ? min(max(tb, max(ta, max(0, band_start(qt_top * BM)) / BN)), tl + 1) : tb;
  const int n_upper = tl - tr + 1;
  auto tile_j0 = [&](int it) {
    if (it < ta) return it * BN;
    const int k = it - ta;
    return (k < n_upper ? tr + k : tb + (k - n_upper)) * BN;
  };

  const int64_t q_row = int64_t(a.hq) * D;
  const int64_t kv_row_bytes = int64_t(a.hkv) * RB;
  const float* qg = static_cast<const float*>(a.q) + (int64_t(b) * n * a.hq + h) * D;
  const char* k_base = static_cast<const char*>(a.k) + (int64_t(b) * n * a.hkv + g) * RB;
  const char* v_base = static_cast<const char*>(a.v) + (int64_t(b) * n * a.hkv + g) * RB;

  // K tile loads: instruction I writes tile bytes [I*1024, I*1024 + 1024), lane
  // L's 16 bytes land at chunk m = I*64 + L (row m / CPR, position m % CPR) and
  // carry global chunk position ^ swz(row).  The buffer resource spans the tile's
  // real rows; rows past the last key re-read it (always masked by causality).
  uint32_t k_src[DPW];
  auto dma_row = [&](int i) { return ((wave * DPW + i) * 64 + lane) / CPR; };
#pragma unroll
  for (int i = 0; i < DPW; ++i) {
    const int m = (wave * DPW + i) * 64 + lane;
    k_src[i] = uint32_t(m / CPR) * uint32_t(kv_row_bytes) + uint32_t((m % CPR) ^ TL::swz(m / CPR)) * 16u;
  }
  auto issue_k = [&](int it) {
    const int j0 = tile_j0(it);
    const int last = static_cast<int>(min(int64_t(BN), n - j0)) - 1;
    const i32x4 rs = make_desc(k_base + j0 * kv_row_bytes, uint32_t(last) * uint32_t(kv_row_bytes) + RB);
    char* const to = &sK[it & 1][wave * DPW * 1024];
    if (last == BN - 1) {
#pragma unroll
      for (int i = 0; i < DPW; ++i) dma16_async(rs, k_src[i], to + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < DPW; ++i) {
        const int r = dma_row(i);
        dma16_async(rs, k_src[i] - uint32_t(r - min(r, last)) * uint32_t(kv_row_bytes), to + i * 1024);
      }
    }
  };
  // V^T[d][key] is written from registers.
  f32x4 vreg[TL::VREG];
  auto issue_v = [&](int it) {
    const int j0 = tile_j0(it);
#pragma unroll
    for (int i = 0; i < TL::VREG; ++i) {
      const int idx = static_cast<int>(threadIdx.x) + i * NW * 64;
      const int64_t j = min(int64_t(j0 + idx / CPR), n - 1);
      vreg[i] = *reinterpret_cast<const f32x4*>(v_base + j * kv_row_bytes + (idx % CPR) * 16);
    }
  };
  auto store_v = [&](int buf) {
    float* vt = reinterpret_cast<float*>(&sV[buf][0]);
#pragma unroll
    for (int i = 0; i < TL::VREG; ++i) {
      const int idx = static_cast<int>(threadIdx.x) + i * NW * 64;
#pragma unroll
      for (int e = 0; e < 4; ++e) vt[((idx % CPR) * 4 + e) * TL::VT_LD + idx / CPR] = vreg[i][e];
    }
  };

  f32x16 oacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) oacc[dt] = f32x16{};
  float m_run = kNegBig, l_run = 0.0f;
  float qf[KS];                                     // elements 2 kk + half of this lane's query row
  issue_v(0);
  issue_k(0);
  {
    const float* row = qg + min(int64_t(my_row), n - 1) * q_row + half;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = row[2 * kk];
  }
  // Q is waited for here, once: the tile loads are invisible to the compiler's
  // wait tracking, which would otherwise wait inside the loop.
  __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0)
  for (int it = 0; it < ntiles; ++it) {
    const int j0 = tile_j0(it);
    __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): this tile has landed
    store_v(it & 1);
    __syncthreads();                                // ... for every thread; the other buffers are free
    if (it + 1 < ntiles) {
      issue_v(it + 1);
      issue_k(it + 1);
    }
    // Does any (row, key) pair of this wave fall inside the mask?
    if (!wave_active || j0 > iw1 - 1 || !(j0 < s || band_start(iw0) <= j0 + BN - 1)) continue;
    const bool all_vis = (j0 + BN - 1 <= iw0) && (iw1 - iw0 == 32) && ((j0 + BN <= s) || band_start(iw1 - 1) <= j0);

    const char* kb = &sK[it & 1][0];
    auto kfrag = [&](int kk, int sub) {
      const int d = 2 * kk + half;
      const int at = lrow * RB + (((d / 4) ^ TL::swz(lrow)) * 16) + (d % 4) * 4;
      return *reinterpret_cast<const float*>(kb + sub * 32 * RB + at);
    };
    f32x16 sacc[2] = {f32x16{}, f32x16{}};
    // Fragments are read two steps ahead; the fence holds that order.
    float kf[3][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      kf[kk][0] = kfrag(kk, 0);
      kf[kk][1] = kfrag(kk, 1);
    }
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      if (kk + 2 < KS) {
        kf[(kk + 2) % 3][0] = kfrag(kk + 2, 0);
        kf[(kk + 2) % 3][1] = kfrag(kk + 2, 1);
      }
      sacc[0] = mma(kf[kk % 3][0], qf[kk], sacc[0]);
      sacc[1] = mma(kf[kk % 3][1], qf[kk], sacc[1]);
      sched_fence();
    }
    // Mask (edge tiles only) and the tile's raw row maximum.
    if (!all_vis) {
      const int jl = j0 + half * 4;                   // key of register 0 of this lane
      const int hi = my_row < i1 ? my_row - jl : -1;  // causal: key offset <= hi
      const int band = band_start(my_row) - jl;       // band: key offset >= band
      const int sink = s - jl;                        // sink: key offset < sink
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dj = sub * 32 + (r >> 2) * 8 + (r & 3);
          const bool vis = (dj <= hi) & ((dj < sink) | (dj >= band));
          sacc[sub][r] = vis ? sacc[sub][r] : -INFINITY;
        }
      }
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sacc[sub][r]);
    tmax = max_xor<32>(tmax) * c2;
    if (__any(tmax > m_run + kRescaleSlack)) {
      const float m_new = fmaxf(m_run, tmax);
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) oacc[dt] *= alpha;
    }
    float psum = 0.0f;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sacc[sub][r] = fast_exp2(mul_then_sub(sacc[sub][r], c2, m_run));
        psum += sacc[sub][r];
      }
    }
    l_run += sum_xor<32>(psum);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      const float* vt = reinterpret_cast<const float*>(&sV[it & 1][0]) + (dt * 32 + lrow) * TL::VT_LD;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          oacc[dt] = mma(vt[sub * 32 + (r >> 2) * 8 + half * 4 + (r & 3)], sacc[sub][r], oacc[dt]);
    }
  }

  if (!wave_active || my_row >= i1) return;
  const float inv_l = 1.0f / l_run;
  float* orow = static_cast<float*>(a.o) + (int64_t(b) * n * a.hq + h) * D + int64_t(my_row) * q_row;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) {
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = oacc[dt][grp * 4 + e] * inv_l;
      *reinterpret_cast<f32x4*>(orow + dt * 32 + grp * 8 + half * 4) = x;
    }
  }
}

int launch_shared(const PrefillArgs& a, void* stream) {
  PrefillArgs copy = a;
  const PrefillGrid g = prefill_grid(a, SharedTiles<64>::BM);
  if (g.blocks >= kMaxGrid) return kGridTooLarge;
  copy.n_qtiles = static_cast<int32_t>(g.tiles);
  copy.qchunk = static_cast<int32_t>(g.qchunk);
  copy.n_chunks = static_cast<int32_t>(g.n_chunks);
  copy.n_units = static_cast<int32_t>(g.n_units);
  void* args[] = {&copy};
  return static_cast<int>(hipLaunchKernel(reinterpret_cast<const void*>(&prefill_f32_shared_kernel<64>),
                                          dim3(static_cast<unsigned>(g.blocks)), dim3(NW * 64), args, 0,
                                          static_cast<hipStream_t>(stream)));
}

template <int D, int KG, int RW>
int launch_t(const PrefillArgs& a, void* stream) {
  const int64_t rows = RW * BR * (NW / KG);
  int64_t pairs = int64_t(a.hkv) * a.batch;
  if (pairs >= kPairsPerDie * kNumXcd) pairs = (pairs + kNumXcd - 1) / kNumXcd * kNumXcd;
  const int64_t blocks = (a.n + rows - 1) / rows * pairs * a.group;
  if (blocks >= kMaxGrid) return kGridTooLarge;
  PrefillArgs copy = a;
  void* args[] = {&copy};
  return static_cast<int>(hipLaunchKernel(reinterpret_cast<const void*>(&prefill_f32_kernel<D, KG, RW>),
                                          dim3(static_cast<unsigned>(blocks)), dim3(NW * 64), args, 0,
                                          static_cast<hipStream_t>(stream)));
}

}  // namespace

int launch_prefill_f32(const PrefillArgs& a, int head_dim, void* stream) {
  const PrefillF32Shape x = prefill_f32_shape(a, head_dim);
  if (head_dim == 64) {
    if (x.shared) return launch_shared(a, stream);
    if (x.row_blocks == 1) return launch_t<64, 4, 1>(a, stream);
    return x.key_groups == 4 ? launch_t<64, 4, 2>(a, stream) : launch_t<64, 2, 2>(a, stream);
  }
  if (head_dim == 128) {
    if (x.key_groups == 4) return launch_t<128, 4, 1>(a, stream);
    return x.key_groups == 2 ? launch_t<128, 2, 1>(a, stream) : launch_t<128, 1, 1>(a, stream);
  }
  return static_cast<int>(hipErrorInvalidValue);
}

}  // namespace moa
