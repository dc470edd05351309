// Prefill attention with a per-KV-head banded-plus-sink causal mask (paper
// Sec. 2.1, Eq. 1, with the Sec. 3.2 span: sink prefix + diagonal band of
// width w_g).  Query i sees key j iff j <= i and (j < s or i - j < w_g).
// With the block band (paper Appendix "Main Setup": 64-token blocks) the band
// of row i instead starts at the first token of block i/64 - ceil(w_g/64) + 1;
// both are "j >= band_start(i)" with band_start(i) = ((i >> sh) - W + 1) << sh.
//
// One work-group = 4 waves = 128 query rows of one (sequence, query head) in a
// large launch (small ones: prefill_rule.h); each wave owns 32 rows.  The
// work-group walks only the 64-key tiles that intersect the sink prefix or the
// band of its rows; every other tile is skipped without being read.  K and V
// tiles are staged in LDS (the global loads of the next tiles are in flight
// while a tile is computed, one barrier per tile) and shared by the 4 waves.
// fp32 plans have a kernel of their own.
//
// Matrix-core formulation (CDNA4 32x32x16 bf16 MFMA):
//   S^T = K Q^T  : A = K tile rows (keys), B = Q^T kept in registers.
//                  Output lane l holds the scores of query row l % 32 for
//                  16 keys, so the row softmax needs one cross-lane step.
//   O^T += V^T P^T : B = P^T taken straight from the score registers
//                  (converted to bf16), A = V^T.  The V tile stays row-major in
//                  LDS and the transposing LDS read (ds_read_b64_tr_b16)
//                  delivers V^T fragments.
// The key order inside each 16-key MFMA step is permuted identically on both
// operands, which leaves the sum unchanged.
// Softmax is online in base 2 with the scale folded into one FMA per score;
// the row sum is accumulated over the bf16-rounded
// probabilities that the PV product uses.
// The running maximum used as the exponent offset is raised only when some
// row of the wave would otherwise see exponents above 2^8 (a wave-uniform
// test), so most tiles skip rescaling the output accumulator; the final
// normalisation by the running sum makes the result independent of that
// offset.  The mask is evaluated only on tiles that are not entirely visible
// to the wave's rows.
#include <algorithm>
#include <type_traits>

#include "moa_device.h"
#include "prefill_rule.h"

namespace moa {

namespace {

constexpr int BN = 64;    // keys per tile
constexpr float kRescaleSlack = 8.0f;   // log2 headroom before the offset is raised

typedef short i16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
#else
  (void)a;
  (void)b;
  return c;
#endif
}

// Transposing LDS read of four bf16: within each 16-lane group, lane 4a+b
// receives element b of the 8-byte reads issued by lanes 4e+a (e = 0..3).
// (The builtin exists only in the device pass; the host pass, which merely
// emits kernel stubs, sees an empty body.)
__device__ __forceinline__ bf16x4 read_tr(const bf16* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  const i16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) i16x4*)(const_cast<bf16*>(p)));
  return __builtin_bit_cast(bf16x4, r);
#else
  (void)p;
  return bf16x4{};
#endif
}

// acc + a + b with a, b in bf16 (v_dot2_f32_bf16 against (1, 1)).
__device__ __forceinline__ float dot2_ones(bf16 a, bf16 b, float acc) {
  typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
#if defined(__HIP_DEVICE_COMPILE__)
  const bf16x2 ab = {a, b};
  const bf16x2 ones = {bf16(1.0f), bf16(1.0f)};
  return __builtin_amdgcn_fdot2_f32_bf16(ab, ones, acc, false);
#else
  return acc + float(a) + float(b);
#endif
}

// NR waves of 32 query rows stage one key group's tiles.
template <int D, int NR>
struct Tiles {
  static constexpr int RB = D * 2;                   // bytes per K/V row
  static constexpr int CPR = RB / 16;                // 16-byte chunks per row
  static constexpr int TILE_BYTES = BN * RB;         // one K or V tile, rows unpadded
  static constexpr int DMA_PER_WAVE = TILE_BYTES / 1024 / NR;   // 1 KB direct-to-LDS loads
  // K is kept two tiles ahead (3 buffers), V one (2): 80 KB at head_dim 128.
  static constexpr int KSTAGES = 3;
  // K rows: chunk c of row r sits at chunk position c ^ swz_k(r), so the 16
  // rows read together by an MFMA operand load hit 16 different bank groups.
  __device__ __forceinline__ static int swz_k(int r) { return CPR >= 16 ? (r & 15) : ((r >> 1) & 7); }
  // V rows: depends on r mod 8 only; the 4 rows x 4 chunks read by half a wave
  // in one transposing load hit 16 different bank groups.
  __device__ __forceinline__ static int swz_v(int r) { return CPR >= 16 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); }
};

// KG key groups of NR waves share the 32 * NR query rows: group kg takes tiles
// kg, kg + KG, ... through LDS stages of its own, and the groups' states meet in
// LDS at the end.
template <int D, int NR, int KG>
__global__ void __launch_bounds__(NR * KG * 64, D == 128 && NR * KG == 4 && KG > 1 ? 1 : 2) prefill_kernel(PrefillArgs a) {
  using TL = Tiles<D, NR>;
  constexpr int BM = 32 * NR;             // query rows per work-group
  constexpr int KS = D / 16;              // MFMA steps over the head dimension
  constexpr int RB = TL::RB, CPR = TL::CPR, KST = TL::KSTAGES;

  constexpr int kGroupBytes = (KST + 2) * TL::TILE_BYTES;
  __shared__ __attribute__((aligned(1024))) char s_tiles[KG * kGroupBytes];

  const int lane = threadIdx.x & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform (scalar)
  const int wave = KG == 1 ? wave_id : wave_id % NR;                    // of the key group: rows
  const int kg = KG == 1 ? 0 : wave_id / NR;
  char* const sK = s_tiles + kg * kGroupBytes;
  char* const sV = sK + KST * TL::TILE_BYTES;
  const int lrow = lane & 31;
  const int half = lane >> 5;

  // Work item.  A dispatch unit is (KV head, sequence, qchunk consecutive
  // query tiles) with all `group` query heads of that KV head, so its work-
  // groups share K/V bands.  Units are ordered heaviest first (latest query
  // chunks first, then widest window) and dealt to the accelerator dies in
  // rounds of kNumXcd, alternating direction each round: work-group i runs on
  // die i % kNumXcd, which walks its units in order, so the work-groups
  // resident on one die at a time share that die's L2, and every die gets a
  // similar mix of heavy and light units.
  const int xcd = static_cast<int>(blockIdx.x % kNumXcd);
  const int local = static_cast<int>(blockIdx.x / kNumXcd);
  const int per_unit = a.group * a.qchunk;
  const int round = local / per_unit;
  const int unit = round * kNumXcd + ((round & 1) ? kNumXcd - 1 - xcd : xcd);
  if (unit >= a.n_units) return;                   // padding unit
  const int within = local % per_unit;
  const int hb = a.hkv * a.batch;
  const int cd = unit / hb;                        // chunk rank, heaviest first
  const int g = a.kv_order[(unit % hb) / a.batch];
  const int b = unit % a.batch;
  const int qt = (a.n_chunks - 1 - cd) * a.qchunk + (a.qchunk - 1 - within / a.group);
  if (qt >= a.n_qtiles) return;                     // past the last query tile
  const int h = g * a.group + within % a.group;
  const int64_t n = a.n;
  // Band of row i: keys from band_start(i) to i; token band (shift 0) or
  // block band (shift 6: whole 64-token blocks, window counted in blocks).
  const int wband = a.window[g];
  const int bsh = a.band_shift;
  auto band_start = [&](int i) { return ((i >> bsh) - wband + 1) * (1 << bsh); };
  const int s = a.num_sink;
  const float c2 = a.scale_log2;

  const int i0 = qt * BM;
  const int i1 = static_cast<int>(min(n, int64_t(i0 + BM)));   // exclusive
  const int iw0 = i0 + wave * 32;                                // this wave's rows
  const int iw1 = min(i1, iw0 + 32);
  const bool wave_active = iw0 < i1;

  // Tiles to visit: sink tiles [0, ta) then band tiles [tb, tl].
  const int ta = (min(s, i1) + BN - 1) / BN;
  const int tl = (i1 - 1) / BN;
  const int tb = max(ta, max(0, band_start(i0)) / BN);
  const int ntiles = ta + max(0, tl - tb + 1);

  const int64_t q_row_stride = int64_t(a.hq) * D;
  const int64_t kv_row_bytes = int64_t(a.hkv) * RB;
  const bf16* qg = static_cast<const bf16*>(a.q) + (int64_t(b) * n * a.hq + h) * D;
  const char* k_base = static_cast<const char*>(a.k) + (int64_t(b) * n * a.hkv + g) * RB;
  const char* v_base = static_cast<const char*>(a.v) + (int64_t(b) * n * a.hkv + g) * RB;

  // Q^T fragments of this lane's query row (loaded after the first tiles' DMA
  // is issued, see the pipeline prologue).
  bf16x8 qf[KS];

  // Direct-to-LDS tile loads: per-lane byte offsets of the sources relative to the
  // tile's first key row (tile independent).  Instruction I writes tile bytes
  // [I*1024, I*1024 + 1024): lane L's 16 bytes land at chunk m = I*64 + L, i.e.
  // row m / CPR, chunk position m % CPR, and carry global chunk
  // position ^ swz(row).  Wave w issues instructions w*DMA_PER_WAVE + i.  Keys
  // past the end re-read the last key (always masked by causality).
  constexpr int DPW = TL::DMA_PER_WAVE;
  uint32_t k_src[DPW], v_src[DPW];
  auto dma_row = [&](int i) { return ((wave * DPW + i) * 64 + lane) / CPR; };
#pragma unroll
  for (int i = 0; i < DPW; ++i) {
    const int m = (wave * DPW + i) * 64 + lane;
    const int r = m / CPR, p = m % CPR;
    k_src[i] = uint32_t(r) * uint32_t(kv_row_bytes) + uint32_t(p ^ TL::swz_k(r)) * 16u;
    v_src[i] = uint32_t(r) * uint32_t(kv_row_bytes) + uint32_t(p ^ TL::swz_v(r)) * 16u;
  }
  // With a.rotate the band tiles are visited in a rotated order: from the
  // unit's common start tile tr (the first band tile of its last query tile,
  // clipped to this work-group's band) up to tl, then from tb up to tr - 1.
  // The work-groups of a unit run side by side on one die, so at every step
  // they read the same key tile (before the wrap: tile tr + step; after it:
  // tile tb + step - (tl - tr + 1), the same for every work-group since tb
  // and tl move with the query tile in step), and each tile comes from memory
  // about once per unit.  Softmax over a set does not depend on the order of
  // its members.  Without a.rotate (keys and values that fit the last-level
  // cache) the band is visited from tb up, which spreads the concurrent reads
  // of a unit over many tiles.
  const int qt_top = min(a.n_qtiles - 1, (a.n_chunks - 1 - cd) * a.qchunk + a.qchunk - 1);
  const int tr = a.rotate ? min(max(tb, max(ta, max(0, band_start(qt_top * BM)) / BN)), tl + 1) : tb;
  const int n_upper = tl - tr + 1;                    // band tiles tr .. tl
  auto tile_j0 = [&](int it) {
    if (it < ta) return it * BN;
    const int k = it - ta;
    return (k < n_upper ? tr + k : tb + (k - n_upper)) * BN;
  };
  // The tiles are visited in runs of consecutive ones: within a run the next
  // tile's first key and byte offset follow by addition.  Scalar work between
  // the barrier and the products is time that the wave waits for: with a search
  // for the tile, two 64-bit products and a stage number modulo 3 per tile
  // instead, calls took 1.5 % (8 x 32 heads x 8,192: 3.17 against 3.13 ms) to 6 %
  // (32 heads x 4,096: 126 against 118.5 us) longer.
  const int64_t step_bytes = int64_t(KG * BN) * kv_row_bytes;
  int run = 0;                                        // steps left in the run of the newest tile
  auto seek = [&](int lt, int& j0, int64_t& off) {    // lt: the tile's number within this key group
    const int x = lt * KG + kg;
    j0 = tile_j0(x);
    off = int64_t(j0) * kv_row_bytes;
    const int end = x < ta ? ta : x - ta < n_upper ? ta + n_upper : 1 << 30;
    run = (end - 1 - x) / KG;
  };
  auto advance = [&](int lt, int& j0, int64_t& off) { // from tile lt - 1
    if (run > 0) {
      --run;
      j0 += KG * BN;
      off += step_bytes;
    } else {
      seek(lt, j0, off);
    }
  };
  // Tile loads go through a buffer resource that spans exactly the tile's real
  // key rows (at most BN), so no address outside the inputs is ever touched;
  // rows past the last key re-read key n-1 (always masked by causality).
  const int n32 = static_cast<int>(n);
  auto tile_dma = [&](const char* base, const auto& src, int j0, int64_t off, char* lds) {
    if (j0 + BN <= n32) {
      const i32x4 rs = make_desc(base + off, uint32_t(BN - 1) * uint32_t(kv_row_bytes) + RB);
#pragma unroll
      for (int i = 0; i < DPW; ++i) dma16_async(rs, src[i], lds + (wave * DPW + i) * 1024);
    } else {
      const int last = n32 - 1 - j0;
      const i32x4 rs = make_desc(base + off, uint32_t(last) * uint32_t(kv_row_bytes) + RB);
#pragma unroll
      for (int i = 0; i < DPW; ++i) {
        const int r = dma_row(i);
        const uint32_t at = src[i] - uint32_t(r - min(r, last)) * uint32_t(kv_row_bytes);
        dma16_async(rs, at, lds + (wave * DPW + i) * 1024);
      }
    }
  };

  // Per-lane byte offsets of the MFMA operand reads (tile independent).
  // K operand: row lrow (+ 32 * sub; the swizzle depends on the row's low bits
  // only), head-dim elements 16 * kk + 8 * half .. +7.
  int k_off[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) k_off[kk] = lrow * RB + (((2 * kk + half) ^ TL::swz_k(lrow)) * 16);
  // Transposing V read: lane 16G + 4e + a points at row (G/2)*4 + e (+ kb0),
  // bf16 column 32*dt + 16*(G%2) + 4a.
  int v_off[D / 32];
  {
    const int vr = (lane >> 5) * 4 + ((lane & 15) >> 2);    // row mod 8
    const int a4 = lane & 3;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      const int q = dt * 4 + ((lane >> 4) & 1) * 2 + (a4 >> 1);
      v_off[dt] = vr * RB + ((q ^ TL::swz_v(vr)) * 16) + (a4 & 1) * 8;
    }
  }

  f32x16 oacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) oacc[dt] = f32x16{};
  float m_run = kNegBig, l_run = 0.0f;
  const int my_row = iw0 + lrow;

  // Pipeline: during tile t, V(t+1) and then K(t+2) stream in; at the top of
  // tile t only the newest K loads may still be in flight.
  const int my_tiles = (ntiles - kg + KG - 1) / KG;   // of this key group
  const int rounds = (ntiles + KG - 1) / KG;          // barriers, the same for every group
  // Tiles of the loop: it (first key jt), it + 1 (V loads), it + 2 (K loads),
  // and the LDS stages they go to.
  int jt, j1, j2;
  int64_t off, off1, off2;
  seek(0, jt, off);
  if (my_tiles > 0) {
    tile_dma(v_base, v_src, jt, off, sV);
    tile_dma(k_base, k_src, jt, off, sK);
  }
  j1 = jt;
  off1 = off;
  advance(1, j1, off1);
  if (my_tiles > 1) tile_dma(k_base, k_src, j1, off1, sK + TL::TILE_BYTES);
  j2 = j1;
  off2 = off1;
  advance(2, j2, off2);
  int k_now = 0, k_next = (KST - 1) * TL::TILE_BYTES, v_now = 0;      // byte offsets of stages
  auto next_tile = [&](int it) {
    jt = j1;
    j1 = j2;
    off1 = off2;
    advance(it + 3, j2, off2);
    k_now = k_now == (KST - 1) * TL::TILE_BYTES ? 0 : k_now + TL::TILE_BYTES;
    k_next = k_next == (KST - 1) * TL::TILE_BYTES ? 0 : k_next + TL::TILE_BYTES;
    v_now ^= TL::TILE_BYTES;
  };
  {
    const int i = iw0 + lrow;
    if (wave_active && i < i1) {
      const bf16* qrow = qg + int64_t(i) * q_row_stride + 8 * half;
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + 16 * kk);
    } else {
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) qf[kk] = bf16x8{};
    }
  }
  // Wait for Q (and the first tiles) here, once.  The tile DMA is opaque to
  // the compiler's wait-count tracking, which would otherwise place waits for
  // the Q loads inside the tile loop, where they would also drain the
  // prefetches in flight.
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  for (int it = 0; it < rounds; next_tile(it), ++it) {
    const int j0 = jt;
    if (it + 1 < my_tiles) {
      // all but the last DPW loads (K(it+1)) have landed: K(it), V(it)
      __builtin_amdgcn_s_waitcnt(0x0F70 | DPW);
    } else {
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    }
    __syncthreads();                      // ... for every thread; K(it-1), V(it-1) buffers are free

    // Does any (row, key) pair of this wave fall inside the mask?
    const bool any_causal = j0 <= iw1 - 1;
    const bool any_vis = wave_active && it < my_tiles && any_causal && (j0 < s || band_start(iw0) <= j0 + BN - 1);
    // The next tiles' loads go between the S products: issued at once after the
    // barrier, the loads of all waves queue for the compute unit's one address
    // unit and the waves stand still meanwhile.  Worth 1 - 4 % at head_dim 128
    // (32 heads x 2,048: 53.7 -> 51.5 us); at 64, where other waves fill the
    // gap, it costs 2 %.
    constexpr bool kSpread = D == 128;
    const bool spread = kSpread && any_vis && it + 2 < my_tiles && j1 + BN <= n32 && j2 + BN <= n32;
    if (!spread) {
      if (it + 1 < my_tiles) tile_dma(v_base, v_src, j1, off1, sV + (v_now ^ TL::TILE_BYTES));
      if (it + 2 < my_tiles) tile_dma(k_base, k_src, j2, off2, sK + k_next);
    }
    if (!any_vis) continue;
    const bool all_vis = (j0 + BN - 1 <= iw0) && (iw1 - iw0 == 32) &&
                         ((j0 + BN <= s) || band_start(iw1 - 1) <= j0);

    // S^T = K Q^T for two 32-key sub-tiles.
    // The two 32-key chains alternate so consecutive MFMAs are independent.
    const char* kb = sK + k_now;
    auto kfrag = [&](int kk, int sub) {
      return *reinterpret_cast<const bf16x8*>(kb + sub * 32 * RB + k_off[kk]);
    };
    f32x16 sacc[2] = {f32x16{}, f32x16{}};
    // Fragments are read two steps ahead.  The fence holds that order: the
    // scheduler otherwise saves the registers and reads each step's fragments
    // right before their use, one LDS latency per step (0.5 - 2 % of a call at
    // head_dim 128, nothing at 64, where four waves share a SIMD).
    bf16x8 kf[3][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      kf[kk][0] = kfrag(kk, 0);
      kf[kk][1] = kfrag(kk, 1);
    }
    auto products = [&](auto with_loads) {
      i32x4 rv = {}, rk = {};
      if constexpr (decltype(with_loads)::value) {
        const uint32_t bytes = uint32_t(BN - 1) * uint32_t(kv_row_bytes) + RB;
        rv = make_desc(v_base + off1, bytes);
        rk = make_desc(k_base + off2, bytes);
      }
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        if (kk + 2 < KS) {
          kf[(kk + 2) % 3][0] = kfrag(kk + 2, 0);
          kf[(kk + 2) % 3][1] = kfrag(kk + 2, 1);
        }
        sacc[0] = mma(kf[kk % 3][0], qf[kk], sacc[0]);
        sacc[1] = mma(kf[kk % 3][1], qf[kk], sacc[1]);
        if constexpr (decltype(with_loads)::value) {
          // V(it + 1) first: only the newest K loads may be in flight at the next tile.
          constexpr int kPerStep = 2 * DPW / KS;
#pragma unroll
          for (int e = 0; e < kPerStep; ++e) {
            const int m = kk * kPerStep + e;
            if (m < DPW) dma16_async(rv, v_src[m % DPW], sV + (v_now ^ TL::TILE_BYTES) + (wave * DPW + m) * 1024);
            else dma16_async(rk, k_src[m % DPW], sK + k_next + (wave * DPW + m - DPW) * 1024);
          }
        }
        sched_fence();
      }
    };
    if constexpr (kSpread) {
      if (spread) products(std::true_type{});
      else products(std::false_type{});
    } else {
      products(std::false_type{});
    }

    // The first V^T fragments are read here, behind the mask and the weights
    // (1 - 2 %: 8 x 32 heads x 8,192: 3.19 -> 3.14 ms).
    const char* vb = sV + v_now;
    auto vfrag = [&](int step, int dt) {
      const int kb0 = (step >> 1) * 32 + 16 * (step & 1);
      const bf16x4 lo4 = read_tr(reinterpret_cast<const bf16*>(vb + kb0 * RB + v_off[dt]));
      const bf16x4 hi4 = read_tr(reinterpret_cast<const bf16*>(vb + (kb0 + 8) * RB + v_off[dt]));
      return __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    bf16x8 vf[2][D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) vf[0][dt] = vfrag(0, dt);
    sched_fence();

    // Mask (edge tiles only; branch-free selects) and the tile's raw row maximum.
    if (!all_vis) {
      const int jl = j0 + half * 4;                 // key of register 0 of this lane
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
    tmax *= c2;
    // Raise the exponent offset only when some row of the wave needs it.  Only
    // then do the two lanes of a row meet; their sums meet after the last tile
    // (an exchange of each per tile: 1 - 2 % of a call).
    if (__any(tmax > m_run + kRescaleSlack)) {
      const float m_new = fmaxf(m_run, max_xor<32>(tmax));
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) oacc[dt] *= alpha;
    }

    // P in bf16; the row sum is taken over the same rounded weights that
    // enter the PV product (dot2 with (1, 1)).
    bf16x8 pf[2][2];
    float psum = 0.0f;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          pf[sub][c][e] = static_cast<bf16>(fast_exp2(__builtin_fmaf(sacc[sub][8 * c + e], c2, -m_run)));
#pragma unroll
        for (int e = 0; e < 8; e += 2) psum = dot2_ones(pf[sub][c][e], pf[sub][c][e + 1], psum);
      }
    }
    l_run += psum;

    // O^T += V^T P^T: for each 16-key step the d-tile accumulators are
    // independent; the V^T fragments of the next step are read meanwhile.
#pragma unroll
    for (int step = 0; step < 4; ++step) {
      if (step + 1 < 4) {
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) vf[(step + 1) & 1][dt] = vfrag(step + 1, dt);
      }
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
        oacc[dt] = mma(vf[step & 1][dt], pf[step >> 1][step & 1], oacc[dt]);
    }
  }

  l_run = sum_xor<32>(l_run);
  if constexpr (KG > 1) {
    // The groups' states of the same rows sit in the same lanes of waves w and
    // w + NR: each group but the first leaves (accumulator, m, l) in LDS.
    constexpr int kRegs = D / 2 + 2;                  // values per lane
    static_assert((KG - 1) * NR * kRegs * 256 <= KG * kGroupBytes, "the states fit the tiles' LDS");
    float* const st = reinterpret_cast<float*>(s_tiles) + lane;
    __syncthreads();                                  // every tile has been read
    if (kg > 0) {
      float* p = st + ((kg - 1) * NR + wave) * kRegs * 64;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) p[(dt * 16 + r) * 64] = oacc[dt][r];
      p[(kRegs - 2) * 64] = m_run;
      p[(kRegs - 1) * 64] = l_run;
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll 1
    for (int v = 0; v < KG - 1; ++v) {
      const float* p = st + (v * NR + wave) * kRegs * 64;
      const float m2 = p[(kRegs - 2) * 64];
      const float m_new = fmaxf(m_run, m2);
      const float f1 = fast_exp2(m_run - m_new), f2 = fast_exp2(m2 - m_new);
      m_run = m_new;
      l_run = l_run * f1 + p[(kRegs - 1) * 64] * f2;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = oacc[dt][r] * f1 + p[(dt * 16 + r) * 64] * f2;
    }
  }

  if (!wave_active || my_row >= i1) return;
  const float inv_l = 1.0f / l_run;
  bf16* orow = static_cast<bf16*>(a.o) + (int64_t(b) * n * a.hq + h) * D + int64_t(my_row) * q_row_stride;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) {
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      const int d0 = dt * 32 + grp * 8 + half * 4;
      bf16x4 outv;
#pragma unroll
      for (int e = 0; e < 4; ++e) outv[e] = static_cast<bf16>(oacc[dt][grp * 4 + e] * inv_l);
      *reinterpret_cast<bf16x4*>(orow + d0) = outv;
    }
  }
}

template <int D, int NR, int KG>
int launch_t(const PrefillArgs& a, void* stream) {
  PrefillArgs copy = a;
  const PrefillGrid g = prefill_grid(a, 32 * NR);
  if (g.blocks >= kMaxGrid) return kGridTooLarge;
  copy.n_qtiles = static_cast<int32_t>(g.tiles);
  copy.qchunk = static_cast<int32_t>(g.qchunk);
  copy.n_chunks = static_cast<int32_t>(g.n_chunks);
  copy.n_units = static_cast<int32_t>(g.n_units);
  void* args[] = {&copy};
  return static_cast<int>(hipLaunchKernel(reinterpret_cast<const void*>(&prefill_kernel<D, NR, KG>),
                                          dim3(static_cast<unsigned>(g.blocks)), dim3(NR * KG * 64), args, 0,
                                          static_cast<hipStream_t>(stream)));
}

template <int D>
int launch_d(const PrefillArgs& a, void* stream) {
  const PrefillShape shape = prefill_shape(a, D);
  if (shape.waves == 2) return launch_t<D, 2, 2>(a, stream);
  if (shape.key_groups == 2) return launch_t<D, 4, 2>(a, stream);
  return launch_t<D, 4, 1>(a, stream);
}

}  // namespace

int launch_prefill(const PrefillArgs& a, int head_dim, void* stream) {
  if (head_dim == 128) return launch_d<128>(a, stream);
  if (head_dim == 64) return launch_d<64>(a, stream);
  return static_cast<int>(hipErrorInvalidValue);
}

}  // namespace moa
