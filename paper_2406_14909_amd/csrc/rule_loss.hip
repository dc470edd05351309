// Rule-loss table (paper Sec. 3.3, Eq. 4): the accuracy loss of giving head h
// rule r at length N is the head's block-averaged attention influence summed
// over the causal pairs the rule masks,
//     dl[h][r] = sum over blocks (I, J) of masked_r(I, J) * ebar[h][I][J],
// where masked_r(I, J) counts the pairs (i, j) of the 64 x 64 block with
// j <= i, j >= s and j < band_start_r(i) (every token of a block carries the
// block's mean).
//
// Between whole blocks past the sinks masked_r depends on the distance
// k = I - J alone, so the profile is first folded along its diagonals, for all
// rules at once: D[k] = sum of ebar[I][I - k].  Two lines of blocks count
// differently and are kept aside, also by distance: the block column that
// holds the sink edge (C[k]) and a last block row of fewer than 64 tokens
// (L[k]).  A rule of band length w masks every block at distance
// k >= k_full completely, k_full = ceil((w + 63) / 64) (w blocks with the
// block band), and with the token band the two distances before it in part;
// so with suffix sums of the three lines it costs three lookups and at most
// seven closed-form counts.  Sums are fp64.
//
// What bounds it: reading the lower triangle once (1024 heads at n = 8192:
// 33.8 MB in 10.0 us, 3.4 TB/s) and, below about 10 MB, the start and the end
// of a work-group.  Each element costs one load, one conversion and one fp64
// add; an earlier version scanned every block row in fp64 and evaluated every
// rule on it, which the vector ALUs bounded (44.0 us).
#include "moa_device.h"

namespace moa {

namespace {

constexpr int kBlock = kInfluenceBlock;

// sum_{x = 0}^{t} clamp(x, 0, m) for 0 <= m <= 64 and |t| < 2^20
__device__ __forceinline__ int clamp_prefix(int t, int m) {
  if (t < 0) return 0;
  if (t <= m) return t * (t + 1) / 2;
  return m * (m + 1) / 2 + (t - m) * m;
}

// Causal pairs of block (I, J) hidden by a rule (band length w in units of
// 2^bsh tokens, s sinks) at length n <= 65536 (at most 64 x 64).
__device__ __forceinline__ int masked_in_block(int I, int J, int n, int s, int w, int bsh) {
  const int r0 = I * kBlock, r1 = min(n, r0 + kBlock);
  const int c0 = J * kBlock, c1 = min(n, c0 + kBlock);
  const int lo = max(c0, s);                       // sinks are never masked
  if (c1 <= lo) return 0;
  if (bsh != 0) {
    const int bs = ((r0 >> bsh) - min(w, (r0 >> bsh) + 2) + 1) * (1 << bsh);   // same start for every row
    return (r1 - r0) * max(0, min(c1, bs) - lo);
  }
  // row i masks [lo, min(c1, i - w + 1)): clamp(i + 1 - w - lo, 0, c1 - lo)
  const int a = 1 - min(w, r1 + 1) - lo, m = c1 - lo;
  return clamp_prefix(r1 - 1 + a, m) - clamp_prefix(r0 - 1 + a, m);
}

// DPP move of an fp64 value (both halves with the same control); lanes with
// no source, or in rows outside row_mask, receive 0.
template <int ctrl, int row_mask>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u & 0xffffffffu), ctrl, row_mask, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), ctrl, row_mask, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo));
}

// Inclusive prefix sum over the 64 lanes: shifts by 1, 2, 4, 8 within each
// row of 16 lanes, then row_bcast:15 (row totals into rows 1 and 3) and
// row_bcast:31 (the first half's total into rows 2 and 3).
__device__ __forceinline__ double wave_inclusive_scan(double v) {
  v += dpp_f64<0x111, 0xF>(v);
  v += dpp_f64<0x112, 0xF>(v);
  v += dpp_f64<0x114, 0xF>(v);
  v += dpp_f64<0x118, 0xF>(v);
  v += dpp_f64<0x142, 0xA>(v);
  v += dpp_f64<0x143, 0xC>(v);
  return v;
}

__device__ __forceinline__ double lane63(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffu), 63);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), 63);
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// One work-group per head.  Thread t folds distance k = t % kDist of block
// rows t / kDist + m * (threads / kDist): consecutive lanes read consecutive
// elements of a row, and kDepth rows are in flight per thread.
template <int kThreads, int kDist, int kDepth>   // kDist: power of two >= nb, <= kThreads
__global__ void __launch_bounds__(kThreads) rule_loss_kernel(RuleLossArgs a) {
  constexpr int kGroups = kThreads / kDist;
  static_assert(kGroups >= 1 && kDist % 64 == 0, "thread mapping");
  __shared__ double s_d[kGroups][kDist];       // diagonal sums; row 0: of all block rows
  __shared__ double s_suf[3][kDist + 64];      // suffix sums of D, C, L (0 from nb on)
  __shared__ float s_line[2][kDist];           // C and L
  __shared__ double s_part[3][kMaxRules];
  const int t = static_cast<int>(threadIdx.x);
  const int lane = t & 63, wave = t >> 6;
  const int h = static_cast<int>(blockIdx.x);
  const int nb = a.nb, n = a.n, s = a.num_sink, bsh = a.band_shift;
  const float* e = a.ebar + int64_t(h) * nb * nb;
  const int ja = (s + kBlock - 1) / kBlock;              // first block with no sink column
  const int js = (s % kBlock) ? s / kBlock : nb;         // block column of the sink edge (nb: none)
  const int rows_last = n - (nb - 1) * kBlock;
  const int nbw = rows_last == kBlock ? nb : nb - 1;     // block rows of 64 tokens

  // D: rows I >= ja + k, so that J = I - k lies past the sinks.  A batch of
  // rows that every lane of the wave sees (k0 .. k0 + 63) loads without a test.
  const int k = t & (kDist - 1), grp = t / kDist;
  const int k0 = __builtin_amdgcn_readfirstlane(k);
  double d = 0.0;
  // first batch that reaches row ja + k0
  const int skip = max(0, ja + k0 - grp) / (kGroups * kDepth) * (kGroups * kDepth);
  for (int i0 = grp + skip; i0 < nbw; i0 += kGroups * kDepth) {
    float x[kDepth];
    if (i0 - (k0 + 63) >= ja && i0 + (kDepth - 1) * kGroups < nbw) {
      const float* p = e + (i0 * nb + (i0 - k));
#pragma unroll
      for (int u = 0; u < kDepth; ++u) x[u] = p[u * kGroups * (nb + 1)];
    } else {
#pragma unroll
      for (int u = 0; u < kDepth; ++u) {
        const int i = i0 + u * kGroups;
        const bool in = i < nbw && i - k >= ja;
        const float y = e[in ? i * nb + (i - k) : 0];
        x[u] = in ? y : 0.0f;
      }
    }
#pragma unroll
    for (int u = 0; u < kDepth; ++u) d += static_cast<double>(x[u]);
  }
  s_d[grp][k] = d;
  if (grp == 0) {
    s_line[0][k] = js + k < nbw ? e[int64_t(js + k) * nb + js] : 0.0f;
    s_line[1][k] = (nbw < nb && nb - 1 - k >= ja) ? e[int64_t(nb - 1) * nb + (nb - 1 - k)] : 0.0f;
  }
  __syncthreads();
  if (kGroups > 1 && grp == 0) {
#pragma unroll
    for (int v = 1; v < kGroups; ++v) d += s_d[v][k];
    s_d[0][k] = d;
  }
  __syncthreads();

  // Suffix sums: one wave per line, from the largest distance down.
  if (wave < 3) {
    double carry = 0.0;
    s_suf[wave][kDist + lane] = 0.0;
    for (int c = kDist - 64; c >= 0; c -= 64) {
      const int kk = c + 63 - lane;
      const double v = wave_inclusive_scan(wave == 0 ? s_d[0][kk] : static_cast<double>(s_line[wave - 1][kk])) + carry;
      s_suf[wave][kk] = v;
      carry = lane63(v);
    }
  }
  __syncthreads();

  // Lane r of wave 0, 1, 2: rule r's share of D, C, L.
  if (wave < 3 && lane < a.num_rules) {
    const int w = a.window[lane];
    const int k_full = bsh ? min(w, kDist) : min((w + 2 * kBlock - 2) / kBlock, kDist);
    const int cols = wave == 1 ? kBlock - s % kBlock : kBlock;      // columns past the sinks
    const int rows = wave == 2 ? rows_last : kBlock;
    double acc = static_cast<double>(rows * cols) * s_suf[wave][k_full];
    if (bsh == 0) {
#pragma unroll
      for (int m = 1; m <= 2; ++m) {
        const int kk = k_full - m;
        if (kk < 0 || kk >= nb) continue;
        // any whole block at distance kk stands for all of them
        int cnt;
        if (wave == 0) cnt = masked_in_block(ja + kk, ja, (ja + kk + 1) * kBlock, s, w, 0);
        else if (wave == 1) cnt = masked_in_block(js + kk, js, (js + kk + 1) * kBlock, s, w, 0);
        else cnt = nb - 1 - kk >= ja ? masked_in_block(nb - 1, nb - 1 - kk, n, s, w, 0) : 0;
        acc += static_cast<double>(cnt) * (wave == 0 ? s_d[0][kk] : static_cast<double>(s_line[wave - 1][kk]));
      }
    }
    if (wave == 2 && nbw < nb && js < nb)                            // where the two lines cross
      acc += static_cast<double>(masked_in_block(nb - 1, js, n, s, w, bsh)) *
             static_cast<double>(e[int64_t(nb - 1) * nb + js]);
    s_part[wave][lane] = acc;
  }
  __syncthreads();
  if (wave != 0 || lane >= a.num_rules) return;
  a.dl[int64_t(h) * a.num_rules + lane] = s_part[0][lane] + (s_part[1][lane] + s_part[2][lane]);
  if (h == 0) a.density[lane] = static_cast<double>(a.kv_len[lane]) / static_cast<double>(n);
}

}  // namespace

// Threads and rows in flight per work-group by the number of block rows; heads
// x n: time before and now (54 rules, graph replays, three profiles in turn).
//   nb <= 64: little to read, the start and the end of a work-group count:
//     1024 x 2000: 12.7 -> 4.4 us (512 threads: 5.5).
//   nb <= 256: 1024 x 8192: 44.0 -> 10.0 us (256 threads 10.7, 1024 12.4);
//     128 x 16000: 71.6 -> 12.2 (18.7, 9.4); 1024 x 16000: 102.8 -> 37.4.
//   above: one row at a time per work-group, so more of them in flight:
//     32 x 32768: 190 -> 15.4 us (8 rows in flight 19.9, 512 threads 31.6);
//     32 x 65536: 538 -> 56.8 (84.0 with 8 rows in flight).
int launch_rule_loss(const RuleLossArgs& a, void* stream) {
  RuleLossArgs copy = a;
  void* args[] = {&copy};
  const void* kernel;
  unsigned threads = 512;
  if (a.nb <= 64) {
    kernel = reinterpret_cast<const void*>(&rule_loss_kernel<256, 64, 8>);
    threads = 256;
  } else if (a.nb <= 128) {
    kernel = reinterpret_cast<const void*>(&rule_loss_kernel<512, 128, 8>);
  } else if (a.nb <= 256) {
    kernel = reinterpret_cast<const void*>(&rule_loss_kernel<512, 256, 8>);
  } else if (a.nb <= 512) {
    kernel = reinterpret_cast<const void*>(&rule_loss_kernel<1024, 512, 32>);
    threads = 1024;
  } else if (a.nb <= 1024) {
    kernel = reinterpret_cast<const void*>(&rule_loss_kernel<1024, 1024, 32>);
    threads = 1024;
  } else {
    return static_cast<int>(hipErrorInvalidValue);
  }
  return static_cast<int>(hipLaunchKernel(kernel, dim3(static_cast<unsigned>(a.num_heads)), dim3(threads), args, 0,
                                          static_cast<hipStream_t>(stream)));
}

}  // namespace moa
