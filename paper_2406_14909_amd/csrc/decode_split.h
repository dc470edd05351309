// How a decode call's virtual key range is cut into workers' pieces: the host
// part that chooses the pieces and the arithmetic that the kernels share.
// Plain C++, so that it also compiles without a GPU toolchain.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "moa_internal.h"

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define MOA_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MOA_HOST_DEVICE inline
#endif

namespace moa {

// Virtual keys of a call, and products of them with the number of workers, stay
// below 2^51, which makes the quotients below exact.
constexpr int64_t kMaxVirtual = int64_t(1) << 51;

// floor(a / b) with inv_b = 1.0 / b: (a + 1/2) / b is at least 1 / 2b away from
// an integer, and the product of the rounded values at most (a / b) 2^-52.  (A
// 64-bit integer division is a chain of several hundred cycles.)
MOA_HOST_DEVICE int64_t mul_floor(int64_t a, double inv_b) {
  return static_cast<int64_t>((static_cast<double>(a) + 0.5) * inv_b);
}

// Worker w's piece is units / workers units of 2^unit_shift keys, and one more
// for `units % workers` of the workers.  Where a unit is a round of the kernel's
// loop, these are the first ones, which sit on all dies and compute units alike
// (spread evenly, every second worker may be a long one, and work-groups go to
// the dies in turn: 16 x 16 heads of 1,294 keys at head_dim 64 24.1 us against
// 20.7).  Where it is a key, they are spread evenly, so that the pieces of equal
// caches or sequences begin with them wherever their number divides the workers'
// (16 x 8 KV heads x 2 query heads of 1,537 keys: 24.0 us against 25.2).
// No branches: the chain up to a work-group's first load counts in a small call.
MOA_HOST_DEVICE int64_t worker_start(const DecodeArgs& a, int w) {
  const int first = w < a.rem ? w : a.rem;
  const int spread = static_cast<int>(mul_floor(w * a.rem, a.inv_workers));
  return (w * a.per_worker + (a.unit_shift ? first : spread)) << a.unit_shift;
}

// The worker whose piece holds virtual key x.
MOA_HOST_DEVICE int worker_of(const DecodeArgs& a, int64_t x) {
  const int64_t u = x >> a.unit_shift;
  const bool later = u >= a.first_units;
  const int64_t num = later ? u - a.first_units : (u + 1) * a.first_mul - 1;
  return static_cast<int>(mul_floor(num, later ? a.inv_later : a.inv_first)) + (later ? a.rem : 0);
}

constexpr int64_t kMaxParts = 64;      // pieces that a cache is cut into, about, in a call of whole rounds
constexpr int64_t kRoundedMax = 2;     // rounds per slot up to which pieces are whole rounds

// Cuts the call for at most `slots` workers, each of which reads 2^round_shift
// keys per round of its loop.
//
// A small call is a chain of latencies, about 3 us per round, and a piece of 257
// keys where a round holds 128 takes three rounds, not two.  So up to kRoundedMax
// rounds per slot the units are rounds and each cache starts a new one.  One round
// per worker is the fastest as long as the slots last and no cache has more than
// about kMaxParts partials for the merge to read (per call: 32 heads of 1,064 keys
// on average 14.1 -> 8.1 us, of 2,112 keys 15.1 -> 12.5; 8 KV heads x 8 query heads
// of 2,112 keys 14.6 -> 9.9; 4 query heads, 8,256 keys, where the limit decides:
// 17.7 -> 15.7, without it 19.5).
// Above, memory bounds the call: every slot gets the same number of keys, to one
// (16 x 8 KV heads x 8 query heads at 3.05, 5.05 and 8.05 rounds per slot: 32.8,
// 48.1 and 70.6 us; in rounds, to one, 34.1, 49.4 and 73.2; ceil(rounds / slots)
// rounds for each worker, which leaves slots without work, 35.8, 51.1 and 72.9.
// At 1.3 rounds per slot 20.0 in keys, 19.4 in rounds).
// `paired` (the matrix-core kernels): where some worker has two rounds anyway, all
// have, up to 4/3 rounds per slot and from 7/4 on: half the partials, and more
// caches begin with a piece (4 x 8 KV heads x 8 query heads at 1.03, 1.15 and 1.75
// rounds per slot: 18.8 -> 17.0, 19.5 -> 17.6 and 25.6 -> 24.3 us).  Between, the
// idle slots cost more (1.45: 22.4 -> 24.1), and the vector kernel needs every
// slot's loads (4 x 16 heads of 4,181 keys at head_dim 64: 18.6 us, paired 20.0).
inline void split_decode(DecodeArgs& a, int64_t slots, int round_shift, bool paired) {
  const int64_t round = int64_t(1) << round_shift;
  int64_t rounds = 0, longest = 0;
  for (int g = 0; g < a.hkv; ++g) {
    const int64_t n = (a.seg_start[g + 1] - a.seg_start[g] + round - 1) >> round_shift;
    rounds += n;
    longest = std::max(longest, n);
  }
  rounds *= a.batch;
  int64_t units = a.seq_keys * a.batch, least = 1;
  a.unit_shift = 0;
  if (rounds <= kRoundedMax * slots) {
    int64_t at = 0, prev = 0;
    for (int g = 0; g < a.hkv; ++g) {
      const int64_t end = a.seg_start[g + 1];
      at += ((end - prev + round - 1) >> round_shift) << round_shift;
      prev = end;
      a.seg_start[g + 1] = at;
    }
    a.seq_keys = at;
    a.unit_shift = round_shift;
    units = rounds;
    const bool twos = paired && rounds > slots && (3 * rounds <= 4 * slots || 4 * rounds >= 7 * slots);
    least = std::max<int64_t>((longest + kMaxParts - 1) / kMaxParts, twos ? 2 : 1);
  }
  const int64_t exact = (kMaxVirtual - 1) / units;   // (decides for no caches that fit in memory)
  a.units = units;
  a.workers = static_cast<int32_t>(std::max<int64_t>(1, std::min({slots, (units + least - 1) / least, exact})));
  a.per_worker = units / a.workers;
  a.rem = static_cast<int32_t>(units % a.workers);
  a.inv_workers = 1.0 / a.workers;
  // worker_of: of the first `rem` pieces and of the later ones, or, spread evenly,
  // the largest w with w * units <= workers * u + workers - 1
  a.first_units = a.unit_shift ? a.rem * (a.per_worker + 1) : units;
  a.first_mul = a.unit_shift ? 1 : a.workers;
  a.inv_first = 1.0 / static_cast<double>(a.unit_shift ? a.per_worker + 1 : units);
  a.inv_later = 1.0 / static_cast<double>(a.per_worker);
  a.inv_seq_keys = 1.0 / static_cast<double>(a.seq_keys);
}

}  // namespace moa
