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

constexpr int64_t kRoundedMax = 16;    // rounds per slot up to which pieces are whole rounds
constexpr int64_t kAlignedMax = 2;     // the same where pieces of equal keys begin with the caches
constexpr int64_t kMaxParts = 256;     // pieces that a cache is cut into, about, in a call of whole rounds
constexpr int64_t kFewParts = 64;      // the same of caches of up to 4 * kFewParts rounds, up to two rounds per slot

// Cuts the call for at most `slots` workers, each of which reads 2^round_shift
// keys per round of its loop.
//
// A small call is a chain of latencies, about 3 us per round, and a piece of 257
// keys where a round holds 128 takes three rounds, not two; so does one of 256
// that crosses from one cache to the next.  So the units are rounds and each cache
// starts a new one.  One round per worker is the fastest as long as the slots last
// and the merge has few partials to read (per call: 32 heads of 1,064 keys on
// average 14.1 -> 8.1 us, of 2,112 keys 15.1 -> 12.5; 8 KV heads x 8 query heads of
// 2,112 keys 14.6 -> 9.9).
// With more rounds than slots every slot gets the same number, to one (windows of a
// rule, one of ceil(rounds / slots) rounds for each worker, of equal keys, of
// rounds dealt: 7 x 8 KV heads x 4 query heads, 2.13 rounds per slot 27.6, 28.1,
// 24.9 us; 14 x 16 heads, head_dim 64, 3.05 41.6, 39.2, 37.5; 20 x 8 x 8 heads, 4.58
// 45.1, 45.7, 43.7; 24 x 32 heads, 5.25 60.6, 58.5, 57.9).  Above kRoundedMax
// a partial round weighs nothing (16 x 32 heads, 23.0: 232, 232, 232).
// Equal caches whose number divides the slots': pieces of equal keys begin with
// them and cross none, so that only the last round of each is partial (16 x 8 KV
// heads x 8 query heads at 3.05, 5.05 and 8.05: 35.8, 51.1 and 72.9 us by
// ceil(rounds / slots), 32.8, 48.1 and 70.6 by keys, 34.1, 49.4 and 73.2 dealt).
// Few long caches have the merge read many partials, and what each costs it is to
// be weighed against longer pieces: up to kMaxParts (1 x 8 heads of 100,064 and
// 131,136 keys 21.7 and 24.0 us; without a limit 27.1 and 40.0, with 64 31.2 and
// 38.1), and kFewParts of caches that this cuts into pieces of at most four rounds
// (8 KV heads x 4 query heads of 12,064 and 24,064 keys 16.5 and 23.8 us; without,
// 17.6 and 25.4), up to two rounds per slot: beyond, fewer parts leave slots without
// work (8 x 4 heads of 25,064 to 100,064 keys, 4.71: 48.9 us; with 64 52.7).
// `paired` (the matrix-core kernels): where some worker has two rounds anyway, all
// have, up to 4/3 rounds per slot and from 7/4 to 2: half the partials, and more
// caches begin with a piece (4 x 8 KV heads x 8 query heads at 1.03, 1.15 and 1.75
// rounds per slot: 18.8 -> 17.0, 19.5 -> 17.6 and 25.6 -> 24.3 us).  Between, the
// idle slots cost more (1.45: 22.4 -> 24.1), and the vector kernel needs every
// slot's loads (4 x 16 heads of 4,181 keys at head_dim 64: 18.6 us, paired 20.0).
inline void split_decode(DecodeArgs& a, int64_t slots, int round_shift, bool paired) {
  const int64_t round = int64_t(1) << round_shift;
  int64_t rounds = 0, least_keys = a.seg_start[1], most_keys = 0;
  for (int g = 0; g < a.hkv; ++g) {
    const int64_t keys = a.seg_start[g + 1] - a.seg_start[g];
    rounds += (keys + round - 1) >> round_shift;
    least_keys = std::min(least_keys, keys);
    most_keys = std::max(most_keys, keys);
  }
  rounds *= a.batch;
  const int64_t longest = (most_keys + round - 1) >> round_shift;
  int64_t units = a.seq_keys * a.batch, least = 1;
  a.unit_shift = 0;
  const bool aligned = slots % (int64_t(a.hkv) * a.batch) == 0 && least_keys == most_keys;
  if (rounds <= (aligned ? kAlignedMax : kRoundedMax) * slots) {
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
    const int64_t parts = rounds <= 2 * slots && longest <= 4 * kFewParts ? kFewParts : kMaxParts;
    least = std::max<int64_t>((longest + parts - 1) / parts, twos ? 2 : 1);
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
