// A sort of a few thousand 32-bit keys with their indices by one workgroup, ties by index, without
// radix passes: four buckets a thread of equal width from the smallest key on (the bucket number
// never falls as the key rises, whatever the rounding), counted with LDS atomics; a scan gives each
// bucket its place, and within its bucket a pair's place is the number of smaller pairs there: six
// barriers in all, where four radix passes take twenty. A bucket of more than bucket_most pairs
// gives up, before the first count if a sample of the keys shows it (up to 0.3 us; of all eight keys a thread 0.6
// of 24 at 8,192 pairs). Keys equal to the smallest or the largest one (idle nodes' zeros, saturated slacks) and
// outliers above the others would crowd buckets, so they get their own treatment (1.4 us of 14.2 at
// 4,096 pairs). Not kept: twice the buckets (no change at 4,096 pairs), and a thread's pairs compared
// round by round together (13.5 against 12.4 us).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace maestro {

constexpr int kBucketWaves = 16;          // at most 1,024 threads
// Pairs of a bucket at most (each is compared with all of them, which one workgroup's LDS serves): with it
// fewer threads and pairs a thread allow longer buckets.
__device__ __forceinline__ uint32_t bucket_most(int n_waves, int items) {
  return n_waves <= 8 ? 256u : items == 1 ? 64u : 32u;
}

// Sorts (key, index) pairs; thread t of wavefront w holds the indices idx[j] = 64 (IPT w + j) + lane,
// those below n count. `above(key, low)` maps keys to floats that never fall as the key rises, 0 at
// `low`. pair: n entries of LDS, count: four words a thread, 16-byte aligned. Both outcomes are
// workgroup-uniform. True: pair[0 .. n-1] holds the pairs in order, behind a barrier. False (a value
// that is not finite, or crowded buckets): both arrays are free again, behind a barrier.
template <int IPT, class Above>
__device__ __forceinline__ bool bucket_sort(const uint32_t (&key)[IPT], const uint32_t (&idx)[IPT], int32_t n,
                                            uint64_t* __restrict__ pair, uint32_t* __restrict__ count, Above above) {
  __shared__ uint32_t s_low[kBucketWaves], s_high[kBucketWaves], s_same[kBucketWaves];
  __shared__ uint32_t s_sum[kBucketWaves], s_ends[kBucketWaves], s_full;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, n_waves = blockDim.x >> 6;
  uint4* own = reinterpret_cast<uint4*>(count) + t;      // four buckets a thread
  *own = make_uint4(0u, 0u, 0u, 0u);
  uint32_t low = 0xFFFFFFFFu, high = 0u;
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if ((int)idx[j] < n) {
      low = min(low, key[j]);
      high = max(high, key[j]);
    }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    low = min(low, __shfl_xor(low, off));
    high = max(high, __shfl_xor(high, off));
  }
  // one key a wavefront, neither its smallest nor its largest (so below the padding's), and how many others
  // equal it there, among four of eight keys a thread: over the wavefronts about as many as share a bucket
  constexpr int kSample = IPT > 4 ? 4 : IPT;
  uint32_t same = 0u;
  const uint64_t between = __ballot((int)idx[0] < n && key[0] != low && key[0] != high);
  if (between) {
    const uint32_t one = __builtin_amdgcn_readlane(key[0], __ffsll((unsigned long long)between) - 1);
#pragma unroll
    for (int j = 0; j < kSample; ++j) same += (uint32_t)__popcll(__ballot(key[j] == one));
    same -= 1u;
  }
  if (lane == 0) {
    s_low[wave] = low;
    s_high[wave] = high;
    s_same[wave] = same;
  }
  if (t == 0) s_full = 0u;
  __syncthreads();
  // the buckets end at the second largest of the wavefronts' largest keys, so that far outliers in
  // one wavefront share the last bucket instead of leaving the others in the first
  uint32_t second = 0u;
  high = same = 0u;
#pragma unroll
  for (int w = 0; w < kBucketWaves; ++w) {                 // reads in flight together
    const uint32_t l = s_low[w], h = s_high[w], c = s_same[w];
    if (w < n_waves) {
      same += c;
      low = min(low, l);
      second = max(second, min(high, h));
      high = max(high, h);
    }
  }
  const uint32_t edge = n > 3 * 64 * IPT ? second : high;
  const float span = above(edge > low ? edge : high, low);
  const int last = 4 * (int)blockDim.x - 1;
  const float scale = (float)last / span;
  const uint32_t most = bucket_most(n_waves, IPT);
  const bool crowded = 5u * (IPT / kSample) * same > 4u * most;
  if (!(above(high, low) < INFINITY) || (low != high && !(scale < INFINITY)) || crowded) return false;
  // The smallest and the largest key are not counted: their pairs' places are the first and the last
  // ones, in index order.
  const uint64_t lanes_below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t bucket[IPT], arrived[IPT], n_low = 0u, n_high = 0u;
  bool inner[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const bool real = (int)idx[j] < n, is_low = real && key[j] == low,
               is_high = real && key[j] == high && high != low;
    const uint64_t lows = __ballot(is_low), highs = __ballot(is_high);
    arrived[j] = is_low ? n_low + (uint32_t)__popcll(lows & lanes_below) : n_high + (uint32_t)__popcll(highs & lanes_below);
    n_low += (uint32_t)__popcll(lows);
    n_high += (uint32_t)__popcll(highs);
    bucket[j] = 0u;
    inner[j] = real && !is_low && !is_high;
    if (inner[j]) {
      bucket[j] = (uint32_t)fminf(above(key[j], low) * scale, (float)last);
      arrived[j] = atomicAdd(&count[bucket[j]], 1u);
    }
  }
  if (lane == 0) s_ends[wave] = n_low | (n_high << 16);
  __syncthreads();
  const uint4 c = *own;
  uint32_t incl = c.x + c.y + c.z + c.w;
  const uint32_t mine = incl;
  if (max(max(c.x, c.y), max(c.z, c.w)) > most) s_full = 1u;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t v = __shfl_up(incl, off);
    if (lane >= off) incl += v;
  }
  if (lane == 63) s_sum[wave] = incl;
  __syncthreads();
  if (s_full != 0u) {
    __syncthreads();                     // read by all before the counts are used again
    return false;
  }
  uint32_t ends = 0u, ends_before = 0u, first = incl - mine;
#pragma unroll
  for (int w = 0; w < kBucketWaves; ++w) {
    const uint32_t e = s_ends[w], f = s_sum[w];
    ends_before += w < wave ? e : 0u;
    ends += w < n_waves ? e : 0u;
    first += w < wave ? f : 0u;
  }
  first += ends & 0xFFFFu;
  const uint32_t inner_end = (uint32_t)n - (ends >> 16);
  *own = make_uint4(first, first + c.x, first + c.x + c.y, first + c.x + c.y + c.z);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if (inner[j]) pair[count[bucket[j]] + arrived[j]] = ((uint64_t)key[j] << 32) | idx[j];
  __syncthreads();
  uint32_t place[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    place[j] = arrived[j] + (key[j] == low ? ends_before & 0xFFFFu : inner_end + (ends_before >> 16));
    if (inner[j]) {
      const uint64_t self = ((uint64_t)key[j] << 32) | idx[j];
      const uint32_t begin = count[bucket[j]];
      const uint32_t end = (int)bucket[j] < last ? count[bucket[j] + 1] : inner_end;
      place[j] = begin;
      if (end - begin > 1u)
        for (uint32_t u = begin; u < end; ++u) place[j] += pair[u] < self ? 1u : 0u;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if ((int)idx[j] < n) pair[place[j]] = ((uint64_t)key[j] << 32) | idx[j];
  __syncthreads();
  return true;
}

}  // namespace maestro
