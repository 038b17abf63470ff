// radix.h -- radix selection of a rank among keys counted by many workgroups:
// digit views, LDS histograms of a digit, the last workgroup of a share of a
// launch, and its decision of the digit (device code shared by the selection of
// whole gradients and of long rows). Internal to libscadles.
#pragma once

#include "scadles_internal.h"

namespace scadles {

// ---- radix-selection digit view ------------------------------------------------------------
struct SelView {
  uint32_t lo, hi, shift, width, prefix;
};

// Width of the pending digit: the remainder bits first and 11-bit digits after,
// the fewest passes with the smallest histogram in the first one, which sees
// the most keys and flushes the most bins.
__device__ inline uint32_t digit_width(uint32_t bits)
{
  const uint32_t r = bits % (uint32_t)kDigitBits;
  return r ? r : (uint32_t)kDigitBits;
}

__device__ inline SelView view_of(const Sel& s)
{
  SelView v;
  v.lo = s.lo;
  v.hi = s.hi;
  v.width = digit_width(s.bits);
  v.shift = s.bits - v.width;
  v.prefix = s.prefix;
  return v;
}

// A selection of the key of descending rank `rank` among those in [lo, hi).
__device__ inline Sel first_sel(uint32_t lo, uint32_t hi, uint64_t rank)
{
  Sel s;
  __builtin_memset(&s, 0, sizeof(s));
  s.active = 1;
  s.lo = lo;
  s.hi = hi;
  s.rank = rank;
  const uint32_t b = bitlen32(hi - lo - 1u);
  s.bits = b ? b : 1u;
  return s;
}

// Whether the pending digit d of a key is counted: the key is in the band and
// matches the digits decided so far. kAll: the band holds every key.
template <bool kAll>
__device__ inline bool digit_of(const SelView& v, uint32_t key, uint32_t& d)
{
  const uint32_t o = kAll ? key : key - v.lo;
  d = (o >> v.shift) & ((1u << v.width) - 1u);
  return (kAll || ((key >= v.lo) & (key < v.hi))) & ((o >> (v.shift + v.width)) == v.prefix);
}

// Counts the pending digit of every lane's key, where there is one, in an LDS
// histogram. Lanes with the first such lane's digit are counted by one
// addition: equal keys -- zeros, ties -- would otherwise queue on one bin.
template <bool kAll>
__device__ inline void count_digit(const SelView& v, uint32_t key, bool valid, uint32_t* h)
{
  uint32_t d;
  const bool in = valid & digit_of<kAll>(v, key, d);
  const uint64_t m = ballot(in);
  const uint32_t lead = m ? (uint32_t)__builtin_ctzll(m) : 0u;
  const bool same = in & (d == (uint32_t)__builtin_amdgcn_readlane(d, lead));
  const uint32_t n = (uint32_t)__builtin_popcountll(ballot(same));
  const bool first = lane_id() == lead;
  if (in & (!same | first)) atomicAdd(&h[d], first ? n : 1u);
}

// The same for N keys per lane, valid where their bit is set. The lanes' first
// keys tell whether equal ones are worth looking for (kTied lanes with one
// digit): where they are not, one addition per key costs less than the ballots
// (exact path, 16 x 25.6 M of continuous values: 3.25 ms per step with the ballots
// always, 2.74 so).
// kAll: the band holds every key.
constexpr uint32_t kTied = 24;
template <bool kAll, int N>
__device__ inline void count_digits(const SelView& v, const uint32_t (&key)[N], uint32_t valid, uint32_t* h)
{
  uint32_t d;
  const bool in = (valid & 1u) & digit_of<kAll>(v, key[0], d);
  const uint64_t m = ballot(in);
  const uint32_t lead = m ? (uint32_t)__builtin_ctzll(m) : 0u;
  const uint64_t same = ballot(in & (d == (uint32_t)__builtin_amdgcn_readlane(d, lead)));
  if (__builtin_popcountll(same) >= (int)kTied) {
#pragma unroll
    for (int i = 0; i < N; ++i) count_digit<kAll>(v, key[i], (valid >> i) & 1u, h);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (((valid >> i) & 1u) & digit_of<kAll>(v, key[i], d)) atomicAdd(&h[d], 1u);
  }
}

__device__ inline void flush_hist(const uint32_t* h, uint32_t* g, int nb)
{
  for (int b = threadIdx.x; b < nb; b += kBlock) {
    uint32_t v = h[b];
    if (v) atomicAdd(g + b, v);
  }
}

// The calling wave's number in its workgroup, known to be uniform.
__device__ inline uint32_t wave_id() { return (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// ---- last workgroup of a device's share of a launch --------------------------------------------
// Every workgroup, once its results are out, adds the `done` units of the
// device's work it did to the device's counter (cleared by the preparation);
// the one that brings it to `all` is the last and returns true in all of its
// threads. It may read what the others produced, provided that they made it
// with device-scope operations (atomicAdd, put) and that it reads with get:
// those pass the caches that are private to an XCD, so that a wait for their
// completion before the counter is all the ordering that is needed -- no fence
// that writes back or drops an L2. No workgroup waits for another.
template <class T>
__device__ inline void put(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class T>
__device__ inline T get(T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ inline bool block_is_last(uint32_t* counter, uint32_t done, uint32_t all)
{
  __shared__ uint32_t s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores and atomics have completed
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(counter, done) + done == all ? 1u : 0u;
  __syncthreads();
  const bool last = s_last != 0u;
  __syncthreads();
  return last;
}

// ---- block-wide rank selection over a histogram -----------------------------------------------
// Among nb bins h(0) .. (nb a multiple of NT) holding counts of keys by digit, finds the
// bin of the key of 1-based descending rank `rank` (the largest digit is the
// top bin) and the number of keys in the bins above it. Every thread returns
// the same result; false when rank exceeds the total.
// The histogram must be complete (a barrier before the call); s_w holds
// NT / 64 + 3 words of LDS.
template <int NT, class Bin>
__device__ inline bool block_find(Bin h, int nb, uint64_t rank, uint32_t* s_w, uint32_t& bin, uint64_t& above)
{
  constexpr int kW = NT / 64;
  const int per = nb / NT;
  const uint32_t tid = threadIdx.x, w = tid >> 6;
  const int b_hi = nb - (int)tid * per;               // this thread's bins [b_hi - per, b_hi), top first
  uint32_t sum = 0;
  for (int i = 0; i < per; ++i) sum += h(b_hi - 1 - i);
  const uint32_t incl = wave_incl_scan(sum);
  if (lane_id() == 63) s_w[w] = incl;
  if (tid == 0) s_w[kW + 2] = 0u;
  __syncthreads();
  uint32_t excl = incl - sum;                         // counts of elements: below 2^32
  for (uint32_t i = 0; i < w; ++i) excl += s_w[i];
  if (excl < rank && rank <= (uint64_t)excl + sum) {
    uint32_t cum = excl;
    for (int i = 0; i < per; ++i) {
      const uint32_t v = h(b_hi - 1 - i);
      if ((uint64_t)cum + v >= rank) {
        s_w[kW] = (uint32_t)(b_hi - 1 - i);
        s_w[kW + 1] = cum;
        s_w[kW + 2] = 1u;
        break;
      }
      cum += v;
    }
  }
  __syncthreads();
  const bool ok = s_w[kW + 2] != 0u;
  bin = ok ? s_w[kW] : 0u;
  above = ok ? s_w[kW + 1] : 0u;
  __syncthreads();
  return ok;
}

// A complete histogram of N bins (device-scope sums of every workgroup) into LDS,
// bin b at h[at(b)], and cleared for the next pass.
template <int N, class At>
__device__ inline void take_hist(uint32_t* g, uint32_t* h, At at)
{
  constexpr int kPer = N / kBlock, kOnce = kPer < 16 ? kPer : 16;
  for (int i0 = 0; i0 < kPer; i0 += kOnce) {
    uint32_t v[kOnce];
#pragma unroll
    for (int i = 0; i < kOnce; ++i) v[i] = get(g + (i0 + i) * kBlock + threadIdx.x);
#pragma unroll
    for (int i = 0; i < kOnce; ++i) {
      const uint32_t b = (i0 + i) * kBlock + threadIdx.x;
      h[at(b)] = v[i];
      g[b] = 0u;
    }
  }
}

// Decides the pending digit of `sel` from its complete histogram g (device-scope
// sums of every workgroup), which is cleared for the next pass. Called by all
// threads of a workgroup, the same result in every thread. h: kBins words of
// LDS, s_w: kWaves + 3. Returns false when the rank exceeds the keys counted.
__device__ inline bool decide_digit(Sel& sel, uint32_t* g, uint32_t* h, uint32_t* s_w)
{
  take_hist<kBins>(g, h, [](uint32_t b) { return b; });
  __syncthreads();
  const uint32_t w = digit_width(sel.bits);
  const int nb = (1 << w) > kBlock ? 1 << w : kBlock;     // bins past the digit's are empty
  uint32_t bin;
  uint64_t above;
  if (!block_find<kBlock>([&](int b) { return h[b]; }, nb, sel.rank, s_w, bin, above)) {
    sel.active = 0;
    sel.found = 0;
    return false;
  }
  sel.rank -= above;
  sel.above += above;
  sel.prefix = (sel.prefix << w) | bin;
  sel.bits -= w;
  if (sel.bits == 0) {
    sel.active = 0;
    sel.found = 1;
    sel.result = sel.lo + sel.prefix;
  }
  return true;
}

}  // namespace scadles
