// select.hip -- Top-k selection kernels for gfx950.
//
// Top-k sparsification (§III-C, §IV "High communication cost" of ScaDLES,
// arXiv 2301.08897) keeps, per device, the k entries of largest |g| (ties to
// the lower index) in ascending index order. Magnitudes are ranked as the
// 31-bit integer key bits(g) & 0x7FFFFFFF, whose order is that of |g| for
// finite values, so every decision below is exact integer work.
//
// Fast path (one read of every gradient, a second one of its hot tiles):
//   1. bracket   : a histogram of a systematic sample (256-element chunks at a
//                  fixed stride), at two ranks around k * (sample/n), gives keys
//                  t_lo <= (k-th largest key) < t_hi with high probability;
//   2. main pass : every gradient is read once; each tile stages its keys >=
//                  t_lo (candidates) and those of them below t_hi (the selection
//                  interval) in its slot in index order; sum g^2 is fused in. A
//                  tile with more candidates than its slot holds is hot: only
//                  its counts are kept, and its interval keys in a list of the
//                  device;
//   3. threshold : the exact k-th largest key is radix-selected on the interval
//                  keys, which the first pass gathers from the slots into a list;
//   4. output    : per tile, the kept entries -- keys above the threshold plus
//                  the lowest-indexed `need` keys equal to it -- are counted,
//                  scanned and written in index order: from the slots, or for
//                  hot tiles from the gradient.
// If the bracket missed (fewer than k candidates) or the interval keys overflow
// their list, the device falls back to the exact path: a radix select over all
// of its data, after which all of its tiles are treated as hot ones.
//
// Small per-device steps (a digit's decision, the tiles' offsets, the adaptive
// decision) are done by the last workgroup of the launch whose results they
// need, not by a launch of their own: see block_is_last.
#include "frame.h"
#include "radix.h"

namespace scadles {

constexpr uint32_t kNoDevice = 0xFFFFFFFFu;

// Threshold and ties kept.
__device__ inline bool threshold_of(const DevState& s, uint32_t& thr, uint32_t& need)
{
  const Sel& sel = s.sel;
  if (!sel.found) {
    thr = kKeyInf;
    need = 0;
    return false;
  }
  thr = sel.result;
  need = (uint32_t)sel.rank;
  return true;
}

// ---- 0. per-call preparation -----------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_prep(Ctx c, PrepArgs a)
{
  const uint32_t K = c.K;
  if (blockIdx.x == 0 && threadIdx.x < K) {
    const uint32_t j = threadIdx.x;
    uint64_t off = 0;
    for (uint32_t i = 0; i < j; ++i) off += (uint64_t)a.seg[i] * c.nseg + a.cap[i];
    DevDesc d;
    d.grad = a.grad[j];
    d.idx_out = a.idx[j];
    d.val_out = a.val[j];
    d.band_off = off;
    d.k = a.k[j];
    d.seg_cap = a.seg[j];
    d.list_cap = a.cap[j];
    d.mode = a.mode[j];
    d.r_lo = a.r_lo[j];
    d.r_hi = a.r_hi[j];
    d.shift = (uint32_t)((reinterpret_cast<uintptr_t>(a.grad[j]) >> 2) & 3u);
    c.desc[j] = d;
    DevState s;
    __builtin_memset(&s, 0, sizeof(s));
    s.t_lo = s.t_hi = kKeyInf;
    s.thr = kKeyInf;
    c.st[j] = s;
  }
  if (blockIdx.x == 0)
    for (uint32_t i = threadIdx.x; i < K * kSegs; i += kBlock) c.list_cnt[i] = 0ull;
  const uint64_t nh = (uint64_t)K * kSampleBins;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < nh; i += stride) c.hist[i] = 0u;
}

// ---- 1. bracket from the systematic sample ---------------------------------------------------
// A histogram of the sample keys' top kBits bits. The bracket only has to be
// conservative (t_lo at or below the sample key of rank r_lo, t_hi above the one
// of rank r_hi), so a rank's bin [B, B + width) gives t_lo = B or t_hi = B +
// width. Small selections stop after one pass of kSampleBits bits (bins of 3% of
// the magnitude); for large ones, whose interval keys cost more than a
// launch, a pass of kDigitBits bits is followed by one that tells apart
// kRefineBits more within the two bins. The device's last workgroup finds the
// bins and, in the last pass, stores the bracket for the main pass.
constexpr int kRefineBits = 11;
constexpr uint32_t kRefineBins = 1u << kRefineBits;

// Sample elements e0 .. of the workgroup: four of every round per thread
// (0 past the sample's end e1).
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));    // four floats at any 4-byte address
constexpr int kSampleRounds = kSBlk / kRound;

__device__ inline void load_sample(const Ctx& c, const DevDesc& d, uint64_t e0, uint64_t e1, f4 (&x)[kSampleRounds])
{
#pragma unroll
  for (int r = 0; r < kSampleRounds; ++r) {
    const uint64_t e = e0 + (uint64_t)r * kRound + threadIdx.x * 4;
    const uint64_t chunk = e / kSChunk, within = e % kSChunk;
    const uint64_t i = chunk * c.s_stride + within;     // real position of sample element e
    if (e + 4 <= e1) x[r] = *(const GLOBAL f4u*)(gptr(d.grad) + i);
    else
      for (int q = 0; q < 4; ++q) x[r][q] = (e + q < e1) ? gptr(d.grad)[i + q] : 0.f;
  }
}

// The bracket from the bins of the two ranks (the upper rank 0: no upper bound).
__device__ inline void store_bracket(DevState& st, const DevDesc& d, uint32_t lo, uint32_t hi, int shift, bool ok)
{
  // t_lo = 0: every key a candidate (a gradient of mostly zeros), more than the
  // lists can hold, so the exact path takes the device from the start
  if (!ok || lo == 0u) {
    st.err |= kErrBracket;
    return;                                       // t_lo = t_hi = kKeyInf from the preparation
  }
  st.t_lo = lo << shift;
  st.t_hi = d.r_hi ? (hi + 1u) << shift : kKeyInf;
}

template <int kBits>
__global__ __launch_bounds__(kBlock) void k_bracket(Ctx c, uint32_t refine)
{
  constexpr uint32_t kN = 1u << kBits;
  constexpr int kShift = 31 - kBits;
  __shared__ uint32_t h[kN + kN / 32];
  __shared__ uint32_t s_w[kWaves + 3];
  const uint32_t j = blockIdx.y, tid = threadIdx.x;
  const DevDesc& d = c.desc[j];
  if (d.mode != kModeFast) return;
  const uint64_t e0 = (uint64_t)blockIdx.x * kSBlk;      // below s_n: the grid is ceil(s_n / kSBlk)
  const uint64_t e1 = (e0 + kSBlk < c.s_n) ? e0 + kSBlk : c.s_n;
  f4 x[kSampleRounds];
  load_sample(c, d, e0, e1, x);
  auto at = [](uint32_t b) { return b + (b >> 5); };     // spreads a thread's run of bins over the banks
  for (uint32_t b = tid; b < kN + kN / 32; b += kBlock) h[b] = 0u;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSampleRounds; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (e0 + (uint64_t)r * kRound + tid * 4 + q < e1) atomicAdd(&h[at(key_of(x[r][q]) >> kShift)], 1u);
  __syncthreads();
  uint32_t* g = c.hist + (uint64_t)j * kSampleBins;
  for (uint32_t b = tid; b < kN; b += kBlock) {
    const uint32_t v = h[at(b)];
    if (v) atomicAdd(g + b, v);
  }
  DevState& st = c.st[j];
  if (!block_is_last(&st.ticket[kTicketSample], 1u, gridDim.x)) return;
  take_hist<kN>(g, h, at);
  __syncthreads();
  auto bin_of = [&](int b) { return h[at((uint32_t)b)]; };
  uint32_t lo, hi = 0;
  uint64_t above_lo, above_hi = 0;
  bool ok = block_find<kBlock>(bin_of, kN, d.r_lo, s_w, lo, above_lo);
  if (d.r_hi) ok = block_find<kBlock>(bin_of, kN, d.r_hi, s_w, hi, above_hi) && ok;
  if (tid != 0) return;
  if (!refine) {
    store_bracket(st, d, lo, hi, kShift, ok);
    return;
  }
  if (!ok) st.err |= kErrBracket;
  st.bin_lo = lo;
  st.bin_hi = hi;
  st.rank_lo = d.r_lo - (uint32_t)above_lo;
  st.rank_hi = d.r_hi - (uint32_t)above_hi;
}

// The second pass: kRefineBits more bits of the sample keys in the two ranks' bins.
__global__ __launch_bounds__(kBlock) void k_refine(Ctx c)
{
  constexpr int kShift = 31 - kDigitBits - kRefineBits;
  __shared__ uint32_t h[2 * kRefineBins];
  __shared__ uint32_t s_w[kWaves + 3];
  const uint32_t j = blockIdx.y, tid = threadIdx.x;
  const DevDesc& d = c.desc[j];
  DevState& st = c.st[j];
  if (d.mode != kModeFast || (st.err & kErrBracket)) return;
  const uint64_t e0 = (uint64_t)blockIdx.x * kSBlk;
  const uint64_t e1 = (e0 + kSBlk < c.s_n) ? e0 + kSBlk : c.s_n;
  f4 x[kSampleRounds];
  load_sample(c, d, e0, e1, x);
  const uint32_t lo = st.bin_lo, hi = st.bin_hi;
  for (uint32_t b = tid; b < 2 * kRefineBins; b += kBlock) h[b] = 0u;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSampleRounds; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (e0 + (uint64_t)r * kRound + tid * 4 + q >= e1) break;
      const uint32_t key = key_of(x[r][q]) >> kShift, bin = key >> kRefineBits;
      if (bin == lo) atomicAdd(&h[key & (kRefineBins - 1)], 1u);
      if (bin == hi) atomicAdd(&h[kRefineBins + (key & (kRefineBins - 1))], 1u);
    }
  __syncthreads();
  uint32_t* g = c.hist + (uint64_t)j * kSampleBins;
  flush_hist(h, g, 2 * kRefineBins);
  if (!block_is_last(&st.ticket[kTicketRefine], 1u, gridDim.x)) return;
  take_hist<2 * kRefineBins>(g, h, [](uint32_t b) { return b; });
  __syncthreads();
  uint32_t sub_lo, sub_hi = 0;
  uint64_t above;
  bool ok = block_find<kBlock>([&](int b) { return h[b]; }, kRefineBins, st.rank_lo, s_w, sub_lo, above);
  if (d.r_hi) ok = block_find<kBlock>([&](int b) { return h[kRefineBins + b]; }, kRefineBins, st.rank_hi, s_w, sub_hi, above) && ok;
  if (tid == 0)
    store_bracket(st, d, (lo << kRefineBits) | sub_lo, (hi << kRefineBits) | sub_hi, kShift, ok);
}

// ---- 2. main pass: one read of every gradient ------------------------------------------------
// No workgroup waits on another: every tile writes its candidates (keys >=
// t_lo) in index order to its own slot with the selection-interval keys among
// them; a hot tile appends the latter to one of the device's list segments
// (in turn, so that the appends do not queue on one address). Only hot tiles
// use atomics: one per tile cost this pass 2% (30 x 143.7M: 2.63 -> 2.68 ms).

// One round of phase 1 for one wave: sum of squares, counts of candidates
// (key >= tlo) and sure keys (key >= thi), and the round's candidates staged in
// LDS in index order (lane, then component) after the `wc` already staged, the
// keys of those below thi (the selection interval) likewise in s_b.
// kEdge: the round may hold pads (pattern 0xFFFFFFFF), so keys are compared as
// rank keys (key + 1, pads 0) and fmax drops the pads' NaN from the squares.
// Counts are wave totals from ballots (scalar popcounts).
// A staged candidate: its index in the low word, its value's bits in the high word.
// A tile's slot region (kSlotWords words, consecutive tiles back to back):
// words 0 .. band - 1 hold the keys of the candidates below t_hi (the
// selection interval), word band + e candidate e's value bits, and the 16-bit
// word (2 * kSlotWords - 1 - e) candidate e's offset in the tile (index = tile
// * kTile - shift + offset). The keys start at a fixed place, so their readers
// load them before the counts arrive. Both ends are written as whole 16-byte
// chunks; a tile whose two parts would meet is hot.
__device__ inline uint32_t slot_off16_at(uint32_t e) { return 2u * kSlotWords - 1u - e; }

__device__ inline uint64_t pack_cand(uint32_t i, float v) { return (uint64_t)i | ((uint64_t)__float_as_uint(v) << 32); }

template <bool kEdge>
__device__ inline void main_stage(const f4& x, uint32_t i0, uint32_t tlo, uint32_t thi, double (&e2)[2], uint32_t& wc,
                                  uint32_t& ws, uint64_t* s_c, uint32_t* s_b)
{
  uint64_t b[4], bb[4];
  bool f[4], fb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double xd = (double)x[q];
    if (kEdge) e2[q & 1] += __builtin_fmax(xd * xd, 0.0);
    else e2[q & 1] = __builtin_fma(xd, xd, e2[q & 1]);
    const uint32_t key = kEdge ? rank_key(x[q]) : key_of(x[q]);
    const uint32_t lo = kEdge ? tlo + 1u : tlo, hi = kEdge ? thi + 1u : thi;
    f[q] = key >= lo;
    fb[q] = f[q] && key < hi;
    b[q] = ballot(f[q]);
    bb[q] = ballot(fb[q]);
  }
  const uint64_t any = b[0] | b[1] | b[2] | b[3];
  if (any == 0ull) return;
  const uint32_t nb = (uint32_t)(__builtin_popcountll(bb[0]) + __builtin_popcountll(bb[1]) +
                                 __builtin_popcountll(bb[2]) + __builtin_popcountll(bb[3]));
  const uint32_t nc = (uint32_t)(__builtin_popcountll(b[0]) + __builtin_popcountll(b[1]) +
                                 __builtin_popcountll(b[2]) + __builtin_popcountll(b[3]));
  // wb, the wave's staged selection keys so far, is wc - ws
  uint32_t pos = wc + mbcnt(b[0]) + mbcnt(b[1]) + mbcnt(b[2]) + mbcnt(b[3]);
  uint32_t bpos = (wc - ws) + mbcnt(bb[0]) + mbcnt(bb[1]) + mbcnt(bb[2]) + mbcnt(bb[3]);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (f[q]) {
      if (pos < (uint32_t)kWaveCap) s_c[pos] = pack_cand(i0 + q, x[q]);
      ++pos;
    }
    if (fb[q]) {
      if (bpos < (uint32_t)kWaveCap) s_b[bpos] = key_of(x[q]);
      ++bpos;
    }
  }
  wc += nc;
  ws += nc - nb;
}

// Each workgroup reads one tile of kTile gradient elements (workgroup b: device
// b / tpd, tile b % tpd). Wave w owns elements [w*4096, (w+1)*4096) of the tile
// and stages its candidates in LDS; the tile's slot is written at the end (the
// only barrier). The gradient pointers come as kernel arguments so that the
// tile's loads issue before anything is read from the workspace.
__global__ __launch_bounds__(kBlock) void k_main(Ctx c, GradArgs ga)
{
  __shared__ uint64_t s_c[kWaves][kWaveCap];
  __shared__ uint32_t s_b[kWaves][kWaveCap];
  const uint32_t l = lane_id(), w = threadIdx.x >> 6;
  const uint32_t jr = blockIdx.x / c.tpd, tile = blockIdx.x - jr * c.tpd;
  const uint32_t j = c.j0 + jr;
  const float* grad = ga.grad[j];
  const uint64_t shift = (reinterpret_cast<uintptr_t>(grad) >> 2) & 3u;
  const uint64_t vbase = (uint64_t)tile * kTile;      // virtual position of the tile
  const Row row{gptr(grad), shift, c.n};
  // Interior tiles hold only real elements: plain aligned loads kept in
  // registers. The (at most two) edge tiles of a device reload per round.
  const bool full = vbase >= row.shift && vbase + kTile <= row.shift + row.n;
  const uint32_t wv0 = (uint32_t)(w * (kTileRounds * 256) + l * 4);   // this lane's first element in the tile
  // real index of virtual position vbase + wv0 (may wrap for leading pads; never written)
  const uint32_t i_base = (uint32_t)(vbase + wv0 - row.shift);

  double e2[2] = {0.0, 0.0};
  uint32_t wc = 0, ws = 0;
  if (full) {
    const GLOBAL float* p = row.p + (vbase - row.shift) + wv0;
    f4 v[kTileRounds];
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) v[r] = ld_stream4(p + r * 256);
    const uint32_t tlo = c.st[j].t_lo, thi = c.st[j].t_hi;
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
      main_stage<false>(v[r], i_base + r * 256, tlo, thi, e2, wc, ws, s_c[w], s_b[w]);
      __builtin_amdgcn_sched_barrier(0);    // keep rounds apart: bounds the live ballot masks
    }
  } else {
    const uint32_t tlo = c.st[j].t_lo, thi = c.st[j].t_hi;
    for (int r = 0; r < kTileRounds; ++r)
      main_stage<true>(load4(row, vbase + wv0 + r * 256, false), i_base + r * 256, tlo, thi, e2, wc, ws, s_c[w],
                     s_b[w]);
  }
  // The tile's slot: the waves' staged candidates one after the other (index
  // order); its counts and sum of squares. A hot tile (a wave chunk over
  // kWaveCap candidates, or more than the region holds) writes no candidates
  // but goes on the device's list of hot tiles.
  __shared__ uint32_t s_cnt[kWaves];
  __shared__ double s_e[kWaves];
  __shared__ uint32_t s_pos;
  const double es = wave_sum_f64(e2[0] + e2[1]);
  if (l == 0) {
    s_cnt[w] = wc | (ws << 16);
    s_e[w] = es;
  }
  __syncthreads();
  // cb[i] / kb[i]: candidates / selection keys of the waves before wave i
  uint32_t cb[kWaves + 1], kb[kWaves + 1];
  bool hot = false;
  cb[0] = kb[0] = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    const uint32_t v = s_cnt[i], wci = v & 0xFFFFu;
    cb[i + 1] = cb[i] + wci;
    kb[i + 1] = kb[i] + wci - (v >> 16);
    hot |= wci > (uint32_t)kWaveCap;
  }
  const uint32_t cand = cb[kWaves], band = kb[kWaves], sure = cand - band;
  const uint32_t na = (cand + band + 3u) / 4u, nbk = ((cand + 1u) / 2u + 3u) / 4u;   // 16-byte chunks of both ends
  hot |= 4u * (na + nbk) > (uint32_t)kSlotWords;
  const uint64_t slot = (uint64_t)j * c.nslot + tile;
  const uint32_t seg = tile % c.nseg;
  if (threadIdx.x == 0) {
    c.slot_cnt[slot] = cand | (hot ? 0x8000u : 0u) | (sure << 16);
    c.epart[slot] = (s_e[0] + s_e[1]) + (s_e[2] + s_e[3]);
  }
  const uint32_t* b32 = &s_b[0][0];
  if (!hot) {
    // The whole workgroup writes both ends, 16 bytes per thread (nontemporal:
    // the slots are read only after the whole pass).
    GLOBAL uint32_t* reg = gptr(c.slot) + slot * kSlotWords;
    const uint32_t* c32 = reinterpret_cast<const uint32_t*>(&s_c[0][0]);
    auto cand_word = [&](uint32_t e, uint32_t half) -> uint32_t {    // half 0: index, 1: value bits
      const uint32_t wi = (uint32_t)(e >= cb[1]) + (uint32_t)(e >= cb[2]) + (uint32_t)(e >= cb[3]);
      const uint32_t base = wi == 0 ? cb[0] : (wi == 1 ? cb[1] : (wi == 2 ? cb[2] : cb[3]));
      return c32[wi * (2 * kWaveCap) + 2u * (e - base) + half];
    };
    auto low_word = [&](uint32_t q) -> uint32_t {
      if (q < band) {
        const uint32_t wi = (uint32_t)(q >= kb[1]) + (uint32_t)(q >= kb[2]) + (uint32_t)(q >= kb[3]);
        const uint32_t base = wi == 0 ? kb[0] : (wi == 1 ? kb[1] : (wi == 2 ? kb[2] : kb[3]));
        return b32[wi * kWaveCap + (q - base)];
      }
      const uint32_t e = q - band;
      return e < cand ? cand_word(e, 1u) : 0u;
    };
    const uint32_t ibase = (uint32_t)(vbase - row.shift);   // index of tile position 0 (mod 2^32)
    auto off16 = [&](uint32_t e) -> uint32_t { return e < cand ? (cand_word(e, 0u) - ibase) & 0xFFFFu : 0u; };
    for (uint32_t t = threadIdx.x; t < na + nbk; t += kBlock) {
      u4 v;
      uint32_t p0;
      if (t < na) {
        p0 = 4u * t;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = low_word(p0 + i);
      } else {
        p0 = kSlotWords - 4u * nbk + 4u * (t - na);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t e_lo = slot_off16_at(2u * (p0 + i));     // candidate in the word's low half
          v[i] = off16(e_lo) | (off16(e_lo - 1u) << 16);
        }
      }
      __builtin_nontemporal_store(v, reinterpret_cast<GLOBAL u4*>(reg + p0));
    }
    return;
  }
  if (threadIdx.x == 0) {
    c.hot_list[(uint64_t)j * c.nslot + atomicAdd(&c.st[j].nhot, 1u)] = tile;
    // the segment's keys and the hot tiles' keys above the interval, in one word
    s_pos = (uint32_t)atomicAdd(&c.list_cnt[(uint64_t)j * kSegs + seg],
                                (unsigned long long)band | ((unsigned long long)sure << 32));
    c.slot_boff[slot] = s_pos;
  }
  if (!band) return;
  // The selection-interval keys, appended in index order. A tile past its
  // segment's end writes nothing (the segment's count tells: the device falls
  // back). A chunk with more keys than were staged is read again.
  __syncthreads();
  const uint32_t pos = s_pos, scap = c.desc[j].seg_cap;
  if (pos > scap || scap - pos < band) return;
  GLOBAL uint32_t* dst = gptr(c.band) + c.desc[j].band_off + (uint64_t)seg * scap + pos;
  for (uint32_t q = threadIdx.x; q < band; q += kBlock) {
    const uint32_t wi = (uint32_t)(q >= kb[1]) + (uint32_t)(q >= kb[2]) + (uint32_t)(q >= kb[3]);
    const uint32_t base = wi == 0 ? kb[0] : (wi == 1 ? kb[1] : (wi == 2 ? kb[2] : kb[3]));
    if (q - base < (uint32_t)kWaveCap) dst[q] = b32[wi * kWaveCap + (q - base)];
  }
  if (wc - ws > (uint32_t)kWaveCap) {
    const uint32_t lo = c.st[j].t_lo + 1u, hi = c.st[j].t_hi + 1u;     // rank keys
    uint32_t run = w == 0 ? kb[0] : (w == 1 ? kb[1] : (w == 2 ? kb[2] : kb[3]));
#pragma unroll 4
    for (int r = 0; r < kTileRounds; ++r) {
      const f4 x = load4(row, vbase + wv0 + (uint64_t)r * 256, false);
      bool fb[4];
      uint64_t bb[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t kq = rank_key(x[q]);
        fb[q] = kq >= lo && kq < hi;
        bb[q] = ballot(fb[q]);
      }
      uint32_t at = run + mbcnt(bb[0]) + mbcnt(bb[1]) + mbcnt(bb[2]) + mbcnt(bb[3]);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (fb[q]) dst[at++] = key_of(x[q]);
      run += (uint32_t)(__builtin_popcountll(bb[0]) + __builtin_popcountll(bb[1]) + __builtin_popcountll(bb[2]) +
                        __builtin_popcountll(bb[3]));
    }
  }
}

__device__ inline uint64_t wave_incl_scan_u64(uint64_t v)
{
  const uint32_t l = lane_id();
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint64_t t = __shfl_up(v, d, 64);
    if (l >= (uint32_t)d) v += t;
  }
  return v;
}

// ---- 3. threshold: histogram passes over the band list (fast devices) or the data (exact ones) ----
// A device takes the exact path when that is asked for or its bracket missed
// (known before the first pass), or when its counts, complete after the first
// pass, show that the selection interval does not hold the k-th largest key or
// the lists not all keys of the interval.
constexpr uint32_t kExactKnown = 1u, kExactFound = 2u;      // DevState::fallback

__device__ inline bool known_exact(const Ctx& c, const DevDesc& d, uint32_t err)
{
  // only the bracket's error bit: the threshold passes may set theirs meanwhile
  return d.mode != kModeFast || c.force_fallback || (err & kErrBracket);
}

// Devices of the launch on the exact path, one bit per device of the group, and
// those of them found after the first pass, which are one pass behind.
__device__ inline uint64_t exact_devices(const Ctx& c, uint32_t pass, uint64_t& behind)
{
  const uint32_t l = lane_id();
  uint32_t fb = 0;
  if (l < c.jn) {
    const uint32_t j = c.j0 + l;
    if (pass == 0) fb = known_exact(c, c.desc[j], c.st[j].err) ? kExactKnown : 0u;
    else fb = c.st[j].fallback;
  }
  behind = ballot(fb == kExactFound);
  return ballot(fb != 0u);
}

// Place of the n-th set bit (n from 0).
__device__ inline uint32_t nth_bit(uint64_t m, uint32_t n)
{
  for (uint32_t i = 0; i < n; ++i) m &= m - 1;
  return (uint32_t)__builtin_ctzll(m);
}

// Fast devices, first pass: `walk` workgroups per device take kBT staged tiles
// per wave: the first 64 keys of every tile are loaded at once, before the
// counts arrive, and all keys are also appended to the device's gathered list
// (one reservation per workgroup, which also counts the tiles' keys above the
// interval). The hot tiles' list, in later passes with
// the gathered one, is shared in chunks by `per_dev` workgroups per device. The
// last workgroup of a device decides the digit.
// Exact devices: the remaining workgroups take equal runs of their (device, block
// of c.fb_rounds rounds) items, device-major: a worker's items of one device share
// its histogram, and a run crosses few devices (grid-stride, every worker flushed and
// waited once per device: 8 x 11.2 M 173 us per pass, 72 so). The worker that completes a device's blocks decides.
constexpr uint32_t kHChunk = 8 * kBlock;

template <int kBT>
__device__ inline void walk_slots(const Ctx& c, uint32_t j, uint32_t b, const DevDesc& d, const SelView& sv, uint32_t* h)
{
  __shared__ uint32_t s_n[kWaves + 1], s_u[kWaves];
  const uint32_t l = lane_id(), w = wave_id();
  const uint32_t t0 = (b * kWaves + w) * kBT, last = c.nslot - 1;
  const uint64_t row = (uint64_t)j * c.nslot;
  const GLOBAL uint32_t* reg = gptr(c.slot);
  uint32_t kv[kBT];
#pragma unroll
  for (int i = 0; i < kBT; ++i) {
    const uint32_t ti = t0 + i < last ? t0 + i : last;
    kv[i] = reg[(row + ti) * kSlotWords + l];
  }
  const uint32_t v = l < (uint32_t)kBT && t0 + l < c.nslot ? c.slot_cnt[row + t0 + l] : 0x8000u;
  const uint32_t nb = v & 0x8000u ? 0u : (v & 0x7FFFu) - (v >> 16);
  const uint32_t incl = wave_incl_scan(nb), pre = incl - nb;
  const uint32_t su = wave_incl_scan(v & 0x8000u ? 0u : v >> 16);
  if (l == 63) {
    s_n[w] = incl;
    s_u[w] = su;
  }
  __syncthreads();
  const uint32_t all = (s_n[0] + s_n[1]) + (s_n[2] + s_n[3]);
  if (threadIdx.x == 0)
    s_n[kWaves] = (uint32_t)atomicAdd(&c.st[j].gathered,
                                      (unsigned long long)all | ((unsigned long long)((s_u[0] + s_u[1]) + (s_u[2] + s_u[3])) << 32));
#pragma unroll
  for (int i = 0; i < kBT; ++i) count_digit<false>(sv, kv[i], l < (uint32_t)__builtin_amdgcn_readlane(nb, i), h);
  __syncthreads();
  uint32_t base = s_n[kWaves];
  // keys past the list's end are only counted: the device takes the exact path
  const bool room = base <= d.list_cap && d.list_cap - base >= all;
  for (uint32_t i = 0; i < w; ++i) base += s_n[i];
  GLOBAL uint32_t* list = gptr(c.band) + d.band_off + (uint64_t)c.nseg * d.seg_cap + base;
#pragma unroll
  for (int i = 0; i < kBT; ++i) {
    const uint32_t n = __builtin_amdgcn_readlane(nb, i);
    GLOBAL uint32_t* dst = list + (uint32_t)__builtin_amdgcn_readlane(pre, i);
    if (room && l < n) dst[l] = kv[i];
    if (n > 64u) {
      const GLOBAL uint32_t* p = reg + (row + t0 + i) * kSlotWords;
      for (uint32_t e = 64; e < n; e += 256) {
        uint32_t x[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) x[m] = e + m * 64 + l < n ? p[e + m * 64 + l] : 0u;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const bool valid = e + m * 64 + l < n;
          if (room && valid) dst[e + m * 64 + l] = x[m];
          count_digit<false>(sv, x[m], valid, h);
        }
      }
    }
  }
}

template <int kBT>
__global__ __launch_bounds__(kBlock) void k_hist(Ctx c, uint32_t walk, uint32_t per_dev, uint32_t pass)
{
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t s_w[kWaves + 3];
  const uint32_t both = walk + per_dev, nfast = both * c.jn;
  if (blockIdx.x < nfast) {
    const uint32_t jr = blockIdx.x / both, wb = blockIdx.x - jr * both;
    const uint32_t j = c.j0 + jr;
    DevState& st = c.st[j];
    const DevDesc& d = c.desc[j];
    Sel sel;
    if (pass == 0) {
      if (known_exact(c, d, st.err)) return;
      sel = first_sel(st.t_lo, st.t_hi, 0);         // the rank follows from the counts
    } else {
      if (st.fallback) return;
      sel = st.sel;
    }
    if (!sel.active) return;
    // lane i: segment i's keys (lane kSegs: the gathered list's), and its
    // chunks with those of the segments before
    const uint32_t l = lane_id();
    const uint64_t lc = l < (uint32_t)kSegs ? (uint64_t)c.list_cnt[(uint64_t)j * kSegs + l] : 0ull;
    const bool over = ballot((uint32_t)lc > d.seg_cap) != 0ull;      // in the first pass only
    uint32_t cnt = over ? 0u : (uint32_t)lc;
    if (pass > 0 && l == (uint32_t)kSegs) cnt = (uint32_t)st.gathered;
    const uint32_t nch = (cnt + kHChunk - 1) / kHChunk;
    const uint32_t incl = wave_incl_scan(nch);
    const uint32_t items = __builtin_amdgcn_readlane(incl, 63);
    if (wb >= walk + items) return;
    for (int i = threadIdx.x; i < kBins; i += kBlock) h[i] = 0u;
    __syncthreads();
    const SelView sv = view_of(sel);
    if (wb < walk) {
      walk_slots<kBT>(c, j, wb, d, sv, h);
    } else {
      for (uint32_t it = wb - walk; it < items; it += per_dev) {
        const uint32_t seg = (uint32_t)__builtin_popcountll(ballot(incl <= it));
        const uint32_t n = __builtin_amdgcn_readlane(cnt, seg);
        const uint32_t e0 = (it - (uint32_t)__builtin_amdgcn_readlane(incl - nch, seg)) * kHChunk + threadIdx.x;
        const GLOBAL uint32_t* p =
            gptr(c.band) + d.band_off + (uint64_t)(seg < (uint32_t)kSegs ? seg : c.nseg) * d.seg_cap;
        uint32_t key[kHChunk / kBlock];
#pragma unroll
        for (int r = 0; r < (int)(kHChunk / kBlock); ++r) {
          const uint32_t e = e0 + r * kBlock;
          key[r] = e < n ? p[e] : 0u;
        }
        uint32_t valid = 0;
#pragma unroll
        for (int r = 0; r < (int)(kHChunk / kBlock); ++r) valid |= e0 + r * kBlock < n ? 1u << r : 0u;
        count_digits<false>(sv, key, valid, h);
      }
    }
    __syncthreads();
    uint32_t* g = c.hist + (uint64_t)j * kSampleBins;
    flush_hist(h, g, kBins);
    if (!block_is_last(&st.ticket[kTicketHist + pass], 1u, walk + (items < per_dev ? items : per_dev))) return;
    bool exact = false;
    if (pass == 0) {
      const uint64_t staged = get(&st.gathered), hot = wave_sum_u64(lc);   // both halves count elements: no carry
      const uint64_t band = (uint64_t)(uint32_t)staged + (uint32_t)hot, sure = (staged >> 32) + (hot >> 32);
      exact = over || (uint32_t)staged > d.list_cap || band + sure < d.k ||
              sure >= d.k;
      sel.rank = exact ? 1u : d.k - sure;
    }
    const bool ok = decide_digit(sel, g, h, s_w);       // clears the histogram in any case
    if (threadIdx.x == 0) {
      if (exact) st.fallback = kExactFound;
      else if (!ok) st.err |= kErrSelect;
      st.sel = sel;
    }
    return;
  }
  const uint32_t worker = blockIdx.x - nfast, G = gridDim.x - nfast;
  uint64_t behind;
  const uint64_t devs = exact_devices(c, pass, behind);
  if (!devs) return;
  const uint64_t items = (uint64_t)__builtin_popcountll(devs) * c.nfb;
  uint32_t cur = kNoDevice, done = 0, own = pass;
  Sel sel{};
  SelView sv{};
  Row row{};
  // the worker's share of the current device is complete
  auto close = [&]() {
    if (!done) return;
    __syncthreads();
    DevState& st = c.st[cur];
    uint32_t* g = c.hist + (uint64_t)cur * kSampleBins;
    flush_hist(h, g, kBins);
    if (block_is_last(&st.ticket[kTicketFull + own], done, c.nfb)) {
      const bool ok = decide_digit(sel, g, h, s_w);
      if (threadIdx.x == 0) {
        if (!ok) st.err |= kErrSelect;
        st.sel = sel;
        if (pass == 0) st.fallback = kExactKnown;
      }
    }
    __syncthreads();
    done = 0;
  };
  const uint64_t it1 = items * (worker + 1) / G;
  for (uint64_t it = items * worker / G; it < it1; ++it) {
    const uint32_t q = (uint32_t)(it / c.nfb), blk = (uint32_t)(it - (uint64_t)q * c.nfb);
    const uint32_t jr = nth_bit(devs, q), j = c.j0 + jr;
    if (j != cur) {
      close();
      cur = j;
      own = pass - (uint32_t)((behind >> jr) & 1ull);         // the device's pass
      sel = own == 0 ? first_sel(0u, kKeyInf, c.desc[j].k) : c.st[j].sel;
      if (sel.active) {
        for (int i = threadIdx.x; i < kBins; i += kBlock) h[i] = 0u;
        __syncthreads();
        sv = view_of(sel);
        row = Row{gptr(c.desc[j].grad), c.desc[j].shift, c.n};
      }
    }
    if (!sel.active) continue;
    const uint64_t vbase = (uint64_t)blk * c.fb_rounds * kRound;
    if (c.fb_rounds == kFbRounds && vbase >= row.shift && vbase + kFbRounds * kRound <= row.shift + row.n) {
      // only real elements: plain aligned loads and no checks. (Four rounds in flight:
      // eight take 93 registers instead of 79 and leave the launch fewer slots beside
      // other layers' main passes, three long layers of 8 x 50 M with ties 592 us against
      // 579; alone they give less than 1%.)
      const GLOBAL float* p = row.p + (vbase - row.shift) + threadIdx.x * 4;
#pragma unroll 1
      for (int r0 = 0; r0 < kFbRounds; r0 += 4) {
        f4 x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = ld_stream4(p + (r0 + r) * kRound);
        uint32_t key[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) key[e] = key_of(x[e / 4][e % 4]);
        count_digits<true>(sv, key, 0xFFFFu, h);
      }
      ++done;
      continue;
    }
    for (uint32_t r0 = 0; r0 < c.fb_rounds; r0 += 4) {
      f4 x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r0 + r < c.fb_rounds) x[r] = load4(row, vbase + (uint64_t)(r0 + r) * kRound + threadIdx.x * 4, true);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (r0 + r >= c.fb_rounds) break;
        const uint64_t v = vbase + (uint64_t)(r0 + r) * kRound + threadIdx.x * 4;
        uint32_t key[4], valid = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          key[e] = key_of(x[r][e]);
          valid |= in_row(row, v + e) ? 1u << e : 0u;
        }
        count_digits<true>(sv, key, valid, h);
      }
    }
    ++done;
  }
  close();
}

// ---- 4. kept counts per tile -----------------------------------------------------------------
// Kept: key > thr, or key == thr while fewer than `need` equal keys came before
// (index order); a kept entry goes to (keys above thr before it) + min(equal
// keys before it, need). The counts and the output below treat two kinds of
// tiles: staged ones (their candidates in the slot), several per wave, and hot
// ones.  All tiles of an
// exact device are hot.

// Calls tile(j, s) for every p-th hot tile s of the launch's devices j, in device
// order from the w-th on: the listed ones of fast devices (kFast), all tiles of
// exact ones (kExact).
template <bool kFast, bool kExact, class Tile>
__device__ inline void for_hot_tiles(const Ctx& c, uint32_t w, uint32_t p, Tile tile)
{
  const uint32_t l = lane_id();
  // lane l: device c.j0 + l's tiles, and those with the devices before
  uint32_t n = 0;
  bool fb = false;
  if (l < c.jn) {
    const DevState& s = c.st[c.j0 + l];
    fb = s.fallback != 0u;
    n = fb ? (kExact ? c.nslot : 0u) : (kFast ? s.nhot : 0u);
  }
  const uint64_t exact = ballot(fb);
  const uint32_t incl = wave_incl_scan(n);      // at most 64 x 2^18 tiles
  const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
  for (uint32_t it = w; it < total; it += p) {
    const uint32_t jr = (uint32_t)__builtin_popcountll(ballot(incl <= it));
    const uint32_t i = it - (uint32_t)__builtin_amdgcn_readlane(incl - n, jr);
    const uint32_t j = c.j0 + jr;
    tile(j, (exact >> jr) & 1ull ? i : c.hot_list[(uint64_t)j * c.nslot + i]);
  }
}

constexpr int kHotBatch = 4;      // rounds loaded at once

// Calls visit(x) for the rounds of the wave's chunk of tile s: lane l's four
// elements x of 256.
// Interior tiles hold only real elements: plain aligned loads; the (at most
// two) edge tiles of a device load round by round.
template <class Visit>
__device__ inline void walk_chunk(const Row& row, uint32_t s, Visit visit)
{
  const uint64_t vbase = (uint64_t)s * kTile, v0 = vbase + wave_id() * (kTileRounds * 256);
  const uint32_t l4 = 4u * lane_id();
  if (vbase >= row.shift && vbase + kTile <= row.shift + row.n) {
    const GLOBAL float* p = row.p + (v0 - row.shift);
    for (int r0 = 0; r0 < kTileRounds; r0 += kHotBatch) {
      f4 x[kHotBatch];
#pragma unroll
      for (int r = 0; r < kHotBatch; ++r) x[r] = ld_stream4(p + (r0 + r) * 256 + l4);
#pragma unroll
      for (int r = 0; r < kHotBatch; ++r) {
        visit(x[r]);
        __builtin_amdgcn_sched_barrier(0);    // keep rounds apart: bounds the live ballot masks
      }
    }
  } else {
    for (int r = 0; r < kTileRounds; ++r) {
      const uint64_t v = v0 + (uint64_t)r * 256;
      visit(load4(row, v + l4, false));
    }
  }
}

// The threshold lies in [t_lo, t_hi): the keys above it and equal to it below
// t_hi are counted on a tile's selection-interval keys, those >= t_hi come from
// its counts. One wave per hot tile, and one per kBT staged tiles: lane l holds
// tile t0 + l's counts; the first 64 keys of every tile are loaded at once,
// before the counts arrive, longer runs four windows at a time. Tiles of exact
// devices are counted on the gradient, one workgroup per tile.
template <int kBT>
__global__ __launch_bounds__(kBlock) void k_count(Ctx c, uint32_t workers, uint32_t per_dev)
{
  const uint32_t l = lane_id(), w = wave_id();
  if (blockIdx.x >= workers) {
    const uint32_t b = blockIdx.x - workers;
    const uint32_t jr = b / per_dev, j = c.j0 + jr;
    const uint32_t t0 = ((b - jr * per_dev) * kWaves + w) * kBT, last = c.nslot - 1;
    if (t0 >= c.nslot) return;
    const uint64_t row = (uint64_t)j * c.nslot;
    const GLOBAL uint32_t* reg = gptr(c.slot);
    uint32_t kv[kBT];
#pragma unroll
    for (int i = 0; i < kBT; ++i) {
      const uint32_t ti = t0 + i < last ? t0 + i : last;
      kv[i] = reg[(row + ti) * kSlotWords + l];
    }
    const uint32_t v = l < (uint32_t)kBT && t0 + l < c.nslot ? c.slot_cnt[row + t0 + l] : 0x8000u;
    const bool staged = !(v & 0x8000u);
    const uint32_t nb = staged ? (v & 0x7FFFu) - (v >> 16) : 0u;
    const DevState& st = c.st[j];
    if (st.fallback) return;
    uint32_t thr, need;
    threshold_of(st, thr, need);
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kBT; ++i) {
      const uint32_t n = __builtin_amdgcn_readlane(nb, i);
      uint32_t gt = (uint32_t)__builtin_amdgcn_readlane(v, i) >> 16, eq = 0;
      auto visit = [&](uint32_t key, bool valid) {
        gt += (uint32_t)__builtin_popcountll(ballot(valid && key > thr));
        eq += (uint32_t)__builtin_popcountll(ballot(valid && key == thr));
      };
      visit(kv[i], l < n);
      if (n > 64u) {
        const GLOBAL uint32_t* p = reg + (row + t0 + i) * kSlotWords;
        for (uint32_t e = 64; e < n; e += 256) {
          uint32_t x[4];
#pragma unroll
          for (int m = 0; m < 4; ++m) x[m] = e + m * 64 + l < n ? p[e + m * 64 + l] : 0u;
#pragma unroll
          for (int m = 0; m < 4; ++m) visit(x[m], e + m * 64 + l < n);
        }
      }
      if (l == (uint32_t)i) mine = gt | (eq << 16);
    }
    if (staged) c.tile_cnt[row + t0 + l] = mine;
    return;
  }
  for_hot_tiles<true, false>(c, blockIdx.x * kWaves + w, workers * kWaves, [&](uint32_t j, uint32_t s) {
    const DevDesc& d = c.desc[j];
    uint32_t thr, need;
    threshold_of(c.st[j], thr, need);
    const uint64_t slot = (uint64_t)j * c.nslot + s;
    const uint32_t v = c.slot_cnt[slot];
    const GLOBAL uint32_t* p = gptr(c.band) + d.band_off + (uint64_t)(s % c.nseg) * d.seg_cap + c.slot_boff[slot];
    uint32_t gt = v >> 16, eq = 0;
    const uint32_t n = (v & 0x7FFFu) - gt;
    for (uint32_t e = 0; e < n; e += 8 * 64) {
      uint32_t x[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) x[m] = e + m * 64 + l < n ? p[e + m * 64 + l] : 0u;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const bool valid = e + m * 64 + l < n;
        gt += (uint32_t)__builtin_popcountll(ballot(valid && x[m] > thr));
        eq += (uint32_t)__builtin_popcountll(ballot(valid && x[m] == thr));
      }
    }
    if (l == 0) c.tile_cnt[slot] = gt | (eq << 16);
  });
  __shared__ uint32_t s_c[kWaves];
  for_hot_tiles<false, true>(c, blockIdx.x, workers, [&](uint32_t j, uint32_t s) {
    const DevDesc& d = c.desc[j];
    uint32_t thr, need;
    threshold_of(c.st[j], thr, need);
    const Row row{gptr(d.grad), d.shift, c.n};
    const uint32_t thr1 = thr + 1u;       // rank keys: pads are never above or equal
    uint32_t n = 0;                       // gt | eq << 16 of the wave's chunk: at most 4096 each
    walk_chunk(row, s, [&](const f4& x) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t kq = rank_key(x[q]);
        n += (uint32_t)__builtin_popcountll(ballot(kq > thr1));
        n += (uint32_t)__builtin_popcountll(ballot(kq == thr1)) << 16;
      }
    });
    __syncthreads();
    if (l == 0) s_c[w] = n;
    __syncthreads();
    // sums of at most kTile each: no carry between the halves
    if (threadIdx.x == 0) c.tile_cnt[(uint64_t)j * c.nslot + s] = (s_c[0] + s_c[1]) + (s_c[2] + s_c[3]);
  });
}

// A tile's counts, gt | eq << 16, as gt | eq << 32.
__device__ inline uint64_t counts_of(uint32_t n) { return (uint64_t)(n & 0xFFFFu) | ((uint64_t)(n >> 16) << 32); }

// One workgroup per device: the exclusive prefix of its tiles' counts (gt | eq <<
// 16) as gt | eq << 32. 1024 threads when it runs alone; 256 when it runs beside another selection's main
// pass, whose stream of small workgroups rarely leaves 16 waves of a compute
// unit free at once.
constexpr int kScanLarge = 1024, kScanSmall = 256;
template <int NT>
__global__ __launch_bounds__(NT) void k_offsets(Ctx c)
{
  constexpr int kPer = 8, kW = NT / 64;
  __shared__ uint32_t h[NT * kPer];
  __shared__ uint64_t s_w[kW];
  const uint32_t j = c.j0 + blockIdx.x, tid = threadIdx.x, w = tid >> 6;
  const uint32_t* cnt = c.tile_cnt + (uint64_t)j * c.nslot;
  uint64_t* pre = c.tile_pre + (uint64_t)j * c.nslot;
  uint64_t base = 0;
  for (uint32_t t0 = 0; t0 < c.nslot; t0 += NT * kPer) {
    uint32_t v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t t = t0 + i * NT + tid;
      v[i] = t < c.nslot ? cnt[t] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) h[i * NT + tid] = v[i];
    __syncthreads();
    uint64_t own[kPer], sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t x = h[tid * kPer + i];
      own[i] = sum;
      sum += counts_of(x);
    }
    const uint64_t incl = wave_incl_scan_u64(sum);
    if (lane_id() == 63) s_w[w] = incl;
    __syncthreads();
    uint64_t ex = base + incl - sum;
    for (uint32_t i = 0; i < (uint32_t)kW; ++i) {
      const uint64_t x = s_w[i];
      ex += i < w ? x : 0ull;
      base += x;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t t = t0 + tid * kPer + i;
      if (t < c.nslot) pre[t] = ex + own[i];
    }
    __syncthreads();
  }
}

// ---- 5. ordered output -----------------------------------------------------------------------
// Where a wave's kept entries go; run_g / run_e count its keys above / equal to
// the threshold so far, from the device's start.
struct Out {
  GLOBAL uint32_t* idx;
  GLOBAL float* val;
  GLOBAL uint32_t* lb;      // aggregation range markers (fused step) or null
  uint32_t thr, need, k, base;
  uint32_t run_g, run_e;
  double e2;
};

__device__ inline Out out_of(const Ctx& c, uint32_t j)
{
  const DevDesc& d = c.desc[j];
  Out o;
  o.idx = gptr(d.idx_out);
  o.val = gptr(d.val_out);
  o.lb = c.lb ? gptr(c.lb) + (uint64_t)j * c.nrange : nullptr;
  threshold_of(c.st[j], o.thr, o.need);
  o.k = d.k;
  o.base = c.idx_base;
  o.run_g = o.run_e = 0;
  o.e2 = 0.0;
  return o;
}

__device__ inline void put_entry(Out& o, uint32_t gt_b, uint32_t eq_b, uint32_t idx, float v)
{
  const uint32_t pos = gt_b + (eq_b < o.need ? eq_b : o.need);
  if (pos < o.k) {
    o.idx[pos] = idx + o.base;
    o.val[pos] = v;
  }
  o.e2 = __builtin_fma((double)v, (double)v, o.e2);
}

// The candidates of staged tile s (cn of them, nb in the selection interval),
// in index order, kWriteBatch
// windows of values and offsets loaded at a time (positions clamped into the
// tile's candidates). Also the range markers of the ranges starting in the
// tile: lb[r] = kept entries with idx < r * kARange, i.e. the output position
// of the first candidate at or after the range start (or the kept total after
// the tile). Ranges from rnext on are open.
constexpr int kWriteBatch = 8;

__device__ inline void write_staged(const Ctx& c, uint32_t j, uint32_t s, uint32_t cn, uint32_t nb, uint32_t shift,
                                    Out& o)
{
  const uint32_t l = lane_id();
  const GLOBAL uint32_t* reg = gptr(c.slot) + ((uint64_t)j * c.nslot + s) * kSlotWords;
  const GLOBAL uint16_t* r16 = reinterpret_cast<const GLOBAL uint16_t*>(reg);
  const GLOBAL uint32_t* vals = reg + nb;
  const uint64_t vg = (uint64_t)s * kTile;
  const uint32_t ibase = (uint32_t)(vg - shift);
  const uint64_t b0 = vg > shift ? vg - shift : 0;
  uint64_t b1 = vg + kTile - shift;
  if (b1 > c.n) b1 = c.n;
  uint32_t rnext = (uint32_t)((b0 + kARange - 1) / kARange);
  const uint32_t rend = (uint32_t)((b1 + kARange - 1) / kARange);
  for (uint32_t e0 = 0; e0 < cn; e0 += kWriteBatch * 64) {
    uint32_t vb[kWriteBatch], ix[kWriteBatch];
#pragma unroll
    for (int m = 0; m < kWriteBatch; ++m) {
      vb[m] = ix[m] = 0u;
      uint32_t e = e0 + m * 64 + l;
      if (e0 + m * 64 < cn) {
        e = e < cn ? e : cn - 1u;
        vb[m] = vals[e];
        ix[m] = ibase + r16[slot_off16_at(e)];
      }
    }
#pragma unroll
    for (int m = 0; m < kWriteBatch; ++m) {
      if (e0 + m * 64 >= cn) break;
      const bool valid = e0 + m * 64 + l < cn;
      const uint32_t key = vb[m] & kKeyMask;
      const bool fg = valid && key > o.thr, fe = valid && key == o.thr;
      const uint64_t bg = ballot(fg), be = ballot(fe);
      const uint32_t gt_b = o.run_g + mbcnt(bg), eq_b = o.run_e + mbcnt(be);
      if (o.lb) {
        const uint32_t ri = ix[m] / (uint32_t)kARange;
        const uint32_t rp = __shfl_up(ri, 1, 64);
        const uint64_t vm = ballot(valid);
        if (valid) {
          const uint32_t p = gt_b + (eq_b < o.need ? eq_b : o.need);
          for (uint32_t r = (l == 0 ? rnext : rp + 1u); r <= ri; ++r) o.lb[r] = p;
        }
        rnext = (uint32_t)__builtin_amdgcn_readlane(ri, 63 - __builtin_clzll(vm)) + 1u;
      }
      if (fg || (fe && eq_b < o.need)) put_entry(o, gt_b, eq_b, ix[m], __uint_as_float(vb[m]));
      o.run_g += (uint32_t)__builtin_popcountll(bg);
      o.run_e += (uint32_t)__builtin_popcountll(be);
    }
  }
  if (o.lb) {
    const uint32_t p = o.run_g + (o.run_e < o.need ? o.run_e : o.need);
    for (uint32_t r = rnext + l; r < rend; r += 64) o.lb[r] = p;
  }
}

// A hot tile, read from the gradient again by a workgroup of kWB threads, every
// wave kHotWindows windows of 64 elements at once, one per lane, all of them in
// registers: the wave counts its keys, the counts before it place it, and the
// kept entries of a window leave as one contiguous run. 16 windows leave the
// kernel 64 registers, 8 waves per SIMD (32 took 72, and the 256-thread kernel
// spilled: see k_write). Their kept squares (lanes in window order, then a
// fixed tree) go to s_e: the tile's energy is the sum of s_e in order, the same for
// every kWB.
constexpr int kHotWindows = 16;
constexpr int kHotSums = kTile / (kHotWindows * 64);

template <int kWB>
__device__ inline void write_hot(const Ctx& c, const DevDesc& d, uint32_t s, uint32_t* s_n, double* s_e, Out& o)
{
  constexpr int kW = kWB / 64;
  const uint32_t l = lane_id(), w = wave_id();
  const uint64_t vbase = (uint64_t)s * kTile;
  const GLOBAL uint32_t* g = reinterpret_cast<const GLOBAL uint32_t*>(gptr(d.grad));
  const uint32_t thr1 = o.thr + 1u;       // rank keys: pads are never above or equal
  const bool full = vbase >= d.shift && vbase + kTile <= d.shift + c.n;
#pragma unroll 1
  for (uint32_t p = 0; p < (uint32_t)kTile; p += kWB * kHotWindows) {
    const uint64_t v0 = vbase + p + w * (kHotWindows * 64);
    uint32_t x[kHotWindows];
    if (full) {
      const GLOBAL uint32_t* gw = g + (v0 - d.shift);
#pragma unroll
      for (int m = 0; m < kHotWindows; ++m) x[m] = __builtin_nontemporal_load(gw + m * 64 + l);
    } else {
      // the (at most two) edge tiles of a device hold positions outside the gradient
#pragma unroll
      for (int m = 0; m < kHotWindows; ++m) {
        const uint64_t v = v0 + m * 64 + l, end = d.shift + c.n;
        const uint64_t at = v < d.shift ? 0 : (v < end ? v - d.shift : c.n - 1);
        const uint32_t y = g[at];
        x[m] = v >= d.shift && v < end ? y : kPadBits;
      }
    }
    uint32_t n = 0;                         // gt | eq << 16: at most 1024 each
#pragma unroll
    for (int m = 0; m < kHotWindows; ++m) {
      const uint32_t key1 = rank_key(__uint_as_float(x[m]));
      n += (uint32_t)__builtin_popcountll(ballot(key1 > thr1));
      n += (uint32_t)__builtin_popcountll(ballot(key1 == thr1)) << 16;
      __builtin_amdgcn_sched_barrier(0);    // keep windows apart: bounds the live ballot masks
    }
    __syncthreads();                        // the counts before have been read
    if (l == 0) s_n[w] = n;
    __syncthreads();
    // the counts of the waves before this one, and of all
    uint32_t bg0 = 0, be0 = 0, ag = 0, ae = 0;
    for (uint32_t i = 0; i < (uint32_t)kW; ++i) {
      const uint32_t v = s_n[i];
      if (i == w) {
        bg0 = ag;
        be0 = ae;
      }
      ag += v & 0xFFFFu;
      ae += v >> 16;
    }
    const uint32_t next_g = o.run_g + ag, next_e = o.run_e + ae;
    o.run_g += bg0;
    o.run_e += be0;
    // The one range start among the wave's positions, if any: its marker is the
    // kept entries before that element (every element of the tile passes by).
    static_assert(kHotWindows * 64 <= kARange, "a wave's positions hold one range start at most");
    const uint64_t first = v0 > d.shift ? v0 - d.shift : 0;
    const uint64_t start = (first + kARange - 1) / kARange * kARange;
    const uint32_t mark = o.lb && start < c.n ? (uint32_t)(start + d.shift - v0) : 0xFFFFFFFFu;
    const uint32_t i0 = (uint32_t)(v0 - d.shift);
#pragma unroll
    for (int m = 0; m < kHotWindows; ++m) {
      const uint32_t key1 = rank_key(__uint_as_float(x[m]));
      const bool fg = key1 > thr1, fe = key1 == thr1;
      const uint64_t bg = ballot(fg), be = ballot(fe);
      const uint32_t gt_b = o.run_g + mbcnt(bg), eq_b = o.run_e + mbcnt(be);
      if (mark == (uint32_t)m * 64 + l) o.lb[start / kARange] = gt_b + (eq_b < o.need ? eq_b : o.need);
      if (fg || (fe && eq_b < o.need)) put_entry(o, gt_b, eq_b, i0 + m * 64 + l, __uint_as_float(x[m]));
      o.run_g += (uint32_t)__builtin_popcountll(bg);
      o.run_e += (uint32_t)__builtin_popcountll(be);
      __builtin_amdgcn_sched_barrier(0);
    }
    const double es = wave_sum_f64(o.e2);
    if (l == 0) s_e[p / (kHotWindows * 64) + w] = es;
    o.e2 = 0.0;
    o.run_g = next_g;
    o.run_e = next_e;
  }
}

// ---- 6. energies of the adaptive rule and per-device decision --------------------------------
// §IV: send Top-k(g) when | ||g||^2 - ||Top-k(g)||^2 | / ||g||^2 <= delta. One
// workgroup per device, after the output pass: a launch of its own, because
// a last workgroup of the output would make every one wait for its stores
// before it ends (16 x 60.2M: the output 36 -> 84 us).
__global__ __launch_bounds__(kBlock) void k_final(Ctx c)
{
  __shared__ double s_e[kWaves];
  const uint32_t j = c.j0 + blockIdx.x;
  DevState& s = c.st[j];
  const double* ea = c.epart + (uint64_t)j * c.nslot;
  const double* ek = c.ekept + (uint64_t)j * c.nslot;
  const uint32_t* cnt = c.tile_cnt + (uint64_t)j * c.nslot;
  double all = 0.0, kept = 0.0;
  uint64_t gt = 0;
#pragma unroll 4
  for (uint32_t b = threadIdx.x; b < c.nslot; b += kBlock) {
    all += ea[b];
    kept += ek[b];
    gt += cnt[b] & 0xFFFFu;
  }
  __shared__ uint64_t s_gt[kWaves];
  gt = wave_sum_u64(gt);
  if (lane_id() == 0) s_gt[threadIdx.x >> 6] = gt;
  const double e_all = block_sum_f64(all, s_e);      // (its barrier covers s_gt)
  const double e_kept = block_sum_f64(kept, s_e);
  if (threadIdx.x != 0) return;
  uint32_t thr, need;
  if (!threshold_of(s, thr, need)) s.err |= kErrNoThreshold;
  s.thr = thr;
  s.need = need;
  s.c_gt = (s_gt[0] + s_gt[1]) + (s_gt[2] + s_gt[3]);
  if (s.c_gt + s.need != c.desc[j].k || (c.inject_count_error && j == 0)) s.err |= kErrCount;
  if (c.err_acc && (s.err & kErrFatal)) atomicOr(c.err_acc + j, s.err & kErrFatal);
  s.e_all = e_all;
  s.e_kept = e_kept;
  // §IV: the rule compares the energies, optionally their moving averages
  s.sparse = adaptive_rule(e_all, e_kept, c.ewma ? c.ewma + 2 * (uint64_t)j : nullptr, c.ewma_beta, c.delta);
  if (c.counters) account(c.counters + 3 * (uint64_t)j, s.sparse, c.desc[j].k, c.n);
  if (c.energies_out) {
    c.energies_out[(uint64_t)c.e_stride * j] = e_all;
    c.energies_out[(uint64_t)c.e_stride * j + 1] = e_kept;
  }
  if (c.compressed_out) c.compressed_out[j] = (uint8_t)s.sparse;
}

// Kept-above | equal << 32 counts of the device's tiles before tile s, by a
// workgroup of NT threads (s_p: one word per wave).
template <int NT>
__device__ inline uint64_t tiles_before(const Ctx& c, uint32_t j, uint32_t s, uint64_t* s_p)
{
  const uint32_t* cnt = c.tile_cnt + (uint64_t)j * c.nslot;
  uint64_t sum = 0;
  for (uint32_t t = threadIdx.x; t < s; t += NT) sum += counts_of(cnt[t]);
  sum = wave_sum_u64(sum);
  __syncthreads();
  if (lane_id() == 0) s_p[wave_id()] = sum;
  __syncthreads();
  uint64_t all = s_p[0];
  for (int i = 1; i < NT / 64; ++i) all += s_p[i];
  return all;
}

// Output pass over the staged tiles of device b / per_dev of the launch,
// kWriteTiles per wave, by workgroup b of kWB threads. The kept sum of squares of
// each tile goes to ekept. kOwnOffsets: the workgroup sums the counts of the tiles
// before its own instead of reading a launch's offsets.
constexpr uint32_t kWriteTiles = 2;

template <int kWB, bool kOwnOffsets>
__device__ inline void write_staged_tiles(const Ctx& c, uint32_t b, uint32_t per_dev, uint64_t* s_p)
{
  constexpr int kW = kWB / 64;
  const uint32_t l = lane_id(), w = wave_id();
  const uint32_t jr = b / per_dev, j = c.j0 + jr;
  const uint32_t tb = (b - jr * per_dev) * (kW * kWriteTiles), s0 = tb + w * kWriteTiles;
  const uint64_t row = (uint64_t)j * c.nslot;
  const bool live = l < kWriteTiles && s0 + l < c.nslot;
  const uint32_t va = live ? c.slot_cnt[row + s0 + l] : 0x8000u;
  uint64_t pre;
  if (kOwnOffsets) {
    if (c.st[j].fallback) return;
    static_assert(kW * kWriteTiles <= 64, "a wave scans its workgroup's tiles");
    const uint32_t n = l < kW * kWriteTiles && tb + l < c.nslot ? c.tile_cnt[row + tb + l] : 0u;
    const uint64_t base = tiles_before<kWB>(c, j, tb, s_p);
    const uint64_t ex = base + wave_incl_scan_u64(counts_of(n)) - counts_of(n);
    pre = __shfl(ex, w * kWriteTiles + (l < kWriteTiles ? l : 0u), 64);
  } else {
    pre = c.tile_pre[live ? row + s0 + l : row];
    if (c.st[j].fallback) return;
  }
  if (ballot(!(va & 0x8000u)) == 0ull) return;
  Out o = out_of(c, j);
  const uint32_t shift = c.desc[j].shift;
  for (uint32_t i = 0; i < kWriteTiles; ++i) {
    const uint32_t v = __builtin_amdgcn_readlane(va, i);
    if (v & 0x8000u) continue;
    o.run_g = __builtin_amdgcn_readlane((uint32_t)pre, i);
    o.run_e = __builtin_amdgcn_readlane((uint32_t)(pre >> 32), i);
    o.e2 = 0.0;
    write_staged(c, j, s0 + i, v & 0x7FFFu, (v & 0x7FFFu) - (v >> 16), shift, o);
    const double es = wave_sum_f64(o.e2);
    if (l == 0) c.ekept[row + s0 + i] = es;
  }
}

// The same over the hot tiles, every workers-th of them from the first on, one
// per workgroup of kWB threads.
template <int kWB, bool kOwnOffsets>
__device__ inline void write_hot_tiles(const Ctx& c, uint32_t first, uint32_t workers, uint64_t* s_p)
{
  __shared__ double s_e[kHotSums];
  __shared__ uint32_t s_n[kWB / 64];
  for_hot_tiles<true, true>(c, first, workers, [&](uint32_t j, uint32_t s) {
    const uint64_t slot = (uint64_t)j * c.nslot + s;
    const uint64_t pre = kOwnOffsets ? tiles_before<kWB>(c, j, s, s_p) : c.tile_pre[slot];
    Out o = out_of(c, j);
    o.run_g = (uint32_t)pre;
    o.run_e = (uint32_t)(pre >> 32);
    write_hot<kWB>(c, c.desc[j], s, s_n, s_e, o);
    __syncthreads();
    if (threadIdx.x == 0) {
      double e = s_e[0];
      for (int i = 1; i < kHotSums; ++i) e += s_e[i];
      c.ekept[slot] = e;
    }
  });
}

// Both in one launch, the hot tiles' workgroups first: theirs is the longer work.
// The staged tiles are bound by the latency of their slots and offsets, so the
// waves in flight count: at 8 per SIMD and 256 threads 32 x 143.7 M take 390 us
// from the main pass to the aggregation, at 7 and 512 threads 454, in two launches
// (each kind its own kernel) 395 and with many hot tiles more than in one
// (30 x 143.7 M with layers of their own scale: 4335 us per step, 4480, 4510).
// Where a workgroup sums its own offsets 8 waves would spill.
template <int kWB, bool kOwnOffsets>
__global__ __launch_bounds__(kWB) __attribute__((amdgpu_waves_per_eu(kOwnOffsets ? 7 : 8, 8))) void k_write(
    Ctx c, uint32_t workers, uint32_t per_dev)
{
  __shared__ uint64_t s_p[kWB / 64];
  if (blockIdx.x >= workers) write_staged_tiles<kWB, kOwnOffsets>(c, blockIdx.x - workers, per_dev, s_p);
  else write_hot_tiles<kWB, kOwnOffsets>(c, blockIdx.x, workers, s_p);
}

// ---- host-side launchers ---------------------------------------------------------------------
// Tiles per wave of the walks over the staged tiles' selection-interval keys (the
// first radix pass and the counts): the most, up to 16, that still give 6000
// waves over the devices of the launch, else 4. Few tiles per wave keep small
// launches wide; many keep large ones from flushing a histogram per few tiles.
// Beside another launch's main pass (a layer of the per-layer selection)
// always 16: fewer workgroups wait less for the slots that pass leaves.
static int band_tiles_per_wave(const Ctx& c, const SelectPlan& p)
{
  if (p.beside) return 16;
  const uint64_t tiles = (uint64_t)c.jn * c.nslot;
  if (tiles / 16 >= 6000) return 16;
  if (tiles / 8 >= 6000) return 8;
  return 4;
}

template <int kBT>
static void launch_threshold(const Ctx& c, const SelectPlan& p, hipStream_t s)
{
  const uint32_t walk = p.any_fast ? (c.nslot + kBT * kWaves - 1) / (kBT * kWaves) : 0u;
  const uint32_t per_dev = p.any_fast ? p.hist_blocks : 0u;
  k_hist<kBT><<<(walk + per_dev) * c.jn + p.full_workers, kBlock, 0, s>>>(c, walk, per_dev, 0u);
  for (uint32_t pass = 1; pass < 3; ++pass)
    k_hist<kBT><<<per_dev * c.jn + p.full_workers, kBlock, 0, s>>>(c, 0u, per_dev, pass);
  // third pass of exact devices found after the first one
  if (p.any_fast) k_hist<kBT><<<p.full_workers, kBlock, 0, s>>>(c, 0u, 0u, 3u);
  k_count<kBT><<<walk * c.jn + p.hot_workers, kBlock, 0, s>>>(c, p.hot_workers, walk);
}

// Whether the output sums the counts of the tiles before its own itself: for up
// to 1024 tiles (16.7 M elements) that is two loads per thread, less than a
// launch (k_offsets, 4.8 us).
static bool own_offsets(const Ctx& c, const SelectPlan& p) { return c.nslot <= 1024 && !p.beside; }

// Everything after the main pass for devices [c.j0, c.j0 + c.jn), on stream s,
// in two halves: 0, the threshold (path decision, radix passes, tile counts and
// offsets), latency-bound and light on memory; 1, the output (ordered
// compaction with the range markers, energies and decision), which moves most
// of the bytes. Workgroups for hot tiles come first: theirs is the longer work.
static void launch_post(const Ctx& c, const SelectPlan& p, hipStream_t s, int half)
{
  if (half == 0) {
    switch (band_tiles_per_wave(c, p)) {
      case 16: launch_threshold<16>(c, p, s); break;
      case 8: launch_threshold<8>(c, p, s); break;
      default: launch_threshold<4>(c, p, s); break;
    }
    if (own_offsets(c, p)) return;
    if (p.beside) k_offsets<kScanSmall><<<c.jn, kScanSmall, 0, s>>>(c);
    else k_offsets<kScanLarge><<<c.jn, kScanLarge, 0, s>>>(c);
    return;
  }
  auto write = [&](auto kernel, int block) {
    const uint32_t tiles = kWriteTiles * block / 64;
    const uint32_t per_dev = p.any_fast ? (c.nslot + tiles - 1) / tiles : 0u;
    kernel<<<per_dev * c.jn + p.hot_workers, block, 0, s>>>(c, p.hot_workers, per_dev);
  };
  // A hot tile's time is its workgroup's: 16 waves where a few tiles are all
  // there is (4 x 61,706: 11.5 us against 17), 8 where they sum their own offsets
  // (8 x 11.2 M: 34 against 40) or are at most 16384 in all (one of 143.7 M whose
  // entries lie in few layers, 8769 tiles: 14 against 20; with the entries spread,
  // 502 us per step with 4, 505 with 8), else 4 (16 x 25.6 M at ratio 0.1, 24960
  // tiles: 725 us per step against 739), also beside a main pass, which rarely
  // leaves 8 free at once (per-layer step of 16 x 143.7 M: 2680 against 2754).
  const uint64_t tiles = (uint64_t)c.jn * c.nslot;
  if (own_offsets(c, p)) {
    if (tiles <= 512) write(k_write<1024, true>, 1024);
    else write(k_write<512, true>, 512);
  } else if (tiles <= 16384 && !p.beside) {
    write(k_write<512, false>, 512);
  } else {
    write(k_write<256, false>, 256);
  }
  k_final<<<c.jn, kBlock, 0, s>>>(c);
}

// One pass over the sample while the devices' expected interval keys are few:
// its wider bins then cost less than a launch. (One / two passes, total: 4 x 1 M
// 84 / 89 us, 8 x 11.2 M 195 / 195, one of 143.7 M 187 / 196, 16 x 60.2 M 1080 /
// 1089 of which the threshold 95 / 78, 30 x 143.7 M 3537 / 3494.)
static void launch_sample(const Ctx& c, const SelectPlan& p, hipStream_t s)
{
  if (!p.any_fast) return;
  const dim3 grid(p.sample_blocks, c.K);
  if (p.interval_keys < (1u << 19)) {
    k_bracket<kSampleBits><<<grid, kBlock, 0, s>>>(c, 0u);
    return;
  }
  k_bracket<kDigitBits><<<grid, kBlock, 0, s>>>(c, 1u);
  k_refine<<<grid, kBlock, 0, s>>>(c);
}

// The whole selection. The devices are split into p.parts groups whose main
// passes run one after the other on s. A main pass is bound by HBM bandwidth,
// the threshold half of the rest of a group's selection by latency: that half
// of group i runs on s2 while the main pass of group i + 1 runs on s, and the
// output half of group i, which moves more bytes, only once that main pass is
// done (the last group's rest runs on s); s waits for s2 at the end.
// done[i] (events of s2's owner) mark the end of main pass i. Profiling events
// (ev, optional; as few as possible, each costs a few microseconds of queue
// time): 0 start, 1 bracket done, 3 + 2i the end of main pass i (main pass i
// starts at the end of the previous one; with profiling these also serve as
// done[i]), 2 + 2 * parts all done.
hipError_t launch_select(const Ctx& c0, const PrepArgs& a, const SelectPlan& p, hipStream_t s, hipStream_t s2,
                         hipEvent_t* done, hipEvent_t join, hipEvent_t* ev)
{
  Ctx c = c0;
  c.j0 = 0;
  c.jn = c.K;
  const uint64_t zero_words = (uint64_t)c.K * kSampleBins;
  uint32_t gprep = (uint32_t)((zero_words + kBlock * 8 - 1) / (kBlock * 8));
  gprep = gprep < 1 ? 1 : (gprep > 2048 ? 2048 : gprep);
  k_prep<<<gprep, kBlock, 0, s>>>(c, a);
  launch_sample(c, p, s);
  if (ev) (void)hipEventRecord(ev[1], s);
  GradArgs ga;
  for (uint32_t j = 0; j < c.K; ++j) ga.grad[j] = a.grad[j];
  const uint32_t parts = p.parts;
  auto group = [&](uint32_t i) {
    Ctx ci = c;
    ci.j0 = c.K * i / parts;
    ci.jn = c.K * (i + 1) / parts - ci.j0;
    return ci;
  };
  for (uint32_t i = 0; i < parts; ++i) {
    const Ctx ci = group(i);
    k_main<<<ci.jn * c.tpd, kBlock, 0, s>>>(ci, ga);
    hipEvent_t de = ev ? ev[3 + 2 * i] : (parts > 1 ? done[i] : nullptr);
    if (de) {
      hipError_t e = hipEventRecord(de, s);
      if (e == hipSuccess && parts > 1) e = hipStreamWaitEvent(s2, de, 0);
      if (e != hipSuccess) return e;
    }
    if (i > 0) launch_post(group(i - 1), p, s2, 1);
    if (i + 1 < parts) {
      launch_post(ci, p, s2, 0);
    } else {
      launch_post(ci, p, s, 0);
      launch_post(ci, p, s, 1);
    }
  }
  if (parts > 1) {
    hipError_t e = hipEventRecord(join, s2);
    if (e == hipSuccess) e = hipStreamWaitEvent(s, join, 0);
    if (e != hipSuccess) return e;
  }
  if (ev) (void)hipEventRecord(ev[2 + 2 * parts], s);
  return hipGetLastError();
}

// The selection of all devices in three parts, for callers that pipeline
// several selections on alternating workspaces (the long layers of a
// per-layer selection): preparation and bracket; the main pass; everything
// after it. The caller orders them and the workspace reuse with events.
hipError_t launch_bracket(const Ctx& c0, const PrepArgs& a, const SelectPlan& p, hipStream_t s)
{
  Ctx c = c0;
  c.j0 = 0;
  c.jn = c.K;
  const uint64_t zero_words = (uint64_t)c.K * kSampleBins;
  uint32_t gprep = (uint32_t)((zero_words + kBlock * 8 - 1) / (kBlock * 8));
  gprep = gprep < 1 ? 1 : (gprep > 2048 ? 2048 : gprep);
  k_prep<<<gprep, kBlock, 0, s>>>(c, a);
  launch_sample(c, p, s);
  return hipGetLastError();
}

hipError_t launch_main(const Ctx& c0, const PrepArgs& a, hipStream_t s)
{
  Ctx c = c0;
  c.j0 = 0;
  c.jn = c.K;
  GradArgs ga;
  for (uint32_t j = 0; j < c.K; ++j) ga.grad[j] = a.grad[j];
  k_main<<<c.K * c.tpd, kBlock, 0, s>>>(c, ga);
  return hipGetLastError();
}

hipError_t launch_rest(const Ctx& c0, const SelectPlan& p, hipStream_t s)
{
  Ctx c = c0;
  c.j0 = 0;
  c.jn = c.K;
  launch_post(c, p, s, 0);
  launch_post(c, p, s, 1);
  return hipGetLastError();
}

}  // namespace scadles
