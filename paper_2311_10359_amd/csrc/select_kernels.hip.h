// Count, sum, minimum, maximum and the nearest-rank p50 / p95 (Section 3.2: sum / count = SK_j, SG_j) of an ID's execution
// times and idle times, which lie next to each other in LDS.  A group of GW lanes takes one of the two, so a wave takes
// 32 / GW IDs at a time, and nothing here waits for another wave.
//
//   1. One pass over the samples: count, sum, minimum, maximum in registers, combined over the group.
//   2. One pass adds to a histogram of 8 * GW bins over [minimum, maximum]: equal steps of the value itself where the range is
//      narrow, of scale_of(value), which follows the value's size, where it is wide.  Every lane then reads eight bins, and a
//      prefix sum over the group says which lane's bins hold the two wanted ranks.
//   3. A bin with many samples that is more than one value wide is cut into 4 * GW bins of equal width and its samples are
//      counted again, until that is not so (seldom needed).
//   4. One pass lists the samples of the two bins that are left, and they are ranked by counting.
#pragma once

#include "common.hip.h"

namespace fikit {

constexpr uint32_t NONE32 = 0xffffffffu;   // "no idle time after this launch" among 32-bit values

// The scale on which histograms over wide ranges lay out their bins: the bit pattern of the value as a float, without
// its lowest 12 bits, i.e. the exponent and the leading 12 bits of the value.  Conversion rounds to nearest, which is
// monotone, so ranks found on the scale are ranks of the values; values below 2^SCALE_EXACT_BITS map one to one and
// come back exactly with value_of_scale.  Durations of one kernel spread over a range in proportion to their size
// (the workloads draw them lognormal): bins of equal width on this scale then hold similar numbers of samples, where
// bins of equal width in nanoseconds would crowd most samples into the lowest few.
constexpr uint32_t SCALE_EXACT_BITS = 12, SCALE_DROP = 12;
__device__ __forceinline__ uint32_t scale_of(uint32_t v) { return __float_as_uint(__uint2float_rn(v)) >> SCALE_DROP; }
__device__ __forceinline__ uint32_t value_of_scale(uint32_t t) { return static_cast<uint32_t>(__uint_as_float(t << SCALE_DROP)); }

// The combination of the values of the GW (16 or 32) lanes of a group, in all of them.  All 64 lanes must call.
template <int GW, typename Op>
__device__ __forceinline__ uint32_t group_all(uint32_t v, Op op) {
  static_assert(GW == 16 || GW == 32, "a row of lanes, or two");
  v = op(v, dpp_move<0xB1>(v));    // quad_perm [1,0,3,2]
  v = op(v, dpp_move<0x4E>(v));    // quad_perm [2,3,0,1]
  v = op(v, dpp_move<0x141>(v));   // row_half_mirror
  v = op(v, dpp_move<0x140>(v));   // row_mirror
  if constexpr (GW == 32) {
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // (rows 0 0 2 2 and 1 1 3 3)
    v = op(p[0], p[1]);
  }
  return v;
}
template <int GW> __device__ __forceinline__ uint32_t group_max(uint32_t v) { return group_all<GW>(v, [](uint32_t a, uint32_t b) { return max_u32(a, b); }); }
template <int GW> __device__ __forceinline__ uint32_t group_min(uint32_t v) { return group_all<GW>(v, [](uint32_t a, uint32_t b) { return min_u32(a, b); }); }
template <int GW> __device__ __forceinline__ uint32_t group_sum(uint32_t v) { return group_all<GW>(v, [](uint32_t a, uint32_t b) { return a + b; }); }
// Inclusive prefix sum over the lanes of a group.
template <int GW>
__device__ __forceinline__ uint32_t group_incl_scan(uint32_t v) {
  v += dpp_or_zero<0x111, 0xf>(v);   // (see wave_incl_scan_u32)
  v += dpp_or_zero<0x112, 0xf>(v);
  v += dpp_or_zero<0x114, 0xf>(v);
  v += dpp_or_zero<0x118, 0xf>(v);
  if (GW == 32) v += dpp_or_zero<0x142, 0xa>(v);
  return v;
}

constexpr uint32_t PICK_HIST = 4 * WAVE;      // words of LDS that the histograms of a wave's groups take (16-byte aligned)
constexpr uint32_t PICK_SAMPLES = 1u << 14;   // most samples of an ID

// Calls use(sample) for every sample of the group's part v[0 .. n), with NONE32 in the place of those that are not there.
// `least` and `most` are the smallest and the largest n of the wave's groups; all 64 lanes call.
template <int GW, typename Use>
__device__ __forceinline__ void each_sample(const uint32_t* v, uint32_t n, uint32_t least, uint32_t most, Use use) {
  constexpr uint32_t UNROLL = 4;
  const uint32_t g = lane_id() & (GW - 1), last = n ? n - 1 : 0u;
  const uint32_t* at = v + g;
  uint32_t i0 = 0;
  for (; i0 + UNROLL * GW <= least; i0 += UNROLL * GW, at += UNROLL * GW) {
    uint32_t x[UNROLL];
#pragma unroll
    for (uint32_t u = 0; u < UNROLL; ++u) x[u] = at[u * GW];
#pragma unroll
    for (uint32_t u = 0; u < UNROLL; ++u) use(x[u]);
  }
  for (; i0 < most; i0 += GW) {
    const uint32_t x = v[min_u32(i0 + g, last)];
    use(i0 + g < n ? x : NONE32);
  }
}

// Histograms have two 16-bit counters to a word (an ID has at most PICK_SAMPLES samples).
__device__ __forceinline__ void count_in(uint32_t* hist, uint32_t bin) { atomicAdd(&hist[bin >> 1], 1u << ((bin << 4) & 31u)); }
__device__ __forceinline__ uint32_t cut_shift(uint32_t width, uint32_t bins_log2) {   // so that width >> shift is below 2^bins_log2
  return width >> bins_log2 ? 32u - static_cast<uint32_t>(__builtin_clz(width)) - bins_log2 : 0u;
}

// scale_of with 0 just below 1.
constexpr uint32_t SCALE_ZERO = (0x3f800000u >> SCALE_DROP) - 1;
__device__ __forceinline__ uint32_t pick_scale(float rounded) {
  return max_u32(__builtin_bit_cast(uint32_t, rounded) >> SCALE_DROP, SCALE_ZERO);
}
// The smallest value whose pick_scale is t or more.  From 2^24 on the values just below a step's own value round up to it: half a
// float's spacing, which is half as wide below a power of two.
__device__ __forceinline__ uint32_t pick_scale_low(uint32_t t) {
  if (t <= SCALE_ZERO) return 0u;
  const uint32_t bits = t << SCALE_DROP, e = (bits >> 23) - 127u;
  if (bits > 0x4f800000u) return NONE32;   // (beyond 2^32)
  const uint32_t own = e == 32 ? 0u : static_cast<uint32_t>(__builtin_ceilf(__builtin_bit_cast(float, bits)));   // (modulo 2^32)
  return own - static_cast<uint32_t>((1ull << e) >> (bits & 0x7fffffu ? 24 : 25));
}

// How the histogram of a group divides [min, max].
template <int GW>
struct Window {
  static constexpr uint32_t BINS_LOG2 = GW == 32 ? 8 : 7;
  uint32_t min, max, from, shift;
  bool linear;
  __device__ __forceinline__ Window(uint32_t min_, uint32_t max_) : min(min_), max(max_) {
    const uint32_t scale_lo = pick_scale(static_cast<float>(min)), by_scale = pick_scale(static_cast<float>(max)) - scale_lo;
    linear = ((max - min) >> BINS_LOG2) == 0 || (by_scale >> BINS_LOG2) == 0;
    from = linear ? min : scale_lo;
    shift = cut_shift(linear ? max - min : by_scale, BINS_LOG2);
  }
  __device__ __forceinline__ uint32_t bin(uint32_t x) const { return ((linear ? x : pick_scale(static_cast<float>(x))) - from) >> shift; }
  // the values of a bin that holds samples
  __device__ __forceinline__ uint32_t low(uint32_t b) const {
    const uint32_t t = from + (b << shift);
    return max_u32(linear ? t : pick_scale_low(t), min);
  }
  __device__ __forceinline__ uint32_t high(uint32_t b) const {
    const uint32_t t = from + ((b + 1) << shift);
    return linear ? (max - from < (b + 1) << shift ? max : t - 1) : min_u32(pick_scale_low(t) - 1, max);
  }
};

// Where a wanted sample is: among the `count` samples of values lo .. lo + width it is the one of rank `rank`.
struct Range {
  uint32_t lo, width, rank, count;
  __device__ __forceinline__ bool wide(uint32_t most) const { return width != 0 && count > most; }
  __device__ __forceinline__ bool has(uint32_t x) const { return x - lo <= width; }   // (never NONE32)
};

// What a pass over the samples has gathered (min NONE32 and max1 0 without any; max1 is one more than the maximum).
struct Tally { uint32_t count, min, max1; uint64_t sum; };
// ... by a lane, on the way: each sample one larger, so that NONE32 adds nothing to sum, count and maximum.
struct LaneTally {
  uint32_t count = 0, min = NONE32, max1 = 0;
  uint64_t sum1 = 0;
  __device__ __forceinline__ void add(uint32_t x) {
    const uint32_t x1 = x + 1;
    min = min_u32(min, x);
    max1 = max_u32(max1, x1);
    sum1 += x1;
    count += x1 != 0 ? 1u : 0u;
  }
  template <int GW>
  __device__ __forceinline__ Tally of_group() const {
    Tally t;
    t.count = group_sum<GW>(count);
    t.min = group_min<GW>(min);
    t.max1 = group_max<GW>(max1);
    // (a lane's sum is below 2^32 * PICK_SAMPLES / 16 = 2^42: two parts whose totals over the group fit 32 bits)
    const uint32_t lo = group_sum<GW>(static_cast<uint32_t>(sum1) & 0xffffffu), hi = group_sum<GW>(static_cast<uint32_t>(sum1 >> 24));
    t.sum = (static_cast<uint64_t>(hi) << 24) + lo - t.count;
    return t;
  }
};

// The bin that holds rank k | the rank inside the bin << 8 | the bin's samples (63 for more) << 22.  Lane g of a group holds the
// words w of bins 8g .. 8g + 7, their samples summed up after each word, and how many samples precede them.
constexpr uint32_t PLACE_MANY = 63;
template <int GW>
__device__ __forceinline__ uint32_t place_word(uint32_t k, uint4 w, uint4 s, uint32_t before) {
  static_assert(8 * GW <= 256 && PICK_SAMPLES <= 1u << 14, "a bin and a rank are packed into 8 and 14 bits");
  const uint32_t t = k - before, w0 = w.x, w1 = w.y, w2 = w.z, w3 = w.w, s0 = s.x, s1 = s.y, s2 = s.z;
  const bool b1 = t >= s0, b2 = t >= s1, b3 = t >= s2;
  const uint32_t word = b3 ? w3 : b2 ? w2 : b1 ? w1 : w0, in = t - (b3 ? s2 : b2 ? s1 : b1 ? s0 : 0u), lower = word & 0xffffu;
  const bool odd = in >= lower;
  const uint32_t bin = 8 * (lane_id() & (GW - 1)) + (b1 ? 2u : 0u) + (b2 ? 2u : 0u) + (b3 ? 2u : 0u) + (odd ? 1u : 0u);
  const uint32_t rank = odd ? in - lower : in, count = odd ? word >> 16 : lower;
  return group_max<GW>(t < s.w ? bin | rank << 8 | min_u32(count, PLACE_MANY) << 22 : 0u);
}
__device__ __forceinline__ uint32_t place_bin(uint32_t word) { return word & 255u; }
__device__ __forceinline__ uint32_t place_rank(uint32_t word) { return (word >> 8) & 0x3fffu; }
__device__ __forceinline__ uint32_t place_count(uint32_t word) { return word >> 22; }

// Looks up both ranks in the wave's histograms.  With `halves` the second one is looked up in the second half.
template <int GW>
__device__ __forceinline__ void search(const uint32_t* hist, uint32_t k50, uint32_t k95, bool halves, uint32_t& at50, uint32_t& at95) {
  const uint32_t lane = lane_id(), g = lane & (GW - 1);
  const uint4 w = reinterpret_cast<const uint4*>(hist)[lane];
  uint4 s;
  s.x = (w.x & 0xffffu) + (w.x >> 16);
  s.y = s.x + (w.y & 0xffffu) + (w.y >> 16);
  s.z = s.y + (w.z & 0xffffu) + (w.z >> 16);
  s.w = s.z + (w.w & 0xffffu) + (w.w >> 16);
  const uint32_t incl = group_incl_scan<GW>(s.w), before = incl - s.w;
  if (halves) k95 += group_max<GW>(g < GW / 2 ? incl : 0u);
  at50 = place_word<GW>(k50, w, s, before);
  at95 = place_word<GW>(k95, w, s, before);
}
__device__ __forceinline__ void clear_hist(uint32_t* hist) {
  __builtin_amdgcn_wave_barrier();
  reinterpret_cast<uint4*>(hist)[lane_id()] = make_uint4(0, 0, 0, 0);
  __builtin_amdgcn_wave_barrier();
}

template <int GW>
__device__ __forceinline__ Window<GW> window_of(const Tally& t) { return Window<GW>(t.count ? t.min : 0u, t.count ? t.max1 - 1 : 0u); }
template <int GW>
__device__ __forceinline__ void add_first(const Window<GW>& win, const uint32_t* v, uint32_t n, uint32_t least, uint32_t most, uint32_t* mine) {
  each_sample<GW>(v, n, least, most, [&](uint32_t x) { if (x != NONE32) count_in(mine, win.bin(x)); });
}
// The ranges that hold the two wanted ranks (0 .. 0 without samples).
template <int GW>
__device__ __forceinline__ void first_ranges(const Window<GW>& win, const uint32_t* hist, uint32_t count, Range& r50, Range& r95) {
  uint32_t at50, at95;
  const bool some = count != 0;
  search<GW>(hist, some ? rank_index_u32(50, count) : NONE32, some ? rank_index_u32(95, count) : NONE32, false, at50, at95);
  auto range = [&](uint32_t at) {
    const uint32_t lo = win.low(place_bin(at));
    return Range{some ? lo : 0u, some ? win.high(place_bin(at)) - lo : 0u, place_rank(at), place_count(at)};
  };
  r50 = range(at50);
  r95 = range(at95);
}
// Counts the samples in the ranges that are too wide, in a half of the group's histogram each; narrows them.
template <int GW>
__device__ __forceinline__ void add_cut(const Range& r50, const Range& r95, const uint32_t* v, uint32_t n, uint32_t least, uint32_t most,
                                        uint32_t* mine) {
  const uint32_t s50 = cut_shift(r50.width, GW == 32 ? 7 : 6), s95 = cut_shift(r95.width, GW == 32 ? 7 : 6);
  const bool go50 = r50.wide(GW), go95 = r95.wide(GW);
  each_sample<GW>(v, n, least, most, [&](uint32_t x) {
    if (go50 && r50.has(x)) count_in(mine, (x - r50.lo) >> s50);
    if (go95 && r95.has(x)) count_in(mine, 4 * GW + ((x - r95.lo) >> s95));
  });
}
template <int GW>
__device__ __forceinline__ void narrow(const uint32_t* hist, Range& r50, Range& r95) {
  uint32_t at50, at95;
  search<GW>(hist, r50.rank, r95.rank, true, at50, at95);
  auto to = [&](Range& r, uint32_t at, uint32_t first) {
    if (!r.wide(GW)) return;
    const uint32_t s = cut_shift(r.width, GW == 32 ? 7 : 6), past = (place_bin(at) - first) << s;
    r = Range{r.lo + past, min_u32(r.width - past, (1u << s) - 1), place_rank(at), place_count(at)};
  };
  to(r50, at50, 0);
  to(r95, at95, 4 * GW);
}

// Lists of the samples in the two ranges: in the space of the histogram, GW places each, behind them how long they are.  Places
// that are not used hold NONE32.
template <int GW>
__device__ __forceinline__ void clear_lists(uint32_t* hist) {
  const uint32_t lane = lane_id(), fill = (lane & (GW - 1)) < GW / 2 ? NONE32 : 0u;
  __builtin_amdgcn_wave_barrier();
  reinterpret_cast<uint4*>(hist)[lane] = make_uint4(fill, fill, fill, fill);
  __builtin_amdgcn_wave_barrier();
}
template <int GW>
__device__ __forceinline__ void add_lists(const Range& r50, const Range& r95, const uint32_t* v, uint32_t n, uint32_t least, uint32_t most,
                                          uint32_t* mine) {
  const bool list50 = r50.width != 0, list95 = r95.width != 0;   // (a range of one value is the answer)
  each_sample<GW>(v, n, least, most, [&](uint32_t x) {
    if (list50 && r50.has(x)) mine[atomicAdd(&mine[2 * GW], 1u) & (GW - 1)] = x;
    if (list95 && r95.has(x)) mine[GW + (atomicAdd(&mine[2 * GW + 1], 1u) & (GW - 1))] = x;
  });
}
// The wanted samples (in all lanes of the group): a lane per listed sample counts the smaller ones; the sample of rank r is the
// largest with at most r smaller ones.
template <int GW>
__device__ __forceinline__ void rank_lists(const uint32_t* mine, const Range& r50, const Range& r95, uint32_t& v50, uint32_t& v95) {
  const uint32_t g = lane_id() & (GW - 1);
  const uint32_t n50 = r50.width ? r50.count : 0u, n95 = r95.width ? r95.count : 0u;
  const uint32_t x50 = mine[g], x95 = mine[GW + g];
  uint32_t lt50 = 0, lt95 = 0;
  for (uint32_t i = 0; ballot(i < n50 || i < n95); i += 4) {
    const uint4 y = *reinterpret_cast<const uint4*>(mine + (i & (GW - 1))), z = *reinterpret_cast<const uint4*>(mine + GW + (i & (GW - 1)));
    lt50 += (y.x < x50 ? 1u : 0u) + (y.y < x50 ? 1u : 0u) + (y.z < x50 ? 1u : 0u) + (y.w < x50 ? 1u : 0u);
    lt95 += (z.x < x95 ? 1u : 0u) + (z.y < x95 ? 1u : 0u) + (z.z < x95 ? 1u : 0u) + (z.w < x95 ? 1u : 0u);
  }
  v50 = group_max<GW>(g < n50 && lt50 <= r50.rank ? x50 : 0u);
  v95 = group_max<GW>(g < n95 && lt95 <= r95.rank ? x95 : 0u);
}

struct Picked {
  uint32_t count, min, max, p50, p95;   // (all 0 without samples)
  uint64_t sum;
};

// Everything about the samples v[0 .. n) of the group, by one wave.  hist: this wave's PICK_HIST words.  All 64 lanes call; the
// result is in all lanes of the group.
template <int GW>
__device__ __forceinline__ Picked pick_group(const uint32_t* v, uint32_t n, uint32_t least, uint32_t most, uint32_t* hist) {
  const uint32_t lane = lane_id(), g = lane & (GW - 1);
  uint32_t* mine = hist + 4 * (lane - g);     // the group's bins, later its two lists
  clear_hist(hist);
  LaneTally lane_tally;
  each_sample<GW>(v, n, least, most, [&](uint32_t x) { lane_tally.add(x); });
  const Tally t = lane_tally.of_group<GW>();
  const Window<GW> win = window_of<GW>(t);
  add_first(win, v, n, least, most, mine);
  __builtin_amdgcn_wave_barrier();
  Range r50, r95;
  first_ranges(win, hist, t.count, r50, r95);
  while (ballot(r50.wide(GW) || r95.wide(GW))) {
    clear_hist(hist);
    add_cut<GW>(r50, r95, v, n, least, most, mine);
    __builtin_amdgcn_wave_barrier();
    narrow<GW>(hist, r50, r95);
  }
  Picked out;
  out.count = t.count; out.sum = t.sum;
  out.min = win.min;
  out.max = win.max;
  out.p50 = r50.lo;
  out.p95 = r95.lo;
  if (ballot(r50.width || r95.width) == 0) return out;
  clear_lists<GW>(hist);
  add_lists<GW>(r50, r95, v, n, least, most, mine);
  __builtin_amdgcn_wave_barrier();
  uint32_t v50, v95;
  rank_lists<GW>(mine, r50, r95, v50, v95);
  if (r50.width) out.p50 = v50;
  if (r95.width) out.p95 = v95;
  return out;
}

}  // namespace fikit
