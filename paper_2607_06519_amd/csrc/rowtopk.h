// Wavefront top-k of a token row (Section 3, the sparse high-frequency
// residual of Eq. 3): the k channels of largest |fl32(x[l] - x[l+1])| of a
// row, ties to the lower channel, found by the lanes that hold the row.
//
// A row of d channels sits on LPR consecutive lanes (a DPP row or part of
// one; 32 lanes for fp32 rows of 128 channels).  A lane's CPL keys form H
// segments of S = CPL / H consecutive channels: key s S + c of lane j is
// channel s LPR S + j S + c (H = 1: lane j holds channels CPL j ..
// CPL j + CPL - 1; H = 2: a lane holds one run in each half of the row, so
// that loads of a segment over the row's lanes are contiguous).  Keys are
// the bit patterns of the non-negative fp32 magnitudes, which order like the
// values.
//
// The search runs on the keys' 16-bit prefixes.  Every lane of a row keeps the
// same bounds lo < hi with #(keys >= lo) >= k > #(keys >= hi), lo and hi
// multiples of 2^16, and halves [lo, hi).  The first lo is a key that k
// disjoint groups of keys all reach (1, 2 or 4 groups a lane: the smallest
// group maximum), the first hi the row maximum's successor.  The prefixes'
// distances from the first lo, saturated at 255, are bytes, four to a
// register: with S(m) = sum |q - m| over the keys, S(m - 1) - S(m) =
// 2 #(q >= m) - #keys, so two v_sad_u8 count four keys, where a compare and
// an add count one.  A row stops once the selection is every key >= lo, the
// bounds are neighbours, or at most three keys lie between them.  A row whose
// threshold lies past the 255 steps, or that has no first lo (k above four
// groups a lane), or that still holds more than three keys in a prefix goes on
// with the full keys, counted one by one.
//
// Then, of the keys in [lo, hi), the last one still needed is the largest (if
// one is needed) or the first one not needed is the smallest (if all but one
// are), found with one max reduction on keys (v_xad_u32 turns both into the
// same max); otherwise lo is the k-th key itself.  Where keys tie at the k-th,
// the first ones in channel order are taken (segment by segment, lanes in
// order within a segment).
// Returns the lane's selection as a CPL-bit mask.
#pragma once

#include "fdkv_common.h"

namespace fdkv {

#ifdef __HIPCC__

template <int LPR>
__device__ __forceinline__ uint32_t row_sum_u32(uint32_t x) {
  static_assert(LPR == 8 || LPR == 16 || LPR == 32, "row width");
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppQuadXor1, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppQuadXor2, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppRowHalfMirror, 0xF, 0xF, false);
  if constexpr (LPR >= 16) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppRowMirror, 0xF, 0xF, false);
  if constexpr (LPR == 32) x += (uint32_t)__shfl_xor((int)x, 16, 64);
  return x;
}

template <int LPR, bool MAX>
__device__ __forceinline__ uint32_t row_ext_u32(uint32_t x) {
  auto op = [](uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, kDppQuadXor1, 0xF, 0xF, false));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, kDppQuadXor2, 0xF, 0xF, false));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, kDppRowHalfMirror, 0xF, 0xF, false));
  if constexpr (LPR >= 16) x = op(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, kDppRowMirror, 0xF, 0xF, false));
  if constexpr (LPR == 32) x = op(x, (uint32_t)__shfl_xor((int)x, 16, 64));
  return x;
}

// Inclusive prefix sum over the row's lanes, in lane order (DPP row shifts
// inside each 16-lane DPP row; a row of 32 lanes adds the lower half's total
// through row_bcast:15; a row of 8 lanes masks the shifts at its boundary).
template <int LPR>
__device__ __forceinline__ uint32_t row_prefix_u32(uint32_t x) {
  static_assert(LPR == 8 || LPR == 16 || LPR == 32, "row width");
  const int lr = (int)(threadIdx.x & (LPR - 1));
  uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += (LPR != 8 || lr >= 1) ? y : 0u;
  y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);           // row_shr:2
  x += (LPR != 8 || lr >= 2) ? y : 0u;
  y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);           // row_shr:4
  x += (LPR != 8 || lr >= 4) ? y : 0u;
  if constexpr (LPR >= 16) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
  if constexpr (LPR == 32) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  return x;
}

// Keys of this lane's CPL channels >= x, summed over the row.
template <int LPR, int CPL>
__device__ __forceinline__ uint32_t row_count_ge(const uint32_t (&key)[CPL], uint32_t x) {
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < CPL; ++i) c += key[i] >= x ? 1u : 0u;
  return row_sum_u32<LPR>(c);
}

// sel = 2 sel + (key >= thr)
__device__ __forceinline__ void push_ge(uint32_t& sel, uint32_t key, uint32_t thr) {
  asm("v_cmp_ge_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(sel) : "v"(key), "v"(thr) : "vcc");
}

// The lane's selected keys (bit i: key i, the channel given above) of the k
// largest keys of its row, ties to the lower channel.  0 <= k <= d.
//
// VALU bound.  A wave of eight rows (8 lanes of 16 keys, k = 16) takes about
// 290 VALU instructions where a count of the full keys at every step took
// about 540: 8B probe at 32768 tokens 1035 -> 862 us, blocks of four (16 lanes
// of 24 keys) 854 -> 673 us for the Gram kernel at 12345 tokens.
template <int LPR, int CPL, int H = 1>
__device__ __forceinline__ uint32_t row_topk_mask(const uint32_t (&key)[CPL], int k) {
  static_assert(H >= 1 && CPL % H == 0 && CPL % 4 == 0 && CPL < 32, "segments, whole registers, one mask bit per key");
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  constexpr int S = CPL / H, NP = CPL / 2, NQ = CPL / 4, N = LPR * CPL;
  constexpr uint32_t kAll = (1u << CPL) - 1u;
  if (k <= 0) return 0u;
  if (k >= N) return kAll;
  // the prefixes, two to a register, and their maxima over the lane's four groups
  u16x2 p[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i)
    p[i] = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(key[2 * i + 1], key[2 * i], 0x07060302u));
  u16x2 ma = p[0], mb = p[NP / 2];
#pragma unroll
  for (int i = 1; i < NP / 2; ++i) {
    ma = __builtin_elementwise_max(ma, p[i]);
    mb = __builtin_elementwise_max(mb, p[NP / 2 + i]);
  }
  const u16x2 mh = __builtin_elementwise_max(ma, mb);
  const uint32_t lmax = max((uint32_t)mh.x, (uint32_t)mh.y);
  const uint32_t rmax = row_ext_u32<LPR, true>(lmax);
  uint32_t base = 0;
  if (k <= LPR) {
    base = row_ext_u32<LPR, false>(lmax);
  } else if (k <= 2 * LPR) {
    base = row_ext_u32<LPR, false>(min((uint32_t)mh.x, (uint32_t)mh.y));
  } else if (k <= 4 * LPR) {
    const u16x2 ml = __builtin_elementwise_min(ma, mb);
    base = row_ext_u32<LPR, false>(min((uint32_t)ml.x, (uint32_t)ml.y));
  }
  // q = min(prefix - base, 255) (0 below base), four to a register
  uint32_t q[NQ];
  {
    const u16x2 b2 = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(base, base, 0x01000100u));
    const u16x2 top = {255, 255};
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const u16x2 x = __builtin_elementwise_min(__builtin_elementwise_sub_sat(p[2 * j], b2), top);
      const u16x2 y = __builtin_elementwise_min(__builtin_elementwise_sub_sat(p[2 * j + 1], b2), top);
      q[j] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, y), __builtin_bit_cast(uint32_t, x), 0x06040200u);
    }
  }
  // Bounds and counts in steps from base; counts as 2 #(q >= m) - N.  The
  // count at lo = 0 is not taken: N bounds it.
  const int kd = 2 * k - N;
  int lo8 = 0, hi8 = (int)min(rmax - base + 1u, 256u), clo2 = N, chi2 = -N;
  auto step = [&]() {
    const int mid = max((lo8 + hi8) >> 1, 1);  // 1: bounds 0 and 1 count at 1 again
    const uint32_t m1 = __builtin_amdgcn_perm((uint32_t)mid, (uint32_t)mid, 0u), m0 = m1 - 0x01010101u;
    uint32_t s0 = 0, s1 = 0;
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      s0 = __builtin_amdgcn_sad_u8(q[j], m0, s0);
      s1 = __builtin_amdgcn_sad_u8(q[j], m1, s1);
    }
    const int c = (int)row_sum_u32<LPR>(s0 - s1);
    const bool up = c >= kd;
    lo8 = up ? mid : lo8;
    clo2 = up ? c : clo2;
    hi8 = up ? hi8 : mid;
    chi2 = up ? chi2 : c;
  };
  // A stopped row may take further steps: they keep the bounds' conditions.
  // (A wave of eight rows of the synthetic keys needs 5.9 steps, hardly ever
  // fewer than five.)
#pragma unroll
  for (int u = 0; u < 4; ++u) step();
  for (int u = 0; u < 5; ++u) {
    step();
    if (__ballot(clo2 != kd && hi8 - lo8 > 1 && clo2 - chi2 > 6) == 0) break;
  }
  uint32_t lo = (base + (uint32_t)lo8) << 16;
  uint32_t hi = (hi8 == 256 ? rmax + 1u : base + (uint32_t)hi8) << 16;
  uint32_t clo = (uint32_t)(clo2 + N) >> 1, chi = (uint32_t)(chi2 + N) >> 1;
  const uint32_t ku = (uint32_t)k;
  for (int round = 0; round < 20; ++round) {
    if (__ballot(clo != ku && hi - lo > 1u && clo - chi > 3u) == 0) break;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t mid = lo + ((hi - lo) >> 1);
      const uint32_t c = row_count_ge<LPR, CPL>(key, mid);
      const bool up = c >= ku;
      lo = up ? mid : lo;
      clo = up ? c : clo;
      hi = up ? hi : mid;
      chi = up ? chi : c;
    }
  }
  // the last key taken (one more is needed above hi), or the first one left
  // out (one too many at or above lo); otherwise every key >= lo
  const uint32_t need = ku - chi, ns = clo - chi;
  const bool take = clo != ku && need == 1u;
  const bool drop = clo != ku && !take && ns == need + 1u;
  uint32_t edge = lo, thr = lo;
  if (__ballot(take || drop) != 0) {
    // the largest key below hi is the largest key - hi in unsigned arithmetic,
    // the smallest key at or above lo the largest ~key + lo
    const uint32_t flip = drop ? 0xFFFFFFFFu : 0u, add = drop ? lo : 0u - hi;
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < CPL; i += 2) m = max(m, max((key[i] ^ flip) + add, (key[i + 1] ^ flip) + add));
    m = (row_ext_u32<LPR, true>(m) - add) ^ flip;
    edge = take || drop ? m : lo;
    thr = drop ? m + 1u : edge;
  }
  uint32_t sel = 0;
#pragma unroll
  for (int i = CPL - 1; i >= 0; --i) push_ge(sel, key[i], thr);
  const bool tied = row_sum_u32<LPR>((uint32_t)__builtin_popcount(sel)) != ku;  // keys equal to edge
  if (__ballot(tied) != 0) {
    // keys above edge, then the first equal keys in channel order
    uint32_t eq = 0;
#pragma unroll
    for (int i = 0; i < CPL; ++i) eq |= key[i] == edge ? 1u << i : 0u;
    const uint32_t gt = sel & ~eq;
    // rank of the lane's first equal key of each segment: the equal keys of
    // the row's earlier segments, then those of the segment's lower lanes
    int left = k - (int)row_sum_u32<LPR>((uint32_t)__builtin_popcount(gt));
    uint32_t s2 = gt;
#pragma unroll
    for (int sg = 0; sg < H; ++sg) {
      constexpr uint32_t kSeg = S == 32 ? ~0u : (1u << S) - 1u;
      uint32_t e = eq & (kSeg << (sg * S));
      const uint32_t n = (uint32_t)__builtin_popcount(e);
      const int mine = left - (int)(row_prefix_u32<LPR>(n) - n);  // how many of the lane's equal keys are taken
      while (__ballot(e != 0u && (int)__builtin_popcount(e) > mine) != 0)
        if ((int)__builtin_popcount(e) > mine) e &= ~(e == 0u ? 0u : 0x80000000u >> __builtin_clz(e));
      s2 |= e;
      if (sg + 1 < H) left -= (int)row_sum_u32<LPR>(n);
    }
    sel = tied ? s2 : sel;
  }
  return sel;
}

#endif  // __HIPCC__

}  // namespace fdkv
