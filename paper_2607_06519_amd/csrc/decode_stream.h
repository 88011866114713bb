// Streaming split-K decode over a bf16 compressed cache (Section 3: the
// reconstruction of Eq. 3 fused into the attention).
//
// A chunk is 512 tokens of one (sequence, KV head), taken by one workgroup of
// 4 waves: a wave walks 128 tokens in 8-row tiles (d = 128; 16 rows at d = 64)
// with an online softmax, keeping the next tiles' loads in flight while it
// computes the current one.  The waves take the workgroup's tiles in turn (tile
// t of wave w: tile 4t + w), so at any time they read one short run of each
// plane; the rows of a token-level set are taken afterwards by the wave whose
// consecutive tokens hold them.
//
// Every call splits its tokens over chunks and waves in this one way, whatever
// its batch, its bound on the lengths or its workspace: a probability is rounded
// to bf16 against the reference max that its wave has reached, so another split
// would give other bits (2e-3 of an output's norm, for the same error against
// exact arithmetic).
//
// One lane layout serves the K pass, the softmax and the V pass: NP = d/8
// lanes per token row, each holding one 16-byte piece (8 channels), so one
// load instruction covers RPL = 64/NP consecutive rows and a lane owns
// NL = TILE/RPL rows of a tile (two).  The NP lanes of a row form a DPP row (d = 128)
// or half row (d = 64).
//  K   - bf16 dot2 of the lane's piece with its piece of every query (held in
//        registers); residual heads add the lane's residual entry
//        w * q[c] * value (B = 2: c the channel, w = +-1 for the stored half
//        difference; B = 4: code 4c + j, w = F_4[j][p] for layer p of the
//        block); a DPP reduce-scatter over the row's lanes then leaves each
//        lane one full (row, head) logit (2G <= NP: d = 128, or d = 64 with
//        G <= 4; d = 64 with G = 8 sums every logit on every lane instead);
//  max - a running reference max per head, equal on the lanes of that head,
//        that moves (the head's max over the wave, rescale by
//        exp2(m_old - m_new)) only when a logit exceeds it by more than 2^8;
//        scale, mask, exp2 and running sum run once per logit;
//  V   - each lane's probability goes back to the row as a bf16 pair (the
//        same head's other row) and an all-gather over the heads, so nothing
//        goes through LDS; the lane's two rows share one dot2 that
//        multiplies two tokens' values by their probabilities; residual heads add
//        w * p * value into LDS accumulators, one copy per row of a load
//        (a row's entries sit on distinct channels for B = 2, so a plain
//        read-add-write is safe; for B = 4 up to three frequencies of one
//        channel sit in adjacent lanes, since codes 4c + j are stored
//        ascending: a DPP pass hands each run's sum to its first lane and
//        only that lane writes, which keeps the adds plain as well -- LDS
//        float atomics tripled the layer time).
// The waves merge in LDS and write one (acc, m, l) record per workgroup;
// decode_merge combines the records.  HBM bound: no MFMA.
//
// What a workgroup spends outside its walk counts too (s_memrealtime stamps at
// 1001 tokens, 8B shape, before the following: unit scalars known 1.3 us after
// the start, first tiles requested at 2.3 us, merge and record 1.9 us).  So the
// launch constants are read in one go and kept in scalar registers, indices are
// divided by multiplication (divu.h), plane sizes are 32-bit, each residual
// flavour computes only its own planes, the wave index is scalar (the tile tests
// are uniform), a move of the reference max crosses rows with permlane swaps, and
// the merge takes two channels a thread from every copy instead of shuffling the
// copies together first.  Per layer (split-K and merge, graph replay): 1001
// tokens 18.2 -> 15.6 us, 32768 tokens 31.3 -> 29.1 us.  (A call of few chunks is bound by the chain of a wave's
// sixteen tiles, some 0.6 us each: a workgroup per wave, which keeps the bits,
// takes 14.9 us at 1001 tokens and 18.7 against 17.0 at 12288, whatever the
// tiles in flight.)
#pragma once

#include "decode_shape.h"
#include "fdkv_common.h"
#include "fdkv_kernels.h"

#include <type_traits>

namespace fdkv {

namespace {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
constexpr int kRsrcDword3 = 0x00020000;  // raw buffer, 32-bit data format (gfx9 family)
constexpr float kSlack = 8.f;            // log2 headroom of the running reference max
constexpr uint32_t kOob = 0x80000000u;   // buffer offset past every plane (planes are < 2^31 bytes): loads read 0

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c,
                                         false);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, uint64_t bytes) {
  const uint32_t n = bytes > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, n, kRsrcDword3);
}

__device__ __forceinline__ uint4 ld128(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// The K and V tile loads and the residual entries: every byte of a plane is
// read once per decode step, so they carry the non-temporal cache hint
// (cache policy NT).
constexpr int kNonTemporal = 2;
__device__ __forceinline__ uint4 ld128_stream(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kNonTemporal);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ uint32_t word(const uint4& v, int w) {
  return w == 0 ? v.x : w == 1 ? v.y : w == 2 ? v.z : v.w;
}

typedef __bf16 bf16x2v_t __attribute__((ext_vector_type(2)));

// Two FP8 E4M3 codes (bytes 0-1 or 2-3 of w) as a bf16 pair; exact, since
// every E4M3 value is a bf16 value.
template <bool HI>
__device__ __forceinline__ uint32_t e4m3x2_bf16(uint32_t w) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HI));
}

// A piece of 8 FP8 channels (raw in .x, .y) as the 8 bf16 channels of a
// bf16 piece.
__device__ __forceinline__ uint4 widen_e4m3(const uint4& raw) {
  return make_uint4(e4m3x2_bf16<false>(raw.x), e4m3x2_bf16<true>(raw.x), e4m3x2_bf16<false>(raw.y),
                    e4m3x2_bf16<true>(raw.y));
}

// Runs of equal channels among the residual V entries of one row (blocks of
// four: codes 4c + j ascending, so a channel's frequencies are adjacent
// entries, at most three).  Lane pc holds entry e with channel c and
// contribution x; entries e - 1, e + 1, e + 2 sit in lanes pc - 1, pc + 1,
// pc + 2 of the same group of NP lanes when they exist (ok1 / ok2 say whether
// e + 1 / e + 2 exist).  Returns the run's sum on the run's first lane.
template <int NP>
__device__ __forceinline__ float run_sum(int c, float x, int pc, bool valid, bool ok1, bool ok2, bool& first) {
  constexpr int kRowShr1 = 0x111, kRowShl1 = 0x101, kRowShl2 = 0x102;
  const int cl = __builtin_amdgcn_update_dpp(-1, c, kRowShr1, 0xF, 0xF, false);
  const int c1 = __builtin_amdgcn_update_dpp(-1, c, kRowShl1, 0xF, 0xF, false);
  const int c2 = __builtin_amdgcn_update_dpp(-1, c, kRowShl2, 0xF, 0xF, false);
  const float x1 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kRowShl1, 0xF, 0xF, false));
  const float x2 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kRowShl2, 0xF, 0xF, false));
  first = valid && (pc == 0 || cl != c);
  const bool n1 = ok1 && pc + 1 < NP && c1 == c;
  const bool n2 = n1 && ok2 && pc + 2 < NP && c2 == c;
  return x + (n1 ? x1 : 0.f) + (n2 ? x2 : 0.f);
}

// Lane exchange across bit B of a row's lane index (rows of 8 or 16 lanes).
// Bits 3 and 2 use the mirrors, which also flip the lower bits: that still
// pairs each lane with one of the other half, and once the lower bits hold
// equal values (duplicates, or lists already gathered) it is the plain swap.
template <int B>
__device__ __forceinline__ uint32_t swap_bit(uint32_t x) {
  constexpr int kCtrl = B == 3 ? kDppRowMirror : B == 2 ? kDppRowHalfMirror : B == 1 ? kDppQuadXor2 : kDppQuadXor1;
  // every source lane lies in the row: bound_ctrl needs no old value
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, 0xF, 0xF, true);
}
template <int B>
__device__ __forceinline__ float swap_bit(float x) {
  return __uint_as_float(swap_bit<B>(__float_as_uint(x)));
}

// The lane NP/2 further along a row of NP lanes (the lane holding the same
// head for the other row of a load): row_ror:8 for 16 lanes; for 8 lanes,
// row_shl:4 into banks 0 and 2 and row_shr:4 into banks 1 and 3.
template <int NP>
__device__ __forceinline__ float swap_half(float x) {
  if constexpr (NP == 16) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, true));
  } else {
    static_assert(NP == 8, "row width");
    int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x104, 0xF, 0x5, false);
    y = __builtin_amdgcn_update_dpp(y, __float_as_int(x), 0x114, 0xF, 0xA, false);
    return __int_as_float(y);
  }
}

// Max over the rows of a load (groups of NP lanes), lane by lane of a row.
template <int NP>
__device__ __forceinline__ float rows_max(float x) {
  if constexpr (NP == 8) x = fmaxf(x, swap_half<16>(x));  // the two groups of a DPP row
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// One reduce-scatter stage across lane bit B: the lanes with the bit clear
// keep the list's lower half and add their partner's copy of it, the others
// the upper half.
template <int B, int H, int V>
__device__ __forceinline__ void scatter_stage(float (&a)[V], int lane) {
  const bool up = (lane >> B) & 1;
#pragma unroll
  for (int t = 0; t < H; ++t) {
    const float keep = up ? a[t + H] : a[t], send = up ? a[t] : a[t + H];
    a[t] = keep + swap_bit<B>(send);
  }
}

// Sum of V values over the 2^NPB lanes of a row, one sum per lane: the
// stages on the top log2(V) lane bits split the list (lane bits b, from the
// top, choose the half), butterflies on the lower bits finish the sums, so
// the lane holds value number (lane % 2^NPB) >> (NPB - log2 V).
template <int NPB, int V>
__device__ __forceinline__ float row_reduce_scatter(float (&a)[V], int lane) {
  constexpr int RB = V == 16 ? 4 : V == 8 ? 3 : V == 4 ? 2 : 1;
  static_assert((1 << RB) == V && RB <= NPB, "one value per lane at most");
  scatter_stage<NPB - 1, V / 2>(a, lane);
  if constexpr (RB >= 2) scatter_stage<NPB - 2, V / 4>(a, lane);
  if constexpr (RB >= 3) scatter_stage<NPB - 3, V / 8>(a, lane);
  if constexpr (RB >= 4) scatter_stage<NPB - 4, V / 16>(a, lane);
  if constexpr (NPB - RB - 1 >= 2) a[0] += swap_bit<2>(a[0]);
  if constexpr (NPB - RB - 1 >= 1) a[0] += swap_bit<1>(a[0]);
  if constexpr (NPB - RB - 1 >= 0) a[0] += swap_bit<0>(a[0]);
  return a[0];
}

// All-gather stage across lane bit B: the list of N values doubles, the
// values of lanes with the bit clear first.
template <int B, int N, int G>
__device__ __forceinline__ void gather_stage(uint32_t (&y)[G], int lane) {
  const bool up = (lane >> B) & 1;
  uint32_t o[N];
#pragma unroll
  for (int t = 0; t < N; ++t) o[t] = swap_bit<B>(y[t]);
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const uint32_t mine = y[t];
    y[t] = up ? o[t] : mine;
    y[t + N] = up ? mine : o[t];
  }
}

// Every lane of a row gets the G values x of head g = (lane >> SH) % G (lanes
// that differ only below bit SH hold equal values).
template <int SH, int G>
__device__ __forceinline__ void row_gather(uint32_t x, uint32_t (&y)[G], int lane) {
  y[0] = x;
  if constexpr (G >= 2) gather_stage<SH, 1>(y, lane);
  if constexpr (G >= 4) gather_stage<SH + 1, 2>(y, lane);
  if constexpr (G >= 8) gather_stage<SH + 2, 4>(y, lane);
}

template <int D, int G>
struct SS {
  static constexpr int NP = D / 8;                 // lanes per row, one 16-byte piece each
  static constexpr int RPL = 64 / NP;              // rows per load instruction
  // d = 128: 8-row tiles (two rows per lane).  Each wait is for 4 KB of K
  // and V instead of 8 KB, and with eight query heads the per-row logits and
  // tile buffers leave room for two waves per SIMD; d = 64 keeps 16 rows
  // (two rows per lane there too)
  static constexpr int TILE = D == 128 ? 8 : 16;
  static constexpr int NL = TILE / RPL;            // rows of a tile per lane
  static constexpr int W = kDecodeWaves;           // waves of the workgroup, which take its tiles in turn
  static constexpr int CW = kDecodeChunk;          // tokens per wave
  static constexpr int NT = CW / TILE;             // tiles per wave
  static constexpr int RS = D + 4;
  // tiles in flight behind the current one: dense heads, and residual heads
  // with one entry per lane
  static constexpr int PD0 = 2;
  static constexpr int PD1 = 1;
  // accumulators of the workgroup's merge (floats), one copy per row of a
  // load of each wave; residual heads add their V entries to them
  static constexpr int SP = W * RPL * G * D;
  static constexpr int NPB = NP == 16 ? 4 : 3;     // log2 NP
  // the NL x G logits of a lane's rows fit one per lane of the row: the
  // softmax runs on a reduce-scatter of them (lane v << SH holds row v / G,
  // head v % G)
  static constexpr bool SCATTER = NL == 2 && NL * G <= NP;
  static constexpr int SH = SCATTER ? NPB - (G == 8 ? 4 : G == 4 ? 3 : G == 2 ? 2 : 1) : 0;
  static_assert(NL == 2 && CW % TILE == 0 && RPL * NP == 64, "shape");
};

template <int NL>
struct TileBuf {
  uint4 k[NL], v[NL];
  // the lane's first residual entry in each of its rows: index and value
  uint32_t ki[NL], kv[NL], vi[NL], vv[NL];
  uint32_t tm;  // token-level residual set: the tile's word of the token mask
};

}  // namespace

// Bit h of the result: byte h of four mode bytes says residual (whatever its fraction).
__device__ __forceinline__ uint32_t residual_bytes(uint32_t m) {
  uint32_t r = 0;
#pragma unroll
  for (int h = 0; h < 4; ++h) r |= ((m >> (8 * h)) & 0xE3u) == (uint32_t)kResidual ? 1u << h : 0u;
  return r;
}

// MULTI: the call has several parts (spans and the exact tail); otherwise
// part 0 is the only one, a compile-time constant, so the per-unit scalars
// load straight from fixed argument offsets with no lookup in front.
template <int D, int G, bool C8K, bool MULTI>
__global__ __launch_bounds__((64 * SS<D, G>::W)) void decode_stream_kernel(DecodeParams P) {
  using S = SS<D, G>;
  constexpr int NTH = 64 * S::W;
  constexpr int NP = S::NP, RPL = S::RPL, TILE = S::TILE, NL = S::NL, CW = S::CW, W = S::W;
  constexpr uint32_t RB = D * 2;
  __shared__ float q_lds[D * G];                        // [c][g] fp32: residual K gathers
  __shared__ __attribute__((aligned(16))) float big[S::SP];
  __shared__ __attribute__((aligned(16))) float m_lds[G][W], l_lds[G][W][RPL];
  auto sp = [&](int w, int cp, int g, int c) -> float& { return big[((w * RPL + cp) * G + g) * D + c]; };

  // % W tells the compiler the wave's range, which readfirstlane hides (28.4 ->
  // 28.2 us a layer on the 8B shape at 32768 tokens)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % W, lane = threadIdx.x & 63;
  // every argument of a one-part call, fetched in one go and kept (left to
  // itself the compiler reads some of them again, tile by tile)
  uint32_t n_slots = (uint32_t)P.n_chunks_total;
  int hkv = P.hkv, n_blocks = P.n_blocks, block = P.block, hq = P.hq, pos = P.pos, nb = P.bsize, k = P.topk;
  float scale_log2 = P.scale_log2, w1 = P.wres[0], w2 = P.wres[1], w3 = P.wres[2];
  const void* q_all = P.q;
  float* ws = P.ws;
  DivU by_chunks = P.by_chunks, by_hkv = P.by_hkv;
  asm volatile("" : "+s"(by_chunks.mul), "+s"(by_chunks.shift), "+s"(by_hkv.mul), "+s"(by_hkv.shift), "+s"(n_slots), "+s"(hkv),
               "+s"(n_blocks), "+s"(block), "+s"(q_all), "+s"(ws), "+s"(hq), "+s"(pos), "+s"(nb), "+s"(k));
  asm volatile("" : "+s"(scale_log2), "+s"(w1), "+s"(w2), "+s"(w3));
  DecodePart pt = P.part[0];
  if constexpr (!MULTI) asm volatile("" : "+s"(pt.lens), "+s"(pt.cache), "+s"(pt.modes), "+s"(pt.seg_off));
  const uint32_t bx = blockIdx.x;
  const uint32_t pair = by_chunks.div(bx);           // (sequence, rank of the KV head)
  const int slot = (int)(bx - pair * n_slots);
  const int seq = (int)by_hkv.div(pair);
  const int rank = (int)pair - seq * hkv;
  const int part = MULTI ? decode_part(P, slot) : 0;
  if constexpr (MULTI) pt = P.part[part];
  const int wgc = MULTI ? slot - P.part_base[part] : slot;
  const bool tail = MULTI && part == P.tail_part;
  // The per-unit values (mode, segment offset, length) are fetched together,
  // as scalar loads that wait on nothing but the arguments, so the start-up
  // costs one round trip that does not queue behind other waves' tile loads.
  // Modes are read through the aligned words of the array (4-byte aligned and
  // padded to a multiple of 4 bytes).  A segment offset is a multiple of 256
  // and a mode is at most kExact; a unit that breaks either reads nothing and
  // writes a record that turns its query heads' outputs into NaN.  (The exact
  // tail of a generation has no unit arrays: its rows are exact.)
  const int T = as_const(pt.lens)[seq];
  int head = rank;
  uint32_t mode_word = (uint32_t)kExact;
  uint64_t seg_off = 0;
  if (!tail) {
    const uint64_t u0 = ((uint64_t)seq * n_blocks + block) * hkv;
    const auto* mw = as_const(reinterpret_cast<const uint32_t*>(pt.modes));
    const auto* so = as_const(pt.seg_off) + u0;
    if (hkv <= 8) {
      // Workgroups are dispatched in index order, and the older of the waves
      // sharing a SIMD are served first, so the heads of a sequence are taken
      // in cost order: residual heads (the most bytes per token) first, then
      // the others, each group in head order.  (More than 8 KV heads keep the
      // head order.)  Heads past the last repeat the
      // last one's loads, which keeps the loads free of branches.
      const int hl = hkv - 1;
      const uint64_t w0 = u0 >> 2, w1 = (u0 + hl) >> 2;
      const uint32_t a = mw[w0], b = mw[min(w0 + 1, w1)], c = mw[min(w0 + 2, w1)];
      uint64_t offs[8];
#pragma unroll
      for (int h = 0; h < 8; ++h) offs[h] = so[min(h, hl)];
      asm volatile("" ::"s"(T), "s"(a), "s"(b), "s"(c), "s"(offs[0]), "s"(offs[1]), "s"(offs[2]), "s"(offs[3]),
                   "s"(offs[4]), "s"(offs[5]), "s"(offs[6]), "s"(offs[7]));
      const uint32_t sft = 8 * (uint32_t)(u0 & 3);
      // modes of heads 0-3 and 4-7, a byte each
      const uint32_t m0 = (uint32_t)((((uint64_t)b << 32) | a) >> sft), m1 = (uint32_t)((((uint64_t)c << 32) | b) >> sft);
      const uint32_t all = (2u << hl) - 1u;
      const uint32_t rmask = (residual_bytes(m0) | residual_bytes(m1) << 4) & all;
      const int nr = __builtin_popcount(rmask);
      uint32_t sel = rank < nr ? rmask : ~rmask & all;
      for (int i = rank < nr ? rank : rank - nr; i > 0; --i) sel &= sel - 1u;  // drop the lower set bits
      head = __builtin_ctz(sel);
      mode_word = (head < 4 ? m0 : m1) >> (8 * (head & 3));
#pragma unroll
      for (int h = 0; h < 8; ++h) seg_off = h == head ? offs[h] : seg_off;
    } else {
      const uint64_t unit = u0 + rank;
      mode_word = mw[unit >> 2];
      seg_off = so[rank];
      asm volatile("" ::"s"(T), "s"(mode_word), "s"(seg_off));
      mode_word >>= 8 * (uint32_t)(unit & 3);
    }
  }
  const int sh = seq * hkv + head;   // the (sequence, KV head) of the record slots
  const uint32_t mbyte = mode_word & 0xFFu;
  const int mode = mode_of(mbyte);
  const int tok0 = wgc * kDecodeWgTokens;  // the chunk's first token
  float* rec = ws + ((uint64_t)sh * n_slots + slot) * G * S::RS;
  const bool bad_unit = !unit_byte_ok(mbyte, P.tokres ? P.n_rates : 0) || (seg_off & 255) != 0;
  if (tok0 >= T || bad_unit) {
    // no tokens here: an empty record, m = -inf, l = 0, acc = 0, since the
    // merge reads every slot; an invalid unit: m = 0, l = 1, acc = NaN, which
    // the merge carries into every output channel of the KV head's queries
    for (int i = threadIdx.x; i < G * S::RS; i += NTH) {
      const int c = i % S::RS;
      rec[i] = bad_unit ? (c == D ? 0.f : c == D + 1 ? 1.f : __builtin_nanf("")) : (c == D ? -INFINITY : 0.f);
    }
    return;
  }

  // residual heads hold either per-token channel entries or a token-level set
  const bool tokres = P.tokres && mode == kResidual;
  const bool resid = !P.tokres && (mode == kResidual) && k > 0;
  // FP8 caches: the shared planes and residual values of shared / residual
  // heads are E4M3 (one byte per channel); exact heads stay bf16
  const bool c8 = C8K && mode != kExact;
  const uint8_t* seg = pt.cache + seg_off;
  // Bytes of the planes a tile reads (below 2^31: 32-bit arithmetic), FP8
  // shared planes in whole 1 KB blocks.  Shared planes: K, then V.  Exact
  // planes: K of the block's layers, then V of its layers.
  const uint32_t dense = c8 ? ((uint32_t)T * D + kC8Block - 1) / kC8Block * kC8Block : (uint32_t)T * RB;
  const uint32_t plane = (dense + kPlaneAlign - 1) / kPlaneAlign * kPlaneAlign;
  const uint32_t kn = mode == kExact ? (uint32_t)pos : 0u, vn = mode == kExact ? (uint32_t)nb : 1u;
  const uint8_t* kbase = seg + (uint64_t)kn * plane;
  const uint8_t* vbase = kbase + (uint64_t)vn * plane;
  if (MULTI && tail) {
    const uint64_t tail_off = (uint64_t)sh * (uint64_t)P.tail_cap * RB;
    kbase = static_cast<const uint8_t*>(P.tail_k) + tail_off;
    vbase = static_cast<const uint8_t*>(P.tail_v) + tail_off;
  }
  const auto kr = rsrc(kbase, dense);
  const auto vr = rsrc(vbase, dense);
  const uint8_t* qbase = static_cast<const uint8_t*>(q_all) + ((uint64_t)seq * hq + (uint64_t)head * G) * RB;
  const auto qr = rsrc(qbase, (uint64_t)G * RB);

  const int rg = lane / NP, pc = lane % NP;  // row of a load, piece of the row
  // the lane's piece of every query, for the whole kernel
  uint4 qreg[G];
#pragma unroll
  for (int g = 0; g < G; ++g) qreg[g] = ld128(qr, (uint32_t)(g * RB + pc * 16));
  // the fp32 query for the residual gathers, read now and staged to LDS after
  // the first tiles have been requested (the waits are in issue order)
  constexpr int QPT = (D * G + NTH - 1) / NTH;
  uint32_t qraw[QPT];
#pragma unroll
  for (int j = 0; j < QPT; ++j) {
    const uint32_t i = threadIdx.x + NTH * j;
    qraw[j] = __builtin_amdgcn_raw_buffer_load_b16(qr, i < D * G ? i * 2 : kOob, 0, 0);
  }

  // the wave's CW consecutive tokens of a token-level set
  const int wtok0 = tok0 + wave * CW;

  float m[G], l[G], acc[G][8];
  // scattered softmax state: the reference max of the lane's head and the
  // running sum of its (row, head) logit (lanes of one head share ms)
  float ms = -INFINITY, ls = 0.f;
  const int s_row = ((lane % NP) >> S::SH) / G;  // the lane's row of the two (0 or 1)
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[g][c] = 0.f;
  }

  // The tile loop is specialised per residual flavour (RES: 0 none, 1 one
  // entry per lane (k = NP), 2 fewer, 4 more (the first two of a lane travel
  // ahead of their tile, others are loaded where they are used), 3 a
  // token-level set: the set's tokens are masked out of the tile loop and
  // taken afterwards in a pass of their own, rebuilt in full) so that every
  // load of a tile is
  // issued unconditionally (k other than NP with its entries loaded in turn where
  // they were used took, per layer of the 8B shape at 32768 tokens, 45.5 us at
  // k = 5 and 59.1 at k = 24, now 29.5 and 35.0; d = 64, k = 16 at 12345 tokens
  // 27.8, now 16.0): a tile past the wave's range takes the
  // out-of-range offset and reads zeros without touching memory.  With no
  // load behind a branch the compiler can wait for exactly the tile it needs
  // and leave the later tiles' loads in flight.
  auto run = [&](auto res_tag, auto c8_tag, auto q4_tag) {
    constexpr int RES = decltype(res_tag)::value;
    constexpr bool C8 = decltype(c8_tag)::value;  // FP8 planes and residual values
    constexpr bool Q4 = decltype(q4_tag)::value;  // block of four: uint16 codes 4c + j
    // planes of the residual entries (bytes below 2^31), after the shared ones
    constexpr bool ENT = RES == 1 || RES == 2 || RES == 4;
    const uint32_t ibytes = ENT ? (uint32_t)T * k * (Q4 ? 2 : 1) : 0, vbytes = ENT ? (uint32_t)T * k * (C8 ? 1 : 2) : 0;
    const uint32_t iplane = (ibytes + kPlaneAlign - 1) / kPlaneAlign * kPlaneAlign;
    const uint32_t vplane = (vbytes + kPlaneAlign - 1) / kPlaneAlign * kPlaneAlign;
    const uint8_t* ent = seg + 2 * (uint64_t)plane;
    const auto ikr = rsrc(ent, ibytes), vkr = rsrc(ent + iplane, vbytes);
    ent += (uint64_t)iplane + vplane;
    const auto ivr = rsrc(ent, ibytes), vvr = rsrc(ent + iplane, vbytes);
    // token-level residual set: token mask, running counts, rows of the set's tokens
    TokLayout Lt{};
    uint64_t tok_rows = 0;
    if constexpr (RES == 3) {
      const int ppm = unit_ppm(P.res_ppm, P.n_rates, P.rates_ppm, mbyte);
      Lt = tok_layout(mode, (uint64_t)T, D, ppm, 2, C8 ? 1 : 2, nb);
      tok_rows = residual_token_count((uint64_t)T, ppm) * (uint64_t)(nb - 1) * D * (C8 ? 1 : 2);
    }
    const auto tmr = rsrc(seg + Lt.mask, (uint64_t)(T + 31) / 32 * 4);
    const auto tcr = rsrc(seg + Lt.count, ((uint64_t)(T + kTokChunk - 1) / kTokChunk + 1) * 4);
    const auto hkr = rsrc(seg + Lt.hk, tok_rows);
    const auto hvr = rsrc(seg + Lt.hv, tok_rows);
    // channel and weight of a residual entry (the weight by bit masks: a
    // select chain here compiles to divergent branches)
    auto entry = [&](uint32_t ix, float& w) -> int {
      if constexpr (Q4) {
        const uint32_t j = ix & 3u;
        const uint32_t m1 = 0u - (uint32_t)(j == 1u), m2 = 0u - (uint32_t)(j == 2u), m3 = 0u - (uint32_t)(j == 3u);
        w = as_f32((as_u32(w1) & m1) | (as_u32(w2) & m2) | (as_u32(w3) & m3));
        return (int)(ix >> 2) & (D - 1);
      } else {
        w = w1;
        return (int)ix & (D - 1);
      }
    };

    constexpr int PD = (RES == 0 || RES == 3) ? S::PD0 : S::PD1, NB = PD + 1;
    // the lane's first and second entry of a row, past k: the out-of-range offset
    const uint32_t past0 = pc < k ? 0u : kOob, past1 = NP + pc < k ? 0u : kOob;
    // the wave's tile t: rows from row0(t), nt of them in the sequence
    // (interleaved over the waves: 1.1% off the 8B decode step against a
    // contiguous 128 tokens a wave)
    auto row0 = [&](int t) -> int { return tok0 + (t * W + wave) * TILE; };
    const int nt = tok0 + wave * TILE < T ? min(CW / TILE, (T - tok0 - wave * TILE + W * TILE - 1) / (W * TILE)) : 0;

    // FP8 planes: a tile is one 1 KB block, and the lane's 16-byte slot of it
    // holds its piece of both of its rows (rows rg and rg + RPL)
    static_assert(!C8 || (TILE * D == kC8Block && NL == 2 && RPL * 2 == TILE), "FP8 tile = one block");
    auto load = [&](int t, TileBuf<NL>& b) {
      // the offset bit that sends a tile past the wave's range out of bounds (a
      // uniform value that the compiler must not turn into a branch around
      // the loads)
      uint32_t out = t < nt ? 0u : kOob;
      asm("" : "+s"(out));
      const uint32_t r0 = (uint32_t)row0(t);
      if constexpr (RES == 3) b.tm = __builtin_amdgcn_raw_buffer_load_b32(tmr, ((r0 >> 5) * 4) | out, 0, 0);
      if constexpr (C8) {
        const uint4 w = ld128_stream(kr, (r0 * D + lane * 16) | out);
        b.k[0] = make_uint4(w.x, w.y, 0u, 0u);
        b.k[1] = make_uint4(w.z, w.w, 0u, 0u);
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const uint32_t row = r0 + i * RPL + rg;
        if constexpr (!C8) b.k[i] = ld128_stream(kr, (row * RB + pc * 16) | out);
        if constexpr (ENT) {
          const uint32_t e = RES == 1 ? row * NP + pc : row * k + pc, off = RES == 1 ? out : out | past0;
          b.ki[i] = Q4 ? __builtin_amdgcn_raw_buffer_load_b16(ikr, (e * 2) | off, 0, kNonTemporal)
                       : __builtin_amdgcn_raw_buffer_load_b8(ikr, e | off, 0, kNonTemporal);
          b.kv[i] = C8 ? __builtin_amdgcn_raw_buffer_load_b8(vkr, e | off, 0, kNonTemporal)
                       : __builtin_amdgcn_raw_buffer_load_b16(vkr, (e * 2) | off, 0, kNonTemporal);
        }
      }
      if constexpr (C8) {
        const uint4 w = ld128_stream(vr, (r0 * D + lane * 16) | out);
        b.v[0] = make_uint4(w.x, w.y, 0u, 0u);
        b.v[1] = make_uint4(w.z, w.w, 0u, 0u);
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const uint32_t row = r0 + i * RPL + rg;
        if constexpr (!C8) b.v[i] = ld128_stream(vr, (row * RB + pc * 16) | out);
        if constexpr (ENT) {
          const uint32_t e = RES == 1 ? row * NP + pc : row * k + pc, off = RES == 1 ? out : out | past0;
          b.vi[i] = Q4 ? __builtin_amdgcn_raw_buffer_load_b16(ivr, (e * 2) | off, 0, kNonTemporal)
                       : __builtin_amdgcn_raw_buffer_load_b8(ivr, e | off, 0, kNonTemporal);
          b.vv[i] = C8 ? __builtin_amdgcn_raw_buffer_load_b8(vvr, e | off, 0, kNonTemporal)
                       : __builtin_amdgcn_raw_buffer_load_b16(vvr, (e * 2) | off, 0, kNonTemporal);
        }
      }
    };

    // RES 4: the lane's second entries of one tile, loaded for the next tile as
    // soon as this one's are used (one set: two would cost the other flavours a
    // wave per SIMD; none with eight query heads, which have no registers left)
    constexpr bool X2 = RES == 4 && G < 8;
    const int rest = X2 ? 2 * NP : NP;  // first entry that is loaded where it is used
    uint32_t xki[NL], xkv[NL], xvi[NL], xvv[NL];
    auto second = [&](int t, auto v_tag, uint32_t (&ix)[NL], uint32_t (&val)[NL]) {
      constexpr bool V = decltype(v_tag)::value;
      uint32_t out = t < nt ? 0u : kOob;
      asm("" : "+s"(out));
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const uint32_t e = (uint32_t)(row0(t) + i * RPL + rg) * k + NP + pc, off = out | past1;
        ix[i] = Q4 ? __builtin_amdgcn_raw_buffer_load_b16(V ? ivr : ikr, (e * 2) | off, 0, kNonTemporal)
                   : __builtin_amdgcn_raw_buffer_load_b8(V ? ivr : ikr, e | off, 0, kNonTemporal);
        val[i] = C8 ? __builtin_amdgcn_raw_buffer_load_b8(V ? vvr : vkr, e | off, 0, kNonTemporal)
                    : __builtin_amdgcn_raw_buffer_load_b16(V ? vvr : vkr, (e * 2) | off, 0, kNonTemporal);
      }
    };

    auto compute = [&](int t, const TileBuf<NL>& b) {
      const int r0 = row0(t);
      float s[NL][G];
#pragma unroll
      for (int i = 0; i < NL; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const uint4 kp = C8 ? widen_e4m3(b.k[i]) : b.k[i];
          float a = 0.f;
#pragma unroll
          for (int w = 0; w < 4; ++w) a = dot2(word(kp, w), word(qreg[g], w), a);
          s[i][g] = a;
        }
      if constexpr (ENT) {
        auto add = [&](int i, uint32_t ix, uint32_t raw) {
          float w;
          const int c = entry(ix, w);
          const float v = w * bf16_to_f32((uint16_t)(C8 ? e4m3x2_bf16<false>(raw) : raw));
#pragma unroll
          for (int g = 0; g < G; ++g) s[i][g] = fmaf(q_lds[c * G + g], v, s[i][g]);
        };
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          if (RES != 2 || pc < k) add(i, b.ki[i], b.kv[i]);
          if constexpr (RES == 4) {
            if (X2 && NP + pc < k) add(i, xki[i], xkv[i]);
            const uint32_t rc = (uint32_t)min(r0 + i * RPL + rg, T - 1);
            for (int e0 = rest; e0 < k; e0 += NP) {
              const int e = e0 + pc;
              const uint32_t x = e < k ? rc * k + e : kOob, x2 = e < k ? 2 * (rc * k + e) : kOob;
              const uint32_t ix = Q4 ? __builtin_amdgcn_raw_buffer_load_b16(ikr, x2, 0, 0)
                                     : __builtin_amdgcn_raw_buffer_load_b8(ikr, x, 0, 0);
              const uint32_t raw = C8 ? __builtin_amdgcn_raw_buffer_load_b8(vkr, x, 0, 0)
                                      : __builtin_amdgcn_raw_buffer_load_b16(vkr, x2, 0, 0);
              if (e < k) add(i, ix, raw);
            }
          }
        }
        if constexpr (X2) second(t + 1, std::false_type{}, xki, xkv);
      }
      // probabilities of the lane's two rows per head as bf16 pairs (row 0
      // low), and as fp32 for the residual V entries
      uint32_t pp[G];
      float p[NL][G];
      if constexpr (S::SCATTER) {
        // Lane pc of the row ends up with the full logit of row s_row, head
        // (pc >> SH) % G, so the scale, the mask, the exp2 and the running sum
        // are taken once per logit rather than on every lane of the row.
        float a[NL * G];
#pragma unroll
        for (int i = 0; i < NL; ++i)
#pragma unroll
          for (int g = 0; g < G; ++g) a[i * G + g] = s[i][g];
        const float red = row_reduce_scatter<S::NPB>(a, lane);
        const int row = r0 + s_row * RPL + rg;
        const bool valid = row < T && (RES != 3 || ((b.tm >> (row & 31)) & 1u) == 0u);
        const float x = valid ? red * scale_log2 : -INFINITY;
        // The reference max moves only when some logit exceeds it by more than
        // kSlack (probabilities then stay below 2^kSlack); moving it takes the
        // head's max over the wave's rows and rescales the running sums.
        if (__ballot(x - ms > kSlack) != 0) {
          const float mt = rows_max<NP>(fmaxf(x, swap_half<NP>(x)));
          const float mn = fmaxf(ms, mt);
          const float al = (ms == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ms - mn);
          ls *= al;
          ms = mn;
#pragma unroll
          for (int g = 0; g < G; ++g) {
            // every lane of head g holds the same factor; lane g << SH is one
            const float alpha = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(al), g << S::SH));
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[g][c] *= alpha;
            if constexpr (ENT) {
#pragma unroll
              for (int cp = 0; cp < RPL; ++cp)
#pragma unroll
                for (int c = lane; c < D; c += 64) sp(wave, cp, g, c) *= alpha;
            }
          }
        }
        // masked rows: exp2(-inf) = 0; a token-level set can mask every row
        // of a tile before any logit has set the reference max, and
        // exp2(-inf - -inf) would be NaN
        const float pv = (RES == 3 && x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(x - ms);
        ls += pv;
        const float pq = swap_half<NP>(pv);  // the same head's other row
        row_gather<S::SH>(s_row == 0 ? cvt_bf16x2(pv, pq) : cvt_bf16x2(pq, pv), pp, lane);
        if constexpr (ENT) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            p[0][g] = bf16_lo(pp[g]);
            p[1][g] = bf16_hi(pp[g]);
          }
        }
      } else {
        float d = -INFINITY;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int row = r0 + i * RPL + rg;
          const bool valid = row < T && (RES != 3 || ((b.tm >> (row & 31)) & 1u) == 0u);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float x = group_sum<NP>(s[i][g]) * scale_log2;
            s[i][g] = valid ? x : -INFINITY;
            d = fmaxf(d, s[i][g] - m[g]);
          }
        }
        if (__ballot(d > kSlack) != 0) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            float mt = s[0][g];
#pragma unroll
            for (int i = 1; i < NL; ++i) mt = fmaxf(mt, s[i][g]);
            mt = rows_max<NP>(mt);
            const float mn = fmaxf(m[g], mt);
            const float alpha = (m[g] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m[g] - mn);
            l[g] *= alpha;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[g][c] *= alpha;
            if constexpr (ENT) {
#pragma unroll
              for (int cp = 0; cp < RPL; ++cp)
#pragma unroll
                for (int c = lane; c < D; c += 64) sp(wave, cp, g, c) *= alpha;
            }
            m[g] = mn;
          }
        }
#pragma unroll
        for (int i = 0; i < NL; ++i)
#pragma unroll
          for (int g = 0; g < G; ++g) {
            if constexpr (RES == 3)
              p[i][g] = s[i][g] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s[i][g] - m[g]);
            else
              p[i][g] = __builtin_amdgcn_exp2f(s[i][g] - m[g]);
            l[g] += p[i][g];
          }
#pragma unroll
        for (int g = 0; g < G; ++g) pp[g] = cvt_bf16x2(p[0][g], p[1][g]);
      }
      // P V over the dense plane: the lane's two rows share one dot2
      {
        const uint4 va = C8 ? widen_e4m3(b.v[0]) : b.v[0];
        const uint4 vb = C8 ? widen_e4m3(b.v[1]) : b.v[1];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t wa = word(va, w), wb = word(vb, w);
          const uint32_t lo = __builtin_amdgcn_perm(wb, wa, 0x05040100u);
          const uint32_t hi = __builtin_amdgcn_perm(wb, wa, 0x07060302u);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            acc[g][2 * w] = dot2(lo, pp[g], acc[g][2 * w]);
            acc[g][2 * w + 1] = dot2(hi, pp[g], acc[g][2 * w + 1]);
          }
        }
      }
      // residual V entries: the lanes of one row hold distinct channels and
      // each row of a load has its own accumulator copy, so a plain
      // read-add-write never collides (masked rows add p = 0)
      // (the lanes of a row take its entries NP at a time, all lanes in every
      // step: entries past k read nothing and write nothing)
      if constexpr (ENT) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          auto step = [&](int e, uint32_t ix, uint32_t raw) {
            float w;
            const int c = entry(ix, w);
            float v = w * bf16_to_f32((uint16_t)(C8 ? e4m3x2_bf16<false>(raw) : raw));
            const bool all = RES == 1;
            bool first = all || e < k;
            if constexpr (Q4) v = run_sum<NP>(c, v, pc, all || e < k, all || e + 1 < k, all || e + 2 < k, first);
            if (first) {
#pragma unroll
              for (int g = 0; g < G; ++g) sp(wave, rg, g, c) += p[i][g] * v;
            }
          };
          step(pc, b.vi[i], b.vv[i]);
          if constexpr (RES == 4) {
            if constexpr (X2) step(NP + pc, xvi[i], xvv[i]);
            const uint32_t rc = (uint32_t)min(r0 + i * RPL + rg, T - 1);
            for (int e0 = rest; e0 < k; e0 += NP) {
              const int e = e0 + pc;
              const uint32_t x = e < k ? rc * k + e : kOob, x2 = e < k ? 2 * (rc * k + e) : kOob;
              const uint32_t ix = Q4 ? __builtin_amdgcn_raw_buffer_load_b16(ivr, x2, 0, 0)
                                     : __builtin_amdgcn_raw_buffer_load_b8(ivr, x, 0, 0);
              step(e, ix, C8 ? __builtin_amdgcn_raw_buffer_load_b8(vvr, x, 0, 0)
                             : __builtin_amdgcn_raw_buffer_load_b16(vvr, x2, 0, 0));
            }
          }
        }
        if constexpr (X2) second(t + 1, std::true_type{}, xvi, xvv);
      }
    };

    // ring of PD + 1 tile buffers: PD tiles stay in flight behind the one
    // being computed
    TileBuf<NL> buf[NB];
#pragma unroll
    for (int i = 0; i < PD; ++i) load(i, buf[i]);
    if constexpr (X2) {
      second(0, std::false_type{}, xki, xkv);
      second(0, std::true_type{}, xvi, xvv);
    }
    if constexpr (ENT) {
      for (int x = lane * 4; x < RPL * G * D; x += 256)
        *reinterpret_cast<float4*>(&sp(wave, 0, 0, x)) = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int j = 0; j < QPT; ++j) {
        const int i = threadIdx.x + NTH * j;
        if (i < D * G) q_lds[(i % D) * G + i / D] = bf16_to_f32((uint16_t)qraw[j]);
      }
      __syncthreads();  // the whole workgroup shares one unit, hence one flavour
    }
    if constexpr (RES == 0) {
      // dense heads: the wave's tiles unrolled at compile time, so every wait
      // is for exactly the tile computed next
      constexpr int NT = S::NT;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t + PD < NT) load(t + PD, buf[(t + PD) % NB]);
        if (t < nt) compute(t, buf[t % NB]);
      }
    } else {
      for (int t = 0; t < nt; t += NB) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          if (S::NT > NB || j + PD < S::NT) load(t + j + PD, buf[(j + PD) % NB]);
          if (j == 0 || t + j < nt) compute(t + j, buf[j]);
        }
      }
    }

    if constexpr (S::SCATTER) {
      // back to values per head: the reference max, and on every lane its
      // row group's sum over both rows (the form the set pass and the merge take)
#pragma unroll
      for (int g = 0; g < G; ++g) m[g] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ms), g << S::SH));
      uint32_t lg[G];
      row_gather<S::SH>(__float_as_uint(ls + swap_half<NP>(ls)), lg, lane);
#pragma unroll
      for (int g = 0; g < G; ++g) l[g] = __uint_as_float(lg[g]);
    }

    if constexpr (RES == 3) {
      // The residual set's tokens among the wave's CW consecutive tokens (the
      // dense walk above skipped them whichever wave read their tile), RPL at a
      // time: the lanes of row group rg rebuild the rg-th one in full,
      // K~ = M + sum_f w_f H_f and V~ alike, and fold it into the online
      // softmax.  The first one's row in the set: the running count before the
      // wave's tokens.
      constexpr int NF = Q4 ? 3 : 1;
      static_assert(CW == kTokChunk, "a running count per wave");
      const uint32_t tw = (uint32_t)wtok0 >> 5;
      const bool in_a = wtok0 + (lane & 32) < T, in_b = wtok0 + 64 + (lane & 32) < T;
      const uint32_t wa = __builtin_amdgcn_raw_buffer_load_b32(tmr, in_a ? (tw + (lane >> 5)) * 4 : kOob, 0, 0);
      const uint32_t wb = __builtin_amdgcn_raw_buffer_load_b32(tmr, in_b ? (tw + 2 + (lane >> 5)) * 4 : kOob, 0, 0);
      const uint32_t base = __builtin_amdgcn_raw_buffer_load_b32(
          tcr, wtok0 < T ? ((uint32_t)wtok0 / kTokChunk) * 4 : kOob, 0, 0);
      const bool bit_a = (wa >> (lane & 31)) & 1u, bit_b = (wb >> (lane & 31)) & 1u;
      const uint64_t ba = __ballot(bit_a), bb = __ballot(bit_b);
      const int na = __builtin_popcountll(ba), nres = na + __builtin_popcountll(bb);
      int* lst = reinterpret_cast<int*>(&sp(wave, 0, 0, 0));  // the wave's own accumulators, not yet in use
      const uint64_t below = (1ull << lane) - 1ull;
      if (bit_a) lst[__builtin_popcountll(ba & below)] = lane;
      if (bit_b) lst[na + __builtin_popcountll(bb & below)] = 64 + lane;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const float wf[3] = {w1, w2, w3};
      for (int j0 = 0; j0 < nres; j0 += RPL) {
        const int j = j0 + rg;
        const bool ok = j < nres;
        const uint32_t row = (uint32_t)(wtok0 + (ok ? lst[j] : 0));
        const uint32_t hrow = (base + (uint32_t)j) * NF * D;  // element index of the token's first row
        uint4 mk, mv, hk[NF], hv[NF];
        if constexpr (C8) {
          const uint32_t o8 = (uint32_t)c8_piece_offset(row, pc, D);
          const auto a = __builtin_amdgcn_raw_buffer_load_b64(kr, ok ? o8 : kOob, 0, 0);
          const auto b2 = __builtin_amdgcn_raw_buffer_load_b64(vr, ok ? o8 : kOob, 0, 0);
          mk = widen_e4m3(make_uint4(a[0], a[1], 0u, 0u));
          mv = widen_e4m3(make_uint4(b2[0], b2[1], 0u, 0u));
#pragma unroll
          for (int f = 0; f < NF; ++f) {
            const uint32_t e = hrow + f * D + pc * 8;
            const auto x = __builtin_amdgcn_raw_buffer_load_b64(hkr, ok ? e : kOob, 0, 0);
            const auto y = __builtin_amdgcn_raw_buffer_load_b64(hvr, ok ? e : kOob, 0, 0);
            hk[f] = widen_e4m3(make_uint4(x[0], x[1], 0u, 0u));
            hv[f] = widen_e4m3(make_uint4(y[0], y[1], 0u, 0u));
          }
        } else {
          mk = ld128(kr, ok ? row * RB + pc * 16 : kOob);
          mv = ld128(vr, ok ? row * RB + pc * 16 : kOob);
#pragma unroll
          for (int f = 0; f < NF; ++f) {
            const uint32_t e = (hrow + f * D + pc * 8) * 2;
            hk[f] = ld128(hkr, ok ? e : kOob);
            hv[f] = ld128(hvr, ok ? e : kOob);
          }
        }
        float kf[8], vf[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int w = c >> 1;
          auto ch = [&](const uint4& v) { return (c & 1) ? bf16_hi(word(v, w)) : bf16_lo(word(v, w)); };
          kf[c] = ch(mk);
          vf[c] = ch(mv);
#pragma unroll
          for (int f = 0; f < NF; ++f) {
            kf[c] = fmaf(wf[f], ch(hk[f]), kf[c]);
            vf[c] = fmaf(wf[f], ch(hv[f]), vf[c]);
          }
        }
        float sres[G];
        float dmax = -INFINITY;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          float a = 0.f;
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const uint32_t qw = word(qreg[g], c >> 1);
            a = fmaf(kf[c], (c & 1) ? bf16_hi(qw) : bf16_lo(qw), a);
          }
          sres[g] = ok ? group_sum<NP>(a) * scale_log2 : -INFINITY;
          dmax = fmaxf(dmax, sres[g] - m[g]);
        }
        if (__ballot(dmax > kSlack) != 0) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float mn = fmaxf(m[g], rows_max<NP>(sres[g]));
            const float alpha = (m[g] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m[g] - mn);
            l[g] *= alpha;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[g][c] *= alpha;
            m[g] = mn;
          }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float pg = __builtin_amdgcn_exp2f(sres[g] - m[g]);  // rows past the set: exp2(-inf) = 0
          l[g] += pg;
#pragma unroll
          for (int c = 0; c < 8; ++c) acc[g][c] = fmaf(pg, vf[c], acc[g][c]);
        }
      }
    }
  };  // run

  using R0 = std::integral_constant<int, 0>;
  using R1 = std::integral_constant<int, 1>;
  using R2 = std::integral_constant<int, 2>;
  using R3 = std::integral_constant<int, 3>;
  using F = std::false_type;
  using Tr = std::true_type;
  using R4 = std::integral_constant<int, 4>;
  // residual heads: one entry per lane of a row (k = NP), fewer or more, by block size
  auto run_res = [&](auto c8_tag) {
    if (nb == 4) {
      if (k == NP)
        run(R1{}, c8_tag, Tr{});
      else if (k < NP)
        run(R2{}, c8_tag, Tr{});
      else
        run(R4{}, c8_tag, Tr{});
    } else {
      if (k == NP)
        run(R1{}, c8_tag, F{});
      else if (k < NP)
        run(R2{}, c8_tag, F{});
      else
        run(R4{}, c8_tag, F{});
    }
  };
  auto run_tok = [&](auto c8_tag) {
    if (nb == 4)
      run(R3{}, c8_tag, Tr{});
    else
      run(R3{}, c8_tag, F{});
  };
  if constexpr (C8K) {
    if (c8) {
      if (resid)
        run_res(Tr{});
      else if (tokres)
        run_tok(Tr{});
      else
        run(R0{}, Tr{}, F{});
    } else {
      run(R0{}, F{}, F{});  // exact heads
    }
  } else {
    if (resid)
      run_res(F{});
    else if (tokres)
      run_tok(F{});
    else
      run(R0{}, F{}, F{});
  }

  // The row groups of a load saw different rows: each lane writes its sums to
  // its row group's accumulator copy (onto the V entries of residual heads),
  // and the merge below adds all copies of the workgroup's waves.
#pragma unroll
  for (int g = 0; g < G; ++g) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float4* dst = reinterpret_cast<float4*>(&sp(wave, rg, g, pc * 8 + 4 * h));
      float4 v = make_float4(acc[g][4 * h], acc[g][4 * h + 1], acc[g][4 * h + 2], acc[g][4 * h + 3]);
      if (resid) {
        const float4 o = *dst;
        v = make_float4(v.x + o.x, v.y + o.y, v.z + o.z, v.w + o.w);
      }
      *dst = v;
    }
  }
  if (pc == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      l_lds[g][wave][rg] = l[g];
      if (rg == 0) m_lds[g][wave] = m[g];
    }
  }
  __syncthreads();
  // Two channels a thread: the copies of a wave, then the workgroup's waves.
  // The thread of channels 0 and 1 takes m and l too.
  for (int i = threadIdx.x; i < G * (D / 2); i += NTH) {
    const int g = i / (D / 2), c = 2 * (i % (D / 2));
    float M = -INFINITY, f[W];
#pragma unroll
    for (int w = 0; w < W; ++w) M = fmaxf(M, m_lds[g][w]);
#pragma unroll
    for (int w = 0; w < W; ++w) f[w] = merge_weight(m_lds[g][w], M);
    // sum over the waves of x(wave, copy)
    auto total = [&](auto x) {
      float o = 0.f;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        float y = 0.f;
#pragma unroll
        for (int cp = 0; cp < RPL; ++cp) y += x(w, cp);
        o = fmaf(f[w], y, o);
      }
      return o;
    };
    float2 v[W][RPL];
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
      for (int cp = 0; cp < RPL; ++cp) v[w][cp] = *reinterpret_cast<const float2*>(&sp(w, cp, g, c));
    float2 o;
    o.x = total([&](int w, int cp) { return v[w][cp].x; });
    o.y = total([&](int w, int cp) { return v[w][cp].y; });
    *reinterpret_cast<float2*>(&rec[g * S::RS + c]) = o;
    if (c == 0)
      *reinterpret_cast<float2*>(&rec[g * S::RS + D]) = make_float2(M, total([&](int w, int cp) { return l_lds[g][w][cp]; }));
  }
}

template <int D, int G>
static hipError_t launch_stream_g(const DecodeParams& P, hipStream_t s) {
  const dim3 grid((unsigned)P.batch * P.hkv * P.n_chunks_total), block(64 * SS<D, G>::W);
  if (P.n_parts > 1 || P.tail_part >= 0) {
    if (P.coef8)
      hipLaunchKernelGGL((decode_stream_kernel<D, G, true, true>), grid, block, 0, s, P);
    else
      hipLaunchKernelGGL((decode_stream_kernel<D, G, false, true>), grid, block, 0, s, P);
    return hipGetLastError();
  }
  if (P.coef8)
    hipLaunchKernelGGL((decode_stream_kernel<D, G, true, false>), grid, block, 0, s, P);
  else
    hipLaunchKernelGGL((decode_stream_kernel<D, G, false, false>), grid, block, 0, s, P);
  return hipGetLastError();
}

// The launches of one head dimension, each compiled in a file of its own.
template <int D>
hipError_t launch_stream(const DecodeParams& P, hipStream_t s);

#ifdef FDKV_STREAM_INSTANCES
template <int D>
hipError_t launch_stream(const DecodeParams& P, hipStream_t s) {
  switch (P.hq / P.hkv) {
    case 1: return launch_stream_g<D, 1>(P, s);
    case 2: return launch_stream_g<D, 2>(P, s);
    case 4: return launch_stream_g<D, 4>(P, s);
    default: return launch_stream_g<D, 8>(P, s);
  }
}
#endif

}  // namespace fdkv
