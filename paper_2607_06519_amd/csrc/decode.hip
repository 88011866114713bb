// Decode attention over an fp32 compressed cache with the reconstruction
// fused in (Section 3, the paragraph after Eq. 3): shared coefficients are read
// once per token and the sparse residual is added only at its indexed
// channels; no reconstructed K/V is ever materialised.  (bf16 and FP8 caches:
// decode_stream.h.)
//
// For layer p of a block of B layers and the G query heads of a KV head:
//   shared   : K~ = MK,                             V~ = MV
//   residual : K~ = MK + sum_e w_e value_e at c_e,  V~ likewise
//   exact    : K~ = K_p,                            V~ = V_p
// where an entry e is a channel c_e with w_e = +1 (p = 0) or -1 (p = 1) for
// the stored half difference of a pair, or a code 4c_e + j with
// w_e = F_4[j][p] for a block of four.  Logits use the algebraic form
// q.K~ = q.MK + sum_e w_e q[c_e] value_e.
//
// A chunk of 512 tokens of one (sequence, KV head) is split over waves in the
// launch shapes of decode_shape.h (kFull: 4 waves of 128 tokens; the groups
// of a small call: 32 tokens a wave, 64 with eight query heads).  Each wave
// takes its tokens in two passes over HBM-resident planes:
//   K pass - 4 to 16 lanes per row read 16-byte pieces against the query pieces
//            held in registers, group reduction by DPP; logits (log2 domain) to
//            LDS.
//   V pass - one row per NP lanes, the probabilities read from LDS; the sparse
//            V residual goes into an LDS accumulator with ds_add_f32.
// The wave's max is exact (two passes), so no rescaling is needed inside a
// wave; the waves merge in LDS and the workgroup writes one (acc, m, l)
// record.  decode_merge (decode_stream.hip) merges the records of a
// sequence with the log-sum-exp rule.
//
// A small call is bound by the chain of loads: of a kSpread wave all K and V
// rows and the first residual entries are requested before the first is used.
// 4 heads of 64 channels, 512 tokens (graph replay, split-K and merge): 19.5 us
// with one workgroup per chunk and a load at a time -> 11.1 us; 8B shape, 512
// tokens 65.8 -> 23.3, 12288 tokens 75.7 -> 48.2, 32768 (kFull) 128 -> 126.
#include "decode_shape.h"
#include "fdkv_common.h"
#include "fdkv_kernels.h"

namespace fdkv {

namespace {

template <int D, int G, int SHAPE>
struct DecodeShape {
  static constexpr int NP = D / 4;               // 16-byte pieces per row
  // lanes per row in the K pass: at most 16 pieces of query a lane
  static constexpr int LPRK = G * NP <= 64 ? 4 : G * NP <= 128 ? 8 : 16;
  static constexpr int PK = NP / LPRK;           // pieces per lane in the K pass
  static constexpr int RPK = 64 / LPRK;          // rows per K pass step
  static constexpr int RPV = 64 / NP;            // rows per V load
  static constexpr int GW = kDecodeWaves, NGRP = SHAPE == kFull ? 1 : decode_groups(G);
  static constexpr int W = SHAPE == kWide ? GW * NGRP : GW;
  static constexpr int GT = kDecodeWgTokens / NGRP, CH = GT / GW;  // tokens of a group, of a wave
  static constexpr int KP = CH / RPK, VP = CH / RPV;               // steps of the passes
  // steps whose rows are in flight together (kSpread: up to 64 registers of each)
  static constexpr int KB = SHAPE != kSpread ? (PK <= 4 ? 2 : 1) : KP * PK <= 16 ? KP : 16 / PK;
  static constexpr int VB = SHAPE != kSpread ? 4 : VP < 16 ? VP : 16;
  static constexpr int ENT = SHAPE == kSpread ? 4 : 0;             // residual entries of a lane requested ahead
  static constexpr int RS = D + 4;               // partial record stride (floats)
  static_assert(LPRK <= 16 && PK >= 1 && KP % KB == 0 && VP % VB == 0 && CH % 32 == 0, "shape");
};

// The wave's LDS writes are visible to its later reads.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

template <int D, int G, int SHAPE>
__global__ __launch_bounds__((64 * DecodeShape<D, G, SHAPE>::W)) void decode_splitk_kernel(DecodeParams P) {
  using S = DecodeShape<D, G, SHAPE>;
  constexpr int NP = S::NP, LPRK = S::LPRK, PK = S::PK, RPK = S::RPK, RPV = S::RPV, CH = S::CH, W = S::W, GW = S::GW;
  constexpr int NTH = 64 * W, NSUB = SHAPE == kSpread ? S::NGRP : 1;
  __shared__ float q_lds[D * G];            // [c][g], for residual gathers
  __shared__ float s_lds[W][G][CH];         // logits, then probabilities
  __shared__ __attribute__((aligned(16))) float sp_lds[W][G][D];  // sparse V accumulator, then the wave's acc
  __shared__ float m_lds[W][G], l_lds[W][G];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t bx = blockIdx.x / NSUB, pair = P.by_chunks.div(bx);
  const int slot = (int)(bx - pair * (uint32_t)P.n_chunks_total);
  const int seq = (int)P.by_hkv.div(pair), head = (int)pair - seq * P.hkv;
  const int sh = (int)pair;                 // seq * hkv + head
  const int grp = SHAPE == kSpread ? (int)(blockIdx.x % NSUB) : wave / GW;
  const int part = decode_part(P, slot);
  const int wgc = slot - P.part_base[part];
  const bool tail = part == P.tail_part;
  const DecodePart pt = P.part[part];
  const int T = as_const(pt.lens)[seq];
  // the exact tail of a generation has no unit arrays; modes are read through
  // the aligned words of the array
  uint32_t mbyte = (uint32_t)kExact;
  uint64_t seg_off = 0;
  if (!tail) {
    const uint64_t unit = ((uint64_t)seq * P.n_blocks + P.block) * P.hkv + head;
    seg_off = as_const(pt.seg_off)[unit];
    mbyte = (as_const(reinterpret_cast<const uint32_t*>(pt.modes))[unit >> 2] >> (8 * (uint32_t)(unit & 3))) & 0xFFu;
  }
  const int mode = mode_of(mbyte);
  const int grp_tok0 = wgc * kDecodeWgTokens + grp * S::GT;
  const int wg_tok0 = SHAPE == kSpread ? grp_tok0 : wgc * kDecodeWgTokens;
  float* rec = P.ws + (((uint64_t)sh * P.n_chunks_total + slot) * NSUB + (SHAPE == kSpread ? grp : 0)) * G * S::RS;
  const bool bad_unit = !unit_byte_ok(mbyte, P.tokres ? P.n_rates : 0) || (seg_off & 255) != 0;
  if (wg_tok0 >= T || bad_unit) {  // uniform over the workgroup
    // an empty record (m = -inf, l = 0, acc = 0): the merge reads every slot;
    // an invalid unit (mode above exact or a misaligned segment) writes
    // m = 0, l = 1, acc = NaN, which turns its query heads' outputs into NaN
    for (int i = threadIdx.x; i < G * S::RS; i += NTH) {
      const int c = i % S::RS;
      rec[i] = bad_unit ? (c == D ? 0.f : c == D + 1 ? 1.f : __builtin_nanf("")) : (c == D ? -INFINITY : 0.f);
    }
    return;
  }

  const bool q4 = P.bsize == 4;
  const int k = P.topk;
  const bool resid = !P.tokres && (mode == kResidual) && k > 0;
  const bool tokres = P.tokres && mode == kResidual;   // token-level residual set
  const uint8_t* seg = tail ? static_cast<const uint8_t*>(P.tail_k) : pt.cache + seg_off;
  const SegLayout L = seg_layout(mode, (uint64_t)T, D, k, 4, 4, P.bsize);
  const uint64_t xplane = plane_bytes((uint64_t)T * D * 4);  // exact planes: K_p at p * xplane, V_p at (B + p) * xplane
  const uint64_t tail_off = (uint64_t)sh * (uint64_t)P.tail_cap * D * 4;
  const uint8_t* kplane = tail ? static_cast<const uint8_t*>(P.tail_k) + tail_off
                               : seg + (mode == kExact ? (uint64_t)P.pos * xplane : L.mk);
  const uint8_t* vplane = tail ? static_cast<const uint8_t*>(P.tail_v) + tail_off
                               : seg + (mode == kExact ? (uint64_t)(P.bsize + P.pos) * xplane : L.mv);
  // raw entry i of an index plane, and its channel and weight
  auto code_at = [&](const uint8_t* ip, uint64_t i) -> uint32_t {
    return q4 ? (uint32_t) reinterpret_cast<const uint16_t*>(ip)[i] : (uint32_t)ip[i];
  };
  const float wr0 = P.wres[0], wr1 = P.wres[1], wr2 = P.wres[2];
  auto entry = [&](uint32_t code, float& w) -> int {
    if (q4) {
      const uint32_t j = code & 3u;
      const uint32_t m1 = 0u - (uint32_t)(j == 1u), m2 = 0u - (uint32_t)(j == 2u), m3 = 0u - (uint32_t)(j == 3u);
      w = as_f32((as_u32(wr0) & m1) | (as_u32(wr1) & m2) | (as_u32(wr2) & m3));
      return (int)(code >> 2) & (D - 1);
    }
    w = wr0;
    return (int)code & (D - 1);
  };
  const uint8_t* ikp = seg + L.ik;
  const float* vkp = reinterpret_cast<const float*>(seg + L.vk);
  const uint8_t* ivp = seg + L.iv;
  const float* vvp = reinterpret_cast<const float*>(seg + L.vv);
  const uint8_t* qbase = static_cast<const uint8_t*>(P.q) + ((uint64_t)seq * P.hq + (uint64_t)head * G) * D * 4;
  const uint64_t RB = (uint64_t)D * 4;
  const float scale_log2 = P.scale_log2;

  const int wtok0 = grp_tok0 + (wave % GW) * CH;
  const int kr = lane / LPRK, ks = lane % LPRK;
  const int vr = lane / NP, vpc = lane % NP;
  // Rows past the sequence repeat its last one (their logits are masked).
  uint4 kv[S::KB][PK], vv[S::VB];
  auto load_k = [&](int p0) {
#pragma unroll
    for (int b = 0; b < S::KB; ++b) {
      const int rc = min(wtok0 + (p0 + b) * RPK + kr, T - 1);
      const uint4* src = reinterpret_cast<const uint4*>(kplane + (uint64_t)rc * RB);
#pragma unroll
      for (int j = 0; j < PK; ++j) kv[b][j] = src[j * LPRK + ks];
    }
  };
  auto load_v = [&](int i0) {
#pragma unroll
    for (int b = 0; b < S::VB; ++b) {
      const int rr = min(wtok0 + (i0 + b) * RPV + vr, T - 1);
      vv[b] = *reinterpret_cast<const uint4*>(vplane + (uint64_t)rr * RB + vpc * 16);
    }
  };
  // residual entries: K's of a row over its lanes, in runs of epl; V's of the
  // wave's tokens over all lanes
  const int epl = (k + LPRK - 1) / LPRK;
  const int e0 = ks * epl, e1 = min(k, e0 + epl);
  const int ne = CH * k, ne_live = min(ne, max(0, T - wtok0) * k);  // entries of the wave's tokens; of those in the sequence
  constexpr int ENT = S::ENT > 0 ? S::ENT : 1;
  uint32_t kc[S::KB][ENT], vc[ENT];
  float kx[S::KB][ENT], vx[ENT];
  auto ahead_k = [&](int p0) {
    if constexpr (S::ENT > 0) {
#pragma unroll
      for (int b = 0; b < S::KB; ++b) {
        const uint64_t rc = (uint64_t)min(wtok0 + (p0 + b) * RPK + kr, T - 1) * k;
#pragma unroll
        for (int i = 0; i < ENT; ++i) {
          const uint64_t e = rc + (e0 + i < e1 ? e0 + i : 0);
          kc[b][i] = code_at(ikp, e);
          kx[b][i] = e0 + i < e1 ? vkp[e] : 0.f;
        }
      }
    }
  };
  load_k(0);
  if (resid) {
    ahead_k(0);
    if constexpr (S::ENT > 0) {
#pragma unroll
      for (int i = 0; i < ENT; ++i) {
        const int e = lane + 64 * i;
        const uint64_t x = (uint64_t)min(wtok0, T - 1) * k + (e < ne_live ? e : 0);
        vc[i] = code_at(ivp, x);
        vx[i] = vvp[x];
      }
    }
  }
  if constexpr (SHAPE == kSpread) load_v(0);

  for (int i = threadIdx.x; i < D * G; i += NTH) {
    const int g = i / D, c = i % D;
    q_lds[c * G + g] = reinterpret_cast<const float*>(qbase)[(uint64_t)g * D + c];
  }
  for (int i = lane; i < G * D; i += 64) (&sp_lds[wave][0][0])[i] = 0.f;
  uint4 qr[G][PK];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int j = 0; j < PK; ++j)
      qr[g][j] = *reinterpret_cast<const uint4*>(qbase + (uint64_t)g * RB + (uint64_t)(j * LPRK + ks) * 16);
  __syncthreads();

  // ------------------------------------------------------------ K pass
  float mx[G];
#pragma unroll
  for (int g = 0; g < G; ++g) mx[g] = -INFINITY;
#pragma unroll 1
  for (int p0 = 0; p0 < S::KP; p0 += S::KB) {
    if (p0 > 0) {
      load_k(p0);
      if (resid) ahead_k(p0);
    }
#pragma unroll
    for (int b = 0; b < S::KB; ++b) {
      const int pass = p0 + b;
      const int row = wtok0 + pass * RPK + kr;
      float a[G];
#pragma unroll
      for (int g = 0; g < G; ++g) a[g] = 0.f;
#pragma unroll
      for (int j = 0; j < PK; ++j) {
        const uint32_t* kw = reinterpret_cast<const uint32_t*>(&kv[b][j]);
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
          for (int g = 0; g < G; ++g)
            a[g] = fmaf(as_f32(kw[w]), as_f32(reinterpret_cast<const uint32_t*>(&qr[g][j])[w]), a[g]);
      }
      if (resid) {
        if constexpr (S::ENT > 0) {
#pragma unroll
          for (int i = 0; i < ENT; ++i) {
            float w;
            const int c = entry(kc[b][i], w);
            const float v = w * kx[b][i];
#pragma unroll
            for (int g = 0; g < G; ++g) a[g] = fmaf(q_lds[c * G + g], v, a[g]);
          }
        }
        const uint64_t rc = (uint64_t)min(row, T - 1) * k;
        for (int e = e0 + S::ENT; e < e1; ++e) {
          float w;
          const int c = entry(code_at(ikp, rc + e), w);
          const float v = w * vkp[rc + e];
#pragma unroll
          for (int g = 0; g < G; ++g) a[g] = fmaf(q_lds[c * G + g], v, a[g]);
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float t = group_sum<LPRK>(a[g]) * scale_log2;
        t = row < T ? t : -INFINITY;
        mx[g] = fmaxf(mx[g], t);
        a[g] = t;
      }
      if (ks == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) s_lds[wave][g][pass * RPK + kr] = a[g];
      }
    }
  }
  // Token-level residual set: the logits of the set's tokens get
  // q . sum_f w_f H_f (lanes over channels, one token at a time) before the
  // max.  The first one's row in the set: the running count before the
  // 128-token chunk, plus the mask bits of the chunk's words before the wave's.
  const int NF = P.bsize - 1;
  uint32_t tbase = 0;
  const float* hkp = nullptr;
  const float* hvp = nullptr;
  const uint32_t* tmask = nullptr;
  const bool set = tokres && wtok0 < T;
  if (set) {
    const TokLayout Lt = tok_layout(mode, (uint64_t)T, D, unit_ppm(P.res_ppm, P.n_rates, P.rates_ppm, mbyte), 4, 4,
                                    P.bsize);
    tmask = reinterpret_cast<const uint32_t*>(seg + Lt.mask);
    tbase = reinterpret_cast<const uint32_t*>(seg + Lt.count)[wtok0 / kTokChunk];
    for (int w = wtok0 / kTokChunk * (kTokChunk / 32); w < wtok0 / 32; ++w) tbase += (uint32_t)__builtin_popcount(tmask[w]);
    hkp = reinterpret_cast<const float*>(seg + Lt.hk);
    hvp = reinterpret_cast<const float*>(seg + Lt.hv);
    wave_sync();  // the K pass's logits are in LDS
    int ntr = 0;
    for (int tl = 0; tl < CH; ++tl) {
      const int row = wtok0 + tl;
      if (row >= T || !((tmask[row >> 5] >> (row & 31)) & 1u)) continue;
      const uint64_t h0 = (uint64_t)(tbase + ntr) * NF * D;
      for (int g = 0; g < G; ++g) {
        float a = 0.f;
        for (int c = lane; c < D; c += 64) {
          float hsum = 0.f;
          for (int f = 0; f < NF; ++f) hsum = fmaf(P.wres[f], hkp[h0 + (uint64_t)f * D + c], hsum);
          a = fmaf(q_lds[c * G + g], hsum, a);
        }
        a = wave_sum(a) * scale_log2;
        if (lane == 0) s_lds[wave][g][tl] += a;
      }
      ++ntr;
    }
    wave_sync();
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float x = -INFINITY;
      for (int tl = lane; tl < CH; tl += 64) x = fmaxf(x, s_lds[wave][g][tl]);
      mx[g] = x;
    }
  }
  float m[G];
#pragma unroll
  for (int g = 0; g < G; ++g) m[g] = wave_max(mx[g]);
  wave_sync();

  // ------------------------------------------------------------ probabilities
  float lsum[G];
#pragma unroll
  for (int g = 0; g < G; ++g) lsum[g] = 0.f;
#pragma unroll
  for (int i = 0; i < (CH + 63) / 64; ++i) {
    const int t = i * 64 + lane;
    if (CH % 64 != 0 && t >= CH) break;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float s = s_lds[wave][g][t];
      const float p = (s == -INFINITY) ? 0.f : exp2f(s - m[g]);
      lsum[g] += p;
      s_lds[wave][g][t] = p;
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) lsum[g] = wave_sum(lsum[g]);
  wave_sync();

  // ------------------------------------------------------------ V pass
  float acc[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[g][c] = 0.f;
#pragma unroll 1
  for (int i0 = 0; i0 < S::VP; i0 += S::VB) {
    if (SHAPE != kSpread || i0 > 0) load_v(i0);
#pragma unroll
    for (int b = 0; b < S::VB; ++b) {
      const int tl = (i0 + b) * RPV + vr;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float p = s_lds[wave][g][tl];
        acc[g][0] = fmaf(p, as_f32(vv[b].x), acc[g][0]);
        acc[g][1] = fmaf(p, as_f32(vv[b].y), acc[g][1]);
        acc[g][2] = fmaf(p, as_f32(vv[b].z), acc[g][2]);
        acc[g][3] = fmaf(p, as_f32(vv[b].w), acc[g][3]);
      }
    }
  }
  if (set) {
    // V of the set's tokens: each lane owns distinct channels of the accumulator
    int j = 0;
    for (int tl = 0; tl < CH; ++tl) {
      const int row = wtok0 + tl;
      if (row >= T || !((tmask[row >> 5] >> (row & 31)) & 1u)) continue;
      const uint64_t h0 = (uint64_t)(tbase + j) * NF * D;
      for (int c = lane; c < D; c += 64) {
        float hsum = 0.f;
        for (int f = 0; f < NF; ++f) hsum = fmaf(P.wres[f], hvp[h0 + (uint64_t)f * D + c], hsum);
#pragma unroll
        for (int g = 0; g < G; ++g) sp_lds[wave][g][c] += s_lds[wave][g][tl] * hsum;
      }
      ++j;
    }
  }
  if (resid) {
    auto add = [&](int e, uint32_t code, float x) {
      const int tl = e / k;
      float w;
      const int c = entry(code, w);
      const float v = w * x;
#pragma unroll
      for (int g = 0; g < G; ++g) atomicAdd(&sp_lds[wave][g][c], s_lds[wave][g][tl] * v);
    };
    if constexpr (S::ENT > 0) {
#pragma unroll
      for (int i = 0; i < ENT; ++i)
        if (lane + 64 * i < ne_live) add(lane + 64 * i, vc[i], vx[i]);
    }
    for (int e = lane + 64 * S::ENT; e < ne_live; e += 64) {
      const uint64_t x = (uint64_t)wtok0 * k + e;
      add(e, code_at(ivp, x), vvp[x]);
    }
  }
#pragma unroll
  for (int off = NP; off < 64; off <<= 1)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[g][c] += __shfl_xor(acc[g][c], off, 64);
  wave_sync();
  if (lane < NP) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float4* dst = reinterpret_cast<float4*>(&sp_lds[wave][g][lane * 4]);
      const float4 o = *dst;
      *dst = make_float4(acc[g][0] + o.x, acc[g][1] + o.y, acc[g][2] + o.z, acc[g][3] + o.w);
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      m_lds[wave][g] = m[g];
      l_lds[wave][g] = lsum[g];
    }
  }
  __syncthreads();

  // ------------------------------------------------------------ merge waves
  // a group's waves, then the workgroup's groups
  for (int i = threadIdx.x; i < G * (D + 2); i += NTH) {
    const int g = i / (D + 2), c = i - g * (D + 2);
    float M = -INFINITY, gm[W / GW], go[W / GW];
#pragma unroll
    for (int u = 0; u < W / GW; ++u) {
      gm[u] = -INFINITY;
#pragma unroll
      for (int w = 0; w < GW; ++w) gm[u] = fmaxf(gm[u], m_lds[u * GW + w][g]);
      go[u] = 0.f;
#pragma unroll
      for (int w = u * GW; w < u * GW + GW; ++w) {
        const float x = c < D ? sp_lds[w][g][c < D ? c : 0] : l_lds[w][g];
        go[u] = fmaf(merge_weight(m_lds[w][g], gm[u]), x, go[u]);
      }
      M = fmaxf(M, gm[u]);
    }
    float o = go[0];
    if constexpr (W > GW) {
      o = 0.f;
#pragma unroll
      for (int u = 0; u < W / GW; ++u) o = fmaf(merge_weight(gm[u], M), go[u], o);
    }
    rec[g * S::RS + c] = c == D ? M : o;
  }
}

template <int D, int G, int SHAPE>
static hipError_t launch_shape(const DecodeParams& P, hipStream_t s) {
  using S = DecodeShape<D, G, SHAPE>;
  const dim3 grid((unsigned)P.batch * P.hkv * P.n_chunks_total * (SHAPE == kSpread ? S::NGRP : 1));
  hipLaunchKernelGGL((decode_splitk_kernel<D, G, SHAPE>), grid, dim3(64 * S::W), 0, s, P);
  return hipGetLastError();
}

template <int D, int G>
static hipError_t launch_decode_t(const DecodeParams& P, hipStream_t s) {
  if (P.n_sub > 1) return launch_shape<D, G, kSpread>(P, s);
  return P.wide ? launch_shape<D, G, kWide>(P, s) : launch_shape<D, G, kFull>(P, s);
}

template <int D>
static hipError_t launch_decode_d(const DecodeParams& P, hipStream_t s) {
  if (P.batch <= 0 || P.n_chunks_total <= 0) return hipSuccess;
  switch (P.hq / P.hkv) {
    case 1: return launch_decode_t<D, 1>(P, s);
    case 2: return launch_decode_t<D, 2>(P, s);
    case 4: return launch_decode_t<D, 4>(P, s);
    default: return launch_decode_t<D, 8>(P, s);
  }
}

hipError_t launch_decode(const DecodeParams& P, hipStream_t s) {
  if (P.bf16) return launch_decode_stream(P, s);
  return P.d == 128 ? launch_decode_d<128>(P, s) : launch_decode_d<64>(P, s);
}

}  // namespace fdkv
