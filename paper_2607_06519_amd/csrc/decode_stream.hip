// Streaming split-K decode over a bf16 or FP8 cache: its launch, and the merge
// of the records (all cache types).  The split-K kernel is in decode_stream.h.
#include "decode_stream.h"

namespace fdkv {

// Wave-wide max / sum: DPP within each row of 16 lanes, then the four row
// results read as uniform values.
__device__ __forceinline__ float wave_max_dpp(float x) {
  x = fmaxf(x, dpp<kDppQuadXor1>(x));
  x = fmaxf(x, dpp<kDppQuadXor2>(x));
  x = fmaxf(x, dpp<kDppRowHalfMirror>(x));
  x = fmaxf(x, dpp<kDppRowMirror>(x));
  const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
  const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
  const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
  const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}
__device__ __forceinline__ float wave_sum_dpp(float x) {
  x += dpp<kDppQuadXor1>(x);
  x += dpp<kDppQuadXor2>(x);
  x += dpp<kDppRowHalfMirror>(x);
  x += dpp<kDppRowMirror>(x);
  const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
  const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
  const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
  const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
  return (a + b) + (c + d);
}

// Log-sum-exp merge of the records of one (sequence, query head), over every
// chunk of the call (compressed spans, then the exact tail; a chunk with no
// tokens holds an empty record, so no lengths are read first):
//   M = max_i m_i,  l = sum_i l_i 2^(m_i - M),  o = sum_i acc_i 2^(m_i - M) / l.
// One workgroup of four waves per query head, chunks taken in blocks of 64.
// Within a block every wave loads the (m, l) pairs (chunk i in lane i) and
// its share of the accumulators (chunk i to wave i mod 4) in one go -- the
// accumulators do not depend on the max -- then reduces M and l itself and
// weights each chunk with the value read from the lane that owns it.  A
// running (M, l, o) carries over between blocks; LDS adds the four waves'
// partial sums.
// SUB: records per chunk.  Above one (the split-K pass of a small fp32 call wrote
// a record per group of a chunk's waves) each chunk's records are first folded
// into one, with the arithmetic of a workgroup that holds all of the chunk's
// groups; chunks are then taken four a wave at a time and those past the end
// skipped, as such launches have few.
template <int D, bool BF16, int G, int SUB>
__global__ __launch_bounds__(256) void decode_merge_kernel(DecodeParams P) {
  constexpr int RS = D + 4;
  constexpr int CPL = D / 64;             // channels per lane
  constexpr int NR = SUB == 1 ? 16 : 4;   // chunks per wave whose accumulators are in flight
  __shared__ float part[4][D];
  const int qh = blockIdx.x % P.hq, seq = blockIdx.x / P.hq;
  const int head = qh / G, g = qh % G;
  const uint64_t rstride = (uint64_t)G * RS;     // floats between consecutive records of one query head
  const uint64_t stride = rstride * SUB;         // ... and between chunks
  const float* base = P.ws + ((uint64_t)(seq * P.hkv + head) * P.n_chunks_total) * stride + g * RS;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nch = P.n_chunks_total, last = nch - 1;  // loads past the end repeat the last record and get weight 0

  float M = -INFINITY, lsum = 0.f, o[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) o[c] = 0.f;
  for (int b0 = 0; b0 < nch; b0 += 64) {
    const int il = b0 + lane;
    float2 ml[SUB];
#pragma unroll
    for (int u = 0; u < SUB; ++u)
      ml[u] = *reinterpret_cast<const float2*>(base + (uint64_t)min(il, last) * stride + u * rstride + D);
    float a[NR][SUB][CPL];
    auto load = [&](int j0) {
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const float* r = base + (uint64_t)min(b0 + wave + 4 * (j0 + j), last) * stride;
#pragma unroll
        for (int u = 0; u < SUB; ++u)
#pragma unroll
          for (int c = 0; c < CPL; ++c) a[j][u][c] = r[u * rstride + lane * CPL + c];
      }
    };
    load(0);
    // the chunk's own (m, l), and its records' weights in it
    float mi = ml[0].x, li = ml[0].y, f[SUB];
    if constexpr (SUB > 1) {
#pragma unroll
      for (int u = 1; u < SUB; ++u) mi = fmaxf(mi, ml[u].x);
      li = 0.f;
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        f[u] = merge_weight(ml[u].x, mi);
        li = fmaf(f[u], ml[u].y, li);
      }
    }
    if (il >= nch) mi = -INFINITY;
    const float Mb = wave_max_dpp(mi);
    const float Mn = fmaxf(M, Mb);
    const float fo = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
    const float w = (il < nch && mi != -INFINITY) ? __builtin_amdgcn_exp2f(mi - Mn) : 0.f;
    lsum = lsum * fo + wave_sum_dpp(w * li);
#pragma unroll
    for (int c = 0; c < CPL; ++c) o[c] *= fo;
#pragma unroll
    for (int j0 = 0; j0 < 16; j0 += NR) {
      if (SUB > 1 && b0 + wave + 4 * j0 >= nch) break;
      if (j0 > 0) load(j0);
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const int il_j = wave + 4 * (j0 + j);
        const float wj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), il_j));
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          float x = a[j][0][c];
          if constexpr (SUB > 1) {
            x = 0.f;
#pragma unroll
            for (int u = 0; u < SUB; ++u)
              x = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(f[u]), il_j)), a[j][u][c], x);
          }
          o[c] = fmaf(wj, x, o[c]);
        }
      }
    }
    M = Mn;
  }
#pragma unroll
  for (int c = 0; c < CPL; ++c) part[wave][lane * CPL + c] = o[c];
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int ch = lane * CPL + c;
      const float s = (part[0][ch] + part[1][ch]) + (part[2][ch] + part[3][ch]);
      const float res = lsum > 0.f ? s / lsum : 0.f;
      const uint64_t oi = ((uint64_t)seq * P.hq + qh) * D + ch;
      if constexpr (BF16)
        reinterpret_cast<uint16_t*>(P.out)[oi] = (uint16_t)f32_to_bf16_bits(res);
      else
        reinterpret_cast<float*>(P.out)[oi] = res;
    }
  }
}

hipError_t launch_decode_stream(const DecodeParams& P, hipStream_t s) {
  if (P.n_chunks_total <= 0) return hipSuccess;
  return P.d == 128 ? launch_stream<128>(P, s) : launch_stream<64>(P, s);
}

template <int D, bool BF16, int G>
static hipError_t launch_merge_g(const DecodeParams& P, hipStream_t s) {
  const dim3 grid((unsigned)P.batch * P.hq);
  if constexpr (!BF16) {
    if (P.n_sub > 1) {
      hipLaunchKernelGGL((decode_merge_kernel<D, BF16, G, decode_groups(G)>), grid, dim3(256), 0, s, P);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((decode_merge_kernel<D, BF16, G, 1>), grid, dim3(256), 0, s, P);
  return hipGetLastError();
}

template <int D, bool BF16>
static hipError_t launch_merge_d(const DecodeParams& P, hipStream_t s) {
  switch (P.hq / P.hkv) {
    case 1: return launch_merge_g<D, BF16, 1>(P, s);
    case 2: return launch_merge_g<D, BF16, 2>(P, s);
    case 4: return launch_merge_g<D, BF16, 4>(P, s);
    default: return launch_merge_g<D, BF16, 8>(P, s);
  }
}

hipError_t launch_decode_merge(const DecodeParams& P, hipStream_t s) {
  if (P.d == 128) return P.bf16 ? launch_merge_d<128, true>(P, s) : launch_merge_d<128, false>(P, s);
  return P.bf16 ? launch_merge_d<64, true>(P, s) : launch_merge_d<64, false>(P, s);
}

}  // namespace fdkv
