// The row layout of the decode kernels: one query token per head, a few heads per wavefront.
#pragma once

#include "thrift_tile.h"

namespace thrift {

// ---- one query row per wavefront: the row layout ----
// With a single head per wavefront the transposed tiles of the prefill kernel would spend a whole wavefront
// instruction on each of the row's 64 scores.  Here the score tiles are formed the other way round, S = Q . K^T
// with the query in rows 0 and 4 of the A operand (all other rows zero): accumulator register 0 of lane (half, r)
// is row 4*half, column r, i.e. the query against key r of the 32-key sub-tile.  Taking sub-tile 0 from the lower 32
// lanes and sub-tile 1 from the upper ones leaves ONE register with the score of key `lane` of the block in every
// lane: the online softmax of Alg. 1 then costs one exponential per block, its maxima come from lane permutes, and
// the probabilities are gathered into lanes 0 and 32 (the B-operand column of the query in O^T += V^T . P^T, 32 keys
// = one MXFP4 group per lane) by a few more permutes.

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x) { return __builtin_amdgcn_update_dpp(0u, x, CTRL, 0xf, 0xf, true); }
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) { return __uint_as_float(dpp_u<CTRL>(__float_as_uint(x))); }
constexpr int kDppSwap1 = 0xb1;        // quad_perm [1,0,3,2]: lane ^ 1
constexpr int kDppSwap2 = 0x4e;        // quad_perm [2,3,0,1]: lane ^ 2
constexpr int kDppQuadHi = 0xee;       // quad_perm [2,3,2,3]: lanes 0,1 of a quad read lanes 2,3
constexpr int kDppHalfMirror = 0x141;  // lane i of each 8 reads lane 7 - i
constexpr int kDppMirror = 0x140;      // lane i of each 16 reads lane 15 - i
constexpr int kDppShl4 = 0x104;        // lane i reads lane i + 4 of its 16-lane row

// natural key order for the row layout: fragment (t, kk) of lane (half, r) = key 32t + r, d-group 2*half + kk
__device__ __forceinline__ K4Tile load_k4_rows(const unsigned char* slot, int lane) {
  const int half = lane >> 5, r = lane & 31;
  const unsigned char* ksrow = slot + kLdsKS + 4 * r + 2 * half;        // sub-tile 1: 32 keys = 128 bytes further
  K4Tile k;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    k.ks[t] = *reinterpret_cast<const uint16_t*>(ksrow + 128 * t);
    k.a[2 * t] = *reinterpret_cast<const v4i*>(slot + kLdsK4 + ((t * 2 + 0) * 64 + lane) * 16);
    k.a[2 * t + 1] = *reinterpret_cast<const v4i*>(slot + kLdsK4 + ((t * 2 + 1) * 64 + lane) * 16);
  }
  return k;
}
// Scores of key `lane` of the block for the wavefront's NH heads (Alg. 1 step 15 for the one-token query block).
// qf / qsc: the fragments and scale bytes of head u in lanes r = u and r = u + 4 (u < 4), zeros elsewhere: accumulator
// register u is then row u + 4*half, head u against key r.
template <int NH>
__device__ __forceinline__ void scores4_row(const K4Tile& k, int lane, const v4i (&qf)[2], uint32_t qsc, float (&sv)[NH]) {
  v16f acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    acc[t] = (v16f){0.f};
    acc[t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(qf[0]), widen(k.a[2 * t]), acc[t], 4, 4, 0, qsc, 0, k.ks[t]);
    acc[t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(qf[1]), widen(k.a[2 * t + 1]), acc[t], 4, 4, 1, qsc, 1, k.ks[t]);
  }
#pragma unroll
  for (int u = 0; u < NH; ++u) sv[u] = (lane >> 5) ? acc[1][u] : acc[0][u];
}
// The same from the 16-bit K tile (Alg. 1 step 9).  Tile rows are keys in natural order, 256 B each, the 16-byte chunk c
// of row `row` stored at chunk position c ^ (row & 7) (eight neighbouring lanes read eight different positions).
// qf[s8]: head u's elements d = 16*s8 + 8*half + [0,8) in lanes r = u and r = u + 4, zeros elsewhere.
template <typename T, int NH>
__device__ __forceinline__ void scores16_row(const unsigned char* ktile, int lane, const v8s (&qf)[8], float (&sv)[NH]) {
  const int half = lane >> 5, r = lane & 31;
  v16f acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const unsigned char* row = ktile + (32 * t + r) * 256;
    acc[t] = (v16f){0.f};
#pragma unroll
    for (int s8 = 0; s8 < 8; ++s8) {
      const v8s kf = *reinterpret_cast<const v8s*>(row + 16 * ((2 * s8 + half) ^ (r & 7)));
      acc[t] = T::mfma(qf[s8], kf, acc[t]);
    }
  }
#pragma unroll
  for (int u = 0; u < NH; ++u) sv[u] = half ? acc[1][u] : acc[0][u];
}
// Online softmax of Alg. 1 (steps 10-12 / 16-17) on the row layout: sv = this lane's raw score.  st.m is the running
// maximum (the same in every lane), st.l this lane's share of the row sum.  Returns (for the whole wavefront) whether
// the maximum rose; only then does alpha hold exp(scale * (m_old - m_new)) and must the accumulators be rescaled.
// p: this lane's unnormalised probability; pbyte: the E8M0 byte of the lane's 32-key group of P (as in softmax_update).
__device__ __forceinline__ bool softmax_row(float sv, float c, RowState& st, float& alpha, uint32_t& pbyte, float& p) {
  float v = sv;
  v = fmaxf(v, dpp_f<kDppSwap1>(v));
  v = fmaxf(v, dpp_f<kDppSwap2>(v));
  v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
  v = fmaxf(v, dpp_f<kDppMirror>(v));                               // maximum of the lane's 16
  const uint32_t vb = __float_as_uint(v);
  const auto s16 = __builtin_amdgcn_permlane16_swap(vb, vb, false, false);   // [0]: the even 16's value on both 16s of a 32, [1]: the odd's
  const float gmax = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));  // maximum of the lane's 32-key group
  const uint32_t gb = __float_as_uint(gmax);
  const auto s32 = __builtin_amdgcn_permlane32_swap(gb, gb, false, false);
  const float m_old = st.m;
  const float m_new = max3(m_old, __uint_as_float(s32[0]), __uint_as_float(s32[1]));
  const bool grew = __builtin_amdgcn_ballot_w64(m_new != m_old) != 0ULL;
  if (grew) {
    float d = m_old - m_new;
    asm volatile("" : "+v"(d));                                    // keeps the exponential inside the branch
    alpha = fast_exp2(d * c);
    float l = st.l;
    asm volatile("s_nop 1\n\tv_mul_f32 %0, %1, %0" : "+v"(l) : "v"(alpha));   // wait states: a transcendental result read by hand-written code
    st.l = l;
  }
  st.m = m_new;
  int e;
  {
    const float x = (gmax - m_new) * c;                            // the group maximum maps to exactly 2^floor(x) or above
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(e) : "v"(x));
  }
  pbyte = (uint32_t)max(e + 125, 1);
  p = fast_exp2(__builtin_fmaf(sv, c, -(m_new * c)));
  st.l += p;
  return grew;
}
// Alg. 1 step 19 on the row layout: every lane turns its probability into an E2M1 code under its group's scale and the
// 32 codes of a group are collected, in key order, into the four registers of lane U (keys 0-31) / lane 32 + U (keys
// 32-63), the B-operand column of head U; what the other lanes receive belongs to no query.
template <int U>
__device__ __forceinline__ v4i gather_p4(float p, uint32_t pb) {
  static_assert(U >= 0 && U < 4, "the head's column must lie in the first four lanes");
  const float pscale = __uint_as_float(pb << 23);
  const float nb = dpp_f<kDppSwap1>(p);
  // even lanes: one byte = the codes of keys (lane, lane + 1)
  const uint32_t b8 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, p, nb, pscale, 0);
  const uint32_t b16 = b8 | (dpp_u<kDppQuadHi>(b8) << 8);          // lanes 4q: keys 4q .. 4q+3
  const uint32_t b32 = b16 | (dpp_u<kDppShl4>(b16) << 16);         // lanes 8q: keys 8q .. 8q+7
  const auto sw = __builtin_amdgcn_permlane16_swap(b32, b32, false, false);
  // lane 0 of a 32: sw[0] = its own word (keys 0-7), sw[1] = lane 16's (keys 16-23); lane 8: keys 8-15 and 24-31.
  // Lane U reads lane 0 (a shift right by U) and lane 8 (a shift left by 8 - U) of its 16.
  constexpr int kFrom0 = 0x110 | U, kFrom8 = 0x100 | (8 - U);
  if constexpr (U == 0) return (v4i){(int)sw[0], (int)dpp_u<kFrom8>(sw[0]), (int)sw[1], (int)dpp_u<kFrom8>(sw[1])};
  else return (v4i){(int)dpp_u<kFrom0>(sw[0]), (int)dpp_u<kFrom8>(sw[0]), (int)dpp_u<kFrom0>(sw[1]), (int)dpp_u<kFrom8>(sw[1])};
}
// Alg. 1 step 13 on the row layout: the probabilities rounded to the input dtype and collected through a 128-byte LDS
// row of the wavefront's own: pf[s] of lane (half, *) = keys 32*half + 8s .. + 7 (the order pv_16_rounded contracts in).
template <typename T>
__device__ __forceinline__ void gather_p16(uint16_t* prow, int lane, float p, v8s (&pf)[4]) {
  prow[lane] = T::from_float(p);
#pragma unroll
  for (int s = 0; s < 4; ++s) pf[s] = *reinterpret_cast<const v8s*>(prow + 32 * (lane >> 5) + 8 * s);
}
// largest value of the 64 lanes, in every lane
__device__ __forceinline__ float wave_max(float x) {
  x = fmaxf(x, dpp_f<kDppSwap1>(x));
  x = fmaxf(x, dpp_f<kDppSwap2>(x));
  x = fmaxf(x, dpp_f<kDppHalfMirror>(x));
  x = fmaxf(x, dpp_f<kDppMirror>(x));
  const uint32_t xb = __float_as_uint(x);
  const auto s16 = __builtin_amdgcn_permlane16_swap(xb, xb, false, false);
  x = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
  return fmaxf(x, other_half(x));
}
// sum over the 64 lanes, in every lane
__device__ __forceinline__ float wave_sum(float x) {
  x += dpp_f<kDppSwap1>(x);
  x += dpp_f<kDppSwap2>(x);
  x += dpp_f<kDppHalfMirror>(x);
  x += dpp_f<kDppMirror>(x);
  const uint32_t xb = __float_as_uint(x);
  const auto s16 = __builtin_amdgcn_permlane16_swap(xb, xb, false, false);
  x = __uint_as_float(s16[0]) + __uint_as_float(s16[1]);
  return x + other_half(x);
}

// Blocks that a decode row of `vis` key blocks promotes.
__device__ __forceinline__ int decode_row_budget(int vis, int fixed_k, long long ppm) {
  if (fixed_k >= 0) return min(fixed_k, vis);
  if (ppm <= 0 || vis == 0) return 0;
  const long long k = (ppm * (long long)vis + 999999LL) / 1000000LL;
  return (int)max(1LL, min(k, (long long)vis));
}

}  // namespace thrift
