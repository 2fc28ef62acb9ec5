// Fused mixed-precision attention for prefill grids of a few hundred groups of 32 query rows.
//
// The walk of thrift_prefill.hip takes a row group through one key block after the other in one wavefront, 0.8 us each however
// idle the chip is: a lone wavefront issues a vector instruction every 9 cycles or so, and a block is about 160 of them (the
// scores of the next block ahead of the softmax of this one did not help: it does not wait for latency).  Here KS = 4 wavefronts,
// one on every SIMD, share the row group and take four key blocks of the walk per step:
//   scores and P.V  wavefront s: the scores of block s of group n and their row maxima, which it leaves in LDS; O^T of channel
//                   tile s for the four blocks of group n - 1, in the order of the walk
//   (barrier)
//   probabilities   wavefront s: the running maximum in front of its block (the maxima of the blocks before it in the group and
//                   of all earlier groups), softmax and, on the 4-bit path, the codes of P, which go to LDS over the K tile that
//                   nobody needs any more
//   (barrier)
// while LDS DMA brings group n + 1.  Every score, maximum, code and sum is formed from the same operands in the same order as by
// one wavefront: the results have the same bits.
//
// A step of four blocks takes 1.8 us where one wavefront takes 3.3 (one head of 2048 tokens: 41 -> 22.5 us, 54 -> 31 with
// the launches before it).  What bounds it: the instruction issue of a lone wavefront, about 1200 cycles for the probabilities, 1300
// for scores and P.V, 1300 for the maxima, the walk and the DMA instructions.  So the loop says which way its branches mostly go and
// masks, promoted and partly filled blocks lie out of line (chunk of 500 tokens on 30720, 16/16 heads, 5 %: 232.4 -> 228.8 us).
//
// RG row groups share the staged blocks of a workgroup of RG x KS wavefronts.
#include "thrift_launch.h"
#include "thrift_tile.h"

namespace thrift {

namespace {

constexpr int KS = 4;                        // wavefronts per row group = key blocks per step = channel tiles of O

template <int RG>
struct SplitLds {
  static constexpr int ring = 0;                                    // [3][KS] 4-bit blocks; codes of P over K's
  static constexpr int k16 = 3 * KS * kLdsBytes4;                   // one 16-bit K tile; rounded P over it
  static constexpr int v16 = k16 + kTile16;                         // one 16-bit V tile
  static constexpr int mx = v16 + kTile16;                          // [RG][32][KS] row maxima of the group's blocks
  static constexpr int sums = mx + RG * KS * 32 * 4;                // [RG][64][KS] row sums, one per lane
  static constexpr int scales = sums + RG * KS * 64 * 4;            // [RG][64][KS] scale bytes of P, one per lane
  static constexpr int total = scales + RG * KS * 64;
  static_assert(RG <= 4, "the codes of P take the place of a K tile");
  static_assert(total <= 160 * 1024, "LDS of a CU");
};

// KS positions of the walk, fewer at its end or in front of a promoted block that has to wait for the tile buffers
struct Group {
  int own;             // key block of this wavefront's position, -1 past the end of the group
  int count;           // positions
  int seen;            // the first ones, whose blocks this wavefront's rows see
  uint32_t promoted;   // bit t: position t is taken in 16 bits (at most one is)
  uint32_t grew;       // bit t: some row's maximum rose with block t
  v4f alpha;           // by that factor
};

}  // namespace

template <typename T, int RG, int ORDER>
__device__ __forceinline__ void prefill_split_item(const PrefillArgs& a, unsigned char* lds, unsigned work) {
  typedef SplitLds<RG> L;
  constexpr int KF = 4 / RG;                 // 1 KiB fragments of a 4-bit K (and of a V) tile per wavefront
  constexpr int C16 = 16 / RG;               // ... of one 16-bit K or V tile
  constexpr int kRows = 32 * RG;

  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, r = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = wave % RG, split = wave / RG;            // row group; position in the group of key blocks, channel tile
  const int N = a.N, Nq = a.Nq, G = a.Hq / a.Hkv;
  const int Tq = (Nq + a.Bq - 1) / a.Bq, Tk = (N + kBk - 1) / kBk, Ts = (Nq + kRows - 1) / kRows;

  // late (long) rows first, the heads of a KV head on one XCD, as in prefill_item
  const int units = a.B * a.Hkv, per_unit = G * Ts;
  int unit, within;
  if ((units & 7) == 0) {
    const int xcd = work & 7, t = work >> 3;
    unit = xcd + 8 * (t / per_unit);
    within = t % per_unit;
  } else {
    unit = work / per_unit;
    within = work % per_unit;
  }
  const int b = unit / a.Hkv, kvh = unit % a.Hkv;
  const int sub = Ts - 1 - within / G;                   // rows kRows * sub ..
  const int hq = kvh * G + within % G;
  const size_t qh = (size_t)b * a.Hq + hq, kh = (size_t)b * a.Hkv + kvh;
  const int i = sub * kRows / a.Bq;                      // query block, whose list this is
  const int q_first = a.q_off * a.Bq + sub * kRows;      // sequence position of the workgroup's first row
  const int q0 = q_first + w * 32;
  const int row = sub * kRows + w * 32 + r, lrow = min(row, Nq - 1);
  const size_t qrow = qh * Nq + lrow;

  v4i qf4[2];
  qf4[0] = *reinterpret_cast<const v4i*>(a.q4 + qrow * 64 + half * 32);
  qf4[1] = *reinterpret_cast<const v4i*>(a.q4 + qrow * 64 + half * 32 + 16);
  const uint32_t qsc = *reinterpret_cast<const uint32_t*>(a.qs + qrow * 4) >> (16 * half);
  const uint8_t* q16head = reinterpret_cast<const uint8_t*>(a.q + qh * Nq * kD);

  const int vis = a.causal ? min(Tk, (q_first + kRows - 1) / kBk + 1) : Tk;
  const int vis_wave = a.causal ? min(vis, (q0 + 31) / kBk + 1) : vis;
  const int key_limit = a.causal ? min(q0 + r + 1, N) : N;
  const int32_t* sel = a.idx + (qh * Tq + i) * a.kmax;
  const int nsel = min(a.cnt[qh * Tq + i], a.kmax);
  auto sel_at = [&](int t) -> int {                      // through the scalar data path, as in prefill_item
    const int32_t* p = sel + __builtin_amdgcn_readfirstlane(t);
    int v;
    asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(p) : "memory");
    return min(max(v, 0), Tk - 1);
  };

  const uint8_t* k4base = a.k4 + kh * N * 64;
  const uint8_t* v4base = a.v4 + kh * (size_t)Tk * 4096;
  const uint8_t* ksbase = a.ks + kh * N * 4;
  const uint8_t* vsbase = a.vs + kh * (size_t)Tk * 2 * kD;
  const uint8_t* k16base = reinterpret_cast<const uint8_t*>(a.k + kh * N * kD);
  const uint8_t* v16base = reinterpret_cast<const uint8_t*>(a.v + kh * N * kD);

  // ---- staging: the RG wavefronts of a position stage its block, layouts as in prefill_item ----
  const uint32_t lds0 = lds_address(lds);
  uint32_t k4off[KF], v4off[KF];
#pragma unroll
  for (int u = 0; u < KF; ++u) {
    const int f = w * KF + u;
    k4off[u] = (uint32_t)(key_of_row(r, f >> 1) * 64 + (2 * half + (f & 1)) * 16);
    v4off[u] = (uint32_t)((32 * f + r) * 32 + half * 16);
  }
  const int last_key_row = (N - 1) & (kBk - 1);
  // rows past the last key do not exist in the row-major arrays: the last key's row again, masked below
  auto clamped = [&](uint32_t off, int shift, uint32_t last) { return (min(off >> shift, last) << shift) | (off & ((1u << shift) - 1u)); };
  auto issue4 = [&](int j, int slot) {
    const int j_ = __builtin_amdgcn_readfirstlane(j);
    const uint32_t to = lds0 + L::ring + (uint32_t)(__builtin_amdgcn_readfirstlane(slot) * KS + split) * kLdsBytes4;
    const uint8_t *kt = k4base + (size_t)j_ * 4096, *vt = v4base + (size_t)j_ * 4096;
    if (__builtin_expect((j_ + 1) * kBk <= N, 1)) {
#pragma unroll
      for (int u = 0; u < KF; ++u) dma_b128(kt, k4off[u], to + kLdsK4 + (w * KF + u) * 1024);
      if (w == 0) dma_b32(ksbase + (size_t)j_ * 256, (uint32_t)lane * 4, to + kLdsKS);
    } else {
      uint32_t last = (uint32_t)last_key_row;
      asm volatile("" : "+s"(last));                     // the clamped offsets are formed here, not ahead of the walk
#pragma unroll
      for (int u = 0; u < KF; ++u) dma_b128(kt, clamped(k4off[u], 6, last), to + kLdsK4 + (w * KF + u) * 1024);
      if (w == 0) dma_b32(ksbase + (size_t)j_ * 256, clamped((uint32_t)lane * 4, 2, last), to + kLdsKS);
    }
#pragma unroll
    for (int u = 0; u < KF; ++u) dma_b128(vt, v4off[u], to + kLdsV4 + (w * KF + u) * 1024);
    if (w == RG - 1) dma_b32(vsbase + (size_t)j_ * 256, (uint32_t)lane * 4, to + kLdsVS);
  };
  // instruction q covers rows 4 q .. 4 q + 3, lane l chunk position l & 15 of row l >> 4
  auto issue16 = [&](const uint8_t* base, int j, bool is_k, uint32_t to) {
    const int j_ = __builtin_amdgcn_readfirstlane(j);
    const uint32_t last = (j_ + 1) * kBk <= N ? kBk - 1 : (uint32_t)last_key_row;
    const uint8_t* tile = base + (size_t)j_ * kTile16;
    int l_ = lane;
    asm volatile("" : "+v"(l_));                         // offsets are formed here, not kept through the walk
    const int r4 = l_ >> 4;
#pragma unroll
    for (int u = 0; u < C16; ++u) {
      const int q = u * RG + w;
      const uint32_t chunk = (uint32_t)(l_ & 15) ^ (is_k ? (uint32_t)(r4 | (q >= 8 ? 4 : 0)) : (uint32_t)(4 * r4));
      dma_b128(tile, clamped((uint32_t)(q * 1024 + r4 * 256) + 16 * chunk, 8, last), to + q * 1024);
    }
  };

  // ---- the walk, KS positions at a time ----
  int pos = 0, at = 0;                                   // next key block; next entry of the list
  int n0 = nsel > 0 ? sel_at(0) : 0x7fffffff;            // that entry
  int nselv = nsel;                                      // ORDER 1: entries inside the visible range (the list is ascending)
  if constexpr (ORDER == 1) {
    if (nsel > 0 && sel_at(nsel - 1) >= vis) {
      nselv = 0;
      while (nselv < nsel && sel_at(nselv) < vis) ++nselv;
    }
    if (nselv == 0) n0 = 0x7fffffff;
  }
  auto advance = [&]() {
    ++at;
    n0 = at < nselv ? sel_at(at) : 0x7fffffff;
  };
  int tail = 0;                                          // ORDER 1: promoted blocks taken
  // the next group; the one before it has a promoted block: `busy`, the 16-bit tile buffers are not free in time
  auto next_group = [&](Group& g, bool busy) {
    g.promoted = 0;
    if (pos + KS <= vis && n0 >= pos + KS) {             // 4-bit blocks that follow each other
      g.own = pos + split;
      g.count = KS;
      g.seen = min(KS, vis_wave - pos);
      pos += KS;
      return;
    }
    g.own = -1;
    g.count = g.seen = 0;
    auto take = [&](int j, bool p) {
      if (g.count == split) g.own = j;
      if (p) g.promoted = 1u << g.count;
      ++g.count;
      if (j < vis_wave) g.seen = g.count;
    };
    if (ORDER == 1 && pos >= vis) {                      // the promoted blocks at the end: one at a time
      if (tail < nselv && !busy) take(sel_at(tail++), true);
      return;
    }
#pragma unroll 1
    while (g.count < KS && pos < vis) {
      if (n0 < pos) {                                    // entries behind the walk (a list that is not ascending) are dropped
        advance();
        continue;
      }
      const bool p = pos == n0;
      if (p) {
        if (ORDER == 0 && busy) break;
        busy = true;
        advance();
      }
      if (ORDER == 0 || !p) take(pos, p);
      ++pos;
    }
  };
  auto more = [&]() { return pos < vis || (ORDER == 1 && tail < nselv); };

  float m = kEmptyMax, l = 0.f;                          // running maximum (every wavefront); row sum (position 0 only)
  v16f o = {0.f};
  const float c = a.scale * 1.4426950408889634f;
  float* mx = reinterpret_cast<float*>(lds + L::mx) + (w * 32 + r) * KS;
  float* sums = reinterpret_cast<float*>(lds + L::sums) + (w * 64 + lane) * KS;
  unsigned char* scales = lds + L::scales + (w * 64 + lane) * KS;
  auto issue_tiles16 = [&](const Group& g) {
    if ((g.promoted >> split) & 1) {
      issue16(k16base, g.own, true, lds0 + L::k16);
      issue16(v16base, g.own, false, lds0 + L::v16);
    }
  };
  // Ordinary arithmetic: a matrix instruction that writes o may just have been issued, and the compiler keeps the 12 wait states
  // behind it only for instructions of its own, not for those inside an asm statement.
  auto rescale_by = [&](float f) {
    l *= f;
    asm volatile("" : "+v"(l));                          // rounded here, not fused with the addition behind
#pragma unroll
    for (int e = 0; e < 16; ++e) o[e] *= f;
  };

  // Step n: the scores of group n and P.V of group n - 1 between one pair of barriers, the probabilities of group n behind
  // them, while the tiles of group n + 1 travel.
  Group g, before, next;
  before.own = -1;
  before.count = before.seen = 0;
  before.promoted = before.grew = 0;
  before.alpha = (v4f){1.f, 1.f, 1.f, 1.f};
  next_group(g, false);
  if (g.own >= 0 && ((g.promoted >> split) & 1) == 0) issue4(g.own, 0);
  issue_tiles16(g);
  int slot_g = 0, slot_b = 2;
  while (g.count > 0 || before.count > 0 || more()) {
    const int j = g.own;
    const bool p16 = ((g.promoted >> split) & 1) != 0;
    const int slot_n = slot_g == 2 ? 0 : slot_g + 1;
    unsigned char* slot = lds + L::ring + (slot_g * KS + split) * kLdsBytes4;
    const unsigned char* behind = lds + L::ring + slot_b * KS * kLdsBytes4;
    vm_wait<0>();
    lds_barrier();                                       // group n has arrived, P of group n - 1 is written, slot_n is free
    next_group(next, g.promoted != 0);
    if (next.own >= 0 && ((next.promoted >> split) & 1) == 0) issue4(next.own, slot_n);
    if (before.promoted == 0) issue_tiles16(next);

    const bool mine = j >= 0 && j < vis_wave;
    const bool usual = before.promoted == 0 && before.seen == KS;
    v16f s[2];
    float mloc = kEmptyMax, mrow = kEmptyMax;
    if (usual) {
      v4i v[KS], pq[KS];
      uint32_t vs[KS];
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        const unsigned char* tile = behind + t * kLdsBytes4;
        v[t] = *reinterpret_cast<const v4i*>(tile + kLdsV4 + lane * 16 + 1024 * split);
        pq[t] = *reinterpret_cast<const v4i*>(tile + kLdsK4 + w * 1024 + lane * 16);
        vs[t] = tile[kLdsVS + half * kD + r + 32 * split];
      }
      const uint32_t pb = *reinterpret_cast<const uint32_t*>(scales);
      if (mine && !p16) scores_fp4(slot, lane, qf4, qsc, s);
      v4f sum;
      if (split == 0) sum = *reinterpret_cast<const v4f*>(sums);
#define THRIFT_BLOCK(TT)                                                                                       \
  if ((before.grew >> TT) & 1) rescale_by(before.alpha[TT]);                                                   \
  if (split == 0) l += sum[TT];                                                                                \
  o = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(v[TT]), widen(pq[TT]), o, 4, 4, 0, vs[TT], TT, pb);
      THRIFT_BLOCK(0) THRIFT_BLOCK(1) THRIFT_BLOCK(2) THRIFT_BLOCK(3)
#undef THRIFT_BLOCK
    } else {
      if (mine && !p16) scores_fp4(slot, lane, qf4, qsc, s);
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        if (t >= before.seen) continue;
        if ((before.grew >> t) & 1) rescale_by(before.alpha[t]);
        if (split == 0) l += sums[t];
        if ((before.promoted >> t) & 1) {
          const unsigned char* pr = lds + L::k16 + w * 4096 + lane * 16;
          v8s pf[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) pf[q] = *reinterpret_cast<const v8s*>(pr + 1024 * q);
          pv_16_tile<T>(lds + L::v16, lane, split, pf, o);
        } else {
          const unsigned char* tile = behind + t * kLdsBytes4;
          const uint32_t pb = scales[t], vs = tile[kLdsVS + half * kD + r + 32 * split];
          o = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(*reinterpret_cast<const v4i*>(tile + kLdsV4 + lane * 16 + 1024 * split)),
                                                              widen(*reinterpret_cast<const v4i*>(tile + kLdsK4 + w * 1024 + lane * 16)), o, 4, 4, 0, vs, 0, pb);
        }
      }
    }
    if (mine) {
      if (__builtin_expect(p16, 0)) {
        v8s qf[8];
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) qf[s8] = *reinterpret_cast<const v8s*>(q16head + (uint32_t)(lrow * (2 * kD) + 32 * s8 + 16 * half));
        scores_16<T>(lds + L::k16, lane, qf, s);
      }
      if (__builtin_expect((a.causal && j * kBk + kBk - 1 > q0) || (j + 1) * kBk > N, 0)) mask_scores(s, half, key_limit - j * kBk);
      mloc = lane_max(s);
      mrow = both_halves_max(mloc);
    }
    if (half == 0) mx[split] = mrow;
    lds_barrier();                                       // maxima of group n are there, group n - 1 is finished
    if (before.promoted != 0) issue_tiles16(next);       // its tile buffers are free only now

    // ---- running maxima, probabilities of block j ----
    const v4f maxima = *reinterpret_cast<const v4f*>(mx);
    const float m_old = m;
    float m_own;
    g.grew = 0;
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      const float m_new = fmaxf(m, maxima[t]);
      g.alpha[t] = m - m_new;
      m = m_new;
      if (t == 0 || t == split) m_own = m;
    }
    if (__builtin_amdgcn_ballot_w64(m != m_old) != 0ULL) {
#pragma unroll
      for (int t = 0; t < KS; ++t)
        if (__builtin_amdgcn_ballot_w64(g.alpha[t] != 0.f) != 0ULL) {
          g.grew |= 1u << t;
          float d = g.alpha[t];
          asm volatile("" : "+v"(d));
          g.alpha[t] = fast_exp2(d * c);
        }
    }
    if (mine) {
      uint32_t pb;
      sums[split] = probabilities(s, mloc, m_own, c, pb);
      if (p16) {
        v8s pf[4];
        round_p16<T>(s, pf);
        unsigned char* to = lds + L::k16 + w * 4096 + lane * 16;
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<v8s*>(to + 1024 * q) = pf[q];
      } else {
        *reinterpret_cast<v4i*>(slot + kLdsK4 + w * 1024 + lane * 16) = quantize_p_group(s, pb);
        scales[split] = (unsigned char)pb;
      }
    }
    before = g;
    g = next;
    slot_b = slot_g;
    slot_g = slot_n;
  }
  vm_wait<0>();

  // ---- epilogue (Alg. 1 step 21): O / l ----
  lds_barrier();
  if (split == 0) {
    const float total = l + other_half(l);
    if (half == 0) mx[0] = total;
  }
  lds_barrier();
  l = mx[0];
  const float inv = l > 0.f ? 1.0f / l : 0.f;
  if (row < Nq) {
#pragma unroll
    for (int q4i = 0; q4i < 4; ++q4i)
      store_out4(a.out, a.out_dt, qrow * kD + 32 * split + 8 * q4i + 4 * half, o[4 * q4i] * inv, o[4 * q4i + 1] * inv, o[4 * q4i + 2] * inv, o[4 * q4i + 3] * inv);
    if (a.lse != nullptr && split == 0 && half == 0) a.lse[qrow] = m * a.scale + __logf(l);
  }
}

// Bounds of 512 threads also for RG = 1: with 256 the compiler counts on one wavefront per SIMD and spreads the matrix results
// over the accumulation registers, which every vector instruction then has to copy from.
template <typename T, int RG, int ORDER>
__global__ void __launch_bounds__(512, 2) prefill_split_kernel(PrefillArgs a) {
  __shared__ __align__(1024) unsigned char lds[SplitLds<RG>::total];
  prefill_split_item<T, RG, ORDER>(a, lds, blockIdx.x);
}

template <int RG>
static void launch_split(const PrefillArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)((long)a.B * a.Hq * ((a.Nq + 32 * RG - 1) / (32 * RG)))), block(RG * KS * 64);
  if (a.dt == THRIFT_F16) {
    if (a.tile_order == 1) prefill_split_kernel<F16, RG, 1><<<grid, block, 0, st>>>(a);
    else prefill_split_kernel<F16, RG, 0><<<grid, block, 0, st>>>(a);
  } else {
    if (a.tile_order == 1) prefill_split_kernel<BF16, RG, 1><<<grid, block, 0, st>>>(a);
    else prefill_split_kernel<BF16, RG, 0><<<grid, block, 0, st>>>(a);
  }
}

// Row groups of 32 query rows up to which four wavefronts each are the faster form: one row group per workgroup while every
// workgroup has a CU of its own, two up to twice as many.  Chunks of queries over 30720 cached tokens at 5 %, 32/8 heads, plain
// kernel / one / two row groups per workgroup: 435 / 264 / 308 us (128 row groups), 437 / 270 / 309 (256), 439 / 496 / 315 (512);
// whole prompts, 8/2 heads: 33 / 28 / 30 us (1000 tokens, 256 row groups), 49 / 47 / 42 (2000, 504).  At 512 row groups and 500
// tokens the walk of 8 key blocks is too short to gain (28.0 / 27.6 us; 27.9 / 28.3 in the order of Sec. 3.3).
// Promoted blocks come one to a group here, and one at a time where they come last: at 10 % 477 / 330 us for the chunk of 128
// row groups, at 25 % 459 / 547.
constexpr int kSplitRowGroups = kCus;
constexpr int kSplitLeastBlocks = 10;        // key blocks, beyond kSplitRowGroups
constexpr int kSplitPercent = 15;            // list length / key blocks (in %) from which the plain kernel is the faster one

bool launch_prefill_split(const PrefillArgs& a, hipStream_t st) {
  if (a.tile_order > 1) return false;                    // these name a schedule of the plain kernel
  const long groups = (long)a.B * a.Hq * ((a.Nq + 31) / 32), Tk = (a.N + kBk - 1) / kBk;
  if ((long)a.kmax * 100 >= Tk * kSplitPercent) return false;
  if (groups <= kSplitRowGroups) launch_split<1>(a, st);
  else if (groups <= 2 * kSplitRowGroups && Tk >= kSplitLeastBlocks) launch_split<2>(a, st);
  else return false;
  return true;
}

}  // namespace thrift
