// Decode for caches that give the one-workgroup-per-partition walk too few workgroups (short caches, few sequences).
//
// The rounding of P follows the running maximum of the partition, so a partition cannot simply be cut into shorter
// recurrences.  It can be computed in two passes that need no order between workgroups:
//   decode_split_scores_kernel  the raw scores of every (query head, key) and the largest score of every chunk;
//   decode_split_values_kernel  softmax, P quantiser and P.V of a chunk, started from the largest score of the chunks in
//                               front of it in the partition: every block sees the running maximum of its partition, as in
//                               the serial walk.
// The scores come from 16 x 16 instead of 32 x 32 matrix instructions.  16-bit scores had equal bits in all of 16 million
// compared; a 4-bit score is exact in both where the products of a row's group scales lie within 2^9 (14 bits hold the sum of
// 128 products of two codes), so that all codes of P are the walk's and only the order of the fp32 sums differs.  With scales
// spread over 2^40, 2.8 % of the scores differed in their last bit, neither side further from 64 bits than the other; a
// probability on a rounding boundary may then fall to either side.
// A chunk is `cw` key blocks and belongs to ONE wavefront, which takes all heads of the KV group at once (a row or
// column of the matrix tiles each: up to 8 heads cost the matrix instructions of one), with tiles in its own LDS and no
// barrier between its blocks.  Four chunks that follow each other make a workgroup,
// whose partials are added up in LDS before they are written.
// Measured against the walk, whole calls or serving steps: 301 -> 74 us for one sequence of 131072 tokens and 32/8 heads,
// 306 -> 43 us for one of 32768, 544 -> 192 us for eight of 16384-32768 tokens and 64/8 heads at a 10 % budget (scores pass
// 70 us, values pass 77 us).
// What bounds it: for short caches the latency of the chain of launches; for long ones the bytes (the scores travel through
// memory once more, 8 bytes per head and token next to 136 bytes of codes and scales per token), of which too few are in
// flight: 4.9 to 5.7 TB/s read and written, against 7.1 of a plain streaming read, with 1.6 to 2.5 wavefronts per SIMD.
#include <type_traits>

#include "thrift_launch.h"
#include "thrift_row.h"

namespace thrift {

namespace {

struct SplitWork {
  int b, kvh;
  int item;            // partial slot of the workgroup
  int j0, j1;          // key blocks of this wavefront (may be none)
  int first_chunk;     // first chunk of the partition
  int chunk;           // this wavefront's chunk
  int n_valid;         // tokens of a block: 64, or those of a partly filled last block
  bool any;            // the workgroup has work
  bool tail;           // the partly filled last block, a partition of its own
};

__device__ __forceinline__ SplitWork split_work(const DecodeSplitArgs& s, int wave) {
  const DecodeArgs& a = s.a;
  SplitWork w;
  const int unit = blockIdx.x / s.items, item = blockIdx.x % s.items;
  w.b = unit / a.Hkv; w.kvh = unit % a.Hkv; w.item = item;
  const int len = a.seqlens ? min(a.Nkv, max(0, a.seqlens[w.b])) : a.Nkv;
  const int full = len / kBk, rest = len % kBk;
  w.n_valid = kBk;
  w.chunk = item * 4 + wave;
  w.tail = item == a.nsplit * s.nsub;
  if (w.tail) {
    w.any = rest > 0;
    w.j0 = full; w.j1 = full + (rest > 0 && wave == 0 ? 1 : 0);
    w.n_valid = rest;
    w.first_chunk = w.chunk;
  } else {
    const int part = item / s.nsub, p0 = part * a.split_blocks, p1 = min(p0 + a.split_blocks, full);
    const int base = p0 + (item % s.nsub) * 4 * s.cw;
    w.any = base < p1;
    w.j0 = min(base + wave * s.cw, p1);
    w.j1 = min(w.j0 + s.cw, p1);
    w.first_chunk = part * s.nsub * 4;
  }
  return w;
}

// Which heads of the group have promoted which of the (at most 32) blocks j0 .. : lane u < G holds head u's bits, bit 0 =
// block j0.
static_assert(kSplitMaxChunk <= 32, "one word of bits per chunk");
__device__ __forceinline__ uint32_t promoted_bits(const DecodeArgs& a, size_t group0, int G, int j0, int lane) {
  if (a.bitmap == nullptr || lane >= G) return 0u;
  const unsigned long long* bm = a.bitmap + (group0 + lane) * a.bitmap_words;
  const int w = j0 >> 6, sh = j0 & 63;
  unsigned long long bits = bm[w] >> sh;
  if (sh != 0 && w + 1 < a.bitmap_words) bits |= bm[w + 1] << (64 - sh);
  return (uint32_t)bits;
}
// mask over the heads for block j0 + i
__device__ __forceinline__ int promoted_mask(uint32_t bits, int i) {
  return (int)__builtin_amdgcn_ballot_w64(((bits >> i) & 1u) != 0u);
}

template <typename T>
__device__ __forceinline__ v4f mfma16(v8s x, v8s y, v4f acc) {
  if constexpr (std::is_same_v<T, F16>)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, x), __builtin_bit_cast(v8h, y), acc, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, x), __builtin_bit_cast(v8bf, y), acc, 0, 0, 0);
}

}  // namespace

// Matrix tiles: 16 x 16, one operand row or column per head (up to 8 of 16 used) and 16 keys or channels.  Lane = 16 g + r:
//   A operand  row r,    contraction slots of group g (32 codes of MXFP4 with a scale each, or 8 elements of 16 bits)
//   B operand  column r, the same slots
//   C / D      column r, rows 4 g + i in register i
// All 128 channels of a 4-bit score are one instruction, and a wavefront's load of 16 keys x 64 bytes is 1 KiB in a row.

// largest value over the lanes that hold the same head (lane % NH), in every one of them: first of each 32 lanes
template <int NH>
__device__ __forceinline__ float head_max32(float v) {
  if constexpr (NH <= 1) v = fmaxf(v, dpp_f<0x121>(v));        // row_ror: lane i of 16 reads lane i - n
  if constexpr (NH <= 2) v = fmaxf(v, dpp_f<0x122>(v));
  if constexpr (NH <= 4) v = fmaxf(v, dpp_f<0x124>(v));
  v = fmaxf(v, dpp_f<0x128>(v));
  const uint32_t b = __float_as_uint(v);
  const auto s = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
template <int NH>
__device__ __forceinline__ float head_sum(float v) {
  if constexpr (NH <= 1) v += dpp_f<0x121>(v);
  if constexpr (NH <= 2) v += dpp_f<0x122>(v);
  if constexpr (NH <= 4) v += dpp_f<0x124>(v);
  v += dpp_f<0x128>(v);
  const uint32_t b = __float_as_uint(v);
  const auto s = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  v = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  return v + other_half(v);
}

// TopK of one row of at most 64 MAXC order keys by one wavefront: word c of the bitmap to out[c].  The k-th largest key is
// searched bit by bit from the top, a step being a comparison and a scalar count per 64 keys: no barrier and no LDS, which
// is what a step of the kernel of its own (decode_select_kernel) waits for.  Ties go to the smaller block id.
template <int MAXC>
__device__ __forceinline__ void wave_select(const uint64_t* keys, int vis, int k, int lane, unsigned long long* out) {
  uint64_t key[MAXC];
#pragma unroll
  for (int c = 0; c < MAXC; ++c) key[c] = c * 64 + lane < vis ? keys[c * 64 + lane] : 0ULL;   // a key is never 0
  uint64_t T = 0;
  if (k < vis) {
    // the upper words alone separate the keys but for a step or two: 32-bit comparisons, none above the largest key
    uint32_t hi[MAXC], top = 0;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
      hi[c] = (uint32_t)(key[c] >> 32);
      top = max(top, hi[c]);
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) top = max(top, (uint32_t)__shfl_xor((int)top, d));
    top = __builtin_amdgcn_readfirstlane(top);
    uint32_t t = 0;
    int n = 0;
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t cand = t | (1u << bit);
      if (cand > top) continue;                            // no key
      n = 0;
#pragma unroll
      for (int c = 0; c < MAXC; ++c)
        if (c * 64 < vis) n += __popcll(__ballot(hi[c] >= cand));
      if (n >= k) t = cand;
      if (n == k) break;                                   // exactly the k largest lie at or above cand
    }
    T = (uint64_t)t << 32;
    if (n != k)
      for (int bit = 31; bit >= 0; --bit) {
        const uint64_t cand = T | (1ULL << bit);
        n = 0;
#pragma unroll
        for (int c = 0; c < MAXC; ++c)
          if (c * 64 < vis) n += __popcll(__ballot(key[c] >= cand));
        if (n >= k) T = cand;
        if (n == k) break;
      }
  }
  int n_gt = 0;
#pragma unroll
  for (int c = 0; c < MAXC; ++c)
    if (c * 64 < vis) n_gt += __popcll(__ballot(key[c] > T));
  const int need = k - n_gt;                               // keys equal to T that are taken
  int seen = 0;
  const uint64_t below = (1ULL << lane) - 1ULL;
#pragma unroll
  for (int c = 0; c < MAXC; ++c) {
    const bool tie = c * 64 + lane < vis && key[c] == T;
    const uint64_t ties = __ballot(tie);
    const uint64_t sel = __ballot(key[c] > T || (tie && seen + __popcll(ties & below) < need));
    seen += __popcll(ties);
    if (lane == 0) out[c] = sel;
  }
}

// NH: heads per KV group, rounded up to 1, 2, 4 or 8.  SELECT: the promoted blocks come from the order keys, selected by every
// workgroup for itself (one row per wavefront) while its first tile is on its way; the first workgroup of a (sequence, KV head)
// leaves the bitmap for the pass behind.  A step of a serving loop, with and without a launch for the selection: 26.2 / 28.8 us
// (1 x 4096 tokens, 32/8 heads), 40.4 / 41.9 us (1 x 32768), 52.8 / 56.1 us (16 x 8192), 176.4 / 178.1 us (16 x 32768).
template <typename T, int NH, bool SELECT>
__global__ void __launch_bounds__(256, 4) decode_split_scores_kernel(DecodeSplitArgs s) {
  const DecodeArgs& a = s.a;
  __shared__ __align__(1024) unsigned char half_tiles[4][kTile16 / 2];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitWork w = split_work(s, wave);
  if (SELECT ? !w.any && w.item != 0 : w.j0 >= w.j1) return;       // uniform over the workgroup where there is a barrier below
  const int G = a.Hq / a.Hkv;
  const size_t group0 = (size_t)w.b * a.Hq + (size_t)w.kvh * G, kh = (size_t)w.b * a.Hkv + w.kvh;
  const uint8_t* k4base = a.k4 + kh * a.Nkv * 64;
  const uint8_t* ksbase = a.ks + kh * a.Nkv * 4;
  const uint8_t* k16base = reinterpret_cast<const uint8_t*>(a.k16 + kh * a.Nkv * kD);
  const uint32_t k4off = (uint32_t)(64 * r + 16 * g), ksoff = (uint32_t)(4 * r + g);   // key 16t + r, channels 32g .. 32g + 31

  const int all = (1 << G) - 1;

  struct Keys {
    v4i k[4];            // key 16t + r, channels 32g .. 32g + 31
    uint32_t ks[4];      // their scale
  };
  auto load4 = [&](int j) {
    Keys x;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      x.k[t] = *reinterpret_cast<const v4i*>(k4base + (size_t)j * 4096 + k4off + 1024 * t);
      x.ks[t] = (ksbase + (size_t)j * 256)[ksoff + 64 * t];
    }
    return x;
  };
  // a block that every head takes in 16 bits is not read in 4
  Keys next;
  uint32_t bits;
  int Mnext;
  if constexpr (SELECT) {
    static_assert(NH <= 4, "a row per wavefront");
    __shared__ unsigned long long sel[NH][kSplitSelectBlocks / 64];
    const int vis = a.seqlens ? (min(a.Nkv, max(0, a.seqlens[w.b])) + kBk - 1) / kBk : a.Nkv / kBk;
    const int k = decode_row_budget(vis, s.fixed_k, s.ppm);
    if (w.j0 < w.j1 && k < vis) next = load4(w.j0);
    if (wave < G) wave_select<kSplitSelectBlocks / 64>(s.keys + (group0 + wave) * (a.Nkv / kBk), vis, k, lane, sel[wave]);
    __syncthreads();
    if (w.item == 0 && tid < NH * (kSplitSelectBlocks / 64)) {
      const int u = tid / (kSplitSelectBlocks / 64), word = tid % (kSplitSelectBlocks / 64);
      if (u < G && word < a.bitmap_words) s.select_out[(group0 + u) * a.bitmap_words + word] = sel[u][word];
    }
    if (w.j0 >= w.j1) return;
    bits = 0u;
    if (lane < G) {
      const int word = w.j0 >> 6, sh = w.j0 & 63;
      unsigned long long x = sel[lane][word] >> sh;
      if (sh != 0 && word + 1 < kSplitSelectBlocks / 64) x |= sel[lane][word + 1] << (64 - sh);
      bits = (uint32_t)x;
    }
    Mnext = promoted_mask(bits, 0);
  } else {
    bits = promoted_bits(a, group0, G, w.j0, lane);
    Mnext = promoted_mask(bits, 0);
    if (Mnext != all) next = load4(w.j0);
  }

  // the query rows as A operand: head r % NR in row r, so that every lane's accumulator registers i are heads
  // (4 g + i) % NR; the lane quantises the MXFP4 group it carries
  constexpr int NR = NH > 4 ? 8 : 4;
  const int hq = r & (NR - 1);
  const bool qlane = hq < G;
  const uint16_t* qrow = a.q + (group0 + (qlane ? hq : 0)) * kD;
  v4i qf4 = {0, 0, 0, 0};
  uint32_t qsc = 127u;
  if (qlane) {
    const uint4* src = reinterpret_cast<const uint4*>(qrow + 32 * g);
    uint32_t pair[16], codes[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint4 x = src[t];
      pair[4 * t] = x.x; pair[4 * t + 1] = x.y; pair[4 * t + 2] = x.z; pair[4 * t + 3] = x.w;
    }
    qsc = quantize_group32<T>(pair, codes);
    qf4 = (v4i){(int)codes[0], (int)codes[1], (int)codes[2], (int)codes[3]};
  }

  // The lane keeps NS scores of NV heads: with four rows of heads, key `lane` (tile g of the four); with eight, heads
  // 4 (g & 1) + i of the keys 16 (g >> 1) + r and 32 more.
  constexpr int NS = NH > 4 ? 2 : 1, NV = NH > 4 ? 4 : NH;
  const int h0 = NH > 4 ? 4 * (g & 1) : 0, key0 = NH > 4 ? 16 * (g >> 1) + r : lane;
  auto mine = [&](const v4f (&acc)[4], float (&v)[NS][NV]) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if constexpr (NH > 4) {
        v[0][i] = g >= 2 ? acc[1][i] : acc[0][i];
        v[1][i] = g >= 2 ? acc[3][i] : acc[2][i];
      } else {
        const float lo = g & 1 ? acc[1][i] : acc[0][i], hi = g & 1 ? acc[3][i] : acc[2][i];
        v[0][i] = g >= 2 ? hi : lo;
      }
    }
  };
  const unsigned char* half_tile = half_tiles[wave];
  const uint32_t lds0 = lds_address(half_tile);
  float top[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) top[i] = kEmptyMax;
  float* out = s.scores + (group0 + h0) * a.Nkv + key0;
  for (int j = w.j0; j < w.j1; ++j) {
    const int M = Mnext;
    float v4[NS][NV], v16[NS][NV];
    if (M != all) {
      v4f acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(widen(qf4), widen(next.k[t]), (v4f){0.f, 0.f, 0.f, 0.f}, 4, 4, 0, qsc, 0, next.ks[t]);
      mine(acc, v4);
    }
    Mnext = j + 1 < w.j1 ? promoted_mask(bits, j + 1 - w.j0) : all;
    if (Mnext != all) next = load4(j + 1);
    if (M != 0) {
      // Half a tile of 32 keys at a time through the wavefront's own LDS: a DMA instruction reads four whole rows, and only
      // reads of whole lines may carry the streaming hint (fragments read from memory directly are 64 bytes of a line each).
      // Rows past the cached tokens reach only their own keys' scores, which are masked below.
      const uint8_t* tile = k16base + (size_t)__builtin_amdgcn_readfirstlane(j) * kTile16;
      v4f acc[4];
      v8s qf[4];
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
        qf[s4] = qlane ? *reinterpret_cast<const v8s*>(qrow + 32 * s4 + 8 * g) : (v8s){0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the reads of the half before are over
        // row 4 q + g of the half; its chunk c stands at position c ^ (row & 7)
#pragma unroll
        for (int q = 0; q < 8; ++q)
          dma_b128<true>(tile + 8192 * hf + 1024 * q, (uint32_t)(256 * g + 16 * (r ^ (4 * (q & 1) + g))), lds0 + 1024 * q);
        vm_wait<0>();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          acc[2 * hf + t] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4)
            acc[2 * hf + t] = mfma16<T>(qf[s4], *reinterpret_cast<const v8s*>(half_tile + 4096 * t + 256 * r + 16 * ((4 * s4 + g) ^ (r & 7))), acc[2 * hf + t]);
        }
      }
      mine(acc, v16);
    }
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if (h0 + i < G) {
          float v = ((M >> (h0 + i)) & 1) ? v16[q][i] : v4[q][i];
          if (key0 + 32 * q >= w.n_valid) v = -INFINITY;
          __builtin_nontemporal_store(v, out + (size_t)i * a.Nkv + (size_t)j * kBk + 32 * q);
          top[i] = fmaxf(top[i], v);
        }
  }
  if (w.tail) return;                                          // a partition of its own: no chunk follows it
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    float m = top[i];                                          // over the 16 keys of the lane's row of lanes, then over the rows with the same heads
    m = fmaxf(m, dpp_f<0x121>(m));
    m = fmaxf(m, dpp_f<0x122>(m));
    m = fmaxf(m, dpp_f<0x124>(m));
    m = fmaxf(m, dpp_f<0x128>(m));
    if constexpr (NH <= 4) {
      const uint32_t b = __float_as_uint(m);
      const auto sw = __builtin_amdgcn_permlane16_swap(b, b, false, false);
      m = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    m = fmaxf(m, other_half(m));
    if (r == 0 && g < (NH > 4 ? 2 : 1) && h0 + i < G) s.cmax[(group0 + h0 + i) * s.chunks + w.chunk] = m;
  }
}

// Softmax layout: lane = NH kg + h holds the NH keys NH kg .. of head h, so that every step of the recurrence that is not
// an exponential costs the heads of a group one instruction together, and each 32 lanes hold one MXFP4 group of P per head.
// The operands of P.V (column = head) are formed through a few hundred bytes of the wavefront's own LDS.
// The accumulators hold channel 8 (4 g + i) + e of head r in o[e][i]: row r of tile e is channel 8 r + e, because a lane's
// 16 bytes of a 16-bit V row are 8 neighbouring channels, which are transposed against 8 rows inside the lane.
template <typename T, int NH>
__global__ void __launch_bounds__(256, 4) decode_split_values_kernel(DecodeSplitArgs s) {
  const DecodeArgs& a = s.a;
  constexpr int kSlot = 4096 + 256;                            // codes and scales of a V block
  __shared__ __align__(1024) unsigned char slots[4][2][kSlot]; // per wavefront; its partial sums at the end
  __shared__ __align__(16) uint16_t prow[4][NH * 64];          // probabilities rounded to 16 bits: [head][key]
  __shared__ __align__(16) uint8_t pcode[4][NH * 32];          // codes of P: [head][key / 2]
  __shared__ uint8_t pscale[4][NH * 2];                        // their E8M0 bytes: [head][group]
  __shared__ float ml[4][NH][2];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitWork w = split_work(s, wave);
  if (!w.any) return;                                          // uniform over the workgroup
  const int G = a.Hq / a.Hkv;
  const size_t group0 = (size_t)w.b * a.Hq + (size_t)w.kvh * G, kh = (size_t)w.b * a.Hkv + w.kvh;
  const float c = a.scale * 1.4426950408889634f;

  const int h = lane & (NH - 1), kg = lane / NH;               // softmax layout
  const size_t qh = group0 + min(h, G - 1);                    // lanes of a padding head follow the last one and are never read
  RowState st = {kEmptyMax, 0.f};
  v4f o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (v4f){0.f, 0.f, 0.f, 0.f};

  if (w.j0 < w.j1) {
    const uint8_t* v4base = a.v4 + kh * (size_t)(a.Nkv / 64) * 4096;
    const uint8_t* vsbase = a.vs + kh * (size_t)(a.Nkv / 32) * kD;
    const uint8_t* v16base = reinterpret_cast<const uint8_t*>(a.v16 + kh * a.Nkv * kD);
    const uint32_t v16off = (uint32_t)(2048 * g + 16 * r);
    // The 4-bit tile of a block travels one block ahead of the arithmetic by LDS DMA, whole lines per instruction.  Its 256
    // bytes of channels 8 R .. 8 R + 7 hold chunk c (channel 8 R + c / 2, token group c & 1) at position c ^ R, so that the
    // 16 rows of a fragment lie in different banks.
    const uint32_t lds0 = lds_address(&slots[wave][0][0]);
    const uint32_t dma_off = (uint32_t)(256 * g + 16 * (r ^ g));              // R = 4 m + g in instruction m
    auto issue4 = [&](int j, int slot) {
      const int j_ = __builtin_amdgcn_readfirstlane(j);
      const uint32_t to = lds0 + (uint32_t)(__builtin_amdgcn_readfirstlane(slot) * kSlot);
      uint32_t off = dma_off;
      asm volatile("" : "+v"(off));                            // one offset kept, not four
#pragma unroll
      for (int m = 0; m < 4; ++m) dma_b128<true>(v4base + (size_t)j_ * 4096 + 1024 * m, off ^ (64u * m), to + 1024 * m);
      dma_b32<true>(vsbase + (size_t)j_ * 256, (uint32_t)(4 * lane), to + 4096);
    };
    const float* sbase = s.scores + group0 * a.Nkv;                          // scalar; the lane's head and keys in 32 bits
    const uint32_t soff = (uint32_t)(min(h, G - 1) * a.Nkv + NH * kg);
    uint16_t* prow_w = prow[wave];
    uint8_t* pcode_w = pcode[wave];
    uint8_t* pscale_w = pscale[wave];
    const uint32_t bits = promoted_bits(a, group0, G, w.j0, lane);
    const int all = (1 << G) - 1, n_blocks = w.j1 - w.j0;
    struct Scores { float v[NH]; };
    auto load_scores = [&](int j) {
      Scores x;
      if constexpr (NH >= 4) {
#pragma unroll
        for (int u = 0; u < NH; u += 4) {
          const float4 y = *reinterpret_cast<const float4*>(sbase + (size_t)j * kBk + soff + u);
          x.v[u] = y.x; x.v[u + 1] = y.y; x.v[u + 2] = y.z; x.v[u + 3] = y.w;
        }
      } else {
#pragma unroll
        for (int u = 0; u < NH; ++u) x.v[u] = (sbase + (size_t)j * kBk)[soff + u];
      }
      return x;
    };
    // keys 32 q + 8 g .. + 7 of block j, channels 8 r ..
    auto load16 = [&](int j, int q, v4i (&row)[8]) {
      const uint8_t* tile = v16base + (size_t)j * kTile16 + 8192 * q;
#pragma unroll
      for (int u = 0; u < 8; ++u) row[u] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(tile + v16off + 256 * u));
    };
    // rows past the cached tokens hold whatever lies there, and zero times that need not be zero
    auto clear16 = [&](int q, v4i (&row)[8]) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (32 * q + 8 * g + u >= w.n_valid) row[u] = (v4i){0, 0, 0, 0};
    };
    int Mnext = promoted_mask(bits, 0);
    if (Mnext != all) issue4(w.j0, 0);
    Scores next = load_scores(w.j0);
    // running maximum in front of the chunk
    const int ahead = w.chunk - w.first_chunk;
    if (ahead > 0) {
      const float* cm = s.cmax + qh * s.chunks + w.first_chunk;
      float m = kEmptyMax;
      for (int e = kg; e < ahead; e += 64 / NH) m = fmaxf(m, cm[e]);
      m = head_max32<NH>(m);
      st.m = fmaxf(m, other_half(m));
    }
    for (int i = 0; i < n_blocks; ++i) {
      const int j = w.j0 + i;
      const int M = Mnext;
      // everything in flight was asked for a block ago: the scores of this one and its 4-bit tile.  The statements on the
      // registers keep the compiler from waiting for the scores again behind the loads issued next.
      vm_wait<0>();
      Scores x = next;
#pragma unroll
      for (int u = 0; u < NH; ++u) asm volatile("" : "+v"(x.v[u]));
      v4i v[8];
      if (M != 0) load16(j, 0, v);                             // needed after the softmax
      Mnext = i + 1 < n_blocks ? promoted_mask(bits, i + 1) : all;
      if (Mnext != all) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the reads of the slot's last block are over
        issue4(j + 1, (i + 1) & 1);
      }
      if (i + 1 < n_blocks) next = load_scores(j + 1);
      // ---- online softmax (Alg. 1 steps 10-12 / 16-17) of all heads ----
      float gmax = x.v[0];
#pragma unroll
      for (int u = 1; u < NH; ++u) gmax = fmaxf(gmax, x.v[u]);
      gmax = head_max32<NH>(gmax);                             // the lane's 32-key group
      const uint32_t gb = __float_as_uint(gmax);
      const auto s32 = __builtin_amdgcn_permlane32_swap(gb, gb, false, false);
      const float m_new = max3(st.m, __uint_as_float(s32[0]), __uint_as_float(s32[1]));
      if (__builtin_amdgcn_ballot_w64(m_new != st.m) != 0ULL) {
        const float alpha = fast_exp2((st.m - m_new) * c);     // lane 16 g + r, r < NH: head r, which is also its column of o
        st.l *= alpha;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] *= alpha;
        st.m = m_new;
      }
      int ex;
      {
        const float d = (gmax - m_new) * c;                    // the group maximum maps to exactly 2^floor(d) or above
        asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(ex) : "v"(d));
      }
      const uint32_t pb = (uint32_t)max(ex + 125, 1);
      const float pscale_f = __uint_as_float(pb << 23), mc = m_new * c;
      float p[NH];
#pragma unroll
      for (int u = 0; u < NH; ++u) {
        p[u] = fast_exp2(__builtin_fmaf(x.v[u], c, -mc));
        st.l += p[u];
      }
      if (M != all) {
        if constexpr (NH == 1) {
          const float nb = dpp_f<kDppSwap1>(p[0]);
          const uint32_t code = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, p[0], nb, pscale_f, 0);
          if ((lane & 1) == 0) pcode_w[lane >> 1] = (uint8_t)code;
        } else {
          uint32_t code = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, p[0], p[1], pscale_f, 0);
          if constexpr (NH >= 4) code = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(code, p[2], p[3], pscale_f, 1);
          if constexpr (NH == 8) {
            code = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(code, p[4], p[5], pscale_f, 2);
            code = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(code, p[6], p[7], pscale_f, 3);
          }
          uint8_t* to = pcode_w + h * 32 + kg * (NH / 2);
          if constexpr (NH == 8) *reinterpret_cast<uint32_t*>(to) = code;
          else if constexpr (NH == 4) *reinterpret_cast<uint16_t*>(to) = (uint16_t)code;
          else *to = (uint8_t)code;
        }
        if ((lane & 31) < NH) pscale_w[h * 2 + (lane >> 5)] = (uint8_t)pb;
        // column r = head r, slots 32 g ..: zeros for padding columns, for the slots past the block's 64 keys and for the
        // heads that take the block in 16 bits
        v4i pq = {0, 0, 0, 0};
        uint32_t pbl = 127u;
        if (r < G && g < 2 && ((M >> r) & 1) == 0) {
          pq = *reinterpret_cast<const v4i*>(pcode_w + r * 32 + g * 16);
          pbl = pscale_w[r * 2 + g];
        }
        const v8i pq8 = widen(pq);
        const unsigned char* slot = slots[wave][i & 1];
        const uint2 vs = *reinterpret_cast<const uint2*>(slot + 4096 + (g & 1) * kD + 8 * r);
        const uint32_t frag = (uint32_t)(256 * r + 16 * (r ^ (g & 1)));     // groups 2 and 3 meet zeros of P: anything finite
#define THRIFT_PV4(E) o[E] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(widen(*reinterpret_cast<const v4i*>(slot + (frag ^ (32u * (E))))), pq8, o[E], 4, 4, (E) & 3, (E) < 4 ? vs.x : vs.y, 0, pbl);
        THRIFT_PV4(0) THRIFT_PV4(1) THRIFT_PV4(2) THRIFT_PV4(3) THRIFT_PV4(4) THRIFT_PV4(5) THRIFT_PV4(6) THRIFT_PV4(7)
#undef THRIFT_PV4
      }
      if (M != 0) {
        int lane_ = lane;                                      // addresses formed here, not kept through the 4-bit blocks
        asm volatile("" : "+v"(lane_));
        const int r_ = lane_ & 15, g_ = lane_ >> 4;
#pragma unroll
        for (int u = 0; u < NH; ++u) prow_w[(lane_ & (NH - 1)) * 64 + NH * (lane_ / NH) + u] = T::from_float(p[u]);
        const bool mine = r_ < G && ((M >> r_) & 1) != 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {                          // keys 32 q + 8 g .. + 7
          if (q == 1) {
            __builtin_amdgcn_sched_barrier(0);                 // into the registers of the first half
            load16(j, 1, v);
          }
          if (w.n_valid != kBk) clear16(q, v);
          const v8s pf = mine ? *reinterpret_cast<const v8s*>(prow_w + r_ * 64 + 32 * q + 8 * g_) : (v8s){0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            v4i col;
#pragma unroll
            for (int u = 0; u < 4; ++u) col[u] = (int)__builtin_amdgcn_perm((uint32_t)v[2 * u + 1][e >> 1], (uint32_t)v[2 * u][e >> 1], sel);
            // zero times an infinity or NaN of V is not zero: the heads that take the block in 4 bits keep their sums
            const v4f sum = mfma16<T>(__builtin_bit_cast(v8s, col), pf, o[e]);
            o[e] = mine ? sum : o[e];
            asm volatile("" : "+v"(o[e]));                     // chosen here: both values of all eight tiles do not fit
            if (e & 1) __builtin_amdgcn_sched_barrier(0);      // the transposed pieces are formed as they are used, not all ahead
          }
        }
      }
    }
    static_assert(NH * kD * 4 <= 2 * kSlot, "the sums of a wavefront take the place of its tiles");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (r < G) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float* to = reinterpret_cast<float*>(slots[wave][0]) + r * kD + 8 * (4 * g + i);
        *reinterpret_cast<float4*>(to) = make_float4(o[0][i], o[1][i], o[2][i], o[3][i]);
        *reinterpret_cast<float4*>(to + 4) = make_float4(o[4][i], o[5][i], o[6][i], o[7][i]);
      }
    }
  }
  {
    const float l = head_sum<NH>(st.l);
    if (lane < NH) { ml[wave][lane][0] = st.m; ml[wave][lane][1] = l; }
  }
  __syncthreads();
  // the workgroup's partial.  A wavefront without blocks has left its sums unwritten; it is skipped by its row sum of zero
  // (with a key it is positive, or the whole chunk weighs nothing, or it is NaN and has to reach the result: bits are
  // compared, because comparisons of numbers are compiled as if there were no NaN).
  for (int e = tid; e < G * kD; e += 256) {
    const int u = e >> 7, ch = e & (kD - 1);
    float m = ml[0][u][0];
#pragma unroll
    for (int v = 1; v < 4; ++v) m = fmaxf(m, ml[v][u][0]);
    float l = 0.f, sum = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float lv = ml[v][u][1];
      if (__float_as_uint(lv) != 0u) {
        const float f = fast_exp2((ml[v][u][0] - m) * c);
        l += f * lv;
        sum += f * reinterpret_cast<const float*>(slots[v][0])[u * kD + ch];
      }
    }
    const size_t slot = (group0 + u) * a.nparts + w.item;
    a.part_o[slot * kD + ch] = sum;
    if (ch == 0) { a.part_ml[2 * slot] = m; a.part_ml[2 * slot + 1] = l; }
  }
}

// Log-sum-exp merge of the partials of one (sequence, query head): 32 channel quads x 8 slots at a time, so that the
// loads of all partials are in flight together.  Slots without work were never written: the lengths say which.
__global__ void __launch_bounds__(256) decode_split_merge_kernel(DecodeSplitArgs s) {
  const DecodeArgs& a = s.a;
  __shared__ float4 red[8][32];
  __shared__ float redl[8];
  const int tid = threadIdx.x, lane = tid & 63, quad = tid & 31, row = tid >> 5;
  const size_t qh = blockIdx.x;
  const int b = (int)(qh / a.Hq);
  const int len = a.seqlens ? min(a.Nkv, max(0, a.seqlens[b])) : a.Nkv;
  const int full = len / kBk;
  const int parts = full / a.split_blocks, left = full % a.split_blocks;
  const int used = parts * s.nsub + (left + 4 * s.cw - 1) / (4 * s.cw);     // slots of full blocks: 0 .. used-1
  const bool tail = len % kBk != 0;                                          // and the last one
  const float c = a.scale * 1.4426950408889634f;
  const float* ml = a.part_ml + qh * a.nparts * 2;
  const float* po = a.part_o + qh * a.nparts * kD;
  const int n = used + (tail ? 1 : 0), last = a.nparts - 1;
  float m = -INFINITY;
  for (int p = lane; p < n; p += 64) m = fmaxf(m, ml[2 * (p < used ? p : last)]);
  m = wave_max(m);
  float l = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int p = row; p < n; p += 8) {
    const int slot = p < used ? p : last;
    const float2 x = *reinterpret_cast<const float2*>(ml + 2 * slot);
    const float4 y = *reinterpret_cast<const float4*>(po + (size_t)slot * kD + 4 * quad);
    const float f = fast_exp2((x.x - m) * c);
    l += f * x.y;
    acc.x += f * y.x; acc.y += f * y.y; acc.z += f * y.z; acc.w += f * y.w;
  }
  red[row][quad] = acc;
  if (quad == 0) redl[row] = l;
  __syncthreads();
  if (tid >= kD) return;
  float sum = 0.f, L = 0.f;
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    sum += reinterpret_cast<const float*>(&red[v][0])[tid];
    L += redl[v];
  }
  const float x = L > 0.f ? sum / L : 0.f;
  if (a.out_dt == THRIFT_F32) ((float*)a.out)[qh * kD + tid] = x;
  else if (a.out_dt == THRIFT_F16) ((uint16_t*)a.out)[qh * kD + tid] = F16::from_float(x);
  else ((uint16_t*)a.out)[qh * kD + tid] = BF16::from_float(x);
}

// The split is used where the walk over whole partitions leaves the chip idle.  A walk takes its 256 key blocks one after
// the other whatever else runs, so with fewer workgroups than the CUs take at once (two each) its time does not shrink.
// Groups of more than 8 heads do not fit the row layout.  Partitions of at most 16 blocks are short walks already.
// Above kSplitMaxItems the walk is the faster one (32/8 heads at 5 %, walk / two passes: 315 / 322 us for 6 x 131072 tokens,
// 353 / 418 us for 8, 681 / 804 us for 16; 16/8 heads, 16 x 65536: 282 / 321 us), but for one query head per KV head in a
// cache of one or two partitions that has lengths: three of a walk's four wavefronts have no head there, its partitions are
// seldom full, and the scores cost 8 bytes a token.  A serving step with 16/16 heads: 242 / 220 us (16 x 32768 tokens, 5 %),
// 344 / 300 us (25 %), 727 / 586 us (100 %), 255 / 167 us (14 x 24576, 10 %); without lengths 249 / 266 us (8 x 65536, 5 %).
bool decode_split_wanted(int B, int Hq, int Hkv, int nsplit, int split_blocks, bool lengths) {
  if (Hq / Hkv > 8) return false;
  if (nsplit > 1 && split_blocks <= 16) return false;
  return (long)B * Hkv * nsplit <= (lengths && Hq == Hkv && nsplit <= 2 ? kSplitMaxItemsOneHead : kSplitMaxItems);
}

// With more heads a wavefront would select two rows one after the other: 58.6 us against 57.5 us for 2 x 20480 tokens, 64/8 heads.
bool decode_split_selects(int Hq, int Hkv, int Tk) { return Hq / Hkv <= 4 && Tk <= kSplitSelectBlocks; }

// Key blocks per wavefront: eight to sixteen wavefronts per CU where there are so many blocks, one block each below that.  Longer
// chunks are longer serial chains, shorter ones more partials and more running maxima to look up.  Chunks of 1 / 2 / 4 / 8,
// whole serving steps or calls in us (B x tokens, heads, budget):
//    512 blocks   1 x 4096, 32/8, 5 %      27.9 /  31.6 /  33.7 /  41.3   takes 1
//   4096          1 x 32768, 32/8, 5 %     47.7 /  41.4 /  43.9 /  49.2         2
//                 1 x 16384, 16/16, 5 %    37.8 /  31.9 /  32.4 /  36.4         2
//  16384          1 x 131072, 32/8, 5 %    99.9 /  81.3 /  76.2 /  76.5         8
//                 16 x 8192, shared, 5 %   79.2 /  60.2 /  54.6 /  54.6         8
//                 4 x 32768, 32/8, 5 %     94.2 /  74.9 /  68.9 /  74.6         8
//                 4 x 32768, 64/8, 100 %  128.5 / 124.0 / 122.8 / 142.7         8
//  32768          8 x 32768, 64/8, 10 %   193.4 / 175.5 / 174.1 / 171.3         8
//                 16 x 16384, 32/8, 5 %   146.5 / 108.2 /  98.8 / 102.6         8
//  65536          16 x 32768, 32/8, 25 %  367.3 / 319.2 / 315.2 / 318.0         8
//                 8 x 32768, 16/16, 10 %  209.6 / 150.2 / 128.0 / 126.3         8
// The line between 4 and 8 is not the best one for all of them: few sequences of uneven lengths would gain up to 14 % by 4, others
// lose 1 to 2 %.
int decode_split_chunk(int B, int Hkv, int Tk) {
  const long blocks = (long)B * Hkv * Tk;
  int cw = 1;
  while (cw < kSplitMaxChunk && blocks >= 4096L * cw) cw *= 2;
  return cw;
}

void launch_decode_split(const DecodeSplitArgs& s, hipStream_t st) {
  const DecodeArgs& a = s.a;
  const dim3 grid((unsigned)((long)a.B * a.Hkv * s.items)), block(256);
  const int G = a.Hq / a.Hkv;
#define THRIFT_SPLIT(T, NH)                                            \
  do {                                                                 \
    if (s.keys != nullptr) decode_split_scores_kernel<T, NH, (NH <= 4)><<<grid, block, 0, st>>>(s);  \
    else decode_split_scores_kernel<T, NH, false><<<grid, block, 0, st>>>(s);                        \
    decode_split_values_kernel<T, NH><<<grid, block, 0, st>>>(s);      \
  } while (0)
#define THRIFT_SPLIT_T(T)                  \
  do {                                     \
    if (G <= 1) THRIFT_SPLIT(T, 1);        \
    else if (G <= 2) THRIFT_SPLIT(T, 2);   \
    else if (G <= 4) THRIFT_SPLIT(T, 4);   \
    else THRIFT_SPLIT(T, 8);               \
  } while (0)
  if (a.dt == THRIFT_F16) THRIFT_SPLIT_T(F16);
  else THRIFT_SPLIT_T(BF16);
#undef THRIFT_SPLIT_T
#undef THRIFT_SPLIT
  decode_split_merge_kernel<<<dim3((unsigned)((long)a.B * a.Hq)), block, 0, st>>>(s);
}

}  // namespace thrift
