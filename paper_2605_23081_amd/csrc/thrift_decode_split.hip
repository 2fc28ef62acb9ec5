// Decode for caches that give the one-workgroup-per-partition walk too few workgroups (short caches, few sequences).
//
// The rounding of P follows the running maximum of the partition, so a partition cannot simply be cut into shorter
// recurrences.  It can be computed in two passes over chunks of a few key blocks:
//   scores  the raw scores of every (query head, key) and the largest score of every chunk;
//   values  softmax, P quantiser and P.V of a chunk, started from the largest score of the chunks in front of it in the
//           partition: every block sees the running maximum of its partition, as in the serial walk.
// A chunk belongs to ONE wavefront, which takes all heads of the KV group at once (a row or column of the matrix tiles each: up
// to 8 heads cost the matrix instructions of one), with tiles in its own LDS and no barrier between its blocks.  Four chunks
// that follow each other make a workgroup, whose partials are added up in LDS before they are written.
//
// Short sequences and many key blocks in all take one launch (pass BOTH): the scores stay in LDS instead of travelling through
// memory twice (8 bytes per head and token next to 136 bytes of codes and scales), and V tiles of some workgroups fill the time
// in which others wait for K.  There a workgroup publishes its largest scores and waits for those of the workgroups in front of
// it in the partition.  Workgroups take their places in a partition by a ticket as they start, so that they wait only for
// workgroups that run already and themselves wait only for still earlier ones: every wait ends, whatever else occupies the
// chip.  Few workgroups with long partitions would mostly wait; there the passes are two launches.
//
// The scores come from 16 x 16 instead of 32 x 32 matrix instructions.  16-bit scores had equal bits in all of 16 million
// compared; a 4-bit score is exact in both where the products of a row's group scales lie within 2^9 (14 bits hold the sum of
// 128 products of two codes), so that all codes of P are the walk's and only the order of the fp32 sums differs.  With scales
// spread over 2^40, 2.8 % of the scores differed in their last bit, neither side further from 64 bits than the other; a
// probability on a rounding boundary may then fall to either side.
//
// Measured, whole calls or serving steps, every pass on buffers of its own (figures below that are said to be back to back repeat one
// pass, which takes 3 to 7 % less), the walk / two launches with a search for every selection / now: 306 / 43.2 / 35.9 us
// for one sequence of 32768 tokens and 32/8 heads, 102 / 28.0 / 21.9 for one of 4096; 301 / 74.0 / 64.2 for one of 131072,
// 544 / 192.4 / 153.8 for eight of 16384-32768 with 64/8 heads at 10 %, 148 / 53.4 / 43.9 for sixteen of 4096-8192 with shared
// selection; back to back - / 324.5 / 261.9 for sixteen of 16384-32768 at 25 %.
// What bounds it: for short caches the chain of launches and of dependent loads inside them (a step of one sequence of 4096 tokens
// reads 0.5 MB; in its 11 us launch 2.0 until the length, the place and the query are there, 1.2 to the first score, 1.0 scores, 2.6 for the
// maxima in front, 0.9 values, 1.4 the sums); for long ones a workgroup's 11 us without tiles in flight (start, wait and end of 30) and
// the last, nearly empty round.
#include <type_traits>

#include "thrift_launch.h"
#include "thrift_row.h"

namespace thrift {

namespace {

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

// Which of the blocks first .. first + n - 1 (at most 32) belong to the k largest of a row's order keys, ties to the smaller
// block id: bit i for block first + i (own: lane i holds its key).  By one wavefront that holds the row, 64 keys per register.
// A block is taken if fewer than k keys are larger.  A workgroup asks for its own blocks only: the counts for one block, most
// often of the upper words alone, cost what one step of a search for the k-th largest key costs, of which that takes 25 to 30
// one after the other.
template <int NR>
__device__ __forceinline__ uint32_t rank_select(const uint64_t (&key)[NR], uint64_t own, int k, int first, int n, int lane) {
  uint32_t taken = 0u;
  for (int i = 0; i < n; ++i) {
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(own >> 32), i);
    int larger = 0;
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      larger += __popcll(__ballot((uint32_t)(key[c] >> 32) > hi));
      // most blocks are out after two registers: 47.0 -> 46.0 us for a step of 4 x 8192-16384 tokens, 34.7 -> 34.4 for 1 x 32768
      if (c % 2 != 0 && c + 1 < NR && larger >= k) break;
    }
    if (larger >= k) continue;
    const uint64_t x = ((uint64_t)hi << 32) | (uint32_t)__builtin_amdgcn_readlane((int)own, i);
    larger = 0;                                            // larger, or equal with a smaller id
#pragma unroll
    for (int c = 0; c < NR; ++c) larger += __popcll(__ballot(key[c] > x || (key[c] == x && 64 * c + lane < first + i)));
    if (larger < k) taken |= 1u << i;
  }
  return taken;
}

// What one launch computes: everything (BOTH), or the raw scores and the largest of every chunk (SCORES) and what comes behind
// them (VALUES).
enum Pass { BOTH, SCORES, VALUES };

// Key blocks per wavefront; with both passes in one the LDS holds their scores.
constexpr int chunk_limit(int nh, bool both) { return both && nh > 4 ? kSplitMaxChunk / 2 : kSplitMaxChunk; }

// Workgroups of four wavefronts that a CU holds, which is also the wavefronts per SIMD whose registers the kernel may have: where one
// launch keeps the scores of 32 (block, head) pairs per wavefront its LDS leaves room for two.
constexpr int kBothOwn = 2 * (4096 + 256) + 128;               // LDS of a wavefront beside its scores
constexpr int workgroups_per_cu(Pass pass, int nh, int nc) { return pass != BOTH ? 4 : 4 * (kBothOwn + 256 * nh * nc) <= 160 * 1024 / 3 ? 3 : 2; }

// NH: heads per KV group, rounded up to 1, 2, 4 or 8.
// NC: key blocks per wavefront, at most, whose scores one launch holds in LDS.
// WK: a promoted block's 16-bit K tile is asked for whole, not half by half (load16 says where that pays).
// NR: the promoted blocks come from the order keys of rows of up to 64 NR key blocks, every workgroup asking for its own blocks
// (a row or two per wavefront); 0: from the bitmap of a launch before.
template <typename T, int NH, Pass PASS, int NR, int NC = 1, bool WK = false>
__global__ void __launch_bounds__(256, workgroups_per_cu(PASS, NH, NC)) decode_split_kernel(DecodeSplitArgs s) {
  const DecodeArgs& a = s.a;
  constexpr bool SELECT = NR > 0;
  constexpr bool kWholeV = PASS == BOTH;                       // both halves of a 16-bit V tile are asked for at once
  static_assert(PASS == BOTH || !WK, "two launches have no registers for it");
  constexpr int kSlot = 4096 + 256;                            // codes and scales of a V block
  // per wavefront: half a 16-bit K tile; then two V blocks, which give way to its partial sums, and behind them its
  // maxima and sums
  constexpr int kTops = 2 * kSlot, kMl = kTops + 64, kOwn = PASS == SCORES ? kTile16 / 2 : kMl + 64;
  __shared__ __align__(1024) unsigned char tiles[4][kOwn];
  static_assert(NH * kD * 4 <= 2 * kSlot && kTile16 / 2 <= 2 * kSlot && NH * 8 <= 64, "they take the tile's place");
  // BOTH: raw scores of the wavefront's blocks, [block][head][key]; those of a block give way to what P.V reads: the
  // probabilities rounded to 16 bits [head][key], the codes of P [head][key / 2] and their E8M0 bytes [head][group].  Before the
  // first scores: the workgroup's place in its partition and the heads' selections
  // VALUES: those alone.  With eight heads the area of a block's scores would leave a CU three workgroups instead of four, and 912 of
  // them (2 x 14464 tokens, 64/8 heads, no block promoted) a second round: 20.8 us, now 16.9.
  constexpr int kArea = PASS == VALUES ? (NH * (64 * 2 + 32 + 2) + 15) / 16 * 4 : NH * 64;
  __shared__ __align__(16) float scores[4][NC][kArea];
  static_assert(PASS != BOTH || (kOwn == kBothOwn && kArea == 64 * NH), "workgroups_per_cu");
  static_assert(PASS != VALUES || 4 * (kOwn + 4 * kArea) <= 160 * 1024 / 4, "four workgroups per CU");
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // y: (partition, workgroup of it), or the partly filled last block.  Two launches walk through the cache of one unit after the
  // other; where workgroups wait for each other the first places of all partitions of all units start first.
  const unsigned units = (unsigned)(a.B * a.Hkv), unit_of_grid = PASS == BOTH ? blockIdx.x % units : blockIdx.x / s.items;
  const int y = (int)(PASS == BOTH ? blockIdx.x / units : blockIdx.x % s.items);
  const bool tail = y == a.nsplit * s.nsub;
  const int part = tail ? 0 : PASS == BOTH ? y % a.nsplit : y / s.nsub;
  // What does not depend on the length is asked for before it arrives: the place, the keys, the query.
  // Where workgroups wait for each other they take the places of a partition in the order in which they start: whoever waits
  // below for the ones in front of it waits for workgroups that run already.  (The places of a partition that the sequence does
  // not reach are nobody's.)
  int at = 0;
  if constexpr (PASS == BOTH) {
    if (tid == 0 && !tail) at = (int)atomicAdd(s.tickets + unit_of_grid * a.nsplit + part, 1u);
  }
  int unit = (int)unit_of_grid;
  asm volatile("" : "+s"(unit));                               // scalar behind the branch: the DMA statements take scalar bases
  const int G = a.Hq / a.Hkv;
  const size_t group0 = (size_t)(unit / a.Hkv) * a.Hq + (size_t)(unit % a.Hkv) * G, kh = (size_t)unit;
  constexpr int kRows = NH > 4 ? 2 : 1;                        // rows of keys per wavefront: heads wave, wave + 4
  uint64_t key[kRows][SELECT ? NR : 1];
  const int Tk = a.Nkv / kBk;
  // the query rows as A operand: head r % 4 (8) in row r, so that every lane's accumulator registers i are heads
  // (4 g + i) % 4 (8); the lane quantises the MXFP4 group it carries
  const int h = lane & (NH - 1), kg = lane / NH;               // softmax layout
  const int hg = min(h, G - 1);                                // lanes of a padding head follow the last one and are never read
  // In two launches the workgroup's place is known, too: the keys of its own blocks; its selection, the largest scores in front of
  // it in the partition and the scores of its first block.  What stands there may never have been written: it is used where the
  // length says that it was.  Asked for one after the other behind the length they took 2.7 us of the 12 us of the values pass, now 0.7:
  // 35.5 -> 34.4 us for 1 x 32768 tokens, 32/8 heads, 5 %, 37.4 -> 36.0 for 2 x 16384 at 10 %, 30.0 -> 29.2 for 1 x 16384.
  const int early = min(part * a.split_blocks + y % s.nsub * 4 * s.cw, Tk - 1);          // (not of a partly filled last block)
  uint64_t own_key[kRows];
  if constexpr (SELECT && PASS == SCORES) {
#pragma unroll
    for (int u = 0; u < kRows; ++u) own_key[u] = s.keys[(group0 + min(wave + 4 * u, G - 1)) * Tk + min(early + lane, Tk - 1)];
  }
  // The first maxima in front, 64 / NH of a head per load: 64 of one head, 128 of two or four, 64 of eight.  Lanes without one read the
  // last again: loads under conditions of their own, and more of them than the longest partition has use for, cost more than the
  // wait where little else is to do (one head, no block promoted: 33.6 us for 14 x 4416 tokens, 16.9 for 20480, like this 32.9 and 16.5,
  // without 32.6 and 16.4).  Only with eight heads, where a load has few, are conditions better (24.8 / 25.1 us for 1 x 32768, 64/8).
  constexpr int kFront = NH == 1 ? 1 : NH == 2 ? 4 : 8;
  float front[kFront];
  uint32_t own_taken = 0u;
  struct Scores { float v[NH]; };
  const float* sbase = s.scores + group0 * a.Nkv;              // scalar; the lane's head and keys in 32 bits
  const uint32_t soff = (uint32_t)(hg * a.Nkv + NH * kg);
  auto load_scores = [&](int j) {
    Scores x;
    if constexpr (NH >= 4) {
#pragma unroll
      for (int u = 0; u < NH; u += 4) {
        const float4 z = *reinterpret_cast<const float4*>(sbase + (size_t)j * kBk + soff + u);
        x.v[u] = z.x; x.v[u + 1] = z.y; x.v[u + 2] = z.z; x.v[u + 3] = z.w;
      }
    } else {
#pragma unroll
      for (int u = 0; u < NH; ++u) x.v[u] = (sbase + (size_t)j * kBk)[soff + u];
    }
    return x;
  };
  Scores next;                                                 // VALUES: the scores of a block are asked for one block ahead
  const int chunk0 = y * 4 + wave, in_front = tail ? 0 : y % s.nsub * 4 + wave;        // chunks of the partition in front
  const float* cm = s.cmax + (group0 + hg) * s.chunks + (tail ? 0 : chunk0 - in_front);
  if constexpr (PASS == VALUES) {
    if constexpr (SELECT) {
      if (lane < G) own_taken = s.taken[(group0 + lane) * s.items + y];
    }
#pragma unroll
    for (int e = 0; e < kFront; ++e) {
      const int at_ = kg + e * (64 / NH);
      if constexpr (NH <= 4) front[e] = cm[max(min(at_, in_front - 1), 0)];
      else front[e] = at_ < in_front ? cm[at_] : kEmptyMax;
    }
    if (!tail) next = load_scores(min(early + wave * s.cw, Tk - 1));
  }
  const int hq = r & (NH > 4 ? 7 : 3);
  const bool qlane = hq < G;
  const uint16_t* qrow = a.q + (group0 + (qlane ? hq : 0)) * kD;
  uint4 qsrc[4];
  if constexpr (PASS != VALUES) {
#pragma unroll
    for (int t = 0; t < 4; ++t) qsrc[t] = reinterpret_cast<const uint4*>(qrow + 32 * g)[t];
  }
  if constexpr (SELECT && PASS != VALUES) {
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      const uint64_t* row = s.keys + (group0 + min(wave + 4 * u, G - 1)) * Tk;
#pragma unroll
      for (int c = 0; c < NR; ++c) key[u][c] = 64 * c + lane < Tk ? row[64 * c + lane] : 0ULL;
    }
  }
  const int len = __builtin_amdgcn_readfirstlane(a.seqlens ? min(a.Nkv, max(0, a.seqlens[unit / a.Hkv])) : a.Nkv);
  const int full = len / kBk, rest = len % kBk, vis = (len + kBk - 1) / kBk;
  if (tail ? rest == 0 : part * a.split_blocks >= full) return;                  // uniform over the workgroup
  if constexpr (SELECT && PASS != VALUES) {
#pragma unroll
    for (int u = 0; u < kRows; ++u)
#pragma unroll
      for (int c = 0; c < NR; ++c) key[u][c] = 64 * c + lane < vis ? key[u][c] : 0ULL;           // a key is never 0
  }
  v4i qf4 = {0, 0, 0, 0};
  uint32_t qsc = 127u;
  if (PASS != VALUES && qlane) {
    uint32_t pair[16], codes[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      pair[4 * t] = qsrc[t].x; pair[4 * t + 1] = qsrc[t].y; pair[4 * t + 2] = qsrc[t].z; pair[4 * t + 3] = qsrc[t].w;
    }
    qsc = quantize_group32<T>(pair, codes);
    qf4 = (v4i){(int)codes[0], (int)codes[1], (int)codes[2], (int)codes[3]};
  }
  int place = tail ? 0 : y % s.nsub;
  if constexpr (PASS == BOTH) {
    if (tid == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) reinterpret_cast<int*>(scores[v][0])[16] = at;
    }
    lds_barrier();
    place = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(scores[wave][0])[16]);
  }
  const int item = tail ? y : part * s.nsub + place;           // partial slot
  const int p1 = tail ? full + 1 : min((part + 1) * a.split_blocks, full);
  const int base = tail ? full : part * a.split_blocks + place * 4 * s.cw;
  if (base >= p1) return;                                      // uniform over the workgroup
  const int j0 = min(base + wave * s.cw, p1), n_blocks = min(j0 + s.cw, p1) - j0;        // this wavefront's key blocks (may be none)
  const int n_valid = tail ? rest : kBk;
  const uint8_t* k4base = a.k4 + kh * a.Nkv * 64;
  const uint8_t* ksbase = a.ks + kh * a.Nkv * 4;
  const uint8_t* k16base = reinterpret_cast<const uint8_t*>(a.k16 + kh * a.Nkv * kD);
  const uint32_t k4off = (uint32_t)(64 * r + 16 * g), ksoff = (uint32_t)(4 * r + g);   // key 16t + r, channels 32g .. 32g + 31
  const int all = (1 << G) - 1;
  const float c = a.scale * 1.4426950408889634f;

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
  Keys kt;                                                     // of the next block, unless every head takes it in 16 bits
  // which heads have promoted which of the wavefront's blocks: lane u < G holds head u's bits
  uint32_t bits = 0u;
  auto load_next = [&](int i) {
    if (i < n_blocks && promoted_mask(bits, i) != all) kt = load4(j0 + i);
  };
  if constexpr (SELECT && PASS == VALUES) {
    bits = own_taken >> (wave * s.cw);
  } else if constexpr (SELECT) {
    const int k = decode_row_budget(vis, s.fixed_k, s.ppm), n = min(4 * s.cw, p1 - base);
    if (n_blocks > 0 && k < vis) kt = load4(j0);
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      if (wave + 4 * u < G) {
        uint64_t own;
        if constexpr (PASS == SCORES) {
          own = u == 0 ? own_key[0] : own_key[kRows - 1];
          if (tail) own = s.keys[(group0 + wave + 4 * u) * Tk + min(base + lane, Tk - 1)];
        } else {
          static_assert(PASS != BOTH || NR <= 2, "one of two registers");
          own = __shfl(key[u][0], (base + lane) & 63);
          if constexpr (NR == 2) {
            const uint64_t x = __shfl(key[u][1], (base + lane) & 63);
            own = base + lane < 64 ? own : x;
          }
        }
        const uint32_t taken = k >= vis ? ~0u : rank_select(key[u], own, k, base, n, lane);
        if (lane < 4) reinterpret_cast<uint32_t*>(scores[lane][0])[wave + 4 * u] = taken;
        if (PASS == SCORES && lane == 0) s.taken[(group0 + wave + 4 * u) * s.items + item] = taken;
      }
    lds_barrier();
    if (lane < G) bits = reinterpret_cast<const uint32_t*>(scores[wave][0])[lane] >> (wave * s.cw);
  } else {
    if (n_blocks > 0) bits = promoted_bits(a, group0, G, j0, lane);
    if constexpr (PASS != VALUES) load_next(0);
  }

  unsigned char* slots = tiles[wave];
  const uint32_t lds0 = lds_address(slots);
  // 16-bit K rows by DMA, whole lines per instruction (only such reads may carry the streaming hint): row 4 q + g, its chunk c
  // at position c ^ (row & 7).  Rows past the cached tokens reach only their own keys' scores, which are masked.
  auto issue_k16 = [&](int j, int q0, int n) __attribute__((always_inline)) {
    const uint8_t* tile = k16base + (size_t)__builtin_amdgcn_readfirstlane(j) * kTile16 + 1024 * q0;
#pragma unroll
    for (int q = 0; q < n; ++q) dma_b128<true>(tile + 1024 * q, (uint32_t)(256 * g + 16 * (r ^ (4 * (q & 1) + g))), lds0 + 1024 * q);
  };
  RowState st = {kEmptyMax, 0.f};
  auto tops = [&](int v) { return reinterpret_cast<float*>(tiles[v] + kTops); };
  if constexpr (PASS != VALUES) {   // ---- scores of the wavefront's blocks and the largest of them ----

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
  float top[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) top[i] = kEmptyMax;
  auto keep = [&](int i, int head, int key, float z) __attribute__((always_inline)) {
    if constexpr (PASS == BOTH) scores[wave][i][head * 64 + key] = z;
    else __builtin_nontemporal_store(z, s.scores + (group0 + head) * a.Nkv + (size_t)(j0 + i) * kBk + key);
  };
  // 4-bit scores of a block for all heads, 16-bit scores for those that have promoted it (which then replace the former)
  auto scores4 = [&](const Keys& x, int i, int M) __attribute__((always_inline)) {
    v4f acc[4];
    float v4[NS][NV];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(widen(qf4), widen(x.k[t]), (v4f){0.f, 0.f, 0.f, 0.f}, 4, 4, 0, qsc, 0, x.ks[t]);
    mine(acc, v4);
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
      for (int u = 0; u < NV; ++u)
        if (h0 + u < G) {
          const float z = key0 + 32 * q < n_valid ? v4[q][u] : -INFINITY;
          if (PASS == BOTH || ((M >> (h0 + u)) & 1) == 0) keep(i, h0 + u, key0 + 32 * q, z);
          top[u] = fmaxf(top[u], ((M >> (h0 + u)) & 1) ? kEmptyMax : z);
        }
  };
  auto keep16 = [&](const v4f (&acc)[4], int i, int M) __attribute__((always_inline)) {
    float v16[NS][NV];
    mine(acc, v16);
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
      for (int u = 0; u < NV; ++u)
        if (h0 + u < G && ((M >> (h0 + u)) & 1)) {
          const float z = key0 + 32 * q < n_valid ? v16[q][u] : -INFINITY;
          keep(i, h0 + u, key0 + 32 * q, z);
          top[u] = fmaxf(top[u], z);
        }
  };
  auto scores16 = [&](const v8s (&qf)[4], int t0, int n, v4f (&acc)[4]) __attribute__((always_inline)) {        // sub-tiles of 16 keys, from the tile's start
#pragma unroll
    for (int t = 0; t < n; ++t) {
      acc[t0 + t] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
        acc[t0 + t] = mfma16<T>(qf[s4], *reinterpret_cast<const v8s*>(slots + 4096 * t + 256 * r + 16 * ((4 * s4 + g) ^ (r & 7))), acc[t0 + t]);
    }
  };
  auto query16 = [&](v8s (&qf)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4)
      qf[s4] = qlane ? *reinterpret_cast<const v8s*>(qrow + 32 * s4 + 8 * g) : (v8s){0, 0, 0, 0, 0, 0, 0, 0};
  };

    for (int i = 0; i < n_blocks; ++i) {
      const int M = promoted_mask(bits, i);
      // The first half of a 16-bit K tile by LDS DMA, the second at the same time into registers, from where it takes the first one's
      // place, or behind it (see load16)
      v4i second[8];
      if (WK && M != 0) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the reads of the tile before are over
        issue_k16(j0 + i, 0, 8);
        const uint8_t* half1 = k16base + (size_t)(j0 + i) * kTile16 + kTile16 / 2 + 16 * lane;
#pragma unroll
        for (int q = 0; q < 8; ++q) second[q] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(half1 + 1024 * q));
      }
      if (M != all) scores4(kt, i, M);
      if (!WK || M == 0) load_next(i + 1);
      if (M != 0) {
        v4f acc[4];
        v8s qf[4];
        query16(qf);
        if constexpr (WK) {
          vm_wait<0>();
          load_next(i + 1);
          scores16(qf, 0, 2, acc);
#pragma unroll
          for (int q = 0; q < 8; ++q) *reinterpret_cast<v4i*>(slots + 1024 * q + 256 * g + 16 * (r ^ (4 * (q & 1) + g))) = second[q];
          scores16(qf, 2, 2, acc);
        } else {
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the reads of the half before are over
            issue_k16(j0 + i, 8 * hf, 8);
            vm_wait<0>();
            scores16(qf, 2 * hf, 2, acc);
          }
        }
        keep16(acc, i, M);
      }
    }

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
    if (r == 0 && g < (NH > 4 ? 2 : 1)) {
      if (PASS == BOTH && h0 + i < NH) tops(wave)[h0 + i] = m;
      if (PASS == SCORES && h0 + i < G && n_blocks > 0 && !tail) s.cmax[(group0 + h0 + i) * s.chunks + item * 4 + wave] = m;
    }
  }
  }
  if constexpr (PASS == SCORES) return;

  const uint8_t* v4base = a.v4 + kh * (size_t)(a.Nkv / 64) * 4096;
  const uint8_t* vsbase = a.vs + kh * (size_t)(a.Nkv / 32) * kD;
  const uint8_t* v16base = reinterpret_cast<const uint8_t*>(a.v16 + kh * a.Nkv * kD);
  const uint32_t v16off = (uint32_t)(2048 * g + 16 * r);
  // The 4-bit tile of a block travels one block ahead of the arithmetic by LDS DMA, whole lines per instruction.  Its 256
  // bytes of channels 8 R .. 8 R + 7 hold chunk c (channel 8 R + c / 2, token group c & 1) at position c ^ R, so that the
  // 16 rows of a fragment lie in different banks.
  const uint32_t dma_off = (uint32_t)(256 * g + 16 * (r ^ g));              // R = 4 m + g in instruction m
  auto issue4 = [&](int j, int slot) {
    const int j_ = __builtin_amdgcn_readfirstlane(j);
    const uint32_t to = lds0 + (uint32_t)(__builtin_amdgcn_readfirstlane(slot) * kSlot);
    uint32_t off = dma_off;
    asm volatile("" : "+v"(off));                              // one offset kept, not four
#pragma unroll
    for (int m = 0; m < 4; ++m) dma_b128<true>(v4base + (size_t)j_ * 4096 + 1024 * m, off ^ (64u * m), to + 1024 * m);
    dma_b32<true>(vsbase + (size_t)j_ * 256, (uint32_t)(4 * lane), to + 4096);
  };
  // Half q of the 16-bit rows of a block, keys 32 q + 8 g .. + 7, channels 8 r ..
  // One launch asks for both halves of V at once.  At once / by halves, back to back: 24.7 / 25.7 us for 4 x 5632 tokens, 32/8 heads, 5 %, 143.5 / 146 for
  // a step of 8 x 16384-32768, 64/8, 10 %, 45.4 / 46.3 for 6 x 4096-8192, 16/16, 25 %; 97.5 / 100.3 for 4 x 16384-32768, 64/8, 100 %, but 70.5 / 68.1 for
  // 4 x 10656-21312, 32/8, 100 %.
  // Of K at once / by halves: where a wavefront has few blocks the wait for a tile is what it does, in short rows with more than two heads and
  // at most four blocks 24.2 / 24.9 us for 2 x 4096, 32/8, 25 %, 36.5 / 37.5 for 5 x 3296-6592, 64/8, 5 %; with eight blocks, or in long rows, the other
  // wavefronts use that time, 45.3 / 43.1 for 16 x 4096-8192, 32/8, 64.8 / 63.1 for 1 x 131072, 146.1 / 143.5 for the 8 x 16384-32768, 41.7 / 40.8 for
  // 5 x 11648-23296, 64/8, 0 %.  One or two heads leave little but the tile on its way in long rows, 109.3 / 116.2 for 11 x 12288, 16/8, 100 %, 106 / 109 for
  // 3 x 13088-26176, 16/16 (an instance of its own: without promoted blocks the code alone costs 47.3 / 45.6, 14 x 12800), and in short ones 61.5 / 58.9 for 6 x 3584-7168,
  // 16/16, 100 %, 34.8 / 33.9 for 7 x 3104-6208, 5 % (but 113 / 117 for 10 x 8192, 100 %).
  // In two launches the registers would leave a CU three workgroups instead of four (44.4 -> 47.7 us for 2 x 28672), and where three
  // are enough it gains nothing (1 x 32768).
  v4i v[kWholeV ? 16 : 8];
  auto load16 = [&](int j, int q0) __attribute__((always_inline)) {
    const uint8_t* tile = v16base + (size_t)j * kTile16 + 8192 * q0;
#pragma unroll
    for (int u = 0; u < 8; ++u) v[(kWholeV ? 8 * q0 : 0) + u] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(tile + v16off + 256 * u));
  };
  int Mnext = n_blocks > 0 ? promoted_mask(bits, 0) : all;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // the last reads of K are over
  if (Mnext != all) issue4(j0, 0);
  // ---- the running maximum in front of the wavefront's blocks ----
  float m = kEmptyMax;
  bool unanswered = false;                                     // BOTH: a wait has ended without a maximum
  if constexpr (PASS == VALUES) {
    if (tail && n_blocks > 0) next = load_scores(j0);
    if (n_blocks > 0) {                                        // (chunks without blocks have left no maximum)
#pragma unroll
      for (int e = 0; e < kFront; ++e) m = fmaxf(m, in_front > 0 ? front[e] : kEmptyMax);
      for (int e = kg + kFront * (64 / NH); e < in_front; e += 64 / NH) m = fmaxf(m, cm[e]);
    }
  } else {
    lds_barrier();
    unsigned* published = s.tops + (group0 + hg) * s.items + item;
    if (wave == 0 && lane < G && !tail) {
      const uint32_t t = __float_as_uint(fmaxf(fmaxf(tops(0)[lane], tops(1)[lane]), fmaxf(tops(2)[lane], tops(3)[lane])));
      __hip_atomic_store(published, t == kUnset ? 0x7fc00000u : t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    bool lost = false;
    for (int e = kg; e < place; e += 64 / NH) {
      uint32_t x = kUnset;
      for (int tries = 0; x == kUnset && tries < s.polls; ++tries) {
        if (tries > 0) __builtin_amdgcn_s_sleep(1);
        x = __hip_atomic_load(published - place + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (x == kUnset) lost = true;
      else m = fmaxf(m, __uint_as_float(x));
    }
    unanswered = __builtin_amdgcn_ballot_w64(lost) != 0ULL;
    for (int u = 0; u < wave; ++u) m = fmaxf(m, tops(u)[hg]);
  }
  m = head_max32<NH>(m);
  st.m = fmaxf(m, other_half(m));

  // ---- softmax, codes of P and P.V of the wavefront's blocks ----
  // Softmax layout: lane = NH kg + h holds the NH keys NH kg .. of head h, so that every step of the recurrence that is not
  // an exponential costs the heads of a group one instruction together, and each 32 lanes hold one MXFP4 group of P per head.
  // The accumulators hold channel 8 (4 g + i) + e of head r in o[e][i]: row r of tile e is channel 8 r + e, because a lane's
  // 16 bytes of a 16-bit V row are 8 neighbouring channels, which are transposed against 8 rows inside the lane.
  v4f o[8];
  // The sums of a wavefront that knows no maximum to start from are NaN, not its row sums: a row sum that is not positive divides
  // nothing in the merge.
  float none = 0.f;
  if constexpr (PASS == BOTH) {
    none = unanswered ? __builtin_nanf("") : 0.f;
    asm volatile("" : "+v"(none));                             // arithmetic is compiled as if there were no NaN
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (v4f){none, none, none, none};
  if (n_blocks > 0) {
    for (int i = 0; i < n_blocks; ++i) {
      const int j = j0 + i;
      const int M = Mnext;
      vm_wait<0>();                                            // the tiles of this block, asked for a block ago or earlier
      float x[NH];
      if constexpr (PASS == VALUES) {
#pragma unroll
        for (int u = 0; u < NH; ++u) {
          x[u] = next.v[u];
          asm volatile("" : "+v"(x[u]));                       // no second wait for them behind the loads issued next
        }
        if (i + 1 < n_blocks) next = load_scores(j + 1);
      } else {
        const float* own = scores[wave][i] + hg * 64 + NH * kg;
        if constexpr (NH >= 4) {
#pragma unroll
          for (int u = 0; u < NH; u += 4) {
            const float4 z = *reinterpret_cast<const float4*>(own + u);
            x[u] = z.x; x[u + 1] = z.y; x[u + 2] = z.z; x[u + 3] = z.w;
          }
        } else {
#pragma unroll
          for (int u = 0; u < NH; ++u) x[u] = own[u];
        }
      }
      uint16_t* prow_w = reinterpret_cast<uint16_t*>(scores[wave][PASS == BOTH ? i : 0]);
      uint8_t* pcode_w = reinterpret_cast<uint8_t*>(prow_w + NH * 64);
      uint8_t* pscale_w = pcode_w + NH * 32;
      if (M != 0) {                                            // needed after the softmax
        load16(j, 0);
        if (kWholeV) load16(j, 1);
      }
      Mnext = i + 1 < n_blocks ? promoted_mask(bits, i + 1) : all;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the scores are here, the reads of the other slot's block are over
      if (Mnext != all) issue4(j + 1, (i + 1) & 1);
      // ---- online softmax (Alg. 1 steps 10-12 / 16-17) of all heads ----
      float gmax = x[0];
#pragma unroll
      for (int u = 1; u < NH; ++u) gmax = fmaxf(gmax, x[u]);
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
        p[u] = fast_exp2(__builtin_fmaf(x[u], c, -mc));
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
        const unsigned char* slot = slots + (i & 1) * kSlot;
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
          if (!kWholeV && q == 1) {
            __builtin_amdgcn_sched_barrier(0);                 // into the registers of the first half
            load16(j, 1);
          }
          v4i* vq = v + (kWholeV ? 8 * q : 0);
          if (n_valid != kBk) {                                // rows past the cached tokens hold whatever lies there, and zero times that need not be zero
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (32 * q + 8 * g + u >= n_valid) vq[u] = (v4i){0, 0, 0, 0};
          }
          const v8s pf = mine ? *reinterpret_cast<const v8s*>(prow_w + r_ * 64 + 32 * q + 8 * g_) : (v8s){0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            v4i col;
#pragma unroll
            for (int u = 0; u < 4; ++u) col[u] = (int)__builtin_amdgcn_perm((uint32_t)vq[2 * u + 1][e >> 1], (uint32_t)vq[2 * u][e >> 1], sel);
            // zero times an infinity or NaN of V is not zero: the heads that take the block in 4 bits keep their sums
            const v4f sum = mfma16<T>(__builtin_bit_cast(v8s, col), pf, o[e]);
            o[e] = mine ? sum : o[e];
            asm volatile("" : "+v"(o[e]));                     // chosen here: both values of all eight tiles do not fit
            if (e & 1) __builtin_amdgcn_sched_barrier(0);      // the transposed pieces are formed as they are used, not all ahead
          }
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (r < G) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float* to = reinterpret_cast<float*>(slots) + r * kD + 8 * (4 * g + i);
        *reinterpret_cast<float4*>(to) = make_float4(o[0][i], o[1][i], o[2][i], o[3][i]);
        *reinterpret_cast<float4*>(to + 4) = make_float4(o[4][i], o[5][i], o[6][i], o[7][i]);
      }
    }
  }
  auto ml = [&](int v, int u) { return reinterpret_cast<float*>(tiles[v] + kMl) + 2 * u; };
  {
    float* own_ml = ml(wave, 0);
    const float l = head_sum<NH>(st.l);
    if (lane < NH) { own_ml[2 * lane] = st.m; own_ml[2 * lane + 1] = l; }
  }
  __syncthreads();
  // the workgroup's partial.  A wavefront without blocks has left its sums unwritten; it is skipped by its row sum of zero
  // (with a key it is positive, or the whole chunk weighs nothing, or it is NaN and has to reach the result: bits are
  // compared, because comparisons of numbers are compiled as if there were no NaN).
  for (int e = tid; e < G * (kD / 2); e += 256) {                 // two channels each: one round for up to four heads (34.9 -> 34.4 us, 1 x 32768)
    const int u = e >> 6, ch = 2 * (e & 63);
    float m = ml(0, u)[0];
#pragma unroll
    for (int v = 1; v < 4; ++v) m = fmaxf(m, ml(v, u)[0]);
    float l = 0.f;
    float2 sum = make_float2(0.f, 0.f);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float lv = ml(v, u)[1];
      if (__float_as_uint(lv) != 0u) {
        const float f = fast_exp2((ml(v, u)[0] - m) * c);
        const float2 x = *reinterpret_cast<const float2*>(tiles[v] + 4 * (u * kD + ch));
        l += f * lv;
        sum.x += f * x.x;
        sum.y += f * x.y;
      }
    }
    const size_t slot = (group0 + u) * a.nparts + item;
    *reinterpret_cast<float2*>(a.part_o + slot * kD + ch) = sum;
    if (ch == 0) { a.part_ml[2 * slot] = m; a.part_ml[2 * slot + 1] = l; }
  }
}

// The tickets and maxima of a call without selection (otherwise decode_scores_kernel clears them).
__global__ void __launch_bounds__(256) decode_split_clear_kernel(unsigned* tickets, int n_tickets, unsigned* tops, long n_tops) {
  const long at = (long)blockIdx.x * 256 + threadIdx.x;
  if (at < n_tickets) tickets[at] = 0u;
  if (at < n_tops) tops[at] = kUnset;
}

// Log-sum-exp merge of the partials of one (sequence, query head): 32 channel quads x 8 slots at a time.  The call is one
// chain of waits, so the first kAhead slots of every row of threads, and the last, are asked for before the length is known;
// slots without work were never written, and the length says which: what they hold is not used.
// With the length, the maxima and the sums asked for one after the other a call of 131072 tokens took 68.6 us instead of 66.8, a step
// of 32768 38.5 instead of 37.2, one of 4096 23.7 instead of 23.3 (four slots ahead: 67.2, 38.3, 23.4).
__global__ void __launch_bounds__(256) decode_split_merge_kernel(DecodeSplitArgs s) {
  const DecodeArgs& a = s.a;
  constexpr int kAhead = 8;
  __shared__ float4 red[8][32];
  __shared__ float redl[8];
  const int tid = threadIdx.x, lane = tid & 63, quad = tid & 31, row = tid >> 5;
  const size_t qh = blockIdx.x;
  const int b = (int)(qh / a.Hq), last = a.nparts - 1;
  const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + qh * a.nparts;
  const float* po = a.part_o + qh * a.nparts * kD + 4 * quad;
  float top = lane < a.nparts ? ml[lane].x : 0.f;
  const float2 ml_last = ml[last];
  const float4 po_last = *reinterpret_cast<const float4*>(po + (size_t)last * kD);
  float2 xa[kAhead];
  float4 ya[kAhead];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    const int p = min(row + 8 * u, last);
    xa[u] = ml[p];
    ya[u] = *reinterpret_cast<const float4*>(po + (size_t)p * kD);
  }
  const int len = a.seqlens ? min(a.Nkv, max(0, a.seqlens[b])) : a.Nkv;
  const int full = len / kBk;
  const int parts = full / a.split_blocks, left = full % a.split_blocks;
  const int used = parts * s.nsub + (left + 4 * s.cw - 1) / (4 * s.cw);     // slots of full blocks: 0 .. used-1
  const bool tail = len % kBk != 0;                                          // and the last one
  const float c = a.scale * 1.4426950408889634f;
  const int n = used + (tail ? 1 : 0);
  float m = -INFINITY;
  if (lane < n) m = lane < used ? top : ml_last.x;
  for (int p = lane + 64; p < n; p += 64) m = fmaxf(m, p < used ? ml[p].x : ml_last.x);
  m = wave_max(m);
  float l = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](float2 x, float4 y) {
    const float f = fast_exp2((x.x - m) * c);
    l += f * x.y;
    acc.x += f * y.x; acc.y += f * y.y; acc.z += f * y.z; acc.w += f * y.w;
  };
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    const int p = row + 8 * u;
    if (p < used) add(xa[u], ya[u]);
  }
#pragma unroll 4
  for (int p = row + 8 * kAhead; p < used; p += 8) add(ml[p], *reinterpret_cast<const float4*>(po + (size_t)p * kD));
  if (tail && row == used % 8) add(ml_last, po_last);
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
// Partitions, walk / one launch: 384: 319 / 275 us (6 x 131072 tokens, 32/8 heads, 5 %), 304 / 230 (16 x 40960); 512: 355 / 366 (8 x
// 131072), 678 / 685 (the same at 25 %), 574 / 528 (16 x 51200, 64/8, 10 %); 1024: 692 / 697 (16 x 131072).  With one query head per
// KV head three of a walk's four wavefronts have no head: 512: 245 / 194 us (a serving step, 16 x 32768, 16/16), 248 / 237 (8 x 65536).
bool decode_split_wanted(int B, int Hq, int Hkv, int nsplit, int split_blocks) {
  if (Hq / Hkv > 8) return false;
  if (nsplit > 1 && split_blocks <= 16) return false;
  return (long)B * Hkv * nsplit <= (Hq == Hkv ? kSplitMaxItemsOneHead : kSplitMaxItems);
}

constexpr int kSelectBoth = 128;

// One launch for both passes, or two.  One launch reads and writes no scores and saves the gap between two; but the places of a
// partition wait for each other, and with few of them in long partitions that wait is what the call takes.  Up to kSelectBoth key
// blocks a sequence nobody waits for long.  Between 129 and kSplitSelectBlocks one launch also needs a launch for the selection that
// two do not.  Two / one in us, B x key blocks of a sequence, heads, budget (blocks of all KV heads):
//   short         1 x    8, 32/8, 5 %   25.7 /  23.0    10 x   48, 64/8, 5 %     41.6 /  32.5    16 x   48, 32/8, 5 %   41.0 / 37.8
//   up to 8192    1 x  512, 32/8        38.0 /  51.7     3 x  320, 32/8, 100 %   63.0 /  67.5     1 x 1024, 32/8, 5 %   51.6 / 56.3
//    8256         1 x 1032, 32/8, 5 %   54.6 /  53.2     1 x 1032, 64/8, 5 %     71.0 /  74.0
//    8448         4 x  264, 32/8, 5 %   48.6 /  53.1     the same at 25 %        68.2 /  76.6     4 x  264, 64/8, 5 %   64.5 / 64.5
//    9216         2 x  576, 32/8, 5 %   51.6 /  52.0     2 x  576, 16/8, 5 %     44.3 /  45.8     2 x  576, 64/8, 5 %   65.5 / 72.0
//   10240         1 x 1280, 32/8, 5 %   58.3 /  57.7     5 x  256, 16/8, 5 %     45.2 /  42.4     1 x 1280, 64/8, 5 %   76.0 / 81.0
//   12288         3 x  512, 32/8, 25 %  91.5 /  82.8     3 x  512, 16/8, 25 %    71.2 /  65.6     3 x  512, 64/8, 25 %   114 /  108
//   14336         7 x  256, 32/8, 25 %  94.9 /  87.9     7 x  256, 16/8, 25 %    73.1 /  68.6     7 x  256, 64/8, 25 %   117 /  109
//   more          4 x  512, 32/8        73.5 /  67.4     1 x 2048, 32/8, 5 %     80.4 /  75.5     4 x  512, 64/8, 100 %  147 /  105
// Without promoted blocks nothing in front of one launch clears its tickets and maxima: it needs a launch of its own for that, and
// gains less the fewer heads read and write scores.  So there two launches go further.  Two / one, no promoted block, serving steps
// (+ append) and calls over full caches:
//    1024         1 x  128, 32/8         16.7 /  19.1    1 x  128, 64/8, call    14.5 /  17.1     1 x   64, 16/16, call  10.1 / 12.6
//    1344         2 x   84, 32/8         17.1 /  21.5    the same, call          13.5 /  18.6     2 x   84, 64/8         19.7 / 23.9
//    2048         2 x  128, 32/8         18.0 /  19.0    4 x   64, 64/8          20.4 /  18.9     8 x   32, 64/8         21.0 / 20.0
//    4096         4 x  128, 32/8         20.7 /  19.8    4 x  128, 64/8          24.6 /  21.8     2 x  128, 16/8, call   13.8 / 14.8
//    8192         8 x  128, 32/8         26.8 /  25.9    8 x  128, 16/8, call    20.8 /  22.6     4 x  128, 16/16, call  19.1 / 22.3
//   10240         1 x 1280, 16/8         29.6 /  32.7    1 x 1280, 64/8          39.8 /  46.6
//   12288         3 x  512, 32/8         35.0 /  32.5    3 x  512, 64/8          41.2 /  46.1     3 x  512, 16/8         32.2 / 30.6
//   14336         7 x  256, 32/8         35.5 /  32.1    7 x  256, 64/8          42.9 /  44.8     7 x  256, 16/8         32.2 / 30.8
//   16384         2 x 1024, 32/8         41.5 /  42.0    2 x 1024, 64/8          47.1 /  49.2     8 x  128, 16/16        32.4 / 32.4
//   32768         8 x  512, 64/8         76.7 /  70.7    2 x 1024, 16/16         54.7 /  55.7     16 x 128, 16/16        51.9 / 54.2
//   40960         5 x  512, 16/16        60.5 /  58.9
// Up to 12800 blocks the scores of eight heads fit the 32 MiB of thrift_attn_decode_static with the rest.
bool decode_split_both(int B, int Hq, int Hkv, int Tk, bool promoted) {
  const long blocks = (long)B * Hkv * Tk;
  const int heads = Hq / Hkv;
  if (promoted) return Tk <= kSelectBoth || blocks > (heads > 4 ? 10240 : 9216);
  if (heads <= 2) return blocks > (heads == 1 ? 32768 : 10240);
  if (Tk <= kSelectBoth) return blocks > 1536;
  return blocks > (heads > 4 ? 12800 : 9216);
}

// Where the kernels select for themselves instead of a launch of its own: rows of key blocks that a wavefront holds, and with one
// launch (whose workgroups ask for more blocks each, among others that wait) only as many as two registers hold: 156 us with a
// launch, 175 without for 8 x 32768 tokens, 64/8 heads; 47.9 us without for 16 x 8192.
bool decode_split_selects(int Tk, bool both) { return Tk <= (both ? kSelectBoth : kSplitSelectBlocks); }

// Key blocks per wavefront.  Longer chunks are longer serial chains, shorter ones more partials and more running maxima to look
// up.  Chunks of 1 / 2 / 4 / 8, whole serving steps or calls in us (blocks of all KV heads; B x tokens, heads, budget):
//   one launch
//     512 blocks   1 x 4096, 32/8, 5 %      25.6 /  28.7 /  32.9 /  42.4   takes 1
//    1344          2 x 5376, 32/8, 100 %    30.0 /  26.6                        2 (more than 20 places in a partition)
//    1280          4 x 2560, 32/8, 5 %      23.7 /  23.9                        1
//                  16 x 640, 64/8, 100 %    27.4 /  30.6                        1
//    2048          8 x 2048, 32/8, 5 %      27.9 /  29.5                        2
//    2048          4 x 4096, 32/8, 5 %             28.7 /  30.1                 2
//    6144          6 x 8192, 16/8, 5 %                    38.5                  4
//   16384          1 x 131072, 32/8, 5 %   115.5 /  88.6 /  78.0 /  76.4         8
//                  16 x 8192, shared, 5 %   80.5 /  60.1 /  54.0 /  47.5         8
//                  4 x 32768, 64/8, 100 %  145.2 / 119.0 / 105.9               4 (eight heads: no more fit the LDS)
// Three or four heads per KV head: the scores of eight blocks leave a CU room for two workgroups, those of four for three.  So
// eight are taken where the grid is one round of two (up to 16384 blocks), unless three of half the length and short rows end
// sooner, and in rows of more than 1024 blocks, where shorter chunks have too many maxima to look up.  Four / eight:
//    9216          9 x 8192, 32/8, 5 %      40.7 /  47.1                        4
//   12288          3 x 32768, 32/8, 5 %     60.5 /  56.1                        8
//   14336          14 x 8192, 32/8, 5 %     54.4 /  55.2                        4
//   20480          10 x 16384, 32/8, 5 %    75.5 /  81.8                        4
//   65536          16 x 32768, 32/8, 25 %  272.3 / 278.1                        4
//                  4 x 131072, 32/8, 25 %  342.0 / 334.7                        8
// One or two heads fit three workgroups per CU with eight blocks too, so that only the number of wavefronts decides.  Four / eight:
//    8192          4 x 8192, 16/16, 25 %    38.0 /  42.6                        4
//    8960          10 x 7168, 16/8, 25 %    46.0 /  52.3                        4
//   10000          2 x 40000, 16/8, 5 %     49.1 /  44.4                        8
//   32768          4 x 32768, 16/16, 25 %   89.0 /  94.7                        4 (one head)
//   20480          5 x 32768, 16/8, 5 %     63.0 /  60.5                        8
//   two launches
//    1280 blocks   1 x 10240, 32/8, 5 %     29.2 /  31.6 /  36.8              takes 1
//    2560          1 x 20480, 32/8, 5 %     36.3 /  34.7 /  39.0                  2
//    7168          2 x 28672, 32/8, 25 %    66.1 /  62.7 /  70.9                  2
//    8192          1 x 65536, 32/8, 5 %     62.2 /  52.7 /  51.6                  4
//                  4 x 16384, 64/8, 5 %     87.6 /  71.0 /  63.4                  4
//    8384          2 x 16768, 16/16, 5 %            40.4 /  36.6                  4
//                  4 x 16768, 16/8, 25 %            54.0 /  53.6                  4
//    3072          2 x 12288, 64/8, 5 %     43.0 /  46.1 /  50.1                  1 (more than four heads: up to 4096)
//   16384          8 x 8192, 16/16, 0 %                     33.5 / 32.4            8 (short rows: they get here without promoted blocks only)
int decode_split_chunk(int B, int Hq, int Hkv, int Tk, bool promoted) {
  const long blocks = (long)B * Hkv * Tk;
  const int heads = Hq / Hkv;
  if (!decode_split_both(B, Hq, Hkv, Tk, promoted))
    return blocks < (heads > 4 ? 4096 : 2048) ? 1 : blocks < 8192 ? 2 : Tk <= kSelectBoth && blocks >= 16384 ? 8 : 4;
  int cw = 1;
  while (cw < chunk_limit(heads, true) && blocks > 1536L * cw) cw *= 2;
  if (cw == 1 && blocks >= 1024 && Tk > 80) cw = 2;
  if (cw == 8 && heads > 2 && Tk <= 1024 && (blocks > 16384 || (Tk <= 256 && blocks <= 14336))) cw = 4;
  if (cw == 8 && heads <= 2 && (blocks <= 9216 || (heads == 1 && blocks > 24576))) cw = 4;
  return cw;
}

void launch_decode_split(const DecodeSplitArgs& s, hipStream_t st) {
  const DecodeArgs& a = s.a;
  const dim3 grid((unsigned)((long)a.B * a.Hkv * s.items)), block(256);
  const int G = a.Hq / a.Hkv;
  if (s.clear && s.both) {
    const long n_tops = (long)a.B * a.Hq * s.items;
    decode_split_clear_kernel<<<dim3((unsigned)((n_tops + 255) / 256)), block, 0, st>>>(s.tickets, a.B * a.Hkv * a.nsplit, s.tops, n_tops);
  }
#define THRIFT_BOTH(T, NH, NC)                                                                            \
  do {                                                                                                    \
    if (s.keys != nullptr) decode_split_kernel<T, NH, BOTH, kSelectBoth / 64, NC, (NH > 2 && NC == 4)><<<grid, block, 0, st>>>(s);        \
    else if (a.bitmap != nullptr) decode_split_kernel<T, NH, BOTH, 0, NC, (NH <= 2)><<<grid, block, 0, st>>>(s);                          \
    else decode_split_kernel<T, NH, BOTH, 0, NC, false><<<grid, block, 0, st>>>(s);                       \
  } while (0)
#define THRIFT_SPLIT(T, NH)                                                                               \
  do {                                                                                                    \
    if (s.both && s.cw <= 4) THRIFT_BOTH(T, NH, (NH == 4 ? 4 : chunk_limit(NH, true)));                   \
    else if (s.both) THRIFT_BOTH(T, NH, (chunk_limit(NH, true)));                                         \
    else if (s.keys != nullptr) {                                                                         \
      decode_split_kernel<T, NH, SCORES, kSplitSelectBlocks / 64><<<grid, block, 0, st>>>(s);             \
      decode_split_kernel<T, NH, VALUES, kSplitSelectBlocks / 64><<<grid, block, 0, st>>>(s);             \
    } else {                                                                                              \
      decode_split_kernel<T, NH, SCORES, 0><<<grid, block, 0, st>>>(s);                                   \
      decode_split_kernel<T, NH, VALUES, 0><<<grid, block, 0, st>>>(s);                                   \
    }                                                                                                     \
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
#undef THRIFT_BOTH
  decode_split_merge_kernel<<<dim3((unsigned)((long)a.B * a.Hq)), block, 0, st>>>(s);
}

}  // namespace thrift
