// Decode for caches that give the one-workgroup-per-partition walk too few workgroups (short caches, few sequences).
//
// The rounding of P follows the running maximum of the partition, so a partition cannot simply be cut into shorter
// recurrences.  It can be computed in two passes that need no order between workgroups:
//   decode_split_scores_kernel  the raw scores of every (query head, key) and the largest score of every chunk;
//   decode_split_values_kernel  softmax, P quantiser and P.V of a chunk, started from the largest score of the chunks in
//                               front of it in the partition: the running maximum of every block, hence every code of P, is
//                               the one of the serial walk.
// A chunk is `cw` key blocks and belongs to ONE wavefront, which takes all heads of the KV group at once (head u in rows u
// and u + 4 of the score tiles, column u of the P.V tiles: up to 8 heads cost the matrix instructions of one), operands
// straight from global memory: no barrier and no LDS on the 4-bit path.  Four chunks that follow each other make a workgroup,
// whose partials are added up in LDS before they are written.
// Measured against the walk (attention kernels alone): 14 + 15 us against 250 us for one sequence of 32768 tokens and 32/8
// heads, 39 + 28 us against 259 us at 131072 tokens, 147 + 94 us against 472 us for eight sequences of 16384-32768 tokens
// and 64/8 heads at a 10 % budget.
// What bounds it: for short caches the latency of the chain of launches; for long ones HBM (the scores travel through
// memory once more, 8 bytes per head and token next to 136 bytes of codes and scales per token).
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

// Which heads of the group have promoted which of the (at most 64) blocks j0 .. : lane u < G holds head u's bits, bit 0 =
// block j0.
__device__ __forceinline__ unsigned long long promoted_bits(const DecodeArgs& a, size_t group0, int G, int j0, int lane) {
  if (a.bitmap == nullptr || lane >= G) return 0ULL;
  const unsigned long long* bm = a.bitmap + (group0 + lane) * a.bitmap_words;
  const int w = j0 >> 6, sh = j0 & 63;
  unsigned long long bits = bm[w] >> sh;
  if (sh != 0 && w + 1 < a.bitmap_words) bits |= bm[w + 1] << (64 - sh);
  return bits;
}
// mask over the heads for block j0 + i
__device__ __forceinline__ int promoted_mask(unsigned long long bits, int i) {
  return (int)__builtin_amdgcn_ballot_w64(((bits >> i) & 1ULL) != 0ULL);
}

}  // namespace

// NH: heads per KV group, rounded up to 1, 2, 4 or 8
template <typename T, int NH>
__global__ void __launch_bounds__(256) decode_split_scores_kernel(DecodeSplitArgs s) {
  const DecodeArgs& a = s.a;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, r = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitWork w = split_work(s, wave);
  if (w.j0 >= w.j1) return;
  const int G = a.Hq / a.Hkv;
  const size_t group0 = (size_t)w.b * a.Hq + (size_t)w.kvh * G, kh = (size_t)w.b * a.Hkv + w.kvh;
  const uint8_t* k4base = a.k4 + kh * a.Nkv * 64;
  const uint8_t* ksbase = a.ks + kh * a.Nkv * 4;
  const uint16_t* k16base = a.k16 + kh * a.Nkv * kD;

  const unsigned long long bits = promoted_bits(a, group0, G, w.j0, lane);
  const int all = (1 << G) - 1;

  // fragment (t, kk): key 32t + r, d-group 2*half + kk
  auto load4 = [&](int j) {
    K4Tile k;
    const uint8_t* kt = k4base + (size_t)j * 4096 + r * 64 + half * 32;
    const uint8_t* st = ksbase + (size_t)j * 256 + r * 4 + half * 2;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      k.a[2 * t] = *reinterpret_cast<const v4i*>(kt + 2048 * t);
      k.a[2 * t + 1] = *reinterpret_cast<const v4i*>(kt + 2048 * t + 16);
      k.ks[t] = *reinterpret_cast<const uint16_t*>(st + 128 * t);
    }
    return k;
  };
  K4Tile next = load4(w.j0);

  // the query rows as A operand: head u in rows u, u + 4 (u < 4) or u + 4, u + 8, so that accumulator register u of both
  // halves is head u; the lane quantises the two MXFP4 groups it carries
  const int hu = (r & 3) + 4 * (r >> 3);
  const bool qlane = r < (NH > 4 ? 16 : 8) && hu < G;
  const uint16_t* qrow = a.q + (group0 + (qlane ? hu : 0)) * kD;
  v4i qf4[2] = {(v4i){0, 0, 0, 0}, (v4i){0, 0, 0, 0}};
  uint32_t qsc = 0x7f7f7f7fu;
  if (qlane) {
    uint32_t sb[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const uint4* src = reinterpret_cast<const uint4*>(qrow + 64 * half + 32 * kk);
      uint32_t pair[16], codes[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint4 x = src[t];
        pair[4 * t] = x.x; pair[4 * t + 1] = x.y; pair[4 * t + 2] = x.z; pair[4 * t + 3] = x.w;
      }
      sb[kk] = quantize_group32<T>(pair, codes);
      qf4[kk] = (v4i){(int)codes[0], (int)codes[1], (int)codes[2], (int)codes[3]};
    }
    qsc = sb[0] | (sb[1] << 8);
  }

  float top[NH];
#pragma unroll
  for (int u = 0; u < NH; ++u) top[u] = kEmptyMax;
  for (int j = w.j0; j < w.j1; ++j) {
    const int M = promoted_mask(bits, j - w.j0);
    const K4Tile k = next;
    if (j + 1 < w.j1) next = load4(j + 1);
    float s4[NH], s16[NH];
    if (M != all) scores4_row<NH>(k, lane, qf4, qsc, s4);
    if (M != 0) {
      // keys past the cached tokens are not read: the last valid row stands in, its scores are masked below
      const uint16_t* kt = k16base + (size_t)j * kBk * kD + 8 * half;
      v16f acc[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const uint16_t* krow = kt + min(32 * t + r, w.n_valid - 1) * kD;
        acc[t] = (v16f){0.f};
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) {
          const v8s qf = qlane ? *reinterpret_cast<const v8s*>(qrow + 16 * s8 + 8 * half) : (v8s){0, 0, 0, 0, 0, 0, 0, 0};
          acc[t] = T::mfma(qf, *reinterpret_cast<const v8s*>(krow + 16 * s8), acc[t]);
        }
      }
#pragma unroll
      for (int u = 0; u < NH; ++u) s16[u] = half ? acc[1][u] : acc[0][u];
    }
#pragma unroll
    for (int u = 0; u < NH; ++u)
      if (u < G) {
        float v = ((M >> u) & 1) ? s16[u] : s4[u];
        if (lane >= w.n_valid) v = -INFINITY;
        s.scores[(group0 + u) * a.Nkv + (size_t)j * kBk + lane] = v;
        top[u] = fmaxf(top[u], v);
      }
  }
  if (w.tail) return;                                          // a partition of its own: no chunk follows it
#pragma unroll
  for (int u = 0; u < NH; ++u)
    if (u < G) {
      const float m = wave_max(top[u]);
      if (lane == 0) s.cmax[(group0 + u) * s.chunks + w.chunk] = m;
    }
}

template <typename T, int NH>
__global__ void __launch_bounds__(256, 2) decode_split_values_kernel(DecodeSplitArgs s) {
  const DecodeArgs& a = s.a;
  __shared__ __align__(1024) unsigned char tiles[4 * kTile16];              // a 16-bit V tile per wavefront; the partials at the end
  __shared__ __align__(16) uint16_t prow[4 * NH * 64];                      // rounded probabilities of the heads, per wavefront
  __shared__ float ml[4][NH][2];
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, r = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitWork w = split_work(s, wave);
  if (!w.any) return;                                          // uniform over the workgroup
  const int G = a.Hq / a.Hkv;
  const size_t group0 = (size_t)w.b * a.Hq + (size_t)w.kvh * G, kh = (size_t)w.b * a.Hkv + w.kvh;
  const uint8_t* v4base = a.v4 + kh * (size_t)(a.Nkv / 64) * 4096;
  const uint8_t* vsbase = a.vs + kh * (size_t)(a.Nkv / 32) * kD;
  const uint8_t* v16base = reinterpret_cast<const uint8_t*>(a.v16 + kh * a.Nkv * kD);
  unsigned char* tile = tiles + wave * kTile16;
  uint16_t* myp = prow + wave * NH * 64;
  const float c = a.scale * 1.4426950408889634f;

  RowState st[NH];
#pragma unroll
  for (int u = 0; u < NH; ++u) st[u] = {kEmptyMax, 0.f};
  v16f o[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) o[n] = (v16f){0.f};

  if (w.j0 < w.j1) {
    const unsigned long long bits = promoted_bits(a, group0, G, w.j0, lane);
    const int all = (1 << G) - 1, n_blocks = w.j1 - w.j0;
    struct Block {
      v4i v[4];
      uint32_t vs[4];
      float sv[NH];
    };
    auto load = [&](int j) {
      Block x;
      const uint8_t* vt = v4base + (size_t)j * 4096 + r * 32 + half * 16;   // channel 32n + r, token half
      const uint8_t* vsr = vsbase + ((size_t)j * 2 + half) * kD + r;
#pragma unroll
      for (int u = 0; u < NH; ++u) x.sv[u] = u < G ? s.scores[(group0 + u) * a.Nkv + (size_t)j * kBk + lane] : 0.f;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        x.v[n] = *reinterpret_cast<const v4i*>(vt + 1024 * n);
        x.vs[n] = vsr[32 * n];
      }
      return x;
    };
    // 16-bit V tile of block j into the wavefront's own buffer: instruction q covers rows 4q .. 4q+3; rows past the cached
    // tokens are never written by anyone: the last valid row in their place
    const uint32_t lds0 = lds_address(tile);
    auto issue16 = [&](int j) {
      const uint8_t* base = v16base + (size_t)__builtin_amdgcn_readfirstlane(j) * kTile16;
      const uint32_t chunk = (uint32_t)((lane & 15) ^ v16_swizzle(lane >> 4)) * 16;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const uint32_t row = (uint32_t)min(4 * q + (lane >> 4), w.n_valid - 1);
        dma_b128(base, row * 256 + chunk, lds0 + q * 1024);
      }
    };
    Block next = load(w.j0);
    // the next promoted block of the chunk is fetched as soon as the buffer is free
    int j16 = w.j0;
    auto advance16 = [&]() {
      while (j16 < w.j1 && promoted_mask(bits, j16 - w.j0) == 0) ++j16;
      if (j16 < w.j1) issue16(j16);
    };
    advance16();
    // running maximum in front of the chunk
    const int ahead = w.chunk - w.first_chunk;
    if (ahead > 0) {
#pragma unroll
      for (int u = 0; u < NH; ++u)
        if (u < G) {
          const float* cm = s.cmax + (group0 + u) * s.chunks + w.first_chunk;
          float m = kEmptyMax;
          for (int e = lane; e < ahead; e += 64) m = fmaxf(m, cm[e]);
          st[u].m = m;
        }
#pragma unroll
      for (int u = 0; u < NH; ++u) st[u].m = wave_max(st[u].m);
    }
    for (int i = 0; i < n_blocks; ++i) {
      const int j = w.j0 + i;
      const int M = promoted_mask(bits, i);
      const Block x = next;
      if (i + 1 < n_blocks) next = load(j + 1);
      float p[NH], alpha_lane = 1.f;
      uint32_t pb[NH];
      bool grew = false;
#pragma unroll
      for (int u = 0; u < NH; ++u)
        if (u < G) {
          float alpha;
          const bool g = softmax_row(x.sv[u], c, st[u], alpha, pb[u], p[u]);
          if (g) alpha_lane = r == u ? alpha : alpha_lane;
          grew |= g;
        }
      rescale(o, grew, alpha_lane);
      if (M != all) {
        // head u's codes in column u; zeros for the heads that take the block in 16 bits
        v4i pq = {0, 0, 0, 0};
        uint32_t pb_lane = 127u;
        auto place = [&](auto uc) {
          constexpr int u = decltype(uc)::value;
          if (u < G && ((M >> u) & 1) == 0) {
            const v4i mine = gather_p4<u>(p[u], pb[u]);
            if (r == u) { pq = mine; pb_lane = pb[u]; }
          }
        };
        place(std::integral_constant<int, 0>{});
        if constexpr (NH > 1) place(std::integral_constant<int, 1>{});
        if constexpr (NH > 2) { place(std::integral_constant<int, 2>{}); place(std::integral_constant<int, 3>{}); }
        if constexpr (NH > 4) {
          place(std::integral_constant<int, 4>{}); place(std::integral_constant<int, 5>{});
          place(std::integral_constant<int, 6>{}); place(std::integral_constant<int, 7>{});
        }
        pv_fp4_codes_regs<false>(pq, pb_lane, x.vs[0], x.vs[1], x.vs[2], x.vs[3], x.v[0], x.v[1], x.v[2], x.v[3], o);
      }
      if (M != 0) {
#pragma unroll
        for (int u = 0; u < NH; ++u)
          if (u < G) myp[u * 64 + lane] = T::from_float(p[u]);
        const bool mine = r < G && ((M >> r) & 1) != 0;
        v8s pf[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          pf[q] = mine ? *reinterpret_cast<const v8s*>(myp + (r & (NH - 1)) * 64 + 32 * half + 8 * q) : (v8s){0, 0, 0, 0, 0, 0, 0, 0};
        vm_wait<0>();                                          // the tile has arrived (only this wavefront reads it)
        pv_16_rounded<T, true>(tile, lane, pf, o);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // its reads are over before the next tile may land
        ++j16;
        advance16();
      }
    }
    // column u of the accumulators: head u
    if (r < G) {
      float* red = reinterpret_cast<float*>(tile) + r * kD;
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
          *reinterpret_cast<float4*>(red + 32 * n + 8 * g4 + 4 * half) =
              make_float4(o[n][4 * g4], o[n][4 * g4 + 1], o[n][4 * g4 + 2], o[n][4 * g4 + 3]);
    }
  }
#pragma unroll
  for (int u = 0; u < NH; ++u) {
    const float l = wave_sum(st[u].l);
    if (lane == 0) { ml[wave][u][0] = st[u].m; ml[wave][u][1] = l; }
  }
  __syncthreads();
  // the workgroup's partial: chunks of one partition share nothing but the maximum they are scaled to.  A wavefront
  // without blocks has left its tile unwritten; it is skipped by its row sum of zero (with a key it is positive, or the
  // whole partial weighs nothing).
  for (int e = tid; e < G * kD; e += 256) {
    const int u = e >> 7, ch = e & (kD - 1);
    float m = ml[0][u][0];
#pragma unroll
    for (int v = 1; v < 4; ++v) m = fmaxf(m, ml[v][u][0]);
    float l = 0.f, sum = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float lv = ml[v][u][1];
      if (lv > 0.f) {
        const float f = fast_exp2((ml[v][u][0] - m) * c);
        l += f * lv;
        sum += f * reinterpret_cast<const float*>(tiles + v * kTile16)[u * kD + ch];
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
bool decode_split_wanted(int B, int Hq, int Hkv, int Tk, int nsplit, int split_blocks) {
  if (Hq / Hkv > 8) return false;
  if (nsplit > 1 && split_blocks <= 16) return false;
  return (long)B * Hkv * nsplit <= kSplitMaxItems;
}

// key blocks per wavefront: as few as leave about eight wavefronts per CU
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
    decode_split_scores_kernel<T, NH><<<grid, block, 0, st>>>(s);      \
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
