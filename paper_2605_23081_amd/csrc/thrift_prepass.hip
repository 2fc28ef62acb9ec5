// Pre-pass kernels of Algorithm 1: block token means (step 3), MXFP4 quantisation (step 2) and
// block-pair scoring + per-row TopK (step 5).  All three are streaming / latency kernels: coalesced
// 16-byte loads, wavefront shuffles and ballots for the reductions, no matrix units.
#include "thrift_device.h"
#include "thrift_launch.h"

namespace thrift {

// ------------------------------------------------------------------------------------------------
// Block means (Sec. 3.2): one workgroup per (b, h, block).  256 threads = 16 row slices x 16 column
// groups of 8 channels; each thread streams rows slice, slice+16, ... with 16-byte loads and adds
// in fp64 (the sum of a block of 16-bit values is then exact, unless bf16 values lie further apart than
// 2^38, so the result does not depend on the order of the additions and matches a serial fp64 mean bit for bit).
// ------------------------------------------------------------------------------------------------
// N need not be a multiple of the block: a head has ceil(N/block) blocks and the last one is the mean
// of the tokens it has.
template <typename T>
__global__ void __launch_bounds__(256) block_means_kernel(const uint16_t* __restrict__ x, float* __restrict__ means,
                                                          int block, int N, int blocks_per_head) {
  const int tid = threadIdx.x;
  const int cg = tid & 15, rs = tid >> 4;
  const int head = blockIdx.x / blocks_per_head, t = blockIdx.x % blocks_per_head;
  const int count = min(block, N - t * block);            // tokens of this block
  const uint16_t* base = x + ((size_t)head * N + (size_t)t * block) * kD + cg * 8;
  double acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.0;
  for (int r = rs; r < count; r += 16) {
    uint4 w = *reinterpret_cast<const uint4*>(base + (size_t)r * kD);
    uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      acc[2 * c] += (double)T::to_float((uint16_t)(ww[c] & 0xffffu));
      acc[2 * c + 1] += (double)T::to_float((uint16_t)(ww[c] >> 16));
    }
  }
  // row slices rs and rs^1, rs^2 sit 16 and 32 lanes apart inside a wavefront
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    acc[c] += __shfl_xor(acc[c], 16);
    acc[c] += __shfl_xor(acc[c], 32);
  }
  __shared__ double part[4][16][8];
  const int wave = tid >> 6;
  if ((tid & 63) < 16) {
#pragma unroll
    for (int c = 0; c < 8; ++c) part[wave][cg][c] = acc[c];
  }
  __syncthreads();
  if (tid < kD) {
    const int g = tid >> 3, c = tid & 7;
    double s = part[0][g][c] + part[1][g][c] + part[2][g][c] + part[3][g][c];
    means[(size_t)blockIdx.x * kD + tid] = (float)(s / (double)count);
  }
}

void launch_block_means(const void* x, thrift_dtype dt, long heads, int N, int block, float* means, hipStream_t st) {
  const int per_head = (N + block - 1) / block;
  const unsigned grid = (unsigned)(heads * per_head);
  if (dt == THRIFT_F16)
    block_means_kernel<F16><<<dim3(grid), dim3(256), 0, st>>>((const uint16_t*)x, means, block, N, per_head);
  else
    block_means_kernel<BF16><<<dim3(grid), dim3(256), 0, st>>>((const uint16_t*)x, means, block, N, per_head);
}

// axis 0: one thread per group of 32 consecutive channels (64 bytes in, 16 code bytes + 1 scale out).
template <typename T>
__global__ void __launch_bounds__(256) quantize_axis0_kernel(const uint16_t* __restrict__ x, uint8_t* __restrict__ codes,
                                                             uint8_t* __restrict__ scales, size_t n_groups) {
  const size_t g = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= n_groups) return;
  const uint4* src = reinterpret_cast<const uint4*>(x + g * 32);
  uint32_t pair[16];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    uint4 w = src[t];
    pair[4 * t] = w.x; pair[4 * t + 1] = w.y; pair[4 * t + 2] = w.z; pair[4 * t + 3] = w.w;
  }
  uint32_t out[4];
  const uint32_t sb = quantize_group32<T>(pair, out);
  *reinterpret_cast<uint4*>(codes + g * 16) = make_uint4(out[0], out[1], out[2], out[3]);
  scales[g] = (uint8_t)sb;
}

// axis 1: one workgroup per (b, h, 64-token block).  The 64 x 128 tile is staged through LDS with
// coalesced 16-byte loads; thread (token group g, channel c) then walks its 32 tokens down a column.
// Output tile: [channel][32 bytes] (tokens 2t, 2t+1 in byte t), scales [2 groups][128 channels].
// N need not be a multiple of 64: a head has ceil(N/64) blocks; tokens past the end count as +0 (they
// do not change a group's largest magnitude and encode as code 0), so a short last group is quantised
// from the tokens it has and the padded codes are zeros.
constexpr int kAxis1Row = kD + 8;  // padded row (in 16-bit elements): keeps 16-byte alignment, spreads banks

template <typename T>
__device__ __forceinline__ void quantize_axis1_block(const uint16_t* __restrict__ x, uint8_t* __restrict__ codes,
                                                     uint8_t* __restrict__ scales, int N, int blocks_per_head, unsigned block,
                                                     uint16_t* tile) {
  constexpr int kRow = kAxis1Row;
  const int tid = threadIdx.x;
  const int head = block / blocks_per_head, t = block % blocks_per_head;
  const int count = min(64, N - t * 64);
  const uint16_t* src = x + ((size_t)head * N + (size_t)t * 64) * kD;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int chunk = tid + 256 * u;           // 1024 chunks of 8 elements
    const int row = chunk >> 4, col = (chunk & 15) * 8;
    *reinterpret_cast<uint4*>(&tile[row * kRow + col]) =
        row < count ? *reinterpret_cast<const uint4*>(src + row * kD + col) : make_uint4(0, 0, 0, 0);
  }
  __syncthreads();
  const int g = tid >> 7, c = tid & 127;
  uint32_t pair[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    uint32_t lo = tile[(32 * g + 2 * u) * kRow + c], hi = tile[(32 * g + 2 * u + 1) * kRow + c];
    pair[u] = lo | (hi << 16);
  }
  uint32_t out[4];
  const uint32_t sb = quantize_group32<T>(pair, out);
  *reinterpret_cast<uint4*>(codes + ((size_t)block * kD + c) * 32 + g * 16) = make_uint4(out[0], out[1], out[2], out[3]);
  scales[((size_t)block * 2 + g) * kD + c] = (uint8_t)sb;
}

template <typename T>
__global__ void __launch_bounds__(256) quantize_axis1_kernel(const uint16_t* __restrict__ x, uint8_t* __restrict__ codes,
                                                             uint8_t* __restrict__ scales, int N, int blocks_per_head) {
  __shared__ __align__(16) uint16_t tile[64 * kAxis1Row];
  quantize_axis1_block<T>(x, codes, scales, N, blocks_per_head, blockIdx.x, tile);
}

void launch_quantize(const void* x, thrift_dtype dt, long bh, int N, int axis, uint8_t* codes, uint8_t* scales, hipStream_t st) {
  const uint16_t* xs = (const uint16_t*)x;
  if (axis == 0) {
    size_t n_groups = (size_t)bh * N * (kD / 32);
    unsigned grid = (unsigned)((n_groups + 255) / 256);
    if (dt == THRIFT_F16) quantize_axis0_kernel<F16><<<dim3(grid), dim3(256), 0, st>>>(xs, codes, scales, n_groups);
    else quantize_axis0_kernel<BF16><<<dim3(grid), dim3(256), 0, st>>>(xs, codes, scales, n_groups);
  } else {
    const int per_head = (N + 63) / 64;
    unsigned grid = (unsigned)(bh * per_head);
    if (dt == THRIFT_F16) quantize_axis1_kernel<F16><<<dim3(grid), dim3(256), 0, st>>>(xs, codes, scales, N, per_head);
    else quantize_axis1_kernel<BF16><<<dim3(grid), dim3(256), 0, st>>>(xs, codes, scales, N, per_head);
  }
}

// ------------------------------------------------------------------------------------------------
// Steps 2 and 3 of Alg. 1 for a whole prompt in one launch: block means and axis-0 codes of Q and K from ONE read of each,
// axis-1 codes of V.  One workgroup per query block, key block and value block.  A thread owns 8 channels of every 16th row,
// as in block_means_kernel; the four lanes of a quad hold one 32-channel group, so a row is quantised where it was loaded
// and 16 lanes store its 64 code bytes together.  Bound by HBM for long prompts (before: five launches, Q and K read twice),
// by the launch for short ones.
// ------------------------------------------------------------------------------------------------
struct PrepassArgs {
  const uint16_t *q, *k, *v;
  float *qmean, *kmean;
  uint8_t *q4, *qs, *k4, *ks, *v4, *vs;
  int N, Bq, Tq, Tk;
  unsigned q_blocks, k_blocks;      // B Hq Tq, B Hkv Tk (as many value blocks as key blocks)
};

template <typename T>
__device__ __forceinline__ void means_and_codes_block(const uint16_t* __restrict__ x, float* __restrict__ means, uint8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ scales, int block, int N, int blocks_per_head, unsigned item,
                                                      double (*part)[16][8]) {
  const int tid = threadIdx.x;
  const int cg = tid & 15, rs = tid >> 4;
  const int head = item / blocks_per_head, t = item % blocks_per_head;
  const int count = min(block, N - t * block);            // tokens of this block
  const size_t row0 = (size_t)head * N + (size_t)t * block;
  const uint16_t* base = x + row0 * kD + cg * 8;
  double acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.0;
#pragma unroll 4
  for (int r = rs; r < count; r += 16) {
    const uint4 w = *reinterpret_cast<const uint4*>(base + (size_t)r * kD);
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      acc[2 * c] += (double)T::to_float((uint16_t)(ww[c] & 0xffffu));
      acc[2 * c + 1] += (double)T::to_float((uint16_t)(ww[c] >> 16));
    }
    uint32_t sb;                                          // the lanes of a quad share the row: all of them are here
    const uint32_t code = quantize_quad8<T>(ww, sb);
    *reinterpret_cast<uint32_t*>(codes + (row0 + r) * (kD / 2) + cg * 4) = code;
    if ((cg & 3) == 0) scales[(row0 + r) * (kD / 32) + (cg >> 2)] = (uint8_t)sb;
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    acc[c] += __shfl_xor(acc[c], 16);
    acc[c] += __shfl_xor(acc[c], 32);
  }
  const int wave = tid >> 6;
  if ((tid & 63) < 16) {
#pragma unroll
    for (int c = 0; c < 8; ++c) part[wave][cg][c] = acc[c];
  }
  __syncthreads();
  if (tid < kD) {
    const int g = tid >> 3, c = tid & 7;
    const double s = part[0][g][c] + part[1][g][c] + part[2][g][c] + part[3][g][c];
    means[(size_t)item * kD + tid] = (float)(s / (double)count);
  }
}

template <typename T>
__global__ void __launch_bounds__(256) prepass_kernel(PrepassArgs p) {
  __shared__ __align__(16) union {
    uint16_t tile[64 * kAxis1Row];
    double part[4][16][8];
  } lds;
  unsigned item = blockIdx.x;
  if (item < p.q_blocks) {
    means_and_codes_block<T>(p.q, p.qmean, p.q4, p.qs, p.Bq, p.N, p.Tq, item, lds.part);
    return;
  }
  item -= p.q_blocks;
  if (item < p.k_blocks) {
    means_and_codes_block<T>(p.k, p.kmean, p.k4, p.ks, kBk, p.N, p.Tk, item, lds.part);
    return;
  }
  quantize_axis1_block<T>(p.v, p.v4, p.vs, p.N, p.Tk, item - p.k_blocks, lds.tile);
}

void launch_prepass(const void* q, const void* k, const void* v, thrift_dtype dt, long heads_q, long heads_kv, int N, int Bq, float* qmean,
                    float* kmean, uint8_t* q4, uint8_t* qs, uint8_t* k4, uint8_t* ks, uint8_t* v4, uint8_t* vs, hipStream_t st) {
  PrepassArgs p;
  p.q = (const uint16_t*)q; p.k = (const uint16_t*)k; p.v = (const uint16_t*)v;
  p.qmean = qmean; p.kmean = kmean; p.q4 = q4; p.qs = qs; p.k4 = k4; p.ks = ks; p.v4 = v4; p.vs = vs;
  p.N = N; p.Bq = Bq; p.Tq = (N + Bq - 1) / Bq; p.Tk = (N + kBk - 1) / kBk;
  p.q_blocks = (unsigned)(heads_q * p.Tq); p.k_blocks = (unsigned)(heads_kv * p.Tk);
  const dim3 grid(p.q_blocks + 2 * p.k_blocks);
  if (dt == THRIFT_F16) prepass_kernel<F16><<<grid, dim3(256), 0, st>>>(p);
  else prepass_kernel<BF16><<<grid, dim3(256), 0, st>>>(p);
}

// ------------------------------------------------------------------------------------------------
// Scores + TopK (Sec. 3.2; Alg. 1 step 5).  A workgroup of 4 wavefronts serves 4 consecutive rows of
// one (b, kv head) in the order (query block, head of the group): they share the staged key-block
// means.  Each wavefront owns one row: lane l scores key blocks l, l+64, ... in fp64, keeps them in
// registers as order-preserving 64-bit keys, finds the k-th largest key by a bitwise search with
// ballot/popcount counting, and emits the selected ids in ascending order.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ int visible_blocks_dev(int i, int Tk, int Bq, int Bk, int causal, int off) {
  if (!causal) return Tk;
  long long last_q = ((long long)i + off + 1) * Bq - 1;
  long long v = last_q / Bk + 1;
  return (int)(v > Tk ? Tk : (v < 0 ? 0 : v));
}

__device__ __forceinline__ int row_budget_dev(int visible, long long ppm, int fixed_k) {
  if (fixed_k >= 0) return fixed_k < visible ? fixed_k : visible;
  if (ppm <= 0) return 0;
  long long k = (ppm * (long long)visible + 999999LL) / 1000000LL;
  if (k < 1) k = 1;
  if (k > visible) k = visible;
  return (int)k;
}

__device__ __forceinline__ uint64_t order_key(double s) {
  uint64_t u = (uint64_t)__double_as_longlong(s);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ULL);   // larger double <=> larger key
}

// Output number n of the SplitMix64 generator seeded with `seed` (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t splitmix64_output(uint64_t seed, uint64_t n) {
  uint64_t z = seed + n * 0x9e3779b97f4a7c15ULL;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
  return z ^ (z >> 31);
}

constexpr int kQuarter = kD / 4;                      // channels staged at a time
constexpr int kStride = kQuarter + 4;                 // padded fp32 quarter row of a staged key mean: conflict-free 16-byte reads

// One staged piece of NC chains per lane: the keys cc * 64 + lane against the row's query mean, U steps of four channels per
// turn of the loop.
template <int NC, int U>
__device__ __forceinline__ void score_piece(const double* q, const float* k, double (&sc)[4]) {
#pragma unroll U
  for (int d = 0; d < kQuarter; d += 4) {
    const double2 qa = *reinterpret_cast<const double2*>(q + d);
    const double2 qb = *reinterpret_cast<const double2*>(q + d + 2);
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) {
      const float4 kv = *reinterpret_cast<const float4*>(k + cc * 64 * kStride + d);
      sc[cc] = fma(qa.x, (double)kv.x, sc[cc]);
      sc[cc] = fma(qa.y, (double)kv.y, sc[cc]);
      sc[cc] = fma(qb.x, (double)kv.z, sc[cc]);
      sc[cc] = fma(qb.y, (double)kv.w, sc[cc]);
    }
  }
}

template <int MAXC, int NW>
__global__ void __launch_bounds__(NW * 64) select_topk_kernel(SelectArgs p) {
  constexpr int kPer = 2048 / (NW * 64);                // 16-byte pieces of a staged piece per thread
  constexpr int kKeys = MAXC < 4 ? 64 * MAXC : 256;     // keys of a staged piece ..
  constexpr int kQuarters = 256 / kKeys;                // .. and quarters of their channels
  __shared__ __align__(16) float kst[256 * kStride];
  __shared__ __align__(16) double qsd[NW][kD];          // the row's query mean (shared mode: summed over the group's heads)
  const int tid = threadIdx.x, lane = tid & 63;
  // wavefront-uniform, and known to the compiler as such: the row, its visible blocks and budget, the threshold and the
  // counts of the search below then live in scalar registers (left as a per-lane value, every count of the search went
  // through vector registers and a branch per chunk: 3600 vector instructions per row instead of 1500)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = p.Hq / p.Hkv;
  const int GR = p.shared ? 1 : G;                      // selection rows per query block and KV head
  const int nheads = p.shared ? G : 1;                  // heads that receive a row's result
  const int rows_per_unit = p.Tq * GR;                  // rows of one (b, kv head), ordered (i, head in group)
  const int wgs_per_unit = (rows_per_unit + NW - 1) / NW;
  // Grid order: the last (under a causal mask: longest) rows of every (b, kv head) first, the units interleaved, so
  // that the launch does not end on its longest workgroups and a KV head's means stay in one XCD's L2 (8 units)
  const int units = p.B * p.Hkv;
  const int unit = blockIdx.x % units;
  const int row0 = (wgs_per_unit - 1 - (int)(blockIdx.x / units)) * NW;
  const int b = unit / p.Hkv, kvh = unit % p.Hkv;
  const float* kbase = p.kmean + (size_t)unit * p.Tk * kD;

  // Every step of a key's chain reads the key mean (per lane) and the query mean (the same address in all lanes, but a
  // full read all the same); with one chain per lane those reads took most of the CU's one LDS pipe.  So a lane walks the
  // chains of four keys (one of each of four 64-key chunks) side by side and reads the query mean once for the four:
  // half the LDS reads per score, and four independent chains of fused multiply-adds.  256 key means are staged a quarter of their channels at a time (36 KiB), fetched into registers while
  // the quarter before is being scored and handed to LDS between two barriers; the workgroup's rows share every
  // staged piece (16 rows: a quarter of the L2 reads of 4).  Rows of one or two chunks, whose time is the waits alone, take four
  // or two quarters of their channels at a time into the same place, and the first piece is asked for before anything else is
  // worked out: 5.0 us instead of 8.9 for 8 workgroups over 32 key blocks, 5.6 / 9.8 for 192 over 47, 9.7 / 13.0 for 512 over 128.
  float4 nx[kPer];
  auto fetch = [&](int t) {                              // piece t of MAXC >= 4: keys 256*(t/4) .. +255, channels 32*(t%4) .. +31
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int chunk = tid + NW * 64 * u;               // 2048 pieces of 4 floats, [quarter][key][channel]
      const int r = (chunk >> 3) % kKeys, q = (chunk >> 3) / kKeys, col = (chunk & 7) * 4;
      const int key0 = MAXC < 4 ? 0 : (t >> 2) * 256, ch0 = MAXC < 4 ? (t * kQuarters + q) * kQuarter : (t & 3) * kQuarter;
      nx[u] = key0 + r < p.Tk ? *reinterpret_cast<const float4*>(kbase + (size_t)(key0 + r) * kD + ch0 + col) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  if (p.selector == 0) fetch(0);
  const int row = row0 + wave;
  const bool active = row < rows_per_unit;
  const int i = active ? row / GR : 0;
  const int hq = kvh * G + (active ? row % GR : 0);     // first (or only) head of the row
  const int cap = p.Tk;
  const int vis = active ? min(cap, visible_blocks_dev(i, p.Tk, p.Bq, p.Bk, p.causal, p.q_block_offset)) : 0;
  const int k = row_budget_dev(vis, p.ppm, p.fixed_k);
  const int last_row = min(row0 + NW - 1, rows_per_unit - 1);
  const int vis_max = min(cap, visible_blocks_dev(last_row / GR, p.Tk, p.Bq, p.Bk, p.causal, p.q_block_offset));
  const size_t rowid = ((size_t)b * p.Hq + hq) * p.Tq + i;

  if (active && p.selector == 0) {
    // fp64 sum over the heads in ascending order (one head: the value itself)
    double q0 = 0.0, q1 = 0.0;
    for (int hh = 0; hh < nheads; ++hh) {
      const float* qm = p.qmean + (rowid + (size_t)hh * p.Tq) * kD;
      q0 += (double)qm[lane];
      q1 += (double)qm[lane + 64];
    }
    qsd[wave][lane] = q0;
    qsd[wave][lane + 64] = q1;
  }

  uint64_t key[MAXC];
#pragma unroll
  for (int c = 0; c < MAXC; ++c) key[c] = 0;
  if (p.selector != 0) {
    // Ablation selectors (App. A): the same k-th-largest search over other keys.  Random: output
    // number n+1 of the SplitMix64 stream of `seed`, n = rowid * 2^32 + j; diagonal: the block id.
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
      const int j = c * 64 + lane;
      if (j < vis) key[c] = p.selector == 1 ? splitmix64_output(p.seed, (((uint64_t)rowid << 32) | (uint64_t)j) + 1ULL) : (uint64_t)j + 1ULL;
    }
  } else if constexpr (MAXC < 4) {
    double sc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 4 / kQuarters; ++t) {
      if (t > 0) __syncthreads();                        // the piece before has been scored by every row
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int chunk = tid + NW * 64 * u;
        *reinterpret_cast<float4*>(&kst[(chunk >> 3) * kStride + (chunk & 7) * 4]) = nx[u];
      }
      if (t + 1 < 4 / kQuarters) fetch(t + 1);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kQuarters; ++q)
        if (vis > 0) score_piece<MAXC, kQuarter / 4>(&qsd[wave][(t * kQuarters + q) * kQuarter], &kst[(q * kKeys + lane) * kStride], sc);
    }
#pragma unroll
    for (int cc = 0; cc < MAXC; ++cc)
      if (cc * 64 + lane < vis) key[cc] = order_key(sc[cc]);
  } else {
#pragma unroll
    for (int cg = 0; cg < MAXC / 4; ++cg) {
      if (cg * 256 < vis_max) {                          // uniform over the workgroup
        double sc[4] = {0.0, 0.0, 0.0, 0.0};             // the chains of keys 256*cg + 64*cc + lane
#pragma unroll 1
        for (int h = 0; h < 4; ++h) {
          __syncthreads();                               // the piece before has been scored by every row
#pragma unroll
          for (int u = 0; u < kPer; ++u) {
            const int chunk = tid + NW * 64 * u;
            const int r = chunk >> 3, col = (chunk & 7) * 4;
            *reinterpret_cast<float4*>(&kst[r * kStride + col]) = nx[u];      // rows beyond Tk: zeros, never used
          }
          const int t1 = cg * 4 + h + 1;
          if (t1 < MAXC && (t1 >> 2) * 256 < vis_max) fetch(t1);              // uniform over the workgroup
          __syncthreads();
          // Uniform over the wavefront; keys past `vis` are scored and dropped, chunks past it left out.  The pieces of one and
          // two chunks take registers that the widest kernel does not have (64 chunks: it spilled, 4070 us instead of 3430
          // for the causal rows of 262144 tokens, 161 instead of 136 for 256 rows of 2100 key blocks), and the kernels of 16
          // rows run whole rows slower with them (267 us instead of 254 for 2048 rows of 1024 key blocks; 90 instead of 92
          // where rows end at 505 to 519): those keep pieces of two, in a loop of their own
          constexpr bool kOne = MAXC == 8 || (NW == 4 && MAXC < 64);
          constexpr int kUnroll = kOne || NW == 4 ? kQuarter / 4 : 2;
          const double* qp = &qsd[wave][h * kQuarter];
          const float* kp = &kst[lane * kStride];
          if (cg * 256 + 128 < vis) score_piece<4, kQuarter / 4>(qp, kp, sc);
          else if (kOne && cg * 256 + 64 < vis) score_piece<2, kUnroll>(qp, kp, sc);
          else if (cg * 256 < vis) score_piece<kOne ? 1 : 2, kUnroll>(qp, kp, sc);
        }
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
          if ((cg * 4 + cc) * 64 + lane < vis) key[cg * 4 + cc] = order_key(sc[cc]);
      }
    }
  }
  if (!active) return;

  if (lane == 0)
    for (int hh = 0; hh < nheads; ++hh) p.cnt[rowid + (size_t)hh * p.Tq] = k;
  if (k <= 0) {
    for (int hh = 0; hh < nheads; ++hh)
      for (int t = lane; t < p.kmax; t += 64) p.idx[(rowid + (size_t)hh * p.Tq) * p.kmax + t] = -1;
    return;
  }
  // k-th largest key: greatest T with |{key >= T}| >= k, built bit by bit from the top
  uint64_t T = 0;
  for (int bit = 63; bit >= 0; --bit) {
    const uint64_t cand = T | (1ULL << bit);
    int n = 0;
#pragma unroll
    for (int c = 0; c < MAXC; ++c)
      if (c * 64 < vis) n += __popcll(__ballot(key[c] >= cand));        // cand > 0 = the key of a lane without a block
    if (n >= k) T = cand;
    if (n == k) break;                                   // exactly the k largest lie at or above cand: done
  }
  int n_gt = 0;
#pragma unroll
  for (int c = 0; c < MAXC; ++c)
    if (c * 64 < vis) n_gt += __popcll(__ballot((c * 64 + lane < vis) && key[c] > T));
  const int need_ties = k - n_gt;                        // ties at T, taken from the smallest id up (0 after an early exit above a gap)
  const uint64_t lt_mask = (1ULL << lane) - 1ULL;
  int written = 0, ties_seen = 0;
#pragma unroll
  for (int c = 0; c < MAXC; ++c) {
    if (c * 64 < vis) {
      const bool valid = c * 64 + lane < vis;
      const bool tie = valid && key[c] == T;
      const uint64_t tie_b = __ballot(tie);
      const bool sel = valid && (key[c] > T || (tie && ties_seen + __popcll(tie_b & lt_mask) < need_ties));
      const uint64_t sel_b = __ballot(sel);
      if (sel)
        for (int hh = 0; hh < nheads; ++hh)
          p.idx[(rowid + (size_t)hh * p.Tq) * p.kmax + written + __popcll(sel_b & lt_mask)] = c * 64 + lane;
      written += __popcll(sel_b);
      ties_seen += __popcll(tie_b);
    }
  }
  for (int hh = 0; hh < nheads; ++hh)
    for (int t = k + lane; t < p.kmax; t += 64) p.idx[(rowid + (size_t)hh * p.Tq) * p.kmax + t] = -1;
}

void launch_select_topk(const SelectArgs& p, hipStream_t st) {
  const int G = p.shared ? 1 : p.Hq / p.Hkv;
  const int chunks = (p.Tk + 63) / 64;
  // 16 rows per workgroup where the keys of a row fit 128 registers per lane, a (b, kv head) has more rows than one workgroup
  // of 4 takes and that many rows leave no CU without a workgroup: a CU works through the chains of its rows one SIMD each,
  // so few rows are better spread (2048 tokens, one head: 18 us with 2 workgroups of 16 rows).  With 16 / 4 rows per
  // workgroup: 71 / 54 us for 4 rows in each of 1024 units and 512 key blocks, 80 / 90 us for 6 rows
  const int nw = (chunks <= 32 && p.Tq * G > 4 && (long)p.B * p.Hkv * ((p.Tq * G + 15) / 16) >= 256) ? 16 : 4;
  const int wgs_per_unit = (p.Tq * G + nw - 1) / nw;
  const dim3 grid((unsigned)((long)p.B * p.Hkv * wgs_per_unit));
  if (nw == 16) {
    if (chunks <= 1) select_topk_kernel<1, 16><<<grid, dim3(1024), 0, st>>>(p);
    else if (chunks <= 2) select_topk_kernel<2, 16><<<grid, dim3(1024), 0, st>>>(p);
    else if (chunks <= 8) select_topk_kernel<8, 16><<<grid, dim3(1024), 0, st>>>(p);
    else if (chunks <= 16) select_topk_kernel<16, 16><<<grid, dim3(1024), 0, st>>>(p);
    else select_topk_kernel<32, 16><<<grid, dim3(1024), 0, st>>>(p);
  } else {
    if (chunks <= 1) select_topk_kernel<1, 4><<<grid, dim3(256), 0, st>>>(p);
    else if (chunks <= 2) select_topk_kernel<2, 4><<<grid, dim3(256), 0, st>>>(p);
    else if (chunks <= 8) select_topk_kernel<8, 4><<<grid, dim3(256), 0, st>>>(p);
    else if (chunks <= 16) select_topk_kernel<16, 4><<<grid, dim3(256), 0, st>>>(p);
    else if (chunks <= 32) select_topk_kernel<32, 4><<<grid, dim3(256), 0, st>>>(p);
    else select_topk_kernel<64, 4><<<grid, dim3(256), 0, st>>>(p);
  }
}

}  // namespace thrift
