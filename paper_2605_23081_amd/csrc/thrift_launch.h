// Host-side launch interface between the C ABI layer and the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "thrift.h"

namespace thrift {

constexpr int kCus = 256;                 // compute units of the MI355X, 32 in each of 8 XCDs

void launch_block_means(const void* x, thrift_dtype dt, long heads, int N, int block, float* means, hipStream_t st);
// block means of q and k, axis-0 codes of both and axis-1 codes of v [B*H, N, D] in one launch (key blocks of 64)
void launch_prepass(const void* q, const void* k, const void* v, thrift_dtype dt, long heads_q, long heads_kv, int N, int Bq, float* qmean,
                    float* kmean, uint8_t* q4, uint8_t* qs, uint8_t* k4, uint8_t* ks, uint8_t* v4, uint8_t* vs, hipStream_t st);
void launch_quantize(const void* x, thrift_dtype dt, long bh, int N, int axis, uint8_t* codes, uint8_t* scales, hipStream_t st);

struct SelectArgs {
  const float* qmean;
  const float* kmean;
  int32_t* idx;
  int32_t* cnt;
  int B, Hq, Hkv, Tq, Tk, Bq, Bk, causal, fixed_k, q_block_offset, kmax;
  long long ppm;                // budget in millionths
  int selector;                 // 0: TopK of the mean scores; 1: random keys; 2: largest block ids
  unsigned long long seed;      // random selector only
  int shared;                   // selector 0 only: one set per KV head from the query means summed over its group
};
void launch_select_topk(const SelectArgs& a, hipStream_t st);

struct PrefillArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const uint8_t* q4;
  const uint8_t* qs;
  const uint8_t* k4;
  const uint8_t* ks;
  const uint8_t* v4;
  const uint8_t* vs;
  const int32_t* idx;
  const int32_t* cnt;
  void* out;
  float* lse;
  int kmax, B, Hq, Hkv, N, Bq, causal;   // N: key tokens per head
  int tile_order;                         // 0: key blocks ascending (Alg. 1); 1: 4-bit blocks first, then promoted (Sec. 3.3)
  int Nq, q_off;                          // query tokens per head; block position of query block 0 in the sequence
  int interleave, fold;                   // launch_prefill's own: order of the workgroups
  float scale;            // softmax scale (already defaulted)
  thrift_dtype dt, out_dt;
};
void launch_prefill(const PrefillArgs& a, hipStream_t st);
// Four wavefronts per 32 query rows where the grid is small (thrift_prefill_split.hip), the same bits: true where it was launched
bool launch_prefill_split(const PrefillArgs& a, hipStream_t st);

struct DecodeArgs {
  const uint16_t* q;
  const uint16_t* k16;
  const uint16_t* v16;
  const uint8_t* k4;
  const uint8_t* ks;
  const uint8_t* v4;
  const uint8_t* vs;
  const int32_t* seqlens;
  const unsigned long long* bitmap;   // [B,Hq,bitmap_words] selected key blocks per query head
  void* out;
  float* part_o;          // [B,Hq,nparts,D] unnormalised partial outputs
  float* part_ml;         // [B,Hq,nparts,2] running max (raw score units) and row sum of each partial
  int* order;             // nullable [B*Hkv*nsplit]: scratch for the launch order of the split-K workgroups (heaviest first)
  int bitmap_words, B, Hq, Hkv, Nkv, split_blocks, nsplit;
  int nparts;             // partial slots per (sequence, query head): 1 per partition + 1 for a partly filled last block
  int nmerge;             // slots the merge reads (the last one only when lengths were given)
  float scale;
  thrift_dtype dt, out_dt;
};
void launch_decode(const DecodeArgs& a, hipStream_t st);
// entries of DecodeArgs::order that launch_decode wants; 0 = so many workgroups that their order does not matter (pass nullptr)
int decode_order_items(int B, int Hkv, int nsplit);
// Two-pass decode for caches that leave the chip idle otherwise (thrift_decode_split.hip)
struct DecodeSplitArgs {
  DecodeArgs a;           // nparts: partial slots per head here: nsplit * nsub + 1; bitmap may be nullptr (no block promoted)
  float* scores;          // two launches: [B,Hq,Nkv] raw scores
  float* cmax;            // two launches: [B,Hq,chunks] largest raw score of every chunk
  uint32_t* taken;        // two launches, with keys: [B,Hq,items] which of the workgroup's blocks the head has promoted, bit i = its block i
  unsigned* tickets;      // one launch: [B,Hkv,nsplit] workgroups of a partition that have started
  unsigned* tops;         // one launch: [B,Hq,items] largest raw score of every workgroup's blocks, as it becomes known
  int cw;                 // key blocks per chunk (wavefront)
  int nsub;               // workgroups (of four chunks) per partition
  int items;              // workgroups per (sequence, KV head): nsplit * nsub, + 1 where lengths can leave a block partly filled
  int both;               // decode_split_both: both passes in one launch
  int chunks;             // nsplit * nsub * 4
  int polls;              // one launch: how often a maximum is asked for that is not published yet (kSplitPolls)
  int clear;              // no selection has cleared tickets and tops: a launch of its own does
  const uint64_t* keys;   // nullable [B,Hq,Nkv/64]: order keys of the block scores; the kernels then select
  int fixed_k;            // the budget of that selection, as in SelectArgs
  long long ppm;
};
constexpr int kSplitSelectBlocks = 512;      // key blocks up to which the kernels select for themselves: eight keys per lane of a wavefront
// `promoted`: the call's budget promotes some block; the form depends on it
bool decode_split_both(int B, int Hq, int Hkv, int Tk, bool promoted);
bool decode_split_selects(int Tk, bool both);
constexpr int kSplitMaxItems = 448;          // partitions up to which the split is faster than one walk of a workgroup each
constexpr int kSplitMaxItemsOneHead = 512;   // the same for one query head per KV head
constexpr int kSplitMaxChunk = 8;
constexpr uint32_t kUnset = 0xffffffffu;   // a maximum that is not published yet: no sum of products of numbers has these bits
// Some hundred milliseconds.  Only a workspace that somebody else writes during the call lets a wait end without its maximum; the
// results of that sequence's KV head then are NaN.
constexpr int kSplitPolls = 1 << 19;
bool decode_split_wanted(int B, int Hq, int Hkv, int nsplit, int split_blocks);
int decode_split_chunk(int B, int Hq, int Hkv, int Tk, bool promoted);
void launch_decode_split(const DecodeSplitArgs& s, hipStream_t st);
// decode-time selection: scores of the cached key-block means against the query heads, then per-row TopK
// as a bitmap ([B*Hq][words], bit j%64 of word j/64) and optionally as ascending id lists
// `split`: nullable; the block scores also clear its tickets and tops
void launch_decode_block_scores(const uint16_t* q16, int q_is_bf16, const float* kmean, const int32_t* seqlens, uint64_t* keys,
                                int B, int Hq, int Hkv, int Tk, int shared, const DecodeSplitArgs* split, hipStream_t st);
void launch_decode_select(const uint16_t* q16, int q_is_bf16, const float* kmean, const int32_t* seqlens, uint64_t* keys,
                          unsigned long long* bitmap, int words, int32_t* idx_out, int32_t* cnt_out, int kmax_out,
                          int B, int Hq, int Hkv, int Tk, int fixed_k, long long ppm, int shared, const DecodeSplitArgs* split, hipStream_t st);

// Append to the dual cache: tokens seqlens[b] .. seqlens[b] + n - 1 of every (sequence, KV head)
struct CacheAppendArgs {
  const uint16_t* k_new;      // [B,Hkv,n_new,D]
  const uint16_t* v_new;
  const int32_t* seqlens;     // [B] tokens cached before the call
  const int32_t* new_lens;    // nullable [B]: tokens to take from k_new / v_new (<= n_new)
  int32_t* seqlens_out;       // nullable [B]: tokens cached after the call (another array than seqlens)
  uint16_t* k16;              // [B,Hkv,Nkv,D]
  uint16_t* v16;
  uint8_t* k4;
  uint8_t* ks;
  uint8_t* v4;
  uint8_t* vs;
  float* kmean;
  int B, Hkv, Nkv, n_new, blocks_per_unit;
};
void launch_cache_append(const CacheAppendArgs& a, thrift_dtype dt, hipStream_t st);

// measurement microbenchmarks (thrift_peak_probe): returns the work of the launch, 0 for an unknown kind
double launch_peak_probe(int kind, thrift_dtype dt, int iters, void* buffer, size_t bytes, hipStream_t st);

}  // namespace thrift
