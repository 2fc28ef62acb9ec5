// Fused mixed-precision flash attention for prefill (Algorithm 1 steps 4-23; Sec. 3.3).
//
// One workgroup = one query block of one (batch, query head), or two of 64 rows; wavefront w owns rows
// 32w .. 32w+31 and keeps Q, the online-softmax state and the O^T accumulators in registers.  Two walks over
// the key blocks are built, both dispatching per tile to the scaled-FP4 or the 16-bit MFMA path:
//   ORDER 0  ascending block order, Alg. 1 as written (a second staging schedule, WIDE, serves high budgets);
//   ORDER 1  the order of the kernel in Sec. 3.3: every 4-bit block first, then the promoted blocks with the
//            16-bit query fragments in registers only for that phase.  This is the benchmarked walk.
//
// The kernel is bound by the vector ALU work of the softmax and the P quantiser (exp and the FP4
// converter run at a quarter of the plain rate), and one wavefront can issue vector instructions at only
// about half the rate its SIMD can execute them.  Everything is therefore sized for THREE workgroups per
// CU (three wavefronts per SIMD): at most 168 vector registers and a third of the LDS per workgroup.
//   * Every block is staged once into LDS for all wavefronts by LDS DMA (global loads that write LDS
//     directly: no staging registers, no LDS write instructions), one block ahead of the arithmetic:
//     MXFP4 codes + scales into one of two 8.5 KiB slots, the 16-bit K and V tiles of a block listed in
//     the row's TopK set into 16 KiB tile buffers.
//   * One workgroup barrier per 4-bit key block orders the traffic, two per promoted block.
//
// Differences from the kernel the paper sketches for Blackwell (Sec. 3.3): MXFP4 instead of NVFP4, 32x32
// MFMA tiles in transposed form (one query per lane column) instead of warp-level MMA tiles, LDS regions
// per precision instead of one aliased region (three workgroups per CU are worth more than the aliasing).
#include <type_traits>

#include "thrift_launch.h"
#include "thrift_tile.h"

namespace thrift {

// LDS map of the prefill kernel (bytes)
constexpr int kLdsRing = 0;                                  // two slots of kLdsBytes4 (block j -> slot j & 1)
constexpr int kLdsV16 = 2 * kLdsBytes4;                      // one swizzled 16-bit V tile
constexpr int kLdsK16 = kLdsV16 + kTile16;                   // one swizzled 16-bit K tile
constexpr int kLdsPrefill = kLdsK16 + kTile16;               // 50176: three workgroups per CU
// LDS map of the wide schedule: two slots that hold one key block each, whatever its path
// (a 4-bit block in the first kLdsBytes4 bytes; a promoted block as its K tile followed by its V tile)
constexpr int kWideSlot = 2 * kTile16;                       // 32768
constexpr int kLdsPrefillWide = 2 * kWideSlot;               // 65536: two workgroups per CU
constexpr int kWidePercent = 15;                             // list length / key blocks (in %) from which the wide schedule is used

// One work item: 32 NW query rows of a (sequence, query head) and all their key blocks.  `work` is the item's position in the
// launch order (what blockIdx.x is in the one-item-per-workgroup launch).
// NL: query blocks among these rows, each with a list of promoted blocks of its own: one, or two of 64 rows.  With two the
// walk takes the blocks of both: a block that only one of them has promoted is staged in both precisions, and each wavefront
// computes what its own list says.  A workgroup per query block of 64 rows had two wavefronts for the LDS of four, one and a half per
// SIMD, and staged every block for half the rows.  One query block / two, 5 %: 542 / 314 us for 8192 tokens, 32/8 heads; 200 / 141
// for 2 x 3000, 16/16, 25 %, no mask; 730 / 597 for a chunk of 1000 on 30720, 10 %; 160 / 120 for 2000, 64/8, 100 %.
// TURNS: see take_turns.  An instance of its own: asked at every key block the question cost grids of at most one workgroup per CU,
// where a lone wavefront per SIMD issues every scalar instruction at its own expense, 2 % (chunk of 1000 tokens on 16384, 32/8
// heads, 5 %: 227.1 us without turns, 231.8 with the question, 224.4 now; 2000 with 16/16: 239.5 / 244.7 / 236.7).  For the same reason the walks
// say which way their branches mostly go (no mask, no promoted block, a whole 4-bit block, rows that see it): that keeps the
// rare ways out of line, 230.4 -> 224.4 us.
template <typename T, int NW, int NL, int ORDER, int WIDE, int TURNS>
__device__ __forceinline__ void prefill_item(const PrefillArgs& a, unsigned char* lds, unsigned work) {
  static_assert(NL == 1 || !WIDE, "a slot of the wide schedule holds a block in one precision");
  constexpr int KF = 4 / NW;                 // 1 KiB fragments of a 4-bit K (and of a V) tile per wavefront
  constexpr int C16 = 16 / NW;               // ... for one 16-bit K or V tile
  constexpr int kSlotStride = WIDE ? kWideSlot : kLdsBytes4;

  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, r = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront-uniform: loop bounds stay scalar
  const int N = a.N, Nq = a.Nq, G = a.Hq / a.Hkv;
  constexpr int kRows = NW * 32, kRowsPerList = kRows / NL;     // of an item; of a query block
  const int Tw = (Nq + kRows - 1) / kRows, Tk = (N + kBk - 1) / kBk;   // the last item / key block may be short
  const int Tq = (Nq + kRowsPerList - 1) / kRowsPerList;

  // ---- work item: heavy (late) query blocks first; KV heads spread over the 8 XCDs so that the query
  // heads and neighbouring query blocks that share a KV head also share an L2 ----
  const int units = a.B * a.Hkv;
  const int xcds = (units & 7) == 0 ? 8 : 1, units_here = units / xcds;
  int t = work / xcds;
  if (a.fold) {                                          // the second workgroup of every CU: shortest first
    const int per = kCus / xcds, end = min(2 * per, (int)gridDim.x / xcds);
    if (t >= per && t < end) t = per + end - 1 - t;
  }
  int unit, within;                                      // the unit's on this XCD; (query block from the last one on, head of the group)
  if (a.interleave) {
    const int rest = t % (units_here * G);
    unit = rest / G;
    within = t / (units_here * G) * G + rest % G;
  } else {
    unit = t / (G * Tw);
    within = t % (G * Tw);
  }
  unit = work % xcds + xcds * unit;
  const int b = unit / a.Hkv, kvh = unit % a.Hkv;
  const int i = Tw - 1 - within / G;
  const int hq = kvh * G + within % G;
  const size_t qh = (size_t)b * a.Hq + hq, kh = (size_t)b * a.Hkv + kvh;
  const int q_first = a.q_off * kRowsPerList + i * kRows;   // sequence position of the first query row
  const int q0 = q_first + wave * 32;                   // ... of this wavefront's
  // The lane's query row inside the head.  Rows past the last query repeat it and are never stored.  Only this
  // 32-bit index is kept; addresses are rebuilt from it and scalar bases where they are needed (registers are
  // what limits this kernel to three wavefronts per SIMD).
  const int lrow = min(i * kRows + wave * 32 + r, Nq - 1);
  const size_t qrow = qh * Nq + lrow;

  // ---- Q fragments ----
  v4i qf4[2];
  // fragment kk: d-group 2*half + kk (scores_fp4); its scale is byte kk of qsc
  qf4[0] = *reinterpret_cast<const v4i*>(a.q4 + qrow * 64 + half * 32);
  qf4[1] = *reinterpret_cast<const v4i*>(a.q4 + qrow * 64 + half * 32 + 16);
  const uint32_t qsc = *reinterpret_cast<const uint32_t*>(a.qs + qrow * 4) >> (16 * half);
  const uint8_t* q16head = reinterpret_cast<const uint8_t*>(a.q + qh * Nq * kD);   // wavefront-uniform

  const int vis = a.causal ? min(Tk, (q_first + kRows - 1) / kBk + 1) : Tk;
  const int own = NL == 1 ? 0 : wave / (NW / NL);      // this wavefront's list
  const int32_t* sel[NL];
  int nsel[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const bool there = l == 0 || NL * i + l < Tq;                  // the last item may have one query block
    const size_t row = qh * Tq + NL * i + (there ? l : 0);
    sel[l] = a.idx + row * a.kmax;
    nsel[l] = there ? min(a.cnt[row], a.kmax) : 0;                 // a count beyond the list length is cut, never followed
  }
  // Entry t of list l, through the scalar data path.  The list index is wavefront-uniform, but the compiler
  // cannot prove that (it depends on list entries read earlier) nor that the list is not written here, and turns a
  // plain read into a vector load plus a wait for EVERY vector load in flight, the tile DMAs included.
  constexpr int kNone = 0x7fffffff;
  auto sel_at = [&](int l, int t) -> int {
    const int32_t* p = sel[l] + __builtin_amdgcn_readfirstlane(t);
    int v;
    asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(p) : "memory");
    return min(max(v, 0), Tk - 1);                      // whatever the list holds, only ids of existing key blocks become addresses
  };
  // the next two promoted block ids of each list at or after the current block (ascending lists)
  int ps[NL], n0[NL], n1[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    ps[l] = 0;
    n0[l] = nsel[l] > 0 ? sel_at(l, 0) : kNone;
    n1[l] = nsel[l] > 1 ? sel_at(l, 1) : kNone;
  }
  // block J, whose next entries are X: promoted by some list, by all of them, by this wavefront's
  auto some = [&](const int (&x)[NL], int j) { return NL == 1 ? x[0] == j : x[0] == j || x[NL - 1] == j; };
  auto all = [&](const int (&x)[NL], int j) { return NL == 1 ? x[0] == j : x[0] == j && x[NL - 1] == j; };
  auto mine = [&](const int (&x)[NL], int j) { return (NL == 1 || own == 0 ? x[0] : x[NL - 1]) == j; };

  const uint8_t* k4base = a.k4 + kh * N * 64;
  const uint8_t* v4base = a.v4 + kh * (size_t)Tk * 4096;
  const uint8_t* ksbase = a.ks + kh * N * 4;
  const uint8_t* vsbase = a.vs + kh * (size_t)Tk * 2 * kD;
  const uint8_t* k16base = reinterpret_cast<const uint8_t*>(a.k + kh * N * kD);
  const uint8_t* v16base = reinterpret_cast<const uint8_t*>(a.v + kh * N * kD);

  // ---- staging: per-lane source offsets of the DMA instructions this wavefront issues.  The LDS side of
  // a DMA is linear in the lane index, so every layout change (MFMA fragment order of the 4-bit tiles,
  // chunk swizzle of the 16-bit tiles) is expressed in the global offsets. ----
  const uint32_t lds0 = lds_address(lds);
  uint32_t k4off[KF], v4off[KF];
#pragma unroll
  for (int u = 0; u < KF; ++u) {
    const int f = wave * KF + u;                         // K: fragment (t, kk) = (f>>1, f&1); V: channels 32f .. 32f+31
    k4off[u] = (uint32_t)(key_of_row(r, f >> 1) * 64 + (2 * half + (f & 1)) * 16);    // d-group 2*half + kk of the key
    v4off[u] = (uint32_t)((32 * f + r) * 32 + half * 16);
  }
  const uint32_t scoff = (uint32_t)lane * 4;
  // the 256 scale bytes of K ride with the even wavefronts, V's with the odd ones: picked once, in scalar registers
  const bool v_scales = (wave & 1) != 0;
  const uint8_t* scbase = v_scales ? vsbase : ksbase;
  const uint32_t sclds = v_scales ? (uint32_t)kLdsVS : (uint32_t)kLdsKS;
  // 16-bit tiles: one instruction covers 4 rows; lane l writes chunk position l&15 of row l>>4
  // (formed from the lane index where a 16-bit tile is issued, one block in twenty on the headline budget,
  // rather than held in registers through every 4-bit block)
#define THRIFT_V16OFF() ((uint32_t)((lane16 >> 4) * 256 + ((lane16 & 15) ^ v16_swizzle(lane16 >> 4)) * 16))
#define THRIFT_K16OFF() ((uint32_t)((lane16 >> 4) * 256 + ((lane16 & 15) ^ (lane16 >> 4)) * 16))   /* rows 32..63: chunk ^ 4 more */

  // A short last key block: the rows past the last key do not exist in the row-major arrays (K codes and
  // scales, 16-bit K and V); their lanes re-read the last key's row instead, and the mask below keeps
  // whatever lands there out of the arithmetic.  (V codes and scales are stored in whole, zero-padded blocks.)
  // The clamped offsets are formed inside the branch that handles the short block (the empty asm keeps the
  // compiler from hoisting a second set of per-lane offsets out of the key loop, which would cost registers
  // on the path every other block takes).
  const int last_key_row = (N - 1) & (kBk - 1);
#define THRIFT_CLAMP_ROWS(OFF, SHIFT, LAST) ((min((uint32_t)(OFF) >> (SHIFT), (LAST)) << (SHIFT)) | ((OFF) & ((1u << (SHIFT)) - 1u)))
#define THRIFT_ISSUE4(J) THRIFT_ISSUE4_SLOT(J, (J) & 1)
#define THRIFT_ISSUE4_SLOT(J, S)                                                                               \
  do {                                                                                                         \
    const int j_ = __builtin_amdgcn_readfirstlane(J), s_ = __builtin_amdgcn_readfirstlane(S); /* scalar operands */ \
    const uint8_t* kt_ = k4base + (size_t)j_ * 4096;                                                           \
    const uint8_t* vt_ = v4base + (size_t)j_ * 4096;                                                           \
    int wave_ = wave;                                                                                          \
    asm volatile("" : "+s"(wave_));   /* LDS destinations are formed here from one scalar, not kept per slot and fragment */ \
    const uint32_t sl_ = lds0 + kLdsRing + s_ * kSlotStride + (uint32_t)(wave_ * (KF * 1024));                 \
    if (__builtin_expect((j_ + 1) * kBk <= N, 1)) {                                                            \
      _Pragma("unroll") for (int u = 0; u < KF; ++u) dma_b128(kt_, k4off[u], sl_ + kLdsK4 + u * 1024);         \
      dma_b32(scbase + (size_t)j_ * 256, scoff, sl_ - (uint32_t)(wave_ * (KF * 1024)) + sclds);                \
    } else {                                                                                                   \
      uint32_t last_ = (uint32_t)last_key_row;                                                                 \
      asm volatile("" : "+s"(last_));                                                                          \
      _Pragma("unroll") for (int u = 0; u < KF; ++u)                                                           \
        dma_b128(kt_, THRIFT_CLAMP_ROWS(k4off[u], 6, last_), sl_ + kLdsK4 + u * 1024);                         \
      /* V scales are stored in whole, zero-padded blocks; K's rows past the last key do not exist */          \
      dma_b32(scbase + (size_t)j_ * 256, v_scales ? scoff : THRIFT_CLAMP_ROWS(scoff, 2, last_),                \
              sl_ - (uint32_t)(wave_ * (KF * 1024)) + sclds);                                                  \
    }                                                                                                          \
    /* V codes: whole blocks */                                                                                \
    _Pragma("unroll") for (int u = 0; u < KF; ++u) dma_b128(vt_, v4off[u], sl_ + kLdsV4 + u * 1024);           \
  } while (0)
  // 16-bit tiles: instruction q_ covers rows 4 q_ .. 4 q_ + 3
#define THRIFT_ISSUE_TILE16(BASE, J, OFFEXPR, LDSBASE)                                                         \
  do {                                                                                                         \
    const int j_ = __builtin_amdgcn_readfirstlane(J);                                                          \
    const uint8_t* t_ = (BASE) + (size_t)j_ * kTile16;                                                         \
    int lane16 = lane, wave_ = wave;                                                                           \
    asm volatile("" : "+v"(lane16), "+s"(wave_));   /* offsets and destinations are computed here, not carried through the key loop */ \
    if ((j_ + 1) * kBk <= N) {                                                                                 \
      _Pragma("unroll") for (int u = 0; u < C16; ++u) {                                                        \
        const int q_ = u * NW + wave_;                                                                         \
        dma_b128(t_ + q_ * 1024, (OFFEXPR), (LDSBASE) + q_ * 1024);                                            \
      }                                                                                                        \
    } else {                                                                                                   \
      uint32_t last_ = (uint32_t)last_key_row;                                                                 \
      asm volatile("" : "+s"(last_));                                                                          \
      _Pragma("unroll") for (int u = 0; u < C16; ++u) {                                                        \
        const int q_ = u * NW + wave_;                                                                         \
        const uint32_t o_ = (uint32_t)(q_ * 1024) + (OFFEXPR);   /* offset from the tile start */              \
        dma_b128(t_, THRIFT_CLAMP_ROWS(o_, 8, last_), (LDSBASE) + q_ * 1024);                                  \
      }                                                                                                        \
    }                                                                                                          \
  } while (0)
#define THRIFT_ISSUE_V16(J) THRIFT_ISSUE_TILE16(v16base, J, THRIFT_V16OFF(), lds0 + kLdsV16)
#define THRIFT_ISSUE_K16(J) THRIFT_ISSUE_TILE16(k16base, J, (u * NW >= 8 ? THRIFT_K16OFF() ^ 64u : THRIFT_K16OFF()), lds0 + kLdsK16)

  RowState st = {kEmptyMax, 0.f};
  v16f o[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) o[n] = (v16f){0.f};
  const float c = a.scale * 1.4426950408889634f;

  // Blocks this wavefront computes: those with at least one key at or before its last query row.  The
  // later blocks of the workgroup (visible only to wavefronts with later rows) are still staged and
  // synchronised on, in a final loop without arithmetic.
  const int vis_wave = a.causal ? min(vis, (q0 + 31) / kBk + 1) : vis;
  // keys at positions below key_limit are visible to the lane's query: those at or before its own position
  // (causal) and only keys that exist
  const int key_limit = a.causal ? min(q0 + r + 1, N) : N;

  // One step of the staging pipeline at block J, with P0 = "some list has promoted block J", P1 / ALL1 = "some / every list
  // has promoted block J+1".
  //  SYNC:  wait for this wavefront's share of block J, then meet the others: block J is complete in LDS
  //         and everyone has finished block J-1 (whose buffers are free again).
  //  ISSUE: block J+1 — its 4-bit tiles into the other slot, unless every list has promoted it; the tiles of a promoted block into
  //         the 16-bit buffers, unless block J is using them (then its K tile follows the score phase of block J and its V
  //         tile the start of step J+1: late_v).
  // Workgroups with rows of one length that share a CU take turns of 16 key blocks with the higher wavefront priority (take_turns).
  const int turn = (int)(work / kCus) & 1;
  bool ahead = false;
  auto take_turn = [&](int j) __attribute__((always_inline)) {
    if constexpr (TURNS) {
      const bool mine_ = ((j >> 4) & 1) == turn;
      if (mine_ != ahead) {
        ahead = mine_;
        if (mine_) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
    }
  };
  bool late_v = false;                                  // block J is promoted and its V tile is not issued yet
#define THRIFT_SYNC()                                                                                          \
  vm_wait<0>();                                                                                                \
  lds_barrier();
#define THRIFT_ISSUE(J, P0, P1, ALL1)                                                                          \
  if ((J) + 1 < vis) {                                                                                         \
    if (!(ALL1)) THRIFT_ISSUE4((J) + 1);                                                                       \
    if ((P1) && !(P0)) {                                                                                       \
      THRIFT_ISSUE_K16((J) + 1);                                                                               \
      THRIFT_ISSUE_V16((J) + 1);                                                                               \
    }                                                                                                          \
  }
#define THRIFT_MASK(J)                                                                                         \
  const bool mask = (a.causal && (J) * kBk + kBk - 1 > q0) || ((J) + 1) * kBk > N;                             \
  const int n_valid = key_limit - (J) * kBk;   /* leading keys of the block this query may see */
  auto next_promoted = [&](int l) {
    ++ps[l];
    n0[l] = n1[l];
    n1[l] = ps[l] + 1 < nsel[l] ? sel_at(l, ps[l] + 1) : kNone;
  };
  // List entries behind the walk's position (a list that is not strictly ascending breaks the contract) are
  // dropped, at the same point of every wavefront's walk: the wavefronts of a workgroup must take identical
  // staging and barrier decisions whatever the list holds.
  auto drop_stale = [&](int j) {
#pragma unroll
    for (int l = 0; l < NL; ++l)
      while (n0[l] < j) next_promoted(l);
  };
  // the lists' entries behind block j, which is the current one
  auto behind = [&](int j, int (&x)[NL]) {
#pragma unroll
    for (int l = 0; l < NL; ++l) x[l] = n0[l] == j ? n1[l] : n0[l];
  };
  auto advance = [&](int j) {
#pragma unroll
    for (int l = 0; l < NL; ++l)
      if (n0[l] == j) next_promoted(l);
  };

  // 16-bit query fragments of the lane's row (the wide schedule keeps them in registers for the whole walk; the
  // three-workgroup schedule has no registers to spare and fetches them again at every promoted block)
#define THRIFT_LOAD_Q16_ROW(QF, LROW)                                                                          \
  _Pragma("unroll") for (int s8 = 0; s8 < 8; ++s8)                                                             \
    QF[s8] = *reinterpret_cast<const v8s*>(q16head + (uint32_t)((LROW) * (2 * kD) + 32 * s8 + 16 * half));     \
  _Pragma("unroll") for (int s8 = 0; s8 < 8; ++s8) asm volatile("" : "+v"(QF[s8]));
#define THRIFT_LOAD_Q16(QF) THRIFT_LOAD_Q16_ROW(QF, lrow)
  // The lane's row index formed again from the thread id (the empty asm hides it from common-subexpression
  // elimination): used where keeping the first copy alive through a long loop would cost a register there.
#define THRIFT_ROW_AGAIN(UNCLAMPED)                                                                            \
  int UNCLAMPED = (int)(threadIdx.x & 31);                                                                     \
  asm volatile("" : "+v"(UNCLAMPED));                                                                          \
  UNCLAMPED += i * kRows + wave * 32;

  if constexpr (WIDE) {
    // ---- wide schedule: every block, 4-bit or promoted, is fetched one whole step ahead into the slot the
    // block before last has left; one barrier per key block, no second rendezvous for promoted blocks ----
#define THRIFT_ISSUE_WIDE(J1, P1)                                                                              \
  if ((J1) < vis) {                                                                                            \
    if (P1) {                                                                                                  \
      THRIFT_ISSUE_TILE16(k16base, J1, (u * NW >= 8 ? THRIFT_K16OFF() ^ 64u : THRIFT_K16OFF()),                \
                          lds0 + (uint32_t)(((J1) & 1) * kWideSlot));                                          \
      THRIFT_ISSUE_TILE16(v16base, J1, THRIFT_V16OFF(), lds0 + (uint32_t)(((J1) & 1) * kWideSlot + kTile16));  \
    } else {                                                                                                   \
      THRIFT_ISSUE4(J1);                                                                                       \
    }                                                                                                          \
  }
    // the 16-bit query fragments stay in registers (this schedule has 256 of them)
    v8s qf[8];
    THRIFT_LOAD_Q16(qf)
    if (vis > 0) { THRIFT_ISSUE_WIDE(0, n0[0] == 0) }
    int j = 0;
    while (j < vis_wave) {
      drop_stale(j);
      const int run_end = min(vis_wave, n0[0]);
      for (; j < run_end; ++j) {                          // a run of 4-bit blocks
        take_turn(j);
        THRIFT_SYNC()
        THRIFT_ISSUE_WIDE(j + 1, j + 1 == n0[0])
        THRIFT_MASK(j)
        const unsigned char* slot = lds + (j & 1) * kWideSlot;
        v16f s[2];
        float alpha;
        uint32_t pb;
        scores_fp4(slot, lane, qf4, qsc, s);
        const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
        rescale(o, grew, alpha);
        pv_fp4(slot, lane, s, pb, o);
      }
      if (j < vis_wave) {                                 // j == n0[0]: a promoted block
        THRIFT_SYNC()
        THRIFT_ISSUE_WIDE(j + 1, j + 1 == n1[0])
        THRIFT_MASK(j)
        const unsigned char* slot = lds + (j & 1) * kWideSlot;
        v16f s[2];
        scores_16<T>(slot, lane, qf, s);
        float alpha;
        uint32_t pb;
        const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
        rescale(o, grew, alpha);
        pv_16<T, true>(slot + kTile16, lane, s, o);
        next_promoted(0);
        ++j;
      }
    }
    for (; j < vis; ++j) {                                // staging only: blocks that later wavefronts still need
      drop_stale(j);
      const bool p0 = j == n0[0];
      THRIFT_SYNC()
      THRIFT_ISSUE_WIDE(j + 1, j + 1 == (p0 ? n1[0] : n0[0]))
      if (p0) next_promoted(0);
    }
#undef THRIFT_ISSUE_WIDE
  } else if constexpr (ORDER == 1) {
    // ---- the order of Sec. 3.3: every 4-bit block in ascending order, then the promoted blocks in ascending
    // order.  Same staging rules; the ring slot follows the step number because block ids now skip. ----
    int nselv[NL];                                      // promoted ids inside the visible range (the list is ascending)
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      nselv[l] = nsel[l];
      if (nsel[l] > 0 && sel_at(l, nsel[l] - 1) >= vis) {
        nselv[l] = 0;
        while (nselv[l] < nsel[l] && sel_at(l, nselv[l]) < vis) ++nselv[l];
      }
    }
    // the lists' next entries at or after a walk's position: of the 4-bit walk, then of the promoted one
    int nx[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) nx[l] = nselv[l] > 0 ? n0[l] : kNone;
    auto first_of = [&](const int (&x)[NL]) { return NL == 1 ? x[0] : min(x[0], x[NL - 1]); };
    auto pass = [&](int l) {                            // to the list's entry behind this one
      ++ps[l];
      nx[l] = ps[l] < nselv[l] ? sel_at(l, ps[l]) : kNone;
    };
    const int first_promoted = first_of(nx);
    int next4;                                          // the next block that some list takes in 4 bits
    bool own4 = true, next_own4;                        // this wavefront's list takes the current / that block in 4 bits
    auto seek = [&](int j) {
      if constexpr (NL == 1) {
        while (__builtin_expect(j == nx[0], 0)) { ++j; pass(0); }
        next_own4 = true;
      } else {
        for (;;) {
          bool p[NL];
#pragma unroll
          for (int l = 0; l < NL; ++l) {
            while (nx[l] < j) pass(l);
            p[l] = nx[l] == j;
          }
          next_own4 = !(own == 0 ? p[0] : p[NL - 1]);
          if (!(p[0] && p[NL - 1])) break;
          ++j;
        }
      }
      next4 = j;
    };
    seek(0);
    int j = next4;
    own4 = next_own4;
    if (j < vis) {
      THRIFT_ISSUE4_SLOT(j, 0);
    } else if (first_promoted < vis) {
      THRIFT_ISSUE_K16(first_promoted);
      THRIFT_ISSUE_V16(first_promoted);
    }
    // Phase A, two steps per trip so that the ring slot of each step is a compile-time constant: every LDS
    // read of the step is then a lane-constant address register plus an immediate offset, no address arithmetic.
    auto step_a = [&](auto slot_c) __attribute__((always_inline)) {
      constexpr int SLOT = decltype(slot_c)::value;
      seek(j + 1);
      take_turn(j);
      THRIFT_SYNC()
      if (__builtin_expect(next4 < vis, 1)) {
        THRIFT_ISSUE4_SLOT(next4, SLOT ^ 1);
      } else if (first_promoted < vis) {
        THRIFT_ISSUE_K16(first_promoted);
        THRIFT_ISSUE_V16(first_promoted);
      }
      if ((NL == 1 || own4) && __builtin_expect(j < vis_wave, 1)) {
        THRIFT_MASK(j)
        const unsigned char* slot = lds + kLdsRing + SLOT * kLdsBytes4;
        v16f s[2];
        float alpha;
        uint32_t pb;
        scores_fp4(slot, lane, qf4, qsc, s);
        const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
        rescale(o, grew, alpha);
        pv_fp4(slot, lane, s, pb, o);
      }
      j = next4;
      own4 = next_own4;
    };
    while (j < vis) {                                   // phase A
      step_a(std::integral_constant<int, 0>{});
      if (j >= vis) break;
      step_a(std::integral_constant<int, 1>{});
    }
    // phase B: the promoted blocks follow each other.  The lane's 16-bit query fragments are fetched once and stay
    // in registers for the whole phase (the 4-bit phase, which has no registers to spare, is over: Sec. 3.3 scopes
    // them the same way).  The 4-bit slots are idle now, so the 16-bit tiles rotate through THREE 16 KiB buffers in
    // the order they are consumed, K(b), V(b), K(b+1), ...: tile t sits in buffer t mod 3 and may be fetched as
    // soon as everyone has finished with tile t-3.  That puts K(b+1) in flight at the start of block b and V(b+1)
    // right after the scores of block b, half a block earlier each than two fixed buffers allow.
    v8s qf[8];
    if (first_promoted < vis_wave) {
      THRIFT_ROW_AGAIN(row_b)
      THRIFT_LOAD_Q16_ROW(qf, min(row_b, Nq - 1))
    }
    // buffer 0: the K region (holds K of the first promoted block), 1: the V region (its V), 2: the 4-bit slots' region
#define THRIFT_TILE_BUFFER(X) ((X) == 0 ? kLdsK16 : (X) == 1 ? kLdsV16 : kLdsRing)
    int kbuf = 0;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      ps[l] = 0;
      nx[l] = nselv[l] > 0 ? n0[l] : kNone;
    }
    int jb = first_promoted;
    while (jb < vis) {
      const bool own16 = NL == 1 || mine(nx, jb), use = own16 && jb < vis_wave;
      if constexpr (NL == 1) {
        pass(0);
      } else {
        do {                                            // (an entry that is not larger than the one before breaks the contract)
#pragma unroll
          for (int l = 0; l < NL; ++l)
            if (nx[l] <= jb) pass(l);
        } while (first_of(nx) <= jb);
      }
      const int jb_next = first_of(nx);
      const bool p1 = jb_next < vis;
      const int vbuf = kbuf == 2 ? 0 : kbuf + 1;
      const int kbuf_next = vbuf == 2 ? 0 : vbuf + 1;
      vm_wait<C16>();                                   // this wavefront's share of K(b); V(b) may still be on its way
      lds_barrier();                                    // K(b) complete; everyone has finished the block before
      if (p1) {
        THRIFT_ISSUE_TILE16(k16base, jb_next, (u * NW >= 8 ? THRIFT_K16OFF() ^ 64u : THRIFT_K16OFF()),
                            lds0 + (uint32_t)THRIFT_TILE_BUFFER(kbuf_next));
      }
      THRIFT_MASK(jb)
      v16f s[2];
      if (use) scores_16<T>(lds + THRIFT_TILE_BUFFER(kbuf), lane, qf, s);
      if (p1) vm_wait<C16>();                           // V(b); K(b+1) may still be on its way
      else vm_wait<0>();
      lds_barrier();                                    // V(b) complete; everyone has its scores, K(b)'s buffer is free
      if (p1) { THRIFT_ISSUE_TILE16(v16base, jb_next, THRIFT_V16OFF(), lds0 + (uint32_t)THRIFT_TILE_BUFFER(kbuf)); }
      if (use) {
        float alpha;
        uint32_t pb;
        const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
        rescale(o, grew, alpha);
        pv_16<T, true>(lds + THRIFT_TILE_BUFFER(vbuf), lane, s, o);
      }
      kbuf = kbuf_next;
      jb = jb_next;
    }
#undef THRIFT_TILE_BUFFER
  } else {
  // prologue: block 0 on its way
  if (vis > 0) {
    if (!all(n0, 0)) THRIFT_ISSUE4(0);
    if (some(n0, 0)) {
      THRIFT_ISSUE_K16(0);
      THRIFT_ISSUE_V16(0);
    }
  }
  // What every wavefront does between its scores and its softmax, and in front of P.V, where some list has promoted block j (P0),
  // whichever path the wavefront itself takes; P1: block j+1 too.
#define THRIFT_BEHIND_SCORES(P0, P1)                                                                           \
  if ((P0) && (P1)) {                                   /* the K buffer is free once every wavefront has its scores */ \
    lds_barrier();                                                                                             \
    THRIFT_ISSUE_K16(j + 1);                                                                                   \
  }
#define THRIFT_BEFORE_PV(P0, P1)                                                                               \
  if ((P0) && late_v) {                                 /* this block's V tile was issued in this step */      \
    if (P1) vm_wait<C16>();                                                                                    \
    else vm_wait<0>();                                                                                         \
    lds_barrier();                                                                                             \
  }
  int j = 0;
  if constexpr (NL == 1) {
  // The walk alternates between runs of 4-bit blocks (tight loop: only the scaled-FP4 path, accumulators
  // updated in place) and single promoted blocks.
  while (j < vis_wave) {
    drop_stale(j);
    const int run_end = min(vis_wave, n0[0]);
    for (; j < run_end; ++j) {
      take_turn(j);
      THRIFT_SYNC()
      THRIFT_ISSUE(j, false, j + 1 == n0[0], j + 1 == n0[0])
      THRIFT_MASK(j)
      const unsigned char* slot = lds + kLdsRing + (j & 1) * kLdsBytes4;
      v16f s[2];
      float alpha;
      uint32_t pb;
      scores_fp4(slot, lane, qf4, qsc, s);
      const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
      rescale(o, grew, alpha);
      pv_fp4(slot, lane, s, pb, o);
      late_v = false;
    }
    if (j < vis_wave) {                                 // j == n0[0]: a promoted block
      const bool p1 = j + 1 == n1[0] && j + 1 < vis;
      v16f s[2];
      float alpha;
      uint32_t pb;
      THRIFT_SYNC()
      THRIFT_ISSUE(j, true, p1, j + 1 == n1[0])
      if (late_v) THRIFT_ISSUE_V16(j);
      THRIFT_MASK(j)
      {
        v8s qf[8];
        THRIFT_LOAD_Q16(qf)
        scores_16<T>(lds + kLdsK16, lane, qf, s);
      }
      THRIFT_BEHIND_SCORES(true, p1)
      const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
      rescale(o, grew, alpha);
      THRIFT_BEFORE_PV(true, p1)
      pv_16<T, true>(lds + kLdsV16, lane, s, o);
      next_promoted(0);
      late_v = p1;
      ++j;
    }
  }
  }
  // Two lists: every block in one loop, whose wavefronts take the path of their own list.  One list: blocks that later wavefronts
  // still need, staged only.
  for (; j < vis; ++j) {
    drop_stale(j);
    int x[NL];
    behind(j, x);
    const bool p0 = some(n0, j), p1 = some(x, j + 1) && j + 1 < vis;
    const bool use = NL > 1 && j < vis_wave, own16 = mine(n0, j);
    if constexpr (NL > 1) take_turn(j);
    THRIFT_SYNC()
    THRIFT_ISSUE(j, p0, p1, all(x, j + 1))
    if (p0 && late_v) THRIFT_ISSUE_V16(j);
    THRIFT_MASK(j)
    if (use && !own16) {
      const unsigned char* slot = lds + kLdsRing + (j & 1) * kLdsBytes4;
      v16f s[2];
      float alpha;
      uint32_t pb;
      scores_fp4(slot, lane, qf4, qsc, s);
      THRIFT_BEHIND_SCORES(p0, p1)
      const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
      rescale(o, grew, alpha);
      THRIFT_BEFORE_PV(p0, p1)
      pv_fp4(slot, lane, s, pb, o);
    }
    if (use && own16) {
      v16f s[2];
      float alpha;
      uint32_t pb;
      {
        v8s qf[8];
        THRIFT_LOAD_Q16(qf)
        scores_16<T>(lds + kLdsK16, lane, qf, s);
      }
      THRIFT_BEHIND_SCORES(true, p1)
      const bool grew = softmax_update(s, lane, mask, n_valid, c, st, alpha, pb);
      rescale(o, grew, alpha);
      THRIFT_BEFORE_PV(true, p1)
      pv_16<T, true>(lds + kLdsV16, lane, s, o);
    }
    if (!use) {
      THRIFT_BEHIND_SCORES(p0, p1)
      THRIFT_BEFORE_PV(p0, p1)
    }
    advance(j);
    late_v = p0 && p1;
  }
  }
  vm_wait<0>();
#undef THRIFT_SYNC
#undef THRIFT_LOAD_Q16
#undef THRIFT_LOAD_Q16_ROW
#undef THRIFT_ISSUE
#undef THRIFT_BEHIND_SCORES
#undef THRIFT_BEFORE_PV
#undef THRIFT_MASK
#undef THRIFT_ISSUE4
#undef THRIFT_ISSUE4_SLOT
#undef THRIFT_ISSUE_V16
#undef THRIFT_ISSUE_K16
#undef THRIFT_ISSUE_TILE16
#undef THRIFT_V16OFF
#undef THRIFT_K16OFF
#undef THRIFT_CLAMP_ROWS

  // ---- epilogue (Alg. 1 step 21): O / l; accumulator i of tile n is channel 32n + 8(i/4) + 4*half + i%4 ----
  const float l = st.l + other_half(st.l);
  const float inv = l > 0.f ? 1.0f / l : 0.f;
  THRIFT_ROW_AGAIN(row_e)
  const bool row_ok = row_e < Nq;
  const int lrow_again = min(row_e, Nq - 1);
  const size_t orow = (qh * Nq + lrow_again) * kD;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int q4i = 0; q4i < 4; ++q4i) {
      const int ch = 32 * n + 8 * q4i + 4 * half;
      if (!row_ok) continue;
      const float x0 = o[n][4 * q4i] * inv, x1 = o[n][4 * q4i + 1] * inv, x2 = o[n][4 * q4i + 2] * inv, x3 = o[n][4 * q4i + 3] * inv;
      store_out4(a.out, a.out_dt, orow + ch, x0, x1, x2, x3);
    }
  if (a.lse != nullptr && half == 0 && row_ok) a.lse[qh * Nq + lrow_again] = st.m * a.scale + __logf(l);
#undef THRIFT_ROW_AGAIN
}

// The second bound is wavefronts per SIMD: three workgroups of four per CU, two (wide), or three workgroups of two, which the SIMDs
// hold as one and a half each and which may have the registers of two.
template <typename T, int NW, int NL, int ORDER, int WIDE, int TURNS>
__global__ void __launch_bounds__(NW * 64, WIDE || NW == 2 ? 2 : 3) prefill_kernel(PrefillArgs a) {
  __shared__ __align__(1024) unsigned char lds[WIDE ? kLdsPrefillWide : kLdsPrefill];
  prefill_item<T, NW, NL, ORDER, WIDE, TURNS>(a, lds, blockIdx.x);
}

// The same items from a persistent launch: as many workgroups as the chip holds at once, each taking the next item
// (heaviest first, like the launch order above) from a device counter until none is left.  An item of this kernel
// leaves no DMA in flight and the barriers below keep the LDS of one item apart from the next.
static __device__ unsigned int prefill_next_item[64];       // one counter per launch in flight would be needed: see launch_prefill

__global__ void prefill_reset_counter_kernel() { prefill_next_item[0] = 0u; }

template <typename T, int ORDER>
__global__ void __launch_bounds__(256, 3) prefill_persistent_kernel(PrefillArgs a, unsigned items) {
  __shared__ __align__(1024) unsigned char lds[kLdsPrefill];
  __shared__ unsigned next;
  // the workgroup's position on its XCD decides nothing here: items keep the XCD of their KV head only while the
  // counter hands consecutive items to consecutive workgroups, which it does at the start and loses later
  for (;;) {
    if (threadIdx.x == 0) next = atomicAdd(&prefill_next_item[0], 1u);
    __syncthreads();
    const unsigned work = next;
    __syncthreads();
    if (work >= items) break;
    prefill_item<T, 4, 1, ORDER, 0, 0>(a, lds, work);
  }
}

// The wide schedule pays for itself once promoted blocks are frequent: their 32 KiB of 16-bit tiles then
// arrive a whole step ahead instead of half a step, at the price of two instead of three workgroups per CU
// for the 4-bit blocks.  The per-row list length bounds the promoted share from above.
static bool wide_schedule(const PrefillArgs& a) {
  if (a.Bq != 128 || a.tile_order == 1 || a.tile_order == 2) return false;
  if (a.tile_order == 3) return true;
  const long Tk = (a.N + kBk - 1) / kBk;
  return (long)a.kmax * 100L >= Tk * (long)kWidePercent;
}

// Longest query blocks of ALL (sequence, KV head) units first, instead of one unit of an XCD after the other.  A causal row is
// up to 2 N / Bq times as long as the first one, and with several units per XCD the long rows of the last unit started when
// the chip was about to run empty: 142 -> 118 us for 2 x 4096 tokens, 16/16 heads, 387 -> 340 us for 2 x 8192, 208 -> 189 us
// for 2 x 4096 with 32/8, 1252 -> 1079 us for 32768 with 8/2.  In grids of more than eight rounds of three workgroups per CU
// the ends weigh little and the units' K/V streams want the L2 one after the other: 1210 / 1260 us for 2 x 8192, 64/8 heads.
static bool interleaved_units(const PrefillArgs& a, unsigned grid) { return a.causal && grid <= 8u * 3u * kCus; }

// Query blocks of 64 rows one to a workgroup of two wavefronts instead of two to one of four.  With the LDS of a CU for three
// workgroups, two wavefronts each are one and a half per SIMD instead of three, and every block is staged for half the rows; but a row's
// walk takes only its own list, in fewer instructions per block, and what counts in a grid of one round is the length of that walk.  The
// second round of causal rows is the short ones, and the more blocks are promoted the longer the second list makes the walk.  Time
// of one / of two query blocks per workgroup, ascending and in the order of Sec. 3.3 (64-row query blocks in the grid):
//   causal, from the first key on            0 %          5 %          10 %         25 %         100 %
//      768   1500 tokens, 32/8           0.91 0.98    0.89 0.91    0.87 0.87    0.83 0.75    0.84 0.84
//      960   1920, 32/8                  0.97 1.03    0.94 1.02    0.92 0.97
//     1024   1000, 64/8                  0.99 1.04    1.00 1.04    0.96 0.97
//     1152   1100, 64/8                               1.04 1.06    1.00 1.01    0.93 0.85    0.89 0.90
//     1152   2 x 549, 64/8 (one block)                1.11 1.06    the same     1.05 1.01    1.00 0.92
//     1136   4500, 16/16                 0.97 1.06    0.92 0.99    0.89 0.93    0.82 0.80    0.84 0.71
//     1280   2560, 32/8                                            0.98 0.98    0.90 0.83    0.84 0.91
//     1376   2700, 32/8                                            1.02 1.01    0.95 0.87    0.87 0.81
//     1504   3000, 32/8                  1.15 1.23    1.11 1.14    1.07 1.07    1.00 0.92    0.92 0.83
//     1600   3200, 32/8                                            1.12 1.11    1.01 0.96    0.92 0.98
//     2528   5000, 32/8                  1.18 1.28    1.14 1.23    1.11 1.16    1.11 1.05    1.17 1.09
//   no mask, or a chunk on 16384
//      416   chunk of 800, 32/8          1.05 1.21    1.00 1.07    0.96 0.98    0.86 0.77    0.86 0.76
//      480   1900, 16/16                 1.09 1.17    1.06 1.09    1.03 1.04
//      544   chunk of 1088, 32/8         0.88 0.93    0.85 0.87    0.83 0.80
//      768   1500, 32/8                  0.94 0.96    0.91 0.92    0.90 0.88    0.86 0.79    0.87 0.89
//      832   1664, 32/8                                            1.23 1.22    1.18 1.09    1.42 1.29
//     1216   chunk of 2400, 32/8         1.45 1.46    1.41 1.31    1.38 1.26    1.30 1.10    1.27 1.25
static bool one_query_block(const PrefillArgs& a) {
  const long blocks = (long)a.B * a.Hq * ((a.Nq + 63) / 64), Tk = (a.N + kBk - 1) / kBk;
  const long percent = (a.kmax * 100L - 50) / Tk;                  // budgets are rounded up to whole blocks: of a short row that is much
  if (a.causal && a.q_off == 0) return blocks <= (percent >= 20 ? 6L : percent >= 8 ? 5L : 3L) * kCus;
  return blocks <= 3L * kCus && (blocks > 2L * kCus || percent >= kWidePercent);         // two to a workgroup are one per CU below that
}

// A grid that the chip holds at once: workgroup n goes to the CU of workgroup n - 256 (read back from the hardware id register), so in
// descending order the same CU gets the longest row of each third, 47 + 31 + 15 key blocks of 3001 tokens, and another one 33 + 17 + 1.  With the
// second third turned round they are 47 + 17 + 15 and 33 + 31 + 1.  Descending / folded: 69.7 / 66.6 us for 3001 tokens, 32/8 heads
// (71.5 / 66.1 in the order of Sec. 3.3), 64.6 / 61.4 for 2 x 2500, 16/16, 47.7 / 45.3 for 1500, 64/8; 49.2 / 48.6 for 2048, 32/8 (two workgroups per CU, of
// which the longer one alone takes the time).  The last third turned round as well is no better (66.4, 67.1), alone worse (68.5, 69.2).
// In the wide schedule a CU holds two and the last third takes the places that are free first, those of the second third's short
// rows: 54.5 / 52.9 us for 1500 tokens, 64/8, 25 %, 78.3 / 77.4 for 3000, 32/8, 53.5 / 53.1 for 2100, 67.3 / 68.5 for 2700, equal at 2500
// and at 100 % (105.2 / 105.1 for 2 x 2900, 16/16, 92.4 / 92.6 for 2700).
static bool folded(const PrefillArgs& a, unsigned grid) { return a.interleave && grid <= 3u * kCus; }

// One round of workgroups whose rows are equally long (no mask, or a chunk behind cached tokens).  A SIMD prefers its oldest wavefront, so that
// the first workgroup of a CU ended when the second was at 60 % (467 and 605 us of a chunk of 2048 tokens on 30720), and the rest ran with
// one wavefront per SIMD, which uses half of its vector rate.  With turns they end together.  Without / with: 592 / 575 us for that
// chunk, 814 / 790 for one of 3072, 780 / 744 for 2500; 102.2 / 97.6 for 3001 tokens without a mask, 62.6 / 60.7 for 2048; with query blocks of 64 rows, two to a
// workgroup, in ascending order 109.9 / 103.2 for 3001 without a mask, 624 / 604 for the chunk of 2048.  In causal prompts the
// first workgroup of a CU is the longest and should run ahead (68.3 / 71.6 for 3001 tokens), and in larger grids the next workgroup fills the
// place that is free: 239 / 265 for 5000 tokens without a mask, 1092 / 1134 for a chunk of 4096; two workgroups per CU (wide): 652 / 634 for the
// chunk of 2048 at 25 %, 123.9 / 127.2 for 3001 tokens without a mask, one and a half rounds.
// The priority holds against every wavefront of the SIMD.  Decode steps on another stream beside chunks of 32/8 heads one after the other,
// without / with turns: where a step finds room it takes as long (34 / 34 us median for one sequence of 4096 beside chunks of 3072, 70.7 / 68.5 for 16 x
// 4096-8192; 39.2 / 38.9 and 86 / 96 beside chunks of 3000 with 16/16 heads, which leave room for most), but the workgroups of a CU leave their places
// together at the chunk's end and not one at three quarters of it: steps that have to wait for one come to 109 / 142 us in the mean (one
// of 4096 beside 3072), 150 / 182 (one of 32768 beside 2048), and beside chunks of 2048 to one per chunk (3.9 / 1.7 steps of 4096 tokens per
// ms); 211 / 224 (16 x 4096-8192), 419 / 438 (8 x 16384-32768, 64/8).  The chunks themselves take 612 / 585, 693 / 678, 725 / 690 and 782 / 762 us there.
static bool take_turns(const PrefillArgs& a, unsigned grid) {
  return (!a.causal || a.q_off > 0) && grid > 1u * kCus && grid <= (wide_schedule(a) ? 2u : 3u) * kCus;
}

void launch_prefill(const PrefillArgs& args, hipStream_t st) {
  if (launch_prefill_split(args, st)) return;
  PrefillArgs a = args;
  const int rows = a.Bq == 64 && one_query_block(a) ? 64 : 128;    // of a workgroup
  const unsigned grid = (unsigned)((long)a.B * a.Hq * ((a.Nq + rows - 1) / rows));
  a.interleave = interleaved_units(a, grid);
  a.fold = folded(a, grid);
  if (a.tile_order == 4 && a.Bq == 128) {
    // persistent launch of the Sec. 3.3 order: three workgroups per CU.  One counter per device: two such launches
    // must not overlap on a device.  The counter is cleared by a kernel (a memset node misbehaves under graph capture).
    int dev = 0, cus = kCus;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const unsigned resident = (unsigned)min((long)grid, 3L * cus);
    a.fold = 0;                                          // its workgroups take the items as they come
    prefill_reset_counter_kernel<<<dim3(1), dim3(1), 0, st>>>();
    if (a.dt == THRIFT_F16) prefill_persistent_kernel<F16, 1><<<dim3(resident), dim3(256), 0, st>>>(a, grid);
    else prefill_persistent_kernel<BF16, 1><<<dim3(resident), dim3(256), 0, st>>>(a, grid);
    return;
  }
  auto launch = [&](auto turns) {
    constexpr int TURNS = decltype(turns)::value;
    const bool order1 = a.tile_order == 1 || a.tile_order == 4, f16 = a.dt == THRIFT_F16;
#define THRIFT_LAUNCH(NW, NL, ORDER, WIDE)                                                                     \
  do {                                                                                                         \
    if (f16) prefill_kernel<F16, NW, NL, ORDER, WIDE, TURNS><<<dim3(grid), dim3(NW * 64), 0, st>>>(a);         \
    else prefill_kernel<BF16, NW, NL, ORDER, WIDE, TURNS><<<dim3(grid), dim3(NW * 64), 0, st>>>(a);            \
  } while (0)
    if (wide_schedule(a)) THRIFT_LAUNCH(4, 1, 0, 1);
    else if (a.Bq == 128 && order1) THRIFT_LAUNCH(4, 1, 1, 0);
    else if (a.Bq == 128) THRIFT_LAUNCH(4, 1, 0, 0);
    else if (rows == 128 && order1) THRIFT_LAUNCH(4, 2, 1, 0);
    else if (rows == 128) THRIFT_LAUNCH(4, 2, 0, 0);
    else if (order1) THRIFT_LAUNCH(2, 1, 1, 0);
    else THRIFT_LAUNCH(2, 1, 0, 0);
#undef THRIFT_LAUNCH
  };
  if (take_turns(a, grid)) launch(std::integral_constant<int, 1>{});
  else launch(std::integral_constant<int, 0>{});
}

}  // namespace thrift
