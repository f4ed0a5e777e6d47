// attn.hip -- ragged, packed verify attention over a paged bf16 GQA KV cache
// for gfx950 (MI355X).
//
// What it computes (Sec. III-D, Eq. (16); packing of Eqs. (10)-(11)): every
// valid row j < k_i of request i reads packed row cu[i]+j and attends, with
// request-local causal masking, to keys 0 .. ctx_i + j of that request.
//
// How (MI355X design; the paper's A100 kernel is a 16-row tile per
// (request, head) on a grid of requests x heads, Sec. III-B):
//  * Tiles follow the live rows.  The G query heads that share a KV head are
//    stacked with the block rows into R = G*k_i live rows (row r -> block row
//    r / G, head r % G), cut into ceil(R/16) MFMA row tiles, so one K/V read
//    serves all G heads (GQA sharing) and a request never pays for rows it
//    does not have (Eq. (2)'s padding applies per 16-row tile, not per 128).
//  * Stream-K work split.  Each (request, KV head) pair is a segment of
//    ceil32(ctx_i + k_i) keys; the segments are laid end to end, each
//    after a lead-in of six blocks that stands for the cost of starting a
//    piece on it, and a persistent grid, sized to the workgroups the GPU
//    holds at once, gives every workgroup one contiguous share of that
//    space (streaming plus piece starts), equal up to a small skew by grid
//    index parity for the XCDs' unequal streaming rates.  A workgroup walks the
//    segments its share touches; a segment it covers whole is written as
//    bf16 directly, a segment cut at a share boundary leaves an fp32 partial
//    (O, m, l) that the combine kernel merges in workgroup order.  Ragged
//    contexts cost no idle workgroups, and there are at most two partials
//    per workgroup.  Results depend only on the request's own data and the
//    batch's total work (the share size), and merge in a fixed order, so
//    they are deterministic.  Small batches, whose even share would fall
//    below eight blocks, instead cut every segment into equal block-aligned
//    pieces, one per workgroup, so that no workgroup straddles two segments.
//  * K/V stream through an LDS ring of three 32-key stages.  Each wave
//    loads one 4 KiB tile per stage (one page's K or V) into registers
//    three stages ahead, as four contiguous 1 KiB loads from a scalar page
//    address, and writes it to the ring when its stage comes up; on gfx950
//    this sustains more bandwidth than LDS-direct loads.  Page ids are
//    staged in LDS per piece.
//  * Transposed scores: S^T = K Q^T and O^T = V^T P^T with
//    v_mfma_f32_16x16x32_bf16.  The score tile comes out with one query row
//    per lane column, which after two row-swap permutes a register pair is
//    exactly the B-operand layout the PV product needs.  Each weight enters
//    PV as a hi + lo pair of bf16 values (two MFMAs per output tile), so the
//    weights carry about 2^-17 of their value and the output's own bf16
//    rounding dominates the error.
//  * Lazy rescaling: the running maximum only moves (and the accumulators
//    are only rescaled) when a key's score exceeds it by more than a
//    factor 2^8, which keeps the weights below 2^8.  It is kept an integer,
//    so rescales and merge weights are exact powers of two.
//  * Waves of a workgroup split the dims when a request has one or two row
//    tiles; beyond that each wave owns one to four tiles, so that every piece
//    reads its K and V once: four waves hold the eight tiles of eight query
//    heads to a KV head and a full block, eight waves, or at D = 64 also four, the
//    sixteen of G = 16.  Only many short segments at G = 16, D = 128, take two
//    passes of K and V, from cache.
//  * The workgroups placed after the first on a CU run at raised wave priority
//    over half of their share, so that a CU's workgroups finish together.
//
// What bounds it, and what it measured (MI355X, split + combine kernels, us a
// call; before: each wave held one tile, so that more than four took a pass of
// K and V for every four, and a step's softmax took 132 vector instructions to
// a tile where it now takes about 60):
//   B=32, 32 query / 8 KV heads, contexts to 8K (0.6 GB): HBM; 105.7 -> 104.1
//     (less than single runs differ by), 5.8 TB/s
//   B=32, 64 / 8 heads, lengths about 8, contexts to 16K (1.2 GB): HBM, with
//     the vector units close behind; 343 -> 228, 5.3 TB/s
//   B=24, 32 / 2 heads, full blocks, contexts to 6K: the matrix and vector
//     units (16 tiles to a key), then 33 MB of partials; 104 -> 59
//   B=32, head_dim 64, contexts to 8K (0.3 GB): HBM; 60.7 -> 58.0, 5.2 TB/s
//   B=8, full blocks, contexts to 2K (40 MB): the chain from launch to the
//     last block; 23.4 -> 20.6
//   B=1, full block, context 700 (3 MB): the same; 16.9 -> 13.2
#include "dsv_internal.h"

#include <math.h>

namespace dsv {
namespace {

// Combine kernel: 1024-thread workgroups (32 rows at D = 128) need a quarter
// of the workgroups that 256 threads do, most of which exit at once; measured
// 0.6 us faster at B=32 with contexts up to 8K (Qwen3-8B attention shape).
constexpr int kCombThreads = 1024;
constexpr int kBlockKeys = kAttnBlockKeys;  // keys per inner step (two pages)
// Smallest stream-K share: with little work (short contexts, few requests)
// eight blocks per workgroup beat spreading it over every resident
// workgroup -- fewer cut segments, so less partial traffic and combine work,
// and a longer pipeline per workgroup.
constexpr int kMinShare = 8 * kBlockKeys;
// Stream-K lead-in: every segment with keys counts kLeadKeys more in the
// linear work space than it holds, the cost of starting a piece on it
// (metadata, page ids, query rows, the ring's first blocks), so that equal
// shares are equal in streaming plus piece starts.  A multiple of the block;
// six blocks measured best across shapes (two to eight were compared).
constexpr int kLeadKeys = kAttnLeadKeys;
// Wave priority.  At D = 128 the persistent grid holds two workgroups per CU
// (one at G = 16), and the one the dispatcher places second (grid index >= number
// of CUs) loses instruction arbitration to the older first one: with equal
// shares and no priorities the first ended at 66 us and the second at 91 (B=32,
// contexts up to 8K).  Its waves therefore run at raised priority until kBoostPct
// percent of its share is done, then at the default, and both end at about 90 us.
// Priority changes no arithmetic.  Drop points, B=32 contexts to 8K / eight
// query heads to a KV head and contexts to 16K, us a call: 50% 104.2 / 226.7,
// 65% 104.4 / 228.8, 80% 106.1 / 229.6, none 113 / 244.
// At D = 64, with two to four workgroups to a CU, all but the first are raised: 8 KV
// heads, B=32 contexts to 8K, groups of 1 / 4 / 8 / 16, us a call: 56.4 / 60.3 /
// 66.3 / 108.4, none raised 57.7 / 61.9 / 70.1 / 116.1, the last alone 56.5 / 60.7 /
// 68.3 / 108.9.
constexpr int kBoostPct = 50;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
  return __builtin_bit_cast(bf16x8, v);
}

// Two bf16 -> one uint32 (low half first), round to nearest even: one
// v_cvt_pk_bf16_f32 (two scalar conversions compile to four instructions).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

__device__ __forceinline__ int round_up_block(int x) {
  return (x + kBlockKeys - 1) / kBlockKeys * kBlockKeys;
}

// Request-level metadata after the cheap device-side checks.  `seg` is the
// request's segment length in keys (ctx + k rounded up to 32), 0 for a
// sentinel or a request whose metadata breaks the contract.
struct ReqMeta {
  int q0, k, ctx, len, seg;
};

__device__ __forceinline__ int segment_of(const AttnParams &p, int q0, int q1, int ctx) {
  const int k = q1 - q0;
  const bool ok = k > 0 && k <= kMaxQlen && q0 >= 0 && q1 <= p.cap && ctx >= 0 &&
                  ctx + k <= p.max_kv_len;
  return ok ? round_up_block(ctx + k) : 0;
}

// Per-thread (non-uniform) segment length of request i.
__device__ __forceinline__ int segment_len(const AttnParams &p, int i) {
  return segment_of(p, p.cu[i], p.cu[i + 1], p.ctx[i]);
}

// Uniform metadata of request i: read with vector loads (the kernel writes
// global memory, so the compiler will not use the scalar cache) and then
// declared uniform.
__device__ __forceinline__ ReqMeta load_req(const AttnParams &p, int i) {
  ReqMeta r;
  r.q0 = __builtin_amdgcn_readfirstlane(p.cu[i]);
  const int q1 = __builtin_amdgcn_readfirstlane(p.cu[i + 1]);
  r.ctx = __builtin_amdgcn_readfirstlane(p.ctx[i]);
  r.k = q1 - r.q0;
  r.len = r.ctx + r.k;
  r.seg = segment_of(p, r.q0, q1, r.ctx);
  return r;
}

// -------------------------------------------------------------------- steps
// The key loop works in steps of one 32-key block, a pair of pages whose tiles
// hold exactly the MFMA operands:
//  K: the 1 KiB chunk c of a page's K tile is the A operand of the score
//     MFMA over dims 32c .. 32c+31, lane l holding slot l & 15.
//  V: lane (kq, m) of d block u takes the 16 bytes of dim 16u+m that hold
//     slots 8*(kq>>1) .. +7 of page kq & 1.
constexpr int kSubKeys = 8192;              // keys whose page ids are staged at a time
constexpr int kSubPages = kSubKeys / kPage;

template <int D>
struct KRegs {
  u32x4 x[2][D / 32];  // [page][chunk]
};
template <int NE>
struct VRegs {
  u32x4 x[NE];  // [d block]
};

// Maximum / sum over the four lanes that hold one query row (lanes n, n+16,
// n+32, n+48), with the gfx950 row-swap permutes.
__device__ __forceinline__ float row_max4(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Sum over the same four lanes.  Each swap hands every lane the pair in the
// same order, so the four lanes end with bitwise equal sums.
__device__ __forceinline__ float row_sum4(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The running maximum is only raised when a block's maximum exceeds it by
// more than this (base-2 units): weights then stay below 2^8, and the
// accumulators are rescaled only on such a jump instead of every block.
// The maximum is kept an integer (the block maximum rounded up), so every
// rescale factor and every merge weight, in the workgroup and in the combine,
// is an exact power of two: where a segment is cut, or which rows share its
// tile, moves a row's weights and sums by powers of two only, and its result
// changes only through fp32 summation order.
constexpr float kRescaleSlack = 8.f;
// Running maximum of a row that has seen no key yet: finite, so that no
// difference of two of them is a NaN.
constexpr float kNoMax = -3.402823466e38f;

// Online-softmax state of one wave, for TW row tiles and NE d blocks.  A lane
// holds one query row (lane & 15) of each tile: its running maximum, its own
// lane's share of the sum of the weights (the row's four lanes are added at
// the end), and for each d block u the outputs of dims 16u + 4*(lane>>4) +
// [0..3] from the wave's first d block on.
template <int TW, int NE>
struct RowState {
  float m[TW];
  float l[TW];
  f32x4 o[TW][NE];
};

// This workgroup's share of the flattened work: [start, end) in units of
// keys over the segments laid end to end (request-major, then KV head).
struct Share {
  int start, end;
  int i, g, off;  // segment and virtual offset where `start` falls
  int lead;       // keys of lead-in per segment: kLeadKeys (stream-K) or 0
  ReqMeta first;  // request i's metadata, as read by the plan
};

// Small batches.  When the even share falls to the minimum, each segment is
// instead cut into pieces of at most `cap` keys, as equal as whole blocks
// allow, one piece per workgroup: no workgroup then pays for a second piece
// (its metadata, page ids and pipeline refill), which at this size is a
// large part of the kernel.  The cap leaves at most one piece per CU -- a
// second workgroup on a CU shares its MFMA and LDS with the first and finishes
// last.  The smallest batches take the smallest cap that does so with at most
// kMaxMerge pieces to a segment, which the combine kernel loads in one round trip
// (one request, 716 keys, four layers: 63.1 -> 58.3 us with three blocks instead
// of eight; 16 pieces to a segment took 70.6 us); the others the smallest of 8 to
// 12 blocks that fits, else eight, if the pieces fit the grid.
//   A cut costs the combine's round trip and the partials, written and read, so
// cut_rule bounds the smallest caps by the elements of a segment's partial: the
// least blocks of a piece, the blocks up to which a segment stays whole, and the
// pieces, in sixteenths of the CUs.  us a call, D = 128, S segments of b blocks, r
// rows each: S=64, b=3, r=16 cut 10.4, whole 9.8; b=4 cut 10.2, whole 10.9; b=5, r=64
// in 192 pieces 14.4, in 128 12.5; S=96, b=4, r=256 in 192 pieces 31.7, whole 21.5.
// Of caps from two to twelve blocks, over 864 shapes, the rule's is 1.8% off the best
// in the mean and 27% at most; with the first line for all it was 4.7% and 68%.
// Piece q of n of a `seg`-key segment starts at piece_begin(seg, n, q).
constexpr int kNumPieceCaps = 5;
__device__ __forceinline__ int piece_cap(int c) { return (8 + c) * kBlockKeys; }  // 8..12 blocks
constexpr int kMaxMerge = 8;
struct CutRule {
  int min_blocks, whole_blocks, cu_sixteenths;
};
// Of `total` partial elements over `segs` segments (no division: this is on the way
// to the first load of every workgroup).
__device__ __forceinline__ CutRule cut_rule(float total, float segs) {
  if (total <= 2048.f * segs) return {2, 3, 16};
  if (total <= 4096.f * segs) return {3, 4, 12};
  if (total <= 8192.f * segs) return {3, 5, 10};
  return {3, 5, 5};
}
__device__ __forceinline__ int seg_pieces(int seg, int cap) { return (seg + cap - 1) / cap; }
__device__ __forceinline__ int piece_begin(int seg, int n, int q) {
  return (int)((long long)(seg / kBlockKeys) * q / n) * kBlockKeys;
}

// Stream-K shares alternate in size with the workgroup's grid index.  The
// dispatcher places workgroup b on XCD b mod 8, and with equal shares the
// workgroups on the odd XCDs finished 6-10 us after those on the even ones
// in every clocked launch of the Qwen3-8B shape at B=32, contexts up to 8K,
// while the shader clocks of all eight XCDs agreed within 2%.  Even
// workgroups therefore take kSkewPct percent more than the mean share and
// odd ones as much less (whole blocks).
constexpr int kSkewPct = 6;
__device__ __forceinline__ int share_skew(int share) {
  return (int)((long long)share * kSkewPct / 100) / kBlockKeys * kBlockKeys;
}
// First virtual key of workgroup b's share.
__device__ __forceinline__ int share_begin(int b, int share, int skew) {
  return b * share + (b & 1) * skew;
}
// The workgroup whose share holds virtual key pos.
__device__ __forceinline__ int share_owner(int pos, int share, int skew) {
  const int pair = pos / (2 * share);
  return 2 * pair + (pos - pair * 2 * share >= share + skew ? 1 : 0);
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP row shifts and
// row broadcasts (lanes without a source add 0): six VALU steps, where a
// shuffle-based scan would take six LDS permutes.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_src(int v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, kRowMask, 0xf, false);
}
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += dpp_src<0x111, 0xf>(v);  // row_shr:1
  v += dpp_src<0x112, 0xf>(v);  // row_shr:2
  v += dpp_src<0x114, 0xf>(v);  // row_shr:4
  v += dpp_src<0x118, 0xf>(v);  // row_shr:8
  v += dpp_src<0x142, 0xa>(v);  // row_bcast:15
  v += dpp_src<0x143, 0xc>(v);  // row_bcast:31
  return v;
}

// Largest of the wave's values (not negative), in lane 63.
__device__ __forceinline__ int wave_max(int v) {
  v = max(v, dpp_src<0x111, 0xf>(v));
  v = max(v, dpp_src<0x112, 0xf>(v));
  v = max(v, dpp_src<0x114, 0xf>(v));
  v = max(v, dpp_src<0x118, 0xf>(v));
  v = max(v, dpp_src<0x142, 0xa>(v));
  v = max(v, dpp_src<0x143, 0xc>(v));
  return v;
}

// Block-wide exclusive scan of one value per thread: the wave scan, then the
// wave totals through LDS (`tot` receives the block total).
template <int NW>
__device__ __forceinline__ int block_excl_scan(int v, int *lds_tot, int &tot) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int incl = wave_incl_scan(v);
  if (lane == kWave - 1) lds_tot[wave] = incl;
  __syncthreads();
  int before = 0;
  tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    before += w < wave ? lds_tot[w] : 0;
    tot += lds_tot[w];
  }
  return before + incl - v;
}

// Computes the share with block-wide scans over the requests' segment
// lengths (each thread owns a contiguous run of requests): a stream-K share
// of the flattened work, or, for small batches, one piece of one segment.
// Workgroup 0 also publishes the per-request prefixes and the plan for the
// combine kernel.  LDS use: lds[0..2*NW) scan totals, then the located
// share.
template <int D, int NW>
__device__ Share plan_share(const AttnParams &p, int *lds) {
  constexpr int kThreads = NW * kWave;
  const int B = p.num_reqs, tid = threadIdx.x;
  int live = p.cu[B];  // packed rows, in flight with the requests' metadata
  const int per = (B + kThreads - 1) / kThreads;
  const int lo = min(B, tid * per), hi = min(B, lo + per);
  int sum = 0;
  // with one request per thread (B <= 256) its metadata stays in registers
  // for the locate step below
  int q0 = 0, q1 = 0, cx = 0;
  if (per == 1) {
    if (lo < hi) {
      q0 = p.cu[lo];
      q1 = p.cu[lo + 1];
      cx = p.ctx[lo];
      sum = segment_of(p, q0, q1, cx);
    }
  } else {
#pragma unroll 4
    for (int i = lo; i < hi; ++i) sum += segment_len(p, i);
  }
  asm volatile("" : "+v"(live));  // or its load is sunk to its use, a round trip later
  int total;
  const int excl = block_excl_scan<NW>(sum, lds, total);  // keys before my requests
  int *loc = lds + 2 * NW;  // located share: i, g, off, q0, q1, ctx, start, end
  const int work = total * p.hkv;
  int share = (work + (int)gridDim.x - 1) / (int)gridDim.x;
  share = max(kMinShare, round_up_block(share));
  // Small batch: the even share is at the minimum.  Count the segment pieces
  // under every candidate cap (block totals only: one wave sum per cap, one
  // barrier) and pick the cap; every workgroup computes the same choice.
  int cap = 0;
  if (share == kMinShare) {
    // pieces under each cap and, last, segments; they fit 16 bits, since a
    // batch at the minimum share has at most eight blocks for every workgroup
    // of the grid
    constexpr int kPacked = kNumPieceCaps / 2 + 1;
    static_assert(kNumPieceCaps % 2 == 1, "the segments take the free half");
    uint32_t cnt[kPacked] = {};
    int longest = 0;
    for (int i = lo; i < hi; ++i) {
      const int seg = per == 1 ? sum : segment_len(p, i);
#pragma unroll
      for (int c = 0; c < kNumPieceCaps; ++c)
        cnt[c / 2] += (uint32_t)seg_pieces(seg, piece_cap(c)) << (16 * (c % 2));
      cnt[kPacked - 1] += seg > 0 ? 1u << 16 : 0u;
      longest = max(longest, seg);
    }
    uint32_t *red = reinterpret_cast<uint32_t *>(loc + 8);  // [kPacked + 1][NW]
    const int lane = tid % kWave, wave = tid / kWave;
#pragma unroll
    for (int c = 0; c <= kPacked; ++c) {
      const int v = c < kPacked ? wave_incl_scan((int)cnt[c < kPacked ? c : 0]) : wave_max(longest);
      if (lane == kWave - 1) red[c * NW + wave] = (uint32_t)v;
    }
    __syncthreads();
    // every piece needs a workgroup of the grid
    const int one_per_cu = min(p.num_cu, (int)gridDim.x);
    longest = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      longest = max(longest, (int)red[kPacked * NW + w]);
    }
    int pieces[kNumPieceCaps + 1];
#pragma unroll
    for (int c = 0; c <= kNumPieceCaps; ++c) {
      int t = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) t += (int)(red[c / 2 * NW + w] >> (16 * (c % 2)) & 0xFFFFu);
      pieces[c] = t * p.hkv;
    }
#pragma unroll
    for (int c = kNumPieceCaps - 1; c >= 0; --c)
      if (pieces[c] <= one_per_cu || (c == 0 && cap == 0 && pieces[c] <= (int)gridDim.x))
        cap = piece_cap(c);
    // below eight blocks: a cap of c blocks leaves at most work / c pieces
    // plus one per segment
    const int segs = pieces[kNumPieceCaps];
    // G = 16 at D = 128, on eight waves, counts as the most
    const CutRule rule = NW == 8 && D == 128
                             ? CutRule{3, 5, 5}
                             : cut_rule((float)live * (float)(p.group * p.hkv * D), (float)segs);
    const int spare = min(p.num_cu * rule.cu_sixteenths / 16, (int)gridDim.x) - segs;
    if (spare > 0 && longest > rule.whole_blocks * kBlockKeys) {
      const int blocks = max(rule.min_blocks, max((longest / kBlockKeys + kMaxMerge - 1) / kMaxMerge,
                                                  (work / kBlockKeys + spare - 1) / spare));
      if (blocks < 8) cap = blocks * kBlockKeys;
    }
  }
  const bool seg_mode = cap > 0;
  int npc = 0;
  if (seg_mode) {
    if (per == 1) {
      npc = seg_pieces(sum, cap);
    } else {
      for (int i = lo; i < hi; ++i) npc += seg_pieces(segment_len(p, i), cap);
    }
  }
  // Stream-K works in the virtual space where each segment with keys is
  // lead keys longer (its lead-in first); the small-batch plan in keys.
  const int lead = seg_mode ? 0 : kLeadKeys;
  int total_pc = 0, total_v = total, excl_pc = 0, excl_v = excl, sum_v = sum;
  if (seg_mode) {
    excl_pc = block_excl_scan<NW>(npc, lds + NW, total_pc);
  } else {
    int nnz = 0;  // this thread's segments with keys
    if (per == 1) {
      nnz = sum > 0 ? 1 : 0;
    } else {
      for (int i = lo; i < hi; ++i) nnz += segment_len(p, i) > 0 ? 1 : 0;
    }
    sum_v = sum + lead * nnz;
    excl_v = block_excl_scan<NW>(sum_v, lds + NW, total_v);
    const int work_v = total_v * p.hkv;
    share = (work_v + (int)gridDim.x - 1) / (int)gridDim.x;
    share = max(kMinShare, round_up_block(share));
  }
  const int work_s = total_v * p.hkv;  // the plan's linear space (= work when seg_mode)
  if (blockIdx.x == 0) {
    int acc = excl_v, acc_pc = excl_pc;
    for (int i = lo; i < hi; ++i) {
      const int seg = segment_len(p, i);
      p.plan[i] = acc;
      p.plan[B + 2 + i] = acc_pc;
      acc += seg > 0 ? seg + lead : 0;
      if (seg_mode) acc_pc += seg_pieces(seg, cap);
    }
    if (tid == 0) {
      p.plan[B] = total_v;
      p.plan[B + 1] = seg_mode ? -cap : share;  // negative: the small-batch cap
      p.plan[2 * B + 2] = total_pc;
    }
  }
  const int b = (int)blockIdx.x;
  int start = work_s, end = work_s;
  if (!seg_mode) {
    const int skew = share_skew(share);
    start = min(work_s, share_begin(b, share, skew));
    end = min(work_s, share_begin(b + 1, share, skew));
  }
  // the thread whose requests contain this workgroup's share locates it and
  // publishes the request's metadata, so the first piece needs no second
  // read of it
  const bool mine = seg_mode ? (b < total_pc * p.hkv && excl_pc * p.hkv <= b &&
                                b < (excl_pc + npc) * p.hkv)
                             : (start < work_s && excl_v * p.hkv <= start &&
                                start < (excl_v + sum_v) * p.hkv);
  if (mine) {
    int acc = excl_v, acc_pc = excl_pc;
    for (int i = lo; i < hi; ++i) {
      if (per != 1) {
        q0 = p.cu[i];
        q1 = p.cu[i + 1];
        cx = p.ctx[i];
      }
      const int seg = segment_of(p, q0, q1, cx);
      const int segv = seg > 0 ? seg + lead : 0;  // seg when seg_mode
      const int n = seg_mode ? seg_pieces(seg, cap) : 0;
      int g = -1, off = 0, s0 = 0, s1 = 0;
      if (seg_mode) {
        if (b < (acc_pc + n) * p.hkv) {
          const int rel = b - acc_pc * p.hkv;
          g = rel / n;
          const int q = rel % n;
          off = piece_begin(seg, n, q);
          s0 = acc * p.hkv + g * seg + off;
          s1 = s0 + piece_begin(seg, n, q + 1) - off;
        }
      } else if (start < (acc + segv) * p.hkv) {
        const int rel = start - acc * p.hkv;
        g = rel / segv;
        off = rel % segv;
        s0 = start;
        s1 = end;
      }
      if (g >= 0) {
        loc[0] = i;
        loc[1] = g;
        loc[2] = off;
        loc[3] = q0;
        loc[4] = q1;
        loc[5] = cx;
        loc[6] = s0;
        loc[7] = s1;
        break;
      }
      acc += segv;
      acc_pc += n;
    }
  }
  __syncthreads();
  // Uniform by construction; declared so, or the compiler would treat every
  // branch on the share as divergent.
  auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  const bool has = uni(seg_mode ? b < total_pc * p.hkv : start < work_s) != 0;
  Share sh;
  sh.lead = uni(lead);
  sh.start = has ? uni(loc[6]) : 0;
  sh.end = has ? uni(loc[7]) : 0;
  sh.i = uni(loc[0]);
  sh.g = uni(loc[1]);
  sh.off = uni(loc[2]);
  const int f0 = uni(loc[3]), f1 = uni(loc[4]);
  sh.first.q0 = f0;
  sh.first.ctx = uni(loc[5]);
  sh.first.k = f1 - f0;
  sh.first.len = sh.first.ctx + sh.first.k;
  sh.first.seg = segment_of(p, f0, f1, sh.first.ctx);
  return sh;
}

// The wave's query operands, and the last key each lane's row may see (-1: a
// row past the live ones).
template <int D, int TW>
struct QOps {
  bf16x8 r[TW][D / 32];
  int row_limit[TW];
};

// Tiles tile0 .. tile0+TW-1 of request rq.  A row past the live ones loads row
// 0 of the request and is zeroed, so that no load sits behind a branch of its
// own.
template <int D, int TW>
__device__ __forceinline__ void load_q(const AttnParams &p, int g, const ReqMeta &rq, int tile0,
                                       int lane, QOps<D, TW> &qv) {
  const int kq = lane >> 4, n = lane & 15;
  const int lg = __builtin_ctz(p.group);
  u32x4 x[TW][D / 32];
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    const int rr = (tile0 + t) * 16 + n;
    const bool valid = rr < p.group * rq.k;
    const int at = valid ? rr : 0;
    const int j = at >> lg, hh = at & (p.group - 1);
    qv.row_limit[t] = valid ? rq.ctx + j : -1;
    const uint16_t *row = p.q + ((size_t)(rq.q0 + j) * p.hq + (size_t)g * p.group + hh) * D;
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
      x[t][c] = *reinterpret_cast<const u32x4 *>(row + 32 * c + 8 * kq);
  }
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    const uint32_t keep = qv.row_limit[t] >= 0 ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
      qv.r[t][c] = as_bf16x8(__builtin_bit_cast(uint4, x[t][c] & u32x4{keep, keep, keep, keep}));
  }
}

template <int TW, int NE>
__device__ __forceinline__ void clear_state(RowState<TW, NE> &st) {
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    st.m[t] = kNoMax;
    st.l[t] = 0.f;
#pragma unroll
    for (int u = 0; u < NE; ++u) st.o[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// Scores of one step for the wave's tiles (raw: the scale is positive and
// applied inside the exponent).  Element (h, q) of a lane is key
// t0 + 16h + 4*(lane>>4) + q.
template <int TW>
struct Scores {
  f32x4 x[TW][2];
};
template <int D, int TW>
__device__ __forceinline__ void step_scores(const KRegs<D> &k, const QOps<D, TW> &qv,
                                            Scores<TW> &s) {
#pragma unroll
  for (int t = 0; t < TW; ++t) {
#pragma unroll
    for (int h = 0; h < 2; ++h) s.x[t][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        s.x[t][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            as_bf16x8(__builtin_bit_cast(uint4, k.x[h][c])), qv.r[t][c], s.x[t][h], 0, 0, 0);
    }
  }
}

// Causal and end-of-request masking of a step that not every live row sees
// whole.  Keys at or past `se` may hold anything (even NaN), so their V is
// zeroed as well.
template <int TW, int NE>
__device__ __forceinline__ void step_mask(int t0, int se, const int (&row_limit)[TW], int lane,
                                          Scores<TW> &s, VRegs<NE> &v) {
  const int kq = lane >> 4;
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int key = t0 + 16 * h + 4 * kq + q;
        if (key > row_limit[t] || key >= se) s.x[t][h][q] = -INFINITY;
      }
  const int tb = t0 + 16 * (kq & 1) + 8 * (kq >> 1);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t mask = (tb + 2 * w < se ? 0x0000FFFFu : 0u) |
                          (tb + 2 * w + 1 < se ? 0xFFFF0000u : 0u);
#pragma unroll
    for (int u = 0; u < NE; ++u) v.x[u][w] &= mask;
  }
}

// Online softmax and the PV product of one step.
template <int TW, int NE>
__device__ __forceinline__ void step_update(const Scores<TW> &s, const VRegs<NE> &v,
                                            float scale_log2, RowState<TW, NE> &st) {
  // a lane's own keys decide whether any row's maximum moves; only then are
  // the row's four lanes brought together
  bool jump = false;
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    float top = -INFINITY;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        top = fmaxf(top, __builtin_fmaf(s.x[t][h][q], scale_log2, -st.m[t]));
    jump |= top > kRescaleSlack;
  }
  if (__builtin_amdgcn_ballot_w64(jump) != 0) {
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      float top = -INFINITY;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q) top = fmaxf(top, s.x[t][h][q]);
      const float m_new = fmaxf(st.m[t], ceilf(row_max4(top) * scale_log2));
      // 0 on a row's first visible step, 1 for a row that still sees nothing
      const float alpha = __builtin_amdgcn_exp2f(st.m[t] - m_new);
      st.l[t] *= alpha;
#pragma unroll
      for (int u = 0; u < NE; ++u) st.o[t][u] *= alpha;
      st.m[t] = m_new;
    }
  }
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    // P enters the bf16 PV product as a pair: hi = P rounded to bf16 and
    // lo = the remainder rounded to bf16, so hi + lo carries P to about
    // 2^-17 of its value and the weights add no error next to the output's
    // own bf16 rounding.  The row sum adds the fp32 weights themselves.
    uint32_t hi[2][2], lo[2][2];
    float psum[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float pw[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        pw[q] = __builtin_amdgcn_exp2f(
            __builtin_fmaf(s.x[t][h][q], scale_log2, -st.m[t]));
      psum[h] = (pw[0] + pw[1]) + (pw[2] + pw[3]);
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const uint32_t x = pack_bf16x2(pw[2 * w], pw[2 * w + 1]);
        hi[h][w] = x;
        lo[h][w] = pack_bf16x2(pw[2 * w] - __uint_as_float(x << 16),
                               pw[2 * w + 1] - __uint_as_float(x & 0xFFFF0000u));
      }
    }
    st.l[t] += psum[0] + psum[1];
    // lane (kq, n) holds slots 4kq .. +3 of both pages; trading odd rows of
    // page 0's against even rows of page 1's leaves it slots 8*(kq>>1) .. +7
    // of page kq & 1, the keys of its V operand
    const auto h0 = __builtin_amdgcn_permlane16_swap(hi[0][0], hi[1][0], false, false);
    const auto h1 = __builtin_amdgcn_permlane16_swap(hi[0][1], hi[1][1], false, false);
    const auto l0 = __builtin_amdgcn_permlane16_swap(lo[0][0], lo[1][0], false, false);
    const auto l1 = __builtin_amdgcn_permlane16_swap(lo[0][1], lo[1][1], false, false);
    const bf16x8 ph = as_bf16x8(make_uint4(h0[0], h1[0], h0[1], h1[1]));
    const bf16x8 pl = as_bf16x8(make_uint4(l0[0], l1[0], l0[1], l1[1]));
#pragma unroll
    for (int u = 0; u < NE; ++u)
      st.o[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          as_bf16x8(__builtin_bit_cast(uint4, v.x[u])), ph, st.o[t][u], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < NE; ++u)
      st.o[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          as_bf16x8(__builtin_bit_cast(uint4, v.x[u])), pl, st.o[t][u], 0, 0, 0);
  }
}

// --------------------------------------------------------------------- ring
// K and V stream through an LDS ring of kStages stages, all of them in flight
// in registers: one step a stage with four waves, two with eight (a tile or
// more for every wave).  Each wave loads its tiles of a stage (a page's K or
// V, contiguous 1 KiB loads), writes them to the ring when the stage comes up,
// and after the barrier the waves read their operands from it.  With four
// waves, stages of two steps (two in flight, 128 KiB to a CU instead of 96)
// measured slower: B=32, contexts to 8K 104.4 -> 107-112 us, with eight query
// heads to a KV head and contexts to 16K 229 -> 238 us.
template <int D, int NW>
struct Ring {
  static constexpr int kSteps = NW / 4;
  static constexpr int kKeys = kSteps * kBlockKeys;
  static constexpr int kPages = kKeys / kPage;
  static constexpr int kTile = kPage * D * 2;          // bytes of a page's K or V
  static constexpr int kStage = 2 * kPages * kTile;    // K tiles, then V tiles (kSteps * 16 KiB)
  static constexpr int kStages = 3;
  static constexpr int kTiles = 2 * kPages / NW;       // tiles a wave loads per stage
  static constexpr int kBytes = kStages * kStage;
  // page and kind (0: K, 1: V) of a wave's q-th tile
  static __device__ __forceinline__ int page(int wave, int q) { return (wave * kTiles + q) >> 1; }
  static __device__ __forceinline__ int kind(int wave, int q) { return (wave * kTiles + q) & 1; }
};

// V tiles sit in the ring with their 16-byte units (dim, half of the slots)
// permuted inside each 1 KiB, so that the operand reads are free of bank
// conflicts: global unit u = 2*dim + half is LDS unit v_unit(u), and
// v_unit_inv is the inverse.  Aligned groups of four lanes still load aligned
// 64-byte pieces.
__device__ __forceinline__ int v_sel(int k) { return ((k >> 1) ^ (k >> 2)) & 1; }
__device__ __forceinline__ int v_unit(int u) {
  const int k = u >> 2, j = (u >> 1) & 1, b = u & 1;
  return 4 * k + 2 * (b ^ v_sel(k)) + j;
}
__device__ __forceinline__ int v_unit_inv(int l) {
  const int k = l >> 2, j = l & 1, b = ((l >> 1) & 1) ^ v_sel(k);
  return 4 * k + 2 * j + b;
}

// What a wave needs to run the ring over one sub-piece.
struct RingCtx {
  const int *ids;        // LDS: page ids of the sub-piece
  const char *kbase;     // K tile of page 0, this KV head, plus the lane's offset
  const char *vbase;     // V tile of page 0, this KV head, plus the lane's offset
  uint32_t page_bytes;   // bytes per page (2 * Hkv tiles)
  int ns;                // stages
  int sb, se, ctx;       // first key, end of the keys, committed context
  int prio_end;          // key at which the wave priority returns to the default
};

template <int D, int NW>
struct StageRegs {
  u32x4 x[Ring<D, NW>::kTiles][D / 32];
};

// Loads the wave's tiles of stage b.  Past the last stage it reads page 0
// instead (in cache, never used): the loop then has one shape, and the
// compiler can wait for exactly the stage each step writes.
template <int D, int NW>
__device__ __forceinline__ void ring_load(const RingCtx &c, int b, int wave,
                                          StageRegs<D, NW> &r) {
  using R = Ring<D, NW>;
#pragma unroll
  for (int q = 0; q < R::kTiles; ++q) {
    const int at = R::kPages * min(b, c.ns - 1) + R::page(wave, q);
    const int id = b < c.ns ? __builtin_amdgcn_readfirstlane(c.ids[at]) : 0;
    const char *t =
        (R::kind(wave, q) ? c.vbase : c.kbase) + (size_t)(uint32_t)id * c.page_bytes;
#pragma unroll
    for (int x = 0; x < D / 32; ++x)
      r.x[q][x] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(t + 1024 * x));
  }
}

// A wave's part of the work on a piece: its row tiles and its d blocks.
struct Role {
  int tile0, e_lo;
  bool active;
};

// One stage in ring slot S: write it, load the stage kStages ahead, and after
// the barrier compute the wave's steps of it.
template <int D, int TW, int NE, int NW, int S>
__device__ __forceinline__ void ring_step(const RingCtx &c, char *ring, int b, int wave, int lane,
                                          StageRegs<D, NW> &r, const QOps<D, TW> &qv,
                                          const Role &role, float scale_log2,
                                          RowState<TW, NE> &st) {
  using R = Ring<D, NW>;
  char *stage = ring + S * R::kStage;
#pragma unroll
  for (int q = 0; q < R::kTiles; ++q) {
    char *dst = stage + (R::kind(wave, q) * R::kPages + R::page(wave, q)) * R::kTile + 16 * lane;
#pragma unroll
    for (int x = 0; x < D / 32; ++x) *reinterpret_cast<u32x4 *>(dst + 1024 * x) = r.x[q][x];
  }
  ring_load<D, NW>(c, b + R::kStages, wave, r);
  __syncthreads();
  if (c.sb + b * R::kKeys >= c.prio_end) __builtin_amdgcn_s_setprio(0);
  if (!role.active) return;
  const int kq = lane >> 4, m = lane & 15;
  const char *vb = stage + (R::kPages + (kq & 1)) * R::kTile + 16 * v_unit(2 * m + (kq >> 1)) +
                   512 * role.e_lo;
#pragma unroll 1
  for (int sub = 0; sub < R::kSteps; ++sub) {
    const int t0 = c.sb + b * R::kKeys + sub * kBlockKeys;
    if (t0 >= c.se) break;
    KRegs<D> k;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int x = 0; x < D / 32; ++x)
        k.x[h][x] = *reinterpret_cast<const u32x4 *>(
            stage + (sub * 2 + h) * R::kTile + 1024 * x + 16 * lane);
    Scores<TW> s;
    step_scores<D, TW>(k, qv, s);
    VRegs<NE> v;
#pragma unroll
    for (int u = 0; u < NE; ++u)
      v.x[u] = *reinterpret_cast<const u32x4 *>(vb + sub * 2 * R::kTile + 512 * u);
    if (t0 + kBlockKeys > min(c.ctx, c.se))
      step_mask<TW, NE>(t0, c.se, qv.row_limit, lane, s, v);
    step_update<TW, NE>(s, v, scale_log2, st);
  }
}

// All stages of one sub-piece.
template <int D, int TW, int NE, int NW>
__device__ __forceinline__ void ring_run(const RingCtx &c, char *ring, int wave, int lane,
                                         const QOps<D, TW> &qv, const Role &role,
                                         float scale_log2, RowState<TW, NE> &st) {
  constexpr int kStages = Ring<D, NW>::kStages;
  StageRegs<D, NW> r[kStages];
  // issued in stage order (the empty asm keeps the compiler from reordering
  // them), so that each step waits only for its own stage
#pragma unroll
  for (int s = 0; s < kStages; ++s) {
    ring_load<D, NW>(c, s, wave, r[s]);
    asm volatile("" ::: "memory");
  }
  for (int b = 0; b < c.ns; b += kStages) {
    ring_step<D, TW, NE, NW, 0>(c, ring, b, wave, lane, r[0], qv, role, scale_log2, st);
    ring_step<D, TW, NE, NW, 1>(c, ring, b + 1, wave, lane, r[1], qv, role, scale_log2, st);
    ring_step<D, TW, NE, NW, 2>(c, ring, b + 2, wave, lane, r[2], qv, role, scale_log2, st);
  }
}

// ------------------------------------------------------------------- pieces
// A piece: the workgroup's keys [key_begin, key_end) of request i, KV head g.
struct Piece {
  int i, g, key_begin, key_end, slot, prio_end;
  bool complete;
  ReqMeta rq;
};

// Writes NE d blocks from e_lo of a finished row tile: bf16 output when the
// piece is the whole segment, otherwise the fp32 partial in this workgroup's
// slot (0: the segment where its share starts, 1: where it ends), with (m, l)
// beside d block 0.
template <int D, int NE>
__device__ __forceinline__ void write_rows(const AttnParams &p, const Piece &x, int rt, int e_lo,
                                           int lane, float m, float l, const f32x4 (&o)[NE]) {
  const int kq = lane >> 4;
  const int rr = rt * 16 + (lane & 15);
  if (rr >= p.group * x.rq.k) return;
  const int dim = 16 * e_lo + 4 * kq;
  if (x.complete) {
    const int lg = __builtin_ctz(p.group);
    const int j = rr >> lg, hh = rr & (p.group - 1);
    const size_t row = (size_t)(x.rq.q0 + j) * p.hq + (size_t)x.g * p.group + hh;
    const float inv = 1.f / l;
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      uint2 w;
      w.x = pack_bf16x2(o[u][0] * inv, o[u][1] * inv);
      w.y = pack_bf16x2(o[u][2] * inv, o[u][3] * inv);
      *reinterpret_cast<uint2 *>(p.out + row * D + dim + 16 * u) = w;
    }
  } else {
    const size_t prow = ((size_t)blockIdx.x * 2 + x.slot) * (p.group * kMaxQlen) + rr;
#pragma unroll
    for (int u = 0; u < NE; ++u)
      *reinterpret_cast<f32x4 *>(p.part_o + prow * D + dim + 16 * u) = o[u];
    if (e_lo == 0 && kq == 0) p.part_ml[prow] = make_float2(m, l);
  }
}

// Wave roles.  NE < D/16 d blocks: the waves split one tile's dims (or two
// tiles', half of the waves each).  All of them: each wave has TW tiles to
// itself.
template <int D, int TW, int NE, int NW>
__device__ __forceinline__ void run_piece(const AttnParams &p, char *buf, int *ids, const Piece &x,
                                          int wave, int lane, int first_tile = 0) {
  using R = Ring<D, NW>;
  constexpr int kParts = D / 16 / NE;  // waves to a tile
  Role role;
  role.tile0 = first_tile + wave / kParts * TW;
  role.e_lo = wave % kParts * NE;
  role.active = role.tile0 * 16 < p.group * x.rq.k;
  RowState<TW, NE> st;
  QOps<D, TW> qv;
  load_q<D, TW>(p, x.g, x.rq, role.tile0, lane, qv);
  clear_state<TW, NE>(st);
  RingCtx c;
  c.ids = ids;
  c.page_bytes = (uint32_t)(2 * p.hkv * kPage * D * (int)sizeof(uint16_t));
  c.kbase = reinterpret_cast<const char *>(p.kv) + (size_t)x.g * kPage * D * sizeof(uint16_t) +
            16 * lane;
  c.vbase = reinterpret_cast<const char *>(p.kv) +
            (size_t)(p.hkv + x.g) * kPage * D * sizeof(uint16_t) + 16 * v_unit_inv(lane);
  c.ctx = x.rq.ctx;
  c.prio_end = x.prio_end;
  for (int sb = x.key_begin; sb < x.key_end; sb += kSubKeys) {
    const int se = min(x.key_end, sb + kSubKeys);
    c.sb = sb;
    c.se = se;
    c.ns = (se - sb + R::kKeys - 1) / R::kKeys;
    // the sub-piece's page ids; an id outside [0, num_pages) breaks the
    // contract and reads page 0 instead (valid memory, result unspecified),
    // pages past the sub-piece read page 0 and are masked
    const int npg = (se - sb + kPage - 1) / kPage;
    const int *pt = p.page_table + (size_t)x.i * p.max_pages + sb / kPage;
    if (sb > x.key_begin) __syncthreads();  // the last ids and stages have been read
    for (int t = threadIdx.x; t < R::kPages * c.ns; t += NW * kWave) {
      const int id = t < npg ? pt[t] : 0;
      ids[t] = (unsigned)id < (unsigned)p.num_pages ? id : 0;
    }
    __syncthreads();
    ring_run<D, TW, NE, NW>(c, buf, wave, lane, qv, role, p.scale_log2, st);
  }
  if (!role.active) return;
#pragma unroll
  for (int t = 0; t < TW; ++t)
    write_rows<D, NE>(p, x, role.tile0 + t, role.e_lo, lane, st.m[t], row_sum4(st.l[t]), st.o[t]);
}

// NW waves, each with up to kTW row tiles: as many as the group's largest
// requests have (16 rows of each head), or as many at a time, K and V read again for
// the rest (kPasses).  Workgroups to a CU, by registers: two of four waves at
// D = 128 (three measured slower: 36 requests, contexts to 2K, four layers 232.8 ->
// 252.9 us), one of eight.  At D = 64 a step is half the bytes and a wave needs half
// the registers: four with one tile to a wave, three with two (four would spill), two
// with four: 16 requests of 10K keys on one KV head take 22.5 us instead of 26.4, 33
// short ones of eight heads to a KV head 39.5 instead of 43.5.
constexpr int min_waves_per_simd(int D, int NW, int kTW) {
  return D == 64 && NW == 4 ? (kTW == 1 ? 4 : (kTW == 2 ? 3 : 2)) : 2;
}
template <int D, int NW, int kTW, bool kPasses = false>
__global__ __launch_bounds__(NW *kWave, min_waves_per_simd(D, NW, kTW)) void attn_streamk_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(1024))) char buf[Ring<D, NW>::kBytes];
  __shared__ int ids[kSubPages];
  __shared__ int lds_plan[2 * NW + 8 + (kNumPieceCaps / 2 + 2) * NW];

  const Share sh = plan_share<D, NW>(p, lds_plan);
  if (sh.start >= sh.end) return;
  int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int lane = threadIdx.x % kWave;

  // keys of the share (virtual) run at raised priority; -1: none
  const bool boost = (int)blockIdx.x >= p.num_cu;
  if (boost) __builtin_amdgcn_s_setprio(1);
  const int boost_end = boost ? sh.start + (int)((long long)(sh.end - sh.start) * kBoostPct / 100) : -1;

  Piece x;
  x.i = sh.i;
  x.g = sh.g;
  x.rq = sh.first;
  int off = sh.off, pos = sh.start, piece = 0;
  // metadata of the request last read: the next KV head's segment of the
  // same request (the usual next piece) needs no second read of it
  int i_meta = sh.i;
  while (pos < sh.end && x.i < p.num_reqs) {
    if (x.i != i_meta) {
      x.rq = load_req(p, x.i);
      i_meta = x.i;
    }
    if (x.rq.seg == 0) {  // sentinel or bad metadata: no keys in the plan
      ++x.i;
      continue;
    }
    // offsets are virtual: the segment's keys follow its lead-in of
    // sh.lead keys (none in the small-batch plan)
    const int segv = x.rq.seg + sh.lead;
    const int take = min(segv - off, sh.end - pos);
    x.key_begin = max(off - sh.lead, 0);
    x.key_end = min(x.rq.len, off + take - sh.lead);
    if (x.key_end <= x.key_begin) break;  // the share ends inside the lead-in
    x.complete = off <= sh.lead && off + take == segv;
    x.slot = piece == 0 ? 0 : 1;
    x.prio_end = boost ? x.key_begin + boost_end - pos : 0x7FFFFFFF;
    if (piece > 0) __syncthreads();  // the last piece's LDS has been read

    // opaque per piece: or the compiler computes every lane's offsets for all
    // the piece forms ahead of the loop, and spills them
    asm volatile("" : "+v"(lane), "+s"(wave));
    const int nt = (p.group * x.rq.k + 15) / 16;  // row tiles
    // one or two tiles split their dims over four waves.  Eight waves don't split
    // them: each would read all of K from LDS (D = 128, 32 requests, contexts to
    // 8K, 8 KV heads, two rows each: 119.5 us, split 135.0).
    constexpr int kBlocks = D / 16;
    if (NW == 4 && nt == 1)
      run_piece<D, 1, kBlocks / 4, NW>(p, buf, ids, x, wave, lane);
    else if (NW == 4 && nt == 2)
      run_piece<D, 1, kBlocks / 2, NW>(p, buf, ids, x, wave, lane);
    else if (kTW == 1 || nt <= NW)
      run_piece<D, 1, kBlocks, NW>(p, buf, ids, x, wave, lane);
    else if constexpr (kTW == 4) {
      if (nt <= 2 * NW)
        run_piece<D, 2, kBlocks, NW>(p, buf, ids, x, wave, lane);
      else
        run_piece<D, 4, kBlocks, NW>(p, buf, ids, x, wave, lane);
    } else if constexpr (kPasses) {
      for (int t = 0; t < nt; t += kTW * NW) {
        if (t > 0) __syncthreads();  // the last pass's LDS has been read
        run_piece<D, kTW, kBlocks, NW>(p, buf, ids, x, wave, lane, t);
      }
    } else if constexpr (kTW == 2)
      run_piece<D, 2, kBlocks, NW>(p, buf, ids, x, wave, lane);

    pos += take;
    off += take;
    ++piece;
    if (off == segv) {
      off = 0;
      if (++x.g == p.hkv) {
        x.g = 0;
        ++x.i;
      }
    }
  }
}

// Merges the partials of segments that straddle share boundaries (in
// workgroup order, so the result is deterministic) and zeroes the tail rows.
// Workgroup (x, g, i) owns kCombThreads/(D/4) live rows of request i and KV head g;
// each thread owns 4 output dims of one row and issues the loads of up to 8
// partials at a time.  Workgroups with z == B zero the tail rows instead.
template <int D>
__global__ __launch_bounds__(kCombThreads) void attn_combine_kernel(AttnParams p) {
  constexpr int kLanesPerRow = D / 4;
  constexpr int kRows = kCombThreads / kLanesPerRow;
  const int g = blockIdx.y, i = blockIdx.z;
  const int G = p.group;
  if (i == p.num_reqs) {
    const int live = min(max(p.cu[p.num_reqs], 0), p.cap);
    const int per_row = G * (D / 8);
    const int total = (p.cap - live) * per_row;
    for (int idx = blockIdx.x * kCombThreads + threadIdx.x; idx < total;
         idx += gridDim.x * kCombThreads) {
      const int r = live + idx / per_row, rem = idx % per_row;
      const int hh = rem / (D / 8), d8 = rem % (D / 8);
      uint16_t *o = p.out + ((size_t)r * p.hq + (size_t)g * G + hh) * D + 8 * d8;
      *reinterpret_cast<uint4 *>(o) = make_uint4(0, 0, 0, 0);
    }
    return;
  }
  // Every plan entry and metadata word this workgroup may need, loaded in
  // one round trip: the empty asm uses them all before the first branch,
  // so the compiler cannot sink the loads that one path needs behind the
  // branches (which made a chain of dependent round trips).
  int prefix = p.plan[i], next = p.plan[i + 1];  // p.plan[B] is the total
  int share = p.plan[p.num_reqs + 1];
  int pc_prefix = p.plan[p.num_reqs + 2 + i];  // read by the small-batch plan only
  int cq0 = p.cu[i], cq1 = p.cu[i + 1], cctx = p.ctx[i];
  asm volatile("" : "+s"(prefix), "+s"(next), "+s"(share), "+s"(pc_prefix), "+s"(cq0),
               "+s"(cq1), "+s"(cctx));
  ReqMeta rq;
  rq.q0 = cq0;
  rq.ctx = cctx;
  rq.k = cq1 - cq0;
  rq.len = cctx + rq.k;
  rq.seg = segment_of(p, cq0, cq1, cctx);
  const int seg = next - prefix;
  if (seg <= 0) return;
  const int start = prefix * p.hkv + g * seg;
  const int skew = share > 0 ? share_skew(share) : 0;
  int b0, b1;
  if (share <= 0) {
    // small-batch plan: the segment's n pieces sit on consecutive workgroups,
    // each the first (and only) piece of its workgroup
    const int n = seg_pieces(seg, -share);
    b0 = pc_prefix * p.hkv + g * n;
    b1 = b0 + n - 1;
  } else {
    // stream-K: seg includes the lead-in, and the first workgroup with any
    // of the segment's keys is the one holding the first key after it
    b0 = share_owner(start + kLeadKeys, share, skew);
    b1 = share_owner(start + seg - 1, share, skew);
  }
  if (b0 == b1) return;  // one workgroup held the whole segment
  const int rr = blockIdx.x * kRows + threadIdx.x / kLanesPerRow;
  if (rr >= G * rq.k) return;
  const int d4 = threadIdx.x % kLanesPerRow;
  const int lg = __builtin_ctz(G);
  const int j = rr >> lg, hh = rr & (G - 1);
  const size_t row = (size_t)(rq.q0 + j) * p.hq + (size_t)g * G + hh;
  const int n_parts = b1 - b0 + 1;
  // partial of workgroup b0 + u: slot 0 if its share starts inside this
  // segment, else slot 1 (the segment is where its share ends)
  auto prow = [&](int u) -> size_t {
    const int b = b0 + u;
    const int slot = share <= 0 || share_begin(b, share, skew) >= start ? 0 : 1;
    return ((size_t)b * 2 + slot) * (G * kMaxQlen) + rr;
  };

  float mx = -INFINITY;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float den = 0.f;
  if (n_parts <= 8) {
    // the common case: every load in one round trip
    float2 l8[8];
    f32x4 o8[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool in = u < n_parts;
      const size_t pr = prow(u);
      l8[u] = in ? p.part_ml[pr] : make_float2(-INFINITY, 0.f);
      o8[u] = in ? *reinterpret_cast<const f32x4 *>(p.part_o + pr * D + 4 * d4)
                 : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) mx = fmaxf(mx, l8[u].x);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float w = exp2f(l8[u].x - mx);
      den += w * l8[u].y;
      acc += w * o8[u];
    }
  } else {
    for (int u0 = 0; u0 < n_parts; u0 += 8) {
      float m8[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        m8[u] = u0 + u < n_parts ? p.part_ml[prow(u0 + u)].x : -INFINITY;
#pragma unroll
      for (int u = 0; u < 8; ++u) mx = fmaxf(mx, m8[u]);
    }
    for (int u0 = 0; u0 < n_parts; u0 += 8) {
      float2 l8[8];
      f32x4 o8[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool in = u0 + u < n_parts;
        const size_t pr = prow(u0 + u);
        l8[u] = in ? p.part_ml[pr] : make_float2(-INFINITY, 0.f);
        o8[u] = in ? *reinterpret_cast<const f32x4 *>(p.part_o + pr * D + 4 * d4)
                   : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float w = exp2f(l8[u].x - mx);
        den += w * l8[u].y;
        acc += w * o8[u];
      }
    }
  }
  const float inv = 1.f / den;
  uint2 w2;
  w2.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
  w2.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
  *reinterpret_cast<uint2 *>(p.out + row * D + 4 * d4) = w2;
}

// Compute units of the current device (cached per device; a host query).
int device_cus() {
  static int cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  if (cache[dev] > 0) return cache[dev];
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  cache[dev] = cus;
  return cus;
}

// The split kernel for a batch's dims, and its threads.  Only G = 16, with up to
// sixteen row tiles to a request, has a choice, between eight waves in one workgroup
// to a CU and forms with more, smaller workgroups; of what it depends on the host
// knows the most segments (requests x KV heads) and the longest context.
//  D = 128: eight waves hold all tiles.  Where there are more segments than CUs and
//   each is short, that leaves every CU several in a row to start: four waves
//   there, eight tiles at a time, the second pass's K and V from cache (64 requests
//   to 200 keys, 8 KV heads, one row each 46.3 -> 33.9 us, full blocks 68.8 -> 53.1; to
//   500 keys 54.8 -> 51.5 and 89.8 -> 102.9).
//  D = 64: four waves can hold all tiles, two workgroups to a CU, which pays with
//   many segments (us, eight waves / four: 32 requests to 8K, 8 KV heads, one row each
//   75.0 / 64.4, geometric lengths 156.6 / 107.0, full blocks 165 / 150; 24 to 6K, 4 KV
//   heads 28.9 / 26.1, 52.7 / 42.9, 59.1 / 61.5); with few the second workgroup only
//   adds partials (1 to 30K, 8 KV heads 23.3 / 27.9, full blocks 46.9 / 59.0; 64 to
//   4K, 1 KV head, full blocks 38.7 / 42.6).
struct SplitKernel {
  void (*fn)(AttnParams);
  int threads;
};
constexpr int kSplitKernels = 8;
constexpr int kManySegments128 = 256, kShortKeys = 256, kManySegments64 = 64;
int split_kernel_index(const dsv_attn_dims &d) {
  const int group = d.num_q_heads / d.num_kv_heads;
  const long long segments = (long long)d.num_reqs * d.num_kv_heads;
  if (d.head_dim == 128) {
    if (group > 8) return segments > kManySegments128 && d.max_kv_len <= kShortKeys ? 3 : 2;
    return group > 4 ? 1 : 0;
  }
  if (group > 8) return segments > kManySegments64 ? 7 : 6;
  return group > 4 ? 5 : 4;
}
SplitKernel split_kernel(int index) {
  constexpr int k4 = 4 * kWave, k8 = 8 * kWave;
  switch (index) {
    case 0: return {attn_streamk_kernel<128, 4, 1>, k4};
    case 1: return {attn_streamk_kernel<128, 4, 2>, k4};
    case 2: return {attn_streamk_kernel<128, 8, 2>, k8};
    case 3: return {attn_streamk_kernel<128, 4, 2, true>, k4};
    case 4: return {attn_streamk_kernel<64, 4, 1>, k4};
    case 5: return {attn_streamk_kernel<64, 4, 2>, k4};
    case 6: return {attn_streamk_kernel<64, 8, 2>, k8};
    default: return {attn_streamk_kernel<64, 4, 4>, k4};
  }
}

// Workgroups the GPU holds at once for the split kernel (cached per device
// and kernel; a host query, so it is safe during graph capture).
int resident_workgroups(int index) {
  static int cache[64][kSplitKernels];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int &slot = cache[dev][index];
  if (slot > 0) return slot;
  const int cus = device_cus();
  int per_cu = 0;
  const SplitKernel k = split_kernel(index);
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, reinterpret_cast<const void *>(k.fn), k.threads, 0);
  if (e != hipSuccess || cus <= 0 || per_cu <= 0) return 0;
  slot = cus * per_cu;
  return slot;
}

}  // namespace

// Upper bound of the persistent grid, known without a device: at most 1024
// workgroups and never more than the 32-key blocks the largest batch could hold.
// The workspace is sized for it.  A 256-CU MI355X holds at once, by head_dim and
// group: 128, up to 8: 512; 128, 16: 256 (512 of the form for many short segments);
// 64, up to 4: 1024; 64, 8: 768; 64, 16: 512 (256 of the form for few segments).
int32_t attn_grid_cap(const dsv_attn_dims &d) {
  constexpr long long kMaxGrid = 1024;
  const long long blocks = (long long)d.num_reqs * d.num_kv_heads *
                           ((d.max_kv_len + kBlockKeys - 1) / kBlockKeys);
  return (int32_t)(blocks < kMaxGrid ? blocks : kMaxGrid);
}

int32_t attn_num_cu() { return device_cus(); }

// Launch grid: the workgroups the current device holds at once, capped.
int32_t attn_grid(const dsv_attn_dims &d) {
  const int r = resident_workgroups(split_kernel_index(d));
  if (r <= 0) return 0;
  const int32_t cap = attn_grid_cap(d);
  return r < cap ? r : cap;
}

AttnWorkspace attn_workspace_layout(const dsv_attn_dims &d) {
  AttnWorkspace w;
  const size_t grid = (size_t)attn_grid_cap(d);
  const size_t rows = grid * 2 * (size_t)(d.num_q_heads / d.num_kv_heads) * kMaxQlen;
  w.grid_cap = (int32_t)grid;
  w.plan_off = 0;
  w.part_ml_off = align_up((size_t)(2 * d.num_reqs + 3) * sizeof(int32_t), 256);
  w.part_o_off = align_up(w.part_ml_off + rows * sizeof(float2), 256);
  w.total = align_up(w.part_o_off + rows * d.head_dim * sizeof(float), 256);
  return w;
}

hipError_t launch_verify_attn(const AttnParams &p, const dsv_attn_dims &d, hipStream_t s) {
  // rows of one request and KV head: G * k_i <= G * 16
  const int comb_rows = d.head_dim == 128 ? kCombThreads / 32 : kCombThreads / 16;
  const dim3 grid_comb((p.group * kMaxQlen + comb_rows - 1) / comb_rows, p.hkv,
                       p.num_reqs + 1);
  timing_mark(kTimeAttnSplit, false, s);
  const SplitKernel split = split_kernel(split_kernel_index(d));
  launch_kernel(split.fn, dim3(p.num_wg), dim3(split.threads), s, p);
  timing_mark(kTimeAttnSplit, true, s);
  timing_mark(kTimeAttnCombine, false, s);
  if (d.head_dim == 128)
    launch_kernel(attn_combine_kernel<128>, grid_comb, dim3(kCombThreads), s, p);
  else
    launch_kernel(attn_combine_kernel<64>, grid_comb, dim3(kCombThreads), s, p);
  timing_mark(kTimeAttnCombine, true, s);
  return hipGetLastError();
}

}  // namespace dsv
