// Decode-step attention over the ragged per-head cache (Sec. 5; weights of Sec. 3.2
// Eq. 2): for every KV head, its G = HQ/H query heads attend to the head's packed
// rows and to the rows still inside the window ring.
//
// The kernel is bound by reading K and V once (512 bytes per row against 4*G*128
// flops), so the design is about streaming rows with as few vector-ALU instructions
// per byte as possible; both contractions run on v_mfma_f32_16x16x32_bf16:
//
//   one wave = an equal part of all heads' rows, or a split of one head's (attend_deal.h), in
//   32-row chunks, the next chunk's loads in flight while the current one is consumed.
//
// Streamed: every load instruction takes four whole rows of K or V (1 KB) with the non-temporal hint, the
// form in which this part's memory gives 7.0 TB/s.  Without the hint, or with it and 64 bytes of a
// 128-byte line per instruction (K in the operand layout straight from memory), a read stream gets 6.1.
// The smallest steps, which a cache serves and whose time is a wavefront's from start to end, do without.
//
//   S^T = K q^T      A = K   lane (i = l%16, kg = l/16) holds 16 bytes of row rho(i) at
//                            byte 64*kk + 16*kg for kk = 0..3 (the k-slices an MFMA
//                            step wants); two 16-row sets per chunk.  Streamed, it is loaded like V
//                            below and turned through 8 KB of LDS of the wavefront's own (pieces
//                            XOR-swizzled with the row: no bank conflicts either way)
//                    B = q   lane (g = l%16, kg) holds q[g][32kk + 8kg ..+8], zero for
//                            g >= G
//                    C       lane (g, s = l/16), register r: row i = 4s + r of the set
//   with rho(t, i) = 16t + 4(i%4) + i/4, so lane (g, s) ends up with the scores of the
//   chunk rows 4j + s, j = 4t + r = 0..7: exactly the eight k-slots of B in
//
//   O^T = V^T P^T    A = V^T lane (c = l%16, s = l/16) loads piece c (8 values,
//                            d = 8c..8c+7) of the rows 4j + s, j = 0..7, fully
//                            coalesced (a load instruction covers 4 whole rows); one
//                            v_perm per register pairs rows (2j', 2j'+1) of one d,
//                            which is the k-pair layout of the A operand for the
//                            d-tile {8c + e : c = 0..15}
//                    B = P^T the exponentiated scores of lane (g, s), packed to bf16
//                    C       lane (g, s), tile e, register r: d = 32s + 8r + e
//   plus one more MFMA with A = ones whose result is the softmax denominator (the sum of
//   the bf16-rounded weights, already reduced over all 32 rows).
//
// The softmax reference m is lazy: scores are exponentiated relative to a per-head
// reference that is only raised (with a rescale of the accumulators) when some score
// exceeds it by more than 2^16; fp32 and bf16 carry that range without loss, so the
// common chunk needs no cross-lane traffic at all.
//
// A second small kernel combines the splits of each head and writes bf16.
#include <limits.h>

#include "attend_deal.h"
#include "kvzap_internal.h"

namespace kvzap {
namespace {

using deal::Deal;

constexpr int kD = 128;                 // head dimension (elements)
constexpr int kChunkRows = 32;
constexpr float kLazyMargin = 16.0f;    // log2 units

// Rows of one head: packed prefix [0, n_p) at row offset `off`, ring [0, n_r).
struct HeadExtent {
  int64_t off;
  int n_p, n_r;
};

// Contiguous layout: head bh owns rows row_offsets[bh] .. of a store of cap_rows rows.
// Paged layout (row_offsets == nullptr): its rows are addressed through its block table and
// cap_rows is what the table can address (max_pages * page_rows, 0 for an empty pool).
__device__ __forceinline__ HeadExtent head_extent(const int64_t* row_offsets,
                                                  const int32_t* lengths,
                                                  const int32_t* seq_pos, int window,
                                                  int64_t cap_rows, int bh, int b, const void* stand_in) {
  // one trip to memory: what is absent is read from `stand_in` (8 bytes) and discarded, since a load
  // behind a branch waits for the ones before it
  const int64_t off = *(row_offsets ? row_offsets + bh : static_cast<const int64_t*>(stand_in));
  const int32_t pos = *(window > 0 ? seq_pos + b : static_cast<const int32_t*>(stand_in));
  HeadExtent e;
  e.off = row_offsets ? off : 0;
  int64_t n = lengths[bh];
  if (e.off < 0 || e.off > cap_rows) { e.off = 0; n = 0; }
  if (n < 0) n = 0;
  if (n > cap_rows - e.off) n = cap_rows - e.off;
  e.n_p = (int)n;
  int r = 0;
  if (window > 0) {
    r = pos;
    r = r < 0 ? 0 : (r > window ? window : r);
  }
  e.n_r = r;
  return e;
}

__device__ __forceinline__ int chunks_of(int rows) { return (rows + kChunkRows - 1) / kChunkRows; }

struct Chunk {
  u32x4 k[8];      // operand layout: [4*t + kk] of set t; streamed: [row group j], as v
  u32x4 v[8];      // [row group j]: piece l%16 of row 4j + l/16
};

// Where the rows of one head live.
struct Source {
  const u32x4* K;            // packed rows of this head (contiguous) or the page pool (paged)
  const u32x4* V;
  const u32x4* Kr;           // ring rows of this head
  const u32x4* Vr;
  const int32_t* pages;      // paged: this head's block-table row
  int log_page, max_pages, num_pages;
  int n_p, n_r;
};

constexpr int kRowVec = kD * 2 / 16;   // 16-byte pieces per row

// Paged prefix: the pool rows of kLookup consecutive chunks' 16-row halves, half i in lane i % 64
// of word i / 64.  Looked up all halves at a time: looked up chunk by chunk, the round trip of every
// entry stood ahead of the chunk's loads.  A table entry outside the pool is clamped into it, so nothing
// outside the pool is ever read.  A part of more than kLookup chunks (64 sequences of 4k..32k rows: 330)
// empties its two buffers for each lookup, which costs such a call 3.5 % over the contiguous layout (701 / 726 us).
constexpr int kLookup = 64;              // chunks
struct Rows {
  int row[2];
};
__device__ __forceinline__ Rows look_up(const Source& s, int chunk0, int lane) {
  Rows w;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int r = chunk0 * kChunkRows + (i * 64 + lane) * 16;
    r = r < s.n_p ? r : (s.n_p > 0 ? s.n_p - 1 : 0);
    int slot = r >> s.log_page;
    slot = slot < s.max_pages - 1 ? slot : s.max_pages - 1;
    int page = s.pages[slot];
    page = page < 0 ? 0 : (page < s.num_pages ? page : s.num_pages - 1);
    w.row[i] = (page << s.log_page) + (r & ((1 << s.log_page) - 1));
  }
  return w;
}

// Where chunk `vc` of the head's chunk list (prefix chunks, then ring chunks) is.  Its 16-row
// halves are each contiguous because a page holds a multiple of 16 rows.  Rows past the end of the
// segment are read from its last row (their weights are forced to zero), so a half that starts
// past it is that row alone.
struct Place {
  bool ring;
  int row0, n_seg;
  size_t half[2];    // first row of each half, in 16-byte pieces from the store, the pool or the ring
};
template <bool kPaged>
__device__ __forceinline__ Place place_of(int vc, int cp, const Source& s, const Rows& rows, int chunk0) {
  Place p;
  p.ring = vc >= cp;
  p.n_seg = p.ring ? s.n_r : s.n_p;
  p.row0 = (p.ring ? vc - cp : vc) * kChunkRows;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int r = p.row0 + 16 * t < p.n_seg ? p.row0 + 16 * t : p.n_seg - 1;
    if (kPaged) {
      const int i = (2 * (vc - chunk0) + t) & 63;
      const int lo = __builtin_amdgcn_readlane(rows.row[0], i), hi = __builtin_amdgcn_readlane(rows.row[1], i);
      const int pool = vc - chunk0 < kLookup / 2 ? lo : hi;
      r = p.ring ? r : pool;
    }
    p.half[t] = (size_t)r * kRowVec;
  }
  return p;
}

// kStream: every load takes four whole rows with the non-temporal hint, K as well (to be turned in LDS).
// Otherwise plain loads, K's in the operand layout: [4*t + kk] of the chunk's set t.
template <bool kStream>
__device__ __forceinline__ void load_chunk(Chunk& c, const Place& p, const Source& s, int li, int lg) {
  const u32x4* Kb = p.ring ? s.Kr : s.K;
  const u32x4* Vb = p.ring ? s.Vr : s.V;
  const bool whole = p.row0 + kChunkRows <= p.n_seg;
  auto at = [&](int t, int r) {                            // piece 0 of row r of half t
    if (!whole) {
      int lim = p.n_seg - 1 - (p.row0 + 16 * t);           // last row of the segment, within the half
      lim = lim < 0 ? 0 : lim;
      r = r < lim ? r : lim;
    }
    return p.half[t] + (size_t)r * kRowVec;
  };
  if constexpr (kStream) {
    if (whole) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        c.k[j] = __builtin_nontemporal_load(Kb + p.half[j >> 2] + (size_t)(4 * (j & 3) + lg) * kRowVec + li);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        c.v[j] = __builtin_nontemporal_load(Vb + p.half[j >> 2] + (size_t)(4 * (j & 3) + lg) * kRowVec + li);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const size_t row = at(j >> 2, 4 * (j & 3) + lg) + li;
        c.k[j] = __builtin_nontemporal_load(Kb + row);
        c.v[j] = __builtin_nontemporal_load(Vb + row);
      }
    }
  } else {
    const int klocal = 4 * (li & 3) + (li >> 2);           // row of this lane inside a 16-row set
    if (whole) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) c.k[4 * t + kk] = Kb[p.half[t] + klocal * kRowVec + lg + kk * 4];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        c.v[j] = Vb[p.half[j >> 2] + (size_t)(4 * (j & 3) + lg) * kRowVec + li];
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const size_t row = at(t, klocal) + lg;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) c.k[4 * t + kk] = Kb[row + kk * 4];
#pragma unroll
        for (int j = 0; j < 4; ++j) c.v[4 * t + j] = Vb[at(t, 4 * j + lg) + li];
      }
    }
  }
}

struct Accum {
  floatx4 o[8];    // [d-tile e][r]: d = 32s + 8r + e
  floatx4 l;       // every register: sum of the weights of head g
  float m;         // reference exponent of head g (scaled log2 units)
};

__device__ __forceinline__ float shfl_xor_f(float x, int mask) {
  return __shfl_xor(x, mask, 64);
}

// turn: 8 KB of LDS of the wavefront's own, where the chunk was streamed
template <bool kStream>
__device__ __forceinline__ void consume_chunk(const Chunk& c, const u32x4 (&qb)[4], Accum& a, u32x4* turn,
                                              int row0, int n_seg, int li, int lg, float cscale) {
  if constexpr (kStream) {
    wave_fence();                                        // the reads of the chunk before
#pragma unroll
    for (int j = 0; j < 8; ++j) turn[(4 * j + lg) * kRowVec + (li ^ ((4 * j + lg) & 15))] = c.k[j];
    wave_fence();
  }
  floatx4 s[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    s[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int row = 4 * (li & 3) + (li >> 2);            // of this lane in the 16-row set
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      u32x4 k;
      if constexpr (kStream) k = turn[(16 * t + row) * kRowVec + ((4 * kk + lg) ^ row)];
      else k = c.k[4 * t + kk];
      s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k),
                                                     __builtin_bit_cast(bf16x8, qb[kk]), s[t],
                                                     0, 0, 0);
    }
  }
  float x[8];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) x[4 * t + r] = s[t][r] * cscale;
  if (row0 + kChunkRows > n_seg) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (row0 + 4 * j + lg >= n_seg) x[j] = -INFINITY;
  }
  float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                   fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
  if (__any(mx > a.m + kLazyMargin)) {
    // raise the reference to the exact running maximum of each head and rescale
    float mn = fmaxf(mx, shfl_xor_f(mx, 16));
    mn = fmaxf(mn, shfl_xor_f(mn, 32));
    mn = fmaxf(mn, a.m);
    const float alpha = __builtin_amdgcn_exp2f(a.m - mn);   // 0 when a.m = -inf
#pragma unroll
    for (int e = 0; e < 8; ++e) a.o[e] *= alpha;
    a.l *= alpha;
    a.m = mn;
  }
  bf16x8 p;
#pragma unroll
  for (int j = 0; j < 8; ++j) p[j] = (__bf16)__builtin_amdgcn_exp2f(x[j] - a.m);

  constexpr unsigned kSelLo = 0x05040100u, kSelHi = 0x07060302u;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    u32x4 vt;
#pragma unroll
    for (int jp = 0; jp < 4; ++jp)
      vt[jp] = __builtin_amdgcn_perm(c.v[2 * jp + 1][e >> 1], c.v[2 * jp][e >> 1],
                                     (e & 1) ? kSelHi : kSelLo);
    a.o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt), p, a.o[e],
                                                     0, 0, 0);
  }
  const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  a.l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones), p, a.l, 0, 0, 0);
}

// What the first pass's kernels are given.  Contiguous layout: K_rows/V_rows are the row store,
// row_offsets the heads' first rows.  Paged layout: K_rows/V_rows are the page pool, row_offsets is
// null, block_table given.  part: [slot][G][128] fp32, ml: [slot][G][2] fp32.
struct Args {
  const u32x4* q; const u32x4* K_rows; const u32x4* V_rows;
  int64_t cap_rows;
  const int64_t* row_offsets; const int32_t* block_table;
  int max_pages, log_page, num_pages;
  const int32_t* lengths; const u32x4* K_ring; const u32x4* V_ring; const int32_t* seq_pos;
  int window;
  float cscale;
  int BH, H, G;
  float* part; float* ml;
};

// Chunks [c0, c1) of head bh, whose sums go to `slot`.
template <bool kPaged, bool kStream>
__device__ __forceinline__ void attend_segment(const Args& a, const HeadExtent& e, int bh, int cp, int c0, int c1,
                                               int slot, u32x4* turn, int lane) {
  const int li = lane & 15, lg = lane >> 4;
  Source src;
  src.K = a.K_rows + (size_t)e.off * kRowVec;
  src.V = a.V_rows + (size_t)e.off * kRowVec;
  src.Kr = a.K_ring + (size_t)bh * (a.window > 0 ? a.window : 0) * kRowVec;
  src.Vr = a.V_ring + (size_t)bh * (a.window > 0 ? a.window : 0) * kRowVec;
  src.pages = kPaged ? a.block_table + (size_t)bh * a.max_pages : nullptr;
  src.log_page = a.log_page; src.max_pages = a.max_pages; src.num_pages = a.num_pages;
  src.n_p = e.n_p; src.n_r = e.n_r;

  // q as the B operand: lane (g = li, kg = lg), k-step kk: q[g][32kk + 8kg ..+8]
  u32x4 qb[4];
  {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const u32x4* qp = a.q + ((size_t)bh * a.G + (li < a.G ? li : 0)) * kRowVec + lg;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qb[kk] = li < a.G ? qp[kk * 4] : zero;
  }

  Accum acc;
#pragma unroll
  for (int t = 0; t < 8; ++t) acc.o[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  acc.l = floatx4{0.f, 0.f, 0.f, 0.f};
  acc.m = -INFINITY;

  // Two chunk buffers; the steady-state loop has no branch around a load, so the
  // compiler's wait counts let the loads of one buffer fly while the other is consumed.
  Chunk ca, cb;
  Rows rows{};
  for (int chunk0 = c0; chunk0 < c1; chunk0 += kLookup) {
    const int end = kPaged && chunk0 + kLookup < c1 ? chunk0 + kLookup : c1;
    if (kPaged) rows = look_up(src, chunk0, lane);
    auto place = [&](int vc) { return place_of<kPaged>(vc, cp, src, rows, chunk0); };
    auto load = [&](Chunk& c, const Place& p) { load_chunk<kStream>(c, p, src, li, lg); };
    auto consume = [&](const Chunk& c, const Place& p) {
      consume_chunk<kStream>(c, qb, acc, turn, p.row0, p.n_seg, li, lg, a.cscale);
    };
    Place pa = place(chunk0), pb;
    load(ca, pa);
    int vc = chunk0;
    while (vc + 2 < end) {
      pb = place(vc + 1);
      load(cb, pb);
      consume(ca, pa);
      pa = place(vc + 2);
      load(ca, pa);
      consume(cb, pb);
      vc += 2;
    }
    if (vc + 1 < end) {
      pb = place(vc + 1);
      load(cb, pb);
      consume(ca, pa);
      consume(cb, pb);
    } else {
      consume(ca, pa);
    }
    if (!kPaged) break;
  }

  if (li < a.G) {
    const size_t out = (size_t)slot * a.G + li;
    float* dst = a.part + out * kD + 32 * lg;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      floatx4 lo = {acc.o[0][r], acc.o[1][r], acc.o[2][r], acc.o[3][r]};
      floatx4 hi = {acc.o[4][r], acc.o[5][r], acc.o[6][r], acc.o[7][r]};
      *reinterpret_cast<floatx4*>(dst + 8 * r) = lo;
      *reinterpret_cast<floatx4*>(dst + 8 * r + 4) = hi;
    }
    if (lg == 0) {
      a.ml[out * 2] = acc.m;
      a.ml[out * 2 + 1] = acc.l[0];
    }
  }
}

// ---- pass 1, head by head: grid (B*H, splits), 64 threads, one split of spc chunks each ----
// The head varies fastest and is shifted by one from split to split: workgroups go to the eight XCDs in
// turn, so the blocks that have work (short heads: the first splits only) come one after the other on all
// of them, and a long head's splits meet every XCD.  Slot head * NS + split.
// Streamed, with K turned in LDS, it is 1 us longer from start to end than without (more to fetch of the
// program, and K's way through LDS), which the smallest steps do not make up for.
template <bool kPaged, bool kStream>
__global__ __launch_bounds__(64, 2) void attend_split_kernel(Args a, int NS, int spc) {
  __shared__ u32x4 s_turn[kStream ? kChunkRows * kRowVec : 1];
  const int split = blockIdx.y + gridDim.y * blockIdx.z;
  if (split >= NS) return;
  const int bh = (int)((blockIdx.x + (unsigned)split) % (unsigned)a.BH);
  const HeadExtent e = head_extent(a.row_offsets, a.lengths, a.seq_pos, a.window, a.cap_rows, bh, bh / a.H, a.q);
  const int cp = chunks_of(e.n_p), ct = cp + chunks_of(e.n_r);
  const int c0 = split * spc;
  // the last split runs to the end of the list, so a head longer than the host's bound
  // is still covered
  const int c1 = split == NS - 1 ? ct : (ct - c0 < spc ? ct : c0 + spc);
  if (c0 >= c1) return;
  attend_segment<kPaged, kStream>(a, e, bh, cp, c0, c1, bh * NS + split, s_turn, threadIdx.x);
}

// ---- pass 1, as one list: grid ceil(nw / waves), streamed ----
// The chunks of all heads, in (b,h) order and each head's prefix before its ring, are one list, and
// each of the nw wavefronts takes an equal part of it: every CU of every XCD reads the same number of
// bytes whatever the heads' lengths are, and all of them end together.  (Cutting every head into
// splits of the same length and handing those out one per wavefront left the XCDs up to 4 % apart and
// paid a wavefront's start for every split: 64 sequences of 4k..32k rows 776 us with splits of 2048
// rows, 815 with 1024, 850 with 512.)
// A block adds up the chunk counts of all heads itself, up to 64 heads a wavefront does.  The part of a
// head that a wavefront handles (a segment) leaves its sums in slot (wavefront + head), which grows from
// segment to segment; span[head] = the first and the last slot of the head, written by the wavefronts
// that hold its ends.
constexpr int kMaxBatches = 1024;        // of 64 heads: B*H <= 65535
constexpr int waves_of(Deal d) { return d == Deal::kBlock ? 4 : 1; }

template <bool kPaged, Deal kDeal>
__global__ __launch_bounds__(waves_of(kDeal) * 64, 2) void attend_list_kernel(Args a, int nw, int2* span) {
  constexpr int kWaves = waves_of(kDeal);
  __shared__ u32x4 s_turn[kWaves][kChunkRows * kRowVec];
  __shared__ int s_batch[kDeal == Deal::kBlock ? kMaxBatches : 1];
  const int tid = threadIdx.x, lane = tid & 63, BH = a.BH;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

  HeadExtent mine;                                       // lane i: head base + i
  int base = 0, chunks;                                  // chunks of that head
  auto extent = [&](int bh) {                            // past the last head: nothing, and no branch around a load
    const int c = bh < BH ? bh : BH - 1;
    HeadExtent e = head_extent(a.row_offsets, a.lengths, a.seq_pos, a.window, a.cap_rows, c, c / a.H, a.q);
    if (bh >= BH) e.n_p = e.n_r = 0;
    return e;
  };
  auto fetch = [&]() {
    mine = extent(base + lane);
    chunks = chunks_of(mine.n_p) + chunks_of(mine.n_r);
  };
  // this wavefront's part of the list; where a third and more have none, those that have are spread over the blocks
  // (16 sequences of 64 rows under a bound of 6208 14.7 -> 12.7 us a call)
  int w = 0, begin = 0, left = 0;
  auto part_of = [&](int total) {
    w = 3ll * total < 2ll * nw * deal::kMinChunks ? wv * (int)gridDim.x + (int)blockIdx.x : (int)blockIdx.x * kWaves + wv;
    const deal::Part part = deal::part_of(total, nw, w);
    begin = part.begin;
    left = part.n;
  };
  int skip;                                              // chunks ahead of `begin` from head `base` on
  if constexpr (kDeal == Deal::kWave) {
    fetch();
    part_of(__builtin_amdgcn_readlane(wave_scan(chunks), 63));
    if (left <= 0) return;
    skip = begin;
  } else {
    // the wavefronts add up 64 heads at a time, the loads of four batches in flight
    const int batches = (BH + 63) / 64;
    for (int i = wv; i < batches; i += 4 * kWaves) {
      int n[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const HeadExtent e = extent((i + u * kWaves) * 64 + lane);
        n[u] = chunks_of(e.n_p) + chunks_of(e.n_r);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int sum = wave_scan(n[u]);
        if (lane == 63 && i + u * kWaves < batches) s_batch[i + u * kWaves] = sum;
      }
    }
    __syncthreads();
    int total = 0;
    for (int i = 0; i < batches; i += 64)
      total += __builtin_amdgcn_readlane(wave_scan(i + lane < batches ? s_batch[i + lane] : 0), 63);
    part_of(total);
    if (left <= 0) return;
    // the batches that end at or before `begin` are passed over
    int passed = 0;
    skip = begin;
    for (int i = 0; i < batches; i += 64) {
      const int upto = wave_scan(i + lane < batches ? s_batch[i + lane] : 0);
      const unsigned long long done = __ballot(upto <= skip);
      if (!done) break;
      passed = i + __popcll(done);
      skip -= __builtin_amdgcn_readlane(upto, 63 - __builtin_clzll(done));
      if (~done) break;
    }
    base = passed * 64;
    fetch();
  }
  int at = 0;                                            // the wavefront's head is base + at
  for (;;) {
    const int upto = wave_scan(chunks);
    const unsigned long long past = __ballot(upto > skip);
    if (past) {
      at = __builtin_ctzll(past);
      skip -= __builtin_amdgcn_readlane(upto - chunks, at);
      break;
    }
    skip -= __builtin_amdgcn_readlane(upto, 63);
    base += 64;
    if (base >= BH) return;                              // (never: begin < total)
    fetch();
  }

  u32x4* const turn = s_turn[wv];
  int first = skip;                                      // its chunk of that head
  for (;;) {
    at = __builtin_amdgcn_readfirstlane(at);
    const int bh = base + at;
    HeadExtent e;
    e.n_p = __builtin_amdgcn_readlane(mine.n_p, at);
    e.n_r = __builtin_amdgcn_readlane(mine.n_r, at);
    e.off = (int64_t)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(mine.off >> 32), at) << 32) |
                      (unsigned)__builtin_amdgcn_readlane((int)mine.off, at));
    const int cp = chunks_of(e.n_p), ct = cp + chunks_of(e.n_r);
    const int c0 = __builtin_amdgcn_readfirstlane(first);
    const int c1 = __builtin_amdgcn_readfirstlane(ct - c0 < left ? ct : c0 + left);
    const int slot = w + bh;
    attend_segment<kPaged, true>(a, e, bh, cp, c0, c1, slot, turn, lane);
    if (lane == 0) {
      if (c0 == 0) span[bh].x = slot;
      if (c1 == ct) span[bh].y = slot;
    }
    left -= c1 - c0;
    if (left <= 0) return;
    // the next head that has chunks: there is one, `left` of the list are still ahead
    unsigned long long more = __ballot(chunks > 0) & (at < 63 ? ~0ull << (at + 1) : 0ull);
    while (!more) {
      base += 64;
      if (base >= BH) return;
      fetch();
      more = __ballot(chunks > 0);
    }
    at = __builtin_ctzll(more);
    first = 0;
  }
}

// ---- pass 2: grid B*H*G, kGroups * 32 threads: thread (c = tid%32, sg = tid/32) folds the slots
// sg, sg + kGroups, ... of output elements 4c..4c+3 with a running reference, then the groups meet
// in LDS.  span: of a list; null where a head has NS slots, one for each spc chunks.
template <int kGroups>
__global__ __launch_bounds__(kGroups * 32) void attend_combine_kernel(
    const float* part, const float* ml, const int2* span, int NS, int spc, int64_t total_rows,
    const int64_t* row_offsets, const int32_t* lengths, const int32_t* seq_pos, int window, int H, int G,
    unsigned short* out) {
  __shared__ floatx4 s_num[kGroups][32];
  __shared__ float s_m[kGroups], s_den[kGroups];
  const int bh = blockIdx.x / G, g = blockIdx.x % G;
  const int c = threadIdx.x & 31, sg = threadIdx.x >> 5;
  int2 slots = *(span ? span + bh : reinterpret_cast<const int2*>(part));
  const HeadExtent e = head_extent(row_offsets, lengths, seq_pos, window, total_rows, bh, bh / H, part);
  const int ct = chunks_of(e.n_p) + chunks_of(e.n_r);
  int ns;
  if (span) {
    ns = ct > 0 ? slots.y - slots.x + 1 : 0;             // of an empty head nobody wrote the span
  } else {
    slots.x = bh * NS;
    ns = (ct + spc - 1) / spc;
    ns = ns < NS ? ns : NS;
  }
  float m = -INFINITY, den = 0.f;
  floatx4 num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = sg; s < ns; s += kGroups) {
    const size_t slot = (size_t)(slots.x + s) * G + g;
    const float ms = ml[slot * 2], ls = ml[slot * 2 + 1];
    const floatx4 a = *reinterpret_cast<const floatx4*>(part + slot * kD + 4 * c);
    const float mn = fmaxf(m, ms);
    const float w_old = __builtin_amdgcn_exp2f(m - mn), w_new = __builtin_amdgcn_exp2f(ms - mn);
    num = num * w_old + a * w_new;
    den = den * w_old + ls * w_new;
    m = mn;
  }
  s_num[sg][c] = num;
  if (c == 0) { s_m[sg] = m; s_den[sg] = den; }
  __syncthreads();
  if (sg == 0) {
    float mm = s_m[0];
#pragma unroll
    for (int k = 1; k < kGroups; ++k) mm = fmaxf(mm, s_m[k]);
    floatx4 n = {0.f, 0.f, 0.f, 0.f};
    float dsum = 0.f;
#pragma unroll
    for (int k = 0; k < kGroups; ++k) {
      // a group that saw no split has m = -inf and zero sums; exp2(-inf - mm) = 0 unless
      // mm is -inf too (no split at all), which the ns > 0 test below covers
      const float w = (s_m[k] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(s_m[k] - mm);
      n += s_num[k][c] * w;
      dsum += s_den[k] * w;
    }
    unsigned short* o = out + (size_t)blockIdx.x * kD + 4 * c;
    typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
    u16x4 r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = float_to_bf16_bits(ns > 0 ? n[k] / dsum : 0.f);
    *reinterpret_cast<u16x4*>(o) = r;
  }
}

long long bound_chunks(int max_rows, int window) {
  return ((long long)max_rows + kChunkRows - 1) / kChunkRows + ((long long)window + kChunkRows - 1) / kChunkRows;
}

struct Layout {
  size_t ml, span, bytes;                // of the workspace: sums, then references and denominators, then spans
};
Layout layout_of(int BH, int G, long long ct) {
  const size_t slots = (size_t)deal::slots_of(BH, ct) * G;
  Layout l;
  l.ml = align_up(slots * kD * sizeof(float), 256);
  l.span = l.ml + align_up(slots * 2 * sizeof(float), 256);
  l.bytes = l.span + align_up((size_t)BH * sizeof(int2), 256);
  return l;
}
}  // namespace

size_t attend_workspace_bytes(int B, int H, int HQ, int max_rows, int window) {
  return layout_of(B * H, HQ / H, bound_chunks(max_rows, window)).bytes;
}

int launch_attend_decode(const void* q, const void* K_rows, const void* V_rows,
                         int64_t total_rows, const int64_t* row_offsets,
                         const int32_t* block_table, int max_pages, int page_rows, int num_pages,
                         const int32_t* lengths, const void* K_ring, const void* V_ring,
                         const int32_t* seq_pos, int window, int max_rows, float scale,
                         void* out, int B, int H, int HQ, void* workspace,
                         hipStream_t stream) {
  const int G = HQ / H, BH = B * H;
  const long long ct = bound_chunks(max_rows, window);
  const Layout lay = layout_of(BH, G, ct);
  char* const ws = static_cast<char*>(workspace);
  float* part = reinterpret_cast<float*>(ws);
  float* ml = reinterpret_cast<float*>(ws + lay.ml);
  int2* span = reinterpret_cast<int2*>(ws + lay.span);
  const float cscale = scale * 1.4426950408889634f;
  const bool paged = block_table != nullptr;
  int log_page = 0;
  while ((1 << log_page) < page_rows) ++log_page;
  // rows a head can address: the whole store, or what its block-table row covers
  const int64_t cap_rows = paged ? (num_pages > 0 ? (int64_t)max_pages * page_rows : 0) : total_rows;
  const int most_rows = (int)(cap_rows < INT_MAX ? cap_rows : INT_MAX);   // of a head: lengths are 32-bit
  const deal::Dealt dealt = deal::deal_of(BH, G, ct, BH * bound_chunks(most_rows, window));
  const Args args{static_cast<const u32x4*>(q), static_cast<const u32x4*>(K_rows), static_cast<const u32x4*>(V_rows), cap_rows,
                  paged ? nullptr : row_offsets, block_table, max_pages, log_page, num_pages, lengths,
                  static_cast<const u32x4*>(K_ring), static_cast<const u32x4*>(V_ring), seq_pos, window, cscale,
                  BH, H, G, part, ml};
  const int NS = dealt.nw / BH;
  if (dealt.deal == Deal::kHead) {
    const unsigned ny = NS < 65535 ? NS : 65535;
    const dim3 grid(BH, ny, (NS + ny - 1) / ny);
    auto launch = [&](auto kernel) { kernel<<<grid, 64, 0, stream>>>(args, NS, dealt.spc); };
    if (dealt.stream) launch(paged ? attend_split_kernel<true, true> : attend_split_kernel<false, true>);
    else launch(paged ? attend_split_kernel<true, false> : attend_split_kernel<false, false>);
    span = nullptr;
  } else {
    const int waves = waves_of(dealt.deal), blocks = (dealt.nw + waves - 1) / waves;
    auto launch = [&](auto kernel) { kernel<<<blocks, waves * 64, 0, stream>>>(args, dealt.nw, span); };
    if (dealt.deal == Deal::kWave) launch(paged ? attend_list_kernel<true, Deal::kWave> : attend_list_kernel<false, Deal::kWave>);
    else launch(paged ? attend_list_kernel<true, Deal::kBlock> : attend_list_kernel<false, Deal::kBlock>);
  }
  if (hipGetLastError() != hipSuccess) return KVZAP_ERR_RUNTIME;
  const int64_t* offsets = paged ? nullptr : row_offsets;
  auto* bits = static_cast<unsigned short*>(out);
  auto combine = [&](auto kernel, int groups) {
    kernel<<<BH * G, groups * 32, 0, stream>>>(part, ml, span, NS, dealt.spc, cap_rows, offsets, lengths, seq_pos, window,
                                               H, G, bits);
  };
  // By the slots that a head can have.  In a list one head may have them all (8 sequences, one head of 60000 rows and 63 of
  // 200: 20.8 us with 8 groups, 17.6 with 16), but past 64 heads the wider blocks cost the usual call more than they
  // give that one (40 sequences of 0.3k..2.4k rows 45.0 / 46.3); one KV head's hundreds took 24 us with 8.
  if (NS > 128) combine(attend_combine_kernel<32>, 32);
  else if (NS > 64 || dealt.deal == Deal::kWave) combine(attend_combine_kernel<16>, 16);
  else combine(attend_combine_kernel<8>, 8);
  if (hipGetLastError() != hipSuccess) return KVZAP_ERR_RUNTIME;
  return KVZAP_OK;
}

}  // namespace kvzap
