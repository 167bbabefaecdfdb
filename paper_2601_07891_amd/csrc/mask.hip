// Threshold + sliding-window mask and per-head index lists (Sec. 3.3, Algorithm 1).
//
// Small launches over scores [B*H, T] (4 bytes per flag, so the whole stage moves
// ~1 % of the bytes of the K/V compaction that follows; it is bound by the ~4 us
// floor of a kernel launch, so the number of launches is what matters):
//   1. count : one block per 1024-token chunk of one (b,h) row counts its kept flags
//   2. emit  : every chunk recomputes its flags (scores are L2-resident by now),
//              ranks them with a wave shuffle scan + LDS and writes the ascending
//              kept positions at its prefix.  With up to kFusedMaxChunks chunks each
//              block derives its own prefix by summing the counts of all chunks
//              before it (a few KB from L2), and the first chunk of every head
//              also writes lengths and offsets; beyond that a single-block scan
//              kernel runs between the two.
// Short inputs take one launch instead (mask_direct_kernel), the gather included.
// No block waits for another, so there is nothing that can spin.
#include <mutex>

#include "kvzap_internal.h"

namespace kvzap {
namespace {

// Scratch of the allocation-free entry point (kvzap_mask_static): the chunk counts and chunk
// prefixes that kvzap_mask keeps in its caller's workspace, for up to kStaticMaskChunks
// 1024-token chunks.  One copy per GPU, at its own address on each, held until the process
// ends; every call on a GPU shares it, so calls that overlap on one GPU race.  Nothing in it
// has to start at zero: the count kernel writes every entry the later kernels read.
constexpr size_t kStaticCountBytes = (size_t)kStaticMaskChunks * sizeof(int32_t);
constexpr size_t kStaticScratchBytes = kStaticCountBytes + (size_t)kStaticMaskChunks * sizeof(int64_t);
static_assert(kStaticCountBytes % 256 == 0, "the prefix part stays 256-byte aligned");
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// In host code `scratch` is only a stand-in for the symbol, not a device address: the address
// on the current GPU is looked up once per device and kept here.
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void* scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KVZAP_ERR_RUNTIME;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return KVZAP_ERR_RUNTIME;
    }
    scratch_ptr[dev] = p;
  }
  *out = scratch_ptr[dev];
  return KVZAP_OK;
}

constexpr int kThreads = 256;            // 4 wavefronts
constexpr int kPerThread = kMaskChunk / kThreads;  // 4 consecutive tokens
static_assert(kPerThread == 4, "one float4 per thread");

// A sequence's own length, clamped into [0, T]: positions at or beyond T do not exist whatever
// the caller's array says (it lives on the device, so the host cannot reject it)
__device__ __forceinline__ int seq_len_of(const int32_t* __restrict__ seq_lens, int b, int T) {
  if (!seq_lens) return T;
  const int n = seq_lens[b];
  return n < 0 ? 0 : (n > T ? T : n);
}

// keep flags of tokens t0..t0+3 of one (b,h) row
__device__ __forceinline__ unsigned keep_bits4(const float* __restrict__ row, int t0, int T,
                                               int Tb, int window, float tau, bool vec_ok) {
  float s[4];
  if (vec_ok && t0 + 3 < T) {
    const floatx4 v = *reinterpret_cast<const floatx4*>(row + t0);
    s[0] = v.x; s[1] = v.y; s[2] = v.z; s[3] = v.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = (t0 + e < T) ? row[t0 + e] : 0.0f;
  }
  const int first_protected = Tb - window;   // may be negative: everything protected
  unsigned bits = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int t = t0 + e;
    const bool keep = (t < Tb) && ((t >= first_protected) || (s[e] >= tau));
    bits |= (keep ? 1u : 0u) << e;
  }
  return bits;
}

__global__ __launch_bounds__(kThreads) void mask_count_kernel(
    const float* __restrict__ scores, float tau_all, const float* __restrict__ tau_head, int window,
    const int32_t* __restrict__ seq_lens, int H, int T, int nchunks,
    int32_t* __restrict__ chunk_counts) {
  const int chunk = blockIdx.x, bh = blockIdx.y;
  const float tau = tau_head ? tau_head[bh] : tau_all;     // one threshold, or one per head
  const int Tb = seq_len_of(seq_lens, bh / H, T);
  const float* row = scores + (size_t)bh * T;
  const bool vec_ok = (T % 4) == 0;
  const int t0 = chunk * kMaskChunk + threadIdx.x * kPerThread;
  const int v = wave_scan(__popc(keep_bits4(row, t0, T, Tb, window, tau, vec_ok)));
  __shared__ int wave_sum[kThreads / 64];
  if ((threadIdx.x & 63) == 63) wave_sum[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) tot += wave_sum[w];
    chunk_counts[(size_t)bh * nchunks + chunk] = tot;
  }
}

constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void mask_scan_kernel(
    const int32_t* __restrict__ chunk_counts, int64_t* chunk_prefix,
    int BH, int nchunks, int32_t* __restrict__ lengths, int64_t* __restrict__ offsets) {
  __shared__ long long wave_tot[kScanThreads / 64];
  __shared__ long long carry_s;
  const int n = BH * nchunks;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (int base = 0; base < n; base += kScanThreads) {
    const int i = base + threadIdx.x;
    const long long v = (i < n) ? (long long)chunk_counts[i] : 0;
    long long incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const long long up = __shfl_up(incl, off, 64);
      if (lane >= off) incl += up;
    }
    if (lane == 63) wave_tot[wid] = incl;
    __syncthreads();
    long long before = carry_s;
    for (int w = 0; w < wid; ++w) before += wave_tot[w];
    if (i < n) chunk_prefix[i] = before + incl - v;
    __syncthreads();
    if (threadIdx.x == kScanThreads - 1) carry_s = before + incl;
    __syncthreads();
  }
  // head starts: the prefix of a head's first chunk; written by this block above
  __threadfence_block();
  __syncthreads();
  for (int bh = threadIdx.x; bh <= BH; bh += kScanThreads) {
    const long long start = (bh < BH) ? chunk_prefix[(size_t)bh * nchunks] : carry_s;
    offsets[bh] = start;
    if (bh < BH) {
      const long long end = (bh + 1 < BH) ? chunk_prefix[(size_t)(bh + 1) * nchunks] : carry_s;
      lengths[bh] = (int32_t)(end - start);
    }
  }
}

constexpr int kFusedMaxChunks = 8192;

// The kernel is a chain of memory round trips: the scores and the counts are loaded side by side, the
// counts four to a load (one by one, the last of 1024 chunks made four dependent trips), and both of a
// head's sums meet at one barrier.  Mask and gather of 8 x 131072 scores 52.9 -> 51.5 us.
template <bool kFused>
__global__ __launch_bounds__(kThreads) void mask_emit_kernel(
    const float* __restrict__ scores, float tau_all, const float* __restrict__ tau_head, int window,
    const int32_t* __restrict__ seq_lens, int H, int T, int nchunks,
    const int64_t* __restrict__ chunk_prefix, const int32_t* __restrict__ chunk_counts,
    int32_t* __restrict__ keep_idx, int32_t* __restrict__ lengths,
    int64_t* __restrict__ offsets) {
  constexpr int kWaves = kThreads / 64;
  const int chunk = blockIdx.x, bh = blockIdx.y;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const float tau = tau_head ? tau_head[bh] : tau_all;
  const int Tb = seq_len_of(seq_lens, bh / H, T);
  const float* row = scores + (size_t)bh * T;
  const bool vec_ok = (T % 4) == 0;
  const int t0 = chunk * kMaskChunk + threadIdx.x * kPerThread;
  int64_t prefix = 0;                                      // kept ahead of this chunk
  int before = 0, own = 0;                                 // this thread's part of it; of the head's
  if (!kFused) prefix = chunk_prefix[(size_t)bh * nchunks + chunk];
  if (kFused) {
    // chunks are ordered (b,h)-major; the first chunk of a head adds up the head's as well.  The array
    // is padded to 256 bytes, so that four counts at a time stay inside it.
    const int mine = bh * nchunks + chunk, end = chunk == 0 ? mine + nchunks : mine;
    typedef int i32x4 __attribute__((ext_vector_type(4)));
#pragma unroll 2
    for (int i = threadIdx.x * 4; i < end; i += kThreads * 4) {
      const i32x4 n = *reinterpret_cast<const i32x4*>(chunk_counts + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        before += i + e < mine ? n[e] : 0;
        own += i + e >= mine && i + e < end ? n[e] : 0;
      }
    }
  }
  const unsigned bits = keep_bits4(row, t0, T, Tb, window, tau, vec_ok);
  const int c = __popc(bits), incl = wave_scan(c);
  __shared__ int s_before[kWaves], s_own[kWaves], s_kept[kWaves];
  before = kFused ? wave_scan(before) : 0;
  own = kFused && chunk == 0 ? wave_scan(own) : 0;         // (uniform)
  if (lane == 63) {
    s_kept[wid] = incl;
    if (kFused) {
      s_before[wid] = before;
      s_own[wid] = own;
    }
  }
  __syncthreads();
  int ahead = 0, head_total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (kFused) {
      prefix += s_before[w];
      head_total += s_own[w];
    }
    ahead += w < wid ? s_kept[w] : 0;
  }
  if (kFused && chunk == 0 && threadIdx.x == 0) {          // this head's length and start
    offsets[bh] = prefix;
    lengths[bh] = head_total;
    if (bh == (int)gridDim.y - 1) offsets[bh + 1] = prefix + head_total;
  }
  int64_t pos = prefix + ahead + incl - c;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (bits & (1u << e)) keep_idx[pos++] = t0 + e;
  }
}

// ---- short inputs: threshold, window and (kLpr > 0) the gather in one launch ----
// A chunk is kDirectChunk tokens of one (b,h) row.  Its block finds its own prefix by testing
// every score ahead of it in (b,h) order -- a few ten thousand floats from L2, which the whole
// block reads at once -- instead of waiting for a launch that counts them, and moves the rows
// it keeps as soon as it has ranked them.  Bound by launch and memory latency.
constexpr int kDirectThreads = 1024;
constexpr int kDirectWaves = kDirectThreads / 64;
constexpr int kDirectChunk = 128;
constexpr int kSegment = 1024;

struct GatherArgs {
  const u32x4* K; const u32x4* V; u32x4* K_out; u32x4* V_out;
  int64_t cap_rows;
};

// kLpr: 16-byte pieces of a K/V row; 0: no gather.  kEager: all rows of the chunk are loaded before it is
// known which are kept
template <int kLpr, bool kEager>
__global__ __launch_bounds__(kDirectThreads) void mask_direct_kernel(
    const float* __restrict__ scores, float tau_all, const float* __restrict__ tau_head, int window,
    const int32_t* __restrict__ seq_lens, int H, int T, int32_t* __restrict__ keep_idx,
    int32_t* __restrict__ lengths, int64_t* __restrict__ offsets, GatherArgs rows) {
  __shared__ int s_before[kDirectWaves], s_own[kDirectWaves], s_first;
  __shared__ int s_keep[kDirectChunk];                     // kept tokens; kEager: the tokens' ranks, -1: dropped
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int bh = blockIdx.y, t_begin = blockIdx.x * kDirectChunk;
  auto tau_of = [&](int row) { return tau_head ? tau_head[row] : tau_all; };
  constexpr int kRows = kLpr > 0 ? kDirectThreads / kLpr : 1;   // rows of one tensor per pass
  constexpr int kPasses = kEager ? kDirectChunk / kRows : 1;
  u32x4 k_row[kPasses], v_row[kPasses];
  if constexpr (kEager) {
#pragma unroll
    for (int u = 0; u < kPasses; ++u) {
      const int t = t_begin + tid / kLpr + u * kRows;
      const size_t from = ((size_t)bh * T + (t < T ? t : T - 1)) * kLpr + tid % kLpr;
      k_row[u] = __builtin_nontemporal_load(rows.K + from);
      v_row[u] = __builtin_nontemporal_load(rows.V + from);
    }
  }
  // this chunk's flags: one lane of the first two wavefronts per token
  bool own = false;
  const int t_mine = t_begin + tid;
  if (tid < kDirectChunk && t_mine < T) {
    const int Tb = seq_len_of(seq_lens, bh / H, T);
    own = t_mine < Tb && (t_mine >= Tb - window || scores[(size_t)bh * T + t_mine] >= tau_of(bh));
  }
  // What is kept ahead of it, in earlier rows and earlier in its own (a head's length is the
  // latter plus its last chunk).  The window's share of a row is known without reading; of the
  // rest a wavefront takes segments of 1024 positions, four 16-byte loads per lane at once, the
  // next segment's ahead of the current one's count.  Two vector operations per score: with a
  // row lookup and a window test per score this part took 20 us on 65536 scores.
  int before = 0, in_row = 0;
  {
    const int cpr = (T + kSegment - 1) / kSegment;
    const int nseg = bh * cpr + (t_begin + kSegment - 1) / kSegment;
    struct Segment { int lo, hi; float tau; int row; };      // linear positions to test
    auto segment = [&](int sg, floatx4 (&q)[4]) {
      Segment s;
      s.row = sg / cpr;
      const int c = sg - s.row * cpr, base = s.row * T;
      const int Tb = seq_len_of(seq_lens, s.row / H, T), end = s.row == bh ? t_begin : T;
      const int limit = Tb < end ? Tb : end;                 // positions that count
      int tested = Tb > window ? Tb - window : 0;            // of those, below the window
      if (tested > limit) tested = limit;
      if (c == 0 && lane == 0) {                             // (limit < tested: none)
        if (s.row == bh) in_row += limit - tested;
        else before += limit - tested;
      }
      s.lo = base + c * kSegment;
      s.hi = base + (tested < (c + 1) * kSegment ? tested : (c + 1) * kSegment);
      s.tau = tau_of(s.row);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = (s.lo & ~3) + (u * 64 + lane) * 4;
        if (i + 3 < s.hi) q[u] = *reinterpret_cast<const floatx4*>(scores + i);
        else
          for (int e = 0; e < 4; ++e) q[u][e] = i + e < s.hi ? scores[i + e] : 0.0f;
      }
      return s;
    };
    auto count = [&](const Segment& s, const floatx4 (&q)[4]) {
      int n = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = (s.lo & ~3) + (u * 64 + lane) * 4;
        if (i >= s.lo && i + 3 < s.hi) {
#pragma unroll
          for (int e = 0; e < 4; ++e) n += q[u][e] >= s.tau;
        } else {
          for (int e = 0; e < 4; ++e) n += i + e >= s.lo && i + e < s.hi && q[u][e] >= s.tau;
        }
      }
      // a row that starts off a 16-byte boundary: the segment's last one to three positions
      const int i = (s.lo & ~3) + 1024 + lane;
      if (i < s.lo + kSegment && i < s.hi) n += scores[i] >= s.tau;
      if (s.row == bh) in_row += n;
      else before += n;
    };
    floatx4 qa[4], qb[4];
    Segment sa, sb;
    int sg = wv;
    if (sg < nseg) sa = segment(sg, qa);
    for (; sg < nseg; sg += 2 * kDirectWaves) {
      if (sg + kDirectWaves < nseg) sb = segment(sg + kDirectWaves, qb);
      count(sa, qa);
      if (sg + 2 * kDirectWaves < nseg) sa = segment(sg + 2 * kDirectWaves, qa);
      if (sg + kDirectWaves < nseg) count(sb, qb);
    }
  }
  before = wave_scan(before);
  in_row = wave_scan(in_row);
  const unsigned long long kept = __ballot(own);
  if (lane == 63) { s_before[wv] = before; s_own[wv] = in_row; }
  if (tid == 0) s_first = __popcll(kept);
  __syncthreads();
  int start = 0, mine = 0;
#pragma unroll
  for (int w = 0; w < kDirectWaves; ++w) { start += s_before[w]; mine += s_own[w]; }
  const int first = s_first, out0 = start + mine;          // of this head; of this chunk
  const int rank = (wv ? first : 0) + __popcll(kept & ((1ull << lane) - 1));
  if (kEager && tid < kDirectChunk) s_keep[tid] = own ? rank : -1;
  if (own) {
    if (!kEager) s_keep[rank] = t_mine;
    keep_idx[out0 + rank] = t_mine;
  }
  const int count = __syncthreads_count(own);
  if (tid == 0) {
    if (blockIdx.x == 0) offsets[bh] = start;
    if (blockIdx.x == gridDim.x - 1) {
      lengths[bh] = mine + count;
      if (bh == (int)gridDim.y - 1) offsets[bh + 1] = out0 + count;
    }
  }
  if constexpr (kEager) {
#pragma unroll
    for (int u = 0; u < kPasses; ++u) {
      const int r = s_keep[tid / kLpr + u * kRows];
      if (r >= 0 && out0 + r < rows.cap_rows) {
        const size_t to = (size_t)(out0 + r) * kLpr + tid % kLpr;
        __builtin_nontemporal_store(k_row[u], rows.K_out + to);
        __builtin_nontemporal_store(v_row[u], rows.V_out + to);
      }
    }
  } else if constexpr (kLpr > 0) {
    const int piece = tid % kLpr;
    const size_t base = (size_t)bh * T * kLpr + piece;
#pragma unroll 4
    for (int j = tid / kLpr; j < count; j += kRows) {
      if (out0 + j >= rows.cap_rows) break;
      const size_t from = base + (size_t)s_keep[j] * kLpr, to = (size_t)(out0 + j) * kLpr + piece;
      const u32x4 k = __builtin_nontemporal_load(rows.K + from), v = __builtin_nontemporal_load(rows.V + from);
      __builtin_nontemporal_store(k, rows.K_out + to);
      __builtin_nontemporal_store(v, rows.V_out + to);
    }
  }
}

// Where one launch is the faster way.  Every block goes over all segments ahead of it, so its
// time grows with their number while count + emit stays at two launches.  Measured, us per call
// (direct / count + emit; with the gather of half the rows: direct / three launches), calls one by one:
//   8 rows of 1024: 4.9 / 7.8 (5.5 / 12.2)   of 2048: 5.0 / 8.2 (6.6 / 12.6)   of 4096 (32
//   segments): 5.9 / 8.2 (8.9 / 12.7)   of 8192 (64): 10.5 / 8.3 (15.6 / 14.8)
//   24 rows of 701: 5.7 / 8.1 (7.0 / 12.3)   128 rows of 512: 21 / 8.3 (25.7 / 18)
// and on a queue that is never empty, where a second launch costs less: 8 rows of 1024 4.0 / 5.6,
// of 4096 5.5 / 5.7, of 5120 (40 segments) 6.4 / 5.7, 40 rows of 1000 6.8 / 5.9; with the gather
// direct wins up to 40 segments there too.
constexpr long long kDirectSegments = 32, kDirectSegmentsGather = 40;

// With a block for every CU at most, the gather is another trip to memory behind the ranks, and reading all
// rows while the scores are tested takes it away, also where few are kept.  The rows' registers leave
// room for one block on a CU, so with more blocks than CUs it loses.  us per call (rows of kept tokens alone /
// all rows, 8 heads, half kept): 2048 x 128 7.6 / 6.8, 4096 x 128 (256 blocks) 9.1 / 8.4, 5000 x 128 (320)
// 11.2 / 13.7, 1024 x 256 9.0 / 7.3, 4096 x 256 13.0 / 11.3; a tenth kept: 4096 x 128 8.2 / 8.2, x 256 11.0 / 11.1.
constexpr long long kEagerBlocks = 256;

bool direct_fits(int B, int H, int T, long long limit) {
  return (long long)B * H * ((T + kSegment - 1) / kSegment) <= limit;
}

template <int kLpr, bool kEager = false>
int launch_direct(const float* scores, float tau, const float* tau_head, int window,
                  const int32_t* seq_lens, int B, int H, int T, int32_t* keep_idx, int32_t* lengths,
                  int64_t* offsets, const GatherArgs& rows, hipStream_t stream) {
  const dim3 grid((T + kDirectChunk - 1) / kDirectChunk, B * H);
  mask_direct_kernel<kLpr, kEager><<<grid, kDirectThreads, 0, stream>>>(scores, tau, tau_head, window, seq_lens, H, T,
                                                                keep_idx, lengths, offsets, rows);
  return hipGetLastError() == hipSuccess ? KVZAP_OK : KVZAP_ERR_RUNTIME;
}

}  // namespace

int launch_mask_compact(const float* scores, float tau, int window, const int32_t* seq_lens, int B,
                        int H, int T, int32_t* keep_idx, int32_t* lengths, int64_t* offsets,
                        const void* K, const void* V, void* K_out, void* V_out, int64_t cap_rows,
                        int D, void* workspace, hipStream_t stream) {
  if (direct_fits(B, H, T, kDirectSegmentsGather)) {
    const GatherArgs rows{static_cast<const u32x4*>(K), static_cast<const u32x4*>(V),
                          static_cast<u32x4*>(K_out), static_cast<u32x4*>(V_out), cap_rows};
    if ((long long)B * H * ((T + kDirectChunk - 1) / kDirectChunk) <= kEagerBlocks) {
      switch (D / 8) {
        case 8: return launch_direct<8, true>(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths, offsets, rows, stream);
        case 16: return launch_direct<16, true>(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths, offsets, rows, stream);
        case 32: return launch_direct<32, true>(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths, offsets, rows, stream);
        default: break;
      }
    }
    switch (D / 8) {
      case 8: return launch_direct<8>(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths, offsets, rows, stream);
      case 16: return launch_direct<16>(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths, offsets, rows, stream);
      case 32: return launch_direct<32>(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths, offsets, rows, stream);
      default: break;
    }
  }
  const int rc = launch_mask(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths,
                             offsets, workspace, stream);
  if (rc != KVZAP_OK) return rc;
  return launch_compact(K, V, keep_idx, lengths, offsets, K_out, V_out, cap_rows, B * H, T, D, stream);
}

int launch_mask(const float* scores, float tau, const float* tau_head, int window,
                const int32_t* seq_lens,
                int B, int H, int T, int32_t* keep_idx, int32_t* lengths,
                int64_t* offsets, void* workspace, hipStream_t stream) {
  if (direct_fits(B, H, T, kDirectSegments))
    return launch_direct<0>(scores, tau, tau_head, window, seq_lens, B, H, T, keep_idx, lengths, offsets,
                            GatherArgs{}, stream);
  const int BH = B * H;
  const int nchunks = mask_chunks(T);
  int32_t* chunk_counts = static_cast<int32_t*>(workspace);
  int64_t* chunk_prefix = reinterpret_cast<int64_t*>(
      static_cast<char*>(workspace) + align_up((size_t)BH * nchunks * sizeof(int32_t), 256));
  const dim3 grid(nchunks, BH);
  mask_count_kernel<<<grid, kThreads, 0, stream>>>(scores, tau, tau_head, window, seq_lens, H, T,
                                                   nchunks, chunk_counts);
  if ((long long)BH * nchunks <= kFusedMaxChunks) {
    mask_emit_kernel<true><<<grid, kThreads, 0, stream>>>(scores, tau, tau_head, window, seq_lens, H, T,
                                                          nchunks, chunk_prefix, chunk_counts,
                                                          keep_idx, lengths, offsets);
  } else {
    mask_scan_kernel<<<1, kScanThreads, 0, stream>>>(chunk_counts, chunk_prefix, BH, nchunks,
                                                     lengths, offsets);
    mask_emit_kernel<false><<<grid, kThreads, 0, stream>>>(scores, tau, tau_head, window, seq_lens, H, T,
                                                           nchunks, chunk_prefix, chunk_counts,
                                                           keep_idx, lengths, offsets);
  }
  return hipGetLastError() == hipSuccess ? KVZAP_OK : KVZAP_ERR_RUNTIME;
}

int launch_mask_static(const float* scores, float tau, int window, const int32_t* seq_lens, int B,
                       int H, int T, int32_t* keep_idx, int32_t* lengths, int64_t* offsets,
                       hipStream_t stream) {
  if ((long long)B * H * mask_chunks(T) > (long long)kStaticMaskChunks) return KVZAP_ERR_STATIC_LIMIT;
  void* ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc != KVZAP_OK) return rc;
  // launch_mask splits its workspace at align_up(chunks * 4, 256) <= kStaticCountBytes
  return launch_mask(scores, tau, nullptr, window, seq_lens, B, H, T, keep_idx, lengths, offsets,
                     ws, stream);
}

}  // namespace kvzap
