// KVzap-Linear forward (Sec. 3.3, Sec. 4.1; App. B Eq. 6): scores = hidden . W^T + b.
//
// With H = 8 outputs the arithmetic intensity is H flop per byte of hidden
// state: the kernel is bound by streaming `hidden` from HBM exactly once.  Plain
// vector ALUs would need 64 FMAs plus bf16 unpacking per 16-byte load, which at
// 8 TB/s is more than the chip's fp32 vector rate; the matrix cores do the same
// work at a few per cent utilisation, so the contraction runs on
// v_mfma_f32_16x16x32_bf16 with tokens on the N side and heads (padded to 16) on
// the M side:
//   A (16 x 32)  = W rows (heads) from LDS, staged once per block
//   B (32 x 16)  = 16 tokens x 32 inputs in the instruction's operand layout (lane = token +
//                  16*k-group, 16 bytes per lane): long inputs in whole lines through LDS
//                  (score_linear_stream_kernel), others straight from global memory.  That way a
//                  128-byte line is consumed by two consecutive load instructions, and with the
//                  non-temporal hint the second one fetches it again (5.1 instead of 6.0 TB/s)
//   C (16 x 16)  = fp32 accumulators, heads 0..15 x 16 tokens
// Each wavefront owns groups of 16 consecutive tokens and walks the whole D_h.
#include "kvzap_internal.h"
#include "score_linear_rule.h"

namespace kvzap {
namespace {

using namespace linear;

// kThreads: wavefronts of a block share one copy of W in LDS; kUnroll: independent 16-byte
// loads in flight per lane
template <int kThreads, int kUnroll>
__global__ __launch_bounds__(kThreads) void score_linear_kernel(
    const unsigned short* __restrict__ hidden, const unsigned short* __restrict__ W,
    const unsigned short* __restrict__ bias, float* __restrict__ scores,
    long long rows, int T, int Dh, int H, int groups_per_block) {
  constexpr int kWaves = kThreads / 64;
  extern __shared__ __align__(16) unsigned char smem[];
  // W as [H][Dh/8 + 4] 16-byte pieces: the 64-byte pad per row spreads the 16
  // (head, k-group) pieces one ds_read_b128 touches over distinct banks
  u32x4* sW = reinterpret_cast<u32x4*>(smem);
  const int pieces_per_row = Dh / 8;
  const int lds_stride = pieces_per_row + 4;
  // W is contiguous ([H][Dh]): piece i of the whole matrix goes to row i / pieces_per_row.
  // Eight loads in flight per thread: one at a time, this staging was a chain of memory
  // round trips that took most of a short call (16 us of 20).
  const int total_pieces = H * pieces_per_row;
  for (int base = 0; base < total_pieces; base += kThreads * 8) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = base + u * kThreads + (int)threadIdx.x;
      v[u] = reinterpret_cast<const u32x4*>(W)[i < total_pieces ? i : total_pieces - 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = base + u * kThreads + (int)threadIdx.x;
      if (i < total_pieces) {
        const int h = i / pieces_per_row, p = i - h * pieces_per_row;
        sW[h * lds_stride + p] = v[u];
      }
    }
  }
  __syncthreads();

  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int col = lane & 15;          // token within the group (B operand) / head (A operand)
  const int kg = lane >> 4;           // which 8 of the 32 inputs of one MFMA
  const long long ngroups = (rows + 15) / 16;
  const long long g_begin = (long long)blockIdx.x * groups_per_block;
  long long g_end = g_begin + groups_per_block;
  if (g_end > ngroups) g_end = ngroups;
  // lanes of the padded heads (col >= H) read a real row and zero it afterwards
  const bool head_ok = col < H;
  const u32x4* sWrow = sW + (size_t)(col % H) * lds_stride + kg;   // + 4*i per MFMA step
  const int steps = Dh / 32;
  const int steps_main = steps / kUnroll * kUnroll;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  for (long long g = g_begin + wid; g < g_end; g += kWaves) {
    long long r = g * 16 + col;
    const bool valid = r < rows;
    if (!valid) r = rows - 1;          // clamp: loads stay in bounds, result discarded
    const u32x4* hrow = reinterpret_cast<const u32x4*>(hidden + (size_t)r * Dh) + kg;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < steps_main; i0 += kUnroll) {
      u32x4 b[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        b[u] = hrow[(size_t)(i0 + u) * 4];
      // the W fragments of the whole batch are read from LDS while the global loads are in
      // flight: read one by one in front of their MFMAs, each exposed its LDS latency when a
      // wavefront is alone on its SIMD (13 of the 18 us of a short call)
      u32x4 a[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const u32x4 w = sWrow[(size_t)(i0 + u) * 4];
        a[u] = head_ok ? w : zero4;
      }
      __builtin_amdgcn_sched_barrier(0);               // keep the reads ahead of the MFMAs
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, a[u]), __builtin_bit_cast(bf16x8, b[u]), acc, 0, 0, 0);
    }
    for (int i = steps_main; i < steps; ++i) {
      const u32x4 b = hrow[(size_t)i * 4];
      const u32x4 a = head_ok ? sWrow[(size_t)i * 4] : zero4;
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    }
    // C layout: lane holds token `col`, heads 4*kg + e
    if (valid) {
      const long long bidx = r / T;
      const long long t = r - bidx * T;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int h = 4 * kg + e;
        if (h < H) {
          const float bv = bias ? bf16_bits_to_float(bias[h]) : 0.0f;
          scores[((size_t)bidx * H + h) * T + t] = acc[e] + bv;
        }
      }
    }
  }
}

// Long inputs: the same contraction with the tokens as a stream of whole lines.  A load instruction
// takes 256 bytes of each of four rows with the non-temporal hint, the form in which this part's
// memory gives 7.0 TB/s (6.0 with the 64 bytes of a row that the operand layout asks for, hint or not),
// and the wavefront turns them into that layout through 4 KB of LDS of its own, pieces XOR-swizzled with
// the row.  One block per CU; a wavefront's groups of 16 tokens are one stream of stages of 256 inputs,
// the next stage loading while the current one is multiplied.
//   Scores wait in LDS until the wavefront is through (or its share of the LDS is full): stored group
// by group, their 0.3 % of the bytes, 64 at a time, took 7 % of the time.
//   Blocks start at different inputs of a row, those of one XCD (every eighth) and neighbours alike: where
// rows are 2^n bytes long, blocks that walk D_h in step read from the same few memory channels (32768 x
// 4096: in step 48 us, with the block index alone as the shift 63, with this one 44).
__global__ __launch_bounds__(kStreamWaves * 64, 2) void score_linear_stream_kernel(
    const unsigned char* __restrict__ hidden, const unsigned short* __restrict__ W,
    const unsigned short* __restrict__ bias, float* __restrict__ scores, long long rows, int T, int Dh, int H,
    int held) {
  extern __shared__ __align__(16) unsigned char smem[];
  u32x4* sW = reinterpret_cast<u32x4*>(smem);            // [H][Dh/8 + 4], as above
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int threads = blockDim.x, waves = threads / 64;
  const int pieces_per_row = Dh / 8, lds_stride = pieces_per_row + 4;
  unsigned char* const own = smem + (size_t)H * lds_stride * 16 + (size_t)wid * (kTurnBytes + held * H * 64);
  u32x4* const turn = reinterpret_cast<u32x4*>(own);
  float* const done = reinterpret_cast<float*>(own + kTurnBytes);          // [H][held * 16]
  const int col = lane & 15, kg = lane >> 4;
  const long long ngroups = (rows + 15) / 16;
  // the block's groups go round its wavefronts: next to each other in memory at any time
  const long long g0 = ngroups * blockIdx.x / gridDim.x + wid, g1 = ngroups * (blockIdx.x + 1) / gridDim.x;
  const int steps = Dh / 32, per_group = (steps + 7) / 8;
  const int n = g0 < g1 ? (int)((g1 - g0 + waves - 1) / waves) * per_group : 0;
  const int k_first = (int)((3 * (blockIdx.x / 8) + blockIdx.x % 8) % (unsigned)per_group);

  long long g_in = g0;
  int k_in = k_first, left_in = per_group;
  unsigned row_off[4];
  auto enter_group = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * i + kg;                        // past the end: clamped, result discarded
      row_off[i] = (unsigned)(rows - g_in * 16 > row ? row : (int)(rows - g_in * 16) - 1) * (unsigned)Dh * 2u;
    }
  };
  auto load = [&](u32x4 (&v)[8]) {
    const unsigned char* base = hidden + (size_t)g_in * 16 * Dh * 2;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      unsigned at = (unsigned)(k_in * 512 + (u >> 2) * 256 + col * 16);
      at = at < (unsigned)Dh * 2u - 16u ? at : (unsigned)Dh * 2u - 16u;    // past D_h: not multiplied
      v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (row_off[u & 3] + at)));
    }
    if (++k_in == per_group) k_in = 0;
    if (--left_in == 0) {
      left_in = per_group;
      g_in += waves;
      if (g_in < g1) enter_group();
    }
  };
  u32x4 va[8], vb[8];
  if (n > 0) {
    enter_group();
    load(va);
  }

  const int total_pieces = H * pieces_per_row;
  for (int base = 0; base < total_pieces; base += threads * 8) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = base + u * threads + (int)threadIdx.x;
      v[u] = reinterpret_cast<const u32x4*>(W)[i < total_pieces ? i : total_pieces - 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = base + u * threads + (int)threadIdx.x;
      if (i < total_pieces) {
        const int h = i / pieces_per_row, p = i - h * pieces_per_row;
        sW[h * lds_stride + p] = v[u];
      }
    }
  }
  __syncthreads();
  if (n == 0) return;

  const bool head_ok = col < H;
  const u32x4* const sWrow = sW + (size_t)(col % H) * lds_stride + kg;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  // Eight sums, one for each of a stage's products, folded into one every eight stages: a product does
  // not wait for the one before it, and the chains of additions are short (one chain through D_h = 4096:
  // 3e-7 of the exact scores, like this 8e-8).
  floatx4 acc[2][4], folded = {0.f, 0.f, 0.f, 0.f}, bias4;
  auto clear = [&]() {
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc[half][kk] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
#pragma unroll
  for (int e = 0; e < 4; ++e)
    bias4[e] = bias ? bf16_bits_to_float(bias[4 * kg + e < H ? 4 * kg + e : H - 1]) : 0.0f;
  long long g_at = g0;                                   // first group whose scores are held
  int k_at = k_first, left_at = per_group, have = 0;
  auto flush = [&]() {
    wave_fence();
    for (int i = lane; i < have * 16; i += 64) {
      const long long r = (g_at + (i >> 4) * waves) * 16 + (i & 15);
      if (r < rows) {
        const long long bidx = r / T;
        float* to = scores + (size_t)bidx * H * T + (r - bidx * T);
        for (int h = 0; h < H; ++h) to[(size_t)h * T] = done[h * held * 16 + i];
      }
    }
    wave_fence();
    g_at += (long long)have * waves;
    have = 0;
  };
  auto consume = [&](const u32x4 (&v)[8]) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      wave_fence();                                      // the reads of the half before
#pragma unroll
      for (int i = 0; i < 4; ++i) turn[(4 * i + kg) * 16 + (col ^ (4 * i + kg))] = v[half * 4 + i];
      wave_fence();
      u32x4 a[4], b[4];
      const int s0 = k_at * 8 + half * 4;                // MFMA step of D_h
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        b[kk] = turn[col * 16 + ((4 * kk + kg) ^ col)];
        const u32x4 w = sWrow[(size_t)(s0 + kk < steps ? s0 + kk : steps - 1) * 4];
        a[kk] = head_ok ? w : zero4;
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        if (s0 + kk < steps)                             // uniform
          acc[half][kk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, a[kk]), __builtin_bit_cast(bf16x8, b[kk]), acc[half][kk], 0, 0, 0);
    }
    if (++k_at == per_group) k_at = 0;
    --left_at;
    if ((left_at & 7) == 0) {
      folded += ((acc[0][0] + acc[0][1]) + (acc[0][2] + acc[0][3])) + ((acc[1][0] + acc[1][1]) + (acc[1][2] + acc[1][3]));
      clear();
    }
    if (left_at == 0) {                                  // C: token `col` of the group, heads 4*kg + e
      left_at = per_group;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * kg + e < H) done[((4 * kg + e) * held + have) * 16 + col] = folded[e] + bias4[e];
      folded = floatx4{0.f, 0.f, 0.f, 0.f};
      if (++have == held) flush();
    }
  };
  int i = 0;
  while (i + 2 < n) {
    load(vb);
    consume(va);
    load(va);
    consume(vb);
    i += 2;
  }
  if (i + 1 < n) {
    load(vb);
    consume(va);
    consume(vb);
  } else {
    consume(va);
  }
  flush();
}

// Short inputs (up to 512 groups of 16 tokens) that the kernel below does not take, with more than eight heads or a
// larger D_h (1024 tokens: 10 us against 18 us): with one group per wavefront the walk over
// D_h above is what a call costs (13 us at D_h = 4096: 128 operand loads through one CU's
// texture path per wavefront, however many are in flight).  Here the four wavefronts of a
// block share ONE group and take a quarter of D_h each, W comes straight from global memory
// (L2) like the tokens, so there is no staging and a single batch of loads; the four partial
// accumulators are added in a fixed order through LDS.
__global__ __launch_bounds__(256) void score_linear_short_kernel(
    const unsigned short* __restrict__ hidden, const unsigned short* __restrict__ W,
    const unsigned short* __restrict__ bias, float* __restrict__ scores,
    long long rows, int T, int Dh, int H) {
  __shared__ floatx4 red[4][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int col = lane & 15, kg = lane >> 4;
  long long r = (long long)blockIdx.x * 16 + col;
  const bool valid = r < rows;
  if (!valid) r = rows - 1;
  const bool head_ok = col < H;
  const int per = Dh / 128;                              // MFMA steps per wavefront (D_h % 128 == 0)
  const u32x4* hrow = reinterpret_cast<const u32x4*>(hidden + (size_t)r * Dh) + kg + (size_t)wid * per * 4;
  const u32x4* wrow = reinterpret_cast<const u32x4*>(W + (size_t)(col % H) * Dh) + kg + (size_t)wid * per * 4;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int kBatch = 16;
  for (int i0 = 0; i0 < per; i0 += kBatch) {
    u32x4 a[kBatch], b[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + u < per ? i0 + u : per - 1;     // clamped; the surplus is not accumulated
      b[u] = hrow[(size_t)i * 4];
      a[u] = wrow[(size_t)i * 4];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (i0 + u < per)                                  // uniform
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, head_ok ? a[u] : zero4), __builtin_bit_cast(bf16x8, b[u]),
            acc, 0, 0, 0);
    }
  }
  red[wid][lane] = acc;
  __syncthreads();
  if (wid == 0 && valid) {
    const floatx4 s = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    const long long bidx = r / T;
    const long long t = r - bidx * T;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int h = 4 * kg + e;
      if (h < H) {
        const float bv = bias ? bf16_bits_to_float(bias[h]) : 0.0f;
        scores[((size_t)bidx * H + h) * T + t] = s[e] + bv;
      }
    }
  }
}

// The shortest inputs, for up to eight heads.  Loads in the operand layout fetch 64 bytes from each
// of 16 rows, which lie D_h * 2 bytes (8 KB) apart: they run at some 24 bytes per clock and CU, and
// those 5 of 10 us are what a call on 16 to 1024 tokens costs, however they are split.  Here every
// load takes 1 KB of ONE row, straight to LDS, and the operands are read from there.
// A block is 8 tokens x all of D_h, a wavefront 512 inputs of it: 8 KB of tokens and 8 KB of W.
// The 16 columns of an MFMA are the 8 tokens twice, with the first and the second 256 inputs, and
// its 16 rows the 8 heads likewise: half the steps, no padded heads, and the two diagonal 8 x 8
// blocks of C are the result.
// Measured, us per call (here / the kernels above): D_h = 4096: 128 tokens 5.2 / 9.7, 1024: 5.0 / 10.0,
// 2048: 5.8 / 10.2, 4096: 9.1 / 10.7, 8192: 16.6 / 18.0, 16384: 34.5 / 29.2; D_h = 5120: 1024: 5.7 /
// 14.1, 8192: 22.1 / 28.0, 16384: 40.8 / 32.4; D_h = 2048: 1024: 3.9 / 6.0, 8192: 8.6 / 9.9.
// W takes its eight rows whatever H is, and the kernels above read fewer: one head at D_h = 4096 12.4 /
// 13.0 on 6144 tokens, 16.2 / 13.6 on 7000, 17.3 / 14.7 on 8192; two 12.4 / 14.8, 16.2 / 15.2, 17.4 /
// 15.9; three 16.3 / 16.8 on 7000.
constexpr int kRowWaveBytes = 2 * kRowTokens * kRowInputs * 2;

// LDS slot <-> 16-byte piece of a 1 KB row (its own inverse): the 16 lanes that are served
// together read one piece, and the one 32 on, of 8 rows, and meet 16 different bank groups
__device__ __forceinline__ int row_slot(int piece, int row) { return piece ^ (2 * row) ^ (piece >> 5); }

__global__ __launch_bounds__(kRowMaxWaves * 64) void score_linear_rows_kernel(
    const unsigned char* hidden, const unsigned char* W, const unsigned short* __restrict__ bias,
    float* __restrict__ scores, long long rows, int T, int Dh, int H) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, kg = lane >> 4, waves = blockDim.x / 64;
  const long long r0 = (long long)blockIdx.x * kRowTokens;
  const int pieces = Dh / 8 - wid * 64 < 64 ? Dh / 8 - wid * 64 : 64;      // of this wavefront, >= 8
  unsigned char* const mine = smem + wid * kRowWaveBytes;
#pragma unroll
  for (int i = 0; i < 2 * kRowTokens; ++i) {
    const int row = i & 7;
    int piece = row_slot(lane, row);
    if (piece > pieces - 1) piece = pieces - 1;                            // past D_h: its products are dropped
    const long long r = r0 + row < rows ? r0 + row : rows - 1;             // past the end: results dropped
    const unsigned char* base = i < kRowTokens ? hidden + (size_t)r * Dh * 2 : W + (size_t)(row < H ? row : H - 1) * Dh * 2;
    load_to_lds_b128(base + wid * (kRowInputs * 2), (unsigned)piece * 16u, lds_address(mine) + i * 1024);
  }
  wait_vmcnt<0>();
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < kRowInputs / 64; ++s) {
    const int piece = (col >> 3) * 32 + s * 4 + kg, row = col & 7;
    const unsigned char* at = mine + row * 1024 + row_slot(piece, row) * 16;
    const u32x4 b = *reinterpret_cast<const u32x4*>(at), w = *reinterpret_cast<const u32x4*>(at + 8 * 1024);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, piece < pieces ? w : zero4),
                                                  __builtin_bit_cast(bf16x8, piece < pieces ? b : zero4), acc, 0, 0, 0);
  }
  // lane (col, kg), register e: row 4*kg + e of C.  The wavefronts' sums meet in LDS.
  *reinterpret_cast<floatx4*>(mine + lane * 16) = acc;
  __syncthreads();
  if (threadIdx.x < 64) {
    const int tok = lane & 7, h = lane >> 3;
    const int first = ((h >> 2) * 16 + tok) * 16 + (h & 3) * 4, second = first + (2 * 16 + 8) * 16;
    float s = 0.0f;
    for (int w = 0; w < waves; ++w) {
      const unsigned char* from = smem + w * kRowWaveBytes;
      s += *reinterpret_cast<const float*>(from + first) + *reinterpret_cast<const float*>(from + second);
    }
    const long long r = r0 + tok;
    if (h < H && r < rows) {
      const long long bidx = r / T;
      scores[((size_t)bidx * H + h) * T + (r - bidx * T)] = s + (bias ? bf16_bits_to_float(bias[h]) : 0.0f);
    }
  }
}

int launch_linear_rows(const void* hidden, const void* W, const void* b, float* scores, long long rows,
                       int T, int Dh, int H, hipStream_t stream) {
  static const hipError_t attr_rc =
      hipFuncSetAttribute(reinterpret_cast<const void*>(score_linear_rows_kernel),
      hipFuncAttributeMaxDynamicSharedMemorySize, kRowMaxWaves * kRowWaveBytes);
  if (attr_rc != hipSuccess) return KVZAP_ERR_RUNTIME;
  const int waves = (Dh + kRowInputs - 1) / kRowInputs;
  score_linear_rows_kernel<<<dim3((unsigned)((rows + kRowTokens - 1) / kRowTokens)), waves * 64,
                             waves * kRowWaveBytes, stream>>>(
      static_cast<const unsigned char*>(hidden), static_cast<const unsigned char*>(W),
      static_cast<const unsigned short*>(b), scores, rows, T, Dh, H);
  return hipGetLastError() == hipSuccess ? KVZAP_OK : KVZAP_ERR_RUNTIME;
}

template <int kThreads, int kUnroll>
int launch_linear(const void* hidden, const void* W, const void* b, float* scores, long long rows,
                  int T, int Dh, int H, long long want_blocks, hipStream_t stream) {
  constexpr int kWaves = kThreads / 64;
  const long long ngroups = (rows + 15) / 16;
  long long gpb = (ngroups + want_blocks - 1) / want_blocks;
  if (gpb < kWaves) gpb = kWaves;                     // at least one group per wavefront
  const long long blocks = (ngroups + gpb - 1) / gpb;
  const size_t lds = (size_t)H * ((size_t)Dh * 2 + 64);   // validated <= 160 KB by the caller
  // once per process, which drives one GPU (thread-safe: a function-local static)
  static const hipError_t attr_rc =
      hipFuncSetAttribute(reinterpret_cast<const void*>(score_linear_kernel<kThreads, kUnroll>),
      hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (attr_rc != hipSuccess) return KVZAP_ERR_RUNTIME;
  score_linear_kernel<kThreads, kUnroll><<<dim3((unsigned)blocks), kThreads, lds, stream>>>(
      static_cast<const unsigned short*>(hidden), static_cast<const unsigned short*>(W),
      static_cast<const unsigned short*>(b), scores, rows, T, Dh, H, (int)gpb);
  return hipGetLastError() == hipSuccess ? KVZAP_OK : KVZAP_ERR_RUNTIME;
}

int launch_linear_stream(const void* hidden, const void* W, const void* b, float* scores, long long rows,
                         int T, int Dh, int H, hipStream_t stream) {
  const Stream st = stream_of(Dh, H);
  // once per process, which drives one GPU (thread-safe: a function-local static)
  static const hipError_t attr_rc =
      hipFuncSetAttribute(reinterpret_cast<const void*>(score_linear_stream_kernel),
      hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (attr_rc != hipSuccess) return KVZAP_ERR_RUNTIME;
  const size_t lds = (size_t)H * ((size_t)Dh * 2 + 64) + (size_t)st.waves * (kTurnBytes + st.held * H * 64);
  score_linear_stream_kernel<<<kStreamBlocks, st.waves * 64, lds, stream>>>(
      static_cast<const unsigned char*>(hidden), static_cast<const unsigned short*>(W),
      static_cast<const unsigned short*>(b), scores, rows, T, Dh, H, st.held);
  return hipGetLastError() == hipSuccess ? KVZAP_OK : KVZAP_ERR_RUNTIME;
}

}  // namespace

int launch_score_linear(const void* hidden, const void* W, const void* b, float* scores,
                        int B, int T, int Dh, int H, hipStream_t stream) {
  const long long rows = (long long)B * T;
  switch (form_of(rows, Dh, H)) {
    case Form::kRows: return launch_linear_rows(hidden, W, b, scores, rows, T, Dh, H, stream);
    case Form::kStream: return launch_linear_stream(hidden, W, b, scores, rows, T, Dh, H, stream);
    case Form::kWide: return launch_linear<1024, 8>(hidden, W, b, scores, rows, T, Dh, H, 1024, stream);
    case Form::kNarrow: return launch_linear<256, 8>(hidden, W, b, scores, rows, T, Dh, H, 1024, stream);
    case Form::kShort: break;
  }
  score_linear_short_kernel<<<dim3((unsigned)((rows + 15) / 16)), 256, 0, stream>>>(
      static_cast<const unsigned short*>(hidden), static_cast<const unsigned short*>(W),
      static_cast<const unsigned short*>(b), scores, rows, T, Dh, H);
  return hipGetLastError() == hipSuccess ? KVZAP_OK : KVZAP_ERR_RUNTIME;
}

}  // namespace kvzap
