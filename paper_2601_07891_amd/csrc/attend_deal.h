// How decode attention's first pass is dealt out to wavefronts, as constant expressions (plain C++14,
// no device code: the kernels and the launch use them, and a host test goes over their sums).
//
// Rows are counted in chunks of 32.  The chunks of all heads, in (b,h) order, are one list, of which
// each of nw wavefronts takes an equal part, or each head is cut into splits of spc chunks of its own.
#pragma once

namespace kvzap {
namespace deal {

constexpr int kMinChunks = 4;            // of a wavefront: fewer, and the combining pass takes longer

// Equal parts of all heads' chunks in 4-wavefront blocks on 28 of an XCD's 32 CUs, or where there are
// no more than 64 heads in one-wavefront blocks on all of them, but at least kMinChunks chunks each and
// no more than 256 wavefronts for one head, whose sums one block combines.  Measured, us per call
// (before, in splits of one head handed out one by one with 64-byte K loads / now): 8 KV heads, 4 query
// heads each: 64 sequences of 4k..32k rows 837 / 699 (6.96 TB/s; with 1024 wavefronts 711, 2048 787),
// 64 of 16000 708 / 614, 24 of 4k..8k 123 / 96, 16 of 0.5k..2k 25.3 / 22.3, 8 of 0.1k..30k 115 / 81, 3 of
// 1k..8k 20.0 / 18.2, 1 of 128k 94 / 87, of 32k 30.2 / 29.1, of 2500 12.2 / 12.2; one KV head of 128k 23.8 /
// 20.9, two 33.6 / 30.4.
// Heads of a few chunks are better off with a wavefront of their own, since a part's every head begins
// with a wait for its first rows: 512 heads of 64 rows beside the window 16.9 us in equal parts, 14.6 head
// by head, 2048 heads 48.4 / 42.9, 8192 194 / 183; 512 of 512 rows (20 chunks) 33.8 / 33.7.  So is a
// list of up to kFewWaves splits at the smallest, all of which are resident at once and start without the sum over
// the heads: 1 of 0.7k..3k rows 7.4 / 6.7 for this pass, 2 of 2000 in pages 8.6 / 8.1; with 4096
// splits 3 of 1k..8k 14.4 / 15.2.
constexpr int kShortHead = 20;           // chunks, by the caller's bound
constexpr long long kFewWaves = 2048;    // eight on each CU
// The list's length is summed on the device in 32 bits, from lengths that only the store's size bounds
// (whatever the caller's array or its bound say, and heads may share pages): where that could come near
// 2^31 chunks no list is made.
constexpr long long kMostListed = 1ll << 30;

enum class Deal { kWave, kBlock, kHead };
struct Dealt {
  Deal deal;
  int nw, spc;
};

// ct: chunks of a head by the caller's bound; most: chunks that all heads together can have
constexpr Dealt deal_of(int BH, long long ct, long long most) {
  if (most > kMostListed || ct <= kShortHead || (ct * BH <= kFewWaves * kMinChunks && ct <= 256 * kMinChunks)) {
    int spc = kMinChunks;
    while (spc < ct && 2048ll * spc < ct * BH) spc *= 2;
    const int splits = (int)((ct + spc - 1) / spc);
    return {Deal::kHead, BH * (splits > 0 ? splits : 1), spc};
  }
  const long long nw = (ct * BH + kMinChunks - 1) / kMinChunks, most_waves = BH > 64 ? 896 : BH < 4 ? 256 * BH : 1024;
  return {BH > 64 ? Deal::kBlock : Deal::kWave, (int)(nw < most_waves ? nw : most_waves), 0};
}

// Slots for the sums of any bound up to ct chunks: a part of the list has fewer than nw + BH segments, and
// splits of spc >= ct * BH / 2048 chunks are no more than BH + 2048.
constexpr long long slots_of(int BH, long long ct) {
  const long long parts = (ct * BH + kMinChunks - 1) / kMinChunks;
  return (parts < 2048 ? parts : 2048) + BH;
}

// Wavefront w's part of a list of `total` chunks; n <= 0: none
struct Part {
  int begin, n;
};
constexpr Part part_of(int total, int nw, int w) {
  int per = (int)(((unsigned)total + (unsigned)nw - 1) / (unsigned)nw);
  per = per > kMinChunks ? per : kMinChunks;
  const int begin = w < nw ? w * per : total;
  return {begin, total - begin < per ? total - begin : per};
}

}  // namespace deal
}  // namespace kvzap
