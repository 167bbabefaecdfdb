// How decode attention's first pass is dealt out to wavefronts, as constant expressions (plain C++14,
// no device code: the kernels and the launch use them, and a host test goes over their sums).
//
// Rows are counted in chunks of 32.  The chunks of all heads, in (b,h) order, are one list, of which
// each of nw wavefronts takes an equal part, or each head is cut into splits of spc chunks of its own.
#pragma once

namespace kvzap {
namespace deal {

constexpr int kMinChunks = 4;            // of a wavefront: fewer, and the combining pass takes longer

// As one list: equal parts of all heads' chunks in 4-wavefront blocks on 28 of an XCD's 32 CUs, or where there
// are no more than 64 heads in one-wavefront blocks on all of them, but at least kMinChunks chunks each. us a
// call of both passes, rows cold in memory, 8 KV heads and 4 query heads each unless named (as streamed
// splits, as plain ones): 64 sequences of 4k..32k rows 702 (766, 843), 6.96 TB/s (with 1024 wavefronts 711,
// 2048 787); 24 of 4k..8k 97.6 (102.8, 117), 40 of 0.3k..2.4k 45.0 (56.2, 66.6), 8 of 0.1k..30k 80.7 (103,
// 117), 3 of 8k..32k 45.0 (51.0, 59.2), 8 of 2k..8k 33.1 (36.7, 42.4), 16 of 2k..8k 58.2 (63.0, 74.6).
//
// Head by head, which starts without a sum over the heads, where the list is short by the caller's bound.
// Plain loads in the operand layout while the rows may be found in the memory-side cache, out of which the
// hint keeps them (a bound of many chunks is seldom full). A decoding step (evict and attend) of three caches
// in turn, us (streamed splits, list): 1 of 0.1k..0.5k rows 17.4 (17.9, 19.5), 4 of 0.3k..2.4k 20.6 (21.1,
// 22.1), 6 of 1500 22.0 (22.8, 24.2), 3 of 1k..8k 26.2 (27.0, 27.3), in pages 26.6 (27.5, 28.7). With every
// row cold the streamed splits are the better from some 8 MB on: a call for 3 of 1k..8k 19.8 (18.0, 18.7).
//
// Streamed splits where the list may be more than that cache holds: a step for 9 of 1500 under a bound of 7644
// in pages 26.2 (list 29.5; plain 25.2), 1 of 32k in pages 38.6 (39.6; 41.7), 16 of 1500 38.4 (39.5; 42.4), 24
// of 1500 49.2 (47.2; 54.9), 64 of 500 48.0 (47.8; 53.9). The line to the list is further up past 64 heads,
// whose sum goes through LDS and a barrier, and from 8 query heads for a KV head on, since the list's parts
// are shorter and the sums of each are as large (16 query heads, 8 of 2k..4k 23.8 a call, as a list 28.4).
//
// Heads of a few chunks go head by head at any number, since a part's every head begins with a wait for its
// first rows: 512 heads of 64 rows under a bound of 512 15.4 a call, as a list 19.3.
constexpr int kShortHead = 20;                                          // chunks, by the caller's bound
constexpr long long plain_chunks(long long ct) { return ct > 128 && ct <= 1024 ? 11264 : 4096; }   // 185 and 67 MB
constexpr long long split_chunks(int BH, int G) { return G >= 8 ? 24576 : BH > 64 ? 18432 : 15360; }   // 403, 302, 252 MB
// The list's length is summed on the device in 32 bits, from lengths that only the store's size bounds
// (whatever the caller's array or its bound say, and heads may share pages): where that could come near
// 2^31 chunks no list is made.
constexpr long long kMostListed = 1ll << 30;

enum class Deal { kWave, kBlock, kHead };   // as one list, for a wavefront or a block; head by head
struct Dealt {
  Deal deal;
  int nw, spc;
  bool stream;
};

// ct: chunks of a head by the caller's bound; most: chunks that all heads together can have
constexpr Dealt deal_of(int BH, int G, long long ct, long long most) {
  const long long all = ct * BH;
  if (most > kMostListed || ct <= kShortHead || all <= split_chunks(BH, G)) {
    // up to 64 chunks for a head in some 96 splits where that leaves a wavefront for every CU (one head of 128k
    // rows 20 us in 257 splits, 40 in 65), about 2048 wavefronts, all resident at once, where there are more
    const long long fill = all / 2048, fold = ct / 96;
    int spc = kMinChunks;
    while (spc < ct && (spc < fill || (spc < 64 && spc < fold && all >= 512ll * spc))) spc *= 2;
    const int splits = (int)((ct + spc - 1) / spc);
    return {Deal::kHead, BH * (splits > 0 ? splits : 1), spc, all > plain_chunks(ct)};
  }
  const long long nw = (all + kMinChunks - 1) / kMinChunks, most_waves = BH > 64 ? 896 : BH < 4 ? 256 * BH : 1024;
  return {BH > 64 ? Deal::kBlock : Deal::kWave, (int)(nw < most_waves ? nw : most_waves), 0, true};
}

// Slots for the sums of any bound up to ct chunks: a part of the list has fewer than nw + BH segments, and
// splits of spc >= 4 chunks, where spc + 1 > ct * BH / 2048, are no more than BH + 2560.
constexpr long long slots_of(int BH, long long ct) {
  const long long parts = (ct * BH + kMinChunks - 1) / kMinChunks;
  return (parts < 2560 ? parts : 2560) + BH;
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
