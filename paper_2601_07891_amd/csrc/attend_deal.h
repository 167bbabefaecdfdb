// How decode attention's first pass is dealt out to wavefronts, as constant expressions (plain C++14,
// no device code: the kernels and the launch use them, and a host test goes over their sums).
//
// Rows are counted in chunks of 32.  The chunks of all heads, in (b,h) order, are one list, of which
// each of nw wavefronts takes an equal part, or each head is cut into splits of spc chunks of its own.
#pragma once

namespace kvzap {
namespace deal {

constexpr int kMinChunks = 4;            // of a wavefront: fewer, and the combining pass takes longer

// Measured below: us per call of both passes, 8 KV heads and 4 query heads each unless named; rows cold in memory /
// three caches in turn, which the 256 MB memory-side cache may hold.
//
// As one list: equal parts of all heads' chunks in 4-wavefront blocks on 28 of an XCD's 32 CUs, or where
// there are no more than 64 heads in one-wavefront blocks on all of them, but at least kMinChunks chunks
// each.  64 sequences of 4k..32k rows 702 (6.96 TB/s; in streamed splits 766, in plain ones 843; with 1024
// wavefronts 711, 2048 787), 24 of 4k..8k 97.6 (102.8, 117), 40 of 0.3k..2.4k 45.0 (56.2, 66.6), 8 of 0.1k..30k 80.7
// (103, 117), 3 of 8k..32k 45.0 (51.0, 59.2).
// Head by head, streamed, where the list is short by the caller's bound: its parts wait for the sum over the heads,
// and most bounds are loose.  3 of 1k..8k 18.0 / 16.7 (as a list 18.7 / 17.6), 1 of 32k 28.6 / 28.3 (29.3 / 28.9), 8 of
// 1500 under a bound of 6500 15.2 / 14.1 (17.3 / 16.1), 32 of 500 under 2500 20.1 / 19.2 (22.1 / 21.2), 64 of 128 under 1012
// 17.8 / 16.6 (21.4 / 20.0).  Ragged heads under a tight bound are the better as a list from there on and a little before: 8 of
// 2k..8k 33.1 (36.7), 16 of 2k..8k 58.2 (63.0), 24 of 0.5k..2k 29.9 / 29.5 (31.3 / 31.0).  Past 64 heads the line is further
// up, since the sum then goes through LDS and a barrier; and from 8 query heads for a KV head on, since the list's parts are
// shorter and the sums of each are as large (16 query heads, 8 of 2k..4k 23.8 / 23.4, as a list 28.4 / 28.1).
// So are heads of a few chunks at any number, since a part's every head begins with a wait for its first
// rows: 512 heads of 64 rows under a bound of 512 15.4 / 14.3 (19.3 / 18.0).
// The smallest lists take plain loads in the operand layout: 1 sequence of 100..500 rows 8.4 / 7.0 (streamed 8.9 /
// 8.2), of 0.7k..3k 10.4 / 8.2 (10.0 / 9.0), of 4000 11.5 / 9.9 (11.0 / 9.9); past the line 4 of 0.3k..2.4k 13.1 / 11.4 (12.2 / 10.9).
constexpr int kShortHead = 20;           // chunks, by the caller's bound
constexpr long long kPlainChunks = 2560;                              // of all heads, by the bound: 42 MB
constexpr long long split_chunks(int BH, int G) { return BH > 64 || G >= 8 ? 24576 : 15360; }   // 403 and 252 MB
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
    return {Deal::kHead, BH * (splits > 0 ? splits : 1), spc, all > kPlainChunks};
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
