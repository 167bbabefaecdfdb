// Which of the linear surrogate's kernels takes an input, as constant expressions (plain C++14, no device
// code: the launch uses them and a host test asks them).
#pragma once

namespace kvzap {
namespace linear {

constexpr int kRowTokens = 8, kRowInputs = 512, kRowMaxWaves = 10;
constexpr long long kRowMaxTokens = 8192, kRowMaxTokensFewHeads = 6144;    // beyond, W per 8 tokens is too much to stage
constexpr int kStreamWaves = 8, kStreamBlocks = 256;
constexpr int kTurnBytes = 16 * 256;

// Wavefronts of a streaming block, as many as W leaves room for, and the groups whose scores each can
// hold (0: no room)
struct Stream {
  int waves, held;
};
constexpr Stream stream_of(int Dh, int H) {
  const long long room = 160 * 1024 - (long long)H * ((long long)Dh * 2 + 64);
  for (int waves = kStreamWaves; waves >= 4; waves -= 2) {
    const long long held = (room / waves - kTurnBytes) / (H * 64);
    if (held > 0) return {waves, (int)(held < 16 ? held : 16)};
  }
  return {0, 0};
}

// short inputs row by row; long ones as a stream of whole lines; what is between in the operand layout, with
// 16- or 4-wavefront blocks, or a block to a group of 16 tokens
enum class Form { kRows, kStream, kWide, kNarrow, kShort };

// The stream from 30 MB on, 32 where there are no more than 65536 tokens of less than 5 KB: below, staging W
// in every block costs more than the streaming gains. us per call (it / the kernels it takes the place of), H
// = 8 unless named: 262144 x 5120 402 (6.7 TB/s) / 450, 131072 x 4096 160 / 195, 65536 x 4096 87 / 103, x 2048
// 46 / 57, 32768 x 4096 44 / 55, 20000 x 5120 37 / 55, 16384 x 4096 24 / 30, 10000 x 2048 11.0 / 12.2; 40000 x
// 8192 109 / 143; 14 heads 8192 x 4096 15.5 / 20.3; one head 262144 x 4096 317 / 375, 20000 x 1024 10.6 /
// 12.0; not taken: 14895 x 1024 8.8 / 8.4, 29788 x 512 8.8 / 8.2, two heads 7449 x 2048 9.3 / 8.4.
// The row kernel's blocks of 8 tokens, which fill a CU's LDS, come in rounds, and the stream wins from the
// fourth on: 4641 x 4096 13.8 / 11.8, 6106: 14.0 / 13.0, 6838: 14.4 / 15.6, 5471 x 5120 16.9 / 14.0, 6253:
// 17.0 / 17.2, 5536 x 3072 11.6 / 11.1, 6187: 11.8 / 13.4.
// The narrow form gives each of 1024 wavefronts one group up to 16384 tokens and takes as long for few as for
// all: near that end it is the faster one up to 90 MB (13674 x 2048 12.9 / 12.4, x 3072 and four heads 17.0 /
// 15.3; not 12210 x 2048 11.6 / 12.0, 16279 x 3072 19.1 / 20.3, 16604 x 2048 15 / 19), for one or two heads,
// whose W is soon staged, earlier (two heads 11233 x 2048 11.1 / 10.6, 13674 x 3072 17.0 / 15.0), and for
// those with rows of 1 KB at most up to the wide form's 65536 (62503 x 512 13.1 / 12.4, 70315: 14.6 / 22.9).
constexpr long long kStreamBytes = 30000000, kStreamBytesMid = 32000000, kLastStretch = 90000000;

constexpr bool streams(long long rows, int Dh, int H) {
  const long long groups = (rows + 15) / 16;
  if (stream_of(Dh, H).held == 0 || groups <= 256) return false;
  if (rows * Dh * 2 < (rows > 65536 || Dh >= 2560 ? kStreamBytes : kStreamBytesMid)) return false;
  if (rows > (H <= 2 ? 10000 : 12700) && rows <= 16384 && rows * Dh * 2 <= kLastStretch) return false;
  return !(H <= 2 && Dh <= 512 && rows <= 65536);
}

constexpr Form form_of(long long rows, int Dh, int H) {
  const long long groups = (rows + 15) / 16;
  if (H <= kRowTokens && Dh <= kRowMaxWaves * kRowInputs && rows <= (H <= 2 ? kRowMaxTokensFewHeads : kRowMaxTokens)) {
    const int per_cu = kRowMaxWaves / ((Dh + kRowInputs - 1) / kRowInputs);          // blocks that the LDS holds
    if (!streams(rows, Dh, H) || rows <= 3ll * kRowTokens * per_cu * kStreamBlocks) return Form::kRows;
  }
  if (streams(rows, Dh, H)) return Form::kStream;
  // where W leaves that kernel no room or the input is short; from 64k tokens 16-wavefront blocks (W is
  // staged into LDS once per block), shorter inputs 4-wavefront blocks so that more CUs take part
  if (groups >= 4096) return Form::kWide;
  // 16k tokens: 26 us in narrow blocks, 32 us in short ones
  return groups > 512 || Dh % 128 != 0 ? Form::kNarrow : Form::kShort;
}

}  // namespace linear
}  // namespace kvzap
