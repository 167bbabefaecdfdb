// Host check of paper_2601_07891_amd/csrc/attend_deal.h: over shapes, bounds and stores, the parts of a list of
// the longest length that a dealt-out call can meet are inside it, in order and cover it (summed in 32 bits,
// as the kernel sums them), and no form writes more slots than the workspace has for its bound or a longer one.
//
// usage: attend_deal_check [--plant]   (--plant takes the store's size for granted: must fail)
//        attend_deal_check BH G max_rows window store_rows   (prints the form of one call)
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "attend_deal.h"

using namespace kvzap::deal;

static long long chunks(long long rows) { return (rows + 31) / 32; }

int main(int argc, char** argv) {
  if (argc == 6) {
    const int BH = std::atoi(argv[1]);
    const long long ring = chunks(std::atoll(argv[4]));
    const Dealt d = deal_of(BH, std::atoi(argv[2]), chunks(std::atoll(argv[3])) + ring, BH * (chunks(std::atoll(argv[5])) + ring));
    if (d.deal == Deal::kHead) std::printf("%s %d\n", d.stream ? "streamed" : "plain", d.nw / BH);
    else std::printf("%s %d\n", d.deal == Deal::kWave ? "list" : "block", d.nw);
    return 0;
  }
  const bool plant = argc > 1 && !std::strcmp(argv[1], "--plant");
  const int heads[] = {1, 2, 3, 4, 8, 24, 63, 64, 65, 72, 512, 513, 2080, 4097, 65535};
  const long long bounds[] = {0, 1, 31, 640, 641, 3000, 6272, 14336, 32768, 39000, 131072, 2000000, INT_MAX};
  const long long stores[] = {0, 1000, 100000, 9608179, 134217728, 1ll << 30, INT_MAX};
  const int windows[] = {0, 33, 128, 4096};
  int checked = 0, failed = 0, lists = 0;
  auto fail = [&](const char* what, int BH, long long ct, long long most) {
    if (failed++ < 8) std::printf("BH=%d, %lld chunks by the bound, %lld in all: %s\n", BH, ct, most, what);
  };
  for (int BH : heads)
    for (int window : windows)
      for (long long bound : bounds)
        for (long long store : stores) {
          const int G = 1 + checked % 16;
          const long long ct = chunks(bound) + chunks(window), most = BH * (chunks(store) + chunks(window));
          const Dealt d = deal_of(BH, G, ct, plant ? 0 : most);
          ++checked;
          if (d.nw < 1) fail("no wavefront", BH, ct, most);
          if (d.deal == Deal::kHead) {
            if (d.nw % BH || d.spc < 1 || (long long)d.nw / BH * d.spc < ct) fail("splits that do not hold the bound", BH, ct, most);
            if (d.nw > slots_of(BH, ct)) fail("more splits than slots", BH, ct, most);
            continue;
          }
          ++lists;
          if (d.nw + BH > slots_of(BH, ct) + 1) fail("more segments than slots", BH, ct, most);
          const long long totals[] = {1, d.nw, ct * BH, most};
          for (long long exact : totals) {
            if (exact > most) continue;
            const int total = (int)(unsigned)exact;           // the device's 32-bit sum
            long long next = 0;
            for (int w = 0; w < d.nw + 4; ++w) {              // a block's last wavefronts may lie past nw
              const Part p = part_of(total, d.nw, w);
              if (p.n <= 0) continue;
              if (p.begin != next || p.begin + (long long)p.n > exact || w >= d.nw) {
                fail("a part outside the list", BH, ct, most);
                break;
              }
              next += p.n;
            }
            if (next != exact) fail("chunks that nobody takes", BH, ct, most);
          }
        }
  // a workspace that was queried for a longer bound serves a shorter one
  for (int BH : heads)
    for (long long ct = 1; ct < 5000; ++ct)
      if (slots_of(BH, ct) < slots_of(BH, ct - 1)) fail("fewer slots for a longer bound", BH, ct, 0);
  std::printf("%d calls checked, %d of them lists, %d faults\n", checked, lists, failed);
  return failed ? 1 : 0;
}
