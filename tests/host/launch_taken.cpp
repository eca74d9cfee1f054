// Reads shapes from stdin, one a line: head-dim Hq Hkv causal sync keep-list CUs then the segment lengths; prints the estimate's
// choice, the launch that is taken, and where a dense sync block finds matrices that lie apart (apart | copied).
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "launch_choice.h"

int main() {
  using namespace fedattn;
  static const char* const names[] = {"four", "four-ordered", "eight", "eight-pairs", "split"};
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    int D, Hq, Hkv, causal, sync, keep, cus, len;
    in >> D >> Hq >> Hkv >> causal >> sync >> keep >> cus;
    if (!in) return 1;
    std::vector<int32_t> seg = {0};
    while (in >> len) seg.push_back(seg.back() + len);
    const int heads = heads_in_common(Hq / Hkv);
    const PrefillShape shape{seg.data(), (int)seg.size() - 1, Hq, Hkv, D, causal != 0, keep != 0, heads, kWaveRows * (4 / heads), cus};
    std::printf("%s %s %s\n", names[choose_prefill_launch(shape, sync != 0)], names[launch_to_take(shape, sync != 0)],
                read_apart(shape) ? "apart" : "copied");
  }
  return 0;
}
