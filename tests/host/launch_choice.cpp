// Reads shapes from stdin, one a line: dtype (bf16 | f32) head-dim Hq Hkv causal sync keep-list CUs then the segment
// lengths; prints the name of the launch each one takes.
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "launch_choice.h"

int main() {
  using namespace fedattn;
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string dtype;
    int D, Hq, Hkv, causal, sync, keep, cus, len;
    in >> dtype >> D >> Hq >> Hkv >> causal >> sync >> keep >> cus;
    if (!in) return 1;
    std::vector<int32_t> seg = {0};
    while (in >> len) seg.push_back(seg.back() + len);
    const int n = (int)seg.size() - 1;
    if (dtype == "f32") {
      std::puts(f32_heads_shared(seg.data(), n, Hq, Hkv, D, 1, cus) ? "shared" : "keys");
    } else {
      static const char* const names[] = {"four", "four-ordered", "eight", "eight-pairs", "split"};
      const int heads = heads_in_common(Hq / Hkv);
      std::puts(names[launch_to_take(PrefillShape{seg.data(), n, Hq, Hkv, D, causal != 0, keep != 0, heads,
                                                  kWaveRows * (4 / heads), cus}, sync != 0)]);
    }
  }
  return 0;
}
