// Answers of the launch rules on the CPU: one query per line of stdin (a name
// and integers), one line of integers per answer.
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "launch_rules.h"

using namespace sherry;

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string fn;
    in >> fn;
    std::vector<int64_t> a;
    for (int64_t v; in >> v;) a.push_back(v);
    if (fn == "quant_streams") {
      std::printf("%d\n", quant_streams(a[0], a[1]) ? 1 : 0);
    } else if (fn == "quant_shape") {
      const QuantShape q = quant_shape(a[0], a[1]);
      std::printf("%d %d\n", q.threads, q.pieces);
    } else {
      std::fprintf(stderr, "unknown query: %s\n", fn.c_str());
      return 1;
    }
  }
  return 0;
}
