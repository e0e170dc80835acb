// Evaluates csrc/launch_rules.h: one rule and its arguments per input line, the choice per
// output line.
#include <iostream>
#include <string>

#include "launch_rules.h"

int main() {
  std::string rule;
  while (std::cin >> rule) {
    if (rule == "permute") {
      int64_t R;
      std::cin >> R;
      std::cout << moe::permute_small_iters(R) << "\n";
    } else if (rule == "combine") {
      int64_t T;
      int k, nvec;
      std::cin >> T >> k >> nvec;
      std::cout << moe::combine_splits(T, k, nvec) << "\n";
    } else {
      return 1;
    }
  }
}
