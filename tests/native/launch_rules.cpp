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
    } else {
      return 1;
    }
  }
}
