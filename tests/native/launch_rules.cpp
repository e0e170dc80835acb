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
    } else if (rule == "grid") {
      int64_t tiles;
      std::cin >> tiles;
      const moe::TileGrid g = moe::tile_grid(tiles);
      std::cout << g.x << " " << g.y << "\n";
    } else if (rule == "stream") {
      // "0", or "wn mr kg stages nt" where the streaming kernels take the GEMM
      int64_t R;
      int E, K, N, num_cu;
      bool swiglu, fp8;
      std::cin >> R >> E >> K >> N >> swiglu >> fp8 >> num_cu;
      if (!moe::stream_is_faster(R, E, K, N, swiglu, fp8, num_cu)) {
        std::cout << "0\n";
        continue;
      }
      const moe::StreamTile t = moe::stream_tile(R, E, N, swiglu, fp8, num_cu);
      std::cout << t.wn << " " << t.mr << " " << t.kg << " " << t.stages << " "
                << moe::stream_nt(R, E, K, N, swiglu, fp8, t.mr) << "\n";
    } else {
      return 1;
    }
  }
}
