// Prints the tile that each query line takes (the library's own selection code, host only).
#include "../paper_2609_33977_amd/csrc/gm_plan.h"

#include <cstdio>
#include <cstring>

int main() {
  char op[32];
  long T, d_in, d_out, g, go, arg;
  while (std::scanf("%31s %ld %ld %ld %ld %ld %ld", op, &T, &d_in, &d_out, &g, &go, &arg) == 7) {
    static const char* const wt[] = {"256x256", "256x128", "128x128"};
    static const char* const dx[] = {"256x256", "256x128", "128x256", "128x128", "64x128", "64x256"};
    const bool packed = !std::strcmp(op, "packed");
    if (packed || !std::strcmp(op, "fwd")) {  // arg: shares of K that the workspace holds
      const gm::FwdPlan p = gm::fwd_plan(T, d_in, d_out, int(g), packed ? 1 : int(go), packed, int(arg));
      if (packed && gm::packed_passes(T, d_in, d_out, int(g), p.ns)) std::printf("passes%d\n", gm::passes_rows(T, d_in, d_out, int(g)));
      else std::printf("%s%s\n", wt[int(p.tile)], p.ks > 1 ? " split" : "");
    } else if (!std::strcmp(op, "dgate")) {
      std::printf("256x%d\n", gm::dgate_columns(T, d_in, d_out, int(go)));
    } else if (!std::strcmp(op, "dx")) {
      if (gm::dx_dense_ok(d_out, int(g))) std::printf("dense %s\n", wt[int(gm::dx_dense_tile(T, d_in, d_out))]);
      else std::printf("%s\n", dx[int(gm::dx_tile(T, d_in, d_out, int(g)))]);
    } else if (!std::strcmp(op, "kinds")) {  // T blocks of d_in ns, then d_out of g
      std::printf("%ld\n", long(gm::two_kinds_ns(T, d_in, d_out, g)));
    } else if (!std::strcmp(op, "first")) {
      std::printf("%s\n", gm::square_dx_first(T, d_in, d_out, int(g)) ? "dX" : "dgate");
    } else if (!std::strcmp(op, "lm")) {  // T: tokens, d_in: hidden size
      std::printf("%s\n", wt[int(gm::lm_bwd_tile(T, d_in))]);
    } else {
      return 1;
    }
  }
  return 0;
}
