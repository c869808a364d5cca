// topk_select (prr_topk.h) on the CPU, for tests/test_topk_host.py.
#include "prr_topk.h"

// Selects kextra of the n pages whose keys are given (and the forced ones), groups of
// 1 << gshift pages having the largest keys gmax.  Returns 0, or 1 if the workgroup does not end.
extern "C" int topk_host(int n, int gshift, int kextra, const int32_t* forced, int n_forced, const uint32_t* keys,
                         const uint32_t* gmax, int32_t* out, int cap, int32_t* out_count, int fill) {
  static prr::TopkLds lds;
  memset(&lds, fill, sizeof(lds));  // (LDS holds what the workgroup before left)
  const bool ended = emu::run(
      [&] {
        prr::topk_select(n, gshift, kextra, forced, n_forced, [&](int g) { return gmax[g]; },
                         [&](int p) { return keys[p]; }, out, cap, out_count, lds);
      },
      20000);
  return ended ? 0 : 1;
}

extern "C" int topk_shift(int n) { return prr::topk_group_shift(n); }
