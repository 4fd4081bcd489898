// CPU-only check of the decode attention's launchers: arguments that their kernel would silently leave out are refused
// before anything is launched.  Built against the library and run by tests/test_host_kernel_names.py.
#include <cstdio>

#include "../../paper_2506_06122_amd/csrc/kernels_fast.h"

template <class F>
static int refused(const char* what, F&& set, void (*launch)(const AttnArgs&, hipStream_t)) {
  AttnArgs a{};
  a.rows = 1;
  a.geom.n_kv_heads = 1;
  a.n_q_heads = 1;
  a.n_splits = 1;
  set(a);
  try {
    launch(a, nullptr);
  } catch (const HipError& e) {
    if (e.code == hipErrorInvalidValue) return 1;
  }
  std::fprintf(stderr, "%s: not refused\n", what);
  return 0;
}

int main() {
  static const int zero = 0;
  static unsigned ticket = 0;
  int n = 0;
  n += refused("row_t0", [](AttnArgs& a) { a.row_t0 = &zero; }, launch_attention_decode_fused);
  n += refused("slot0", [](AttnArgs& a) { a.slot0 = 1; }, launch_attention_decode_fused);
  n += refused("n_slots", [](AttnArgs& a) { a.n_slots = 2; }, launch_attention_decode_fused);
  n += refused("n_groups", [](AttnArgs& a) { a.n_groups = 1; }, launch_attention_decode_fused);
  n += refused("splits without tickets", [](AttnArgs& a) { a.n_splits = 2; }, launch_attention_decode_fused);
  n += refused("17 splits", [](AttnArgs& a) { a.n_splits = 17, a.tickets = &ticket; }, launch_attention_decode_fused);
  n += refused("tickets, grouped", [](AttnArgs& a) { a.n_splits_a = a.n_groups = 1, a.tickets = &ticket; }, launch_attention_decode_grouped);
  std::printf("%d refused\n", n);
  return n != 7;
}
