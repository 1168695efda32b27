// The library's dispatch rules (dispatch.hpp) behind a C interface, compiled
// with g++ by tests/routes.py.
#include "dispatch.hpp"

extern "C" {
int rule_one_kernel(int64_t m, int64_t n, int64_t k, int64_t lda, int64_t ldb) {
  return oz::one_kernel(m, n, k, lda, ldb);
}
int rule_fused_a(int64_t m, int64_t n) { return oz::fused_a(m, n); }
int rule_fused_moduli(int64_t m) { return oz::fused_moduli(m); }
int rule_reconstruct_strips(int64_t m, int64_t n) { return oz::reconstruct_strips(m, n); }
int rule_xcd_ranges(int64_t tiles, int64_t stages, int64_t splits) { return oz::xcd_ranges(tiles, stages, splits); }
int rule_both_at_once(int64_t m, int64_t n, int64_t k, int64_t kp, int64_t room) {
  return oz::both_at_once(m, n, k, kp, room);
}
int64_t rule_scan_both_slabs(int64_t n, int64_t k) { return oz::scan_both_slabs(n, k); }
int64_t rule_scan_both_blocks(int64_t m, int64_t n, int64_t k) { return oz::scan_both_blocks(m, n, k); }
}
