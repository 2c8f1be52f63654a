// Solve-kernel variants and the autotuned choice per (precision, block size).
#pragma once
#include <stddef.h>

namespace fb {

// variant v: the tile width (right-hand sides per job).  Two kernels exist, v =
// 0 and v = 2; the other numbers are choices that older tune files may hold
// and stand for the kernel of their tile width.
constexpr int kNumVariants = 10;
inline int variant_tile(int v) { return ((v >= 2 && v < 6) || v == 9) ? 32 : 16; }
constexpr int kTimedVariants[2] = {0, 2};
// dynamic LDS of the block-solve kernel: three NB x T slots of the factors'
// element type, the block's permutation (2 NB window rows) and the gather
// order of its first NB rows (16-bit LDS offsets)
inline size_t solve_lds_bytes(int nb, int t, size_t elem) {
  return (size_t)3 * nb * t * elem + (size_t)3 * nb * 2;
}
bool variant_fits(size_t rsize, int nb, int v);
// the chosen variant, or -1 (the rule chooses); setting -1 takes a choice back
int tuned_variant(size_t rsize, int nb);
void set_tuned_variant(size_t rsize, int nb, int v);

}  // namespace fb
