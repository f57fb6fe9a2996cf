// Instantiations of the direct-to-LDS tiled kernel for float layers.
#include "igemm_split_kernel.hpp"

namespace sc {

template <int KS, bool TAPS, int VEC_OUT>
static LaunchFn pick_tile(int bm, int bn) {
  if constexpr (KS <= 2) {
    if (bm == 128 && bn == 64) return igemm_split_launch<128, 64, KS, TAPS, VEC_OUT>;
    if (bm == 128 && bn == 32) return igemm_split_launch<128, 32, KS, TAPS, VEC_OUT>;
    if (bm == 64 && bn == 64) return igemm_split_launch<64, 64, KS, TAPS, VEC_OUT>;
  }
  if (bm == 64 && bn == 32) return igemm_split_launch<64, 32, KS, TAPS, VEC_OUT>;
  return nullptr;
}

template <int KS>
static LaunchFn pick(int bm, int bn, bool taps, int vec_out) {
  if (vec_out == 1) return taps ? pick_tile<KS, true, 1>(bm, bn) : pick_tile<KS, false, 1>(bm, bn);
  if (vec_out == 2) return taps ? pick_tile<KS, true, 2>(bm, bn) : pick_tile<KS, false, 2>(bm, bn);
  return nullptr;
}

LaunchFn split_kernel(int bm, int bn, int groups, bool taps, int vec_out) {
  if (groups == 1) return pick<1>(bm, bn, taps, vec_out);
  if (groups == 2) return pick<2>(bm, bn, taps, vec_out);
  if (groups == 4) return pick<4>(bm, bn, taps, vec_out);
  return nullptr;
}

}  // namespace sc
