// Instantiations of the buffer-load tiled kernel (16-bit operands, float accumulate).
#include "igemm_buf_kernel.hpp"

namespace sc {

// ring of two tiles for layers with at most two K tiles (less LDS, more workgroups per CU)
template <int DT>
static LaunchFn pick_shallow(int bm, int bn) {
  if (bm == 128 && bn == 64) return igemm_buf_launch<DT, 128, 64, 2, 2, 2>;
  if (bm == 96 && bn == 128) return igemm_buf_launch<DT, 96, 128, 1, 4, 2>;
  if (bm == 64 && bn == 128) return igemm_buf_launch<DT, 64, 128, 2, 2, 2>;
  if (bm == 64 && bn == 64) return igemm_buf_launch<DT, 64, 64, 2, 2, 2>;
  if (bm == 128 && bn == 32) return igemm_buf_launch<DT, 128, 32, 4, 1, 2>;
  if (bm == 32 && bn == 128) return igemm_buf_launch<DT, 32, 128, 1, 4, 2>;
  return nullptr;
}

template <int DT>
static LaunchFn pick(int bm, int bn) {
  if (bm == 256 && bn == 128) return igemm_buf_launch<DT, 256, 128, 4, 2, 3>;   // eight wavefronts
  if (bm == 128 && bn == 256) return igemm_buf_launch<DT, 128, 256, 2, 4, 3>;   // eight wavefronts
  if (bm == 128 && bn == 128) return igemm_buf_launch<DT, 128, 128, 2, 4, 3>;   // eight wavefronts
  if (bm == 128 && bn == 64) return igemm_buf_launch<DT, 128, 64, 2, 2, 3>;
  if (bm == 96 && bn == 128) return igemm_buf_launch<DT, 96, 128, 1, 4, 3>;
  if (bm == 64 && bn == 128) return igemm_buf_launch<DT, 64, 128, 2, 2, 3>;
  if (bm == 64 && bn == 64) return igemm_buf_launch<DT, 64, 64, 2, 2, 3>;
  if (bm == 128 && bn == 32) return igemm_buf_launch<DT, 128, 32, 4, 1, 3>;
  if (bm == 32 && bn == 128) return igemm_buf_launch<DT, 32, 128, 1, 4, 3>;
  return nullptr;
}

template <int DT>
static LaunchFn pick_splitk(int bm, int bn) {
  if (bm == 256 && bn == 128) return igemm_buf_launch<DT, 256, 128, 4, 2, 3, true>;
  if (bm == 128 && bn == 256) return igemm_buf_launch<DT, 128, 256, 2, 4, 3, true>;
  if (bm == 128 && bn == 128) return igemm_buf_launch<DT, 128, 128, 2, 4, 3, true>;
  if (bm == 96 && bn == 128) return igemm_buf_launch<DT, 96, 128, 1, 4, 3, true>;
  if (bm == 64 && bn == 128) return igemm_buf_launch<DT, 64, 128, 2, 2, 3, true>;
  return nullptr;
}

// Measured (us, s = 0.5, 64 x 64 with one group / two): 64 x 512 -> 512 @7 24.4 / 20.3 (split K of 128 x 128, the choice
// before: 22.0), 64 x 256 -> 512 @7 13.8 / 12.1, 2 x 256 -> 256 @40 13.6 / 11.8, 30 x 384 -> 384 @13 19.3 / 16.8 (20.7); with more
// workgroups than compute units 17.1 / 22.7 (64 x 256 -> 256 @14).  64 x 128 and 128 x 64 with two groups: up to 12 % faster
// alone than one group of 64 x 64, no faster behind other layers (filters cold), left out.  Chosen by the model in the place of a
// split of K only (see model_pick).
template <int DT>
static LaunchFn pick_groups(int bm, int bn) {
  if (bm == 64 && bn == 64) return igemm_buf_launch<DT, 64, 64, 2, 2, 3, false, 2>;
  return nullptr;
}

LaunchFn buf_groups_kernel(int dtype, int bm, int bn) {
  if (dtype == kBF16) return pick_groups<kBF16>(bm, bn);
  if (dtype == kF16) return pick_groups<kF16>(bm, bn);
  return nullptr;
}

LaunchFn buf_splitk_kernel(int dtype, int bm, int bn) {
  if (dtype == kBF16) return pick_splitk<kBF16>(bm, bn);
  if (dtype == kF16) return pick_splitk<kF16>(bm, bn);
  return nullptr;
}

LaunchFn buf_kernel(int dtype, int bm, int bn, bool shallow) {
  if (dtype == kBF16) return shallow ? pick_shallow<kBF16>(bm, bn) : pick<kBF16>(bm, bn);
  if (dtype == kF16) return shallow ? pick_shallow<kF16>(bm, bn) : pick<kF16>(bm, bn);
  return nullptr;
}

}  // namespace sc
