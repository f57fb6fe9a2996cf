// Instantiations of the window kernel (16-bit operands, float accumulate).
#include "igemm_window_kernel.hpp"

namespace sc {

template <int DT, int KS>
static LaunchFn pick(int bm, int bn) {
  if (bm == 256 && bn == 128) return igemm_window_launch<DT, 256, 128, KS>;
  if (bm == 128 && bn == 128) return igemm_window_launch<DT, 128, 128, KS>;
  if (bm == 128 && bn == 64) return igemm_window_launch<DT, 128, 64, KS>;
  if (bm == 64 && bn == 128) return igemm_window_launch<DT, 64, 128, KS>;
  if (bm == 64 && bn == 64) return igemm_window_launch<DT, 64, 64, KS>;
  return nullptr;
}

LaunchFn window_kernel(int dtype, int ks, int bm, int bn) {
  if (dtype == kBF16) return ks == 3 ? pick<kBF16, 3>(bm, bn) : ks == 5 ? pick<kBF16, 5>(bm, bn) : nullptr;
  if (dtype == kF16) return ks == 3 ? pick<kF16, 3>(bm, bn) : ks == 5 ? pick<kF16, 5>(bm, bn) : nullptr;
  return nullptr;
}

size_t window_lds_bytes(int bm, int bn, int slab_bytes, int chunks) {
  if (bm == 256) return win_lds_bytes<256, 128>(slab_bytes, chunks);
  if (bm == 128) return bn == 128 ? win_lds_bytes<128, 128>(slab_bytes, chunks) : win_lds_bytes<128, 64>(slab_bytes, chunks);
  return bn == 128 ? win_lds_bytes<64, 128>(slab_bytes, chunks) : win_lds_bytes<64, 64>(slab_bytes, chunks);
}

}  // namespace sc
