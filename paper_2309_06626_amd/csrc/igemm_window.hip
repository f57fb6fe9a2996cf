// Instantiations of the window kernel (16-bit operands, float accumulate).
#include "igemm_window_kernel.hpp"

namespace sc {

template <int DT>
static LaunchFn pick(int bm, int bn) {
  if (bm == 256 && bn == 128) return igemm_window_launch<DT, 256, 128>;
  if (bm == 128 && bn == 128) return igemm_window_launch<DT, 128, 128>;
  if (bm == 128 && bn == 64) return igemm_window_launch<DT, 128, 64>;
  if (bm == 64 && bn == 128) return igemm_window_launch<DT, 64, 128>;
  if (bm == 64 && bn == 64) return igemm_window_launch<DT, 64, 64>;
  return nullptr;
}

LaunchFn window_kernel(int dtype, int bm, int bn) {
  if (dtype == kBF16) return pick<kBF16>(bm, bn);
  if (dtype == kF16) return pick<kF16>(bm, bn);
  return nullptr;
}

size_t window_lds_bytes(int bm, int bn, int slab_bytes, int chunks) {
  if (bm == 256) return win_lds_bytes<256, 128>(slab_bytes, chunks);
  if (bm == 128) return bn == 128 ? win_lds_bytes<128, 128>(slab_bytes, chunks) : win_lds_bytes<128, 64>(slab_bytes, chunks);
  return bn == 128 ? win_lds_bytes<64, 128>(slab_bytes, chunks) : win_lds_bytes<64, 64>(slab_bytes, chunks);
}

}  // namespace sc
