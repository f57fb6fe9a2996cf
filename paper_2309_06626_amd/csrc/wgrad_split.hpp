// Filter gradient of float layers on the bf16 matrix pipes (wgrad_split.hip).
#pragma once
#include "conv_params.hpp"

namespace sc {

struct WgradSplitParams {
  const void* x;
  const void* g;             // g map [M][Cout]
  const int32_t* row_idx;    // kept rows, or null for the identity
  float* out;                // [splits][Cout][K]
  int32_t rows, rows_per_split, splits;
  int32_t h, w, c_in, ho_wo, wo, c_out;
  int32_t kh, kw, sh, sw, ph, pw, dil_h, dil_w;
  int32_t k;                 // kh * kw * c_in
  int32_t co_tiles, k_tiles;
  uint32_t x_bytes, g_bytes;
  uint32_t div_howo_mul, div_howo_shift, div_wo_mul, div_wo_shift;
};

constexpr int kWsTile = 64;        // output channels and window entries of a workgroup
constexpr int kWsRows = 64;        // kept rows of a step of the workgroup: 16 per wavefront

// windows up to 8 x 8 (validity bits), tensors below 2 GiB (32-bit byte offsets)
inline bool wgrad_split_applies(int kh, int kw, uint64_t x_bytes, uint64_t g_bytes) {
  return kh <= 8 && kw <= 8 && x_bytes < (1ull << 31) && g_bytes < (1ull << 31);
}
// row splits: two workgroups per compute unit, at least two steps each
inline int wgrad_split_splits(int64_t rows, int c_out, int k, size_t most_bytes) {
  const int64_t tiles = (int64_t)((c_out + kWsTile - 1) / kWsTile) * ((k + kWsTile - 1) / kWsTile);
  int64_t want = 512 / tiles;
  const int64_t by_rows = (rows + 2 * kWsRows - 1) / (2 * kWsRows), by_bytes = (int64_t)(most_bytes / ((size_t)c_out * k * 4));
  want = want < by_rows ? want : by_rows;
  want = want < by_bytes ? want : by_bytes;
  return (int)(want > 1 ? want : 1);
}
hipError_t wgrad_split_launch(const WgradSplitParams& p, hipStream_t stream);

}  // namespace sc
