// Instantiations of the register-staged tiled kernel, and the plan-time kernels that pack its filters and its gather table.
#include "igemm_stage_kernel.hpp"

namespace sc {

template <int DT, int GATHER, bool NCHW>
static LaunchFn stage_tile(int bm, int bn, int groups) {
  if (groups == 2) {
    if (bm == 64 && bn == 128) return igemm_stage_launch<DT, 64, 128, 2, 2, GATHER, NCHW, 2>;
    if (bm == 64 && bn == 64) return igemm_stage_launch<DT, 64, 64, 2, 2, GATHER, NCHW, 2>;
    return nullptr;
  }
  if (groups != 1) return nullptr;
  if (bm == 128 && bn == 64) return igemm_stage_launch<DT, 128, 64, 2, 2, GATHER, NCHW>;
  if (bm == 128 && bn == 32) return igemm_stage_launch<DT, 128, 32, 4, 1, GATHER, NCHW>;
  if (bm == 64 && bn == 128) return igemm_stage_launch<DT, 64, 128, 2, 2, GATHER, NCHW>;
  if (bm == 64 && bn == 64) return igemm_stage_launch<DT, 64, 64, 2, 2, GATHER, NCHW>;
  return nullptr;
}

template <int DT>
static LaunchFn stage_gather(int gather, bool nchw, int bm, int bn, int groups) {
  if (gather == kStageRaggedGroups) return stage_tile<DT, kStageRaggedGroups, false>(bm, bn, groups);
  if (gather == kStageChunks) return stage_tile<DT, kStageChunks, true>(bm, bn, groups);
  if (gather == kStageEntries)
    return nchw ? stage_tile<DT, kStageEntries, true>(bm, bn, groups) : stage_tile<DT, kStageEntries, false>(bm, bn, groups);
  if constexpr (DT == kF32) {
    if (gather == kStageGroups) return stage_tile<DT, kStageGroups, false>(bm, bn, groups);
  }
  return nullptr;          // (16-byte groups of a 16-bit type go straight into LDS: other kernels)
}

LaunchFn stage_kernel(int dtype, int gather, bool nchw, int bm, int bn, int groups) {
  if (dtype == kF32) return stage_gather<kF32>(gather, nchw, bm, bn, groups);
  if (dtype == kF16) return stage_gather<kF16>(gather, nchw, bm, bn, groups);
  return stage_gather<kBF16>(gather, nchw, bm, bn, groups);
}

// The K order of a gather: entry k of the tiles is channel `ci` of tap `tap`, or a filter entry that stays zero.
struct StageOrder {
  int gather, v, c_in, taps, cpad;
  __device__ bool at(int k, int* tap, int* ci) const {
    if (gather <= kStageRaggedGroups) {
      *tap = k / cpad;
      int e = k - *tap * cpad;
      if (e + v >= cpad && cpad > c_in) {              // the pixel's last group ends at its last channel
        e += c_in - cpad;
        *ci = e;
        return *tap < taps && e >= cpad - v;          // (what it repeats of the group before meets zeros)
      }
      *ci = e;
    } else {
      *tap = k / c_in;
      *ci = k - *tap * c_in;
    }
    return *tap < taps;
  }
};

// Eight filter entries in three parts, K steps of a part apart.  An entry that is not finite, or becomes so by the scaling, is
// stored as its two halves with a second part that is not a number, so that every sum it enters asks for the careful pass.
__device__ __forceinline__ void store_filter_parts(const float (&e)[8], v4i* __restrict__ dst) {
  using D = StageDims<kF32>;
  uint16_t parts[3][8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t bits = __builtin_bit_cast(uint32_t, e[i]);
    const float v = e[i] * kPartScale, a = (float)(__bf16)v, r = v - a, b = (float)(__bf16)r, c = r - b;
    const bool fits = (__builtin_bit_cast(uint32_t, a) & 0x7f800000u) != 0x7f800000u;
    parts[0][i] = (uint16_t)((fits ? __builtin_bit_cast(uint32_t, a) : bits) >> 16);
    parts[1][i] = fits ? (uint16_t)(__builtin_bit_cast(uint32_t, b) >> 16) : (uint16_t)0x7fc0;
    parts[2][i] = fits ? (uint16_t)(__builtin_bit_cast(uint32_t, c) >> 16) : (uint16_t)bits;
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    v4i v;
    __builtin_memcpy(&v, parts[q], 16);
    dst[q * D::KSTEPS * 64] = v;
  }
}

// One thread per 16 bytes of the packed filters: [32 channels][K tile][part][K step][lane].  Channel rows are permuted so
// that a lane of the MFMA result owns 16 consecutive channels.
template <int DT>
__global__ void stage_pack_kernel(const typename Elem<DT>::T* __restrict__ w, v4i* __restrict__ wp, StageOrder o, int c_out,
                                  int blocks, int k_tiles, int kh, int kw, int nchw) {
  using D = StageDims<DT>;
  using T = typename Elem<DT>::T;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)blocks * k_tiles * D::KSTEPS * 64) return;
  const int lane = (int)(idx & 63);
  const int64_t unit = idx >> 6;
  const int ks = (int)(unit % D::KSTEPS);
  const int64_t tile = unit / D::KSTEPS;
  const int kt = (int)(tile % k_tiles), nb = (int)(tile / k_tiles);
  const int m = lane & 31, half = lane >> 5;
  const int co = nb * 32 + 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3);
  T e[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    int tap, ci;
    const bool real = o.at(kt * D::K_TILE + (2 * ks + half) * 8 + i, &tap, &ci) && co < c_out;
    e[i] = !real ? (T)0.0f : nchw ? w[((int64_t)co * o.c_in + ci) * o.taps + tap] : w[((int64_t)co * o.taps + tap) * o.c_in + ci];
  }
  v4i* dst = wp + tile * (D::BLOCK_BYTES / 16) + ks * 64 + lane;
  if constexpr (DT == kF32) {
    store_filter_parts(e, dst);
  } else {
    v4i v;
    __builtin_memcpy(&v, e, 16);
    dst[0] = v;
  }
}

// Table entry: byte offset from the window's corner, and the validity bits its tap needs.
__global__ void stage_table_kernel(KEntry* __restrict__ tab, int entries, int per, StageOrder o, int kw, int dil_h, int dil_w,
                                   int eb, int xs_h, int xs_w, int xs_c) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= entries) return;
  int tap, ci;
  // (of a last group the entry that counts is its last one: the group ends there)
  o.at(i * per, &tap, &ci);
  KEntry e;
  e.off = 0;
  e.dydx = (int32_t)kStageNoTap;
  if (tap < o.taps) {
    const int ky = tap / kw, kx = tap % kw;
    e.off = (ky * dil_h * xs_h + kx * dil_w * xs_w + ci * xs_c) * eb;
    uint32_t bits = (1u << ky) | (1u << (8 + kx));
    if (o.gather == kStageRaggedGroups && (i * per) % o.cpad + per == o.cpad) bits |= kStageTail;
    e.dydx = (int32_t)bits;
  }
  tab[i] = e;
}

hipError_t stage_pack(int dtype, int gather, const void* w, void* wp, KEntry* tab, int c_out, int blocks, int c_in, int kh, int kw,
                      int dil_h, int dil_w, int k_tiles, bool nchw, int h, int w_cols, hipStream_t stream) {
  const int v = dtype == kF32 ? 4 : 8, eb = dtype == kF32 ? 4 : 2;
  const StageOrder o = {gather, v, c_in, kh * kw, (c_in + v - 1) / v * v};
  const int ksteps = dtype == kF32 ? StageDims<kF32>::KSTEPS : StageDims<kBF16>::KSTEPS;
  const int64_t total = (int64_t)blocks * k_tiles * ksteps * 64;
  const dim3 grid((unsigned)((total + 255) / 256)), block(256);
  if (!w) (void)0;      // (the table alone)
  else if (dtype == kF32)
    hipLaunchKernelGGL(stage_pack_kernel<kF32>, grid, block, 0, stream, (const float*)w, (v4i*)wp, o, c_out, blocks, k_tiles, kh, kw, nchw ? 1 : 0);
  else      // 16-bit patterns are moved verbatim
    hipLaunchKernelGGL(stage_pack_kernel<kF16>, grid, block, 0, stream, (const _Float16*)w, (v4i*)wp, o, c_out, blocks, k_tiles, kh, kw, nchw ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !tab) return e;
  const int per = gather <= kStageRaggedGroups ? v : gather == kStageChunks ? 8 : 1;
  const int entries = k_tiles * (dtype == kF32 ? StageDims<kF32>::K_TILE : StageDims<kBF16>::K_TILE) / per;
  const int xs_h = nchw ? w_cols : w_cols * c_in, xs_w = nchw ? 1 : c_in, xs_c = nchw ? h * w_cols : 1;
  hipLaunchKernelGGL(stage_table_kernel, dim3((entries + 255) / 256), dim3(256), 0, stream, tab, entries, per, o, kw, dil_h, dil_w, eb,
                     xs_h, xs_w, xs_c);
  return hipGetLastError();
}

// Filters of an NHWC layer whose channels are whole 16-byte groups, into the layout of the tiled and band kernels
// ([channel row][K], rows permuted like above) and, for float, into the parts of the direct-to-LDS kernel: one launch, 16
// bytes a thread.  ROT: `w` holds the filters of the layer whose input gradient this is ([Cin][kh][kw][Cout], rotated by 180
// degrees); lanes then run over the channel rows, along which those lie.
template <int DT, bool ROT>
__global__ void repack_kernel(const typename Elem<DT>::T* __restrict__ w, v4i* __restrict__ wp, v4i* __restrict__ parts, int c_out,
                              int c_in, int taps, int k_stride, int rows, int row_blocks, int part_blocks, int k_tiles) {
  using D = StageDims<DT>;
  using T = typename Elem<DT>::T;
  constexpr int V = Elem<DT>::V;
  const int k = taps * c_in;
  auto channel = [](int row) { return (row & ~31) + 16 * ((row >> 2) & 1) + 4 * ((row & 31) >> 3) + (row & 3); };
  auto group = [&](int co, int kk, T* dst) {        // V entries from kk on: one tap
    if (co >= c_out || kk >= k) {
#pragma unroll
      for (int i = 0; i < V; ++i) dst[i] = (T)0.0f;
      return;
    }
    if constexpr (ROT) {
      const int tap = kk / c_in, ci = kk - tap * c_in;
#pragma unroll
      for (int i = 0; i < V; ++i) dst[i] = w[((int64_t)(ci + i) * taps + taps - 1 - tap) * c_out + co];
    } else {
      const v4i v = *reinterpret_cast<const v4i*>(w + (int64_t)co * k + kk);
      __builtin_memcpy(dst, &v, 16);
    }
  };
  if ((int)blockIdx.x < row_blocks) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x, per_row = k_stride / V;
    int row, g;
    if constexpr (ROT) {
      const int rest = idx >> 5;
      g = rest % per_row;
      row = rest / per_row * 32 + (idx & 31);
    } else {
      row = idx / per_row;
      g = idx - row * per_row;
    }
    if (row >= rows) return;
    T e[V];
    group(channel(row), g * V, e);
    v4i v;
    __builtin_memcpy(&v, e, 16);
    wp[(int64_t)row * per_row + g] = v;
    return;
  }
  if constexpr (DT != kF32) {      // for the window kernel: [32 channels][chunk][K step][tap][lane], k_tiles chunks
    const int idx = (blockIdx.x - row_blocks) * blockDim.x + threadIdx.x;
    // (the four wavefronts of a workgroup take the four K steps of a tap, so that the 128 bytes of a chunk are read by one compute unit;
    // with taps side by side instead they came from L2 four times: 512 -> 512 3x3 7.8 -> 6.4 us a launch, 128 -> 128 the same)
    const int lane = idx & 63, unit = idx >> 6, ks = unit & 3, part = unit >> 2, tap = part % taps, rest = part / taps;
    const int chunk = rest % k_tiles, nb = rest / k_tiles;
    if (nb >= part_blocks) return;
    T e[8];
    const int ci = chunk * 64 + ks * 16 + (lane >> 5) * 8;
    group(nb * 32 + channel(lane & 31), ci < c_in ? tap * c_in + ci : k, e);      // (zeros behind the last channel)
    v4i v;
    __builtin_memcpy(&v, e, 16);
    parts[((rest * 4 + ks) * taps + tap) * 64 + lane] = v;
  }
  if constexpr (DT == kF32) {
    const int idx = (blockIdx.x - row_blocks) * blockDim.x + threadIdx.x;
    const int lane = idx & 63, unit = idx >> 6, ks = unit % D::KSTEPS, tile = unit / D::KSTEPS;
    const int kt = tile % k_tiles, nb = tile / k_tiles;
    if (nb >= part_blocks) return;
    const int co = nb * 32 + channel(lane & 31), kk = kt * D::K_TILE + (2 * ks + (lane >> 5)) * 8;
    float e[8];
    group(co, kk, e);
    group(co, kk + 4, e + 4);
    store_filter_parts(e, parts + (int64_t)tile * (D::BLOCK_BYTES / 16) + ks * 64 + lane);
  }
}

hipError_t repack_filters(int dtype, const void* w, void* wp, void* parts, int c_out, int c_in, int taps, int k_stride, int rows,
                          int part_blocks, int k_tiles, bool rotated, hipStream_t stream) {
  const int v = dtype == kF32 ? 4 : 8;
  const int row_blocks = (int)(((int64_t)rows * (k_stride / v) + 255) / 256);
  const int64_t units = (int64_t)part_blocks * k_tiles * (dtype == kF32 ? StageDims<kF32>::KSTEPS : 4 * taps);
  const int blocks = row_blocks + (parts ? (int)((units * 64 + 255) / 256) : 0);
  auto launch = [&](auto kern, auto* src) {
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, stream, src, (v4i*)wp, (v4i*)parts, c_out, c_in, taps, k_stride, rows, row_blocks,
                       part_blocks, k_tiles);
  };
  if (dtype == kF32) {
    if (rotated) launch(repack_kernel<kF32, true>, (const float*)w);
    else launch(repack_kernel<kF32, false>, (const float*)w);
  } else {       // 16-bit patterns are moved verbatim
    if (rotated) launch(repack_kernel<kF16, true>, (const _Float16*)w);
    else launch(repack_kernel<kF16, false>, (const _Float16*)w);
  }
  return hipGetLastError();
}

}  // namespace sc
