// Host side of the C ABI (validation, workspace carving, tile choice, launches) and the small
// plan-time kernels: mask -> row-index compaction, filter packing, gather-table build, and
// the glue operators of the test networks.
#include "../../include/sparse_conv.h"

#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <numeric>
#include <new>

#include "band_kernel.hpp"
#include "bandpp_kernel.hpp"
#include "bandrow_kernel.hpp"
#include "bandstream_kernel.hpp"
#include "bandtap_kernel.hpp"
#include "conv_params.hpp"
#include "igemm_buf_kernel.hpp"
#include "igemm_slab_kernel.hpp"
#include "igemm_split_kernel.hpp"
#include "igemm_stage_kernel.hpp"
#include "igemm_streamk_kernel.hpp"
#include "igemm_window_kernel.hpp"
#include "igemm_panel_kernel.hpp"

namespace sc {

static thread_local int32_t g_last_hip = 0;
#ifdef SC_TIMING
static long long* g_dbg = nullptr;   // development builds only
#endif

static inline bool hip_failed(hipError_t e) {
  if (e != hipSuccess) { g_last_hip = (int32_t)e; return true; }
  return false;
}
#define SC_HIP(expr) do { if (hip_failed((expr))) return SC_ERR_HIP; } while (0)

// the other translation units of the library report their HIP failures through this
void note_hip_error(int32_t code) { g_last_hip = code; }

// ------------------------------------------------------------------------------------------------
// Mask -> ascending list of kept rows (Alg. 2, indirection init: positions are visited in
// ascending order and appended only where the mask is set).  Two passes, no inter-workgroup
// waiting: each wavefront owns a segment of kSeg rows; pass 1 counts with ballots, pass 2 sums
// the counts of the earlier segments and scatters with ballot + lane rank.
// ------------------------------------------------------------------------------------------------
constexpr int kSeg = 1024;

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// (copy, may be null: the plan's private copy of the mask, mask_len bytes, written on the way -- the first mask_len
// rows read exactly those bytes)
__global__ __launch_bounds__(256) void mask_count_kernel(const uint8_t* __restrict__ mask, int m, int period,
                                                         int nseg, int32_t* __restrict__ counts,
                                                         uint8_t* __restrict__ copy, int mask_len) {
  const int lane = threadIdx.x & 63;
  const int seg = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (seg >= nseg) return;
  const int r0 = seg * kSeg;
  int cnt = 0;
  for (int it = 0; it < kSeg / 64; ++it) {
    int r = r0 + it * 64 + lane;
    const uint8_t v = r < m ? mask[period ? r % period : r] : (uint8_t)0;
    if (copy && r < mask_len) copy[r] = v;
    bool keep = v != 0;
    cnt += __popcll(__ballot(keep));
  }
  if (lane == 0) counts[seg] = cnt;
}

__global__ __launch_bounds__(256) void mask_scatter_kernel(const uint8_t* __restrict__ mask, int m, int period,
                                                           int nseg, const int32_t* __restrict__ counts,
                                                           int32_t* __restrict__ row_idx,
                                                           int32_t* __restrict__ kept_out) {
  const int lane = threadIdx.x & 63;
  const int seg = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (seg >= nseg) return;
  int part = 0;
  for (int i = lane; i < seg; i += 64) part += counts[i];
  int base = wave_sum(part);
  const int r0 = seg * kSeg;
  for (int it = 0; it < kSeg / 64; ++it) {
    int r = r0 + it * 64 + lane;
    bool keep = r < m && mask[period ? r % period : r] != 0;
    unsigned long long b = __ballot(keep);
    int rank = __popcll(b & ((1ull << lane) - 1ull));
    if (keep) row_idx[base + rank] = r;
    base += __popcll(b);
  }
  if (seg == nseg - 1 && lane == 0) {
    kept_out[0] = base;
    kept_out[1] = 0;      // the per-band maximum, raised by band_rows_kernel
    kept_out[2] = 0;      // the widest slab of a 64-row / 128-row / 256-row tile, raised by slab_span_kernel
    kept_out[3] = kept_out[4] = 0;
  }
}

// Slab and window kernels: virtual rows between the window corner of the first and of the last kept row of every tile of 64, 128 and
// 256 kept rows, plus the window height; the maximum over the tiles sizes the LDS slab.
__global__ __launch_bounds__(256) void slab_span_kernel(const int32_t* __restrict__ row_idx, const int32_t* __restrict__ kept_dev,
                                                        int ho_wo, int wo, int hp, int kh, int32_t* __restrict__ span_out) {
  __shared__ int s_span[3];
  if (threadIdx.x < 3) s_span[threadIdx.x] = 0;
  __syncthreads();
  const int kept = kept_dev[0];
  const int tile = blockIdx.x * 256 + threadIdx.x;
  auto vrow = [&](int r) { return (r / ho_wo) * hp + (r % ho_wo) / wo; };
  for (int b = 0; b < 3; ++b) {
    const int bm = 64 << b;
    const int64_t m0 = (int64_t)tile * bm;
    if (m0 >= kept) continue;
    const int last = (int)min((int64_t)kept, m0 + bm) - 1;
    atomicMax(&s_span[b], vrow(row_idx[last]) + kh - vrow(row_idx[m0]));
  }
  __syncthreads();
  if (threadIdx.x < 3) atomicMax(span_out + threadIdx.x, s_span[threadIdx.x]);
}

// The inverse map for a compact tensor: rank[r] = position of row r among the kept rows, -1 for a dropped
// row.  Same two passes (counts from mask_count_kernel).
__global__ __launch_bounds__(256) void mask_rank_kernel(const uint8_t* __restrict__ mask, int m, int period,
                                                        int nseg, const int32_t* __restrict__ counts,
                                                        int32_t* __restrict__ rank_out,
                                                        int32_t* __restrict__ kept_out) {
  const int lane = threadIdx.x & 63;
  const int seg = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (seg >= nseg) return;
  int part = 0;
  for (int i = lane; i < seg; i += 64) part += counts[i];
  int base = wave_sum(part);
  const int r0 = seg * kSeg;
  for (int it = 0; it < kSeg / 64; ++it) {
    int r = r0 + it * 64 + lane;
    bool keep = r < m && mask[period ? r % period : r] != 0;
    unsigned long long b = __ballot(keep);
    int rank = __popcll(b & ((1ull << lane) - 1ull));
    if (r < m) rank_out[r] = keep ? base + rank : -1;
    base += __popcll(b);
  }
  if (seg == nseg - 1 && lane == 0) *kept_out = base;
}

// ------------------------------------------------------------------------------------------------
// Filter packing: [cout_pad][k_pad] with K = (ky, kx, ci) contiguous, zero padded.  Inside every
// group of 32 output channels the rows are permuted so that MFMA output row 8j + 4h + i holds
// channel 16h + 4j + i: a lane of the result then owns 16 consecutive channels.
// ------------------------------------------------------------------------------------------------
// epad > 0 selects the row-segment K order of the small-channel gather: K' = (ky, e) with e = kx*c_in + ci
// padded to epad entries per window row (the padding holds zeros).
template <typename T>
__global__ void pack_filters_kernel(const T* __restrict__ w, T* __restrict__ wp, int c_out, int c_in, int kh, int kw,
                                    int k, int k_pad, int cout_pad, int nchw, int epad) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)cout_pad * k_pad) return;
  int prow = (int)(idx / k_pad), kk = (int)(idx % k_pad);
  int rho = prow & 31;
  int co = (prow & ~31) + 16 * ((rho >> 2) & 1) + 4 * (rho >> 3) + (rho & 3);
  T v = (T)0.0f;
  bool real = co < c_out && kk < k;
  if (epad > 0 && real) {
    int ky = kk / epad, e = kk % epad;
    real = e < kw * c_in;
    kk = ky * kw * c_in + e;   // position in the plain (ky, kx, ci) order
  }
  if (real) {
    int tap = kk / c_in, ci = kk % c_in;
    int ky = tap / kw, kx = tap % kw;
    int64_t src = nchw ? (((int64_t)co * c_in + ci) * kh + ky) * kw + kx
                       : (((int64_t)co * kh + ky) * kw + kx) * c_in + ci;
    v = w[src];
  }
  wp[idx] = v;
}

// Gather table: entry g covers K entries [g*vec, (g+1)*vec) (vec = 1 for the element gather).
__global__ void build_ktab_kernel(KEntry* __restrict__ tab, int entries, int vec, int k, int c_in, int kw, int dil_h,
                                  int dil_w, int xs_h, int xs_w, int xs_c) {
  int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= entries) return;
  int kk = g * vec;
  KEntry e;
  if (kk < k) {
    int tap = kk / c_in, ci = kk % c_in;
    int dy = (tap / kw) * dil_h, dx = (tap % kw) * dil_w;
    e.off = dy * xs_h + dx * xs_w + ci * xs_c;
    e.dydx = dy | (dx << 16);
  } else {
    e.off = 0;
    e.dydx = 0x7fff;  // row offset no image reaches: the padded K entries read as zero
  }
  tab[g] = e;
}

// Small-channel gather: copy x [N][H][W][C] into the interior of the zero-margined buffer
// [N][Hp][Wp][C] (margins are zeroed once at plan time), 16 bytes per thread; rows of W*C elements are
// a multiple of 8 elements here.
template <typename T>
__global__ void pad_input_kernel(const T* __restrict__ x, T* __restrict__ xp, int n, int h, int row_elems, int hp,
                                 int prow_elems, int top, int left_elems) {
  typedef T vec8 __attribute__((ext_vector_type(8)));
  const int gpr = row_elems >> 3;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = (int64_t)n * h * gpr;
  if (idx >= total) return;
  int g = (int)(idx % gpr);
  int64_t r = idx / gpr;
  int iy = (int)(r % h), b = (int)(r / h);
  const vec8 v = *reinterpret_cast<const vec8*>(x + r * row_elems + g * 8);
  T* dst = xp + ((int64_t)b * hp + iy + top) * prow_elems + left_elems + g * 8;
  __builtin_memcpy(dst, &v, 16);   // destination is only element-aligned
}

__global__ void fill_zero_kernel(uint4* __restrict__ dst, int64_t n16, unsigned char* tail, int ntail) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) dst[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

// First compacted row of every band: lower bound of the band's first dense row in the kept-row list.
__global__ void band_start_kernel(const int32_t* __restrict__ row_idx, const int32_t* __restrict__ kept_dev,
                                  int32_t* __restrict__ band_i0, int n_bands, int bands_per_image, int bh, int split,
                                  int ho, int wo) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b > n_bands) return;
  const int kept = *kept_dev;
  int target;
  if (b == n_bands) {
    target = 0x7fffffff;
  } else {
    int img = b / bands_per_image, first, end;
    band_pixel_range(b - img * bands_per_image, bh, split, ho, wo, &first, &end);
    target = img * ho * wo + first;
  }
  int lo = 0, hi = kept;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (row_idx[mid] < target) lo = mid + 1; else hi = mid;
  }
  band_i0[b] = lo;
}

// Band-ordered copy of the kept-row list: the kept rows of band b, ascending, stored from index
// r_lo(b) (the band's first dense row) on, so the band kernel finds them without knowing counts.
// The first kept row of every band also raises band_max to the band's kept-row count (it sizes the accumulator blocks of
// the streaming kernel and picks the MFMA block shape of the others: the fullest band is the one a launch waits for).
__global__ void band_rows_kernel(const int32_t* __restrict__ row_idx, const int32_t* __restrict__ kept_dev,
                                 const int32_t* __restrict__ band_i0, int32_t* __restrict__ band_rows,
                                 int bands_per_image, int bh, int split, int ho, int wo, int32_t* __restrict__ band_max) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= *kept_dev) return;
  const int r = row_idx[i];
  const int ho_wo = ho * wo;
  const int img = r / ho_wo;
  const int bi = band_of_pixel(r - img * ho_wo, bh, split, ho, wo);
  const int band = img * bands_per_image + bi;
  int first, end;
  band_pixel_range(bi, bh, split, ho, wo, &first, &end);
  const int i0 = band_i0[band];
  band_rows[img * ho_wo + first + (i - i0)] = r;
  if (i == i0) atomicMax(band_max, band_i0[band + 1] - i0);
}

// ------------------------------------------------------------------------------------------------
// The same tables -- row list, private mask copy, band starts, band-ordered rows -- and the spans of slabs in
// ONE launch, for maps of up to kTableMostRows rows.  A workgroup owns 1 024 rows and counts the ones in front of them by
// itself (16-byte loads of a mask that lies in L2) instead of waiting for a pass of its own, so a refresh of a small map is
// one launch in place of four or five.  Every workgroup leaves what the host wants to know -- its kept rows, the fullest
// band that ends in its rows, the spans -- in host memory (`result`, kTableWords words each), where the host finds it behind the
// synchronisation without a copy.
// ------------------------------------------------------------------------------------------------
constexpr int kTableThreads = 256, kTableRows = 4 * kTableThreads;
constexpr int kTableMostRows = 1 << 17, kTableMostWgs = kTableMostRows / kTableRows;
// Words that a workgroup leaves for the host: kept rows, most kept rows of a band; for tiles of 64, 128 and 256 kept rows the widest span of
// those inside the segment, the virtual row at which the one open at its end begins and at which the one open at its start ends (-1: none);
// the virtual row of its last kept row.
enum { kTableKept, kTableFullest, kTableInner, kTableOpen = kTableInner + 3, kTableClose = kTableOpen + 3, kTableEnd = kTableClose + 3, kTableWords };

// The widest span of a tile of 64, 128 and 256 kept rows, in virtual rows, from the words of all workgroups in order.
static void table_spans(const int32_t* words, int wgs, int kh, int32_t (&span)[3]) {
  for (int b = 0; b < 3; ++b) {
    int open = -1, end = -1;
    span[b] = 0;
    for (int i = 0; i < wgs; ++i) {
      const int32_t* w = words + i * kTableWords;
      span[b] = std::max(span[b], w[kTableInner + b]);
      if (w[kTableClose + b] >= 0) {
        span[b] = std::max(span[b], w[kTableClose + b] + kh - open);
        open = -1;
      }
      if (w[kTableOpen + b] >= 0) open = w[kTableOpen + b];
      if (w[kTableEnd] >= 0) end = w[kTableEnd];
    }
    if (open >= 0) span[b] = std::max(span[b], end + kh - open);      // the last tile, which the kept rows do not fill
  }
}

struct TableParams {
  const uint8_t* mask;
  uint8_t* copy;
  int32_t *row_idx, *kept_out, *band_i0, *band_rows, *result;
  int32_t m, period, mask_len;
  int32_t n_bands, bands_per_image, bh, split, ho, wo;      // n_bands == 0: no band tables
  int32_t slab_hp, slab_kh;                                 // slab_hp == 0: no spans
  uint32_t howo_mul, howo_shift, wo_mul, wo_shift, bh_mul, bh_shift;
};

__global__ __launch_bounds__(kTableThreads) void row_tables_kernel(const TableParams p) {
  __shared__ unsigned long long s_bits[kTableRows / 64];    // which rows of the segment are kept
  __shared__ int s_before[kTableRows / 64];                 // kept rows of the segment in front of each word
  __shared__ int s_wave[4], s_red[3];
  constexpr int TILES = kTableRows / 64 + 1;                // tiles of 64 kept rows that a segment touches
  __shared__ int s_tile[2][TILES];                          // virtual rows of their first and last rows (-1: not of this segment)
  __shared__ int s_out[kTableWords];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int r0 = blockIdx.x * kTableRows;
  const int ho_wo = p.ho * p.wo;

  // the segment's rows, and where a band that began in front of it started
  unsigned char v[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int r = r0 + wave * 256 + it * 64 + lane;
    const int q = p.period ? r - fast_div(r, p.howo_mul, p.howo_shift) * p.period : r;
    v[it] = r < p.m ? p.mask[q] : (uint8_t)0;
    if (r < p.mask_len) p.copy[r] = v[it];
  }
  auto band_at = [&](int r, int* band, int* first, int* end) {      // rows [first, end) of the band that row r lies in
    const int img = fast_div(r, p.howo_mul, p.howo_shift), pix = r - img * ho_wo;
    const int run = fast_div(fast_div(pix, p.wo_mul, p.wo_shift), p.bh_mul, p.bh_shift);
    const int p0 = run * p.bh * p.wo, px = min(p.ho - run * p.bh, p.bh) * p.wo, half = (px + 1) >> 1;
    const int second = p.split && pix - p0 >= half ? 1 : 0;
    *band = img * p.bands_per_image + (p.split ? 2 * run + second : run);
    *first = img * ho_wo + p0 + (second ? half : 0);
    *end = img * ho_wo + p0 + (p.split && !second ? half : px);
  };
  int start = r0;
  if (p.n_bands && r0 > 0) {
    int band, end;
    band_at(r0, &band, &start, &end);
  }
  // kept rows in [0, start) and in [start, r0)
  auto kept_in = [&](int from, int to) {       // this thread's share of mask[from .. to)
    int n = 0;
    const uintptr_t base = (uintptr_t)p.mask;
    const int a = (int)min((int64_t)to, (int64_t)((from + base + 15) / 16 * 16 - base)), b = (int)max((int64_t)a, (int64_t)((to + base) / 16 * 16 - base));
    for (int i = from + t; i < a; i += kTableThreads) n += p.mask[i] != 0;
    for (int i = a + 16 * t; i < b; i += 4 * 16 * kTableThreads) {      // four loads on their way
      uint4 w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int at = i + u * 16 * kTableThreads;
        w[u] = at < b ? *reinterpret_cast<const uint4*>(p.mask + at) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t d[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) n += __popc((((d[e] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | d[e]) & 0x80808080u);
      }
    }
    for (int i = b + t; i < to; i += kTableThreads) n += p.mask[i] != 0;
    return n;
  };
  auto kept_before = [&](int r) {              // this thread's share of the kept rows in front of row r
    if (!p.period) return kept_in(0, r);
    const int img = fast_div(r, p.howo_mul, p.howo_shift), rem = r - img * p.period;
    return (img ? img * kept_in(0, p.period) : 0) + kept_in(0, rem);
  };
  if (t < 3) s_red[t] = 0;
  if (t < 2 * TILES) s_tile[t / TILES][t % TILES] = -1;
  if (t < kTableWords) s_out[t] = t >= kTableOpen ? -1 : 0;
  __syncthreads();
  if (r0 > 0) {
    const int to_start = wave_sum(kept_before(start)), to_r0 = wave_sum(start == r0 ? 0 : kept_before(r0));
    if (lane == 0) {
      atomicAdd(&s_red[0], to_start);
      atomicAdd(&s_red[1], start == r0 ? to_start : to_r0);
    }
  }
  int own = 0;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const unsigned long long bits = __ballot(v[it] != 0);
    if (lane == 0) { s_bits[wave * 4 + it] = bits; s_before[wave * 4 + it] = own; }
    own += __popcll(bits);
  }
  if (lane == 0) s_wave[wave] = own;
  __syncthreads();
  int before_wave = 0, total = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < wave) before_wave += s_wave[w];
    total += s_wave[w];
  }
  if (lane < 4) s_before[wave * 4 + lane] += before_wave;
  const int start_rank = s_red[0], base = s_red[1];
  __syncthreads();
  auto rank_at = [&](int r) {                  // kept rows in front of row r, a row of the segment or `start`
    if (r < r0) return start_rank;
    const int q = r - r0;
    return base + s_before[q >> 6] + (int)__popcll(s_bits[q >> 6] & ((1ull << (q & 63)) - 1ull));
  };
  auto mark = [&](int r, int rank) {           // for spans: a kept row that is the first or the last of 64, or the segment's last
    const bool first = (rank & 63) == 0, last = (rank & 63) == 63, end = rank == base + total - 1;
    if (!first && !last && !end) return;
    const int img = fast_div(r, p.howo_mul, p.howo_shift);
    const int vrow = img * p.slab_hp + fast_div(r - img * ho_wo, p.wo_mul, p.wo_shift);
    if (first) s_tile[0][(rank >> 6) - (base >> 6)] = vrow;
    if (last) s_tile[1][(rank >> 6) - (base >> 6)] = vrow;
    if (end) s_out[kTableEnd] = vrow;
  };
  int fullest = 0;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int r = r0 + wave * 256 + it * 64 + lane;
    if (r >= p.m) break;
    const bool keep = v[it] != 0;
    const int rank = rank_at(r);
    if (keep) p.row_idx[rank] = r;
    if (p.slab_hp && keep) mark(r, rank);
    if (p.n_bands) {
      int band, first, end;
      band_at(r, &band, &first, &end);
      const int i0 = rank_at(first);
      if (r == first) p.band_i0[band] = rank;
      if (keep) p.band_rows[first + (rank - i0)] = r;
      if (r == end - 1) fullest = max(fullest, rank + (keep ? 1 : 0) - i0);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) fullest = max(fullest, __shfl_xor(fullest, off, 64));
  if (lane == 0) atomicMax(&s_red[2], fullest);
  __syncthreads();
  if (p.slab_hp && t < TILES) {
    // Spans of the tiles of 64, 128 and 256 kept rows that lie in this segment whole.  A tile that crosses the segment's end leaves its
    // first virtual row there, one that crosses its start its last; the host puts the two together (table_spans).
    const int unit = (base >> 6) + t;
    for (int b = 0; b < 3; ++b) {
      const int n = 1 << b;
      if ((unit & (n - 1)) == 0 && s_tile[0][t] >= 0) {
        const int end = t + n - 1 < TILES ? s_tile[1][t + n - 1] : -1;
        if (end >= 0) atomicMax(&s_out[kTableInner + b], end + p.slab_kh - s_tile[0][t]);
        else s_out[kTableOpen + b] = s_tile[0][t];
      }
      if (((unit + 1) & (n - 1)) == 0 && s_tile[1][t] >= 0 && (t + 1 < n || s_tile[0][t + 1 - n] < 0)) s_out[kTableClose + b] = s_tile[1][t];
    }
  }
  if (t == 0) {
    s_out[kTableKept] = total;
    s_out[kTableFullest] = s_red[2];
  }
  __syncthreads();
  if (t < kTableWords) p.result[blockIdx.x * kTableWords + t] = s_out[t];
  if (t == 0 && blockIdx.x == gridDim.x - 1) {
    p.kept_out[0] = base + total;
    p.kept_out[1] = p.kept_out[2] = p.kept_out[3] = p.kept_out[4] = 0;
    if (p.n_bands) p.band_i0[p.n_bands] = base + total;
  }
}

// Host memory that kernels write their few words for the host into: kHostSlots slots in one allocation, made on first use
// (in a way that a capture in another thread is not disturbed by) and held until the process ends.  A call holds a slot from its
// launch to its synchronisation; one that finds none free (or no such memory), or whose stream is being captured, copies from
// the device instead.  SPARSE_CONV_HOST_SLOTS=0: always (tests).
constexpr int kHostSlots = 32, kHostSlotWords = kTableMostWgs * kTableWords;
struct HostSlots {
  std::mutex lock;
  int32_t* base = nullptr;
  bool tried = false;
  uint32_t used = 0;
  int32_t* take(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
    if (status != hipStreamCaptureStatusNone) return nullptr;      // (the call is refused at its synchronisation)
    if (const char* env = std::getenv("SPARSE_CONV_HOST_SLOTS"); env && env[0] == '0') return nullptr;
    std::lock_guard<std::mutex> hold(lock);
    if (!tried) {
      tried = true;
      void* mem = nullptr;
      hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
      const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
      if (hipHostMalloc(&mem, sizeof(int32_t) * kHostSlots * kHostSlotWords, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) base = static_cast<int32_t*>(mem);
      else (void)hipGetLastError();
      if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    if (!base) return nullptr;
    for (int i = 0; i < kHostSlots; ++i)
      if (!(used >> i & 1u)) { used |= 1u << i; return base + i * kHostSlotWords; }
    return nullptr;
  }
  void give_back(int32_t* slot) {
    std::lock_guard<std::mutex> hold(lock);
    used &= ~(1u << ((slot - base) / kHostSlotWords));
  }
};
static HostSlots g_host_slots;

// ------------------------------------------------------------------------------------------------
// Glue operators for network runs
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ void maxpool_nhwc_kernel(const T* __restrict__ x, T* __restrict__ y, int n, int h, int w, int c, int k,
                                    int s, int p, int ho, int wo) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = (int64_t)n * ho * wo * c;
  if (idx >= total) return;
  int ch = (int)(idx % c);
  int64_t pos = idx / c;
  int ox = (int)(pos % wo);
  int oy = (int)((pos / wo) % ho);
  int b = (int)(pos / ((int64_t)wo * ho));
  float best = -INFINITY;
  for (int ky = 0; ky < k; ++ky) {
    int iy = oy * s - p + ky;
    if (iy < 0 || iy >= h) continue;
    for (int kx = 0; kx < k; ++kx) {
      int ix = ox * s - p + kx;
      if (ix < 0 || ix >= w) continue;
      float v = (float)x[(((int64_t)b * h + iy) * w + ix) * c + ch];
      best = fmaxf(best, v);
    }
  }
  y[idx] = (T)best;
}

// 16-bit types, channel count a multiple of 8: a thread owns 8 consecutive channels of one output
// position (16-byte loads and stores; the scalar kernel above moves 2 bytes per thread and access)
template <typename T>
__global__ void maxpool_nhwc_vec8_kernel(const T* __restrict__ x, T* __restrict__ y, int n, int h, int w, int c, int k,
                                         int s, int p, int ho, int wo) {
  typedef T vec8 __attribute__((ext_vector_type(8)));
  const int cg = c >> 3;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = (int64_t)n * ho * wo * cg;
  if (idx >= total) return;
  int g = (int)(idx % cg);
  int64_t pos = idx / cg;
  int ox = (int)(pos % wo);
  int oy = (int)((pos / wo) % ho);
  int b = (int)(pos / ((int64_t)wo * ho));
  float best[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) best[e] = -INFINITY;
  for (int ky = 0; ky < k; ++ky) {
    int iy = oy * s - p + ky;
    if (iy < 0 || iy >= h) continue;
    for (int kx = 0; kx < k; ++kx) {
      int ix = ox * s - p + kx;
      if (ix < 0 || ix >= w) continue;
      const vec8 v = *reinterpret_cast<const vec8*>(x + (((int64_t)b * h + iy) * w + ix) * c + g * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) best[e] = fmaxf(best[e], (float)v[e]);
    }
  }
  vec8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (T)best[e];
  *reinterpret_cast<vec8*>(y + pos * c + g * 8) = o;
}

// The same for the 3x3 window: the nine loads are unconditional (clamped coordinates; a padded tap is replaced by
// minus infinity afterwards), so they are all in flight at once.
template <typename T>
__global__ void maxpool3_nhwc_vec8_kernel(const T* __restrict__ x, T* __restrict__ y, int n, int h, int w, int c, int s,
                                          int p, int ho, int wo, uint32_t cg_mul, uint32_t cg_shift, uint32_t wo_mul,
                                          uint32_t wo_shift, uint32_t ho_mul, uint32_t ho_shift) {
  typedef T vec8 __attribute__((ext_vector_type(8)));
  const int cg = c >> 3;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;          // (the launcher keeps n * ho * wo * cg below 2^31)
  if (idx >= n * ho * wo * cg) return;
  const int pos = fast_div(idx, cg_mul, cg_shift), g = idx - pos * cg;
  const int row = fast_div(pos, wo_mul, wo_shift), ox = pos - row * wo;
  const int b = fast_div(row, ho_mul, ho_shift), oy = row - b * ho;
  const int iy0 = oy * s - p, ix0 = ox * s - p;
  vec8 v[9];
  bool ok[9];
#pragma unroll
  for (int ky = 0; ky < 3; ++ky)
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      const int iy = iy0 + ky, ix = ix0 + kx;
      ok[ky * 3 + kx] = (unsigned)iy < (unsigned)h && (unsigned)ix < (unsigned)w;
      const int cy = min(max(iy, 0), h - 1), cx = min(max(ix, 0), w - 1);
      v[ky * 3 + kx] = *reinterpret_cast<const vec8*>(x + (((int64_t)b * h + cy) * w + cx) * c + g * 8);
    }
  float best[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) best[e] = -INFINITY;
#pragma unroll
  for (int tap = 0; tap < 9; ++tap)
#pragma unroll
    for (int e = 0; e < 8; ++e) best[e] = fmaxf(best[e], ok[tap] ? (float)v[tap][e] : -INFINITY);
  vec8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (T)best[e];
  *reinterpret_cast<vec8*>(y + (int64_t)pos * c + g * 8) = o;
}

template <typename T, bool RELU>
__global__ void add_vec8_kernel(const T* a, const T* b, T* y, int64_t groups) {   // y may alias a or b
  typedef T vec8 __attribute__((ext_vector_type(8)));
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < groups; i += stride) {
    const vec8 va = reinterpret_cast<const vec8*>(a)[i], vb = reinterpret_cast<const vec8*>(b)[i];
    vec8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = (float)va[e] + (float)vb[e];
      o[e] = (T)(RELU ? fmaxf(v, 0.0f) : v);
    }
    reinterpret_cast<vec8*>(y)[i] = o;
  }
}

template <typename T, bool RELU>
__global__ void add_kernel(const T* a, const T* b, T* y, int64_t count) {   // y may alias a or b
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < count; i += stride) {
    const float v = (float)a[i] + (float)b[i];
    y[i] = (T)(RELU ? fmaxf(v, 0.0f) : v);
  }
}

// y = post(0 + shortcut): what a fused launch leaves when the mask keeps no row at all
template <typename T>
__global__ void shortcut_only_kernel(const T* __restrict__ res, T* __restrict__ y, int64_t count, int relu) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < count; i += stride) {
    float v = 0.0f + (float)res[i];
    if (relu) v = fmaxf(v, 0.0f);
    y[i] = (T)v;
  }
}

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline int elem_bytes(int dtype) { return dtype == SC_F32 ? 4 : 2; }

// float partial sums of a split-K launch at most (one BM x BN block per workgroup)
constexpr size_t kSplitKPartialBytes = (size_t)48 << 20;
constexpr int kStreamKMostWgs = 1024;   // persistent workgroups of a stream-K launch at most
constexpr int kSplitKMost = 64;   // splits per output tile at most

struct Geometry {
  int32_t ho, wo;
  int64_t m;
  int32_t k, k_pad, k_stride, k_tiles, vec, cout_pad;
  bool vec_gather, vec_out, vec_out8;
  int64_t x_elems, y_elems, mask_len;
  int32_t nseg;
  // workspace carve (byte offsets)
  size_t off_rows, off_counts, off_kept, off_zeros, off_mask, off_wp, off_ktab, off_band, off_band_rows, off_counters, off_partial, total;
  bool splitk_ok;          // the layer may run the split-K kernel (workspace reserved for it)
  // small-channel gather (NHWC, 16-bit, Cin*eb not a multiple of 16 bytes, e.g. the 3-channel stem): a
  // window row of kw*Cin contiguous elements is fetched as ceil(kw*Cin/8) unaligned 16-byte groups
  // from a zero-margined copy of the input, so no tap needs a bounds check
  bool depthwise;          // groups == Cin == Cout: its own kernel, no lowering
  bool rowseg;
  int32_t epad, hp, wp_cols;   // K entries per window row (padded to 8), padded input height and width
  size_t off_xpad;
  // register-staged tiled kernel (igemm_stage_kernel.hpp): its gather (-1: the layer does not run it), K tiles in that
  // gather's order, repeated entries of a pixel's last group, 32-channel blocks of its packed filters
  int32_t stage_gather, stage_k_tiles, stage_tail, stage_blocks;
  size_t off_stage_w, off_stage_tab;
  bool window;             // the layer may run the window kernel (igemm_window_kernel.hpp): its packed filters at off_window_w
  size_t off_window_w;
  size_t off_xrank, off_xcounts;   // depthwise layers with windows: rank map of a compact input, its segment counts
};

static int out_extent(int in, int k, int stride, int pad, int dil) {
  int64_t eff = (int64_t)in + 2 * (int64_t)pad - (int64_t)dil * (k - 1) - 1;
  if (eff < 0) return 0;
  return (int)(eff / stride) + 1;
}

static sc_status check_desc(const sc_conv_desc* d, Geometry* g) {
  if (!d) return SC_ERR_NULL;
  // one group (the paper's lowering) or one channel per group (depthwise, NHWC)
  const bool depthwise = d->groups != 1;
  if (depthwise && !(d->groups == d->c_in && d->c_in == d->c_out && d->layout == SC_NHWC)) return SC_ERR_UNSUPPORTED;
  if (d->dtype != SC_F32 && d->dtype != SC_F16 && d->dtype != SC_BF16) return SC_ERR_UNSUPPORTED;
  if (d->layout != SC_NHWC && d->layout != SC_NCHW) return SC_ERR_UNSUPPORTED;
  if (d->mask_mode != SC_MASK_ROW && d->mask_mode != SC_MASK_SPATIAL) return SC_ERR_UNSUPPORTED;
  if (d->out_mode != SC_OUT_ZERO_FILL && d->out_mode != SC_OUT_SCATTER_ONLY) return SC_ERR_UNSUPPORTED;
  if (d->n < 1 || d->c_in < 1 || d->h < 1 || d->w < 1 || d->c_out < 1 || d->kh < 1 || d->kw < 1 ||
      d->stride_h < 1 || d->stride_w < 1 || d->pad_h < 0 || d->pad_w < 0 || d->dil_h < 1 || d->dil_w < 1)
    return SC_ERR_BAD_SHAPE;
  if (!(d->sparsity < 1.0f)) return SC_ERR_BAD_SHAPE;  // also rejects NaN
  // the gather table packs window offsets into 15 bits
  if (d->h > 16000 || d->w > 16000 || d->pad_h > 16000 || d->pad_w > 16000 ||
      (int64_t)(d->kh - 1) * d->dil_h > 16000 || (int64_t)(d->kw - 1) * d->dil_w > 16000)
    return SC_ERR_BAD_SHAPE;
  g->ho = out_extent(d->h, d->kh, d->stride_h, d->pad_h, d->dil_h);
  g->wo = out_extent(d->w, d->kw, d->stride_w, d->pad_w, d->dil_w);
  if (g->ho < 1 || g->wo < 1) return SC_ERR_BAD_SHAPE;
  const int64_t lim = (int64_t)1 << 31;
  g->m = (int64_t)d->n * g->ho * g->wo;
  g->x_elems = (int64_t)d->n * d->h * d->w * d->c_in;
  g->y_elems = g->m * d->c_out;
  int64_t k = (int64_t)d->kh * d->kw * (depthwise ? 1 : d->c_in);
  g->depthwise = depthwise;
  if (g->m >= lim || g->x_elems >= lim - (1 << 20) || g->y_elems >= lim || k >= (1 << 24) || d->c_out >= (1 << 24))
    return SC_ERR_BAD_SHAPE;
  const int eb = elem_bytes(d->dtype);
  g->vec = 16 / eb;
  g->rowseg = false;
  g->epad = g->hp = g->wp_cols = 0;
  // (window-row gather; not for pointwise layers, whose window row is one pixel and which may be handed
  // the kept rows of their input only)
  if (d->layout == SC_NHWC && d->dtype != SC_F32 && d->c_in % g->vec != 0 && d->dil_w == 1 && d->kw * d->c_in <= 64 &&
      (d->w * d->c_in) % 8 == 0 && d->kh * d->kw > 1 && !depthwise) {
    const int epad = (d->kw * d->c_in + 7) / 8 * 8;
    const int over = (epad - d->kw * d->c_in + d->c_in - 1) / d->c_in;      // pixels the last group reads past the window
    const int max_iy = (g->ho - 1) * d->stride_h - d->pad_h + (d->kh - 1) * d->dil_h;
    const int max_ix = (g->wo - 1) * d->stride_w - d->pad_w + d->kw - 1 + over;
    const int64_t hp = d->pad_h + std::max<int64_t>(d->h, max_iy + 1), wpc = d->pad_w + std::max<int64_t>(d->w, max_ix + 1);
    if ((int64_t)d->n * hp * wpc * d->c_in + 64 < lim - (1 << 20)) {
      g->rowseg = true;
      g->epad = epad;
      g->hp = (int32_t)hp;
      g->wp_cols = (int32_t)wpc;
      k = (int64_t)d->kh * epad;
    }
  }
  g->k = (int32_t)k;
  const int bk = 8 * g->vec;
  g->k_pad = (int32_t)((k + bk - 1) / bk * bk);
  g->k_tiles = g->k_pad / bk;
  // filter rows are spaced by an odd number of K tiles: the band kernel's LDS swizzle relies on it
  g->k_stride = (g->k_tiles & 1) ? g->k_pad : g->k_pad + bk;
  g->cout_pad = (d->c_out + 255) / 256 * 256;
  g->vec_gather = d->layout == SC_NHWC && d->c_in % g->vec == 0;
  g->vec_out = d->layout == SC_NHWC && d->c_out % 16 == 0;
  // output rows that are whole 16-byte groups but no multiple of 16 channels (e.g. 40, 56, 104): vectorised
  // stores in the register-staged tiled kernel only
  g->vec_out8 = d->layout == SC_NHWC && !g->vec_out && d->c_out % g->vec == 0;
  g->mask_len = d->mask_mode == SC_MASK_ROW ? g->m : (int64_t)g->ho * g->wo;
  g->nseg = (int32_t)((g->m + kSeg - 1) / kSeg);
  size_t off = 0;
  g->off_rows = off;   off = align_up(off + (size_t)g->m * 4, 256);
  g->off_counts = off; off = align_up(off + ((size_t)g->nseg * 4 + 16 + (size_t)std::min(g->nseg, kTableMostWgs) * kTableWords) * 4, 256);      // (and the words of row_tables_kernel)
  g->off_kept = off;   off += 256;
  g->off_zeros = off;  off += 256;
  g->off_mask = off;   off = align_up(off + (size_t)g->mask_len, 256);
  g->off_wp = off;     off = align_up(off + (size_t)g->cout_pad * g->k_stride * eb, 256);
  g->off_ktab = off;   off = align_up(off + (size_t)g->k_pad * sizeof(KEntry), 256);
  g->off_band = off;   off = align_up(off + ((size_t)d->n * g->ho + 1) * 4, 256);
  g->off_band_rows = off; off = align_up(off + (size_t)g->m * 4, 256);
  g->off_xpad = off;
  if (g->rowseg) off = align_up(off + ((size_t)d->n * g->hp * g->wp_cols * d->c_in + 64) * eb, 256);
  g->off_xrank = g->off_xcounts = off;
  if (depthwise && d->kh * d->kw > 1) {
    const size_t pixels = (size_t)d->n * d->h * d->w;
    g->off_xrank = off;   off = align_up(off + pixels * 4, 256);
    g->off_xcounts = off; off = align_up(off + ((pixels + kSeg - 1) / kSeg + 1) * 4, 256);
  }
  // split-K (16-bit operands, direct-to-LDS gather, 128-channel tiles, deep K): arrival counters for
  // every output tile (64 x 64 is the smallest split-K tile) and the float partial sums
  g->splitk_ok = d->dtype != SC_F32 && g->vec_gather && g->vec_out && d->c_out >= 128 && g->k_tiles >= 16 && !depthwise;
  g->off_counters = g->off_partial = off;
  if (g->splitk_ok) {
    const size_t tiles = (size_t)((g->m + 63) / 64) * ((d->c_out + 63) / 64);
    g->off_counters = off; off = align_up(off + tiles * 4, 256);
    g->off_partial = off;  off = align_up(off + kSplitKPartialBytes, 256);
  }
  // Register-staged kernel: float layers, and layers whose tensors the 16-byte gathers do not fit (channels first, or
  // channel counts off the 16-byte group).  Windows up to 8 x 8 (validity bits), x below 2 GiB (32-bit byte offsets).
  g->stage_gather = -1;
  g->stage_k_tiles = g->stage_tail = g->stage_blocks = 0;
  g->off_stage_w = g->off_stage_tab = off;
  if (!depthwise && !g->rowseg && (d->dtype == SC_F32 || !g->vec_gather) && d->kh <= 8 && d->kw <= 8 && g->x_elems * eb < lim) {
    const bool nhwc = d->layout == SC_NHWC;
    g->stage_gather = nhwc ? (g->vec_gather ? kStageGroups : d->c_in >= g->vec ? kStageRaggedGroups : kStageEntries)
                           : (d->c_in % 8 == 0 ? kStageChunks : kStageEntries);
    const int cpad = g->stage_gather == kStageRaggedGroups ? (d->c_in + g->vec - 1) / g->vec * g->vec : d->c_in;
    const int tile = d->dtype == SC_F32 ? StageDims<kF32>::K_TILE : StageDims<kBF16>::K_TILE;
    const int block_bytes = d->dtype == SC_F32 ? StageDims<kF32>::BLOCK_BYTES : StageDims<kBF16>::BLOCK_BYTES;
    g->stage_tail = cpad - d->c_in;
    g->stage_k_tiles = (int32_t)(((int64_t)d->kh * d->kw * cpad + tile - 1) / tile);
    g->stage_blocks = (d->c_out + 127) / 128 * 4;      // (tiles are up to 128 channels wide)
    g->off_stage_w = off;   off = align_up(off + (size_t)g->stage_blocks * g->stage_k_tiles * block_bytes, 256);
    g->off_stage_tab = off; off = align_up(off + (size_t)g->stage_k_tiles * tile * sizeof(KEntry), 256);
  }
  // Window kernel: 3 x 3 or 5 x 5 at stride 1, whole 16-byte groups, tensors and virtual pixels in 31 bits.  Its packed filters hold whole chunks.
  const int64_t window_k = (int64_t)d->kh * d->kw * ((d->c_in + kWinChunk - 1) / kWinChunk) * kWinChunk;
  g->window = g->vec_gather && (g->vec_out || g->vec_out8) && d->dtype != SC_F32 && (d->kh == 3 || d->kh == 5) && d->kw == d->kh && d->stride_h == 1 && d->stride_w == 1 &&
              d->dil_h == 1 && d->dil_w == 1 && !depthwise && g->x_elems * eb < lim &&
              (int64_t)d->n * (d->h + 2 * (int64_t)d->pad_h) * (d->w + 2 * (int64_t)d->pad_w) < lim &&
              (int64_t)((d->c_out + 31) / 32) * 32 * window_k * eb < lim && (int64_t)g->cout_pad * g->k_stride < lim;
  g->off_window_w = off;
  if (g->window) off = align_up(off + (size_t)((d->c_out + 31) / 32) * 32 * window_k * eb, 256);
  g->total = off;
  return SC_OK;
}

// Band kernel applicability and band height.
struct BandPlan {
  bool ok;
  bool stream;       // filters streamed through an LDS ring instead of resident
  bool pp;           // persistent workgroups, two wavefront groups alternating between transfer and MFMA
  bool tap;          // one band per workgroup of eight wavefronts, filters arriving tap by tap under the MFMAs
  int pp_grid;       // workgroups of that kernel
  int max_kept;      // most kept rows in one band
  int bh, bands_per_image, n_bands, n_tiles, ni_idx, ni;
  int split;         // alternating-group kernel only: every run of bh rows is two bands of half its pixels
  size_t b_bytes, x_bytes, lds;
  bool rowband;      // small-channel layers: window rows read from a zero-margined slab (row-segment K order)
  int rb_pitch, rb_left, rb_in_rows, rb_gpw, rb_tail;
};

constexpr size_t kLdsLimit = 160 * 1024;
// behind the band kernel's slabs: a zeroed KiB and 128 bias floats
constexpr size_t kBandExtraLds = 1024 + 128 * 4;

// 32-row MFMA units the busiest of four wavefronts runs for a band with `cnt` rows, with 32-row (MI = 1) or
// 64-row (MI = 2) blocks dealt round robin; `mi_idx` receives the better shape (at a tie the 64-row block, whose
// two row blocks share every filter fragment read from LDS).
static double band_units(double cnt, int* mi_idx) {
  const double units1 = std::ceil(std::ceil(cnt / 32.0) / 4.0), units2 = 2.0 * std::ceil(std::ceil(cnt / 64.0) / 4.0);
  if (mi_idx) *mi_idx = units1 < units2 ? 0 : 1;
  return std::min(units1, units2);
}

static bool tap_is_automatic(const sc_conv_desc& d, const Geometry& g, const BandPlan& tp, int64_t rows);
static int device_cus();

// Band kernel of the small-channel layers (row-segment K order): window starts must be 4-byte aligned in the slab, K
// at most 24 groups of 16 bytes, 64 output channels per workgroup, bands of at most 512 output pixels.  The tallest
// such band that still leaves a workgroup per compute unit.  SPARSE_CONV_BAND_KERNEL=none keeps such a layer on the
// tiled row-segment kernel, SPARSE_CONV_BAND_HEIGHT=<bh> fixes the band height (tuning and tests).
static BandPlan plan_rowband(const sc_conv_desc& d, const Geometry& g) {
  BandPlan bp;
  std::memset(&bp, 0, sizeof(bp));
  const int eb = elem_bytes(d.dtype);
  const char* variant = std::getenv("SPARSE_CONV_BAND_KERNEL");
  if (variant && std::strcmp(variant, "none") == 0) return bp;
  if (eb != 2 || !g.vec_out || d.dil_w != 1 || (d.stride_w * d.c_in * eb) % 4 != 0) return bp;
  const int gpw = g.epad / 8;
  if (d.kh * gpw > kRowBandMostGroups || (int64_t)d.kh * g.epad > g.k_stride) return bp;
  if (g.wo > kRowBandMaxRows) return bp;
  const int64_t reach = (int64_t)(g.wo - 1) * d.stride_w * d.c_in * eb + (int64_t)gpw * 16;   // end of the last window row
  const int64_t pitch = (int64_t)align_up((size_t)std::max<int64_t>((int64_t)(d.pad_w + d.w) * d.c_in * eb, reach), 16);
  const char* env = std::getenv("SPARSE_CONV_BAND_HEIGHT");
  const int forced_bh = env ? std::atoi(env) : 0;
  auto fits = [&](int bh) {
    const int64_t in_rows = (int64_t)(bh - 1) * d.stride_h + (int64_t)(d.kh - 1) * d.dil_h + 1;
    return (int64_t)bh * g.wo <= kRowBandMaxRows && rowband_slab_at(d.kh * gpw) + in_rows * pitch <= (int64_t)kLdsLimit;
  };
  if (!fits(1)) return bp;
  int bh = 1;
  while (bh < g.ho && fits(bh + 1)) ++bh;
  const int n_tiles = (d.c_out + 63) / 64;
  // (measured on the 7x7 stem at batch 4 .. 64: halving pays only while the bands do not cover the compute units once)
  while (bh > 1 && (int64_t)d.n * ((g.ho + bh - 1) / bh) * n_tiles < (int64_t)device_cus()) bh = (bh + 1) / 2;
  if (forced_bh > 0) { if (!fits(forced_bh)) return bp; bh = forced_bh; }
  bp.ok = bp.rowband = true;
  bp.ni = 2; bp.ni_idx = 1;
  bp.n_tiles = n_tiles;
  bp.bh = bh;
  bp.bands_per_image = (g.ho + bh - 1) / bh;
  bp.n_bands = d.n * bp.bands_per_image;
  bp.rb_pitch = (int)pitch;
  bp.rb_left = d.pad_w;
  bp.rb_in_rows = (bh - 1) * d.stride_h + (d.kh - 1) * d.dil_h + 1;
  bp.rb_gpw = gpw;
  bp.rb_tail = d.kw * d.c_in - (gpw - 1) * 8;
  bp.b_bytes = (size_t)64 * rowband_filter_pitch(d.kh * gpw);
  bp.x_bytes = (size_t)bp.rb_in_rows * pitch;
  bp.lds = rowband_slab_at(d.kh * gpw) + bp.x_bytes;
  return bp;
}

// `rows`: the rows the run is expected to contract (the kept rows of a sparse run, M of a dense one).
static BandPlan plan_band(const sc_conv_desc& d, const Geometry& g, int64_t rows) {
  BandPlan bp;
  std::memset(&bp, 0, sizeof(bp));
  const int eb = elem_bytes(d.dtype);
  if (g.depthwise) return bp;
  if (g.rowseg) return plan_rowband(d, g);
  if (d.layout != SC_NHWC || !g.vec_gather || !g.vec_out) return bp;
  if ((d.c_in / g.vec) % 2 != 0) return bp;      // a K step of two 16-byte groups must stay inside one tap
  if (d.kh * d.kw == 1) return bp;               // no window overlap to exploit: gather kept rows directly
  bp.ni = d.c_out <= 32 ? 1 : d.c_out <= 64 ? 2 : 4;
  bp.ni_idx = bp.ni == 1 ? 0 : bp.ni == 2 ? 1 : 2;
  bp.n_tiles = (d.c_out + 32 * bp.ni - 1) / (32 * bp.ni);
  bp.b_bytes = (size_t)32 * bp.ni * g.k_stride * eb;
  // Alternating-group kernel (persistent workgroups, filters resident, two input slabs): 3x3
  // windows of 16-bit operands with 4 or 8 channel groups per pixel.  It pays once a workgroup
  // walks several bands (measured on MI355X: from three steps on); with fewer, one band per
  // workgroup is faster.  SPARSE_CONV_BAND_KERNEL=single|alternating|tap|no-tap overrides (tuning and tests).
  const char* variant = std::getenv("SPARSE_CONV_BAND_KERNEL");
  const bool want_single = variant && std::strcmp(variant, "single") == 0;
  const bool want_pp = variant && std::strcmp(variant, "alternating") == 0;
  const bool want_tap = variant && std::strcmp(variant, "tap") == 0;
  const bool no_tap = variant && std::strcmp(variant, "no-tap") == 0;      // the automatic choice among the other kernels
  // Tap-pipelined kernel: 3x3 windows of 16-bit operands with 4 or 8 channel groups per pixel, one band per
  // workgroup; the tallest band that fits LDS and 512 rows and costs the fewest rounds of workgroups.
  if (!want_single && !want_pp && !no_tap && d.kh == 3 && d.kw == 3 && d.dtype != SC_F32 &&
      (d.c_in / g.vec == 8 || d.c_in / g.vec == 4)) {
    BandPlan tp = bp;
    tp.ni = d.c_out <= 32 ? 1 : 2;
    tp.ni_idx = tp.ni - 1;
    tp.n_tiles = (d.c_out + 32 * tp.ni - 1) / (32 * tp.ni);
    tp.b_bytes = (size_t)9 * 32 * tp.ni * (d.c_in / g.vec) * 16;
    const char* env = std::getenv("SPARSE_CONV_BAND_HEIGHT");
    const int forced_bh = env ? std::atoi(env) : 0;
    double best = 1e300;
    for (int bh = 1; bh <= g.ho; ++bh) {
      const int64_t ih = (int64_t)(bh - 1) * d.stride_h + (int64_t)2 * d.dil_h + 1;
      const size_t xbytes = align_up((size_t)ih * d.w * d.c_in * eb, 1024);
      if (tp.b_bytes + kTapFixedLds + xbytes > kLdsLimit) break;
      if ((int64_t)bh * g.wo > kTapMaxRows) break;
      const int bpi = (g.ho + bh - 1) / bh;
      const int64_t nb = (int64_t)d.n * bpi * tp.n_tiles;
      const double rounds = std::ceil((double)nb / (double)device_cus());
      const double cost = rounds * ((double)xbytes + (double)tp.b_bytes + 64.0 * bh * g.wo);
      const bool take = forced_bh > 0 ? bh == forced_bh : cost <= best;
      if (take) {
        best = cost;
        tp.ok = true;
        tp.tap = true;
        tp.bh = bh;
        tp.bands_per_image = bpi;
        tp.n_bands = d.n * bpi;
        tp.x_bytes = xbytes;
        tp.lds = tp.b_bytes + kTapFixedLds + xbytes;
      }
    }
    if (tp.ok && (want_tap || tap_is_automatic(d, g, tp, rows))) return tp;
  }
  if (!want_single && d.kh == 3 && d.kw == 3 && d.dtype != SC_F32 &&
      (d.c_in / g.vec == 8 || d.c_in / g.vec == 4)) {
    BandPlan pp = bp;
    pp.ni = d.c_out <= 32 ? 1 : 2;
    pp.ni_idx = pp.ni - 1;
    pp.n_tiles = (d.c_out + 32 * pp.ni - 1) / (32 * pp.ni);
    pp.b_bytes = (size_t)32 * pp.ni * g.k_stride * eb;
    // SPARSE_CONV_BAND_HEIGHT=<bh> or <bh>,split overrides the search (tuning and tests)
    const char* env = std::getenv("SPARSE_CONV_BAND_HEIGHT");
    const int forced_bh = env ? std::atoi(env) : 0;
    const int forced_split = (env && std::strstr(env, ",split")) ? 1 : 0;
    const int lanes_max = std::max(1, 256 / pp.n_tiles);
    int best_steps = 0;
    double best = 1e300;
    // whole runs of bh rows, and runs cut into two bands of half their pixels
    for (int bh = 1; bh <= g.ho; ++bh) {
      for (int split = 0; split <= 1; ++split) {
        // rows of output a band touches: a half band of an odd run reaches into the middle row from either side
        const int rows_out = split ? bh / 2 + 1 : bh;
        if (split && bh < 2) continue;
        int64_t ih = (int64_t)(rows_out - 1) * d.stride_h + (int64_t)(d.kh - 1) * d.dil_h + 1;
        size_t xbytes = align_up((size_t)ih * d.w * d.c_in * eb, 1024);
        if (pp.b_bytes + 2 * xbytes + kPPFixedLds > kLdsLimit) continue;
        const int64_t band_px = split ? ((int64_t)bh * g.wo + 1) / 2 : (int64_t)bh * g.wo;
        if (band_px > kPPMaxRows) continue;
        int bpi = bands_in_image(g.ho, bh, split);
        int64_t nb = (int64_t)d.n * bpi;
        int lanes = (int)std::min<int64_t>(nb, lanes_max);
        int steps = (int)((nb + lanes - 1) / lanes);
        // a step costs its band plus a fixed part (halo rows, barrier, transfer latency)
        double cost = steps * ((split ? 0.5 * bh : (double)bh) + 1.5);
        const bool take = forced_bh > 0 ? (bh == forced_bh && split == forced_split) : cost <= best;
        if (take) {
          best = cost;
          best_steps = steps;
          pp.ok = true;
          pp.pp = true;
          pp.bh = bh;
          pp.split = split;
          pp.bands_per_image = bpi;
          pp.n_bands = (int)nb;
          pp.x_bytes = xbytes;
          pp.lds = pp.b_bytes + 2 * xbytes + kPPFixedLds;
          pp.pp_grid = lanes * pp.n_tiles;
        }
      }
    }
    // two channel tiles would transfer every band twice: measured slower than the tiled kernel
    if (pp.ok && (want_pp || (best_steps >= 3 && pp.n_tiles == 1))) return pp;
    // Exactly two equal steps per workgroup (split bands, as many runs of rows as workgroups): the second band's
    // transfer hides behind the first one's MFMAs and stores, which is worth 4-8 % on the stage-1 ResNet layer at
    // batch 32 -- unless halving the bands costs MFMA blocks (64-row blocks that a whole run fills well fall apart
    // into more 32-row blocks: s = 0.25 there, 3 units per run against 2 + 2 per pair of halves).
    // The slowest workgroup sets the kernel's time, so the counts are those of a band three standard deviations
    // above the mean of a random mask (at s = 0.4 a half band keeps 118 rows on average, but more than the 128 of
    // four blocks in some workgroup of nearly every launch).
    if (pp.ok && pp.split && best_steps == 2 && pp.n_tiles == 1 && pp.n_bands == 2 * pp.pp_grid && !want_single) {
      const double drop = 1.0 - (double)rows / (double)g.m;
      auto busiest = [&](double mean) { return mean + 3.0 * std::sqrt(std::max(mean * drop, 0.0)); };
      const double whole = band_units(busiest((double)rows / (pp.n_bands / 2)), nullptr);
      const double halves = 2.0 * band_units(busiest((double)rows / pp.n_bands), nullptr);
      if (halves <= std::max(whole, 2.0)) return pp;
    }
  }
  if (bp.b_bytes > 96 * 1024) {
    // Filters too large to stay resident: stream them (16-bit types, whole 128-byte K tiles per tap,
    // 64 or 128 channels per workgroup).  Taller bands amortise the filter traffic, which every
    // workgroup pays in full; rows are capped by the accumulator registers (128 rows per MI step).
    if (d.dtype == SC_F32 || (d.c_in / g.vec) % 8 != 0 || bp.ni < 2) return bp;
    bp.stream = true;
    bp.b_bytes = (size_t)kStreamStages * 32 * bp.ni * kRowBytes;
    const char* env = std::getenv("SPARSE_CONV_BAND_HEIGHT");
    const int forced_bh = env ? std::atoi(env) : 0;
    int best_bh = 0;
    int64_t best_wg = 0;
    for (int bh = 1; bh <= g.ho; ++bh) {
      int64_t ih = (int64_t)(bh - 1) * d.stride_h + (int64_t)(d.kh - 1) * d.dil_h + 1;
      size_t xbytes = align_up((size_t)ih * d.w * d.c_in * eb, 1024);
      if (bp.b_bytes + xbytes + kBandExtraLds > kLdsLimit) break;
      if ((int64_t)bh * g.wo > (bp.ni == 4 ? 384 : 512)) break;   // accumulator registers: 3 / 4 blocks of 128 rows
      int bpi = (g.ho + bh - 1) / bh;
      int64_t nwg = (int64_t)d.n * bpi * bp.n_tiles;
      // the tallest band that still gives every CU a workgroup; failing that, one output row per
      // band (the most workgroups); SPARSE_CONV_BAND_HEIGHT overrides (tuning and tests)
      const bool take = forced_bh > 0 ? bh == forced_bh : (nwg >= 256 || best_bh == 0);
      if (take) { best_bh = bh; best_wg = nwg; bp.x_bytes = xbytes; }
    }
    (void)best_wg;
    if (best_bh == 0) { bp.stream = false; return bp; }
    bp.ok = true;
    bp.bh = best_bh;
    bp.bands_per_image = (g.ho + best_bh - 1) / best_bh;
    bp.n_bands = d.n * bp.bands_per_image;
    bp.lds = bp.b_bytes + bp.x_bytes + kBandExtraLds;
    return bp;
  }
  double best = 1e300;
  for (int bh = 1; bh <= g.ho; ++bh) {
    int64_t ih = (int64_t)(bh - 1) * d.stride_h + (int64_t)(d.kh - 1) * d.dil_h + 1;
    size_t xbytes = align_up((size_t)ih * d.w * d.c_in * eb, 1024);
    if (bp.b_bytes + xbytes + kBandExtraLds > kLdsLimit) break;
    if ((int64_t)bh * g.wo > kBandMaxRows) break;
    int bpi = (g.ho + bh - 1) / bh;
    int64_t nb = (int64_t)d.n * bpi * bp.n_tiles;
    double rounds = std::ceil((double)nb / 256.0);
    double cost = rounds * ((double)xbytes + (double)bp.b_bytes + 64.0 * bh * g.wo);
    if (cost <= best) {
      best = cost;
      bp.ok = true;
      bp.bh = bh;
      bp.bands_per_image = bpi;
      bp.n_bands = d.n * bpi;
      bp.x_bytes = xbytes;
      bp.lds = bp.b_bytes + xbytes + kBandExtraLds;
    }
  }
  return bp;
}

// Compute units of the current device (256 on MI355X), asked once per process.
static int device_cus() {
  static std::atomic<int> cached{0};
  int v = cached.load();
  if (v > 0) return v;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
    (void)hipGetLastError();
    cus = 256;
  }
  cached.store(cus);
  return cus;
}

// When the tap-pipelined kernel is the automatic choice: one channel tile (two would transfer every band twice) and
// at most one workgroup per compute unit.  Measured on MI355X, sparse run / dense run in us: ResNet18 stage-1 layer
// at batch 32, s = 0.5: 8.7 / 11.4 against 10.9 / 13.9 with the alternating-group kernel (s = 0.25: 10.5 against
// 13.6 with one band per workgroup); detector y2: 10.5 / 11.6 against 17.4 / 17.2; at batch 64 (two rounds of
// workgroups, nothing to overlap the second round's transfers with) 17.8 against 16.6 for persistent workgroups.
static bool tap_is_automatic(const sc_conv_desc& d, const Geometry& g, const BandPlan& tp, int64_t rows) {
  (void)d; (void)g; (void)rows;
  return tp.n_tiles == 1 && (int64_t)tp.n_bands * tp.n_tiles <= device_cus();
}

}  // namespace sc

using namespace sc;

// tile of the register-staged and of the direct float kernel; groups of wavefronts that share K; asked for by the environment
struct StageTile { int bm, bn, groups; bool asked; };

struct sc_plan {
  sc_conv_desc desc;
  Geometry geo;
  BandPlan band;                   // of the sparse run (the band tables in the workspace follow it)
  BandPlan band_dense;             // of the dense run, which needs no tables: it may cut the bands differently
  const BandTable* band_table;
  const BandStreamTable* stream_table;
  const BandPPTable* pp_table;
  const BandTapTable* tap_table;
  unsigned char* ws;
  int64_t kept;
  const KernelEntry* table;
  int table_count;
  // grouped: tile whose launch with two groups of wavefronts, sharing K inside the workgroup, stands in for the split into
  // `splits` shares where group_candidates allows it (-1: none); asked: by the environment; us: its predicted time (0: not priced)
  struct Pick { int ti, splits; bool masked; int grouped = -1; bool asked = false; double us = 0.0; };
  Pick pick[2];                    // tiled launch of the sparse / dense run when nothing is forced: tile, K splits, and
                                   // (sparse run) whether every row is contracted and the mask decides at the store
  bool prefer_tiled[2];            // measured by sparse_conv_plan_tune: the tiled launch beat the band / row-panel kernel
  bool tuned;                      // pick and prefer_tiled come from measurements on this device, not from the cost model
  LaunchFn panel;                  // row-panel kernel of the plan's dtype (null: none)
  int tile_splitk;                 // index of the 64 x 128 entry, the tile of automatic split-K launches (-1: none)
  int forced[2];                   // -1 = automatic, >= 0 generic tile index, kForceBand = band kernel
  int gather_pipeline;             // 0 = automatic, 1 = through registers, 2 = straight into LDS
  int split_k;                     // 0 = automatic, 1 = never, n >= 2 = n splits wherever the kernel applies
  int row_panel;                   // 0 = automatic, 1 = never, 2 = wherever the kernel applies
  int stream_k;                    // 0 = automatic, 1 = never, n >= 2 = n persistent workgroups wherever the kernel applies
  int masked_store;                // 0 = automatic, 1 = never, 2 = wherever it applies (sparse runs of dense NHWC operands)
  bool x_rank_set;                 // sparse_conv_plan_set_input_mask has filled the rank map of a compact input
  // slab form of the tiled kernel (deep 3x3 layers)
  struct Slab { int bm, splits; };
  StageTile stage_pick[2];         // tile of the register-staged kernel for the sparse / dense run (bm == 0: another kernel)
  int depthwise_kernel;            // asked for by SPARSE_CONV_DEPTHWISE_KERNEL=staged|walk (tests): 0 none, 1 staged, 2 column walk
  int stage_tuned;                 // sparse_conv_plan_tune measured that kernel fastest (1) or slower than another (-1); 0: not timed
  bool slab_ok;                    // the layer's geometry admits it
  int slab;                        // 0 = automatic, 1 = never, 2 = wherever it applies, 128 / 256 = with tiles of that many rows
  struct Window { int bm, bn; bool before_bands, plain_only = false, asked = false; };
  Window window[2];                // tile of the window kernel for the sparse / dense run (bm == 0: another kernel), whether a band kernel gives way,
                                   // whether only plain runs take it (the others never went to that band kernel); asked for by the environment
  int slab_span[2][3];             // [sparse, dense run][64-row, 128-row, 256-row tiles]: virtual rows of the widest tile's slab
  Slab slab_auto[2];               // what an automatic launch of the sparse / dense run takes (bm == 0: another kernel)
};
constexpr int kForceBand = -2;

namespace sc {

// Tile choice for a GEMM of `rows` x c_out x K.  The row count is the compacted one, so a heavily masked layer
// gets other tiles than its dense twin (Sec. 3.2: the GEMM range shrinks with the sparsity).  Every candidate
// (tile shape x K splits, and for the sparse run the variant that contracts every row and masks at the store)
// is priced with a small model of one launch on this device and the cheapest wins.  The constants are
// measurements on MI355X, each of one quantity:
//   kLaunchUs     what a launch costs beyond the lifetime of its workgroups (dispatch ramp and drain)
//   kWgFixedUs    set-up and epilogue of a workgroup; kRowListUs more when rows come through the row list
//                 (a dependent round trip to memory before the first transfer, and the zero fill)
//   kIngestKBus   what a compute unit moves from L2 into LDS per microsecond with 1, 2, 3+ workgroups resident
//                 (the K loops of these kernels are bound by that path, not by the matrix pipes)
//   kMfmaShare    share of the matrix peak a K loop sustains when it is the bound
//   kExchangeKBus rate at which float partial sums of a split K walk travel between workgroups (device-scope
//                 stores and loads: across the fabric between the dies' L2 caches)
// The model is good to about 15 %; sparse_conv_plan_tune replaces its choice by a measured one.
constexpr double kLaunchUs = 3.0, kWgFixedUs = 1.0, kRowListUs = 0.6, kMfmaShare = 0.85, kExchangeKBus = 4000.0;
//   kGroupUs      what two groups of wavefronts that share K add to a workgroup: their sums through LDS; such a workgroup
//                 alone on a compute unit takes in kIngestGroupsKBus
constexpr double kIngestKBus[3] = {62.0, 110.0, 120.0}, kGroupUs = 0.2, kIngestGroupsKBus = 85.0;
constexpr double kIngestEightWavesKBus = 76.0;      // one resident workgroup of eight wavefronts
constexpr double kClockPerUs = 2100.0;

// LDS bytes of the kernel form a tile of this layer runs (decides how many workgroups share a compute unit)
static size_t tile_lds_bytes(const sc_plan* pl, const KernelEntry& ke) {
  const Geometry& g = pl->geo;
  if (g.vec_gather && g.vec_out && pl->gather_pipeline != 1) {
    const int stages = g.k_tiles <= 2 ? 2 : 3;
    return (size_t)stages * (ke.bm + ke.bn) * kRowBytes + (ke.bm + 4) * 4 + (size_t)ke.bn * 4;
  }
  return 2 * (size_t)(ke.bm + ke.bn) * kRowBytes + (size_t)ke.bm * 4;
}

// predicted microseconds of one tiled launch: `rows` rows through tile ke with K cut into `splits`;
// `listed`: rows come through the kept-row list and dropped rows are zero-filled by their owners
static double predict_us(const sc_plan* pl, const KernelEntry& ke, int64_t rows, int splits, bool listed, int groups = 1) {
  const Geometry& g = pl->geo;
  const sc_conv_desc& d = pl->desc;
  const int cus = device_cus();
  const int64_t tiles = ((rows + ke.bm - 1) / ke.bm) * ((d.c_out + ke.bn - 1) / ke.bn);
  const int64_t wgs = tiles * splits;
  const int n_kt = (g.k_tiles + splits - 1) / splits;
  const double kb_wg = (double)(ke.bm + ke.bn) * kRowBytes * n_kt / 1024.0;          // through the L1 path
  const double peak = d.dtype == SC_F32 ? 4096.0 * 157.3 / 2500.0 : 4096.0;          // FLOP per clock and compute unit
  const int bk = kRowBytes / elem_bytes(d.dtype);
  const double mfma_us = 2.0 * ke.bm * ke.bn * bk * n_kt / (peak * kMfmaShare * kClockPerUs);
  const bool eight_waves = ke.bm * ke.bn >= 128 * 128 && g.vec_gather && g.vec_out && d.dtype != SC_F32 && d.c_in % 64 == 0;
  int occ = (int)std::min<size_t>(kLdsLimit / std::max<size_t>(tile_lds_bytes(pl, ke), 1), eight_waves ? 2 : 4);
  occ = std::max(occ, 1);
  if (groups > 1) occ = std::max<int>(1, (int)std::min<size_t>(kLdsLimit / (tile_lds_bytes(pl, ke) * groups), 2));
  const int c = (int)std::max<int64_t>(1, std::min<int64_t>(occ, (wgs + cus - 1) / cus));   // resident per compute unit
  const double rounds = std::ceil((double)wgs / ((double)cus * c));
  const double ingest = c == 1 && groups > 1 ? kIngestGroupsKBus : c == 1 && eight_waves ? kIngestEightWavesKBus : kIngestKBus[std::min(c * groups, 3) - 1];
  const double round_us = kWgFixedUs + (groups > 1 ? kGroupUs : 0.0) + (listed ? kRowListUs : 0.0) + std::max(c * kb_wg / ingest, c * mfma_us);
  double t = kLaunchUs + rounds * round_us;
  if (splits > 1)   // every split writes its tile of floats, the last arrival reads them all
    t += 2.0 * (double)tiles * splits * ke.bm * ke.bn * 4.0 / 1024.0 / kExchangeKBus;
  return t;
}

static int most_splits(const sc_plan* pl, const KernelEntry& ke, int64_t rows);
static LaunchFn splitk_launcher(const sc_plan* pl, const KernelEntry& ke);
static int group_candidates(const sc_plan* pl, const KernelEntry& ke, int64_t rows);
static bool buf_applies(const sc_plan* pl, const KernelEntry& ke);

// K splits the automatic choice considers for a tile: up to four, and only the buffer-load form of the split kernel
// (the older form of the small tiles measured slower than their unsplit launches everywhere)
static int split_candidates(const sc_plan* pl, const KernelEntry& ke, int64_t rows) {
  if (pl->split_k == 1 || !buf_applies(pl, ke) || pl->geo.k_tiles <= 2) return 1;
  if (!buf_splitk_kernel(pl->desc.dtype == SC_BF16 ? kBF16 : kF16, ke.bm, ke.bn)) return 1;
  return std::min(4, most_splits(pl, ke, rows));
}

// groups of wavefronts the automatic choice considers for a tile: two, where the buffer-load kernel has that form and the
// workgroups cover half to all of the compute units (fewer leave the filters, cold behind other layers, to too few of them:
// a ResNet18 stack at batch 8 and 160 x 160 208 -> 212 us; more wait for a second round)
static int group_candidates(const sc_plan* pl, const KernelEntry& ke, int64_t rows) {
  const int64_t wgs = ((rows + ke.bm - 1) / ke.bm) * ((pl->desc.c_out + ke.bn - 1) / ke.bn);
  if (wgs * 2 < device_cus() || wgs > device_cus()) return 1;
  if (pl->split_k != 0 || pl->stream_k >= 2 || pl->geo.k_tiles < 8 || !buf_applies(pl, ke)) return 1;
  return buf_groups_kernel(pl->desc.dtype == SC_BF16 ? kBF16 : kF16, ke.bm, ke.bn) ? 2 : 1;
}

// the cheapest tiled launch by the model.  Layers the fast gathers do not serve keep their one measured shape.
static sc_plan::Pick model_pick(const sc_plan* pl, int which, int64_t rows) {
  const Geometry& g = pl->geo;
  const sc_conv_desc& d = pl->desc;
  sc_plan::Pick best = {0, 1, false};
  auto find = [&](int bm, int bn) {
    for (int i = 0; i < pl->table_count; ++i)
      if (pl->table[i].bm == bm && pl->table[i].bn == bn) return i;
    return 0;
  };
  if (g.rowseg) { best.ti = d.c_out <= 32 ? find(128, 32) : find(64, 64); return best; }   // window-row gather (stems)
  if (!g.vec_gather) { best.ti = find(128, 64); return best; }                              // element gather
  // SPARSE_CONV_TILE_GROUPS=<bm>x<bn>x<1|2>: that tile with so many groups of wavefronts sharing K (tuning and tests)
  int fbm = 0, fbn = 0, fgr = 0;
  if (const char* env = std::getenv("SPARSE_CONV_TILE_GROUPS"); env && std::sscanf(env, "%dx%dx%d", &fbm, &fbn, &fgr) == 3) {
    const int i = find(fbm, fbn);
    const bool grouped = fgr == 2 && buf_applies(pl, pl->table[i]) && buf_groups_kernel(d.dtype == SC_BF16 ? kBF16 : kF16, fbm, fbn);
    if (pl->table[i].bm == fbm && pl->table[i].bn == fbn && (fgr == 1 || grouped)) return {i, grouped ? 2 : 1, false, grouped ? i : -1, grouped};
  }
  double best_us = 1e300;
  const bool can_mask = which == 0 && rows < g.m && rows > 0;
  for (int i = 0; i < pl->table_count; ++i) {
    const KernelEntry& ke = pl->table[i];
    if (tile_lds_bytes(pl, ke) > kLdsLimit) continue;
    if (ke.bn > 128 && d.c_out <= 128) continue;                      // more than half of such a tile would be padding
    const int most = split_candidates(pl, ke, rows);
    for (int sp = 1; sp <= most; ++sp) {
      const double t = predict_us(pl, ke, rows, sp, which == 0 && rows < g.m);
      if (t < best_us) { best_us = t; best = {i, sp, false}; }
    }
    if (can_mask && pl->masked_store != 1) {       // every row contracted, the mask decides at the store: the dense launch plus a mask byte per row
      const double t = predict_us(pl, ke, g.m, 1, false) + 0.1;
      if (t < best_us) { best_us = t; best = {i, 1, true}; }
    }
  }
  // Two groups of wavefronts only where they add what the best launch adds in its order, i.e. in the place of a split into two
  // or (where the four shares are whole turns of the ring of three tiles) four: one order of additions whichever of the two
  // runs.  64 x 512 -> 512 @7 in bf16 at s = 0.5: four shares of 128 x 128 20.0 us, two groups 18.9.
  if (!best.masked && (best.splits == 2 || (best.splits == 4 && g.k_tiles % 12 == 0)))
    for (int i = 0; i < pl->table_count; ++i) {
      if (group_candidates(pl, pl->table[i], rows) < 2) continue;
      const double t = predict_us(pl, pl->table[i], rows, 1, which == 0 && rows < g.m, 2);
      if (t < best_us) { best_us = t; best.grouped = i; }
    }
  best.us = best_us;
  return best;
}

// Split K?  Layers deep in a network have few rows and a long K: large output tiles cannot fill
// 256 CUs, and with small tiles every workgroup walks the whole K, one L2 round trip after the other.
// Dividing K among workgroups shortens that walk and still gives every CU work.
struct TilePick { int ti, splits; bool masked; int shares = 0; };      // (shares of K added by two groups of wavefronts; 0: none)

// Row-panel kernel: short K (pointwise layers), several 64-channel tiles, enough rows to fill the
// CUs with 128-row panels.  There the tiled kernels are bound by the instructions every
// (row tile, channel tile) workgroup repeats; the panel kernel pays them once per row tile.
static bool use_panel(const sc_plan* pl, int which, int64_t rows) {
  const Geometry& g = pl->geo;
  const sc_conv_desc& d = pl->desc;
  const bool applies = pl->panel && pl->forced[which] < 0 && !(pl->prefer_tiled[which] && pl->row_panel != 2) &&
                       pl->gather_pipeline != 1 && pl->row_panel != 1 &&
                       g.vec_gather && g.vec_out && g.k_tiles <= kPanelMaxKTiles && d.c_out <= 1024;
  // (from 96 channels on, i.e. more than one channel tile per panel: 16 -> 96 channels on a 112 x 112 map,
  // batch 64, measured 52 -> 44 us with dense and 38 -> 27 us with compact operands)
  return applies && (pl->row_panel == 2 || (d.c_out >= 96 && rows >= 128 * 256));
}

static bool buf_applies(const sc_plan* pl, const KernelEntry& ke);

// the split-K launcher of a tile: the buffer-load form where the layer admits it, else the direct-to-LDS form
static LaunchFn splitk_launcher(const sc_plan* pl, const KernelEntry& ke) {
  if (buf_applies(pl, ke) && pl->geo.k_tiles > 2) {
    LaunchFn fn = buf_splitk_kernel(pl->desc.dtype == SC_BF16 ? kBF16 : kF16, ke.bm, ke.bn);
    if (fn) return fn;
  }
  return ke.splitk;
}

static int most_splits(const sc_plan* pl, const KernelEntry& ke, int64_t rows) {
  const Geometry& g = pl->geo;
  if (!g.splitk_ok || !splitk_launcher(pl, ke) || pl->split_k == 1 || pl->gather_pipeline == 1) return 1;
  const int64_t tiles = ((rows + ke.bm - 1) / ke.bm) * ((pl->desc.c_out + ke.bn - 1) / ke.bn);
  const int64_t by_buffer = (int64_t)(kSplitKPartialBytes / ((size_t)ke.bm * ke.bn * sizeof(float))) / std::max<int64_t>(tiles, 1);
  return (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(by_buffer, g.k_tiles / 4), kSplitKMost));
}

// Buffer-load form of the tiled kernel: Cin a multiple of the K tile (a K tile then lies inside one tap),
// windows up to 8 x 8, tensors below 2 GiB (the out-of-range marker is offset 2^31).
static bool buf_applies(const sc_plan* pl, const KernelEntry& ke) {
  const sc_conv_desc& d = pl->desc;
  const Geometry& g = pl->geo;
  if (d.dtype == SC_F32) return false;
  const int eb = 2;
  const uint64_t xb = (uint64_t)d.n * d.h * d.w * d.c_in * eb, wb = (uint64_t)g.cout_pad * g.k_stride * eb;
  return buf_kernel(d.dtype == SC_BF16 ? kBF16 : kF16, ke.bm, ke.bn, g.k_tiles <= 2) && g.vec_gather && g.vec_out &&
         pl->gather_pipeline == 0 && d.c_in % 64 == 0 && d.kh <= 8 && d.kw <= 8 && xb < ((uint64_t)1 << 31) &&
         wb < ((uint64_t)1 << 31) && !g.rowseg;
}

// Stream-K launch of the buffer-load tiled kernel: how many persistent workgroups (0: an ordinary launch).
// Needs the split-K workspace (counters per tile, two partial-sum slots per workgroup), at least four K
// steps per workgroup, and step counts the kernel's 32-bit arithmetic holds.
static int stream_k_workgroups(const sc_plan* pl, const KernelEntry& ke, int64_t rows) {
  const Geometry& g = pl->geo;
  if (!g.splitk_ok || pl->stream_k == 1 || g.k_tiles <= 2 || !buf_applies(pl, ke)) return 0;
  if (!streamk_kernel(pl->desc.dtype == SC_BF16 ? kBF16 : kF16, ke.bm, ke.bn)) return 0;
  int want = pl->stream_k >= 2 ? pl->stream_k : 0;      // automatic: off
  if (want == 0) return 0;
  want = std::min((want + 7) / 8 * 8, kStreamKMostWgs);
  const int64_t tiles = ((rows + ke.bm - 1) / ke.bm) * ((pl->desc.c_out + ke.bn - 1) / ke.bn);
  const int64_t total = tiles * g.k_tiles;
  const int64_t by_buffer = (int64_t)(kSplitKPartialBytes / (2 * (size_t)ke.bm * ke.bn * sizeof(float))) / 8 * 8;
  want = (int)std::min<int64_t>(want, by_buffer);
  want = (int)std::min<int64_t>(want, total / 4 / 8 * 8);
  if (want < 8 || total * (want + 1) >= ((int64_t)1 << 31)) return 0;
  return want;
}

// ---- slab form of the tiled kernel --------------------------------------------------------------------
// 3x3 windows, stride 1, no dilation, 16-bit NHWC, input channels in chunks of 32, tensors below 2 GiB.
static int span_of(int bm) { return bm == 256 ? 2 : bm == 128 ? 1 : 0; }      // index of a tile's span
static bool slab_geometry_ok(const sc_conv_desc& d, const Geometry& g) {
  if (g.depthwise || g.rowseg || d.dtype == SC_F32 || d.layout != SC_NHWC || !g.vec_out) return false;
  if (d.kh != 3 || d.kw != 3 || d.stride_h != 1 || d.stride_w != 1 || d.dil_h != 1 || d.dil_w != 1) return false;
  if (d.pad_h > 2 || d.pad_w > 2 || d.c_in % kSlabCh != 0 || d.c_out < 96) return false;
  const uint64_t xb = (uint64_t)d.n * d.h * d.w * d.c_in * 2, wb = (uint64_t)g.cout_pad * g.k_stride * 2;
  return xb < ((uint64_t)1 << 31) && wb < ((uint64_t)1 << 31) && (int64_t)d.n * (d.h + 2 * d.pad_h) < ((int64_t)1 << 30);
}
// bytes of one slab buffer for tiles of bm rows whose widest slab spans `span` virtual rows (0: it does not fit)
static int slab_buffer_bytes(const sc_conv_desc& d, int bm, int span) {
  const int round = (bm == 256 ? 512 : 256) * 16;      // what one transfer of the whole workgroup covers
  const int64_t bytes = ((int64_t)span * (d.w + 2 * d.pad_w) * kSlabPixelBytes + round - 1) / round * round;
  return span > 0 && bytes <= kSlabMostBytes ? (int)bytes : 0;
}
// dense run: tiles are runs of bm consecutive pixels.  Where they begin in an image repeats after one period, and no tile spans more than one
// that begins in the last column of some row would (us a plan of 64 x 64 -> 64 @56, all tiles / until one is as wide as that: 130 / 85).
static int slab_dense_span(const sc_conv_desc& d, const Geometry& g, int bm) {
  const uint32_t hp = d.h + 2 * d.pad_h, ho_wo = g.ho * g.wo, wo = g.wo, m = (uint32_t)g.m;
  auto vrow = [&](uint32_t r) { return r / ho_wo * hp + r % ho_wo / wo; };
  uint32_t most = 0, span = 0;
  for (uint32_t q = wo - 1; q < ho_wo; q += wo) most = std::max(most, vrow(q + bm - 1) + d.kh - vrow(q));
  const uint32_t tiles = (m - 1) / bm + 1, period = ho_wo / std::gcd(ho_wo, (uint32_t)bm);
  for (uint32_t i = 0; i < std::min(tiles, period) && span < most; ++i) {
    const uint32_t m0 = i * bm, last = m - m0 > (uint32_t)bm ? m0 + bm - 1 : m - 1;
    span = std::max(span, vrow(last) + d.kh - vrow(m0));
  }
  return (int)span;
}
// K splits (by chunks of input channels) of a slab launch with tiles of bm rows: one workgroup per compute unit
static int slab_splits(const sc_plan* pl, int bm, int64_t rows) {
  const Geometry& g = pl->geo;
  if (!g.splitk_ok || pl->split_k == 1) return 1;
  const int64_t tiles = ((rows + bm - 1) / bm) * ((pl->desc.c_out + kSlabBN - 1) / kSlabBN);
  int64_t want = pl->split_k >= 2 ? pl->split_k : std::max<int64_t>(1, device_cus() / std::max<int64_t>(tiles, 1));
  const int64_t by_buffer = (int64_t)(kSplitKPartialBytes / ((size_t)bm * kSlabBN * sizeof(float))) / std::max<int64_t>(tiles, 1);
  want = std::min<int64_t>(std::min<int64_t>(want, by_buffer), std::min<int64_t>(pl->desc.c_in / kSlabCh, kSplitKMost));
  return (int)std::max<int64_t>(want, 1);
}
// the slab launch the options ask for, or the automatic one (bm == 0: none)
static sc_plan::Slab slab_pick(const sc_plan* pl, int which, int64_t rows) {
  const sc_plan::Slab none = {0, 1};
  if (!pl->slab_ok || pl->slab == 1 || rows == 0 || pl->gather_pipeline == 1) return none;
  if (pl->slab == 0) {
    if (pl->forced[which] != -1 || pl->split_k != 0 || pl->stream_k >= 2 || pl->masked_store == 2) return none;
    return pl->slab_auto[which];
  }
  for (int bm = 256; bm >= 128; bm >>= 1) {
    if (pl->slab >= 128 && pl->slab != bm) continue;
    if (slab_buffer_bytes(pl->desc, bm, pl->slab_span[which][span_of(bm)])) return {bm, slab_splits(pl, bm, rows)};
  }
  return none;
}
// ---- window kernel ------------------------------------------------------------------------------------------
// bytes of one of its slabs for tiles of bm rows (0: they do not fit)
static int window_slab_bytes(const sc_plan* pl, int which, int bm) {
  const sc_conv_desc& d = pl->desc;
  int span = pl->slab_span[which][span_of(bm)];
  if (pl->kept == pl->geo.m) span = std::max(span, pl->slab_span[1][span_of(bm)]);      // (such a run goes over the identity map)
  const int64_t px = (int64_t)span * (d.w + 2 * d.pad_w);
  if (span <= 0 || px > kWinMostPixels) return 0;
  return (int)((px * kWinPitch + 8191) / 8192 * 8192);
}
// Does the band kernel of a run stay, whatever the mask?  The alternating and the tap-pipelined one are ahead of the window kernel (us, band
// kernel / window kernel: 32 x 64 -> 64 @56 10.3 / 16, 1 x 64 -> 64 @56 5.7 / 6.7), and so is the plain one with few channels and few
// outputs (8 x 32 -> 16 @48 4.4 / 6.5).
static bool band_stays(const sc_conv_desc& d, const BandPlan& band) {
  return band.ok && !band.stream && (band.pp || band.tap || band.rowband || (d.c_in < 48 && d.c_out < 80) || std::getenv("SPARSE_CONV_BAND_KERNEL"));
}
// Predicted microseconds of a run by the plain band kernel (one band a workgroup, a 16-bit layer).  A round of workgroups costs its fixed
// part, the slabs of filters and input of those that share a compute unit, the rows they store, and the walk of the busiest wavefront: blocks
// of 32 or 64 rows, K steps of 16, each with an instruction a 32 x 32 block and, where the window shape is not known to the compiler
// (band_kernel's KH, KW, CPP), a fixed part; beyond the rounds a megabyte of y.  Fitted to 1 604 runs of 802 layers (16 to 160 channels in,
// 16 to 512 out, maps of 7 to 80, 3 x 3 and 5 x 5): standard deviation 5 % (2 to 6 % in each of the three walks, sparse and dense).
static double band_us(const sc_plan* pl, int which) {
  const sc_conv_desc& d = pl->desc;
  const Geometry& g = pl->geo;
  const BandPlan& b = which ? pl->band_dense : pl->band;
  const int cus = device_cus(), rows = which || pl->kept == g.m ? std::min(b.bh, g.ho) * g.wo : b.max_kept;
  int mi_idx = 0;
  const double blocks = band_units((double)rows, &mi_idx) / (mi_idx + 1);
  const int walk = d.kh == 3 && d.kw == 3 ? (d.c_in == 32 ? 1 : d.c_in == 64 ? 2 : 0) : 0;
  static const double steps[3][2] = {{0.0798, 0.0478}, {0.0019, 0.0517}, {0.0034, 0.0239}};      // fixed part, block of 32 x 32
  const double k_us = blocks * ((g.k + 15) / 16) * (steps[walk][0] + steps[walk][1] * (mi_idx + 1) * b.ni);
  const double kb = (double)(b.b_bytes + b.x_bytes) / 1024;
  const int64_t wgs = (int64_t)b.n_bands * b.n_tiles;
  const int resident = (int)std::min<size_t>(std::max<size_t>(kLdsLimit / b.lds, 1), 8);
  auto round_us = [&](int64_t on_cu) { return (which ? 2.75 : 3.71) + on_cu * (0.0171 * kb + 0.0009 * rows * b.ni) + k_us; };
  const int64_t full = (wgs - 1) / ((int64_t)cus * resident), rest = wgs - full * cus * resident;
  return full * round_us(resident) + round_us((rest + cus - 1) / cus) + 0.185 * 2e-6 * g.y_elems;
}
// may it run a tile?  (its slabs fit)
static bool window_fits(const sc_plan* pl, int which, int bm, int bn) {
  const int sb = pl->geo.window && window_kernel(kBF16, pl->desc.kh, bm, bn) ? window_slab_bytes(pl, which, bm) : 0;
  return sb > 0 && window_lds_bytes(bm, bn, sb, (pl->desc.c_in + kWinChunk - 1) / kWinChunk) <= kLdsLimit;
}
static constexpr int kWindowTiles[][2] = {{256, 128}, {128, 128}, {128, 64}, {64, 128}, {64, 64}};
// Its tile for the sparse / dense run, where it is expected to be faster than the cheapest tiled launch (bm == 0: it is not).
// SPARSE_CONV_WINDOW_TILE=<bm>x<bn> overrides, in the place of band kernels too (tuning and tests); 0x0 switches the kernel off.
static sc_plan::Window window_tile_for(const sc_plan* pl, int which) {
  const sc_plan::Window none = {0, 0, false};
  const sc_conv_desc& d = pl->desc;
  const int64_t rows = which ? pl->geo.m : pl->kept;
  if (!pl->geo.window || rows == 0) return none;
  const int chunks = (d.c_in + kWinChunk - 1) / kWinChunk;
  int fbm = 0, fbn = 0;
  if (const char* env = std::getenv("SPARSE_CONV_WINDOW_TILE"); env && std::sscanf(env, "%dx%d", &fbm, &fbn) == 2)
    return fbm > 0 && window_fits(pl, which, fbm, fbn) ? sc_plan::Window{fbm, fbn, true, false, true} : sc_plan::Window{0, 0, false, false, true};
  // A plain band kernel that does not stay is priced (band_us).  From 48 channels on it runs where it is cheaper than this kernel's tiles and
  // the others, by 3 % unless its walk is the unrolled one of 64 channels, whose price is good to 2 % (us, band / this kernel / another tile:
  // 3 x 48 -> 32 @17x22 8.1 / 6.3, 4 x 128 -> 16 @10x8 14.5 / 6.8, 58 x 128 -> 16 @31x36, every row, 41.9 / 15.8 / 12.0, but 62 x 64 -> 32 @53
  // 15.2 / 26.1 / 16.4 and, every row, 13.9 / 31.3 / 21.0, 56 x 64 -> 64 @45 at s = 0.25 16.4 / 20.8 / 19.1).  With fewer channels and many
  // outputs only this kernel takes its place, where it is 5 % cheaper (the price of the others is not made for a short K): over 263 layers
  // 0.80 and 0.77 of the band kernel's time.  Over 400 layers drawn at random, with rows dropped here and there, in blocks and at the end, the 205 sparse
  // and 270 dense runs that these rules give to this kernel take 0.58 times the time of the kernels without it, one 1.06 times, the others at most 1.03.
  const BandPlan& band = which ? pl->band_dense : pl->band;
  if (band_stays(d, band)) return none;
  const bool plain_band = band.ok && !band.stream, deep = d.c_in >= 48;
  // Priced like the other tiled launches (us, MI355X): a launch and its first round of workgroups, every further round, a chunk of 64
  // channels in a round, what a chunk takes longer the more compute units it keeps busy, and a megabyte of y.  Fitted to the runs of 170
  // layers (1 to 8 chunks, 16 to 512 outputs, maps of 7 to 80): standard deviation 4 to 8 %.  The others' price leaves out y and the
  // round trip of a split walk's sums; with both added it is as good.  On those layers the choice between these tiles and the cheapest
  // other launch takes 1.004 (sparse) and 1.006 times (dense) the time of the best one, and 1 / 1.34 and 1 / 1.35 of the others' alone.
  // 256 rows are for runs over every row: a sparse one of so many spans too many pixels.
  struct Shape { int bm, bn; double us[2][5]; };      // [sparse, dense]: first, further round, chunk, chunk by load, megabyte
  static const Shape shapes[] = {{256, 128, {{0, 0, 0, 0, 0}, {5.10, 6.0, 4.73, 0.61, 0.245}}},
                                 {128, 128, {{5.82, 3.34, 2.53, 0.04, 0.339}, {5.25, 3.67, 2.43, 0.49, 0.261}}},
                                 {128, 64, {{5.72, 3.76, 1.37, 0.23, 0.257}, {5.33, 3.66, 1.28, 0.42, 0.197}}},
                                 {64, 128, {{5.10, 0.82, 1.35, 0.43, 0.280}, {4.49, 1.16, 1.31, 0.66, 0.224}}},
                                 {64, 64, {{5.30, 1.32, 0.72, 0.44, 0.219}, {4.84, 1.59, 0.69, 0.55, 0.0}}}};
  const int cus = device_cus(), form = which || pl->kept == pl->geo.m ? 1 : 0;
  const sc_plan::Pick& other = pl->pick[which];
  const double mb = (double)pl->geo.y_elems * 2e-6;
  // The other launch by the model's price of it, y and a split walk's round trip: of the buffer-load kernel, of the direct-to-LDS one
  // and of the one through registers, whose K tiles cost more than the model has them (direct-to-LDS, 5 x 104 -> 96 @30: 7.9, takes 11).
  static const double others[3][2][3] = {{{-0.38, 0.99, 0.372}, {-0.75, 1.017, 0.515}},
                                         {{-2.99, 1.647, 0.209}, {-2.745, 1.621, 0.180}},
                                         {{-3.73, 1.91, 0.278}, {-3.74, 1.892, 0.381}}};
  const int family = !pl->geo.vec_out ? 2 : d.c_in % 64 != 0 ? 1 : 0;
  const double* o = others[family][form];
  double other_us = o[0] + o[1] * other.us + o[2] * mb + (other.splits > 1 ? 2.6 : 0.0);
  if (other.us == 0.0) return none;                               // (a launch that was asked for)
  const double band_price = plain_band ? band_us(pl, which) : 0.0;
  sc_plan::Window best = {0, 0, plain_band && deep};
  // (what has to be won: one chunk or less leaves this kernel's set-up uncovered, 10 x 64 -> 224 @16 6.35 / 6.6)
  const double ahead = d.c_in < 48 ? 0.9 : family ? 0.943 : chunks == 1 ? 0.97 : 1.0;
  double best_us = plain_band && !deep ? 0.95 * band_price : ahead * other_us;
  for (const Shape& sh : shapes) {
    if ((sh.bm == 256 && form == 0) || !window_fits(pl, which, sh.bm, sh.bn)) continue;
    const int64_t wgs = ((rows + sh.bm - 1) / sh.bm) * ((d.c_out + sh.bn - 1) / sh.bn);
    const double load = (double)wgs / cus, rounds = (double)((wgs + cus - 1) / cus);
    if (rounds > 1.0 && sh.bm == 64) continue;      // (set-up and sums again each round: 36 x 128 -> 432 @26x24 in three 24.0 / 30.0)
    const double* c = sh.us[form];
    const int kg = sh.bm == 256 ? 1 : sh.bn == 128 ? 2 : 4, last = (d.c_in - (chunks - 1) * kWinChunk + 15) / 16;      // K groups, K steps of the last chunk
    const double walk = (chunks - 1 + (double)((last + kg - 1) / kg * kg) / 4) * (d.kh * d.kw / 9.0);      // (in chunks of a 3 x 3 window)
    // (where a tile's share of the map holds more dropped rows than have their zeros written ahead of the products, two thirds for 64 rows, the
    // others come behind them, and the slab grows.  us beyond the price in one chunk, 64 x 64: s = 0.6 0.0, 0.7 0.5, 0.8 0.6, the other tiles
    // alike.  17 x 32 -> 40 @14x15 at s = 0.7 takes 6.6 to 6.9, priced 6.0, in another tile 6.3.  The price of 5 x 5 windows, 10 % high, has room for it.)
    const bool over = form == 0 && d.kh == 3 && pl->geo.m * sh.bm > rows * (2 * sh.bm + 64);
    const double between = over ? 0.5 + 0.5 * std::max(0.0, std::log((double)pl->geo.m / (3.3 * rows))) : 0.0;
    // (two prices are low.  Half of the wavefronts of 256 x 128 hold no outputs where there are 64 or fewer: 57 x 48 -> 40 @23x26, every row, 10.4 us,
    // in other tiles 9.3, 37 x 72 -> 40 @31 13.1 / 12.0, but 60 x 72 -> 40 @45x48 26.1 / 29.0.  And 128 rows and more over every row of one whole
    // chunk, where much of y goes out at once: 20 x 64 -> 320 @22 9.8 / 9.0, 40 x 64 -> 384 @14 9.9 / 9.3, but 64 x 64 -> 512 @12 12.4 / 14.2.)
    const double low = sh.bm == 256 && d.c_out <= 64 ? 1.08 : sh.bm >= 128 && form && chunks == 1 && family == 0 ? 1.055 : 1.0;
    const double us = (c[0] + c[1] * (rounds - 1) + walk * (c[2] * rounds + c[3] * load) + c[4] * mb) * low + between;
    if (us < best_us) { best_us = us; best = {sh.bm, sh.bn, plain_band, plain_band && !deep}; }
  }
  if (plain_band && deep && band_price < (d.c_in == 64 ? 1.0 : 0.97) * best_us / ahead) return none;
  return best;
}
// (not where a tile or a form of another kernel was asked for or measured faster)
static bool window_is_free(const sc_plan* pl, int which, int64_t rows) {
  return rows > 0 && pl->forced[which] == -1 && !pl->prefer_tiled[which] && pl->gather_pipeline == 0 && pl->split_k == 0 &&
         pl->stream_k < 2 && pl->masked_store != 2 && pl->slab == 0 && pl->row_panel != 2 && !pl->slab_auto[which].bm;
}
// does a run of a dense input take the window kernel?
static bool use_window(const sc_plan* pl, int which, int64_t rows, bool plain = true) {
  return pl->window[which].bm > 0 && (plain || !pl->window[which].plain_only) && window_is_free(pl, which, rows);
}
// is the band kernel that applies left out for it, or for a tile?
static bool bands_give_way(const sc_plan* pl, int which, int64_t rows) {
  return pl->window[which].before_bands && window_is_free(pl, which, rows);
}
// ---- register-staged kernel ------------------------------------------------------------------------------
// The direct-to-LDS form serves the float NHWC layers whose rows are whole 16-byte groups.
static bool stage_is_direct(const sc_conv_desc& d, const Geometry& g) {
  return g.stage_gather == kStageGroups && d.c_out % 4 == 0 &&
         (int64_t)g.stage_blocks * g.stage_k_tiles * StageDims<kF32>::BLOCK_BYTES < ((int64_t)1 << 31);
}
static LaunchFn stage_launcher(const sc_conv_desc& d, const Geometry& g, StageTile t) {
  if (stage_is_direct(d, g))
    return split_kernel(t.bm, t.bn, t.groups, d.c_in % StageDims<kF32>::K_TILE == 0, d.c_out % 16 == 0 ? 1 : 2);
  return stage_kernel(d.dtype == SC_BF16 ? kBF16 : d.dtype == SC_F16 ? kF16 : kF32, g.stage_gather, d.layout == SC_NCHW, t.bm, t.bn, t.groups);
}
// Its tile for a run of `rows` rows.  SPARSE_CONV_STAGE_TILE=<bm>x<bn>[x<groups>] overrides (tuning and tests), 0x0 switches the
// kernel off.
// `groups` > 0 fixes the number of groups: both runs of a plan take the same, so that they add a row's products in the same order
// and a kept row carries the same bits in either (stage_tiles_for).  price: of the direct form, its predicted time.
static StageTile stage_tile_for(const sc_conv_desc& d, const Geometry& g, int64_t rows, int groups = 0, double* price = nullptr) {
  StageTile none = {0, 0, 1, false};
  if (g.stage_gather < 0 || rows == 0) return none;
  int fbm = 0, fbn = 0, fgr = 1;
  if (const char* env = std::getenv("SPARSE_CONV_STAGE_TILE"); env && std::sscanf(env, "%dx%dx%d", &fbm, &fbn, &fgr) >= 2)
    return fbm > 0 && stage_launcher(d, g, {fbm, fbn, fgr, true}) ? StageTile{fbm, fbn, fgr, true} : none;
  const int kt = g.stage_k_tiles;
  if (stage_is_direct(d, g)) {
    // Priced like the other tiled launches (us, MI355X): what a K tile costs a compute unit with enough workgroups on it, what it costs
    // a workgroup alone, and a round of workgroups beyond its K loop, where the stores and the zero fill of a tile count.  The figures
    // are fitted to the sparse and dense runs of all nine tiles on 90 layers (1 to 100 K tiles, 8 to 400 channels).  Chosen tile against
    // the fastest one, geometric mean over 150 layers: sparse runs 1.015, dense 1.024, fused 1.036; with one figure for every tile's round
    // 1.023, 1.026 and 1.048.  Sparse runs at s = 0.5, chosen tile / 128 x 64 in one group / the float-MFMA kernel:  32 x 64 -> 64 @56
    // 27.5 / 27.5 / 60;  128 -> 128 @28 25.5 / 28.6 / 55;  256 -> 256 @14 30.8 / 47 / 61;  16 x 384 -> 384 @12 29.2 / 67 / 88;
    // 1 x 128 -> 128 @28 12.2 / 25 / 32 (batch 32 where not said; where few workgroups walk a long K, groups share it).
    struct Shape { StageTile t; double per_tile, alone, round; int waves; };
    static const Shape shapes[] = {
        {{128, 64, 1, false}, 0.57, 0.57, 5.5, 4},  {{128, 64, 2, false}, 0.46, 0.93, 5.9, 8}, {{128, 32, 1, false}, 0.40, 0.48, 4.7, 4},
        {{128, 32, 2, false}, 0.33, 0.77, 5.0, 8},  {{64, 64, 1, false}, 0.32, 0.49, 5.6, 2},  {{64, 64, 2, false}, 0.30, 0.63, 5.4, 4},
        {{64, 32, 1, false}, 0.215, 0.44, 4.5, 2}, {{64, 32, 2, false}, 0.21, 0.53, 4.6, 4}, {{64, 32, 4, false}, 0.19, 0.86, 4.7, 8}};
    const int cus = device_cus();
    StageTile best = none;
    double best_us = 1e300;
    for (const Shape& sh : shapes) {
      if (groups > 0 && sh.t.groups != groups) continue;
      const int64_t wgs = ((rows + sh.t.bm - 1) / sh.t.bm) * ((d.c_out + sh.t.bn - 1) / sh.t.bn);
      const int lds = sh.t.groups * 2 * (sh.t.bm * kRowBytes + sh.t.bn / 32 * StageDims<kF32>::BLOCK_BYTES);
      const int resident = std::max(1, std::min((int)(kLdsLimit / lds), (sh.t.bn == 64 ? 8 : 12) / sh.waves));
      const int steps = (kt + sh.t.groups - 1) / sh.t.groups;
      auto round_us = [&](int64_t on_cu) {
        double step = std::max(sh.alone, (double)on_cu * sh.t.groups * sh.per_tile);
        if (sh.waves == 2 && on_cu >= 2) step = std::max(step, 0.81);       // (their wavefronts share two of the four SIMDs)
        return sh.round + steps * step;
      };
      const int64_t full = wgs / ((int64_t)cus * resident), rest = wgs - full * cus * resident;
      const double us = full * round_us(resident) + (rest ? round_us((rest + cus - 1) / cus) : 0.0);
      if (us < best_us) { best_us = us; best = sh.t; }
    }
    if (price) *price = best_us;
    return best;
  }
  // Through registers (us a sparse run, s = 0.5 where not said).  64 rows keep most workgroups in flight: 64 x 64 / 128 x 64
  // 40 / 48 for 32 x 128 -> 128 @28 channels first in float, 40 / 42 for 64 x 51 -> 51 @56 in bf16 at s = 0.3, 27 / 38 for
  // 64 x 410 -> 410 @7.  Where 128 channels in a workgroup still cover the compute units once, half of the gathers are saved and
  // a second group of wavefronts hides one's transfers behind the other's products, 64 x 64 / 64 x 128 in two groups: 40 / 37
  // for the first layer, 29 / 21 in bf16; not for the groups of ragged pixels, which are few loads: 32 x 102 -> 102 @28 in
  // float 33.4 / 34.3, in fp16 14.2 / 16.3.  Beyond one round two groups lose (their LDS leaves one workgroup on a compute
  // unit): 64 x 102 -> 102 @28 in fp16 at s = 0.3 28.1 / 40, 25.7 for 64 x 128 in one group.
  // Two groups of 64 x 64 / one where they are at most one round: 4 x 128 -> 128 @28 channels first in float 21.8 / 26.6,
  // 16 x 256 -> 256 @14 39 / 49, 410 -> 410 @7 22.4 / 27.2, 8 x 205 -> 205 @14 in fp16 14.2 / 17.2; two rounds: 20 x 37 -> 77
  // @30 24.5 / 17.6; short K: 33 -> 30 @56 in bf16 (five tiles) no difference; at one to three tiles the dense run, which takes the
  // sparse run's groups in several rounds, loses up to half (16 x 3 -> 256 @28 in float 25.0 with two groups, 12.1 with one).
  // Tiles of 32 channels keep a wavefront to a row block of its own and pay from a round of workgroups on: 64 x 64 / 128 x 32 for
  // 16 x 33 -> 30 @56 in bf16 13.6 / 16.0.
  const int cus = device_cus();
  auto wgs_of = [&](int bm, int bn) { return ((rows + bm - 1) / bm) * ((d.c_out + bn - 1) / bn); };
  if (groups <= 1) {
    if (d.c_out <= 32 && wgs_of(128, 32) >= cus) return {128, 32, 1, false};
    if (kt <= 2 && wgs_of(128, 64) >= cus) return {128, 64, 1, false};
  }
  const bool wide = d.c_out > 64 && (d.c_out % 128 == 0 || d.c_out % 128 > 64);
  const int64_t wgs = wgs_of(64, 128);
  if (wide && wgs >= cus * 3 / 4 && wgs <= cus && g.stage_gather >= kStageChunks && (groups == 0 ? kt >= 4 : groups == 2))
    return {64, 128, 2, false};
  if (wide && wgs > cus && d.dtype != SC_F32 && groups != 2) return {64, 128, 1, false};
  if (groups > 0) return {64, 64, groups, false};
  if (wgs_of(64, 64) <= cus && kt >= (d.dtype == SC_F32 ? 4 : 8)) return {64, 64, 2, false};
  return {64, 64, 1, false};
}
// The tiles of both runs.
static void stage_tiles_for(const sc_conv_desc& d, const Geometry& g, int64_t kept, StageTile (&out)[2]) {
  out[0] = stage_tile_for(d, g, kept);
  if (out[0].bm && !out[0].asked && stage_is_direct(d, g)) {
    // the number of groups that is best for both, the sparse run counting three times: by itself it would cut a short walk in four
    // where the dense one then takes several rounds (4 x 96 -> 256 @28 pointwise, sparse / dense: 7.3 / 11.2 us)
    double own[2], best = 1e300;
    StageTile t[2];
    (void)stage_tile_for(d, g, kept, 0, &own[0]);
    (void)stage_tile_for(d, g, g.m, 0, &own[1]);
    for (int groups = 1; groups <= 4; groups *= 2) {
      double us[2];
      t[0] = stage_tile_for(d, g, kept, groups, &us[0]);
      t[1] = stage_tile_for(d, g, g.m, groups, &us[1]);
      const double cost = 3.0 * us[0] / own[0] + us[1] / own[1];
      if (t[0].bm && t[1].bm && cost < best) { best = cost; out[0] = t[0]; out[1] = t[1]; }
    }
    return;
  }
  // Through registers, one or two K tiles before many outputs: the stores are what counts, and the element gather, of which more
  // workgroups share a compute unit, is as fast or faster where it stores 16-byte groups: 32 x 13 -> 256 @56 pointwise
  // 35.7 / 37.8 us in bf16, 52 / 61 in float; 16 x 51 -> 256 @28 in bf16 8.2 / 9.1; fewer outputs 8.9 / 7.4 (half of the rows).
  if (out[0].bm && !out[0].asked && d.layout == SC_NHWC && g.vec_out && g.stage_k_tiles <= (d.dtype == SC_F32 ? 2 : 1) &&
      kept * d.c_out >= (int64_t)5 << 19) {
    out[0] = out[1] = {0, 0, 1, false};
    return;
  }
  out[1] = stage_tile_for(d, g, g.m, out[0].bm ? out[0].groups : 0);
}
enum LaunchForm { kPlainRun, kCompactRun, kFusedRun };      // dense operands; a compact one; with a shortcut sum
// Layers that stay with the other kernels though the staged one could run them (one line for the sparse and the dense run, see
// above; us, another kernel / staged).
static bool leave_to_others(const sc_plan* pl, LaunchForm form) {
  const sc_conv_desc& d = pl->desc;
  const Geometry& g = pl->geo;
  // Float layers that a band kernel serves, while they are small (there are no such bands for the other forms): 16 -> 16 @16, one
  // image, 6.4 / 7.1; 16 -> 16 @56, four images, 6.9 / 7.3; with 2.3e8 multiply-adds in all rows 10.4 and 11.4 / 9.5 and 10.8.
  if (form == kPlainRun && pl->band.ok && (double)g.m * g.k * d.c_out < 8e7) return true;
  // Float layers with a short K and few outputs: the launch is most of the time, and the tiles that contract every row and mask at
  // the store save the row list's round trip (fused launches do not have that form; compact and dense runs, which would gain, add in the
  // order of the plain one).  Half of the rows, another kernel / staged, plain, compact output and dense, by K tiles of 32 entries,
  // pointwise @28: 16 x 32 -> 64 (1) 5.1 / 5.9, 4.55 / 4.15, 5.0 / 4.7; 64 -> 64 (2) 5.8 / 6.1, 5.2 / 4.6, 5.7 / 5.2; 32 x 32 -> 32 (1) 5.5 / 5.8, 4.8 / 4.1, 5.3 /
  // 4.7; 16 x 128 -> 64 (4) 7.3 / 6.6, 6.9 / 5.5, 7.3 / 6.0; more outputs: 32 -> 256 (1) 9.9 / 7.85, 7.4 / 5.6, 11.3 / 7.7, 96 -> 96 (3) 7.4 / 7.2, 6.2 / 5.4, 9.3 /
  // 6.3.
  return form != kFusedRun && stage_is_direct(d, g) && g.stage_k_tiles <= 4 && (double)g.m * d.c_out * g.stage_k_tiles < 2.4e6;
}
// does a run take it?  (not where a tile, a band kernel or another form of the tiled kernel was asked for)
static bool use_stage(const sc_plan* pl, int which, LaunchForm form = kPlainRun) {
  if (form == kPlainRun && pl->stage_tuned < 0) return false;
  if (pl->stage_tuned <= 0 && !pl->stage_pick[which].asked && leave_to_others(pl, form)) return false;
  // (options that name a form of the other kernels count only where that form applies)
  return pl->stage_pick[which].bm > 0 && pl->forced[which] == -1 && (pl->gather_pipeline == 0 || !pl->geo.vec_gather) &&
         !(pl->masked_store == 2 && which == 0 && form == kPlainRun && pl->desc.layout == SC_NHWC) && !pl->prefer_tiled[which];
}
static TilePick pick_tile(const sc_plan* pl, int which, int64_t rows) {
  TilePick tp;
  tp.masked = false;
  if (pl->forced[which] >= 0) {          // tuning: the forced tile, split as requested
    tp.ti = pl->forced[which];
    tp.splits = pl->split_k >= 2 ? std::min(pl->split_k, most_splits(pl, pl->table[tp.ti], rows)) : 1;
    tp.masked = pl->masked_store == 2 && which == 0;
    return tp;
  }
  tp.ti = pl->pick[which].ti;
  tp.splits = pl->split_k == 1 ? 1 : std::min(pl->pick[which].splits, most_splits(pl, pl->table[tp.ti], rows));
  tp.masked = pl->masked_store == 2 ? which == 0 : pl->masked_store == 1 ? false : pl->pick[which].masked;
  const sc_plan::Pick& pick = pl->pick[which];
  if (pick.grouped >= 0 && !tp.masked && (pick.asked || group_candidates(pl, pl->table[pick.grouped], rows) > 1))
    tp = {pick.grouped, 1, false, pick.splits};
  if (pl->split_k >= 2 && pl->tile_splitk >= 0) {      // on request: that many splits of the 64 x 128 tile
    const int want = std::min(pl->split_k, most_splits(pl, pl->table[pl->tile_splitk], rows));
    if (want >= 2) tp = {pl->tile_splitk, want, false};
  }
  return tp;
}


// residual (may be null): shortcut tensor in the format of y, fused into the epilogue of a tiled kernel:
// y = post(act(conv + bias) + residual); dropped rows of a dense-layout output receive post(residual).
static sc_status launch_conv(const sc_plan* pl, bool dense, const void* x, const float* bias, void* y,
                             hipStream_t stream, bool x_compact = false, bool y_compact = false,
                             const void* residual = nullptr, int residual_relu = 0) {
  const sc_conv_desc& d = pl->desc;
  const Geometry& g = pl->geo;
  const int which = dense ? 1 : 0;
  const int64_t rows = dense ? g.m : pl->kept;
  const bool zero_fill = !dense && !y_compact && d.out_mode == SC_OUT_ZERO_FILL && pl->kept < g.m;
  // a mask that keeps every row makes the row list the identity: skip the indirection; so does a run
  // whose input and output both hold the kept rows only (row i in, row i out)
  // (not for a depthwise layer with windows: its compact input follows the input's mask, not its own)
  const bool ranked_input = x_compact && g.depthwise && d.kh * d.kw > 1;
  const bool identity = dense || pl->kept == g.m || (x_compact && y_compact && !ranked_input);
  const bool compact = !identity && (x_compact || y_compact);
  const int eb = elem_bytes(d.dtype);
  if (rows == 0) {
    if (d.out_mode == SC_OUT_ZERO_FILL && !y_compact && residual) {
      const dim3 grid((unsigned)std::min<int64_t>((g.y_elems + 255) / 256, 65536)), block(256);
      if (d.dtype == SC_F32)
        hipLaunchKernelGGL(shortcut_only_kernel<float>, grid, block, 0, stream, (const float*)residual, (float*)y, g.y_elems, residual_relu);
      else if (d.dtype == SC_F16)
        hipLaunchKernelGGL(shortcut_only_kernel<_Float16>, grid, block, 0, stream, (const _Float16*)residual, (_Float16*)y, g.y_elems, residual_relu);
      else
        hipLaunchKernelGGL(shortcut_only_kernel<__bf16>, grid, block, 0, stream, (const __bf16*)residual, (__bf16*)y, g.y_elems, residual_relu);
      SC_HIP(hipGetLastError());
    } else if (d.out_mode == SC_OUT_ZERO_FILL && !y_compact) {
      int64_t bytes = g.y_elems * eb;
      int64_t n16 = bytes / 16;
      int ntail = (int)(bytes - n16 * 16);
      int grid = (int)std::min<int64_t>((n16 + 255) / 256 + 1, 4096);
      hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, stream, (uint4*)y, n16,
                         (unsigned char*)y + n16 * 16, ntail);
      SC_HIP(hipGetLastError());
    }
    return SC_OK;
  }
  // the streaming variant measured no faster than the tiled kernel on the benchmark layers, so the
  // automatic choice takes it only on request
  if (g.depthwise) {
    if (residual) return SC_ERR_UNSUPPORTED;
    DepthwiseParams q;
    std::memset(&q, 0, sizeof(q));
    q.x = x;
    q.wp = pl->ws + g.off_wp;
    q.bias = d.has_bias ? bias : nullptr;
    q.y = y;
    // zero-fill runs walk the dense rows and look at the mask; the others walk the kept rows
    q.row_idx = (identity || zero_fill) ? nullptr : reinterpret_cast<const int32_t*>(pl->ws + g.off_rows);
    q.mask = identity ? nullptr : pl->ws + g.off_mask;
    // Only the zero-fill walk visits all M dense rows.  Every other run visits `rows` items: M for a dense run or
    // a mask that keeps everything, the kept rows otherwise -- through the row list, or as the identity over the
    // kept rows when both operands are compact (x and y then hold kept * C elements, not M * C).
    q.items = zero_fill ? g.m : rows;
    q.zero_fill = zero_fill ? 1 : 0;
    q.rank = (compact && y_compact) ? reinterpret_cast<const int32_t*>(pl->ws + g.off_band_rows) : nullptr;
    q.n = d.n; q.ho = g.ho; q.cus = device_cus(); q.kernel = pl->depthwise_kernel;
    q.c = d.c_in; q.h = d.h; q.w = d.w; q.ho_wo = g.ho * g.wo; q.wo = g.wo;
    q.kh = d.kh; q.kw = d.kw; q.sh = d.stride_h; q.sw = d.stride_w; q.ph = d.pad_h; q.pw = d.pad_w;
    q.dil_h = d.dil_h; q.dil_w = d.dil_w;
    q.relu = d.relu;
    q.mask_spatial = d.mask_mode == SC_MASK_SPATIAL;
    q.x_compact = (compact && x_compact) || ranked_input ? 1 : 0;
    q.y_compact = compact && y_compact ? 1 : 0;
    // A 1x1 layer whose compact input feeds a zero-filled dense output walks the dense rows, so the item number is
    // no longer the row of x: a kept pixel finds its row in the layer's own rank table (input and output pixels
    // coincide for such a window; dropped pixels leave before they read).
    const bool own_rank_input = compact && x_compact && !ranked_input && zero_fill;
    q.x_rank = ranked_input     ? reinterpret_cast<const int32_t*>(pl->ws + g.off_xrank)
               : own_rank_input ? reinterpret_cast<const int32_t*>(pl->ws + g.off_band_rows)
                                : nullptr;
    magic_div((uint32_t)q.ho_wo, &q.div_howo_mul, &q.div_howo_shift);
    magic_div((uint32_t)q.wo, &q.div_wo_mul, &q.div_wo_shift);
    SC_HIP(depthwise_launch(d.dtype == SC_BF16 ? kBF16 : d.dtype == SC_F16 ? kF16 : kF32, q, stream));
    return SC_OK;
  }
  // the band kernels address input and output by dense position: runs with a compact operand take a tiled kernel
  const BandPlan& band = dense ? pl->band_dense : pl->band;
  // (of the band and row-panel kernels only the alternating-group band kernel has a shortcut path: any other
  // fused launch takes a tiled kernel)
  const sc_plan::Slab slab = x_compact ? sc_plan::Slab{0, 1} : slab_pick(pl, which, rows);
  const bool staged = use_stage(pl, which, residual ? kFusedRun : x_compact || y_compact ? kCompactRun : kPlainRun);
  const bool use_band = band.ok && !x_compact && !y_compact && (!residual || ((band.pp || band.tap) && !band.stream)) &&
                        (pl->forced[which] == kForceBand || (pl->forced[which] == -1 && !band.stream && !pl->prefer_tiled[which])) &&
                        !(slab.bm && pl->slab >= 2) && !staged && !bands_give_way(pl, which, rows);
  if (use_band) {
    const BandPlan& b = band;
    BandParams q;
    std::memset(&q, 0, sizeof(q));
    q.x = x;
    q.wp = pl->ws + g.off_wp;
    q.bias = d.has_bias ? bias : nullptr;
    q.y = y;
    q.row_idx = identity ? nullptr : reinterpret_cast<const int32_t*>(pl->ws + g.off_rows);
    q.mask = pl->ws + g.off_mask;
    q.band_i0 = reinterpret_cast<const int32_t*>(pl->ws + g.off_band);
    q.band_rows = reinterpret_cast<const int32_t*>(pl->ws + g.off_band_rows);
    q.h = d.h; q.w = d.w; q.c_in = d.c_in; q.ho = g.ho; q.wo = g.wo; q.c_out = d.c_out;
    q.kh = d.kh; q.kw = d.kw; q.sh = d.stride_h; q.sw = d.stride_w; q.ph = d.pad_h; q.pw = d.pad_w;
    q.dil_h = d.dil_h; q.dil_w = d.dil_w;
    q.k_stride = g.k_stride;
    q.bh = b.bh; q.split = b.split; q.bands_per_image = b.bands_per_image; q.n_bands = b.n_bands; q.n_tiles = b.n_tiles;
    q.b_bytes = (int32_t)b.b_bytes;
    q.x_groups = (int32_t)(b.x_bytes / 16);
    q.relu = d.relu;
    q.zero_fill = zero_fill ? 1 : 0;
    q.mask_spatial = d.mask_mode == SC_MASK_SPATIAL;
    magic_div((uint32_t)g.wo, &q.div_wo_mul, &q.div_wo_shift);
#ifdef SC_TIMING
    q.dbg = g_dbg;
#endif
    if (b.rowband) {
      RowBandParams rq;
      rq.b = q;
      rq.pitch = b.rb_pitch; rq.left = b.rb_left; rq.in_rows = b.rb_in_rows;
      rq.gpw = b.rb_gpw; rq.groups = d.kh * b.rb_gpw; rq.tail = b.rb_tail;
      rq.fpitch = rowband_filter_pitch(rq.groups);
      magic_div((uint32_t)(b.rb_pitch / 16), &rq.div_cpr_mul, &rq.div_cpr_shift);
      int mi_idx = 0;
      band_units(dense || identity ? (double)(std::min(b.bh, g.ho) * g.wo) : (double)b.max_kept, &mi_idx);
      if (4 * b.lds <= kLdsLimit) mi_idx = 0;      // four workgroups per compute unit: only the 32-row form has the registers
      RowBandLaunchFn fn = bandrow_kernel_for(d.dtype == SC_BF16 ? kBF16 : kF16, mi_idx + 1, d.kh, b.rb_gpw);
      if (!fn) return SC_ERR_UNSUPPORTED;
      SC_HIP(fn(rq, b.lds, stream));
      return SC_OK;
    }
    if (b.stream) {
      // every kept row of a band sits in accumulators: 128 rows per MI step
      const int most = dense ? b.bh * g.wo : b.max_kept;
      const int mi = std::max(1, (most + 127) / 128);
      if (mi > (b.ni == 4 ? 3 : 4)) return SC_ERR_UNSUPPORTED;   // cannot happen: the planner caps the band rows
      SC_HIP(pl->stream_table->fn[b.ni == 4 ? 1 : 0][mi - 1](q, b.lds, stream));
      return SC_OK;
    }
    // 32-row (MI = 1) or 64-row (MI = 2) MFMA blocks, dealt to the four wavefronts round robin: the
    // shape that leaves the busiest wavefront fewer 32-row units
    int mi_idx = 0;
    const int band_px = (std::min(b.bh, g.ho) * g.wo + (b.split ? 1 : 0)) / (b.split ? 2 : 1);
    band_units(dense || identity ? (double)band_px : (double)b.max_kept, &mi_idx);
    if (b.tap) {
      // 32-row blocks b = wave, wave + 8: one or two per wavefront, by the fullest band of the run
      const int most = dense || identity ? band_px : b.max_kept;
      if (most > kTapMaxRows) return SC_ERR_UNSUPPORTED;   // cannot happen: the planner caps the band rows
      q.residual = residual;
      q.residual_relu = residual_relu ? 1 : 0;
      const auto& table = residual ? pl->tap_table->fn_res : pl->tap_table->fn;
      SC_HIP(table[d.c_in / g.vec == 8 ? 0 : 1][b.ni - 1][most > 256 ? 1 : 0](q, b.lds, stream));
      return SC_OK;
    }
    if (b.pp) {
      q.residual = residual;
      q.residual_relu = residual_relu ? 1 : 0;
      const auto& table = residual ? pl->pp_table->fn_res : pl->pp_table->fn;
      SC_HIP(table[d.c_in / g.vec == 8 ? 0 : 1][b.ni - 1][mi_idx](q, b.lds, b.pp_grid, stream));
      return SC_OK;
    }
    // (one line for the sparse and the dense run: both add a row's products in the same order)
    if (d.dtype == SC_F32 && (int64_t)std::max(pl->band.bh, pl->band_dense.bh) * g.wo <= 32 &&
        std::min(pl->band.b_bytes, pl->band_dense.b_bytes) >= (size_t)3 * 4096 * b.ni) {
      q.share_k = 1;
      mi_idx = 0;
    }
    const int cpp = d.c_in / g.vec;
    const int shape = (d.kh == 3 && d.kw == 3 && cpp == 8) ? 1 : (d.kh == 3 && d.kw == 3 && cpp == 4) ? 2 : 0;
    SC_HIP(pl->band_table->fn[shape][b.ni_idx][mi_idx](q, b.lds, stream));
    return SC_OK;
  }
  if (!x_compact && !slab.bm && use_window(pl, which, rows, !residual && !y_compact)) {
    const sc_plan::Window win = pl->window[which];
    ConvParams p;
    std::memset(&p, 0, sizeof(p));
    p.x = x;
    p.wp = pl->ws + g.off_window_w;
    p.bias = d.has_bias ? bias : nullptr;
    p.y = y;
    p.row_idx = identity ? nullptr : reinterpret_cast<const int32_t*>(pl->ws + g.off_rows);
    p.mask = pl->ws + g.off_mask;
    p.rows = (int32_t)rows;
    p.m_total = (int32_t)g.m;
    p.h = d.h; p.w = d.w; p.ho_wo = g.ho * g.wo; p.wo = g.wo;
    magic_div((uint32_t)p.ho_wo, &p.div_howo_mul, &p.div_howo_shift);
    magic_div((uint32_t)p.wo, &p.div_wo_mul, &p.div_wo_shift);
    p.ph = d.pad_h; p.pw = d.pad_w;
    p.c_in = d.c_in; p.c_out = d.c_out;
    p.relu = d.relu;
    p.zero_fill = zero_fill ? 1 : 0;
    p.mask_spatial = d.mask_mode == SC_MASK_SPATIAL;
    p.y_compact = compact && y_compact ? 1 : 0;
    p.residual = residual;
    p.residual_relu = residual_relu ? 1 : 0;
    p.m_tiles = (int32_t)((rows + win.bm - 1) / win.bm);
    p.n_tiles = (d.c_out + win.bn - 1) / win.bn;
    p.splits = p.m_tiles * p.n_tiles <= device_cus() ? 1 : 0;
    p.x_bytes = (uint32_t)(g.x_elems * eb);
    p.w_bytes = (uint32_t)((uint64_t)((d.c_out + 31) / 32) * 32 * d.kh * d.kw * ((d.c_in + kWinChunk - 1) / kWinChunk) * kWinChunk * eb);
    p.vec_out = g.vec_out ? 1 : 2;
    p.slab_bytes = window_slab_bytes(pl, which, win.bm);
    p.zero_share = (int32_t)((g.m + p.m_tiles - 1) / p.m_tiles);
    p.slab_hp = d.h + 2 * d.pad_h;
    p.slab_wp = d.w + 2 * d.pad_w;
    magic_div((uint32_t)p.slab_hp, &p.div_hp_mul, &p.div_hp_shift);
    magic_div((uint32_t)p.slab_wp, &p.div_wp_mul, &p.div_wp_shift);
#ifdef SC_TIMING
    p.dbg = g_dbg;
#endif
    LaunchFn fn = window_kernel(d.dtype == SC_BF16 ? kBF16 : kF16, d.kh, win.bm, win.bn);
    if (!fn || !p.slab_bytes) return SC_ERR_UNSUPPORTED;    // cannot happen: the pick checked both
    SC_HIP(fn(p, stream));
    return SC_OK;
  }
  if (slab.bm) {
    ConvParams p;
    std::memset(&p, 0, sizeof(p));
    p.x = x;
    p.wp = pl->ws + g.off_wp;
    p.bias = d.has_bias ? bias : nullptr;
    p.y = y;
    p.row_idx = identity ? nullptr : reinterpret_cast<const int32_t*>(pl->ws + g.off_rows);
    p.mask = pl->ws + g.off_mask;
    p.rows = (int32_t)rows;
    p.m_total = (int32_t)g.m;
    p.h = d.h; p.w = d.w; p.ho_wo = g.ho * g.wo; p.wo = g.wo;
    magic_div((uint32_t)p.ho_wo, &p.div_howo_mul, &p.div_howo_shift);
    magic_div((uint32_t)p.wo, &p.div_wo_mul, &p.div_wo_shift);
    p.sh = 1; p.sw = 1; p.ph = d.pad_h; p.pw = d.pad_w;
    p.c_in = d.c_in; p.kh = d.kh; p.kw = d.kw; p.dil_h = 1; p.dil_w = 1;
    p.c_out = d.c_out;
    p.k_pad = g.k_stride; p.k_tiles = g.k_tiles;
    p.relu = d.relu;
    p.zero_fill = zero_fill ? 1 : 0;
    p.mask_spatial = d.mask_mode == SC_MASK_SPATIAL;
    p.vec_out = 1;
    p.y_compact = compact && y_compact ? 1 : 0;
    p.residual = residual;
    p.residual_relu = residual_relu ? 1 : 0;
    p.m_tiles = (int32_t)((rows + slab.bm - 1) / slab.bm);
    p.n_tiles = (d.c_out + kSlabBN - 1) / kSlabBN;
    p.x_bytes = (uint32_t)((uint64_t)d.n * d.h * d.w * d.c_in * eb);
    p.w_bytes = (uint32_t)((uint64_t)g.cout_pad * g.k_stride * eb);
    // (a mask that keeps every row runs over the identity map: its tiles are those of the dense run)
    p.slab_bytes = slab_buffer_bytes(d, slab.bm, std::max(pl->slab_span[which][span_of(slab.bm)],
                                                          identity ? pl->slab_span[1][span_of(slab.bm)] : 0));
    p.slab_hp = d.h + 2 * d.pad_h;
    p.slab_wp = d.w + 2 * d.pad_w;
    magic_div((uint32_t)p.slab_hp, &p.div_hp_mul, &p.div_hp_shift);
    magic_div((uint32_t)p.slab_wp, &p.div_wp_mul, &p.div_wp_shift);
    if (p.slab_bytes == 0) return SC_ERR_UNSUPPORTED;    // cannot happen: slab_pick checked the span
    const int splits = std::min(slab.splits, d.c_in / kSlabCh);
    if (splits > 1) {
      p.splits = splits;
      p.partial = reinterpret_cast<float*>(pl->ws + g.off_partial);
      p.counters = reinterpret_cast<int32_t*>(pl->ws + g.off_counters);
    }
    LaunchFn fn = slab_kernel(d.dtype == SC_BF16 ? kBF16 : kF16, slab.bm, splits > 1);
    if (!fn) return SC_ERR_UNSUPPORTED;
    SC_HIP(fn(p, stream));
    return SC_OK;
  }
  if (staged) {
    ConvParams p;
    std::memset(&p, 0, sizeof(p));
    const StageTile tile = pl->stage_pick[which];
    p.x = x;
    p.wp = pl->ws + g.off_stage_w;
    p.bias = d.has_bias ? bias : nullptr;
    p.y = y;
    p.row_idx = identity ? nullptr : reinterpret_cast<const int32_t*>(pl->ws + g.off_rows);
    p.mask = pl->ws + g.off_mask;
    p.ktab = reinterpret_cast<const KEntry*>(pl->ws + g.off_stage_tab);
    p.zeros = pl->ws + g.off_zeros;
    p.rows = (int32_t)rows;
    p.m_total = (int32_t)g.m;
    p.h = d.h; p.w = d.w; p.ho_wo = g.ho * g.wo; p.wo = g.wo;
    magic_div((uint32_t)p.ho_wo, &p.div_howo_mul, &p.div_howo_shift);
    magic_div((uint32_t)p.wo, &p.div_wo_mul, &p.div_wo_shift);
    p.sh = d.stride_h; p.sw = d.stride_w; p.ph = d.pad_h; p.pw = d.pad_w;
    p.c_in = d.c_in; p.kh = d.kh; p.kw = d.kw; p.dil_h = d.dil_h; p.dil_w = d.dil_w;
    p.c_out = d.c_out;
    p.k_tiles = g.stage_k_tiles;
    p.seg_tail = g.stage_tail;
    if (d.layout == SC_NHWC) {
      p.xs_n = (int64_t)d.h * d.w * d.c_in; p.xs_h = d.w * d.c_in; p.xs_w = d.c_in;
      p.ys_n = (int64_t)p.ho_wo * d.c_out; p.ys_p = d.c_out; p.ys_c = 1;
    } else {
      p.xs_n = (int64_t)d.c_in * d.h * d.w; p.xs_h = d.w; p.xs_w = 1;
      p.ys_n = (int64_t)d.c_out * p.ho_wo; p.ys_p = 1; p.ys_c = p.ho_wo;
    }
    p.x_bytes = (uint32_t)(g.x_elems * eb);
    p.relu = d.relu;
    p.zero_fill = zero_fill ? 1 : 0;
    p.mask_spatial = d.mask_mode == SC_MASK_SPATIAL;
    p.x_compact = compact && x_compact ? 1 : 0;
    p.y_compact = compact && y_compact ? 1 : 0;
    p.residual = residual;
    p.residual_relu = residual && residual_relu ? 1 : 0;
    p.m_tiles = (int32_t)((rows + tile.bm - 1) / tile.bm);
    p.n_tiles = (d.c_out + tile.bn - 1) / tile.bn;
    p.w_bytes = (uint32_t)((uint64_t)g.stage_blocks * g.stage_k_tiles * (d.dtype == SC_F32 ? StageDims<kF32>::BLOCK_BYTES : StageDims<kBF16>::BLOCK_BYTES));
    LaunchFn fn = stage_launcher(d, g, tile);
    if (!fn) return SC_ERR_UNSUPPORTED;      // cannot happen: the pick checked it
    SC_HIP(fn(p, stream));
    return SC_OK;
  }
  TilePick tp = pick_tile(pl, which, rows);
  // every row contracted, the mask looked at only at the store: plain sparse runs of dense operands without a shortcut
  const bool masked = tp.masked && !dense && !identity && !compact && !x_compact && !y_compact && !residual &&
                      d.layout == SC_NHWC && !g.rowseg;
  if (tp.masked && !masked) tp = {tp.ti, 1, false};
  const int ti = tp.ti, splits = masked ? 1 : tp.splits;
  const KernelEntry& ke = pl->table[ti];
  const bool panel = !residual && !masked && use_panel(pl, which, rows);
  ConvParams p;
  std::memset(&p, 0, sizeof(p));
  p.x = x;
  p.wp = pl->ws + g.off_wp;
  p.bias = d.has_bias ? bias : nullptr;
  p.y = y;
  p.row_idx = (identity || masked) ? nullptr : reinterpret_cast<const int32_t*>(pl->ws + g.off_rows);
  p.mask = pl->ws + g.off_mask;
  p.ktab = reinterpret_cast<const KEntry*>(pl->ws + g.off_ktab);
  p.zeros = pl->ws + g.off_zeros;
  p.rows = (int32_t)(masked ? g.m : rows);
  p.masked_store = masked ? (d.out_mode == SC_OUT_ZERO_FILL ? 1 : 2) : 0;
  p.m_total = (int32_t)g.m;
  p.h = d.h; p.w = d.w; p.ho_wo = g.ho * g.wo; p.wo = g.wo;
  magic_div((uint32_t)p.ho_wo, &p.div_howo_mul, &p.div_howo_shift);
  magic_div((uint32_t)p.wo, &p.div_wo_mul, &p.div_wo_shift);
  p.sh = d.stride_h; p.sw = d.stride_w; p.ph = d.pad_h; p.pw = d.pad_w;
  p.c_in = d.c_in; p.kh = d.kh; p.kw = d.kw; p.dil_h = d.dil_h; p.dil_w = d.dil_w;
  p.c_out = d.c_out;
  p.k_pad = g.k_stride; p.k_tiles = g.k_tiles;
  if (d.layout == SC_NHWC) {
    p.xs_n = (int64_t)d.h * d.w * d.c_in; p.xs_h = d.w * d.c_in; p.xs_w = d.c_in;
    p.ys_n = (int64_t)p.ho_wo * d.c_out; p.ys_p = d.c_out; p.ys_c = 1;
  } else {
    p.xs_n = (int64_t)d.c_in * d.h * d.w; p.xs_h = d.w; p.xs_w = 1;
    p.ys_n = (int64_t)d.c_out * p.ho_wo; p.ys_p = 1; p.ys_c = p.ho_wo;
  }
  p.relu = d.relu;
  p.zero_fill = zero_fill && !masked ? 1 : 0;
  p.mask_spatial = d.mask_mode == SC_MASK_SPATIAL;
  p.vec_out = g.vec_out ? 1 : g.vec_out8 ? 2 : 0;
  p.x_compact = compact && x_compact ? 1 : 0;
  p.y_compact = compact && y_compact ? 1 : 0;
  p.residual = residual;
  p.residual_relu = residual_relu ? 1 : 0;
#ifdef SC_TIMING
  p.dbg = g_dbg;
#endif
  p.m_tiles = (int32_t)(((masked ? g.m : rows) + ke.bm - 1) / ke.bm);
  p.n_tiles = (d.c_out + ke.bn - 1) / ke.bn;
  // shallow K (pointwise layers): the workgroup lives for one or two K tiles, so residency, not
  // read-ahead, hides the latency -- take the two-tile ring and fit more workgroups per CU
  LaunchFn fn = !g.vec_gather ? ke.elem
                : (g.vec_out && pl->gather_pipeline != 1) ? (g.k_tiles <= 2 ? ke.dma2 : ke.dma) : ke.vec;
  if (g.rowseg && x_compact) return SC_ERR_UNSUPPORTED;   // the zero-margined copy is built from a dense input
  if (g.rowseg) {
    // small-channel gather: refresh the interior of the zero-margined input copy, then gather window rows
    // from it (no padding in the copy's coordinates: the margins are the padding)
    const int dt = d.dtype == SC_BF16 ? kBF16 : kF16;
    LaunchFn rs = rowseg_kernel(dt, ke.bm, ke.bn);
    if (!rs) return SC_ERR_UNSUPPORTED;
    const int row_elems = d.w * d.c_in, prow_elems = g.wp_cols * d.c_in;
    const int64_t groups = (int64_t)d.n * d.h * (row_elems / 8);
    _Float16* xp = reinterpret_cast<_Float16*>(pl->ws + g.off_xpad);   // 16-bit patterns are moved verbatim
    hipLaunchKernelGGL(pad_input_kernel<_Float16>, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const _Float16*>(x), xp, d.n, d.h, row_elems, g.hp, prow_elems, d.pad_h,
                       d.pad_w * d.c_in);
    SC_HIP(hipGetLastError());
    p.x = xp;
    p.h = g.hp; p.w = g.wp_cols; p.ph = 0; p.pw = 0;
    p.xs_n = (int64_t)g.hp * prow_elems; p.xs_h = prow_elems; p.xs_w = d.c_in;
    p.seg_gpk = g.epad / 8;
    p.seg_gpk_inv = 65536 / p.seg_gpk + 1;   // (g * inv) >> 16 == g / gpk for g < 4096
    p.seg_tail = d.kw * d.c_in - (p.seg_gpk - 1) * 8;
    fn = rs;
  }
  bool fn_is_buf = false;
  if (buf_applies(pl, ke)) {
    const int dt = d.dtype == SC_BF16 ? kBF16 : kF16;
    p.x_bytes = (uint32_t)((uint64_t)d.n * d.h * d.w * d.c_in * eb);
    p.w_bytes = (uint32_t)((uint64_t)g.cout_pad * g.k_stride * eb);
    fn = buf_kernel(dt, ke.bm, ke.bn, g.k_tiles <= 2);
    fn_is_buf = true;
  }
  if (fn_is_buf && splits == 1 && !panel && !masked) {
    const int dt = d.dtype == SC_BF16 ? kBF16 : kF16;
    const int wgs = stream_k_workgroups(pl, ke, rows);
    LaunchFn sk = wgs ? streamk_kernel(dt, ke.bm, ke.bn) : nullptr;
    if (sk) {
      p.stream_wgs = wgs;
      p.partial = reinterpret_cast<float*>(pl->ws + g.off_partial);
      p.counters = reinterpret_cast<int32_t*>(pl->ws + g.off_counters);
      fn = sk;
    }
  }
  if (tp.shares > 0 && fn_is_buf && splits == 1 && !panel && !masked && !p.stream_wgs) {
    fn = buf_groups_kernel(d.dtype == SC_BF16 ? kBF16 : kF16, ke.bm, ke.bn);
    p.splits = tp.shares;
  }
  if (splits > 1) {
    p.splits = splits;
    p.partial = reinterpret_cast<float*>(pl->ws + g.off_partial);
    p.counters = reinterpret_cast<int32_t*>(pl->ws + g.off_counters);
    fn = splitk_launcher(pl, ke);
  }
  if (panel) {
    p.m_tiles = (int32_t)((rows + kPanelBM - 1) / kPanelBM);
    p.n_tiles = (d.c_out + kPanelBN - 1) / kPanelBN;
    fn = pl->panel;
  }
  SC_HIP(fn(p, stream));
  return SC_OK;
}

static sc_status check_run_args(const sc_plan* plan, const void* x, const float* bias, void* y) {
  if (!plan || !x || !y) return SC_ERR_NULL;
  if (plan->desc.has_bias && !bias) return SC_ERR_NULL;
  if (((uintptr_t)x & 15) || ((uintptr_t)y & 15) || (plan->desc.has_bias && ((uintptr_t)bias & 15)))
    return SC_ERR_ALIGN;
  return SC_OK;
}

// Everything of a plan that depends on the filters: the packed filter matrix (and, once, the gather table).  copies: of the filters of a
// layer that the window kernel may run, those in rows (of the other kernels), in fragment order, or both.
enum { kRowCopy = 1, kWindowCopy = 2, kBothCopies = 3 };
static sc_status pack_filters(const sc_conv_desc& d, const Geometry& g, unsigned char* ws, const void* w_dev, bool tables,
                              bool rotated, hipStream_t stream, int copies = kBothCopies) {
  if (g.depthwise) {
    const int dt = d.dtype == SC_BF16 ? kBF16 : d.dtype == SC_F16 ? kF16 : kF32;
    SC_HIP(depthwise_pack(dt, w_dev, ws + g.off_wp, d.c_in, d.kh * d.kw, stream));
    return SC_OK;
  }
  const int dt = d.dtype == SC_BF16 ? kBF16 : d.dtype == SC_F16 ? kF16 : kF32;
  // Whole 16-byte groups: one launch, which leaves out the rows of padding channels once they hold zeros (us per refresh of
  // 64 x 3 x 3 x 64 in float: 4.7 + 4.7 element by element in two launches; with the rotation in front of it 4.6 more).
  const bool by_groups = g.vec_gather && !g.rowseg && d.layout == SC_NHWC && (int64_t)g.cout_pad * g.k_stride < ((int64_t)1 << 31);
  if (rotated && !by_groups) return SC_ERR_UNSUPPORTED;      // (the caller rotates by itself)
  if (by_groups) {
    const bool parts = g.stage_gather == kStageGroups;
    const int blocks32 = (d.c_out + 31) / 32;
    const int rows = !(copies & kRowCopy) ? 0 : tables ? g.cout_pad : blocks32 * 32;
    SC_HIP(repack_filters(dt, w_dev, ws + g.off_wp, parts ? ws + g.off_stage_w : g.window && (copies & kWindowCopy) ? ws + g.off_window_w : nullptr,
                          d.c_out, d.c_in, d.kh * d.kw, g.k_stride, rows, tables && parts ? g.stage_blocks : blocks32,
                          parts ? g.stage_k_tiles : (d.c_in + kWinChunk - 1) / kWinChunk, rotated, stream));
  } else {
    int64_t total = (int64_t)g.cout_pad * g.k_stride;
    int grid = (int)((total + 255) / 256);
    const int nchw = d.layout == SC_NCHW;
    if (d.dtype == SC_F32)
      hipLaunchKernelGGL(pack_filters_kernel<float>, dim3(grid), dim3(256), 0, stream, (const float*)w_dev,
                         (float*)(ws + g.off_wp), d.c_out, d.c_in, d.kh, d.kw, g.k, g.k_stride, g.cout_pad, nchw, g.rowseg ? g.epad : 0);
    else  // 16-bit patterns are moved verbatim
      hipLaunchKernelGGL(pack_filters_kernel<_Float16>, dim3(grid), dim3(256), 0, stream, (const _Float16*)w_dev,
                         (_Float16*)(ws + g.off_wp), d.c_out, d.c_in, d.kh, d.kw, g.k, g.k_stride, g.cout_pad, nchw, g.rowseg ? g.epad : 0);
    SC_HIP(hipGetLastError());
  }
  if (g.stage_gather >= 0 && (tables || !by_groups)) {
    SC_HIP(stage_pack(dt, g.stage_gather, by_groups ? nullptr : w_dev, ws + g.off_stage_w, tables ? reinterpret_cast<KEntry*>(ws + g.off_stage_tab) : nullptr,
                      d.c_out, g.stage_blocks, d.c_in, d.kh, d.kw, d.dil_h, d.dil_w, g.stage_k_tiles, d.layout == SC_NCHW, d.h, d.w, stream));
  }
  // gather table (depends on the geometry only)
  if (tables) {
    const int vec = g.vec_gather ? g.vec : 1;
    const int entries = g.k_pad / vec;
    int xs_h, xs_w, xs_c;
    if (d.layout == SC_NHWC) { xs_h = d.w * d.c_in; xs_w = d.c_in; xs_c = 1; }
    else { xs_h = d.w; xs_w = 1; xs_c = d.h * d.w; }
    hipLaunchKernelGGL(build_ktab_kernel, dim3((entries + 255) / 256), dim3(256), 0, stream,
                       reinterpret_cast<KEntry*>(ws + g.off_ktab), entries, vec, g.k, d.c_in, d.kw, d.dil_h, d.dil_w,
                       xs_h, xs_w, xs_c);
    SC_HIP(hipGetLastError());
  }
  return SC_OK;
}

// Everything of a plan that depends on the mask (Alg. 2, indirection init): the private mask copy, the
// ascending list of kept rows and its length, the band tables, the rank table of depthwise layers.
// Synchronises the stream (the kept count decides the launch shapes) and checks the count against the
// descriptor's sparsity.
static sc_status build_row_tables(const sc_conv_desc& d, const Geometry& g, unsigned char* ws, const uint8_t* mask_dev,
                                  hipStream_t stream, BandPlan* bp_io, int32_t* kept_out, int32_t* slab_span_out) {
  BandPlan& bp = *bp_io;
  const int period = d.mask_mode == SC_MASK_SPATIAL ? g.ho * g.wo : 0;
  int32_t* counts = reinterpret_cast<int32_t*>(ws + g.off_counts);
  int32_t* rows = reinterpret_cast<int32_t*>(ws + g.off_rows);
  int32_t* kept_dev = reinterpret_cast<int32_t*>(ws + g.off_kept);
  int32_t host_vals[5] = {-1, 0, 0, 0, 0};   // kept count, most kept rows in one band, widest slab of a 64-row / 128-row / 256-row tile
  // (where a band kernel stays, tuning asks for the spans itself: two of 24 us of a refresh of a small map, of 58 past 2^17 rows nine)
  const bool slab = slab_geometry_ok(d, g) || (g.window && (!band_stays(d, bp) || std::getenv("SPARSE_CONV_WINDOW_TILE")));
  // One launch up to 2^17 rows (where a run of rows cut in two leaves both halves a pixel); beyond that every workgroup's
  // count of the rows in front of it costs more than a pass of its own.  Measured per refresh on a
  // 56 x 56 map of one image, us of GPU time: 13 in five launches and a copy, 5 in one.
  if (g.m <= kTableMostRows && !(bp.ok && bp.split && g.wo == 1)) {
    TableParams p;
    std::memset(&p, 0, sizeof(p));
    const int wgs = (int)((g.m + kTableRows - 1) / kTableRows);
    p.mask = mask_dev;
    p.copy = ws + g.off_mask;
    p.row_idx = rows;
    p.kept_out = kept_dev;
    p.band_i0 = reinterpret_cast<int32_t*>(ws + g.off_band);
    p.band_rows = reinterpret_cast<int32_t*>(ws + g.off_band_rows);
    p.m = (int32_t)g.m; p.period = period; p.mask_len = (int32_t)g.mask_len;
    p.ho = g.ho; p.wo = g.wo; p.bh = 1;
    if (bp.ok) { p.n_bands = bp.n_bands; p.bands_per_image = bp.bands_per_image; p.bh = bp.bh; p.split = bp.split; }
    if (slab) { p.slab_hp = d.h + 2 * d.pad_h; p.slab_kh = d.kh; }
    magic_div((uint32_t)(g.ho * g.wo), &p.howo_mul, &p.howo_shift);
    magic_div((uint32_t)g.wo, &p.wo_mul, &p.wo_shift);
    magic_div((uint32_t)p.bh, &p.bh_mul, &p.bh_shift);
    int32_t* slot = g_host_slots.take(stream);
    p.result = slot ? slot : counts;
    int32_t copied[kHostSlotWords];
    const sc_status s = [&]() -> sc_status {
      hipLaunchKernelGGL(row_tables_kernel, dim3(wgs), dim3(kTableThreads), 0, stream, p);
      SC_HIP(hipGetLastError());
      if (g.depthwise)
        SC_HIP(depthwise_rank(rows, kept_dev, reinterpret_cast<int32_t*>(ws + g.off_band_rows), g.m, stream));
      if (!slot) SC_HIP(hipMemcpyAsync(copied, counts, sizeof(int32_t) * kTableWords * wgs, hipMemcpyDeviceToHost, stream));
      SC_HIP(hipStreamSynchronize(stream));
      return SC_OK;
    }();
    if (s != SC_OK) {
      // (a launch may still be on its way to the slot: it stays taken)
      return s;
    }
    const int32_t* res = slot ? slot : copied;
    int kept = 0, fullest = 0;
    for (int i = 0; i < wgs; ++i) {
      kept += res[kTableWords * i + kTableKept];
      fullest = std::max(fullest, (int)res[kTableWords * i + kTableFullest]);
    }
    int32_t span[3] = {0, 0, 0};
    if (slab) table_spans(res, wgs, d.kh, span);
    for (int b = 0; b < 3; ++b) host_vals[2 + b] = span[b];
    if (slot) g_host_slots.give_back(slot);
    host_vals[0] = kept;
    host_vals[1] = fullest;
  } else {
    const int cgrid = (g.nseg + 3) / 4;
    // pass 1 also leaves the plan's private copy of the mask (the zero fill of every run reads it)
    hipLaunchKernelGGL(mask_count_kernel, dim3(cgrid), dim3(256), 0, stream, mask_dev, (int)g.m, period,
                       g.nseg, counts, ws + g.off_mask, (int)g.mask_len);
    SC_HIP(hipGetLastError());
    hipLaunchKernelGGL(mask_scatter_kernel, dim3(cgrid), dim3(256), 0, stream, ws + g.off_mask, (int)g.m, period,
                       g.nseg, counts, rows, kept_dev);
    SC_HIP(hipGetLastError());
    if (g.depthwise)   // position of every kept row in the row list (compact output of the LDS-tiled kernels)
      SC_HIP(depthwise_rank(rows, kept_dev, reinterpret_cast<int32_t*>(ws + g.off_band_rows), g.m, stream));

    if (bp.ok) {
      hipLaunchKernelGGL(band_start_kernel, dim3((bp.n_bands + 1 + 255) / 256), dim3(256), 0, stream, rows, kept_dev,
                         reinterpret_cast<int32_t*>(ws + g.off_band), bp.n_bands, bp.bands_per_image, bp.bh, bp.split, g.ho, g.wo);
      SC_HIP(hipGetLastError());
      // kept_dev + 1 holds the per-band maximum (zeroed by the scatter pass, raised by band_rows_kernel)
      hipLaunchKernelGGL(band_rows_kernel, dim3((unsigned)((g.m + 255) / 256)), dim3(256), 0, stream, rows, kept_dev,
                         reinterpret_cast<const int32_t*>(ws + g.off_band),
                         reinterpret_cast<int32_t*>(ws + g.off_band_rows), bp.bands_per_image, bp.bh, bp.split, g.ho, g.wo,
                         kept_dev + 1);
      SC_HIP(hipGetLastError());
    }

    if (slab) {
      hipLaunchKernelGGL(slab_span_kernel, dim3((unsigned)((g.m + 63) / 64 + 255) / 256), dim3(256), 0, stream, rows, kept_dev,
                         g.ho * g.wo, g.wo, d.h + 2 * d.pad_h, d.kh, kept_dev + 2);
      SC_HIP(hipGetLastError());
    }

    SC_HIP(hipMemcpyAsync(host_vals, kept_dev, sizeof(host_vals), hipMemcpyDeviceToHost, stream));
    SC_HIP(hipStreamSynchronize(stream));
  }
  *kept_out = host_vals[0];
  bp.max_kept = host_vals[1];
  for (int b = 0; b < 3; ++b) slab_span_out[b] = host_vals[2 + b];

  if (d.sparsity >= 0.0f) {
    // Sec. 3.2: rows in the GEMM = output_size - sparsity * output_size (rounded half up).  The descriptor carries
    // the ratio as a float: where the product falls on a half within that float's rounding interval (0.9 of 135
    // rows), either neighbour is the count the caller's own ratio demands, and both are accepted.
    const double sp = (double)d.sparsity, eps = std::ldexp(std::fabs(sp), -24) + 1e-12;
    const int64_t want_hi = (int64_t)std::floor((1.0 - (sp - eps)) * (double)g.mask_len + 0.5);
    const int64_t want_lo = (int64_t)std::floor((1.0 - (sp + eps)) * (double)g.mask_len + 0.5);
    int64_t have = d.mask_mode == SC_MASK_ROW ? host_vals[0] : host_vals[0] / d.n;
    if (have < want_lo || have > want_hi) return SC_ERR_MASK_COUNT;
  }
  return SC_OK;
}

}  // namespace sc

extern "C" {

sc_status sparse_conv_output_shape(const sc_conv_desc* desc, int32_t* ho, int32_t* wo, int64_t* m) {
  Geometry g;
  sc_status s = check_desc(desc, &g);
  if (s != SC_OK) return s;
  if (ho) *ho = g.ho;
  if (wo) *wo = g.wo;
  if (m) *m = g.m;
  return SC_OK;
}

sc_status sparse_conv_workspace_bytes(const sc_conv_desc* desc, size_t* bytes) {
  if (!bytes) return SC_ERR_NULL;
  Geometry g;
  sc_status s = check_desc(desc, &g);
  if (s != SC_OK) return s;
  *bytes = g.total;
  return SC_OK;
}

sc_status sparse_conv_plan(const sc_conv_desc* desc, const uint8_t* mask_dev, const void* w_dev,
                           void* workspace_dev, size_t workspace_bytes, void* hip_stream, sc_plan** out) {
  if (!out) return SC_ERR_NULL;
  *out = nullptr;
  Geometry g;
  sc_status s = check_desc(desc, &g);
  if (s != SC_OK) return s;
  if (!mask_dev || !w_dev || !workspace_dev) return SC_ERR_NULL;
  if (workspace_bytes < g.total) return SC_ERR_WORKSPACE;
  if (((uintptr_t)workspace_dev & 255) || ((uintptr_t)w_dev & 15)) return SC_ERR_ALIGN;

  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace_dev);
  const sc_conv_desc& d = *desc;
  const int eb = elem_bytes(d.dtype);

  SC_HIP(hipMemsetAsync(ws + g.off_zeros, 0, 256, stream));
  if (g.rowseg)      // margins of the padded input copy stay zero; every run rewrites the interior
    SC_HIP(hipMemsetAsync(ws + g.off_xpad, 0, ((size_t)d.n * g.hp * g.wp_cols * d.c_in + 64) * eb, stream));
  if (g.splitk_ok)   // arrival counters start at zero; every launch leaves them at zero again
    SC_HIP(hipMemsetAsync(ws + g.off_counters, 0, g.off_partial - g.off_counters, stream));
  // (the kept-row count is not known yet: the descriptor's sparsity says what to expect, half the rows if it is silent)
  const int64_t rows_hint = d.sparsity >= 0.0f ? (int64_t)((1.0 - (double)d.sparsity) * (double)g.m + 0.5) : g.m / 2;
  BandPlan bp = plan_band(d, g, rows_hint);
  int32_t kept_host = 0;
  s = pack_filters(d, g, ws, w_dev, true, false, stream);
  if (s != SC_OK) return s;
  int32_t slab_span[3] = {0, 0, 0};
  s = build_row_tables(d, g, ws, mask_dev, stream, &bp, &kept_host, slab_span);   // synchronises the stream
  if (s != SC_OK) return s;

  sc_plan* pl = new (std::nothrow) sc_plan;
  if (!pl) return SC_ERR_NULL;
  pl->desc = d;
  pl->geo = g;
  pl->ws = ws;
  pl->kept = kept_host;
  pl->table = d.dtype == SC_BF16 ? kernels_bf16(&pl->table_count)
              : d.dtype == SC_F16 ? kernels_f16(&pl->table_count)
                                  : kernels_f32(&pl->table_count);
  pl->forced[0] = pl->forced[1] = -1;
  pl->prefer_tiled[0] = pl->prefer_tiled[1] = false;
  pl->tuned = false;
  const char* depthwise_kernel = std::getenv("SPARSE_CONV_DEPTHWISE_KERNEL");
  pl->depthwise_kernel = !depthwise_kernel ? 0 : std::strcmp(depthwise_kernel, "staged") == 0 ? 1 : std::strcmp(depthwise_kernel, "walk") == 0 ? 2 : 0;
  pl->gather_pipeline = 0;
  pl->split_k = 0;
  pl->row_panel = 0;
  pl->stream_k = 0;
  pl->masked_store = 0;
  pl->x_rank_set = false;
  pl->tile_splitk = -1;
  for (int i = 0; i < pl->table_count; ++i)
    if (pl->table[i].splitk && pl->table[i].bm == 64 && pl->table[i].bn == 128) pl->tile_splitk = i;
  if (pl->tile_splitk < 0) pl->geo.splitk_ok = false;
  pl->pick[0] = model_pick(pl, 0, pl->kept);
  pl->pick[1] = model_pick(pl, 1, g.m);
  pl->band = bp;
  pl->band_dense = plan_band(d, g, g.m);
  pl->stage_tuned = 0;
  stage_tiles_for(d, g, pl->kept, pl->stage_pick);
  pl->slab = 0;
  pl->slab_ok = slab_geometry_ok(d, g) && slab_kernel(d.dtype == SC_BF16 ? kBF16 : kF16, 128, false);
  for (int b = 0; b < 3; ++b) {
    pl->slab_span[0][b] = slab_span[b];
    pl->slab_span[1][b] = pl->slab_ok || g.window ? slab_dense_span(d, g, 64 << b) : 0;
  }
  pl->window[0] = window_tile_for(pl, 0);
  pl->window[1] = window_tile_for(pl, 1);
  // (automatic launches take the slab form only where sparse_conv_plan_tune measured it faster: the cost model's
  // quantities -- bytes through the L1 path, matrix time -- do not rank it, its K loop is bound by LDS reads)
  pl->slab_auto[0] = pl->slab_auto[1] = sc_plan::Slab{0, 1};
  pl->band_table = d.dtype == SC_BF16 ? band_bf16() : d.dtype == SC_F16 ? band_f16() : band_f32();
  pl->stream_table = d.dtype == SC_BF16 ? bandstream_bf16() : d.dtype == SC_F16 ? bandstream_f16() : nullptr;
  pl->pp_table = d.dtype == SC_BF16 ? bandpp_bf16() : d.dtype == SC_F16 ? bandpp_f16() : nullptr;
  pl->tap_table = d.dtype == SC_BF16 ? bandtap_bf16() : d.dtype == SC_F16 ? bandtap_f16() : nullptr;
  pl->panel = d.dtype == SC_BF16 ? panel_bf16() : d.dtype == SC_F16 ? panel_f16() : nullptr;
  (void)eb;
  *out = pl;
  return SC_OK;
}

sc_status sparse_conv_plan_set_mask(sc_plan* plan, const uint8_t* mask_dev, void* hip_stream) {
  if (!plan || !mask_dev) return SC_ERR_NULL;
  const sc_conv_desc& d = plan->desc;
  const Geometry& g = plan->geo;
  BandPlan bp = plan->band;
  int32_t kept_host = 0;
  int32_t slab_span[3] = {0, 0, 0};
  sc_status s = build_row_tables(d, g, plan->ws, mask_dev, static_cast<hipStream_t>(hip_stream), &bp, &kept_host, slab_span);
  if (s != SC_OK) return s;
  plan->kept = kept_host;
  plan->band = bp;
  plan->pick[0] = model_pick(plan, 0, plan->kept);      // (a measured choice belonged to the previous mask's row count)
  plan->prefer_tiled[0] = false;
  if (plan->stage_tuned) plan->prefer_tiled[1] = false;      // (both runs were chosen together)
  plan->stage_tuned = 0;
  stage_tiles_for(d, g, plan->kept, plan->stage_pick);
  for (int b = 0; b < 3; ++b) plan->slab_span[0][b] = slab_span[b];
  plan->slab_auto[0] = sc_plan::Slab{0, 1};
  plan->window[0] = window_tile_for(plan, 0);
  return SC_OK;
}

sc_status sparse_conv_plan_set_input_mask(sc_plan* plan, const uint8_t* mask_in_dev, int64_t* kept_in,
                                          void* hip_stream) {
  if (!plan || !mask_in_dev) return SC_ERR_NULL;
  const sc_conv_desc& d = plan->desc;
  const Geometry& g = plan->geo;
  if (!g.depthwise || d.kh * d.kw == 1) return SC_ERR_UNSUPPORTED;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const int64_t pixels = (int64_t)d.n * d.h * d.w;
  if (pixels >= ((int64_t)1 << 31)) return SC_ERR_BAD_SHAPE;
  const int period = d.mask_mode == SC_MASK_SPATIAL ? d.h * d.w : 0;
  const int nseg = (int)((pixels + kSeg - 1) / kSeg);
  int32_t* counts = reinterpret_cast<int32_t*>(plan->ws + g.off_xcounts);
  int32_t* kept_dev = counts + nseg;
  const int cgrid = (nseg + 3) / 4;
  hipLaunchKernelGGL(mask_count_kernel, dim3(cgrid), dim3(256), 0, stream, mask_in_dev, (int)pixels, period, nseg, counts, nullptr, 0);
  SC_HIP(hipGetLastError());
  hipLaunchKernelGGL(mask_rank_kernel, dim3(cgrid), dim3(256), 0, stream, mask_in_dev, (int)pixels, period, nseg, counts,
                     reinterpret_cast<int32_t*>(plan->ws + g.off_xrank), kept_dev);
  SC_HIP(hipGetLastError());
  int32_t kept_host = 0;
  SC_HIP(hipMemcpyAsync(&kept_host, kept_dev, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
  SC_HIP(hipStreamSynchronize(stream));
  plan->x_rank_set = true;
  if (kept_in) *kept_in = kept_host;
  return SC_OK;
}

sc_status sparse_conv_plan_set_filters(sc_plan* plan, const void* w_dev, void* hip_stream) {
  if (!plan || !w_dev) return SC_ERR_NULL;
  if ((uintptr_t)w_dev & 15) return SC_ERR_ALIGN;
  return pack_filters(plan->desc, plan->geo, plan->ws, w_dev, false, false, static_cast<hipStream_t>(hip_stream));
}

// (of the backward pass: a plan of the input gradient, from the filters of the layer itself.  Its only runs are plain dense ones, of a kernel
// that is chosen once, so the copy that this kernel does not read is left out: us a training step of 512 -> 512 @7, batch 16 73.2 / 71.8, 64 91.7 / 89.2)
__attribute__((visibility("hidden"))) sc_status sc_plan_set_rotated_filters(sc_plan* plan, const void* w_dev, void* hip_stream) {
  const int copies = !plan->geo.window ? kBothCopies : use_window(plan, 1, plan->geo.m) ? kWindowCopy : kRowCopy;
  return pack_filters(plan->desc, plan->geo, plan->ws, w_dev, false, true, static_cast<hipStream_t>(hip_stream), copies);
}

sc_status sparse_conv_run(const sc_plan* plan, const void* x_dev, const float* bias_dev, void* y_dev,
                          void* hip_stream) {
  sc_status s = check_run_args(plan, x_dev, bias_dev, y_dev);
  if (s != SC_OK) return s;
  return launch_conv(plan, false, x_dev, bias_dev, y_dev, static_cast<hipStream_t>(hip_stream));
}

sc_status sparse_conv_run_rows(const sc_plan* plan, const void* x_dev, int32_t x_rows, const float* bias_dev,
                               void* y_dev, int32_t y_rows, void* hip_stream) {
  sc_status s = check_run_args(plan, x_dev, bias_dev, y_dev);
  if (s != SC_OK) return s;
  if ((x_rows != SC_ROWS_DENSE && x_rows != SC_ROWS_COMPACT) || (y_rows != SC_ROWS_DENSE && y_rows != SC_ROWS_COMPACT))
    return SC_ERR_UNSUPPORTED;
  const sc_conv_desc& d = plan->desc;
  const bool xc = x_rows == SC_ROWS_COMPACT, yc = y_rows == SC_ROWS_COMPACT;
  if ((xc || yc) && d.layout != SC_NHWC) return SC_ERR_UNSUPPORTED;
  const bool pixel_window = d.kh == 1 && d.kw == 1 && d.stride_h == 1 && d.stride_w == 1 && d.pad_h == 0 && d.pad_w == 0;
  // a window that is the pixel itself never reads a dropped pixel; a depthwise layer with larger windows looks
  // every pixel up in the rank map of its input
  if (xc && !pixel_window && !(plan->geo.depthwise && plan->x_rank_set)) return SC_ERR_UNSUPPORTED;
  return launch_conv(plan, false, x_dev, bias_dev, y_dev, static_cast<hipStream_t>(hip_stream), xc, yc);
}

sc_status sparse_conv_run_residual(const sc_plan* plan, const void* x_dev, int32_t x_rows, const float* bias_dev,
                                   const void* residual_dev, int32_t residual_relu, void* y_dev, int32_t y_rows,
                                   void* hip_stream) {
  sc_status s = check_run_args(plan, x_dev, bias_dev, y_dev);
  if (s != SC_OK) return s;
  if (!residual_dev) return SC_ERR_NULL;
  if ((uintptr_t)residual_dev & 15) return SC_ERR_ALIGN;
  if ((x_rows != SC_ROWS_DENSE && x_rows != SC_ROWS_COMPACT) || (y_rows != SC_ROWS_DENSE && y_rows != SC_ROWS_COMPACT))
    return SC_ERR_UNSUPPORTED;
  const sc_conv_desc& d = plan->desc;
  const bool xc = x_rows == SC_ROWS_COMPACT, yc = y_rows == SC_ROWS_COMPACT;
  if ((xc || yc) && d.layout != SC_NHWC) return SC_ERR_UNSUPPORTED;
  const bool pixel_window = d.kh == 1 && d.kw == 1 && d.stride_h == 1 && d.stride_w == 1 && d.pad_h == 0 && d.pad_w == 0;
  if (plan->geo.depthwise || (xc && !pixel_window)) return SC_ERR_UNSUPPORTED;
  return launch_conv(plan, false, x_dev, bias_dev, y_dev, static_cast<hipStream_t>(hip_stream), xc, yc, residual_dev,
                     residual_relu);
}

sc_status dense_conv_run_residual(const sc_plan* plan, const void* x_dev, const float* bias_dev,
                                  const void* residual_dev, int32_t residual_relu, void* y_dev, void* hip_stream) {
  sc_status s = check_run_args(plan, x_dev, bias_dev, y_dev);
  if (s != SC_OK) return s;
  if (!residual_dev) return SC_ERR_NULL;
  if ((uintptr_t)residual_dev & 15) return SC_ERR_ALIGN;
  if (plan->geo.depthwise) return SC_ERR_UNSUPPORTED;
  return launch_conv(plan, true, x_dev, bias_dev, y_dev, static_cast<hipStream_t>(hip_stream), false, false,
                     residual_dev, residual_relu);
}

sc_status dense_conv_run(const sc_plan* plan, const void* x_dev, const float* bias_dev, void* y_dev,
                         void* hip_stream) {
  sc_status s = check_run_args(plan, x_dev, bias_dev, y_dev);
  if (s != SC_OK) return s;
  return launch_conv(plan, true, x_dev, bias_dev, y_dev, static_cast<hipStream_t>(hip_stream));
}

sc_status sparse_conv_plan_tune(sc_plan* plan, const void* x_dev, const float* bias_dev, void* y_dev, void* hip_stream) {
  sc_status st = check_run_args(plan, x_dev, bias_dev, y_dev);
  if (st != SC_OK) return st;
  if (plan->geo.depthwise) return SC_OK;       // one kernel per window shape: nothing to choose
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  SC_HIP(hipStreamSynchronize(stream));
  // Candidates are timed as graphs of back-to-back launches on a stream of the library's own: launched one by one
  // from the host, layers of a few microseconds would all measure the host's launch rate.
  hipStream_t ts = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  SC_HIP(hipStreamCreateWithFlags(&ts, hipStreamNonBlocking));
  if (hip_failed(hipEventCreate(&e0))) { (void)hipStreamDestroy(ts); return SC_ERR_HIP; }
  if (hip_failed(hipEventCreate(&e1))) { (void)hipEventDestroy(e0); (void)hipStreamDestroy(ts); return SC_ERR_HIP; }
  // microseconds per launch of the run as the plan stands (negative: something failed)
  auto time_us = [&](bool dense, int launches, int replays) -> double {
    if (launch_conv(plan, dense, x_dev, bias_dev, y_dev, ts) != SC_OK) return -1.0;     // also sets kernel attributes
    if (hipStreamBeginCapture(ts, hipStreamCaptureModeThreadLocal) != hipSuccess) return -1.0;
    bool ok = true;
    for (int i = 0; i < launches && ok; ++i) ok = launch_conv(plan, dense, x_dev, bias_dev, y_dev, ts) == SC_OK;
    hipGraph_t graph = nullptr;
    if (hipStreamEndCapture(ts, &graph) != hipSuccess || !ok || !graph) {
      if (graph) (void)hipGraphDestroy(graph);
      (void)hipGetLastError();
      return -1.0;
    }
    hipGraphExec_t exec = nullptr;
    double best = -1.0;
    if (hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) == hipSuccess) {
      for (int rep = 0; rep <= replays; ++rep) {       // replay 0 warms up
        float ms = 0.0f;
        if (hipEventRecord(e0, ts) != hipSuccess || hipGraphLaunch(exec, ts) != hipSuccess ||
            hipEventRecord(e1, ts) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { best = -1.0; break; }
        const double us = (double)ms * 1e3 / launches;
        if (rep > 0 && (best < 0.0 || us < best)) best = us;
      }
      (void)hipGraphExecDestroy(exec);
    }
    (void)hipGraphDestroy(graph);
    return best;
  };
  sc_status result = SC_OK;
  // every tile x split (and the masked-store variant) of the tiled kernels that the model prices within 1.6 x of its best:
  // the first that beats best_us by 1.5 % and all after it that beat the last
  auto try_tiled = [&](int which, sc_plan::Pick* best_pick, double* best_us) -> bool {
    const bool dense = which == 1;
    const int64_t rows = dense ? plan->geo.m : plan->kept;
    struct Cand { sc_plan::Pick pick; double predicted; };
    Cand cands[128];
    int n = 0;
    double best_pred = 1e300;
    const bool can_mask = which == 0 && rows < plan->geo.m;
    for (int i = 0; i < plan->table_count && n < 120; ++i) {
      const KernelEntry& ke = plan->table[i];
      if (tile_lds_bytes(plan, ke) > kLdsLimit) continue;
      const int most = split_candidates(plan, ke, rows);
      for (int sp = 1; sp <= most; ++sp) {
        cands[n] = {{i, sp, false}, predict_us(plan, ke, rows, sp, which == 0 && rows < plan->geo.m)};
        best_pred = std::min(best_pred, cands[n++].predicted);
      }
      if (most >= 2 && group_candidates(plan, ke, rows) > 1) {
        cands[n] = {{i, 2, false, i}, predict_us(plan, ke, rows, 1, which == 0 && rows < plan->geo.m, 2)};
        best_pred = std::min(best_pred, cands[n++].predicted);
      }
      if (can_mask && plan->masked_store != 1) {
        cands[n] = {{i, 1, true}, predict_us(plan, ke, plan->geo.m, 1, false) + 0.1};
        best_pred = std::min(best_pred, cands[n++].predicted);
      }
    }
    bool found = false;
    for (int c = 0; c < n; ++c) {
      if (cands[c].predicted > 1.6 * best_pred) continue;
      plan->pick[which] = cands[c].pick;
      plan->prefer_tiled[which] = true;
      const double us = time_us(dense, 40, 3);
      if (us > 0.0 && us < 0.985 * *best_us) { *best_us = us; *best_pick = cands[c].pick; found = true; }
    }
    return found;
  };
  // Layers of the staged kernel: its tiles and shares of K, the band kernel and the tiled ones.  The sparse run decides (where
  // no row is kept the dense one), and the other run takes the fastest form of the same kernel with the same shares, so that
  // both go on adding a row's products in one order.
  const int lead = plan->kept > 0 ? 0 : 1;
  const bool staged = plan->stage_pick[lead].bm > 0 && !plan->stage_pick[lead].asked && plan->forced[0] == -1 && plan->forced[1] == -1 &&
                      (plan->gather_pipeline == 0 || !plan->geo.vec_gather) && plan->masked_store != 2;
  if (staged) {
    const sc_conv_desc& d = plan->desc;
    plan->prefer_tiled[0] = plan->prefer_tiled[1] = false;
    plan->stage_tuned = 0;
    for (int which = 0; which < 2; ++which) plan->pick[which] = model_pick(plan, which, which ? plan->geo.m : plan->kept);
    const bool band_first = !use_stage(plan, lead);
    auto try_staged = [&](int which, int groups, StageTile* best, double* best_us) {
      for (const int bm : {64, 128})
        for (const int bn : {32, 64, 128}) {
          const StageTile t = {bm, bn, groups, false};
          if ((bn > 32 && d.c_out <= bn / 2) || !stage_launcher(d, plan->geo, t)) continue;
          plan->stage_pick[which] = t;
          double us = time_us(which == 1, 10, 1);      // (a look first: what takes 1.6 x as long is no serious candidate)
          if (us > 1.6 * *best_us) continue;
          us = time_us(which == 1, 40, 3);
          if (us > 0.0 && us < *best_us) { *best_us = us; *best = t; }
        }
    };
    if (time_us(lead == 1, 100, 4) < 0.0) result = SC_ERR_HIP;                // clocks up before anything is compared
    plan->stage_tuned = 1;
    StageTile tile = plan->stage_pick[lead];
    double staged_us = result == SC_OK ? time_us(lead == 1, 40, 3) : -1.0;
    if (staged_us < 0.0) result = SC_ERR_HIP;
    for (int groups = 1; groups <= 4 && result == SC_OK; groups *= 2) try_staged(lead, groups, &tile, &staged_us);
    plan->stage_pick[lead] = tile;
    if (lead == 0) plan->stage_pick[1] = stage_tile_for(d, plan->geo, plan->geo.m, tile.groups);
    double best_us = staged_us;
    if (result == SC_OK && plan->geo.vec_gather) {
      const bool bands = plan->band.ok && !plan->band.stream && plan->band_dense.ok && !plan->band_dense.stream;
      plan->stage_tuned = -1;
      const double band_us = bands ? time_us(lead == 1, 40, 3) : -1.0;
      bool band_wins = band_us > 0.0 && band_us < (band_first ? best_us / 0.985 : 0.985 * best_us);
      if (band_wins) best_us = band_us;
      sc_plan::Pick pick[2] = {plan->pick[0], plan->pick[1]};
      const bool tiled_wins = try_tiled(lead, &pick[lead], &best_us);
      plan->pick[lead] = pick[lead];
      plan->prefer_tiled[lead] = tiled_wins;
      plan->stage_tuned = tiled_wins || band_wins ? -1 : 1;
      if (tiled_wins && lead == 0) {
        double us = 1e300;
        (void)try_tiled(1, &pick[1], &us);
        plan->pick[1] = pick[1];
        plan->prefer_tiled[1] = true;
      }
    }
    if (result == SC_OK && lead == 0 && plan->stage_tuned > 0) {
      StageTile other = plan->stage_pick[1];
      double us = time_us(true, 40, 3);
      if (us < 0.0) result = SC_ERR_HIP;
      else try_staged(1, tile.groups, &other, &us);
      plan->stage_pick[1] = other;
    }
  }
  for (int which = 0; which < 2 && result == SC_OK && !staged; ++which) {
    const bool dense = which == 1;
    const int64_t rows = dense ? plan->geo.m : plan->kept;
    if (plan->forced[which] != -1 || rows == 0) continue;
    plan->pick[which] = model_pick(plan, which, rows);
    plan->prefer_tiled[which] = false;
    plan->slab_auto[which] = sc_plan::Slab{0, 1};
    plan->window[which] = window_tile_for(plan, which);
    if (time_us(dense, 100, 4) < 0.0) { result = SC_ERR_HIP; break; }     // clocks up before anything is compared
    sc_plan::Pick best_pick = plan->pick[which];
    bool best_tiled = false;
    double best_us = time_us(dense, 40, 3);
    if (best_us < 0.0) { result = SC_ERR_HIP; break; }
    if (!plan->geo.vec_gather || plan->geo.rowseg) {                   // one tile shape serves these gathers
      const BandPlan& rb = dense ? plan->band_dense : plan->band;
      if (rb.ok && rb.rowband) {                                       // band kernel of the small-channel layers or that tile
        plan->prefer_tiled[which] = true;
        const double us = time_us(dense, 40, 3);
        if (!(us > 0.0 && us < 0.985 * best_us)) plan->prefer_tiled[which] = false;
      }
      continue;
    }
    // the band kernel, where it had given way, and every tile of the window kernel
    const BandPlan& bsel = dense ? plan->band_dense : plan->band;
    const bool band_applies = bsel.ok && !bsel.stream;
    if (plan->geo.window && !plan->window[which].asked && window_is_free(plan, which, rows)) {
      if (which == 0 && plan->slab_span[0][0] == 0) {      // (the row tables left the spans out)
        const Geometry& g = plan->geo;
        const sc_conv_desc& d = plan->desc;
        int32_t* kept_dev = reinterpret_cast<int32_t*>(plan->ws + g.off_kept);
        int32_t span[3] = {0, 0, 0};
        hipLaunchKernelGGL(slab_span_kernel, dim3((unsigned)((g.m + 63) / 64 + 255) / 256), dim3(256), 0, ts,
                           reinterpret_cast<const int32_t*>(plan->ws + g.off_rows), kept_dev, g.ho * g.wo, g.wo, d.h + 2 * d.pad_h, d.kh, kept_dev + 2);
        if (hip_failed(hipGetLastError()) || hip_failed(hipMemcpyAsync(span, kept_dev + 2, sizeof(span), hipMemcpyDeviceToHost, ts)) ||
            hip_failed(hipStreamSynchronize(ts))) { result = SC_ERR_HIP; break; }
        for (int b = 0; b < 3; ++b) plan->slab_span[0][b] = span[b];
      }
      const sc_plan::Window priced = plan->window[which];
      sc_plan::Window best_window = priced;
      auto try_window = [&](sc_plan::Window w) {
        plan->window[which] = w;
        const double us = time_us(dense, 40, 3);
        if (us > 0.0 && us < 0.985 * best_us) { best_us = us; best_window = w; }
      };
      if (band_applies && priced.before_bands) try_window({0, 0, false});
      for (const auto& tile : kWindowTiles)
        if ((tile[0] != priced.bm || tile[1] != priced.bn) && window_fits(plan, which, tile[0], tile[1]))
          try_window({tile[0], tile[1], band_applies, band_applies && !bsel.pp && !bsel.tap && plan->desc.c_in < 48});
      plan->window[which] = best_window;
    }
    best_tiled = try_tiled(which, &best_pick, &best_us);
    plan->pick[which] = best_pick;
    plan->prefer_tiled[which] = best_tiled;
    // the slab form of the tiled kernel (deep 3x3 layers): both tile heights, the K splits around one workgroup per
    // compute unit; it replaces the choice so far only where it measures faster
    if (plan->slab_ok && plan->slab == 0 && plan->split_k == 0 && !(band_applies && !best_tiled && !bands_give_way(plan, which, rows))) {
      plan->prefer_tiled[which] = best_tiled || band_applies;      // (or the band kernel would run in its place)
      sc_plan::Slab best_slab = {0, 1};
      for (int bm = 256; bm >= 128; bm >>= 1) {
        if (!slab_buffer_bytes(plan->desc, bm, plan->slab_span[which][span_of(bm)])) continue;
        const int around = slab_splits(plan, bm, rows);
        int tried[4] = {0, 0, 0, 0}, n_tried = 0;
        for (int sp : {around, around - 1, around + 1, 1}) {
          if (sp < 1 || sp > plan->desc.c_in / kSlabCh || (sp > 1 && !plan->geo.splitk_ok)) continue;
          if ((int64_t)((rows + bm - 1) / bm) * ((plan->desc.c_out + kSlabBN - 1) / kSlabBN) * sp * bm * kSlabBN * 4 > (int64_t)kSplitKPartialBytes) continue;
          bool seen = false;
          for (int i = 0; i < n_tried; ++i) seen = seen || tried[i] == sp;
          if (seen) continue;
          tried[n_tried++] = sp;
          plan->slab_auto[which] = {bm, sp};
          const double us = time_us(dense, 40, 3);
          if (us > 0.0 && us < 0.985 * best_us) { best_us = us; best_slab = {bm, sp}; }
        }
      }
      plan->slab_auto[which] = best_slab;
      if (!best_slab.bm) plan->prefer_tiled[which] = best_tiled;
    }
  }
  // A sparse run must not lose to the dense run of its own plan: where it still does, try the dense run's tile with
  // every row contracted and the mask applied at the store.
  if (result == SC_OK && !staged && plan->forced[0] == -1 && plan->forced[1] == -1 && plan->kept > 0 && plan->kept < plan->geo.m &&
      plan->masked_store != 1 && plan->geo.vec_gather && !plan->geo.rowseg && plan->desc.layout == SC_NHWC) {
    const double us_sparse = time_us(false, 40, 3), us_dense = time_us(true, 40, 3);
    // (where the dense run takes a band or row-panel kernel, the tile is the one the dense run would take as a tiled launch)
    if (us_sparse > 0.0 && us_dense > 0.0 && us_sparse > us_dense) {
      const sc_plan::Pick keep = plan->pick[0];
      const bool keep_tiled = plan->prefer_tiled[0];
      const sc_plan::Slab keep_slab = plan->slab_auto[0];
      plan->pick[0] = {plan->pick[1].ti, 1, true};
      plan->prefer_tiled[0] = true;
      plan->slab_auto[0] = sc_plan::Slab{0, 1};
      const double us = time_us(false, 40, 3);
      if (!(us > 0.0 && us < us_sparse)) { plan->pick[0] = keep; plan->prefer_tiled[0] = keep_tiled; plan->slab_auto[0] = keep_slab; }
    }
  }
  plan->tuned = result == SC_OK;
  if (hip_failed(hipStreamSynchronize(ts)) && result == SC_OK) result = SC_ERR_HIP;
  if (result == SC_OK) result = launch_conv(plan, false, x_dev, bias_dev, y_dev, stream);   // y = the masked convolution
  if (hip_failed(hipStreamSynchronize(stream)) && result == SC_OK) result = SC_ERR_HIP;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipStreamDestroy(ts);
  return result;
}

sc_status sparse_conv_plan_info(const sc_plan* plan, int64_t* m, int64_t* kept, int32_t* ho, int32_t* wo,
                                const int32_t** row_idx_dev) {
  if (!plan) return SC_ERR_NULL;
  if (m) *m = plan->geo.m;
  if (kept) *kept = plan->kept;
  if (ho) *ho = plan->geo.ho;
  if (wo) *wo = plan->geo.wo;
  if (row_idx_dev) *row_idx_dev = reinterpret_cast<const int32_t*>(plan->ws + plan->geo.off_rows);
  return SC_OK;
}

const uint8_t* sparse_conv_plan_mask(const sc_plan* plan) {
  return plan ? plan->ws + plan->geo.off_mask : nullptr;
}

sc_status sparse_conv_plan_tiles(const sc_plan* plan, int32_t which, int32_t* tile_m, int32_t* tile_n,
                                 int64_t* workgroups) {
  if (!plan) return SC_ERR_NULL;
  if (which != 0 && which != 1) return SC_ERR_UNSUPPORTED;
  if (plan->geo.depthwise) {   // one lane per pixel and 16-byte channel group, 256 lanes per workgroup
    const int eb = elem_bytes(plan->desc.dtype);
    const int v = plan->desc.c_in % (16 / eb) == 0 ? 16 / eb : 1;
    const bool walk_dense = which == 1 || plan->desc.out_mode == SC_OUT_ZERO_FILL;
    if (tile_m) *tile_m = 1;
    if (tile_n) *tile_n = v;
    if (workgroups) *workgroups = ((walk_dense ? plan->geo.m : plan->kept) * (plan->desc.c_in / v) + 255) / 256;
    return SC_OK;
  }
  const BandPlan& band = which ? plan->band_dense : plan->band;
  if (band.ok && (plan->forced[which] == kForceBand || (plan->forced[which] == -1 && !band.stream && !plan->prefer_tiled[which])) &&
      !(plan->slab >= 2 && slab_pick(plan, which, which ? plan->geo.m : plan->kept).bm) && !use_stage(plan, which) &&
      !bands_give_way(plan, which, which ? plan->geo.m : plan->kept)) {
    if (tile_m) *tile_m = -band.bh;     // (rows per run; split bands hold half a run each)
    if (tile_n) *tile_n = 32 * band.ni;
    if (workgroups) *workgroups = band.pp && !band.tap ? band.pp_grid : (int64_t)band.n_bands * band.n_tiles;
    return SC_OK;
  }
  int64_t rows = which ? plan->geo.m : plan->kept;
  const bool window = use_window(plan, which, rows);
  if (const sc_plan::Slab sl = slab_pick(plan, which, rows); sl.bm) {
    if (tile_m) *tile_m = sl.bm;
    if (tile_n) *tile_n = kSlabBN;
    if (workgroups) *workgroups = ((rows + sl.bm - 1) / sl.bm) * ((plan->desc.c_out + kSlabBN - 1) / kSlabBN) * std::min(sl.splits, plan->desc.c_in / kSlabCh);
    return SC_OK;
  }
  if (window) {
    const sc_plan::Window win = plan->window[which];
    if (tile_m) *tile_m = win.bm;
    if (tile_n) *tile_n = win.bn;
    if (workgroups) *workgroups = ((rows + win.bm - 1) / win.bm) * ((plan->desc.c_out + win.bn - 1) / win.bn);
    return SC_OK;
  }
  if (use_stage(plan, which)) {
    const StageTile st = plan->stage_pick[which];
    if (tile_m) *tile_m = st.bm;
    if (tile_n) *tile_n = st.bn;
    if (workgroups) *workgroups = ((rows + st.bm - 1) / st.bm) * ((plan->desc.c_out + st.bn - 1) / st.bn);
    return SC_OK;
  }
  if (use_panel(plan, which, rows)) {
    if (tile_m) *tile_m = kPanelBM;
    if (tile_n) *tile_n = kPanelBN;
    if (workgroups) *workgroups = (rows + kPanelBM - 1) / kPanelBM;
    return SC_OK;
  }
  const TilePick tp = pick_tile(plan, which, rows);
  const int splits = tp.masked ? 1 : tp.splits;
  if (tp.masked && which == 0) rows = plan->geo.m;
  const KernelEntry& ke = plan->table[tp.ti];
  if (tile_m) *tile_m = ke.bm;
  if (tile_n) *tile_n = ke.bn;
  if (workgroups) *workgroups = ((rows + ke.bm - 1) / ke.bm) * ((plan->desc.c_out + ke.bn - 1) / ke.bn) * splits;
  const int sk = splits == 1 ? stream_k_workgroups(plan, ke, rows) : 0;
  if (sk && workgroups) *workgroups = sk;      // persistent workgroups of a stream-K launch
  return SC_OK;
}

// name of the tiled kernel a launch of this plan takes when no band or row-panel kernel applies
static const char* tiled_kernel_name(const sc_plan* plan, int32_t which, LaunchForm form) {
  const Geometry& g = plan->geo;
  if (use_stage(plan, which, form)) return "tile_staged";
  if (use_window(plan, which, which ? g.m : plan->kept, form == kPlainRun)) return "tile_window";
  const TilePick tp = pick_tile(plan, which, which ? g.m : plan->kept);
  if (tp.masked) return "tile_masked_store";
  if (tp.splits > 1) return "tile_split_k";
  if (stream_k_workgroups(plan, plan->table[tp.ti], which ? g.m : plan->kept)) return "tile_stream_k";
  if (g.rowseg) return "tile_row_segments";
  if (!g.vec_gather) return "tile_elements";
  return (g.vec_out && plan->gather_pipeline != 1) ? "tile_lds_direct" : "tile_registers";
}

const char* sparse_conv_plan_kernel(const sc_plan* plan, int32_t which) {
  if (!plan || (which != 0 && which != 1)) return nullptr;
  if (plan->geo.depthwise) return "depthwise";
  const BandPlan& band = which ? plan->band_dense : plan->band;
  if (band.ok && (plan->forced[which] == kForceBand || (plan->forced[which] == -1 && !band.stream && !plan->prefer_tiled[which])) &&
      !(plan->slab >= 2 && slab_pick(plan, which, which ? plan->geo.m : plan->kept).bm) && !use_stage(plan, which) &&
      !bands_give_way(plan, which, which ? plan->geo.m : plan->kept))
    return band.rowband ? "band_row_segments" : band.stream ? "band_stream" : band.tap ? "band_tap" : band.pp ? "band_alternating" : "band";
  const Geometry& g = plan->geo;
  if (slab_pick(plan, which, which ? g.m : plan->kept).bm) return "tile_slab";
  if (use_panel(plan, which, which ? g.m : plan->kept)) return "tile_row_panel";
  return tiled_kernel_name(plan, which, kPlainRun);
}

const char* sparse_conv_plan_fused_kernel(const sc_plan* plan, int32_t which) {
  if (!plan || (which != 0 && which != 1) || plan->geo.depthwise) return nullptr;
  const BandPlan& band = which ? plan->band_dense : plan->band;
  if (band.ok && (band.pp || band.tap) && !band.stream &&
      (plan->forced[which] == kForceBand || (plan->forced[which] == -1 && !plan->prefer_tiled[which])) &&
      !(plan->slab >= 2 && slab_pick(plan, which, which ? plan->geo.m : plan->kept).bm) &&
      !bands_give_way(plan, which, which ? plan->geo.m : plan->kept))
    return band.tap ? "band_tap" : "band_alternating";
  if (slab_pick(plan, which, which ? plan->geo.m : plan->kept).bm) return "tile_slab";
  return tiled_kernel_name(plan, which, kFusedRun);
}

sc_status sparse_conv_plan_set_tiles(sc_plan* plan, int32_t which, int32_t tile_m, int32_t tile_n) {
  if (!plan) return SC_ERR_NULL;
  if (which != 0 && which != 1) return SC_ERR_UNSUPPORTED;
  if (tile_m == 0 && tile_n == 0) { plan->forced[which] = -1; return SC_OK; }
  if (plan->geo.depthwise) return SC_ERR_UNSUPPORTED;   // one kernel, no tiles to choose
  if (tile_m < 0) {
    if (!(which ? plan->band_dense : plan->band).ok) return SC_ERR_UNSUPPORTED;
    plan->forced[which] = kForceBand;
    return SC_OK;
  }
  for (int i = 0; i < plan->table_count; ++i)
    if (plan->table[i].bm == tile_m && plan->table[i].bn == tile_n) { plan->forced[which] = i; return SC_OK; }
  return SC_ERR_UNSUPPORTED;
}

sc_status sparse_conv_plan_set_option(sc_plan* plan, int32_t option, int32_t value) {
  if (!plan) return SC_ERR_NULL;
  if (option == SC_OPT_GATHER_PIPELINE && value >= 0 && value <= 2) { plan->gather_pipeline = value; return SC_OK; }
  if (option == SC_OPT_ROW_PANEL && value >= 0 && value <= 2) { plan->row_panel = value; return SC_OK; }
  if (option == SC_OPT_SPLIT_K && value >= 0 && value <= kSplitKMost) { plan->split_k = value; return SC_OK; }
  if (option == SC_OPT_STREAM_K && value >= 0 && value <= kStreamKMostWgs) { plan->stream_k = value; return SC_OK; }
  if (option == SC_OPT_MASKED_STORE && value >= 0 && value <= 2) { plan->masked_store = value; return SC_OK; }
  if (option == SC_OPT_SLAB && ((value >= 0 && value <= 2) || value == 128 || value == 256)) { plan->slab = value; return SC_OK; }
  return SC_ERR_UNSUPPORTED;
}

void sparse_conv_plan_destroy(sc_plan* plan) { delete plan; }

const char* sc_status_string(sc_status s) {
  switch (s) {
    case SC_OK: return "ok";
    case SC_ERR_NULL: return "a required pointer is NULL";
    case SC_ERR_BAD_SHAPE: return "bad shape (non-positive extent, empty output or tensor too large)";
    case SC_ERR_UNSUPPORTED: return "unsupported (groups other than 1 or depthwise NHWC, or unknown dtype/layout/mode/tile/format)";
    case SC_ERR_MASK_COUNT: return "mask popcount differs from the count the sparsity ratio demands";
    case SC_ERR_WORKSPACE: return "workspace too small";
    case SC_ERR_ALIGN: return "device pointer not sufficiently aligned";
    case SC_ERR_HIP: return "a HIP call failed (see sc_last_hip_error)";
  }
  return "unknown status";
}

int32_t sc_last_hip_error(void) { return sc::g_last_hip; }

#ifdef SC_TIMING
void sc_debug_set_buffer(void* p) { sc::g_dbg = static_cast<long long*>(p); }
#endif

sc_status sc_maxpool2d_nhwc(const void* x_dev, void* y_dev, int32_t dtype, int32_t n, int32_t h, int32_t w,
                            int32_t c, int32_t k, int32_t s, int32_t p, void* hip_stream) {
  if (!x_dev || !y_dev) return SC_ERR_NULL;
  if (dtype != SC_F32 && dtype != SC_F16 && dtype != SC_BF16) return SC_ERR_UNSUPPORTED;
  if (n < 1 || h < 1 || w < 1 || c < 1 || k < 1 || s < 1 || p < 0 || 2 * p > k) return SC_ERR_BAD_SHAPE;
  int ho = out_extent(h, k, s, p, 1), wo = out_extent(w, k, s, p, 1);
  if (ho < 1 || wo < 1) return SC_ERR_BAD_SHAPE;
  int64_t total = (int64_t)n * ho * wo * c;
  if (total >= ((int64_t)1 << 31) * 256) return SC_ERR_BAD_SHAPE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  dim3 grid((unsigned)((total + 255) / 256)), block(256);
  const bool vec8 = dtype != SC_F32 && c % 8 == 0 && (((uintptr_t)x_dev | (uintptr_t)y_dev) & 15) == 0;
  if (vec8 && k == 3 && total / 8 < ((int64_t)1 << 31)) {
    dim3 vgrid((unsigned)((total / 8 + 255) / 256));
    uint32_t cm, cs, wm, ws_, hm, hs;
    sc::magic_div((uint32_t)(c / 8), &cm, &cs);
    sc::magic_div((uint32_t)wo, &wm, &ws_);
    sc::magic_div((uint32_t)ho, &hm, &hs);
    if (dtype == SC_F16)
      hipLaunchKernelGGL(maxpool3_nhwc_vec8_kernel<_Float16>, vgrid, block, 0, stream, (const _Float16*)x_dev,
                         (_Float16*)y_dev, n, h, w, c, s, p, ho, wo, cm, cs, wm, ws_, hm, hs);
    else
      hipLaunchKernelGGL(maxpool3_nhwc_vec8_kernel<__bf16>, vgrid, block, 0, stream, (const __bf16*)x_dev,
                         (__bf16*)y_dev, n, h, w, c, s, p, ho, wo, cm, cs, wm, ws_, hm, hs);
  } else if (vec8) {
    dim3 vgrid((unsigned)((total / 8 + 255) / 256));
    if (dtype == SC_F16)
      hipLaunchKernelGGL(maxpool_nhwc_vec8_kernel<_Float16>, vgrid, block, 0, stream, (const _Float16*)x_dev,
                         (_Float16*)y_dev, n, h, w, c, k, s, p, ho, wo);
    else
      hipLaunchKernelGGL(maxpool_nhwc_vec8_kernel<__bf16>, vgrid, block, 0, stream, (const __bf16*)x_dev,
                         (__bf16*)y_dev, n, h, w, c, k, s, p, ho, wo);
  } else if (dtype == SC_F32)
    hipLaunchKernelGGL(maxpool_nhwc_kernel<float>, grid, block, 0, stream, (const float*)x_dev, (float*)y_dev, n, h,
                       w, c, k, s, p, ho, wo);
  else if (dtype == SC_F16)
    hipLaunchKernelGGL(maxpool_nhwc_kernel<_Float16>, grid, block, 0, stream, (const _Float16*)x_dev,
                       (_Float16*)y_dev, n, h, w, c, k, s, p, ho, wo);
  else
    hipLaunchKernelGGL(maxpool_nhwc_kernel<__bf16>, grid, block, 0, stream, (const __bf16*)x_dev, (__bf16*)y_dev, n,
                       h, w, c, k, s, p, ho, wo);
  SC_HIP(hipGetLastError());
  return SC_OK;
}

}  // extern "C"

template <bool RELU>
static sc_status add_launch(const void* a_dev, const void* b_dev, void* y_dev, int32_t dtype, int64_t count,
                            void* hip_stream) {
  if (!a_dev || !b_dev || !y_dev) return SC_ERR_NULL;
  if (dtype != SC_F32 && dtype != SC_F16 && dtype != SC_BF16) return SC_ERR_UNSUPPORTED;
  if (count < 0) return SC_ERR_BAD_SHAPE;
  if (count == 0) return SC_OK;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  dim3 grid((unsigned)std::min<int64_t>((count + 255) / 256, 65536)), block(256);
  const bool vec8 = dtype != SC_F32 && count % 8 == 0 &&
                    (((uintptr_t)a_dev | (uintptr_t)b_dev | (uintptr_t)y_dev) & 15) == 0;
  if (vec8) {
    dim3 vgrid((unsigned)std::min<int64_t>((count / 8 + 255) / 256, 65536));
    if (dtype == SC_F16)
      hipLaunchKernelGGL((add_vec8_kernel<_Float16, RELU>), vgrid, block, 0, stream, (const _Float16*)a_dev,
                         (const _Float16*)b_dev, (_Float16*)y_dev, count / 8);
    else
      hipLaunchKernelGGL((add_vec8_kernel<__bf16, RELU>), vgrid, block, 0, stream, (const __bf16*)a_dev,
                         (const __bf16*)b_dev, (__bf16*)y_dev, count / 8);
  } else if (dtype == SC_F32)
    hipLaunchKernelGGL((add_kernel<float, RELU>), grid, block, 0, stream, (const float*)a_dev, (const float*)b_dev,
                       (float*)y_dev, count);
  else if (dtype == SC_F16)
    hipLaunchKernelGGL((add_kernel<_Float16, RELU>), grid, block, 0, stream, (const _Float16*)a_dev,
                       (const _Float16*)b_dev, (_Float16*)y_dev, count);
  else
    hipLaunchKernelGGL((add_kernel<__bf16, RELU>), grid, block, 0, stream, (const __bf16*)a_dev, (const __bf16*)b_dev,
                       (__bf16*)y_dev, count);
  SC_HIP(hipGetLastError());
  return SC_OK;
}

extern "C" {

sc_status sc_add_relu(const void* a_dev, const void* b_dev, void* y_dev, int32_t dtype, int64_t count,
                      void* hip_stream) {
  return add_launch<true>(a_dev, b_dev, y_dev, dtype, count, hip_stream);
}

sc_status sc_add(const void* a_dev, const void* b_dev, void* y_dev, int32_t dtype, int64_t count, void* hip_stream) {
  return add_launch<false>(a_dev, b_dev, y_dev, dtype, count, hip_stream);
}

}  // extern "C"
