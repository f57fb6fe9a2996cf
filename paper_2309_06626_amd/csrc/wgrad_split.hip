// Filter gradient of float layers: dw[co][k] = sum over the kept rows of g[row][co] * A[row][k], the contraction on the bf16
// matrix pipes with three exact parts per operand, main and small products in sums of their own (see igemm_stage_kernel.hpp).
//
// A workgroup has 64 output channels x 64 window entries x one split of the kept rows.  The contraction runs over rows, and
// its four wavefronts divide a step's 64 rows: each has the whole tile for its own 16 rows, in LDS tiles of its own, so no
// value is split twice and the loop has no barrier.  Both operands lie row-major in LDS as panels of 16 rows x 256 bytes,
// filled by `buffer_load ... lds` (an offset past the end of a buffer writes the zeros of padded taps, absent rows and
// columns past the tile); an MFMA lane reads the eight rows of its column with four `ds_read2st64_b32`, whose two dwords lie
// a row apart.  The 16-byte groups of the lower eight rows are exchanged by eight, which puts the two halves of a wavefront
// on different halves of the banks.  A lane decodes one row a step and hands it round.
// The sums of the four wavefronts meet in LDS and are added in order; partial sums per split, added in split order by the
// reduction: results do not depend on scheduling.
// A wavefront whose sums are not all finite contracts its rows again with the float MFMA on the unsplit
// values, which gives the infinities of the plain sum.
//
// What bounds it: the vector instructions that split and decode (about 300 per 24 MFMAs of a wavefront's step; the vector issue is
// busy 59 % of the time, the matrix pipes 29 %, LDS 21 %: counters) next to the matrix work, with two wavefronts per SIMD.
// 16 x 64 -> 64 @56 at s = 0.5 (25 088 rows to contract): 72 us on the float MFMA (wgrad_f32_kernel, which stays for windows past
// the validity bits and tensors past 2 GiB), 20 us here.
#include "wgrad_split.hpp"

#include "igemm_stage_kernel.hpp"

namespace sc {

typedef float v2f __attribute__((ext_vector_type(2)));
constexpr int kWsPanel = 16 * 256;                 // 16 rows x 64 floats
constexpr int kWsStage = 2 * kWsPanel;             // one panel of g, one of the lowered rows
constexpr int kWsWaveLds = 2 * kWsStage;           // two stages

// two dwords of this lane's column, rows R and R + 1 of a panel
template <int ROW> __device__ __forceinline__ v2f lds_read_rows(unsigned addr) {
  v2f v;
  asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(v) : "v"(addr), "n"(ROW), "n"(ROW + 1));
  return v;
}

__global__ __launch_bounds__(256, 2) void wgrad_split_kernel(const WgradSplitParams p) {
  __shared__ __align__(16) unsigned char smem[4 * kWsWaveLds];
  const int tiles = p.co_tiles * p.k_tiles, nwg = tiles * p.splits;
  const int per_xcd = (nwg + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);      // the tiles of a split share an XCD's L2
  if (logical >= nwg) return;
  const int split = logical / tiles, tile = logical - split * tiles;
  const int co0 = (tile / p.k_tiles) * kWsTile, k0 = (tile % p.k_tiles) * kWsTile;
  const int i_begin = split * p.rows_per_split, i_end = min(p.rows, i_begin + p.rows_per_split);
  const int steps = (i_end - i_begin + kWsRows - 1) / kWsRows;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int fp = lane & 31, fh = lane >> 5;
  unsigned char* mine = smem + wave * kWsWaveLds;

  // ---- columns this lane transfers: logical 16-byte group lane % 16, exchanged by eight for rows 8 .. 15 --------------------
  int g_col[2], a_off[2];
  uint32_t a_bits[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int grp = (lane & 15) ^ (8 * f);
    const int co = co0 + grp * 4, kc = k0 + grp * 4;
    g_col[f] = co < p.c_out ? co * 4 : -1;
    const int tap = kc / p.c_in, ci = kc - tap * p.c_in;          // (Cin is a multiple of eight: a group lies in one tap)
    const int ky = tap / p.kw, kx = tap - ky * p.kw;
    a_off[f] = ((ky * p.dil_h * p.w + kx * p.dil_w) * p.c_in + ci) * 4;
    a_bits[f] = kc < p.k ? (1u << ky) | (1u << (8 + kx)) : kStageNoTap;
  }
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)p.x_bytes, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.g), 0, (int)p.g_bytes, kBufferWord3);
  typedef __attribute__((address_space(3))) void lds_void;

  // the row this lane decodes: row lane % 16 of its wavefront's step
  auto row_at = [&](int step) {
    const int i = min(i_begin + step * kWsRows + wave * 16 + (lane & 15), i_end - 1);
    return p.row_idx ? p.row_idx[i] : i;
  };
  int row = 0;
  auto issue = [&](int step, int slot) {
    const bool present = i_begin + step * kWsRows + wave * 16 + (lane & 15) < i_end;
    const int n = fast_div(row, p.div_howo_mul, p.div_howo_shift), rem = row - n * p.ho_wo;
    const int oy = fast_div(rem, p.div_wo_mul, p.div_wo_shift), ox = rem - oy * p.wo;
    const int iy0 = oy * p.sh - p.ph, ix0 = ox * p.sw - p.pw;
    const int corner = (((n * p.h + iy0) * p.w + ix0) * p.c_in) * 4;
    uint32_t bits = 0;
    for (int ky = 0; ky < p.kh; ++ky) bits |= ((unsigned)(iy0 + ky * p.dil_h) < (unsigned)p.h ? 1u : 0u) << ky;
    for (int kx = 0; kx < p.kw; ++kx) bits |= ((unsigned)(ix0 + kx * p.dil_w) < (unsigned)p.w ? 1u : 0u) << (8 + kx);
    if (!present) bits = 0;
    const int g_at = present ? row * p.c_out * 4 : (int)kOutOfRange;
    unsigned char* dst = mine + slot * kWsStage;
#pragma unroll
    for (int i = 0; i < 4; ++i) {                    // four rows at a time
      const int from = (4 * i + (lane >> 4)) * 4, f = i >> 1;
      const int c = __builtin_amdgcn_ds_bpermute(from, corner), ga = __builtin_amdgcn_ds_bpermute(from, g_at);
      const uint32_t b = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)bits);
      const uint32_t vg = g_col[f] >= 0 ? (uint32_t)(ga + g_col[f]) : kOutOfRange;
      const uint32_t va = (b & a_bits[f]) == a_bits[f] ? (uint32_t)(c + a_off[f]) : kOutOfRange;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rg, (lds_void*)(dst + i * 1024), 16, vg, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)(dst + kWsPanel + i * 1024), 16, va, 0, 0, 0);
    }
    row = row_at(step + 1);
  };

  floatx16 acc[2][2], small[2][2];
  auto clear = [&]() {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = small[a][b][v] = 0.0f;
  };
  // this lane's column of the even and the odd 32-column block, in the half of the rows its half of the wavefront reads
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)mine;
  unsigned col_at[2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
    col_at[b] = lds0 + (unsigned)(fh * 8 * 256 + (((8 * b + (fp >> 2)) ^ (8 * fh)) << 4) + (fp & 3) * 4);
  struct Column { v2f d[4]; };
  auto read = [&](auto slot_c, auto panel_c, int b, Column& c) {
    constexpr int R = decltype(slot_c)::value * (kWsStage / 256) + decltype(panel_c)::value * 16;
    c.d[0] = lds_read_rows<R>(col_at[b]);
    c.d[1] = lds_read_rows<R + 2>(col_at[b]);
    c.d[2] = lds_read_rows<R + 4>(col_at[b]);
    c.d[3] = lds_read_rows<R + 6>(col_at[b]);
  };
  auto landed = [&](auto n_c, Column& c) {
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(c.d[0]), "+v"(c.d[1]), "+v"(c.d[2]), "+v"(c.d[3]) : "n"(decltype(n_c)::value));
  };
  using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>;
  auto step = [&](auto slot_c, int s, auto careful_c) {
    constexpr bool CAREFUL = decltype(careful_c)::value;
    constexpr int SLOT = decltype(slot_c)::value;
    wait_vmcnt<0>();                                  // the step's panels have landed (and the next step's row number)
    if (s + 1 < steps) issue(s + 1, SLOT ^ 1);
    Column g[2], a[2];
    read(slot_c, I0{}, 0, g[0]);
    read(slot_c, I0{}, 1, g[1]);
    read(slot_c, I1{}, 0, a[0]);
    landed(std::integral_constant<int, 8>{}, g[0]);
    landed(std::integral_constant<int, 4>{}, g[1]);
    read(slot_c, I1{}, 1, a[1]);
    auto values = [](const Column& c, float (&f)[8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = c.d[e >> 1][e & 1];
    };
    if constexpr (CAREFUL) {
      landed(I0{}, a[0]);
      landed(I0{}, a[1]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(g[i].d[e >> 1][e & 1], a[j].d[e >> 1][e & 1], acc[i][j], 0, 0, 0);
    } else {
      using H = Elem<kBF16>;
      float f[8];
      v4i pg[2][3], pa[3];
      values(g[0], f); split3(f, pg[0][0], pg[0][1], pg[0][2]);
      values(g[1], f); split3(f, pg[1][0], pg[1][1], pg[1][2]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j == 0) landed(std::integral_constant<int, 4>{}, a[0]);
        else landed(I0{}, a[1]);
        values(a[j], f);
        split3(f, pa[0], pa[1], pa[2]);
#pragma unroll
        for (int i = 0; i < 2; ++i) H::mma(acc[i][j], pg[i][0], pa[0]);
#pragma unroll
        for (int i = 0; i < 2; ++i) H::mma(small[i][j], pg[i][1], pa[0]);
#pragma unroll
        for (int i = 0; i < 2; ++i) H::mma(small[i][j], pg[i][0], pa[1]);
#pragma unroll
        for (int i = 0; i < 2; ++i) H::mma(small[i][j], pg[i][1], pa[1]);
#pragma unroll
        for (int i = 0; i < 2; ++i) H::mma(small[i][j], pg[i][2], pa[0]);
#pragma unroll
        for (int i = 0; i < 2; ++i) H::mma(small[i][j], pg[i][0], pa[2]);
      }
    }
  };
  auto contract = [&](auto careful_c) {
    clear();
    row = row_at(0);
    issue(0, 0);
    for (int s = 0; s < steps; s += 2) {
      step(I0{}, s, careful_c);
      if (s + 1 < steps) step(I1{}, s + 1, careful_c);
    }
  };
  contract(std::false_type{});
  float odd = 0.0f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc[i][j][v] = (acc[i][j][v] + small[i][j][v]) * kSumScale;
        odd = not_finite(acc[i][j][v], odd);
      }
  if (__ballot(odd != odd)) contract(std::true_type{});

  // ---- the four wavefronts' sums: [wavefront][block][16 bytes of a lane], block b of the tile added by wavefront b ------------
  __syncthreads();
  v4f* sums = reinterpret_cast<v4f*>(smem);
  static_assert(4 * 4 * 4 * 64 * 16 <= 4 * kWsWaveLds, "the sums lie where the panels were");
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      sums[((wave * 4 + b) * 4 + q) * 64 + lane] = v4f{acc[b >> 1][b & 1][4 * q], acc[b >> 1][b & 1][4 * q + 1],
                                                       acc[b >> 1][b & 1][4 * q + 2], acc[b >> 1][b & 1][4 * q + 3]};
  __syncthreads();
  // MFMA result row 8j + 4h + i sits in register 4j + i of lane half h; column = lane % 32
  float* __restrict__ out = p.out + (int64_t)split * p.c_out * p.k;
  const int kc = k0 + (wave & 1) * 32 + fp;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v4f tot = sums[(wave * 4 + q) * 64 + lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const v4f v = sums[((w * 4 + wave) * 4 + q) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) tot[e] += v[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int co = co0 + (wave >> 1) * 32 + 8 * q + 4 * fh + e;
      if (co < p.c_out && kc < p.k) out[(int64_t)co * p.k + kc] = tot[e];
    }
  }
}

hipError_t wgrad_split_launch(const WgradSplitParams& p, hipStream_t stream) {
  const int nwg = p.co_tiles * p.k_tiles * p.splits;
  hipLaunchKernelGGL(wgrad_split_kernel, dim3(((nwg + 7) / 8) * 8), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace sc
