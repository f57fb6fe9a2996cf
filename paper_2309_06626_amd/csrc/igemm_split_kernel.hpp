// Tiled masked-convolution kernel for float NHWC layers (Cin and Cout multiples of four): operands straight into LDS, the
// contraction on the bf16 matrix pipes in three parts per operand (see igemm_stage_kernel.hpp for the arithmetic, which is
// the same, and for the pass over values that are not finite).
//
// A wavefront owns 32 rows of the tile and all of its channels, so a row's values are split into their parts by one
// wavefront only, in registers, behind the matrix work of the step before; LDS holds the rows as they are (128 bytes of
// K, 16-byte groups exchanged like in igemm_dma_kernel) and the filters in the order of the plan's packed parts.  Both
// arrive through `buffer_load ... lds`: no registers, no LDS stores.
//
// What bounds it: a wavefront's own chain, splitting, then multiplying.  Six MFMAs per pair of blocks are 0.35 us a K tile of
// 128 x 64 at the matrix pipes' rate; it costs 0.53 us with two workgroups on a compute unit, and a workgroup alone takes
// 0.69 us a tile, one wait after the other, which is what the groups that share K are for.  On 64 -> 64 @56 at batch 32 the matrix
// pipes and the vector issue are busy 31 % of the time each, LDS 11 % (counters), and 392 workgroups are one and a half per compute
// unit.  Measured at s = 0.5 (float MFMA before / this kernel, us; batch 32): 64 -> 64 @56 58 / 31 (119 TFLOP/s of float
// arithmetic), 128 -> 128 @28 55 / 31, 256 -> 256 @14 61 / 38, batch 16 384 -> 384 @12 88 / 32, one image of 128 -> 128 @28
// 32 / 15.  Error of the first against 64 bits: 3.0e-7 before, 1.0e-7 now.
//
// Two tiles in LDS a group: 56 KB and four wavefronts for 128 x 64, 44 for 128 x 32, 40 KB and two for 64 x 64, 28 for 64 x 32, so
// that two to five workgroups of one group share a compute unit and fill each other's waits.
#pragma once
#include "igemm_stage_kernel.hpp"

namespace sc {

template <int BM, int BN, int KS> constexpr size_t split_lds_bytes() {
  return KS * 2 * ((size_t)BM * kRowBytes + (size_t)(BN / 32) * StageDims<kF32>::BLOCK_BYTES);
}

// TAPS: a K tile lies inside one window tap (Cin a multiple of 32): the walk over the window is scalar.  Otherwise each
// lane finds its 16-byte group in the plan's table.
// VEC_OUT: 1 = Cout a multiple of 16, 2 = a multiple of four.
// KS: the K tiles are divided among KS groups of wavefronts, each with LDS tiles of its own; the first group adds the others'
// sums in order and stores.  For launches with few workgroups, whose time is one K tile's latency after the other.
template <int BM, int BN, int KS, bool TAPS, int VEC_OUT>
__global__ __launch_bounds__(2 * BM * KS, 2) void igemm_split_kernel(const ConvParams p) {
  using D = StageDims<kF32>;
  constexpr int NT = 2 * BM;                       // threads of a group: a wavefront per 32 rows
  constexpr int NTALL = NT * KS;
  constexpr int NI = BN / 32;
  static_assert(NI <= 2, "the registers hold two blocks of channels: two sums and two K steps of fragments each");
  constexpr int A_BYTES = BM * kRowBytes, B_BYTES = NI * D::BLOCK_BYTES, STAGE_BYTES = A_BYTES + B_BYTES;
  constexpr int RPR = NT / 8;                      // rows one transfer of the workgroup covers
  constexpr int A_LOADS = BM / RPR;                // = 4
  constexpr int WAVES = NT / 64;
  constexpr int B_UNITS = B_BYTES / 1024, B_LOADS = (B_UNITS + WAVES - 1) / WAVES;

  extern __shared__ __align__(16) unsigned char smem_all[];
  // (nothing beside the two tiles: 64 x 64 is exactly a quarter of a compute unit's LDS; behind the K loop the first words
  // hold the workgroup's flag and the bias slice)
  int32_t* s_flag = reinterpret_cast<int32_t*>(smem_all);
  float* s_bias = reinterpret_cast<float*>(smem_all + 16);                    // [BN]

  const int nwg = p.m_tiles * p.n_tiles;
  const int per_xcd = (nwg + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= nwg) return;
  const int tile_m = logical / p.n_tiles;
  const int tile_n = logical - tile_m * p.n_tiles;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int t = threadIdx.x;
  const int lane = t & 63, group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(t / NT);
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6) - group * WAVES;      // within the group
  unsigned char* smem = smem_all + group * (2 * STAGE_BYTES);
  const int kt_lo = KS == 1 ? 0 : group * p.k_tiles / KS, kt_hi = KS == 1 ? p.k_tiles : (group + 1) * p.k_tiles / KS;
  const int steps = (p.k_tiles + KS - 1) / KS;        // (of the longest share: every wavefront passes every barrier)
  const int wm0 = wave * 32;
  const int fp = lane & 31, fh = lane >> 5;
  float* __restrict__ y = static_cast<float*>(p.y);

  // ---- rows, bias slice, the dense row range this workgroup owns: one round trip ---------------------------------------
  const int lrow = wave * 8 + (lane >> 3);            // tile row of this lane's transfers (plus RPR per transfer)
  const int lc = (lane & 7) ^ ((lrow >> 1) & 7);      // the 16-byte group it fetches
  int32_t a_row[A_LOADS];
#pragma unroll
  for (int j = 0; j < A_LOADS; ++j) {
    const int icc = min(m0 + lrow + RPR * j, p.rows - 1);
    a_row[j] = p.row_idx ? p.row_idx[icc] : icc;
  }
  const int my_row = m0 + wm0 + fp;                   // the row of this lane's results
  const int out_row = my_row >= p.rows ? -1 : p.y_compact || !p.row_idx ? my_row : p.row_idx[my_row];
  const float bias_v = t < BN && p.bias && n0 + t < p.c_out ? p.bias[n0 + t] : 0.0f;
  int z_lo = 0, z_hi = p.m_total;
  if (p.zero_fill) {
    if (tile_m != 0) z_lo = p.row_idx[m0];
    if (m0 + BM < p.rows) z_hi = p.row_idx[m0 + BM];
  }
  KEntry ke = {0, 0};
  int32_t a_at[A_LOADS];       // byte offset of the window's corner (and this lane's group), possibly negative
  uint32_t a_taps[A_LOADS];    // which window rows (bits 0..7) and columns (bits 8..15) lie inside the image
#pragma unroll
  for (int j = 0; j < A_LOADS; ++j) {
    const int ic = m0 + lrow + RPR * j;
    const bool present = ic < p.rows;
    const int rc = p.x_compact ? min(ic, p.rows - 1) : a_row[j];
    const int n = fast_div(rc, p.div_howo_mul, p.div_howo_shift), rem = rc - n * p.ho_wo;
    const int oy = fast_div(rem, p.div_wo_mul, p.div_wo_shift), ox = rem - oy * p.wo;
    const int iy0 = oy * p.sh - p.ph, ix0 = ox * p.sw - p.pw;
    a_at[j] = (int32_t)((n * p.xs_n + (int64_t)iy0 * p.xs_h + (int64_t)ix0 * p.xs_w + (TAPS ? lc * 4 : 0)) * 4);
    uint32_t bits = 0;
    for (int ky = 0; ky < p.kh; ++ky) bits |= ((unsigned)(iy0 + ky * p.dil_h) < (unsigned)p.h ? 1u : 0u) << ky;
    for (int kx = 0; kx < p.kw; ++kx) bits |= ((unsigned)(ix0 + kx * p.dil_w) < (unsigned)p.w ? 1u : 0u) << (8 + kx);
    a_taps[j] = present ? bits : 0u;
  }

  // mask bytes of the first passes of the zero fill, requested here and looked at behind the first K tile
  constexpr int CPR = BN / 4, RPI = NTALL / CPR, ZB = 8;
  const int zc = t % CPR, zr = t / CPR;
  unsigned mk[ZB];
  auto mask_of = [&](int r) -> unsigned {
    if (p.mask_spatial) r -= fast_div(r, p.div_howo_mul, p.div_howo_shift) * p.ho_wo;
    return p.mask[r];
  };
#pragma unroll
  for (int u = 0; u < ZB; ++u) mk[u] = p.zero_fill ? mask_of(min(z_lo + zr + u * RPI, p.m_total - 1)) : 1u;

  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)p.x_bytes, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.wp), 0, (int)p.w_bytes, kBufferWord3);
  typedef __attribute__((address_space(3))) void lds_void;

  const int step_x = p.dil_w * p.xs_w * 4, step_y = p.dil_h * p.xs_h * 4;
  int s_ci, s_ky, s_kx, s_off, s_kt;      // scalar walk over the window (TAPS), next K tile to issue
  uint32_t s_bits;
  auto rewind = [&]() {
    s_kt = kt_lo;
    if constexpr (TAPS) {
      const int tap = kt_lo * 32 / p.c_in;
      s_ci = kt_lo * 32 - tap * p.c_in;
      s_ky = tap / p.kw;
      s_kx = tap - s_ky * p.kw;
      s_off = s_ci * 4 + s_kx * step_x + s_ky * step_y;
      s_bits = (1u << s_ky) | (1u << (8 + s_kx));
    } else {
      ke = p.ktab[min(s_kt, p.k_tiles - 1) * 8 + lc];
    }
  };
  rewind();
  const int w_tile0 = (n0 / 32) * p.k_tiles;                  // packed filters: [32 channels][K tile]
  auto issue_tile = [&](int stage) {
    unsigned char* sa = smem + stage * STAGE_BYTES + wave * 8 * kRowBytes;
    const uint32_t need = TAPS ? s_bits : (uint32_t)ke.dydx;
    const int off = TAPS ? s_off : ke.off;
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j) {
      const uint32_t voff = (a_taps[j] & need) == need ? (uint32_t)(a_at[j] + off) : kOutOfRange;     // out of range: zeros
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)(sa + j * RPR * kRowBytes), 16, voff, 0, 0, 0);
    }
    unsigned char* sb = smem + stage * STAGE_BYTES + A_BYTES;
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) {
      // (a wavefront without a unit of its own in the last round repeats the last one: the same bytes to the same place)
      const int u = min(wave + WAVES * j, B_UNITS - 1);
      constexpr int PER = D::BLOCK_BYTES / 1024;
      const int nb = u / PER, in = u - nb * PER;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)(sb + u * 1024), 16, (uint32_t)(lane * 16),
                                               (w_tile0 + nb * p.k_tiles + s_kt) * D::BLOCK_BYTES + in * 1024, 0, 0);
    }
    ++s_kt;
    if constexpr (TAPS) {
      s_ci += 32;
      s_off += 128;
      if (s_ci == p.c_in) {
        s_ci = 0;
        s_off += step_x - p.c_in * 4;
        if (++s_kx == p.kw) {
          s_kx = 0;
          ++s_ky;
          s_off += step_y - p.kw * step_x;
        }
        s_bits = (1u << s_ky) | (1u << (8 + s_kx));
      }
    } else {
      ke = p.ktab[min(s_kt, p.k_tiles - 1) * 8 + lc];         // (used by the next call, a tile later)
    }
  };

  floatx16 acc[NI], small[NI];
  auto clear = [&]() {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[ni][v] = small[ni][v] = 0.0f;
  };

  // fragment addresses: lane (fp, fh) of K step ks holds entries 16 ks + 8 fh .. + 7 of row wm0 + fp: two groups
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  unsigned frag_a[2][2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int g = 0; g < 2; ++g)
      frag_a[ks][g] = lds0 + (unsigned)((wm0 + fp) * kRowBytes + (((4 * ks + 2 * fh + g) ^ (((wm0 + fp) >> 1) & 7)) << 4));
  const unsigned frag_b = lds0 + (unsigned)(A_BYTES + lane * 16);

  struct Frags { v4i x[2]; v4i w[NI][3]; };
  auto read_x = [&](auto stage_c, int ks, Frags& f) {
    constexpr int SO = decltype(stage_c)::value * STAGE_BYTES;
    f.x[0] = lds_read16_big<SO>(frag_a[ks][0]);
    f.x[1] = lds_read16_big<SO>(frag_a[ks][1]);
  };
  auto read_w = [&](auto stage_c, auto ks_c, Frags& f) {
    constexpr int SO = decltype(stage_c)::value * STAGE_BYTES + decltype(ks_c)::value * 1024;
    auto block = [&](auto ni_c) {
      constexpr int ni = decltype(ni_c)::value;
      if constexpr (ni < NI) {
        f.w[ni][0] = lds_read16_big<SO + ni * D::BLOCK_BYTES>(frag_b);
        f.w[ni][1] = lds_read16_big<SO + ni * D::BLOCK_BYTES + 2048>(frag_b);
        f.w[ni][2] = lds_read16_big<SO + ni * D::BLOCK_BYTES + 4096>(frag_b);
      }
    };
    block(std::integral_constant<int, 0>{});
    block(std::integral_constant<int, 1>{});
  };
  // at most N LDS reads still on their way; the fragments pass through, so nothing that uses them moves above
  auto landed = [&](auto n_c, Frags& f) {
    constexpr int N = decltype(n_c)::value;
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(f.x[0]), "+v"(f.x[1]) : "n"(N));
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) asm volatile("" : "+v"(f.w[ni][0]), "+v"(f.w[ni][1]), "+v"(f.w[ni][2]));
  };
  auto contract_step = [&](const Frags& f, auto careful_c) {
    constexpr bool CAREFUL = decltype(careful_c)::value;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = __builtin_bit_cast(v4f, f.x[e >> 2])[e & 3];
    if constexpr (CAREFUL) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          auto part = [&](int q) {
            const uint32_t v = (uint32_t)f.w[ni][q][e >> 1];
            return (e & 1) ? bf16_hi(v) : bf16_lo(v);
          };
          acc[ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(join3(part(0), part(1), part(2)), x[e], acc[ni], 0, 0, 0);
        }
    } else {
      using H = Elem<kBF16>;
      v4i p1, p2, p3;
      split3(x, p1, p2, p3);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) H::mma(acc[ni], f.w[ni][0], p1);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) H::mma(small[ni], f.w[ni][1], p1);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) H::mma(small[ni], f.w[ni][0], p2);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) H::mma(small[ni], f.w[ni][1], p2);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) H::mma(small[ni], f.w[ni][2], p1);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) H::mma(small[ni], f.w[ni][0], p3);
    }
  };

  auto fill_zeros = [&]() {
    const int valid = min(BN, p.c_out - n0) / 4;
    if (zc >= valid) return;
    unsigned char* ybase = reinterpret_cast<unsigned char*>(y) + (int64_t)n0 * 4 + zc * 16;
    const int64_t res_at = (int64_t)n0 * 4 + zc * 16;
    const v4i z = {0, 0, 0, 0};
    auto pass = [&](int r, unsigned keep) {
      if (r < z_hi && keep == 0) {
        const int64_t at = (int64_t)r * p.c_out * 4;
        *reinterpret_cast<v4i*>(ybase + at) = p.residual ? dropped_row_group<kF32>(p.residual, res_at + at, p.residual_relu) : z;
      }
    };
#pragma unroll
    for (int u = 0; u < ZB; ++u) pass(z_lo + zr + u * RPI, mk[u]);
    for (int r0 = z_lo + zr + ZB * RPI; r0 < z_hi; r0 += ZB * RPI) {
      unsigned m[ZB];
#pragma unroll
      for (int u = 0; u < ZB; ++u) m[u] = mask_of(min(r0 + u * RPI, z_hi - 1));
#pragma unroll
      for (int u = 0; u < ZB; ++u) pass(r0 + u * RPI, m[u]);
    }
  };

  auto k_tile = [&](auto stage_c, int kt, auto careful_c) {      // kt: of this group's share
    constexpr int ST = decltype(stage_c)::value;
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();        // the tile has landed for every wavefront, and all have left the one before
    asm volatile("" ::: "memory");
    if (kt + 1 < kt_hi) issue_tile(ST ^ 1);
    if (KS > 1 && kt >= kt_hi) return;
    Frags f0, f1;
    read_x(stage_c, 0, f0);
    read_w(stage_c, std::integral_constant<int, 0>{}, f0);
    read_x(stage_c, 1, f1);
    read_w(stage_c, std::integral_constant<int, 1>{}, f1);
    landed(std::integral_constant<int, 2 + 3 * NI>{}, f0);
    contract_step(f0, careful_c);
    landed(std::integral_constant<int, 0>{}, f1);
    contract_step(f1, careful_c);
  };
  auto contract = [&](auto careful_c) {
    clear();
    if (kt_lo < kt_hi) issue_tile(0);
    for (int i = 0; i < steps; i += 2) {
      k_tile(std::integral_constant<int, 0>{}, kt_lo + i, careful_c);
      if constexpr (!decltype(careful_c)::value) {
        if (i == 0 && p.zero_fill) fill_zeros();        // (these stores drain under the K loop)
      }
      if (i + 1 < steps) k_tile(std::integral_constant<int, 1>{}, kt_lo + i + 1, careful_c);
    }
    __syncthreads();
    if constexpr (!decltype(careful_c)::value) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[ni][v] = (acc[ni][v] + small[ni][v]) * kSumScale;
    }
    if constexpr (KS > 1) {
      v4f* part = reinterpret_cast<v4f*>(smem_all) + wave * (NI * 4 * 64) + lane;
      constexpr int SLOT = WAVES * NI * 4 * 64;
      static_assert((KS - 1) * SLOT * 16 <= KS * 2 * STAGE_BYTES, "the partial sums lie where the tiles were");
      if (group > 0) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            part[(group - 1) * SLOT + (ni * 4 + q) * 64] = v4f{acc[ni][4 * q], acc[ni][4 * q + 1], acc[ni][4 * q + 2], acc[ni][4 * q + 3]};
      }
      __syncthreads();
      if (group == 0) {
#pragma unroll
        for (int g = 0; g < KS - 1; ++g)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const v4f v = part[g * SLOT + (ni * 4 + q) * 64];
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[ni][4 * q + e] += v[e];
            }
      }
      __syncthreads();
    }
  };
  contract(std::false_type{});
  float odd = 0.0f;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int v = 0; v < 16; ++v) odd = not_finite(acc[ni][v], odd);
  if (t == 0) *s_flag = 0;
  __syncthreads();
  if (odd != odd) *s_flag = 1;
  __syncthreads();
  if (*s_flag) {
    __syncthreads();
    rewind();
    contract(std::true_type{});
  }
  for (int i = t; i < BN; i += NTALL) s_bias[i] = i == t ? bias_v : p.bias && n0 + i < p.c_out ? p.bias[n0 + i] : 0.0f;
  __syncthreads();

  // ---- epilogue --------------------------------------------------------------------------------------------------------------
  if (group == 0) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int c0 = n0 + ni * 32 + 16 * fh;
      if (c0 >= p.c_out) continue;
      store_block_pairs<kF32, VEC_OUT == 1>(acc[ni], out_row, false, c0, y, p.bias ? s_bias + (c0 - n0) : nullptr, p.relu, p.c_out,
                                            static_cast<const float*>(p.residual), p.residual_relu);
    }
  }
}

template <int BM, int BN, int KS, bool TAPS, int VEC_OUT>
hipError_t igemm_split_launch(const ConvParams& p, hipStream_t stream) {
  constexpr size_t lds = split_lds_bytes<BM, BN, KS>();
  auto kern = igemm_split_kernel<BM, BN, KS, TAPS, VEC_OUT>;
  static std::atomic<bool> attr_set{false};
  if (lds > 64 * 1024 && !attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int nwg = p.m_tiles * p.n_tiles;
  hipLaunchKernelGGL(kern, dim3(((nwg + 7) / 8) * 8), dim3(2 * BM * KS), lds, stream, p);
  return hipGetLastError();
}

// the kernel of tile bm x bn with K in `groups` shares, or null (igemm_split.hip)
LaunchFn split_kernel(int bm, int bn, int groups, bool taps, int vec_out);

}  // namespace sc
