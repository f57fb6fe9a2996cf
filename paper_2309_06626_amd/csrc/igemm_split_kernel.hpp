// Tiled masked-convolution kernel for float NHWC layers (Cin and Cout multiples of four): operands straight into LDS, the
// contraction on the bf16 matrix pipes in three parts per operand (see igemm_stage_kernel.hpp for the arithmetic, which is
// the same, and for the pass over values that are not finite).
//
// A wavefront owns 32 rows of the tile and all of its channels, so a row's values are split into their parts by one
// wavefront only, in registers, behind the matrix work of the step before; LDS holds the rows as they are (128 bytes of
// K, 16-byte groups exchanged like in igemm_dma_kernel) and the filters in the order of the plan's packed parts.  Both
// arrive through `buffer_load ... lds`: no registers, no LDS stores.
//
// What bounds it: the issue slots of a wavefront.  A K tile of 128 x 64 is 24 MFMAs (768 cycles), and about 110 instructions that
// split, 16 LDS reads and 7 transfers at 5, 8 and 40 cycles; one after the other they took 1 950 cycles (0.885 us for a workgroup
// alone), now 1 300 (0.57 to 0.6): the split of the next step and the transfers lie behind the MFMAs of this one, across the barrier, the
// places of a tap's rows are worked out once a tap, and what was left of the loop's own bookkeeping (700 cycles without any work) went
// with its branches.  Deeper rings of tiles (three, four) change nothing: no transfer is waited for.  Two workgroups on a compute unit
// still take 1.15 us a pair of tiles, LDS and the address unit (1 300 and 900 cycles) beside 1 540 of products.
// On 64 -> 64 @56 at batch 32 (392 workgroups) the matrix pipes are busy 38 % of the time, the address units 39, the vector issue 36, LDS 13.
// Measured at s = 0.5 (float MFMA / split one after the other, stores in single lanes / this kernel, us; batch 32):  64 -> 64 @56 58 / 32 /
// 28.5 (130 TFLOP/s of float arithmetic), 128 -> 128 @28 55 / 31 / 25.8, 256 -> 256 @14 61 / 38 / 30.7, batch 16 384 -> 384 @12 88 / 31 / 29.1, one image
// of 128 -> 128 @28 32 / 14.5 / 12.2, batch 16 96 -> 256 @28 pointwise - / 11.9 / 9.0.  The same bits for the same tile.
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
// FUSED: with a shortcut sum.  Its groups of the dropped rows are asked for several passes at a time: one by one, each a round trip to
// memory, the tiles of few threads had become slower than the two groups that were chosen before (us, one by one / together:
// 4 x 244 -> 104 @70 pointwise 20.3 / 17.0; 64 x 32 -> 32 @28 10.8 / 9.05; 32 x 32 -> 256 @56 89.6 / 66.4).
// KS: the K tiles are divided among KS groups of wavefronts, each with LDS tiles of its own; the first group adds the others'
// sums in order and stores.  For launches with few workgroups, whose time is one K tile's latency after the other.
template <int BM, int BN, int KS, bool TAPS, int VEC_OUT, bool FUSED>
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
  uint32_t a_voff[A_LOADS];               // where the rows of that tile lie (TAPS: up to s_ci channels into the tap)
  const int w_step = p.k_tiles * D::BLOCK_BYTES;
  int s_w;                                // and its filters
  auto aim = [&](int off, uint32_t need) {
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j) a_voff[j] = (a_taps[j] & need) == need ? (uint32_t)(a_at[j] + off) : kOutOfRange;     // out of range: zeros
  };
  auto rewind = [&]() {
    s_kt = kt_lo;
    s_w = ((n0 / 32) * p.k_tiles + kt_lo) * D::BLOCK_BYTES;     // packed filters: [32 channels][K tile]
    if constexpr (TAPS) {
      const int tap = kt_lo * 32 / p.c_in;
      s_ci = kt_lo * 32 - tap * p.c_in;
      s_ky = tap / p.kw;
      s_kx = tap - s_ky * p.kw;
      s_off = s_kx * step_x + s_ky * step_y;
      aim(s_off, (1u << s_ky) | (1u << (8 + s_kx)));
    } else {
      ke = p.ktab[min(s_kt, p.k_tiles - 1) * 8 + lc];
    }
  };
  rewind();
  // Transfer number l of the next tile into slot `stage`: its filters, then its rows.  Past the end of a share the next one's
  // tile, past the end of the walk the last filters and rows of the last window row arrive; nothing uses them.
  constexpr int LOADS = A_LOADS + B_LOADS;
  auto fetch_filters = [&](unsigned char* dst, int at) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)dst, 16, (uint32_t)(lane * 16), at, 0, 0);
  };
  auto fetch_rows = [&](unsigned char* dst, uint32_t at) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)dst, 16, at, TAPS ? s_ci * 4 : 0, 0, 0);
  };
  auto issue_one = [&](int stage, auto l_c) {
    constexpr int l = decltype(l_c)::value;
    if constexpr (l < B_LOADS) {
      // (a wavefront without a unit of its own in the last round repeats the last one: the same bytes to the same place)
      const int u = min(wave + WAVES * l, B_UNITS - 1);
      constexpr int PER = D::BLOCK_BYTES / 1024;
      const int nb = u / PER, in = u - nb * PER;
      fetch_filters(smem + stage * STAGE_BYTES + A_BYTES + u * 1024, s_w + nb * w_step + in * 1024);
    } else {
      constexpr int j = l - B_LOADS;
      if constexpr (!TAPS && j == 0) aim(ke.off, (uint32_t)ke.dydx);
      fetch_rows(smem + stage * STAGE_BYTES + (wave * 8 + j * RPR) * kRowBytes, a_voff[j]);
    }
  };
  auto walk_on = [&]() {
    if (++s_kt < p.k_tiles) s_w += D::BLOCK_BYTES;
    if constexpr (TAPS) {
      s_ci += 32;
      if (s_ci == p.c_in) {
        s_ci = 0;
        s_off += step_x;
        if (++s_kx == p.kw) {
          s_kx = 0;
          s_ky = min(s_ky + 1, p.kh - 1);
          s_off = s_ky * step_y;
        }
        aim(s_off, (1u << s_ky) | (1u << (8 + s_kx)));
      }
    } else {
      ke = p.ktab[min(s_kt, p.k_tiles - 1) * 8 + lc];         // (used by the next call, a tile later)
    }
  };
  auto issue_tile = [&](int stage) {
    static_for<LOADS>([&](auto l_c) { issue_one(stage, l_c); });
    walk_on();
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

  struct Filters { v4i q[NI][3]; };
  struct Parts { v4i q[3]; };
  auto read_step = [&](auto stage_c, auto ks_c, v4i (&x)[2], Filters& f, unsigned more = 0) {
    constexpr int ST = decltype(stage_c)::value * STAGE_BYTES, ks = decltype(ks_c)::value;
    x[0] = lds_read16_big<ST>(frag_a[ks][0] + more);
    x[1] = lds_read16_big<ST>(frag_a[ks][1] + more);
    static_for<NI>([&](auto ni_c) {
      constexpr int at = ST + ks * 1024 + decltype(ni_c)::value * D::BLOCK_BYTES;
      f.q[decltype(ni_c)::value][0] = lds_read16_big<at>(frag_b + more);
      f.q[decltype(ni_c)::value][1] = lds_read16_big<at + 2048>(frag_b + more);
      f.q[decltype(ni_c)::value][2] = lds_read16_big<at + 4096>(frag_b + more);
    });
  };
  // the rows' fragments (behind them the filters' may still be on their way), or all of them, have landed; they pass through,
  // so nothing that uses them moves above
  auto rows_landed = [&](v4i (&x)[2]) { asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(x[0]), "+v"(x[1]) : "n"(3 * NI)); };
  auto all_landed = [&](Filters& f) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.q[0][0]), "+v"(f.q[0][1]), "+v"(f.q[0][2]));
    if constexpr (NI == 2) asm volatile("" : "+v"(f.q[NI - 1][0]), "+v"(f.q[NI - 1][1]), "+v"(f.q[NI - 1][2]));
  };
  // product number i of a K step
  auto product = [&](auto i_c, const Filters& f, const Parts& x) {
    constexpr int i = decltype(i_c)::value / NI, ni = decltype(i_c)::value % NI;
    constexpr int WQ[6] = {0, 1, 0, 1, 2, 0}, XQ[6] = {0, 0, 1, 1, 0, 2};
    Elem<kBF16>::mma(i == 0 ? acc[ni] : small[ni], f.q[ni][WQ[i]], x.q[XQ[i]]);
  };
  // The products of one K step and, behind them, the split of the next step's rows and the transfers of the next tile: four to
  // six vector instructions behind every MFMA, where the issue slot is free while the matrix unit works (a fifth costs nothing, an
  // eighth 12 cycles), dealt out so that none waits for the one before it (8 cycles instead of 5).
  constexpr int NP = 6 * NI, HEAD = NI == 2 ? 3 : 1, PIECES = 9;
  auto products = [&](const Filters& f, const Parts& x, v4i (&nx)[2], Parts& np, auto transfer) {
    float v[8], part[8];
    int pk[3][4];
    auto scale = [&](int e) { v[e] = __builtin_bit_cast(v4f, nx[e >> 2])[e & 3] * kPartScale; asm volatile("" : "+v"(v[e])); };
    auto pack = [&](int third, int i) {
      pk[third][i] = third == 2 ? (int)upper_halves(__builtin_bit_cast(uint32_t, v[2 * i]), __builtin_bit_cast(uint32_t, v[2 * i + 1]))
                                : (int)bf16_pair(v[2 * i], v[2 * i + 1]);
      asm volatile("" : "+v"(pk[third][i]));      // (not sunk to where the parts are used)
      np.q[third][i] = pk[third][i];
    };
    auto widen = [&](int third, int e) {
      part[e] = e & 1 ? bf16_hi((uint32_t)pk[third][e >> 1]) : bf16_lo((uint32_t)pk[third][e >> 1]);
      asm volatile("" : "+v"(part[e]));
    };
    auto rest = [&](int e) { v[e] -= part[e]; asm volatile("" : "+v"(v[e])); };
    auto piece = [&](auto c_c) {
      constexpr int c = decltype(c_c)::value;
      if constexpr (c == 0) for (int e = 0; e < 6; ++e) scale(e);
      if constexpr (c == 1) { scale(6); scale(7); for (int i = 0; i < 4; ++i) pack(0, i); }
      if constexpr (c == 2) for (int e = 0; e < 6; ++e) widen(0, e);
      if constexpr (c == 3) { widen(0, 6); widen(0, 7); for (int e = 0; e < 4; ++e) rest(e); }
      if constexpr (c == 4) { for (int e = 4; e < 8; ++e) rest(e); pack(1, 0); pack(1, 1); }
      if constexpr (c == 5) { pack(1, 2); pack(1, 3); for (int e = 0; e < 4; ++e) widen(1, e); }
      if constexpr (c == 6) { for (int e = 4; e < 8; ++e) widen(1, e); rest(0); rest(1); }
      if constexpr (c == 7) for (int e = 2; e < 8; ++e) rest(e);
      if constexpr (c == 8) for (int i = 0; i < 4; ++i) pack(2, i);
    };
    static_for<NP>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      product(i_c, f, x);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int l0 = i * LOADS / NP, l1 = (i + 1) * LOADS / NP;
      static_for<l1 - l0>([&](auto l_c) { transfer(std::integral_constant<int, l0 + decltype(l_c)::value>{}); });
      if constexpr (i == HEAD - 1) rows_landed(nx);
      if constexpr (i >= HEAD) {
        constexpr int c0 = (i - HEAD) * PIECES / (NP - HEAD), c1 = (i - HEAD + 1) * PIECES / (NP - HEAD);
        static_for<c1 - c0>([&](auto c_c) { piece(std::integral_constant<int, c0 + decltype(c_c)::value>{}); });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  auto fill_zeros = [&]() {
    const int valid = min(BN, p.c_out - n0) / 4;
    if (zc >= valid) return;
    unsigned char* ybase = reinterpret_cast<unsigned char*>(y) + (int64_t)n0 * 4 + zc * 16;
    auto passes = [&](int r0, const unsigned (&keep)[ZB]) {
      v4i v[ZB];
      auto each = [&](auto fn) {
#pragma unroll
        for (int u = 0; u < ZB; ++u) {
          const int r = r0 + u * RPI;
          if (r < z_hi && keep[u] == 0) fn(v[u], (int64_t)r * p.c_out * 4);
        }
      };
      if constexpr (FUSED) {
        const unsigned char* res = static_cast<const unsigned char*>(p.residual) + (int64_t)n0 * 4 + zc * 16;
        each([&](v4i& g, int64_t at) { g = *reinterpret_cast<const v4i*>(res + at); });
        __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0), said once: the compiler would have the K loop wait for them
        each([&](v4i& g, int64_t at) { *reinterpret_cast<v4i*>(ybase + at) = shortcut_alone<kF32>(g, p.residual_relu); });
      } else {
        each([&](v4i&, int64_t at) { *reinterpret_cast<v4i*>(ybase + at) = v4i{0, 0, 0, 0}; });
      }
    };
    passes(z_lo + zr, mk);
    for (int r0 = z_lo + zr + ZB * RPI; r0 < z_hi; r0 += ZB * RPI) {
      unsigned m[ZB];
#pragma unroll
      for (int u = 0; u < ZB; ++u) m[u] = mask_of(min(r0 + u * RPI, z_hi - 1));
      passes(r0, m);
    }
  };

  using Zero = std::integral_constant<int, 0>;
  using One = std::integral_constant<int, 1>;
  const int n_kt = kt_hi - kt_lo;
  auto arrive = [&]() {
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();        // the tile has landed for every wavefront, and all have read the one before
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto pipeline = [&]() {
    Filters w0, w1;
    Parts p0, p1;
    v4i x[2];
    issue_tile(0);
    arrive();
    if (steps > 1) issue_tile(1);
    read_step(Zero{}, Zero{}, x, w0);
    rows_landed(x);
    {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = __builtin_bit_cast(v4f, x[e >> 2])[e & 3];
      split3(v, p0.q[0], p0.q[1], p0.q[2]);
    }
    all_landed(w0);
    // a tile of the share, in slot S; the first half of the next one is read, and split, behind its second half
    auto tile = [&](auto stage_c) {
      constexpr int S = decltype(stage_c)::value;
      read_step(stage_c, One{}, x, w1);
      products(w0, p0, x, p1, [](auto) {});
      all_landed(w1);
      arrive();
      // (behind the last tile of a share that is shorter than another this reads what lies there, and nothing uses it)
      read_step(std::integral_constant<int, S ^ 1>{}, Zero{}, x, w0);
      products(w1, p1, x, p0, [&](auto l_c) { issue_one(S, l_c); });
      walk_on();
      all_landed(w0);
    };
    if (steps > 1) tile(Zero{});
    if (p.zero_fill) fill_zeros();        // (under the products of a tile's first half: the next arrive waits for the stores too)
    int i = 1;
#pragma unroll 1
    for (; i + 2 < steps; i += 2) {
      tile(One{});
      tile(Zero{});
    }
    if (i + 1 < steps) tile(One{});
    // The last tile: nothing follows that would have to be asked for, waited for or split (us, like the others / so: fused, one image of
    // 32 -> 64 @28 pointwise 7.30 / 6.94, 64 x 32 -> 32 @28 11.2 / 10.9; plain, one image of 128 -> 128 @28 12.8 / 12.2, dense 32 x 32 -> 256
    // @56 pointwise 45.9 / 42.8).
    if (KS == 1 || n_kt == steps) {
      const unsigned at = (steps & 1) ? 0u : (unsigned)STAGE_BYTES;
      read_step(Zero{}, One{}, x, w1, at);
      products(w0, p0, x, p1, [](auto) {});
      all_landed(w1);
      static_for<NP>([&](auto i_c) { product(i_c, w1, p1); });
    }
    wait_vmcnt<0>();
  };
  // the same sums on the float MFMA
  auto careful_tile = [&](auto stage_c, int i) {
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue_tile(decltype(stage_c)::value ^ 1);
    if (KS > 1 && i >= n_kt) return;
    static_for<2>([&](auto ks_c) {
      v4i x[2];
      Filters f;
      read_step(stage_c, ks_c, x, f);
      rows_landed(x);
      all_landed(f);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          auto part = [&](int q) {
            const uint32_t v = (uint32_t)f.q[ni][q][e >> 1];
            return (e & 1) ? bf16_hi(v) : bf16_lo(v);
          };
          acc[ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(join3(part(0), part(1), part(2)), __builtin_bit_cast(v4f, x[e >> 2])[e & 3], acc[ni], 0, 0, 0);
        }
    });
  };
  auto careful_walk = [&]() {
    issue_tile(0);
#pragma unroll 1
    for (int i = 0; i < steps; i += 2) {
      careful_tile(Zero{}, i);
      if (i + 1 < steps) careful_tile(One{}, i + 1);
    }
    wait_vmcnt<0>();
  };
  auto finish = [&](auto careful_c) {          // the sums of the groups together
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
  clear();
  pipeline();
  finish(std::false_type{});
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
    clear();
    careful_walk();
    finish(std::true_type{});
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
                                            FUSED ? static_cast<const float*>(p.residual) : nullptr, FUSED ? p.residual_relu : 0);
    }
  }
}

template <int BM, int BN, int KS, bool TAPS, int VEC_OUT>
hipError_t igemm_split_launch(const ConvParams& p, hipStream_t stream) {
  constexpr size_t lds = split_lds_bytes<BM, BN, KS>();
  auto kern = p.residual ? igemm_split_kernel<BM, BN, KS, TAPS, VEC_OUT, true> : igemm_split_kernel<BM, BN, KS, TAPS, VEC_OUT, false>;
  static std::atomic<bool> attr_set[2] = {{false}, {false}};
  std::atomic<bool>& set = attr_set[p.residual ? 1 : 0];
  if (lds > 64 * 1024 && !set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    set = true;
  }
  const int nwg = p.m_tiles * p.n_tiles;
  hipLaunchKernelGGL(kern, dim3(((nwg + 7) / 8) * 8), dim3(2 * BM * KS), lds, stream, p);
  return hipGetLastError();
}

// the kernel of tile bm x bn with K in `groups` shares, or null (igemm_split.hip)
LaunchFn split_kernel(int bm, int bn, int groups, bool taps, int vec_out);

}  // namespace sc
