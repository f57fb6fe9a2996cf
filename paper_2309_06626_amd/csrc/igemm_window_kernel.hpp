// Tiled masked-convolution kernel for 3 x 3 and 5 x 5 windows at stride 1 (16-bit NHWC, Cin and Cout multiples of 8): every input pixel of a tile
// passes into LDS once, the filters go straight into registers.
//
// What bounds the tiled kernels whose K tiles pass a ring in LDS (igemm_buf_kernel), taken apart by leaving one thing out at a time
// (128 x 128, 18 K tiles of 32 KB, 8.8 us): transfers alone 5.4 (46 to 56 bytes a clock come through the L1 path, however many are on
// their way), LDS reads alone 4.1, products alone 4.6; they do not hide each other, because eight wavefronts meet at a barrier every
// K tile.  Here a K tile costs 22 KB of transfers instead of 32 (a pixel's nine uses share one), half of the LDS writes, and no barrier:
//   * the slab: for a chunk of 64 channels, the run of virtual zero-padded pixels under the windows of the tile's rows, so that a tap is
//     one displacement for all of them; the next chunk's slab lands while this one is contracted, and wavefronts meet once a chunk;
//   * filters, packed in fragment order (repack_kernel), nine fragments a wavefront (five of 25) on their way at any time;
//   * wavefronts stand side by side over the channels, so that no two load the same filters, and share K where that leaves some over:
//     a K group takes every KG-th step of 16 channels, and the groups' sums are added through LDS in order at the end.
// A pixel takes nine 16-byte groups in LDS, of which eight hold channels: reads of sixteen consecutive pixels touch every bank once.  The
// kept rows of a mask are not consecutive, and which ones stand side by side is chosen for that (below); a fifth of the rows of a 64-row tile
// finds every set of its residue full and takes a hole all the same, and 43 % of the LDS cycles are conflict cycles (64 x 512 -> 512 @7).
//
// Measured at s = 0.5 in bf16, launches behind each other on one card, the tiled kernels / this one, us: 64 x 512 -> 512 @7 20.7 / 15.3 (dense
// 28.6 / 20.6), 64 x 256 -> 256 @14 17.6 / 15.2 (21.8 / 20.1), 16 x 256 -> 256 @14 12.7 / 9.6 (13.0 / 8.7), 64 x 128 -> 128 @28 15.8 / 14.5
// (22.2 / 19.1), 1 x 128 -> 128 @28 9.6 / 7.1 (8.9 / 6.4), 2 x 512 -> 48 @8x6 21.3 / 11.5 (21.2 / 11.1), 5 x 5, 1 x 360 -> 104 @19x24 73 / 16
// (73 / 15).  Of the 12 us a workgroup of the first takes, 1.8 pass before the first row number is known, 1.5 until the first slab has
// landed, 0.6 go into the groups' sums and as much into the stores.
// Tried and left out: reads of the next tap ahead of all products of this one (12.7 -> 13.0 of a loop), the zeros of dropped rows between
// the products of the first pass (their acknowledgements hold up the filters' waits: 7.4 -> 8.0).
//
// Workgroup = BM kept rows x BN channels, eight wavefronts; the epilogue is that of the other tiled kernels.  The zeros of the dropped rows are
// shared out by rows of the map, as many for every tile wherever its kept rows lie: a tile that wrote those up to the next tile's first row,
// as in the other kernels, had them all where half of a map is dropped in one piece (38 x 160 -> 64 @21x19 with the
// lower half dropped 30.4 us, now 8.1; as many rows dropped here and there 8.2).
#pragma once
#include <type_traits>

#include "igemm_buf_kernel.hpp"

namespace sc {

constexpr int kWinChunk = 64;                            // channels of a slab
constexpr int kWinPitch = 2 * kWinChunk + 16;            // bytes of a pixel in LDS: nine 16-byte groups, the last one unused
constexpr int kWinGroups = kWinPitch / 16;
constexpr int kWinMostPixels = 512;                      // of a slab (a thread decodes each)
constexpr int kWinRounds = (kWinMostPixels * kWinPitch + 8191) / 8192;      // transfers of the whole workgroup for a slab at most

template <int BM, int BN> struct WinDims {
  static constexpr int WAVES_M = BM == 256 ? 2 : 1, WAVES_N = BN / 32, KG = 8 / (WAVES_M * WAVES_N);
  static constexpr int MI = BM / WAVES_M / 32;
  static constexpr int PASSES = 4 / KG;                  // of a wavefront over the taps of a chunk, one K step of 16 channels each
  static constexpr int FIN = KG < MI ? KG : MI;          // K groups that store
  static constexpr int MINE = MI / FIN;                  // 32 x 32 blocks such a wavefront stores
  static constexpr int ZERO_ROWS = BM + 64;              // dropped rows whose zeros go out before the K loop
  static constexpr size_t sums_bytes() { return KG > 1 ? (size_t)MI * 8 * 4096 : 0; }
  static constexpr size_t tail_bytes() { return BM * 12 + BN * 4 + kWinMostPixels * 4 + 128 + ZERO_ROWS * 4; }
};
template <int BM, int BN> size_t win_lds_bytes(int slab_bytes, int chunks) {
  using D = WinDims<BM, BN>;
  const size_t slabs = (size_t)slab_bytes * (chunks > 1 ? 2 : 1);
  return (slabs > D::sums_bytes() ? slabs : D::sums_bytes()) + D::tail_bytes();
}

template <int DT, int BM, int BN, int KS>      // KS x KS windows
__global__ __launch_bounds__(512) void igemm_window_kernel(const ConvParams p) {
  using E = Elem<DT>;
  using T = typename E::T;
  using D = WinDims<BM, BN>;
  constexpr int EB = sizeof(T), MI = D::MI, KG = D::KG;
  constexpr int TAPS = KS * KS, AHEAD = KS == 3 ? 9 : 5;      // filter fragments a wavefront has on their way: a whole part of a pass
  static_assert(TAPS % AHEAD == 0, "whole turns");
  constexpr int CPR = BN * EB / 16, RPI = 512 / CPR;      // 16-byte groups of a row slice, dense rows a pass of the zero fill covers
  constexpr int NZ = WinDims<BM, BN>::ZERO_ROWS / RPI;    // passes that go out before the K loop
  static_assert(EB == 2 && D::WAVES_M * D::WAVES_N * KG == 8, "16-bit operands, eight wavefronts");

  extern __shared__ __align__(16) unsigned char smem[];
  const int chunks = (p.c_in + kWinChunk - 1) / kWinChunk, last_ci = p.c_in - (chunks - 1) * kWinChunk;      // channels of the last chunk
  const size_t slabs = (size_t)p.slab_bytes * (chunks > 1 ? 2 : 1);
  int32_t* s_rows = reinterpret_cast<int32_t*>(smem + (slabs > D::sums_bytes() ? slabs : D::sums_bytes()));      // [BM] row of y
  int32_t* s_corner = s_rows + BM;                        // [BM] LDS byte of the window's first pixel
  float* s_bias = reinterpret_cast<float*>(s_corner + BM);      // [BN]
  int32_t* s_px = reinterpret_cast<int32_t*>(s_bias + BN);      // [kWinMostPixels] byte offset of a slab pixel in x
  int32_t* s_count = s_px + kWinMostPixels;                     // [16] rows of a residue, then the rows beyond the last set
  int32_t* s_drops = s_count + 24;                              // [8] dropped rows that a wavefront has found
  int32_t* s_hole = s_count + 32;                               // [BM]
  int32_t* s_drop = s_hole + BM;                                // [ZERO_ROWS] the first dropped rows of this workgroup's share

  const int nwg = p.m_tiles * p.n_tiles;
  const int per_xcd = (nwg + 7) >> 3;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= nwg) return;
  const int tile_m = tile / p.n_tiles, tile_n = tile - tile_m * p.n_tiles;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int pos = wave % (D::WAVES_M * D::WAVES_N), kg = wave / (D::WAVES_M * D::WAVES_N);
  const int wm0 = (pos / D::WAVES_N) * (MI * 32), wn0 = (pos % D::WAVES_N) * 32;
  const int fp = lane & 31, fh = lane >> 5;
  const int hp = p.slab_hp, wp = p.slab_wp;
  T* __restrict__ y = static_cast<T*>(p.y);

  // ---- first round trip: row numbers, the mask of this workgroup's share of the map, bias; the first filters need none of them ----------------
  const int i_last = min(m0 + BM, p.rows) - 1;
  const int r_first = p.row_idx ? p.row_idx[m0] : m0;
  const int r_last = p.row_idx ? p.row_idx[i_last] : i_last;
  const int z_lo = tile_m * p.zero_share, z_hi = (int)min((int64_t)z_lo + p.zero_share, (int64_t)p.m_total);
  auto mask_of = [&](int r) { return (int)p.mask[p.mask_spatial ? r - fast_div(r, p.div_howo_mul, p.div_howo_shift) * p.ho_wo : r]; };
  int keeps[2] = {0, 0};                                 // mask of rows z_lo + t and z_lo + 512 + t
  if (p.zero_fill) {
    keeps[0] = mask_of(min(z_lo + t, p.m_total - 1));
    if (p.zero_share > 512) keeps[1] = mask_of(min(z_lo + 512 + t, p.m_total - 1));
  }
  int my_row = 0;                                        // row of tile row t
  if (t < BM) {
    const int i = min(m0 + t, p.rows - 1);
    my_row = p.row_idx ? p.row_idx[i] : i;
  }
  float bias_v = 0.0f;
  if (t < BN && p.bias && n0 + t < p.c_out) bias_v = p.bias[n0 + t];

  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)p.x_bytes, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.wp), 0, (int)p.w_bytes, kBufferWord3);
  const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)0x7fffffff, kBufferWord3);
  typedef __attribute__((address_space(3))) void lds_void;

  // Filters, packed in the order in which the matrix unit takes them: [32 channels][chunk][K step][tap][lane] of 16 bytes.  A
  // wavefront of K group kg takes K steps kg, kg + KG, ... of a chunk, one pass over the taps each; AHEAD fragments are on their way at any time.
  const int n_pass = chunks * D::PASSES;
  const int nb = min((n0 + wn0) >> 5, (p.c_out - 1) >> 5);
  const uint32_t w_lane = (uint32_t)(lane * 16);
  auto pass_at = [&](int pass) {
    const int q = min(pass, n_pass - 1);
    return ((nb * chunks + q / D::PASSES) * 4 + kg + KG * (q % D::PASSES)) * (TAPS * 1024);
  };
  v4i bf[AHEAD];
  {
    const int at = pass_at(0);
#pragma unroll
    for (int tap = 0; tap < AHEAD; ++tap) bf[tap] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, w_lane, at + tap * 1024, 0));
  }

  const int zc = t % CPR, zr = t / CPR;
  const bool fill_ahead = p.zero_fill && !p.residual && (int64_t)p.m_total * p.c_out * EB < ((int64_t)1 << 31);      // (byte offsets of a buffer)
  // ---- the slab: a run of pixels of the images with their zero margins (virtual rows of wp pixels, hp of them an image), from the
  // corner of the first row's window to the end of the last one's.  A tap is then one displacement, the same for every row. -----------
  auto corner = [&](int r) {
    const int n = fast_div(r, p.div_howo_mul, p.div_howo_shift), rem = r - n * p.ho_wo;
    const int oy = fast_div(rem, p.div_wo_mul, p.div_wo_shift);
    return (n * hp + oy) * wp + rem - oy * p.wo;
  };
  const int v_lo = corner(r_first);
  const int slab_px = min(corner(r_last) + (KS - 1) * wp + KS - v_lo, kWinMostPixels);
  const int rounds = min((slab_px * kWinPitch + 8191) >> 13, p.slab_bytes >> 13);
  {
    const int v = v_lo + t;
    const int vr = fast_div(v, p.div_wp_mul, p.div_wp_shift), n = fast_div(vr, p.div_hp_mul, p.div_hp_shift);
    const int iy = vr - n * hp - p.ph, ix = v - vr * wp - p.pw;
    const bool ok = t < slab_px && (unsigned)iy < (unsigned)p.h && (unsigned)ix < (unsigned)p.w;
    s_px[t] = ok ? (((n * p.h + iy) * p.w + ix) * p.c_in) * EB : (int)kOutOfRange;
  }
  const int my_px = t < BM ? corner(my_row) - v_lo : 0;
  if (t < 32) s_count[t] = 0;
  if (t < BN) s_bias[t] = bias_v;
  __syncthreads();
  uint32_t s_voff[kWinRounds], in_last = 0;               // (bit j: the group lies inside the last chunk)
#pragma unroll
  for (int j = 0; j < kWinRounds; ++j) {
    const int g = j * 512 + t, px = g / kWinGroups, in = g - px * kWinGroups;
    const uint32_t at = px < kWinMostPixels ? (uint32_t)s_px[min(px, kWinMostPixels - 1)] : kOutOfRange;
    s_voff[j] = in < kWinGroups - 1 && at != kOutOfRange ? at + in * 16 : kOutOfRange;      // out of range: LDS gets zeros
    in_last |= (in * 8 < last_ci ? 1u : 0u) << j;
  }
  auto ask_slab = [&](int chunk) {
    unsigned char* dst = smem + (chunk & 1) * p.slab_bytes + wave * 1024;
    const uint32_t in_chunk = chunk + 1 < chunks ? ~0u : in_last;
#pragma unroll
    for (int j = 0; j < kWinRounds; ++j) {
      const uint32_t voff = in_chunk >> j & 1u ? s_voff[j] : kOutOfRange;
      if (j < rounds) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)(dst + j * 8192), 16, voff, chunk * kWinChunk * EB, 0, 0);
    }
  };
  ask_slab(0);

  // ---- rows are dealt to lanes while the slab is on its way.  Sixteen lanes read 16 bytes each in one go unless two of them meet in a
  // bank group, i.e. their pixels are congruent modulo 16 (the pitch is an odd number of groups).  The k-th row of a residue goes to the
  // k-th set of sixteen lanes; rows beyond the last set fill its holes, from the last set on, so that few sets read twice. ------------
  auto lds_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  constexpr int SETS = BM / 16;
  int place = -1, spare = 0;
  int n_drop = 0;                                         // dropped rows among the first 1 024 of the share
  unsigned long long drop_bits[2] = {0, 0};
  if (p.zero_fill) {
    asm volatile("" : "+v"(keeps[0]), "+v"(keeps[1]));    // (waited for here, behind the slab's transfers)
    drop_bits[0] = __ballot(keeps[0] == 0 && z_lo + t < z_hi);
    drop_bits[1] = __ballot(keeps[1] == 0 && z_lo + 512 + t < z_hi);
    if (lane == 0) s_drops[wave] = (int)__popcll(drop_bits[0]) | (int)__popcll(drop_bits[1]) << 16;
  }
  if (t < BM) {
    const int k = atomicAdd(&s_count[my_px & 15], 1);
    if (k < SETS) place = k * 16 + (my_px & 15);
    else spare = atomicAdd(&s_count[16], 1);
  }
  lds_barrier();
  if (wave == 0) {
    int found = 0;
#pragma unroll
    for (int i = SETS - 4; i >= 0; i -= 4) {
      const int k = i + (lane >> 4);
      const bool hole = k >= s_count[lane & 15];
      const unsigned long long b = __ballot(hole);
      if (hole) s_hole[found + __popcll(b & ((1ull << lane) - 1ull))] = k * 16 + (lane & 15);
      found += __popcll(b);
    }
  }
  if (p.zero_fill) {
    int in_front[2] = {0, 0}, all = 0;                    // (the counts of rows z_lo + 0 .. 511 and of the 512 behind them in halves of a word)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i == wave) in_front[0] = in_front[1] = all;
      all += s_drops[i];
    }
    n_drop = (all & 0xffff) + (all >> 16);
    in_front[0] &= 0xffff;
    in_front[1] = (in_front[1] >> 16) + (all & 0xffff);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = in_front[u] + (int)__popcll(drop_bits[u] & ((1ull << lane) - 1ull));
      if ((drop_bits[u] >> lane & 1) && i < D::ZERO_ROWS) s_drop[i] = z_lo + u * 512 + t;
    }
  }
  const int n_list = min(n_drop, D::ZERO_ROWS);
  lds_barrier();
  if (t < BM) {
    if (place < 0) place = s_hole[spare];
    s_rows[place] = m0 + t >= p.rows ? -1 : p.y_compact ? m0 + t : my_row;
    s_corner[place] = my_px * kWinPitch;
  }
  lds_barrier();
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  unsigned a_base[MI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) a_base[mi] = lds0 + (unsigned)s_corner[wm0 + mi * 32 + fp] + (unsigned)((2 * kg + fh) * 16);

  // ---- zeros of the dropped rows of this workgroup's share (Alg. 2, mask == 0 branch), the first passes -------------------------
  if (fill_ahead) {
    const int valid = (min(BN, p.c_out - n0) * EB) >> 4;
#pragma unroll
    for (int u = 0; u < NZ; ++u) {      // unconditional (out of range where nothing is to be stored): their number is counted on below
      const int i = zr + u * RPI;
      const int r = s_drop[i];
      unsigned at = i < n_list && zc < valid ? (unsigned)(r * p.c_out + n0) * EB + zc * 16 : kOutOfRange;
      asm volatile("" : "+v"(at));
      __builtin_amdgcn_raw_buffer_store_b128(v4i{0, 0, 0, 0}, ry, at, 0, 0);
    }
  }

  floatx16 acc[MI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[mi][v] = 0.0f;

  if (fill_ahead) wait_vmcnt<NZ>();
  else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // ---- K loop: a chunk's slab lands while the one before it is contracted; wavefronts meet once a chunk ------------------------------
  const int tap_row = wp * kWinPitch;
  int pass = 0;
#pragma unroll 1
  for (int chunk = 0; chunk < chunks; ++chunk) {
    if (chunk + 1 < chunks) ask_slab(chunk + 1);
    const unsigned slab_at = (unsigned)((chunk & 1) * p.slab_bytes);
#pragma unroll 1
    for (int q = 0; q < D::PASSES; ++q, ++pass) {
      if (chunk + 1 == chunks && (kg + KG * q) * 16 >= last_ci) break;      // (no channels left in the last chunk)
      const int this_at = pass_at(pass), next_at = pass_at(pass + 1);
      const unsigned from = slab_at + (unsigned)(q * KG * 32);
      v4i xa[3][MI];
      auto read = [&](int tap, int mi) {
        xa[tap % 3][mi] = lds_read16_at<0>(a_base[mi] + from + (unsigned)((tap / KS) * tap_row + (tap % KS) * kWinPitch));
      };
#pragma unroll
      for (int tap = 0; tap < 2; ++tap)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) read(tap, mi);
#pragma unroll
      for (int tap = 0; tap < TAPS; ++tap) {      // a fragment of the tap two ahead is asked for behind every product
        if (tap + 1 < TAPS) wait_frags<MI>(xa[tap % 3]);
        else wait_frags<0>(xa[tap % 3]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
          E::mma(acc[mi], bf[tap % AHEAD], xa[tap % 3][mi]);
          __builtin_amdgcn_sched_barrier(0);
          if (tap + 2 < TAPS) read(tap + 2, mi);
          __builtin_amdgcn_sched_barrier(0);
        }
        const int next = tap + AHEAD < TAPS ? this_at + (tap + AHEAD) * 1024 : next_at + (tap + AHEAD - TAPS) * 1024;
        bf[tap % AHEAD] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, w_lane, next, 0));
      }
    }
    if (chunk + 1 < chunks) {
      // the next slab has landed when at most the filters asked for since are on their way, a pass at least
      __builtin_amdgcn_sched_barrier(0);
      wait_vmcnt<AHEAD>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- the K groups' sums, in order; each of the first FIN groups ends up with a share of the blocks ----------------------------------
  floatx16 sum[D::MINE];
  if constexpr (KG == 1) {
#pragma unroll
    for (int b = 0; b < MI; ++b) sum[b] = acc[b];
  } else {
    __syncthreads();                                          // every wavefront has left the slabs
    v4f* part = reinterpret_cast<v4f*>(smem) + lane;          // [K group][position][block][4][64]
    auto at = [&](int g, int b, int q) { return (((g * (8 / KG) + pos) * MI + b) * 4 + q) * 64; };
#pragma unroll
    for (int b = 0; b < MI; ++b)
      if (b / D::MINE != kg) {
#pragma unroll
        for (int q = 0; q < 4; ++q) part[at(kg, b, q)] = v4f{acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]};
      } else {
        sum[b % D::MINE] = acc[b];
      }
    __syncthreads();
    if (kg < D::FIN) {
      floatx16 total[D::MINE];
#pragma unroll
      for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int b = 0; b < D::MINE; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            v4f v;
            if (g == kg) v = v4f{sum[b][4 * q], sum[b][4 * q + 1], sum[b][4 * q + 2], sum[b][4 * q + 3]};
            else v = part[at(g, kg * D::MINE + b, q)];
#pragma unroll
            for (int e = 0; e < 4; ++e) total[b][4 * q + e] = g == 0 ? v[e] : total[b][4 * q + e] + v[e];
          }
#pragma unroll
      for (int b = 0; b < D::MINE; ++b) sum[b] = total[b];
    }
  }

  // ---- zero fill: the rows behind the listed ones, and those too where they have not had their zeros yet (a shortcut is fused) --------
  if (p.zero_fill && (!fill_ahead || n_drop > n_list || z_hi - z_lo > 1024)) {
    const int valid = (min(BN, p.c_out - n0) * EB) >> 4;
    if (zc < valid) {
      const int64_t at0 = (int64_t)n0 * EB + zc * 16;
      unsigned char* ybase = reinterpret_cast<unsigned char*>(y) + at0;
      if (!fill_ahead) {
        const unsigned char* rbase = static_cast<const unsigned char*>(p.residual) + at0;
        v4i g[NZ];
#pragma unroll
        for (int u = 0; u < NZ; ++u) {
          g[u] = v4i{0, 0, 0, 0};
          if (p.residual && zr + u * RPI < n_list) g[u] = *reinterpret_cast<const v4i*>(rbase + (int64_t)s_drop[zr + u * RPI] * p.c_out * EB);
        }
#pragma unroll
        for (int u = 0; u < NZ; ++u)
          if (zr + u * RPI < n_list)
            sc_store16(reinterpret_cast<v4i*>(ybase + (int64_t)s_drop[zr + u * RPI] * p.c_out * EB), p.residual ? shortcut_alone<DT>(g[u], p.residual_relu) : g[u]);
      }
      const int z_from = n_drop > n_list ? s_drop[D::ZERO_ROWS - 1] + 1 : min(z_lo + 1024, z_hi);
      for (int r0 = z_from + zr; r0 < z_hi; r0 += 4 * RPI) {
        int m4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          m4[u] = mask_of(min(r0 + u * RPI, z_hi - 1));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = r0 + u * RPI;
          if (r < z_hi && m4[u] == 0) {
            const int64_t at = (int64_t)r * p.c_out * EB;
            sc_store16(reinterpret_cast<v4i*>(ybase + at), dropped_row_group<DT>(p.residual, at0 + at, p.residual_relu));
          }
        }
      }
    }
  }

  // ---- epilogue ------------------------------------------------------------------------------------------------------------------
  const int c0 = n0 + wn0 + 16 * fh;
  if (kg < D::FIN && c0 < p.c_out) {
#pragma unroll
    for (int b = 0; b < D::MINE; ++b) {
      const int rr = s_rows[wm0 + ((KG == 1 ? 0 : kg * D::MINE) + b) * 32 + fp];
      if (rr < 0) continue;
      store_kept_block_res<DT>(sum[b], rr, c0, y, p.bias ? s_bias + (c0 - n0) : nullptr, 0, p.relu, p.vec_out, p.c_out, p.ho_wo, 0, 0, 0,
                               static_cast<const T*>(p.residual), p.residual_relu);
    }
  }
}

template <int DT, int BM, int BN, int KS>
hipError_t igemm_window_launch(const ConvParams& p, hipStream_t stream) {
  // (p.splits: at most one workgroup a compute unit, so that none waits beside an idle one: 64 x 512 -> 512 @7 takes 7 % less)
  size_t lds = win_lds_bytes<BM, BN>(p.slab_bytes, (p.c_in + kWinChunk - 1) / kWinChunk);
  if (p.splits == 1 && lds < 81 * 1024) lds = 81 * 1024;
  auto kern = igemm_window_kernel<DT, BM, BN, KS>;
  static std::atomic<bool> attr_set{false};
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int nwg = p.m_tiles * p.n_tiles;
  hipLaunchKernelGGL(kern, dim3((nwg + 7) / 8 * 8), dim3(512), lds, stream, p);
  return hipGetLastError();
}

// the window kernel of tile bm x bn for a 16-bit dtype and ks x ks windows, or null; LDS it needs
LaunchFn window_kernel(int dtype, int ks, int bm, int bn);
size_t window_lds_bytes(int bm, int bn, int slab_bytes, int chunks);

}  // namespace sc
