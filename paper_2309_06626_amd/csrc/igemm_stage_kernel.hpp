// Tiled masked-convolution kernel whose operand tiles pass through registers on their way into LDS.
//
// Serves the layers whose rows cannot be transferred as they lie in memory:
//   * float operands.  The float MFMA runs at a sixteenth of the 16-bit rate, so a float tile is staged as three bf16
//     parts of the value times 2^24: x1 = bf16(2^24 x), x2 = bf16(2^24 x - x1), x3 = 2^24 x - x1 - x2, both rounded to
//     nearest.  The split is exact for every float, subnormal ones included: the 24 significand bits go into three times
//     eight, |x2| <= 2^-8 |2^24 x|, |x3| <= 2^-17 |2^24 x|, and the last bit of the smallest float is 2^-125 after the
//     scaling, inside the range of a normal bf16 (unscaled, later parts of operands below 2^-110 would fall out of it).
//     Of the nine products of a pair of parts the six largest are contracted: x1w1, x1w2, x2w1, x2w2, x1w3, x3w1.  What is
//     left out (x2w3, x3w2, x3w3) is at most 2^-24 (1 + 2^-10) of |x w|, about the half unit of one rounding, and of no
//     common sign.  The products themselves are exact in the matrix unit, x1w1 and the five small ones go to accumulators
//     of their own, and one MFMA adds sixteen of them, so fewer roundings happen than with the float MFMA (two per addition
//     step).  The sums are scaled back by 2^-48.  A value that is not finite makes its remainder not-a-number and with it
//     the sums it enters; operands from 2^104 on, and sums from 2^80 on, become infinite by the scaling: a workgroup whose
//     sums are not all finite contracts its tile again with the float MFMA on the unsplit values (`careful` pass), which
//     gives the infinities of the plain sum and no others.
//   * NHWC channel counts that are no multiple of the 16-byte group (a pruned network run as it is): a group is an
//     element-aligned 16-byte load inside one pixel.  The last group of a pixel is the one that ENDS at its last
//     channel; the entries it repeats meet zero filter entries, and the careful pass clears them.
//   * channels-first tensors, and pixels with fewer channels than a group: one load per entry.  A wavefront's lanes are
//     64 rows of the tile and the entry is the same for all of them, so what a lane adds is one 32-bit offset, and a
//     load touches the few cache lines that hold the row's neighbours along a map row.
//
// K is cut into chunks of eight entries; a K tile is four chunks of floats or eight of a 16-bit type.  In LDS a tile
// lies in the order in which the MFMA reads it -- [part][32 rows][K step][lane] of 16 bytes -- with the row exchanged by
// a multiple of the chunk number so that the sixteen lanes of a write phase hit sixteen different bank groups.  The
// filters are packed in the same order at plan time, so their transfer is a plain copy.
//
// What bounds it: no unit alone.  The rows of a K tile pass LDS twice (written by the threads that fetched them, read by the
// wavefronts); the split and the stores of the next tile go out behind the products of this one where that pays; the address units
// are the busiest, 49 % of the time channels first in float (one load per entry), 57 % with the element-aligned groups of
// 102 channels, next to 26 and 14 % of the matrix pipes, 20 % of the vector issue and 14 and 19 % of LDS (counters).  Row loads
// run two tiles ahead in registers; the table that says where they go runs three ahead, because waiting for a load waits for
// all that were issued before it, and is read by scalar loads where a wavefront shares its entries.  The filters need no
// registers: they go from memory to LDS as they lie, a tile ahead.
// Measured at s = 0.5 (element gather / all through registers / this kernel, us): 32 x 128 -> 128 @28 channels first in float
// 115 / 45 / 35.4, in bf16 84 / 27.5 / 20.9, 32 x 51 -> 64 @28 in bf16 - / 19.6 / 13.8; at s = 0.3 64 x 102 -> 102 @28 in fp16
// 98 / 27.5 / 25.5, 51 -> 51 @56 110 / 44 / 40, 410 -> 410 @7 186 / 27 / 22.5.
//
// Workgroup = BM kept rows x BN channels, four wavefronts (or KG groups of four); zero-fill ownership and the order of the
// epilogue are those of the other tiled kernels.
#pragma once
#include "igemm_buf_kernel.hpp"

namespace sc {

// fn(integral_constant 0), ..., fn(integral_constant N - 1)
template <int N, typename F> __device__ __forceinline__ void static_for(F fn) {
  if constexpr (N > 0) {
    static_for<N - 1>(fn);
    fn(std::integral_constant<int, N - 1>{});
  }
}

// how window entries reach a tile
enum StageGather { kStageGroups = 0,         // NHWC, Cin a multiple of the 16-byte group
                   kStageRaggedGroups = 1,   // NHWC, Cin at least one group, not a multiple of it
                   kStageChunks = 2,         // one load per entry, eight channels of a tap per table entry (NCHW, Cin % 8 == 0)
                   kStageEntries = 3 };      // one load per entry, a table entry each (any layout, any Cin)

constexpr uint32_t kStageNoTap = 1u << 30;       // a validity bit no row has: entries beyond the last one
constexpr uint32_t kStageTail = 1u << 31;        // the group repeats entries of the one before it

template <int DT> struct StageDims {
  static constexpr int PARTS = DT == kF32 ? 3 : 1;
  static constexpr int CHUNKS = DT == kF32 ? 4 : 8;        // chunks of eight entries in a K tile
  static constexpr int KSTEPS = CHUNKS / 2;                // 32x32x16 steps
  static constexpr int SWZ = 16 / CHUNKS;                  // row exchanged with (chunk * SWZ)
  static constexpr int BLOCK_BYTES = PARTS * KSTEPS * 1024;   // 32 rows (or channels) x one K tile
  static constexpr int K_TILE = 8 * CHUNKS;
};
template <int DT, int BM, int BN> constexpr size_t stage_lds_bytes(int groups) {
  return 2 * (size_t)((BM + BN) / 32) * StageDims<DT>::BLOCK_BYTES * groups + (BM + BN) * 4;
}

// not-a-number once one of the values that passed through is infinite or not a number, else zero (an instruction a value)
__device__ __forceinline__ float not_finite(float v, float before) { return __builtin_fmaf(v, 0.0f, before); }
constexpr float kPartScale = 0x1p24f, kSumScale = 0x1p-48f;      // of the parts of a value, and back for their products
// (the two float halves of a packed pair of bf16, exactly)
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __builtin_bit_cast(float, v & 0xffff0000u); }
// upper halves of two registers side by side
__device__ __forceinline__ uint32_t upper_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
// two floats, rounded to nearest, side by side
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 h2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{lo, hi}), h2));
}
// Eight floats -> three parts of eight bf16.  Both remainders are exact, and the last one has at most eight significand bits.
__device__ __forceinline__ void split3(const float (&f)[8], v4i& p1, v4i& p2, v4i& p3) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float v0 = f[2 * i] * kPartScale, v1 = f[2 * i + 1] * kPartScale;
    const uint32_t h = bf16_pair(v0, v1);
    const float r0 = v0 - bf16_lo(h), r1 = v1 - bf16_hi(h);
    const uint32_t m = bf16_pair(r0, r1);
    p1[i] = (int)h;
    p2[i] = (int)m;
    p3[i] = (int)upper_halves(__builtin_bit_cast(uint32_t, r0 - bf16_lo(m)), __builtin_bit_cast(uint32_t, r1 - bf16_hi(m)));
  }
}
// the float a triple of packed filter parts stands for (igemm_stage.hip: where the second part is not a number, the others
// hold the two halves of the value itself)
__device__ __forceinline__ float join3(float a, float b, float c) {
  if (b != b) return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a) | (__builtin_bit_cast(uint32_t, c) >> 16));
  return ((a + b) + c) * (1.0f / kPartScale);
}

// Bias, activation, shortcut and store of a lane's 16 channels c0 .. c0 + 15 of output row rr, for any layout: 16-byte
// groups at element alignment for NHWC, elements for NCHW.
template <int DT, bool NCHW>
__device__ __forceinline__ void stage_store_row(const float (&acc)[16], int rr, int c0, const ConvParams& p, const float* s_bias_at) {
  using T = typename Elem<DT>::T;
  constexpr int V = Elem<DT>::V;
  int64_t at;
  if constexpr (!NCHW) at = (int64_t)rr * p.c_out + c0;
  else {
    const int n = fast_div(rr, p.div_howo_mul, p.div_howo_shift);
    at = n * p.ys_n + (rr - n * p.ho_wo) + (int64_t)c0 * p.ys_c;
  }
  const int ok = min(16, p.c_out - c0);
  T* y = static_cast<T*>(p.y) + at;
  const T* res = p.residual ? static_cast<const T*>(p.residual) + at : nullptr;
  T out[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    float f = acc[v] + (s_bias_at ? s_bias_at[v] : 0.0f);
    if (p.relu) f = fmaxf(f, 0.0f);
    if (res && v < ok) f += (float)(NCHW ? res[(int64_t)v * p.ys_c] : res[v]);
    if (p.residual_relu) f = fmaxf(f, 0.0f);
    out[v] = Elem<DT>::from_float(f);
  }
  if constexpr (NCHW) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (v < ok) y[(int64_t)v * p.ys_c] = out[v];
  } else {
#pragma unroll
    for (int g = 0; g < 16 / V; ++g) {
      if (V * g + V <= ok) __builtin_memcpy(y + V * g, out + V * g, 16);
      else {
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (V * g + e < ok) y[V * g + e] = out[V * g + e];
      }
    }
  }
}

// KG > 1: the K tiles are divided among KG groups of four wavefronts, each with LDS tiles of its own; the first group adds the
// others' sums in order and stores.  For launches of at most a workgroup per compute unit, whose four wavefronts leave it idle
// between their phases (measured where the launcher chooses).
template <int DT, int BM, int BN, int WAVES_M, int WAVES_N, int GATHER, bool NCHW, int KG = 1>
__global__ __launch_bounds__(kThreads * KG, 2) void igemm_stage_kernel(const ConvParams p) {
  using D = StageDims<DT>;
  using E = Elem<DT>;
  using T = typename E::T;
  constexpr int V = E::V, EB = sizeof(T);
  constexpr int PARTS = D::PARTS, CHUNKS = D::CHUNKS, KSTEPS = D::KSTEPS, SWZ = D::SWZ;
  constexpr bool SPLIT = PARTS == 3;
  constexpr bool BY_ENTRY = GATHER >= kStageChunks;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int MI = WM / 32, NI = WN / 32;
  constexpr int A_BYTES = (BM / 32) * D::BLOCK_BYTES, B_BYTES = (BN / 32) * D::BLOCK_BYTES;
  constexpr int PART_A = (BM / 32) * KSTEPS * 1024;             // one part of the A tile
  constexpr int B_UNITS = B_BYTES / 1024;                       // 1 KiB a wavefront copies at a time
  constexpr int B_LOADS = (B_UNITS + 3) / 4;
  constexpr int AHEAD = PARTS * (MI + NI) <= 9 && MI * NI < 4 ? 2 : 1;      // (as the registers allow)
  static_assert(WAVES_M * WAVES_N == 4 && WM % 32 == 0 && WN % 32 == 0 && BM % 64 == 0, "four wavefronts of 32x32 blocks");

  constexpr int RING = 2 * (A_BYTES + B_BYTES);
  extern __shared__ __align__(16) unsigned char smem_all[];
  const int t_all = threadIdx.x, group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(t_all / kThreads);
  unsigned char* smem = smem_all + group * RING;
  unsigned char* s_a = smem;                                    // [2][A_BYTES]
  unsigned char* s_b = smem + 2 * A_BYTES;                      // [2][B_BYTES]
  int32_t* s_rows = reinterpret_cast<int32_t*>(smem_all + KG * RING);             // [BM]
  float* s_bias = reinterpret_cast<float*>(s_rows + BM);        // [BN]

  const int nwg = p.m_tiles * p.n_tiles;
  const int per_xcd = (nwg + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= nwg) return;
  const int tile_m = logical / p.n_tiles;
  const int tile_n = logical - tile_m * p.n_tiles;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int t = t_all - group * kThreads;                        // within the group, like `wave`
  const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int kt_lo = group * p.k_tiles / KG, n_kt = (group + 1) * p.k_tiles / KG - kt_lo;
  const int steps = (p.k_tiles + KG - 1) / KG;                   // of the longest share; a shorter one ends in a tile of zeros
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  const int fp = lane & 31, fh = lane >> 5;

  // ---- the rows this thread stages and the chunks of a K tile it fetches for each of them -----------------------------
  //   groups:  CHUNKS lanes side by side hold the chunks of one row; rows 256 / CHUNKS apart
  //   entries: lane = row, the chunk is the same for the whole wavefront
  constexpr int ROWS = BY_ENTRY ? 1 : BM * CHUNKS / kThreads;
  constexpr int ROW_STEP = kThreads / CHUNKS;
  constexpr int PER_ROW = BY_ENTRY ? BM * CHUNKS / kThreads : 1;
  const int row0 = BY_ENTRY ? t % BM : t / CHUNKS;
  const int chunk0 = BY_ENTRY ? __builtin_amdgcn_readfirstlane(t / BM) * PER_ROW : t % CHUNKS;
  int32_t a_at[ROWS];           // byte offset of the window's corner, possibly negative
  uint32_t a_taps[ROWS];        // bit ky: that window row lies inside the image; bit 8 + kx: that window column
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const int ic = m0 + row0 + ROW_STEP * j;
    const bool present = ic < p.rows;
    const int icc = present ? ic : p.rows - 1;
    const int rr = p.row_idx ? p.row_idx[icc] : icc;
    if (BY_ENTRY ? t < BM : chunk0 == 0) s_rows[row0 + ROW_STEP * j] = !present ? -1 : p.y_compact ? ic : rr;
    const int rc = p.x_compact ? icc : rr;
    const int n = fast_div(rc, p.div_howo_mul, p.div_howo_shift), rem = rc - n * p.ho_wo;
    const int oy = fast_div(rem, p.div_wo_mul, p.div_wo_shift), ox = rem - oy * p.wo;
    const int iy0 = oy * p.sh - p.ph, ix0 = ox * p.sw - p.pw;
    a_at[j] = (int32_t)((n * p.xs_n + (int64_t)iy0 * p.xs_h + (int64_t)ix0 * p.xs_w) * EB);
    uint32_t bits = 0;
    for (int ky = 0; ky < p.kh; ++ky) bits |= ((unsigned)(iy0 + ky * p.dil_h) < (unsigned)p.h ? 1u : 0u) << ky;
    for (int kx = 0; kx < p.kw; ++kx) bits |= ((unsigned)(ix0 + kx * p.dil_w) < (unsigned)p.w ? 1u : 0u) << (8 + kx);
    a_taps[j] = present ? bits : 0u;
  }
  if (t_all < BN) s_bias[t_all] = p.bias && n0 + t_all < p.c_out ? p.bias[n0 + t_all] : 0.0f;
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)p.x_bytes, kBufferWord3);
  const unsigned char* xb = static_cast<const unsigned char*>(p.x);
  const unsigned char* wb = static_cast<const unsigned char*>(p.wp) + ((int64_t)(n0 / 32) * p.k_tiles) * D::BLOCK_BYTES;

  // what a thread holds of a K tile: 16-byte groups, or one register per entry
  constexpr int A_REGS = BY_ENTRY ? PER_ROW * 8 : ROWS * (8 * EB / 4);
  struct Regs { uint32_t a[A_REGS]; uint32_t tails; };
  constexpr int A_LOADS = BY_ENTRY ? PER_ROW * 8 : ROWS * (8 / V);      // loads of a tile's rows
  // The loads of a tile go out between the products of an earlier one, where the issue slot is free while the matrix unit works;
  // all at once a wavefront sits in the issue stage until the address unit has taken them (us, at once / between: 128 -> 128 @28
  // channels first in float, batch 4 26.3 / 21.9, batch 32 39.1 / 37.1; 16 x 256 -> 256 @14 46 / 39; 410 -> 410 @7 24.2 / 22.5).
  // Where they are many beside few products their addresses crowd the registers (128 rows by entry in bf16 23 / 41).
  constexpr bool BETWEEN = A_LOADS <= (GATHER == kStageEntries ? 8 : 16);
  constexpr int GPC = 8 / V;          // 16-byte groups per chunk
  const int last = max(kt_lo + n_kt - 1, 0);

  // The table entries of the next tile to be loaded.  They are fetched a tile ahead of the loads that need them, so that
  // waiting for them (loads return in order) never waits for a tile that is still on its way.
  // Where they are the same for a wavefront they are scalar loads (named as such: behind the barriers' clobbers the compiler
  // would use vector loads, or a branch around the offset of an entry outside the image).
  constexpr int ENTRIES = GATHER == kStageChunks ? 1 : 8;       // of a chunk
  constexpr bool TABLE_AHEAD = PER_ROW * ENTRIES <= 16;         // (as the scalar registers allow)
  constexpr int TABS = BY_ENTRY ? PER_ROW * ENTRIES : GPC;
  typedef const __attribute__((address_space(4))) KEntry ScalarEntry;
  typedef const __attribute__((address_space(4))) v4i ScalarPair;
  KEntry ke[TABS];
  auto load_table = [&](int kt) {
    if constexpr (!BY_ENTRY) {
#pragma unroll
      for (int g = 0; g < GPC; ++g) ke[g] = p.ktab[(kt * CHUNKS + chunk0) * GPC + g];
    } else {
      const KEntry* at = p.ktab + (kt * CHUNKS + chunk0) * ENTRIES;
      if constexpr (TABS % 2 != 0) {
        const auto* one = reinterpret_cast<ScalarEntry*>(reinterpret_cast<uint64_t>(at));
        ke[0].off = one->off;
        ke[0].dydx = one->dydx;
      } else {
        const auto* two = reinterpret_cast<ScalarPair*>(reinterpret_cast<uint64_t>(at));
#pragma unroll
        for (int i = 0; i < TABS / 2; ++i) {
          const v4i v = two[i];
          ke[2 * i] = KEntry{v[0], v[1]};
          ke[2 * i + 1] = KEntry{v[2], v[3]};
        }
      }
    }
  };
  // Where the loads of tile i of the share go (unconditional: past the last one that is loaded again, and not used); load_one
  // issues the j-th of them.
  struct Places { uint32_t at[BY_ENTRY ? PER_ROW * (GATHER == kStageChunks ? 1 : 8) : ROWS * GPC]; };
  auto aim_tile = [&](int i, Regs& r, Places& pl) {
    const int kt_want = kt_lo + i, kt = min(kt_want, last);
    if (BY_ENTRY && !TABLE_AHEAD) load_table(kt);
    KEntry now[TABS];
#pragma unroll
    for (int i = 0; i < TABS; ++i) now[i] = ke[i];
    if (!BY_ENTRY || TABLE_AHEAD) load_table(min(kt_want + 1, last));
    if constexpr (!BY_ENTRY) r.tails = 0;
#pragma unroll
    for (int g = 0; g < TABS; ++g) {
      uint32_t need = (uint32_t)now[g].dydx & ~(BY_ENTRY ? 0u : kStageTail);
      if (KG > 1 && i >= n_kt) need = kStageNoTap;
      if constexpr (GATHER == kStageRaggedGroups) r.tails |= ((uint32_t)now[g].dydx >> 31) << g;
#pragma unroll
      for (int j = 0; j < ROWS; ++j) pl.at[j * TABS + g] = (a_taps[j] & need) == need ? (uint32_t)(a_at[j] + now[g].off) : kOutOfRange;
    }
  };
  auto load_one = [&](int j, Regs& r, const Places& pl) {
    if constexpr (!BY_ENTRY) {
      v4i v;
      if constexpr (GATHER == kStageGroups) {
        v = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, pl.at[j], 0, 0));
      } else {
        const unsigned char* src = pl.at[j] != kOutOfRange ? xb + (int64_t)(int32_t)pl.at[j] : static_cast<const unsigned char*>(p.zeros);
        __builtin_memcpy(&v, src, 16);          // element-aligned
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) r.a[j * 4 + i] = (uint32_t)v[i];
    } else {
      const uint32_t voff = pl.at[GATHER == kStageChunks ? j / 8 : j];
      const int soff = GATHER == kStageChunks ? (j % 8) * p.h * p.w * EB : 0;
      if constexpr (EB == 4) r.a[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rx, voff, soff, 0);
      else r.a[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rx, voff, soff, 0);
    }
  };
  auto load_all = [&](Regs& r, const Places& pl) {
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j) load_one(j, r, pl);
  };
  auto load_tile = [&](int i, Regs& r) {
    Places pl;
    aim_tile(i, r, pl);
    load_all(r, pl);
  };
  // the filters of tile i go straight into LDS; tile i + 1 is asked for when every wavefront has left the place it takes
  typedef __attribute__((address_space(3))) void lds_void;
  auto issue_filters = [&](int i, int buf) {
    const int kt = min(kt_lo + i, last);
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) {
      // (a wavefront without a unit of its own in the last round repeats the last one: the same bytes to the same place)
      const int u = min(wave + 4 * j, B_UNITS - 1);
      constexpr int PER = D::BLOCK_BYTES / 1024;
      const int nb = u / PER, in = u - nb * PER;
      const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<unsigned char*>(wb + ((int64_t)nb * p.k_tiles + kt) * D::BLOCK_BYTES), 0, KG > 1 && i >= n_kt ? 0 : D::BLOCK_BYTES, kBufferWord3);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)(s_b + buf * B_BYTES + u * 1024), 16, (uint32_t)(lane * 16), in * 1024, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);       // (ahead of the row loads that follow: the order is counted on below)
  };

  // LDS byte offset of (row, chunk) inside one part of a tile
  auto a_place = [&](int row, int chunk) {
    return ((row >> 5) * KSTEPS + (chunk >> 1)) * 1024 + (chunk & 1) * 512 + (((row ^ (chunk * SWZ)) & 31) << 4);
  };
  auto store_tile = [&](int buf, const Regs& r, auto careful_c) {
    constexpr bool CAREFUL = decltype(careful_c)::value;
    unsigned char* pa = s_a + buf * A_BYTES;
#pragma unroll
    for (int j = 0; j < ROWS; ++j)
#pragma unroll
      for (int c = 0; c < PER_ROW; ++c) {
        unsigned char* dst = pa + a_place(row0 + ROW_STEP * j, chunk0 + c);
        if constexpr (SPLIT) {
          float f[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) f[e] = __builtin_bit_cast(float, r.a[(j * PER_ROW + c) * 8 + e]);
          if constexpr (CAREFUL) {
            if constexpr (GATHER == kStageRaggedGroups) {
#pragma unroll
              for (int e = 0; e < 8; ++e)
                if (((r.tails >> (e / 4)) & 1u) && (e & 3) < p.seg_tail) f[e] = 0.0f;
            }
            v4f lo = {f[0], f[1], f[2], f[3]}, hi = {f[4], f[5], f[6], f[7]};
            *reinterpret_cast<v4f*>(dst) = lo;
            *reinterpret_cast<v4f*>(dst + PART_A) = hi;
          } else {
            v4i p1, p2, p3;
            split3(f, p1, p2, p3);
            *reinterpret_cast<v4i*>(dst) = p1;
            *reinterpret_cast<v4i*>(dst + PART_A) = p2;
            *reinterpret_cast<v4i*>(dst + 2 * PART_A) = p3;
          }
        } else {
          v4i v;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (BY_ENTRY) v[i] = (int)((r.a[c * 8 + 2 * i] & 0xffffu) | (r.a[c * 8 + 2 * i + 1] << 16));
            else v[i] = (int)r.a[j * 4 + i];
            if constexpr (CAREFUL && GATHER == kStageRaggedGroups) {
              if (r.tails & 1u) {
                if (2 * i < p.seg_tail) v[i] &= (int)0xffff0000u;
                if (2 * i + 1 < p.seg_tail) v[i] &= 0xffff;
              }
            }
          }
          *reinterpret_cast<v4i*>(dst) = v;
        }
      }
  };

  // The same in pieces that go between the products of the tile before (the place was left at the last barrier): a float chunk in ten
  // of four to six vector instructions, none of which waits for the one before it, the last one with the stores; a 16-bit chunk in one.
  constexpr int CHUNK_PIECES = SPLIT ? 10 : 1, PIECES = ROWS * PER_ROW * CHUNK_PIECES;
  struct Split { float v[8], part[8]; uint32_t pk[3][4]; };
  auto store_piece = [&](int buf, const Regs& r, Split& sp, int piece) {
    const int chunk = piece / CHUNK_PIECES, j = chunk / PER_ROW, c = chunk % PER_ROW, step = piece % CHUNK_PIECES;
    unsigned char* dst = s_a + buf * A_BYTES + a_place(row0 + ROW_STEP * j, chunk0 + c);
    if constexpr (!SPLIT) {
      v4i v;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (BY_ENTRY) v[i] = (int)((r.a[c * 8 + 2 * i] & 0xffffu) | (r.a[c * 8 + 2 * i + 1] << 16));
        else v[i] = (int)r.a[j * 4 + i];
      }
      *reinterpret_cast<v4i*>(dst) = v;
    } else {
      auto scale = [&](int e) { sp.v[e] = __builtin_bit_cast(float, r.a[chunk * 8 + e]) * kPartScale; asm volatile("" : "+v"(sp.v[e])); };
      auto pack = [&](int q, int i) {
        sp.pk[q][i] = q == 2 ? upper_halves(__builtin_bit_cast(uint32_t, sp.v[2 * i]), __builtin_bit_cast(uint32_t, sp.v[2 * i + 1])) : bf16_pair(sp.v[2 * i], sp.v[2 * i + 1]);
        asm volatile("" : "+v"(sp.pk[q][i]));      // (not sunk to the stores)
      };
      auto widen = [&](int q, int e) {
        sp.part[e] = e & 1 ? bf16_hi(sp.pk[q][e >> 1]) : bf16_lo(sp.pk[q][e >> 1]);
        asm volatile("" : "+v"(sp.part[e]));
      };
      auto rest = [&](int e) { sp.v[e] -= sp.part[e]; asm volatile("" : "+v"(sp.v[e])); };
      if (step == 0) for (int e = 0; e < 6; ++e) scale(e);
      if (step == 1) { scale(6); scale(7); for (int i = 0; i < 4; ++i) pack(0, i); }
      if (step == 2) for (int e = 0; e < 6; ++e) widen(0, e);
      if (step == 3) { widen(0, 6); widen(0, 7); for (int e = 0; e < 4; ++e) rest(e); }
      if (step == 4) { for (int e = 4; e < 8; ++e) rest(e); pack(1, 0); pack(1, 1); }
      if (step == 5) { pack(1, 2); pack(1, 3); for (int e = 0; e < 4; ++e) widen(1, e); }
      if (step == 6) { for (int e = 4; e < 8; ++e) widen(1, e); rest(0); rest(1); }
      if (step == 7) for (int e = 2; e < 8; ++e) rest(e);
      if (step == 8) for (int i = 0; i < 4; ++i) pack(2, i);
      if (step == 9) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
          *reinterpret_cast<v4i*>(dst + q * PART_A) = v4i{(int)sp.pk[q][0], (int)sp.pk[q][1], (int)sp.pk[q][2], (int)sp.pk[q][3]};
      }
    }
  };

  floatx16 acc[MI][NI], small[SPLIT ? MI : 1][SPLIT ? NI : 1];
  auto clear = [&]() {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc[mi][ni][v] = 0.0f;
          if constexpr (SPLIT) small[mi][ni][v] = 0.0f;
        }
  };

  // (LDS reads by hand: the compiler would have them wait for the filters on their way to the other half)
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  unsigned frag_a[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) frag_a[ks] = lds0 + a_place(wm0 + fp, 2 * ks + fh);
  const unsigned frag_b = lds0 + 2 * A_BYTES + (wn0 / 32) * D::BLOCK_BYTES + lane * 16;

  // (r, pl: the loads of a later tile, issued between the products; st: the next tile, stored between them)
  auto compute_tile = [&](auto buf_c, auto careful_c, Regs* r, const Places* pl, const Regs* st) {
    Split sp;
    constexpr bool CAREFUL = decltype(careful_c)::value;
    constexpr int BUF = decltype(buf_c)::value;
    auto steps_of = [&](auto k2_c) {      // AHEAD K steps of fragments are read before their products start
      constexpr int k2 = decltype(k2_c)::value;
      v4i xf[AHEAD][MI][PARTS], wf[AHEAD][NI][PARTS];
      static_for<AHEAD>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        static_for<PARTS>([&](auto q_c) {
          constexpr int q = decltype(q_c)::value;
          static_for<NI>([&](auto ni_c) {
            constexpr int ni = decltype(ni_c)::value;
            wf[i][ni][q] = lds_read16_big<BUF * B_BYTES + ni * D::BLOCK_BYTES + (q * KSTEPS + k2 + i) * 1024>(frag_b);
          });
          static_for<MI>([&](auto mi_c) {
            constexpr int mi = decltype(mi_c)::value;
            xf[i][mi][q] = lds_read16_big<BUF * A_BYTES + q * PART_A + mi * KSTEPS * 1024>(frag_a[k2 + i]);
          });
        });
      });
      static_for<AHEAD>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        // the step's fragments have landed, those of the next one may be on their way; they pass through, so that nothing
        // that uses them moves above
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"((AHEAD - 1 - i) * PARTS * (MI + NI)));
#pragma unroll
        for (int q = 0; q < PARTS; ++q) {
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) asm volatile("" : "+v"(wf[i][ni][q]));
#pragma unroll
          for (int mi = 0; mi < MI; ++mi) asm volatile("" : "+v"(xf[i][mi][q]));
        }
        constexpr int ROUNDS = (SPLIT && !CAREFUL ? 6 : 1) * MI * NI, ALL = KSTEPS * ROUNDS, FIRST = ALL / 4;
        int done = (k2 + i) * ROUNDS;
        auto each = [&](auto fn) {
#pragma unroll
          for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
              fn(mi, ni);
              if (r) {
#pragma unroll
                for (int j = 0; j < A_LOADS; ++j)
                  if (j * ALL / A_LOADS == done) load_one(j, *r, *pl);
              }
              if (!CAREFUL && st) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < PIECES; ++i)
                  if (FIRST + i * (ALL - FIRST) / PIECES == done) store_piece(BUF ^ 1, *st, sp, i);
                __builtin_amdgcn_sched_barrier(0);
              } else if (r) {
                __builtin_amdgcn_sched_barrier(0x6);
              }
              ++done;
            }
        };
        if constexpr (!SPLIT) {
          each([&](int mi, int ni) { E::mma(acc[mi][ni], wf[i][ni][0], xf[i][mi][0]); });
        } else if constexpr (CAREFUL) {
          each([&](int mi, int ni) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              auto part = [&](int q) {
                const uint32_t v = (uint32_t)wf[i][ni][q][e >> 1];
                return (e & 1) ? bf16_hi(v) : bf16_lo(v);
              };
              const float w = join3(part(0), part(1), part(2));
              const float x = __builtin_bit_cast(v4f, xf[i][mi][e >> 2])[e & 3];
              acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, x, acc[mi][ni], 0, 0, 0);
            }
          });
        } else {
          using H = Elem<kBF16>;
          each([&](int mi, int ni) { H::mma(acc[mi][ni], wf[i][ni][0], xf[i][mi][0]); });
          each([&](int mi, int ni) { H::mma(small[mi][ni], wf[i][ni][1], xf[i][mi][0]); });
          each([&](int mi, int ni) { H::mma(small[mi][ni], wf[i][ni][0], xf[i][mi][1]); });
          each([&](int mi, int ni) { H::mma(small[mi][ni], wf[i][ni][1], xf[i][mi][1]); });
          each([&](int mi, int ni) { H::mma(small[mi][ni], wf[i][ni][2], xf[i][mi][0]); });
          each([&](int mi, int ni) { H::mma(small[mi][ni], wf[i][ni][0], xf[i][mi][2]); });
        }
      });
    };
    static_for<KSTEPS / AHEAD>([&](auto k_c) { steps_of(std::integral_constant<int, decltype(k_c)::value * AHEAD>{}); });
  };

  // ---- zero fill of the dropped rows this workgroup owns (Alg. 2, mask == 0 branch), behind the first K tile: the stores
  // drain under the others.  Mask bytes are fetched several passes at a time.
  auto fill_zeros = [&]() {
    const int lo = tile_m == 0 ? 0 : p.row_idx[m0];
    const int hi = (m0 + BM >= p.rows) ? p.m_total : p.row_idx[m0 + BM];
    auto mask_of = [&](int r) -> unsigned {
      if (p.mask_spatial) r -= fast_div(r, p.div_howo_mul, p.div_howo_shift) * p.ho_wo;
      return p.mask[r];
    };
    T* y = static_cast<T*>(p.y);
    const T* res = static_cast<const T*>(p.residual);
    auto fill_one = [&](int64_t at) {
      float f = 0.0f;
      if (res) {
        f += (float)res[at];
        if (p.residual_relu) f = fmaxf(f, 0.0f);
      }
      y[at] = E::from_float(f);
    };
    const int cols = min(BN, p.c_out - n0);
    if constexpr (!NCHW) {      // lanes side by side on the 16-byte groups of a row
      constexpr int CPR = BN / V, RPI = kThreads * KG / CPR, ZB = 8;
      const int c = (t_all % CPR) * V;
      if (c >= cols) return;
      for (int r0 = lo + t_all / CPR; r0 < hi; r0 += ZB * RPI) {
        unsigned mk[ZB];
#pragma unroll
        for (int u = 0; u < ZB; ++u) mk[u] = mask_of(min(r0 + u * RPI, hi - 1));
#pragma unroll
        for (int u = 0; u < ZB; ++u) {
          const int r = r0 + u * RPI;
          if (r >= hi || mk[u] != 0) continue;
          const int64_t at = (int64_t)r * p.c_out + n0 + c;
          if (!res && c + V <= cols) {
            const v4i z = {0, 0, 0, 0};
            __builtin_memcpy(y + at, &z, 16);
          } else {
            for (int e = 0; e < min(V, cols - c); ++e) fill_one(at + e);
          }
        }
      }
    } else {                    // lanes side by side on the positions of a channel's map
      constexpr int ZB = 4;
      for (int r0 = lo + lane; r0 < hi; r0 += ZB * 64) {
        unsigned mk[ZB];
#pragma unroll
        for (int u = 0; u < ZB; ++u) mk[u] = mask_of(min(r0 + u * 64, hi - 1));
#pragma unroll
        for (int u = 0; u < ZB; ++u) {
          const int r = r0 + u * 64;
          if (r >= hi || mk[u] != 0) continue;
          const int n = fast_div(r, p.div_howo_mul, p.div_howo_shift);
          const int64_t at = n * p.ys_n + (r - n * p.ho_wo) + (int64_t)n0 * p.ys_c;
          for (int c = wave + 4 * group; c < cols; c += 4 * KG) fill_one(at + (int64_t)c * p.ys_c);
        }
      }
    }
  };

  // ---- K loop: two tiles ahead in registers, one ahead in LDS ------------------------------------------------------------
  auto contract = [&](auto careful_c) {
    // The next tile's split and stores behind the products of this one, or after them (us, after / behind: 32 x 128 -> 128 @28 channels
    // first in float 36.9 / 35.4, in bf16 21.3 / 20.9;  16 x 256 -> 256 @14 38.8 / 36.9;  32 x 102 -> 102 @28 NHWC in float 33.3 / 31.2).
    // The few stores of 16-bit groups gain nothing (64 x 102 -> 102 @28 in fp16 26.5 / 26.6), and a table entry for every load leaves
    // no registers for it (16 x 3 -> 64 @56 channels first in float 9.8 / 10.1).  Nor have the 128-row tiles of 16-bit chunks, whose loads
    // go out at once: both register slots would lie in scratch memory (32 x 32 -> 32 @56 in bf16 19.0 / 38.5, pointwise 64 -> 256 @28
    // 15.1 / 20.2; dense runs up to four times as long).
    constexpr bool BEHIND = !decltype(careful_c)::value && BETWEEN && (GATHER == kStageChunks || (SPLIT && GATHER != kStageEntries));
    constexpr std::integral_constant<int, 0> even;
    constexpr std::integral_constant<int, 1> odd;
    Regs r0, r1;
    Places pl;
    // (a wavefront's loads return in order: when at most A_LOADS, those of a later tile's rows, are on their way, the
    // filters asked for before them have landed)
    auto arrive = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(A_LOADS) : "memory");      // (and this wavefront's stores to LDS are done)
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    load_table(min(kt_lo, last));
    issue_filters(0, 0);
    load_tile(0, r0);
    load_tile(1, r1);
    store_tile(0, r0, careful_c);
    arrive();
    // (two tiles per turn and no way out in the middle: the accumulators and the register slots keep their places)
#pragma unroll 1
    for (int kt = 0; kt + 1 < steps; kt += 2) {
      issue_filters(kt + 1, 1);
      aim_tile(kt + 2, r0, pl);
      if constexpr (!BETWEEN) load_all(r0, pl);
      __builtin_amdgcn_sched_barrier(0);
      compute_tile(even, careful_c, BETWEEN ? &r0 : nullptr, &pl, BEHIND ? &r1 : nullptr);
      if (!decltype(careful_c)::value && kt == 0 && p.zero_fill) fill_zeros();
      if constexpr (!BEHIND) store_tile(1, r1, careful_c);
      arrive();
      issue_filters(kt + 2, 0);
      aim_tile(kt + 3, r1, pl);
      if constexpr (!BETWEEN) load_all(r1, pl);
      __builtin_amdgcn_sched_barrier(0);
      compute_tile(odd, careful_c, BETWEEN ? &r1 : nullptr, &pl, BEHIND ? &r0 : nullptr);
      if constexpr (!BEHIND) store_tile(0, r0, careful_c);
      arrive();
    }
    if (steps & 1) compute_tile(even, careful_c, (Regs*)nullptr, (const Places*)nullptr, (const Regs*)nullptr);
    if (!decltype(careful_c)::value && steps == 1 && p.zero_fill) fill_zeros();
    wait_vmcnt<0>();                         // (no filters are on their way into LDS any more)
    if constexpr (SPLIT && !decltype(careful_c)::value) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[mi][ni][v] = (acc[mi][ni][v] + small[mi][ni][v]) * kSumScale;
    }
    if constexpr (KG > 1) {
      __syncthreads();                       // every wavefront has left its tiles: their place takes the sums
      constexpr int SLOT = 4 * MI * NI * 4 * 64;
      static_assert((KG - 1) * SLOT * 16 <= KG * RING, "the sums lie where the tiles were");
      v4f* part = reinterpret_cast<v4f*>(smem_all) + wave * (MI * NI * 4 * 64) + lane;
      auto each = [&](auto fn) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q) fn(acc[mi][ni], (mi * NI + ni) * 4 + q, 4 * q);
      };
      if (group > 0)
        each([&](floatx16& a, int at, int v) { part[(group - 1) * SLOT + at * 64] = v4f{a[v], a[v + 1], a[v + 2], a[v + 3]}; });
      __syncthreads();
      if (group == 0) {
#pragma unroll
        for (int g = 0; g < KG - 1; ++g)
          each([&](floatx16& a, int at, int v) {
            const v4f s = part[g * SLOT + at * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[v + e] += s[e];
          });
      }
      __syncthreads();
    }
  };
  clear();
  contract(std::false_type{});
  if constexpr (SPLIT || GATHER == kStageRaggedGroups) {
    bool odd = false;
    float mark = 0.0f;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          if constexpr (SPLIT) mark = not_finite(acc[mi][ni][v], mark);
          else odd |= acc[mi][ni][v] != acc[mi][ni][v];
        }
    if (__syncthreads_or((odd || mark != mark) && group == 0)) {
      clear();
      contract(std::true_type{});
    }
  }
  __syncthreads();

  // ---- epilogue --------------------------------------------------------------------------------------------------------------
  if (KG > 1 && group > 0) return;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    const int rr = s_rows[wm0 + mi * 32 + fp];
    if (rr < 0) continue;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int c0 = wn0 + ni * 32 + 16 * fh;
      if (n0 + c0 >= p.c_out) continue;
      float vals[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) vals[v] = acc[mi][ni][v];
      stage_store_row<DT, NCHW>(vals, rr, n0 + c0, p, p.bias ? s_bias + c0 : nullptr);
    }
  }
}

template <int DT, int BM, int BN, int WAVES_M, int WAVES_N, int GATHER, bool NCHW, int KG = 1>
hipError_t igemm_stage_launch(const ConvParams& p, hipStream_t stream) {
  constexpr size_t lds = stage_lds_bytes<DT, BM, BN>(KG);
  auto kern = igemm_stage_kernel<DT, BM, BN, WAVES_M, WAVES_N, GATHER, NCHW, KG>;
  static std::atomic<bool> attr_set{false};
  if (lds > 64 * 1024 && !attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int nwg = p.m_tiles * p.n_tiles;
  hipLaunchKernelGGL(kern, dim3(((nwg + 7) / 8) * 8), dim3(kThreads * KG), lds, stream, p);
  return hipGetLastError();
}

// the kernel of tile bm x bn with K in `groups` shares for a dtype and a gather, or null (igemm_stage.hip)
LaunchFn stage_kernel(int dtype, int gather, bool nchw, int bm, int bn, int groups);
// filters into the order of the kernel's tiles, and the gather's table (igemm_stage.hip)
hipError_t stage_pack(int dtype, int gather, const void* w, void* wp, KEntry* tab, int c_out, int blocks, int c_in, int kh, int kw,
                      int dil_h, int dil_w, int k_tiles, bool nchw, int h, int w_cols, hipStream_t stream);
// the filters of an NHWC layer with whole 16-byte groups of channels into the tiled layout and (parts not null) the float
// parts; rotated: from the filters of the layer whose input gradient this is (igemm_stage.hip)
hipError_t repack_filters(int dtype, const void* w, void* wp, void* parts, int c_out, int c_in, int taps, int k_stride, int rows,
                          int part_blocks, int k_tiles, bool rotated, hipStream_t stream);

}  // namespace sc
