// Key-key Gram stages of the DensityKV update on bf16 MFMA (gfx950).
//
// Every Gram stage evaluates Soft-Riesz weights w(k_i, k_j) (Eq. 2) for a set
// of "row" items against a stream of "column" items and reduces them per row:
//
//   k_score_mfma       rows = candidates, columns = bank states:
//                      S_x = sum_i RNE(w_ix bs_i)  (Eq. 6), or an approximation
//                      for the banks that k_score_probe picks (then k_order_mark,
//                      k_rescore and k_order_fix make the order exact)
//   k_first_part_mfma  per bank state, over the first 256 ordered candidates:
//                      64-candidate chunk sums (the prefix checkpoints of
//                      Eqs. 8-9) and the first prefix that reaches tau b
//   k_chunk_part_mfma  the chunk sums of the rest of the order, and
//   k_cross_mfma       the whole crossing search, for the groups that the first
//                      part leaves open (Eqs. 9-11)
//   k_rowsum_mfma      row sums: the r* fix-up
//   k_maint_mfma       the exact maintenance (Supp. C): row sums, and the symmetric
//                      Gram of the admitted candidates
//   k_density_mfma     from-scratch bank densities (Eq. 3), a symmetric Gram
//
// The column range of every Gram is split over workgroups (grid dimension y);
// partial integer sums are combined with 64-bit atomic adds, which are exact
// and order-independent.
//
// Layout: a workgroup of 4 waves owns 128 row items; wave w owns 32 of them,
// held for the whole kernel as the B operand of v_mfma_f32_32x32x16_bf16
// (lane l <-> row item l % 32).  Column items stream through LDS in stages of 64
// (two or three stages resident, loaded global -> LDS directly, key rows swizzled)
// and form the A operand, so each lane ends up with 16 weights of its own row
// item and reduces them in registers.
//
// Exactness: with keys on the 1/64 grid every partial sum of the contraction
// is an exact multiple of 2^-18 below 2^24 units, so the MFMA result
//   u = (|k_i|^2 + |k_j|^2 - 2 <k_i, k_j>) / sigma^2
// is exact.  The norms enter through one extra K step (each norm / sigma^2 is
// split exactly into three bf16 pieces) and the row keys are pre-scaled by
// -2 / sigma^2 (exact in bf16).  The epilogue is the binary32 contract:
// t = 1 + u, t^p, correctly rounded reciprocal (rcp + one FMA correction, exact
// for every significand), RNE(w * 2^23) via one FMA, integer sums.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dkv_internal.hpp"

namespace dkv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;  // waves per workgroup of the crossing search, and of the Gram stages at D <= 128
// Waves per workgroup of the Gram stages: 8 at descriptor dimension 256, whose
// three column stages (about 100 KB of LDS) allow one workgroup per CU, so that
// each SIMD still holds two waves.
template <int D>
constexpr int gram_waves() { return D > 128 ? 8 : kWaves; }
constexpr int kCT = 32;  // column items per MFMA tile
constexpr int kSI = 64;  // column items per LDS stage (two tiles, two independent MFMA chains)

template <int D>
struct TileCfg {
  static constexpr int kSteps = D / 16;     // K steps over the key
  static constexpr int kChunks = D / 8;     // 16-byte chunks per key
};

__device__ __forceinline__ uint16_t bf16_rne_bits(float f) { return f32_to_bf16_bits(f); }

// Exact split of x (at most 24 significant bits) into three bf16 values.
__device__ __forceinline__ void split3(float x, uint16_t &h, uint16_t &m, uint16_t &l) {
  h = bf16_rne_bits(x);
  float r = x - bf16_bits_to_f32(h);
  m = bf16_rne_bits(r);
  float r2 = r - bf16_bits_to_f32(m);
  l = bf16_rne_bits(r2);
}

constexpr uint16_t kOne = 0x3F80;  // bf16 1.0

// FOLD: the MFMA already added the 1 of t = 1 + u (exact when sigma^2 <= 2^11,
// where every partial sum stays below 2^24 units of 2^-12 / sigma^2).
template <int P, bool FOLD>
__device__ __forceinline__ uint32_t weight_raw(float u, float scale) {
  // raw bits of fma(w, scale, 2^23): kMagic + RNE(w * scale)
  const float t = FOLD ? u : 1.0f + u;
  float tp = t;
  if constexpr (P >= 2) tp = t * t;
  if constexpr (P == 4) tp = tp * tp;
  const float w = clamp_weight(rcp_rn(tp));
  return __float_as_uint(__builtin_fmaf(w, scale, 8388608.0f));
}

// Source of retention descriptors of dimension D: row r's descriptor is k[r]
// (rows of D elements) or, for the [K; V] geometry (SPLIT), the concatenation
// [k[r]; v[r]] of two rows of D / 2 elements.  desc_chunk gives its 16-byte
// chunk c (8 bf16).
struct Desc {
  const uint16_t *k;
  const uint16_t *v;
};

template <int D, bool SPLIT>
__device__ __forceinline__ const uint16_t *desc_chunk(const Desc &s, int64_t row, int c) {
  if constexpr (!SPLIT) {
    return s.k + row * D + 8 * c;
  } else {
    constexpr int H = D / 2;
    return c < H / 8 ? s.k + row * H + 8 * c : s.v + row * H + 8 * (c - H / 8);
  }
}

// Row fragment: B operand of every K step for this lane's row item.
template <int D>
struct RowFrag {
  bf16x8 b[TileCfg<D>::kSteps + 1];
};

// Load the B operand for row item (lane % 32): keys scaled by -2/sigma^2, then
// the aug step [1, 1, 1, n_hi, n_mid, n_lo, fold, 0] (half 0) / zeros (half 1).
template <int D, bool FOLD, bool SPLIT>
__device__ __forceinline__ void load_row_frag(RowFrag<D> &rf, const Desc &src, int64_t row, float norm, bool valid,
                                              float neg2_inv_s2, float inv_s2) {
  const int h = (threadIdx.x & 63) >> 5;
#pragma unroll
  for (int kk = 0; kk < TileCfg<D>::kSteps; ++kk) {
    u32x4 raw = {0, 0, 0, 0};
    if (valid) raw = *reinterpret_cast<const u32x4 *>(desc_chunk<D, SPLIT>(src, row, 2 * kk + h));
    u32x4 sc;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // both halves times a power of two (exact), back to bf16 in one packed conversion
      const float lo = __uint_as_float(raw[q] << 16) * neg2_inv_s2;
      const float hi = __uint_as_float(raw[q] & 0xFFFF0000u) * neg2_inv_s2;
      sc[q] = pack_bf16x2(lo, hi);
    }
    rf.b[kk] = __builtin_bit_cast(bf16x8, sc);
  }
  u32x4 aug = {0, 0, 0, 0};
  if (valid && h == 0) {
    uint16_t nh, nm, nl;
    split3(norm * inv_s2, nh, nm, nl);
    aug[0] = (uint32_t)kOne | ((uint32_t)kOne << 16);
    aug[1] = (uint32_t)kOne | ((uint32_t)nh << 16);
    aug[2] = (uint32_t)nm | ((uint32_t)nl << 16);
    aug[3] = FOLD ? (uint32_t)kOne : 0u;
  }
  rf.b[TileCfg<D>::kSteps] = __builtin_bit_cast(bf16x8, aug);
}

// ---------------------------------------------------------------------------
// Column stages in LDS: 64 column items per stage, three stages resident (two
// loading while one is used), or two where the registers allow a fourth workgroup
// per CU (the score up to descriptor dimension 128) or hide nothing more (the
// crossing search).  Keys go global -> LDS with 16-byte direct-to-LDS
// loads (no VGPR staging); a key row is 2 d bytes with its 16-byte chunk c
// stored at c ^ (row % chunks), so that the A-operand reads (32 rows, one chunk
// each) are free of bank conflicts.  Each item's extra K step (column_aug,
// precomputed per update) and, for the score, its score scale follow.
// ---------------------------------------------------------------------------
template <int D, int W = kWaves>
struct SCfg {
  static constexpr int CH = D / 8;             // 16-byte chunks per key row
  static constexpr int RB = 2 * D;             // key row bytes
  static constexpr int RPL = 1024 / RB;        // rows per 1 KB load
  static constexpr int NB = kSI * RB / 1024;   // 1 KB loads per stage
  static constexpr int PER = NB / W;           // key loads per thread per stage
  static constexpr int KEYB = kSI * RB;        // key bytes per stage
  static constexpr int AUGB = kSI * 16;        // aug bytes per stage
  static constexpr int ITEMS = kSI / W;       // aug / scale items per wave (its lanes 0 .. ITEMS - 1)
  static_assert(NB % W == 0 && kSI % W == 0, "loads split evenly over the waves");
};
// direct-to-LDS loads per thread per stage: keys, aug (+ score scale)
template <int D, bool kBs, int W = kWaves>
constexpr int stage_ops() { return SCfg<D, W>::PER + 1 + (kBs ? 1 : 0); }

typedef __attribute__((address_space(3))) void lds_void;

// Global rows fetched by this thread for the stage starting at column j0 (its
// key loads, then its aug / scale item); items past ncols repeat the last one.
template <int D, int W>
using StageRows = int32_t[SCfg<D, W>::PER + 1];

template <int D, int W, class RowOf>
__device__ __forceinline__ void stage_rows(StageRows<D, W> &rows, int j0, int ncols, RowOf row_of) {
  using C = SCfg<D, W>;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < C::PER; ++q) {
    const int r = (wave * C::PER + q) * C::RPL + l / C::CH;
    rows[q] = (int32_t)row_of(min(j0 + r, ncols - 1));
  }
  rows[C::PER] = (int32_t)row_of(min(j0 + C::ITEMS * wave + l % C::ITEMS, ncols - 1));
}

// Word 3 of a raw buffer resource: 32-bit data format, no swizzle, no
// thread-id addressing.
constexpr int kBufferRsrcWord3 = 0x00020000;

// One 16-byte (4-byte) raw buffer load per lane to LDS, dst + 16 lane
// (dst + 4 lane), from base + voff, with the bytes [base, base + nbytes) as
// the buffer's extent.
__device__ __forceinline__ void buffer_to_lds16(const void *base, int nbytes, int voff, char *dst) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, nbytes, kBufferRsrcWord3);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)dst, 16, voff, 0, 0, 0);
}
__device__ __forceinline__ void buffer_to_lds4(const void *base, int nbytes, int voff, char *dst) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, nbytes, kBufferRsrcWord3);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)dst, 4, voff, 0, 0, 0);
}

// Stage loads.  Every row of a call lies in one bank's region of its arrays,
// rows [row0, row0 + nrows) (uniform), so whole-key-row descriptors go through
// raw buffer loads to LDS over that region: with a global load to LDS in flight
// the compiler counts every later LDS read as possibly out of order and waits
// for all of them before each use.  [K; V] descriptors, whose two halves come
// from two arrays chosen per lane, keep the global loads to LDS.
template <int D, bool kBs, bool SPLIT, int W = kWaves>
__device__ __forceinline__ void stage_dma(const StageRows<D, W> &rows, const Desc &keys,
                                          const uint4 *augs, const float *bs, char *kb, char *ab, float *sb,
                                          int64_t row0, int nrows) {
  using C = SCfg<D, W>;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  if constexpr (!SPLIT) {
    const void *kbase = keys.k + row0 * D;
    const int kbytes = nrows * C::RB;
#pragma unroll
    for (int q = 0; q < C::PER; ++q) {
      const int blk = wave * C::PER + q;
      const int r = blk * C::RPL + l / C::CH;
      const int c = (l % C::CH) ^ (r % C::CH);
      buffer_to_lds16(kbase, kbytes, (int)(rows[q] - row0) * C::RB + 16 * c, kb + blk * 1024);
    }
  } else {
#pragma unroll
    for (int q = 0; q < C::PER; ++q) {
      const int blk = wave * C::PER + q;
      const int r = blk * C::RPL + l / C::CH;
      const int c = (l % C::CH) ^ (r % C::CH);
      __builtin_amdgcn_global_load_lds((void *)desc_chunk<D, SPLIT>(keys, (int64_t)rows[q], c),
                                       (lds_void *)(kb + blk * 1024), 16, 0, 0);
    }
  }
  // items ITEMS w .. ITEMS (w + 1) - 1: lanes 0 .. ITEMS - 1 of wave w (LDS address = base + lane * size)
  if (l < C::ITEMS) {
    const int rel = (int)(rows[C::PER] - row0);
    buffer_to_lds16(augs + row0, nrows * 16, rel * 16, ab + 16 * C::ITEMS * wave);
    if constexpr (kBs) buffer_to_lds4(bs + row0, nrows * 4, rel * 4, reinterpret_cast<char *>(sb + C::ITEMS * wave));
  }
}

// Stages whose rows are consecutive (row i of a stage = the stage's first row
// + i: bank slots in order, or the ordered candidates): each lane's byte
// offsets are the same for every stage, and the stage's first row goes into the
// uniform buffer base, so no per-stage row arithmetic runs on the VALU.
template <int D, int W = kWaves>
struct StageOff {
  int key[SCfg<D, W>::PER];  // key loads: row r of the stage, swizzled chunk c, as r RB + 16 c
  int item;                  // aug / scale item of lanes 0 .. ITEMS - 1 of each wave: ITEMS w + lane
};

template <int D, int W = kWaves>
__device__ __forceinline__ StageOff<D, W> stage_offsets() {
  using C = SCfg<D, W>;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  StageOff<D, W> o;
#pragma unroll
  for (int q = 0; q < C::PER; ++q) {
    const int r = (wave * C::PER + q) * C::RPL + l / C::CH;
    o.key[q] = r * C::RB + 16 * ((l % C::CH) ^ (r % C::CH));
  }
  o.item = C::ITEMS * wave + l % C::ITEMS;
  return o;
}

// Loads of the stage whose first row is row0 + first (whole-row descriptors).
// The buffers end where the region [row0, row0 + nrows) ends, so rows past it
// read as zero; rows past the Gram's last column are real rows of the region,
// masked by the epilogue like the repeated last row they replace.
template <int D, bool kBs, int W = kWaves>
__device__ __forceinline__ void stage_dma_seq(const StageOff<D, W> &o, int first, const uint16_t *keys,
                                              const uint4 *augs, const float *bs, char *kb, char *ab, float *sb,
                                              int64_t row0, int nrows) {
  using C = SCfg<D, W>;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int64_t r0 = row0 + first;
  const int left = nrows - first;  // rows from the stage's first to the region's end
#pragma unroll
  for (int q = 0; q < C::PER; ++q)
    buffer_to_lds16(keys + r0 * D, left * C::RB, o.key[q], kb + (wave * C::PER + q) * 1024);
  if (l < C::ITEMS) {
    buffer_to_lds16(augs + r0, left * 16, o.item * 16, ab + 16 * C::ITEMS * wave);
    if constexpr (kBs) buffer_to_lds4(bs + r0, left * 4, o.item * 4, reinterpret_cast<char *>(sb + C::ITEMS * wave));
  }
}

// s_waitcnt immediate (gfx9 encoding): at most n vector-memory operations
// outstanding and no LDS operation outstanding (expcnt left alone).
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

// Stage barrier without a memory fence: each thread has waited for its own
// loads of the stage about to be read, so the loads of later stages stay in
// flight; the "memory" clobber keeps LDS accesses from moving across it.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_barrier" ::: "memory"); }

// u for both 32-item tiles of a stage: A fragments from the swizzled key rows
// and the aug step, two interleaved MFMA chains.
template <int D, int AHEAD>
__device__ __forceinline__ void stage_u(const char *kb, const char *ab, const RowFrag<D> &rf, f32x16 &u0,
                                        f32x16 &u1) {
  constexpr int KS = TileCfg<D>::kSteps;
  const int l = threadIdx.x & 63, h = l >> 5, r0 = l & 31, r1 = 32 + r0;
  bf16x8 a0[KS + 1], a1[KS + 1];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    const int c = 2 * kk + h;
    a0[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(
                                            kb + r0 * SCfg<D>::RB + 16 * (c ^ (r0 % SCfg<D>::CH))));
    a1[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(
                                            kb + r1 * SCfg<D>::RB + 16 * (c ^ (r1 % SCfg<D>::CH))));
  }
  // the aug step: both half-waves read the item's 16 bytes; the row fragment's
  // second half is zero, so the h = 1 copy contributes nothing
  a0[KS] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(ab + 16 * r0));
  a1[KS] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(ab + 16 * r1));
  f32x16 x0 = {}, x1 = {};
#pragma unroll
  for (int kk = 0; kk <= KS; ++kk) {
    x0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[kk], rf.b[kk], x0, 0, 0, 0);
    x1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[kk], rf.b[kk], x1, 0, 0, 0);
  }
  // AHEAD > 0: keep AHEAD fragment reads in flight ahead of the MFMAs (the LDS
  // latency is several MFMAs long), i.e. AHEAD reads, then one MFMA and one read
  // at a time; 0 leaves the order to the compiler (kernels with less register room)
  if constexpr (AHEAD > 0) {
    constexpr int kFrags = 2 * (KS + 1), kAhead = kFrags < AHEAD ? kFrags : AHEAD;
    __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);  // LDS reads
#pragma unroll
    for (int i = 0; i < kFrags - kAhead; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kAhead, 0);
  }
  u0 = x0;
  u1 = x1;
}

// Tile-granular software pipeline of the Gram stages (descriptors of up to 128
// elements): the 9 MFMAs of the next 32-column tile are issued interleaved with
// the epilogue of the current tile, so that one wave keeps the matrix cores and
// the VALU busy at the same time instead of relying on other waves.
// frag_offsets: byte offsets of this lane's A fragments in a stage buffer
// (tile 0; tile 1 is 32 rows further: rows r and r + 32 share the swizzle).
template <int D>
__device__ __forceinline__ void frag_offsets(int (&off)[TileCfg<D>::kSteps]) {
  static_assert(32 % SCfg<D>::CH == 0, "rows r and r + 32 share the swizzle");
  const int l = threadIdx.x & 63, h = l >> 5, r0 = l & 31;
#pragma unroll
  for (int kk = 0; kk < TileCfg<D>::kSteps; ++kk) off[kk] = r0 * SCfg<D>::RB + 16 * ((2 * kk + h) ^ (r0 % SCfg<D>::CH));
}
// The exact t = 1 + d2 / sigma^2 of one 32-column tile (half 0 or 1 of a
// stage): the column items' A fragments from LDS times the row fragment, one
// MFMA chain
template <int D>
__device__ __forceinline__ f32x16 tile_mfma(const char *kb, const char *ab, int half, const RowFrag<D> &rf,
                                            const int (&off)[TileCfg<D>::kSteps]) {
  constexpr int KS = TileCfg<D>::kSteps;
  const int r0 = threadIdx.x & 31;
  bf16x8 a[KS + 1];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk)
    a[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kb + 32 * half * SCfg<D>::RB + off[kk]));
  a[KS] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(ab + 16 * (32 * half + r0)));
  f32x16 x = {};
#pragma unroll
  for (int kk = 0; kk <= KS; ++kk) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], rf.b[kk], x, 0, 0, 0);
  return x;
}
// Scheduling of the region that holds one tile_mfma and one tile epilogue:
// LEAD LDS reads first (3 fragments, plus any other reads of the region), then
// per MFMA one read and a slice of the epilogue.
template <int D, int LEAD = 3>
__device__ __forceinline__ void tile_interleave() {
  __builtin_amdgcn_sched_group_barrier(0x100, LEAD, 0);  // LDS reads
#pragma unroll
  for (int i = 0; i <= TileCfg<D>::kSteps; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);  // VALU
  }
}

__device__ __forceinline__ int col_of_reg(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

// Sum over this lane's 16 weights (as integers), columns >= nvalid masked out.
template <int P, bool MASK, bool FOLD>
__device__ __forceinline__ uint32_t lane_wsum(const f32x16 &u, int nvalid, int h) {
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    uint32_t raw = weight_raw<P, FOLD>(u[i], 8388608.0f);
    if constexpr (MASK) raw = col_of_reg(i, h) < nvalid ? raw : kMagic;
    s += raw;
  }
  return s - 16u * kMagic;
}

// ---------------------------------------------------------------------------
// Score: rows = candidates, columns = bank states [c0, c1) of this split.
// ---------------------------------------------------------------------------
constexpr int kColsPerSplit = 1024;

// APPROX: the sums with the hardware reciprocal in place of the correctly rounded
// one and in binary32 within a tile, for calls that need the candidates' order
// only: |S~ - S| <= score_tol(S~, m).  Per pair 16 instead of 26 VALU cycles, so
// that the matrix cores bound the loop; where the bound leaves a position open,
// k_rescore computes the exact scores (below).  Which banks take it: k_score_probe.
//   v_rcp_f32 is within 1 ulp (2^-23) of 1 / t^p, the correctly rounded weight
//   within 2^-24: together 3 2^-24 per term; eight terms in a chain and the sum of
//   the two chains add at most 9 2^-24; the exact terms are rounded to integers
//   (1/2 each), the tile's sum once (1/2 per 32 terms and half-wave): 12 2^-24 S +
//   (1/2 + 1/32) m, below S / 2^20 + m.
__device__ __forceinline__ int64_t score_tol(int64_t s, int m) { return (s >> 20) + m + 2; }

// The LDS stages of a score workgroup: column keys and aug steps (the third stage at
// descriptor dimension 256 only) and score scales.
template <int D>
struct ScoreBufs {
  char *k0, *k1, *k2, *a0, *a1, *a2;
  float *s0, *s1, *s2;
};
template <int D>
constexpr int score_key2() { return D <= 128 ? 1024 : SCfg<D>::KEYB; }
template <int D>
constexpr int score_aug2() { return D <= 128 ? 16 : SCfg<D>::AUGB; }
#define DKV_SCORE_BUFS(sb)                                                                                        \
  __shared__ __attribute__((aligned(1024))) char sb##_k0[SCfg<D>::KEYB], sb##_k1[SCfg<D>::KEYB], sb##_k2[score_key2<D>()]; \
  __shared__ __attribute__((aligned(16))) char sb##_a0[SCfg<D>::AUGB], sb##_a1[SCfg<D>::AUGB], sb##_a2[score_aug2<D>()];   \
  __shared__ __attribute__((aligned(16))) float sb##_s0[kSI], sb##_s1[kSI], sb##_s2[kSI];                             \
  const ScoreBufs<D> sb{sb##_k0, sb##_k1, sb##_k2, sb##_a0, sb##_a1, sb##_a2, sb##_s0, sb##_s1, sb##_s2}

// Rows of a score work item: 32 W of the bank's candidates in order from 32 W bx
// on; entries [e0, e1) of its list from e0 + 32 W bx on; or 32 W of them spread
// over the block, whose sums go to `probe`.
enum ScoreRows { ROWS_ALL, ROWS_LIST, ROWS_PROBE };

// Scores of a work item's candidates over the states [c0, c0 + ncols) of bank b.
template <int D, int P, bool FOLD, bool KV, bool APPROX, int ROWS>
__device__ __forceinline__ void score_item(const dkv_bank &bank, const void *seg_k, const void *seg_v, const Geom &g,
                                           const Prm &p, const Workspace &ws, int b, int bx, int c0, int ncols,
                                           const ScoreBufs<D> &sb, int e0, int e1, uint64_t *probe) {
  constexpr int W = gram_waves<D>();
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, h = l >> 5, n = l & 31;
  const int x = e0 + bx * 32 * W + wave * 32 + n;
  char *const k0 = sb.k0, *const k1 = sb.k1, *const k2 = sb.k2, *const a0 = sb.a0, *const a1 = sb.a1, *const a2 = sb.a2;
  float *const s0 = sb.s0, *const s1 = sb.s1, *const s2 = sb.s2;
  const Desc K{static_cast<const uint16_t *>(seg_k), static_cast<const uint16_t *>(seg_v)};
  const Desc BK{static_cast<const uint16_t *>(bank.k), static_cast<const uint16_t *>(bank.v)};
  const bool rv = x < e1;
  size_t xr = (size_t)b * g.N + (rv ? x : 0);
  if constexpr (ROWS == ROWS_LIST) xr = (size_t)b * g.N + ws.adm_list[(size_t)b * g.N + min(x, e1 - 1)];
  if constexpr (ROWS == ROWS_PROBE) xr = (size_t)b * g.N + x * g.N / (32 * W);
  RowFrag<D> rf;
  load_row_frag<D, FOLD, KV>(rf, K, (int64_t)xr, rv ? ws.cnorm[xr] : 0.0f, rv, -2.0f * p.inv_sigma2, p.inv_sigma2);
  const size_t rb = (size_t)b * g.Mcap + c0;
  const int64_t bank_row0 = (int64_t)b * g.Mcap;  // the stage rows lie in bank b's slots
  auto row_of = [&](int i) -> int64_t { return (int64_t)(rb + i); };
  uint64_t A64 = 0;
  const int ns = (ncols + kSI - 1) / kSI;
  // epilogue of one 32-column tile: integer sum of the scaled score terms
  auto epi = [&](auto mask_tag, const f32x16 &u, const float *tb, int nvalid, uint32_t &sa)
      __attribute__((always_inline)) {
    constexpr bool MASK = decltype(mask_tag)::value;
    float bsv[16];
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const float4 v = *reinterpret_cast<const float4 *>(&tb[8 * gq + 4 * h]);
      bsv[4 * gq + 0] = v.x;
      bsv[4 * gq + 1] = v.y;
      bsv[4 * gq + 2] = v.z;
      bsv[4 * gq + 3] = v.w;
    }
    sa = 0;
    float fa[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float tt = FOLD ? u[i] : 1.0f + u[i];
      float tp = tt;
      if constexpr (P >= 2) tp = tt * tt;
      if constexpr (P == 4) tp = tp * tp;
      if constexpr (APPROX) {
        const float f = __builtin_fmaf(clamp_weight(__builtin_amdgcn_rcpf(tp)), bsv[i], fa[i & 1]);
        // the sum is selected, not the weight: the scales past the last live state are whatever the workspace
        // held, and 0 times an infinity or a NaN is a NaN
        fa[i & 1] = !MASK || col_of_reg(i, h) < nvalid ? f : fa[i & 1];
      } else {
        const float w = clamp_weight(rcp_rn(tp));
        uint32_t ra = __float_as_uint(__builtin_fmaf(w, bsv[i], 8388608.0f));
        if constexpr (MASK) ra = col_of_reg(i, h) < nvalid ? ra : kMagic;
        sa += ra;
      }
    }
    if constexpr (APPROX) sa = (uint32_t)__builtin_rintf(fa[0] + fa[1]);
    else sa -= 16u * kMagic;
  };
  using Full = std::integral_constant<bool, false>;
  using Part = std::integral_constant<bool, true>;
  constexpr int kOps = stage_ops<D, true, W>();
  StageRows<D, W> rows;
  // stage s: rows s kSI .. of this split; whole-row descriptors take the
  // per-lane offsets of consecutive rows, [K; V] ones (two arrays) the row list
  [[maybe_unused]] const StageOff<D, W> soff = stage_offsets<D, W>();
  auto stage_rows_for = [&](int st) __attribute__((always_inline)) {
    if constexpr (KV) stage_rows<D, W>(rows, st * kSI, ncols, row_of);
  };
  auto stage_dma_for = [&](int st, char *kd, char *ad, float *sd) __attribute__((always_inline)) {
    if constexpr (KV) stage_dma<D, true, KV, W>(rows, BK, ws.baug, ws.bs, kd, ad, sd, bank_row0, g.Mcap);
    else stage_dma_seq<D, true, W>(soff, c0 + st * kSI, BK.k, ws.baug, ws.bs, kd, ad, sd, bank_row0, g.Mcap);
  };
  // stage t in buffers (t % 3); rows of stage t + 2 loaded one step ahead
  auto step = [&](int t, const char *kb, const char *ab, const float *sb, char *kn, char *an, float *sn)
      __attribute__((always_inline)) {
    if (t + 1 < ns) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kOps));
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
    stage_barrier();
    if (t + 2 < ns) {
      stage_dma_for(t + 2, kn, an, sn);
      if (t + 3 < ns) stage_rows_for(t + 3);
    }
    f32x16 u0, u1;
    stage_u<D, 0>(kb, ab, rf, u0, u1);
    const int nv0 = ncols - t * kSI;
    uint32_t sa;
    if (nv0 >= kSI) {
      epi(Full{}, u0, sb, kCT, sa);
      A64 += sa;
      epi(Full{}, u1, sb + kCT, kCT, sa);
      A64 += sa;
    } else {
      epi(Part{}, u0, sb, nv0, sa);
      A64 += sa;
      if (nv0 > kCT) {
        epi(Part{}, u1, sb + kCT, nv0 - kCT, sa);
        A64 += sa;
      }
    }
  };
  stage_rows_for(0);
  stage_dma_for(0, k0, a0, s0);
  if (ns > 1) stage_rows_for(1);
  if constexpr (D <= 128) {
    // Tile-granular software pipeline (see tile_interleave) over two stage
    // buffers (the score scales keep three): iteration t: tile 1 of stage t with
    // the epilogue of tile 0; the wait for stage t + 1 and the barrier; stage
    // t + 2 issued into stage t's buffers; tile 0 of stage t + 1 with the epilogue
    // of tile 1.
    int aoff[TileCfg<D>::kSteps];
    frag_offsets<D>(aoff);
    auto epi_full = [&](const f32x16 &u, const float *tb) __attribute__((always_inline)) -> uint32_t {
      uint32_t sa = 0;
      float fa[2] = {0.0f, 0.0f};
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const float4 v = *reinterpret_cast<const float4 *>(&tb[8 * gq + 4 * h]);
        const float bsv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float tt = FOLD ? u[4 * gq + q] : 1.0f + u[4 * gq + q];
          float tp = tt;
          if constexpr (P >= 2) tp = tt * tt;
          if constexpr (P == 4) tp = tp * tp;
          if constexpr (APPROX) {
            fa[q & 1] = __builtin_fmaf(clamp_weight(__builtin_amdgcn_rcpf(tp)), bsv[q], fa[q & 1]);
          } else {
            const float w = clamp_weight(rcp_rn(tp));
            sa += __float_as_uint(__builtin_fmaf(w, bsv[q], 8388608.0f));
          }
        }
      }
      return APPROX ? (uint32_t)__builtin_rintf(fa[0] + fa[1]) : sa - 16u * kMagic;
    };
    f32x16 u;
    auto pstep = [&](int t, const char *kc, const char *ac, const float *sc, const char *kn, const char *an, char *kd,
                     char *ad, float *sd) __attribute__((always_inline)) {
      f32x16 xx = tile_mfma<D>(kc, ac, 1, rf, aoff);
      uint32_t sa = epi_full(u, sc);
      tile_interleave<D, 7>();  // the 4 score-scale reads lead
      asm volatile("" : "+v"(sa));  // the epilogue of tile 0 stays beside the MFMAs of tile 1
      u = xx;
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      stage_barrier();
      if (t + 2 < ns) {
        stage_dma_for(t + 2, kd, ad, sd);
        if (t + 3 < ns) stage_rows_for(t + 3);
      }
      xx = tile_mfma<D>(kn, an, 0, rf, aoff);
      sa += epi_full(u, sc + kCT);
      tile_interleave<D, 7>();
      u = xx;
      A64 += sa;
    };
    if (ns > 0) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      stage_barrier();
      if (ns > 1) {
        stage_dma_for(1, k1, a1, s1);
        if (ns > 2) stage_rows_for(2);
      }
      u = tile_mfma<D>(k0, a0, 0, rf, aoff);
    }
    for (int t = 0; t + 1 < ns; t += 6) {
      pstep(t, k0, a0, s0, k1, a1, k0, a0, s2);
      if (t + 2 < ns) pstep(t + 1, k1, a1, s1, k0, a0, k1, a1, s0);
      if (t + 3 < ns) pstep(t + 2, k0, a0, s2, k1, a1, k0, a0, s1);
      if (t + 4 < ns) pstep(t + 3, k1, a1, s0, k0, a0, k1, a1, s2);
      if (t + 5 < ns) pstep(t + 4, k0, a0, s1, k1, a1, k0, a0, s0);
      if (t + 6 < ns) pstep(t + 5, k1, a1, s2, k0, a0, k1, a1, s1);
    }
    if (ns > 0) {  // the last stage (possibly partial): u holds its tile 0
      const int t = ns - 1;
      const int nv0 = ncols - t * kSI;
      const float *sb = t % 3 == 0 ? s0 : (t % 3 == 1 ? s1 : s2);
      // one call per buffer: the LDS arrays stay compile-time known
      auto last = [&](const char *kb, const char *ab) __attribute__((always_inline)) {
        uint32_t sa;
        epi(Part{}, u, sb, nv0, sa);
        A64 += sa;
        if (nv0 > kCT) {
          const f32x16 xx = tile_mfma<D>(kb, ab, 1, rf, aoff);
          epi(Part{}, xx, sb + kCT, nv0 - kCT, sa);
          A64 += sa;
        }
      };
      if (t % 2 == 0) last(k0, a0);
      else last(k1, a1);
    }
  } else {
  if (ns > 1) {
    stage_dma_for(1, k1, a1, s1);
    if (ns > 2) stage_rows_for(2);
  }
  for (int t = 0; t < ns; t += 3) {
    step(t, k0, a0, s0, k2, a2, s2);
    if (t + 1 < ns) step(t + 1, k1, a1, s1, k0, a0, s0);
    if (t + 2 < ns) step(t + 2, k2, a2, s2, k1, a1, s1);
  }
  }
  const uint64_t At = A64 + __shfl_xor(A64, 32, 64);
  if (!rv || h != 0) return;
  if constexpr (ROWS == ROWS_PROBE) probe[x] = At;
  else atomicAdd(reinterpret_cast<unsigned long long *>(&(ROWS == ROWS_LIST ? ws.sub_adm : ws.acol)[xr]), (unsigned long long)At);
}

template <int D, int P, bool FOLD, bool KV, bool APPROX>
__global__ __launch_bounds__(64 * gram_waves<D>(), gram_waves<D>() == 4 ? 4 : 2) void k_score_mfma(
    dkv_bank bank, const void *seg_k, const void *seg_v, Geom g, Prm p, Workspace ws) {
  constexpr int W = gram_waves<D>();
  // One-dimensional grid over (row block, column split, bank), row blocks
  // fastest.  Workgroup L is dispatched to XCD L % 8; ranking the workgroups
  // XCD by XCD (r = workgroups on lower XCDs + L / 8) keeps all the work items
  // of a bank on one XCD, in order, so that its keys and the candidates' stay
  // in that XCD's L2.
  const int nx = (g.N + 32 * W - 1) / (32 * W), ny = (g.Mcap + kColsPerSplit - 1) / kColsPerSplit;
  const int T = (int)gridDim.x, L = (int)blockIdx.x, xcd = L % 8;
  const int r = xcd * (T / 8) + min(xcd, T % 8) + L / 8;
  const int b = r / (nx * ny), by = (r / nx) % ny, bx = r % nx;
  const int m = ws.m[b];
  const int c0 = by * kColsPerSplit;
  if (c0 >= m || ws.whole[b] == 2) return;  // the order of a block that enters whole is not needed
  DKV_SCORE_BUFS(sb);
  const int ncols = min(kColsPerSplit, m - c0);
  if (APPROX && !ws.exact[b])
    score_item<D, P, FOLD, KV, true, ROWS_ALL>(bank, seg_k, seg_v, g, p, ws, b, bx, c0, ncols, sb, 0, g.N, nullptr);
  else
    score_item<D, P, FOLD, KV, false, ROWS_ALL>(bank, seg_k, seg_v, g, p, ws, b, bx, c0, ncols, sb, 0, g.N, nullptr);
}

// Whether a bank's scores are worth approximating (exact[b] = 0).
//   Where the order is needed beyond its head, as in a group whose crossing
// search goes on past the first part, the exact scores of the open neighbours cost
// more than the approximation saves (48 full banks of 9,360 states, 18 to 28% of
// the candidates open: update 2,340 -> 2,580 us).  So the bank's group has to be
// replaced whole, or one of its banks has to be near its bound (k_begin).
//   And the share of neighbours in the order that the error bound leaves open has
// to be small.  It is estimated from the exact scores of 32 W candidates spread
// over the block, over the bank's first states: in the sorted sample the distance
// of eight places gives the local spacing, scaled to the whole block and bank.
// Estimate and truth were 0.11 and 0.09 for clustered keys, 0.20 and 0.15 without
// clusters, 0.81 and 0.59 with one baseline at a tenth of the next (the scores' unit
// follows the smallest), 1.0 and 1.0 with tied candidates; a bank that turned out
// open throughout took twice the exact score's time.
constexpr int kProbeStates = 256;
constexpr float kProbeMax = 0.25f;

template <int D, int P, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * gram_waves<D>(), gram_waves<D>() == 4 ? 4 : 2) void k_score_probe(
    dkv_bank bank, const void *seg_k, const void *seg_v, Geom g, Prm p, Workspace ws) {
  constexpr int W = gram_waves<D>(), S = 32 * W, kApart = 8;
  const int b = blockIdx.x, t = threadIdx.x, m = ws.m[b];
  // an order that is needed beyond the first part (or one position) pays for more exact scores than it saves
  bool near = ws.whole[b] != 0;
  const int g0 = (b / g.gs) * g.gs;
  for (int j = t & 63; j < g.gs; j += 64) near |= ws.n_ev[g0 + j] != 0;
  near = __any(near);
  if (g.N < S || m == 0 || ws.whole[b] == 2 || !near) {  // too few to tell; nothing to score; not worth it
    if (t == 0) ws.exact[b] = g.N < S || !near;
    return;
  }
  DKV_SCORE_BUFS(sb);
  __shared__ uint64_t raw[S], sorted[S];
  __shared__ float part[W];
  const int ncols = min(kProbeStates, m);
  score_item<D, P, FOLD, KV, false, ROWS_PROBE>(bank, seg_k, seg_v, g, p, ws, b, 0, 0, ncols, sb, 0, S, raw);
  __syncthreads();
  if (t < S) {
    const uint64_t s = raw[t];
    int r = 0;
    for (int j = 0; j < S; ++j) r += raw[j] < s || (raw[j] == s && j < t);
    sorted[r] = s;
  }
  __syncthreads();
  float open = 0.0f;
  if (t + kApart < S) {
    const float up = (float)m / (float)ncols;
    const float tol = 2.0f * (float)score_tol((int64_t)((float)sorted[t] * up), m);
    const float gap = (float)(sorted[t + kApart] - sorted[t]) * up * ((float)S / ((float)kApart * (float)g.N));
    open = tol < gap ? tol / gap : 1.0f;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) open += __shfl_xor(open, o, 64);
  if ((t & 63) == 0) part[t >> 6] = open;
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < W; ++w) open += part[w];
    ws.exact[b] = open > kProbeMax * (S - kApart);
  }
}

// ---------------------------------------------------------------------------
// Exact order from approximate scores.  Neighbours in the approximate order whose
// difference is within the two bounds (score_tol grows with the score, so a clear
// gap separates everything before it from everything after it) form clusters;
// inside them the exact scores decide.  k_order_mark lists the members in
// position order: first those of clusters that begin within the first part of the
// crossing search (or, for a bank replaced whole with fewer states than
// candidates, the cluster across position R: only the set matters), then the
// rest, whose order only the groups that the first part leaves open need.
// k_rescore sums their exact scores, k_order_fix places them.
// Storage: adm_list = candidate, adm_dest = position | ambiguous with the next
// (bit 30), n_ev / e = members in the first list / in both, sub_adm = exact sums
// (cleared again when read); all of it is free until the selection.
// ---------------------------------------------------------------------------
constexpr int kOrderThreads = 1024;
constexpr int kAmbiguous = 1 << 30;
constexpr int kWalkMax = 16;  // steps to either side; beyond, the whole list is sorted

__global__ __launch_bounds__(kOrderThreads) void k_order_mark(Geom g, Workspace ws) {
  const int b = blockIdx.x, m = ws.m[b], R = ws.R[b], N = g.N, whole = ws.whole[b];
  const size_t nb = (size_t)b * N;
  __shared__ int64_t S[kSortMax];
  __shared__ int tmp[2][kOrderThreads / 64];
  __shared__ int lo, hi;  // positions [lo, hi): whole = 1: the cluster across R; else the first list's
  constexpr int kPer = kSortMax / kOrderThreads;
  if (m == 0 || whole == 2 || ws.exact[b]) {  // every score is exact, or no order is needed
    if (threadIdx.x == 0) ws.n_ev[b] = ws.e[b] = 0;
    return;
  }
  int xs[kPer];  // positions threadIdx.x + u kOrderThreads
#pragma unroll
  for (int u = 0; u < kPer; ++u) xs[u] = ws.order[nb + min((int)threadIdx.x + u * kOrderThreads, N - 1)];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int64_t v = ws.acol[nb + xs[u]];
    if ((int)threadIdx.x + u * kOrderThreads < N) S[threadIdx.x + u * kOrderThreads] = v;
  }
  if (threadIdx.x == 0) lo = whole ? 0 : -1, hi = N;
  __syncthreads();
  auto amb = [&](int p) {  // position p with p + 1
    return p >= 0 && p + 1 < N && S[p + 1] - S[p] <= score_tol(S[p], m) + score_tol(S[p + 1], m);
  };
  const int cut = whole ? R : kCrossFirst;  // a cluster is wanted first if it reaches across (whole), or begins before, this position
  for (int p = threadIdx.x; p < N; p += kOrderThreads)
    if (!amb(p)) {
      if (p >= cut - 1) atomicMin(&hi, p + 1);
      else if (whole) atomicMax(&lo, p + 1);
    }
  __syncthreads();
  if (whole && !(R > 0 && amb(R - 1))) hi = lo;  // (the same value from every thread)
  __syncthreads();
  const int l0 = whole ? lo : 0, l1 = hi;
  // members in position order: each thread's contiguous positions, then a scan
  const int per = (N + kOrderThreads - 1) / kOrderThreads;
  const int p0 = min(N, (int)threadIdx.x * per), p1 = min(N, p0 + per);
  int head = 0, all = 0;
  for (int p = p0; p < p1; ++p) {
    const bool f = (amb(p - 1) || amb(p)) && (!whole || (p >= l0 && p < l1));
    all += f;
    head += f && p < l1;
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int ia = all, ih = head;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int ya = __shfl_up(ia, o, 64), yh = __shfl_up(ih, o, 64);
    if (lane >= o) ia += ya, ih += yh;
  }
  if (lane == 63) tmp[0][wid] = ia, tmp[1][wid] = ih;
  __syncthreads();
  int k = ia - all, ta = 0, th = 0;
  for (int w = 0; w < kOrderThreads / 64; ++w) {
    if (w < wid) k += tmp[0][w];
    ta += tmp[0][w];
    th += tmp[1][w];
  }
  for (int p = p0; p < p1; ++p) {
    const bool next = amb(p);
    if (!((amb(p - 1) || next) && (!whole || (p >= l0 && p < l1)))) continue;
    ws.adm_list[nb + k] = ws.order[nb + p];
    ws.adm_dest[nb + k] = p | (next ? kAmbiguous : 0);
    ++k;
  }
  if (threadIdx.x == 0) {
    ws.n_ev[b] = th;
    ws.e[b] = ta;
  }
}

// Entries [k0, k1) of a bank's members: the first list, or (rest) the others of an open group.
__device__ __forceinline__ void order_range(const Geom &g, const Workspace &ws, int b, int rest, int &k0, int &k1) {
  k0 = rest ? ws.n_ev[b] : 0;
  k1 = rest ? (ws.more[b / g.gs] >= kMoreOpen ? ws.e[b] : k0) : ws.n_ev[b];
}

// Exact scores of the listed candidates, with the score kernel's tiles (32 W of
// them and 1,024 bank states per work item).
template <int D, int P, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * gram_waves<D>(), gram_waves<D>() == 4 ? 3 : 2) void k_rescore(
    dkv_bank bank, const void *seg_k, const void *seg_v, Geom g, Prm p, Workspace ws, int rest) {
  constexpr int kRpw = 32 * gram_waves<D>();
  __shared__ int pre[65];
  DKV_SCORE_BUFS(sb);
  auto blocks = [&](int k0, int k1) { return (k1 - k0 + kRpw - 1) / kRpw; };
  walk_items(
      g.B, pre,
      [&](int b) {
        int k0, k1;
        order_range(g, ws, b, rest, k0, k1);
        return blocks(k0, k1) * ((ws.m[b] + kColsPerSplit - 1) / kColsPerSplit);
      },
      [&](int b, int i) __attribute__((always_inline)) {
        int k0, k1;
        order_range(g, ws, b, rest, k0, k1);
        const int nx = blocks(k0, k1), c0 = i / nx * kColsPerSplit;
        __syncthreads();  // the previous item's LDS stages are done with
        score_item<D, P, FOLD, KV, false, ROWS_LIST>(bank, seg_k, seg_v, g, p, ws, b, i % nx, c0,
                                                     min(kColsPerSplit, ws.m[b] - c0), sb, k0, k1, nullptr);
      });
}

// The members of a cluster take its positions in the order of (exact score,
// source index); one workgroup per bank.  A member counts the smaller ones of
// its cluster while the clusters are short.  With a longer one (nearly tied
// scores: a block of equal rows, or one state whose baseline is far below the
// others') the whole list is sorted instead: clusters are separated by a gap
// that the error bound does not reach, so in the order of the exact scores the
// list's k-th member takes its k-th position.
__global__ __launch_bounds__(kOrderThreads) void k_order_fix(Geom g, Workspace ws, int rest) {
  const int b = blockIdx.x;
  const size_t nb = (size_t)b * g.N;
  int k0, k1;
  order_range(g, ws, b, rest, k0, k1);
  if (k0 >= k1) return;
  __shared__ uint64_t S[kSortMax];
  __shared__ uint32_t X[kSortMax];  // candidate, and in bit 31: ambiguous with the next position
  for (int k = k0 + (int)threadIdx.x; k < k1; k += kOrderThreads) {
    const int x = ws.adm_list[nb + k];
    S[k - k0] = (uint64_t)ws.sub_adm[nb + x];
    ws.sub_adm[nb + x] = 0;
    X[k - k0] = (uint32_t)x | (ws.adm_dest[nb + k] & kAmbiguous ? 0x80000000u : 0u);
  }
  __syncthreads();
  const int cnt = k1 - k0;
  bool walked = true;
  for (int k = threadIdx.x; k < cnt && walked; k += kOrderThreads) {
    const int x = (int)(X[k] & 0x7FFFFFFFu);
    const uint64_t s = S[k];
    int first = k, j = k, less = 0;
    // members are listed by position, so a cluster is a run whose entries are ambiguous with their next
    while (first > 0 && (X[first - 1] >> 31) && k - first < kWalkMax) {
      --first;
      const int y = (int)(X[first] & 0x7FFFFFFFu);
      less += S[first] < s || (S[first] == s && y < x);
    }
    while (X[j] >> 31 && j - k < kWalkMax) {
      ++j;
      const int y = (int)(X[j] & 0x7FFFFFFFu);
      less += S[j] < s || (S[j] == s && y < x);
    }
    walked = !(first > 0 && X[first - 1] >> 31) && !(X[j] >> 31);
    if (walked) {
      const int pos = (ws.adm_dest[nb + k0 + first] & ~kAmbiguous) + less;
      ws.order[nb + pos] = x;
      ws.rank[nb + x] = pos;
    }
  }
  if (__syncthreads_and(walked)) return;
  // bitonic sort of (score, source index), padded to a power of two
  int n2 = kOrderThreads;
  while (n2 < cnt) n2 *= 2;
  for (int k = threadIdx.x; k < n2; k += kOrderThreads)
    S[k] = k < cnt ? (S[k] << 13) | (X[k] & 0x1FFFu) : ~0ull;
  __syncthreads();
  for (int len = 2; len <= n2; len <<= 1) {
    for (int d = len >> 1; d > 0; d >>= 1) {
      for (int t = threadIdx.x; t < n2 / 2; t += kOrderThreads) {
        // the t-th index i with bit d clear, against i + d; ascending where bit len of i is clear
        const int i = ((t & ~(d - 1)) << 1) | (t & (d - 1));
        const uint64_t x = S[i], y = S[i + d];
        if (((i & len) == 0) == (x > y)) {
          S[i] = y;
          S[i + d] = x;
        }
      }
      __syncthreads();
    }
  }
  for (int k = threadIdx.x; k < cnt; k += kOrderThreads) {
    const int x = (int)(S[k] & 0x1FFFu), pos = ws.adm_dest[nb + k0 + k] & ~kAmbiguous;
    ws.order[nb + pos] = x;
    ws.rank[nb + x] = pos;
  }
}

// ---------------------------------------------------------------------------
// Row sums.  MODE selects rows, columns and where the sum goes.
// ---------------------------------------------------------------------------
enum RowSumMode { RS_CHUNK = 0, RS_FIXUP = 1, RS_SURV_EV = 2, RS_ADM_BASE = 3 };

static_assert(kCrossFirst % kCkStride == 0, "the first part ends on a chunk boundary");

// The three LDS stages of a Gram workgroup (separate arrays: with the stage
// known at compile time, reads of one stage never wait for loads into another).
template <int D>
struct StageBufs {
  char *k0, *k1, *k2, *a0, *a1, *a2;
  uint32_t *cb;  // [3][kSI] sums of the stages' streamed items (symmetric Grams only), or null
};

// DPP move (the partner lane's value) with a compile-time control.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
// Transposing reduction over the 16 lanes of a DPP row: the lane holds eight
// values a[i] (the first butterfly level already applied), returns the row
// sum for value index lane % 16.  Each level keeps the half of the values
// selected by one lane bit and adds the partner's copy of it: half-row mirror
// (bit 2), quad permutations (bits 1, 0).
__device__ __forceinline__ uint32_t row_transpose_tail(const uint32_t (&a)[8], int l) {
  uint32_t c[4], d[2];
  const bool b2 = (l >> 2) & 1, b1 = (l >> 1) & 1, b0 = l & 1;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t keep = b2 ? a[i + 4] : a[i], send = b2 ? a[i] : a[i + 4];
    c[i] = keep + dpp_mov<0x141>(send);  // row_half_mirror: lane 7 - x within 8 (bit 2 flipped)
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t keep = b1 ? c[i + 2] : c[i], send = b1 ? c[i] : c[i + 2];
    d[i] = keep + dpp_mov<0x4E>(send);  // quad_perm [2,3,0,1]: lane x ^ 2
  }
  const uint32_t keep = b0 ? d[1] : d[0], send = b0 ? d[0] : d[1];
  return keep + dpp_mov<0xB1>(send);  // quad_perm [1,0,3,2]: lane x ^ 1
}

// Body of one row-sum workgroup (bx, by, bz) = (row block, column split, bank).
template <int D, int P, int MODE, bool FOLD, bool KV>
__device__ __forceinline__ void rowsum_body(const dkv_bank &bank, const void *seg_k, const void *seg_v, const Geom &g,
                                            const Prm &p, const Workspace &ws, int64_t *out, int bx, int by, int bz,
                                            const StageBufs<D> &sb, int cfirst = 0, int per = 0) {
  constexpr int W = gram_waves<D>();
  constexpr int kRowsPerWG = 32 * W;
  const int b = bz;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, h = l >> 5, n = l & 31;
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  const int m = ws.m[b];
  // descriptors: candidates, bank states, ordered candidates (stored concatenated)
  const Desc SK{static_cast<const uint16_t *>(seg_k), static_cast<const uint16_t *>(seg_v)};
  const Desc BK{static_cast<const uint16_t *>(bank.k), static_cast<const uint16_t *>(bank.v)};
  const Desc OK{ws.sk, nullptr};
  constexpr bool kNeedEv = MODE == RS_SURV_EV || MODE == RS_ADM_BASE;
  const int n_ev = kNeedEv ? ws.n_ev[b] : 0;
  const int rs = (MODE == RS_FIXUP || kNeedEv) ? ws.r_star[b / g.gs] : 0;
  const int n_surv = m - n_ev;
  // rows
  int nrows;
  if constexpr (MODE == RS_CHUNK || MODE == RS_FIXUP) nrows = m;
  else if constexpr (MODE == RS_SURV_EV) nrows = n_surv;
  else nrows = rs;
  if ((int)bx * kRowsPerWG >= nrows) return;
  if constexpr (MODE == RS_FIXUP) {
    if (ws.whole[b]) return;        // no state survives
    if (rs == 0 && !out) return;    // rho~ = rho: the commit reads rho itself
  }
  // columns of this workgroup: [c0, c1) of the mode's column list
  int c0 = 0, c1 = 0;
  if constexpr (MODE == RS_CHUNK) {  // prefixes from cfirst on, `per` (whole chunks) per split
    c0 = cfirst + by * per;
    c1 = min(ws.R[b], c0 + per);
  } else if constexpr (MODE == RS_FIXUP) {
    c0 = (rs / kCkStride) * kCkStride;
    c1 = rs;
  } else {
    c0 = by * kColsPerSplit;
    c1 = min(MODE == RS_SURV_EV ? n_ev : n_surv, c0 + kColsPerSplit);
  }
  if (MODE != RS_FIXUP && c0 >= c1) return;  // the fix-up always writes rho~, even for r* % 256 == 0
  const int v = bx * kRowsPerWG + wave * 32 + n;
  const bool rv = v < nrows;
  // fix-up: rho~ = rho + the whole chunks before r* + (below) the partial chunk
  auto fixup_finish = [&](uint64_t tot) __attribute__((always_inline)) {
    // the two half-waves sum alternate 4-chunk groups
    const int full = rs / kCkStride;
    if (rv) {
      const uint4 *ckr = reinterpret_cast<const uint4 *>(ws.ck + (rb + v) * ws.nck);
      for (int c4 = h; 4 * c4 < full; c4 += 2) {
        const uint4 q = ckr[c4];
        const int c = 4 * c4;
        tot += (uint64_t)q.x + (c + 1 < full ? (uint64_t)q.y : 0) + (c + 2 < full ? (uint64_t)q.z : 0) +
               (c + 3 < full ? (uint64_t)q.w : 0);
      }
    }
    tot += __shfl_xor(tot, 32, 64);
    if (!rv || h != 0) return;
    const size_t row = rb + v;
    const int64_t rt = bank.rho[row] + (int64_t)tot;
    ws.rho_t[row] = rt;
    if (out) out[row] = rt;
  };
  if constexpr (MODE == RS_FIXUP) {
    // r* on a chunk boundary (uniform over the workgroup): no Gram, whole chunks only
    if (c0 >= c1) {
      fixup_finish(0);
      return;
    }
  }
  // row item
  Desc rsrc = BK;
  int64_t rrow = (int64_t)rb;
  float rnorm = 0.0f;
  size_t out_idx = 0;
  if (rv) {
    if constexpr (MODE == RS_CHUNK || MODE == RS_FIXUP) {
      rrow = (int64_t)(rb + v);
      rnorm = bank.knorm[rb + v];
      out_idx = rb + v;
    } else if constexpr (MODE == RS_SURV_EV) {
      const int s = ws.surv_list[rb + v];
      rrow = (int64_t)(rb + s);
      rnorm = bank.knorm[rb + s];
      out_idx = rb + s;
    } else {
      const int x = ws.adm_list[nb + v];
      rsrc = SK;
      rrow = (int64_t)(nb + x);
      rnorm = ws.cnorm[nb + x];
      out_idx = nb + v;
    }
  }
  RowFrag<D> rf;
  load_row_frag<D, FOLD, KV>(rf, rsrc, rrow, rnorm, rv, -2.0f * p.inv_sigma2, p.inv_sigma2);
  // column items (absolute index j in the mode's list)
  auto row_of = [&](int j) -> int64_t {
    if constexpr (MODE == RS_CHUNK) return (int64_t)(nb + j);
    else if constexpr (MODE == RS_FIXUP) return (int64_t)(nb + ws.order[nb + j]);
    else if constexpr (MODE == RS_SURV_EV) return (int64_t)(rb + ws.ev_list[rb + j]);
    else return (int64_t)(rb + ws.surv_list[rb + j]);
  };
  const Desc colbase = MODE == RS_CHUNK ? OK : (MODE == RS_FIXUP ? SK : BK);
  // the ordered candidates are stored as whole descriptors; the others are split for [K; V]
  constexpr bool kColSplit = KV && MODE != RS_CHUNK;
  const uint4 *colaug = MODE == RS_CHUNK ? ws.saug : (MODE == RS_FIXUP ? ws.caug : ws.baug);
  // the column rows lie in bank b's candidates or in its slots
  constexpr bool kColCand = MODE == RS_CHUNK || MODE == RS_FIXUP;
  const int64_t col_row0 = kColCand ? (int64_t)nb : (int64_t)rb;
  const int col_nrows = kColCand ? g.N : g.Mcap;  // rows of that region
  // software-pipelined (below); the fix-up has one stage, and descriptor
  // dimension 256 no registers for it
  constexpr bool kPipe = MODE != RS_FIXUP && D <= 128;
  uint64_t S64 = 0;
  uint32_t chunk_sum = 0;
  const int ncols = c1 - c0;
  const int ns = (ncols + kSI - 1) / kSI;
  auto row_of_rel = [&](int j) -> int64_t { return row_of(c0 + j); };
  // sum of the lane's 16 weights of one 32-column tile, columns >= nvalid masked
  auto tile_sum = [&](const f32x16 &u, int nvalid) __attribute__((always_inline)) -> uint32_t {
    return nvalid >= kCT ? lane_wsum<P, false, FOLD>(u, kCT, h) : lane_wsum<P, true, FOLD>(u, nvalid, h);
  };
  constexpr int kOps = stage_ops<D, false, W>();
  // Stage t in buffers t % 3.  The global rows of stage t + 2 were fetched one
  // step earlier (list lookups for the maintenance stages), so issuing its
  // loads never waits for the loads still in flight.
  // Two row sets used alternately (the loop is unrolled 6 = lcm(3, 2) times),
  // so that no register copy waits for a lookup still in flight.
  StageRows<D, W> rowsA, rowsB;
  using Rows = StageRows<D, W>;
  // stage s covers list entries c0 + s kSI ..; where those are consecutive rows
  // of one region (ordered candidates, bank slots in order) and whole-row
  // descriptors, the loads take the per-lane offsets of consecutive rows and no
  // row list is built
  constexpr bool kSeqRows = !kColSplit && MODE == RS_CHUNK;
  [[maybe_unused]] const StageOff<D, W> soff = stage_offsets<D, W>();
  auto stage_rows_for = [&](Rows &r, int st) __attribute__((always_inline)) {
    if constexpr (!kSeqRows) stage_rows<D, W>(r, st * kSI, ncols, row_of_rel);
  };
  auto stage_dma_for = [&](const Rows &r, int st, char *kd, char *ad) __attribute__((always_inline)) {
    if constexpr (kSeqRows)
      stage_dma_seq<D, false, W>(soff, c0 + st * kSI, colbase.k, colaug, nullptr, kd, ad, nullptr, col_row0, col_nrows);
    else stage_dma<D, false, kColSplit, W>(r, colbase, colaug, nullptr, kd, ad, nullptr, col_row0, col_nrows);
  };
  auto step = [&](int t, const char *kb, const char *ab, char *kn, char *an, Rows &use, Rows &fill)
      __attribute__((always_inline)) {
    if (t + 1 < ns) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kOps));
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
    stage_barrier();
    if (t + 2 < ns) {
      if (t + 3 < ns) stage_rows_for(fill, t + 3);
      stage_dma_for(use, t + 2, kn, an);
    }
    f32x16 u0, u1;
    stage_u<D, D <= 128 ? 4 : 0>(kb, ab, rf, u0, u1);
    const int nv0 = ncols - t * kSI;
    const int j0 = c0 + t * kSI;
    uint32_t s2 = tile_sum(u0, nv0);
    if (nv0 > kCT) s2 += tile_sum(u1, nv0 - kCT);
    if constexpr (MODE == RS_CHUNK) {
      chunk_sum += s2;
      const bool chunk_end = ((t + 1) % (kCkStride / kSI)) == 0 || t + 1 == ns;
      if (chunk_end) {
        const uint32_t tot = chunk_sum + __shfl_xor(chunk_sum, 32, 64);
        if (rv && h == 0) ws.ck[(rb + v) * ws.nck + (j0 / kCkStride)] = tot;
        chunk_sum = 0;
      }
    } else {
      S64 += s2;
    }
  };
  if (ns > 0) {
    stage_rows_for(rowsA, 0);
    stage_dma_for(rowsA, 0, sb.k0, sb.a0);
    if (ns > 1) {
      stage_rows_for(rowsB, 1);
      stage_dma_for(rowsB, 1, sb.k1, sb.a1);
      if (ns > 2) stage_rows_for(rowsA, 2);
    }
  }
  if constexpr (kPipe) {
    // Software pipeline at the granularity of one 32-column tile: the MFMAs of the next tile run interleaved with the
    // epilogue of the current one, so that one wave keeps the matrix cores and
    // the VALU busy at the same time.  Stage s (tiles 2 s, 2 s + 1) uses
    // buffers s % 3 and rows (s even ? rowsA : rowsB).  Iteration t: tile 1
    // of stage t with the epilogue of tile 0; then the wait for stage t + 1,
    // the barrier (every wave is done with the buffers of stage t), stage t + 3
    // issued into them, and tile 0 of stage t + 1 with the epilogue of tile 1.
    static_assert(kCkStride == kSI, "one prefix chunk per stage");
    int aoff[TileCfg<D>::kSteps];
    frag_offsets<D>(aoff);
    auto tile_mfma_ = [&](const char *kb, const char *ab, int half) __attribute__((always_inline)) -> f32x16 {
      return tile_mfma<D>(kb, ab, half, rf, aoff);
    };
    auto store_chunk = [&](int t, uint32_t s2) __attribute__((always_inline)) {
      if constexpr (MODE != RS_CHUNK) {
        S64 += s2;
        return;
      }
      const uint32_t tot = s2 + __shfl_xor(s2, 32, 64);
      if (rv && h == 0) ws.ck[(rb + v) * ws.nck + ((c0 + t * kSI) / kCkStride)] = tot;
    };
    f32x16 u;
    // iteration t for a full stage t that is not the last
    auto pstep = [&](int t, const char *kc, const char *ac, const char *kn, const char *an, char *kd, char *ad,
                     Rows &use, Rows &fill) __attribute__((always_inline)) {
      f32x16 x = tile_mfma_(kc, ac, 1);
      uint32_t s2 = lane_wsum<P, false, FOLD>(u, kCT, h);
      tile_interleave<D>();
      asm volatile("" : "+v"(s2));  // the epilogue of tile 0 stays beside the MFMAs of tile 1
      u = x;
      if (t + 2 < ns) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kOps));
      else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      stage_barrier();
      if (t + 3 < ns) {
        if (t + 4 < ns) stage_rows_for(fill, t + 4);
        stage_dma_for(use, t + 3, kd, ad);
      }
      x = tile_mfma_(kn, an, 0);
      s2 += lane_wsum<P, false, FOLD>(u, kCT, h);
      tile_interleave<D>();
      u = x;
      store_chunk(t, s2);
    };
    if (ns > 0) {
      if (ns > 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kOps));
      else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      stage_barrier();
      if (ns > 2) {
        if (ns > 3) stage_rows_for(rowsB, 3);
        stage_dma_for(rowsA, 2, sb.k2, sb.a2);
      }
      u = tile_mfma_(sb.k0, sb.a0, 0);
    }
    // iteration t: stage t in buffers t % 3, stage t + 1 in (t + 1) % 3, stage t + 3
    // issued into t % 3 with rows (t odd ? rowsA : rowsB), rows of t + 4 fetched
    for (int t = 0; t + 1 < ns; t += 6) {
      pstep(t, sb.k0, sb.a0, sb.k1, sb.a1, sb.k0, sb.a0, rowsB, rowsA);
      if (t + 2 < ns) pstep(t + 1, sb.k1, sb.a1, sb.k2, sb.a2, sb.k1, sb.a1, rowsA, rowsB);
      if (t + 3 < ns) pstep(t + 2, sb.k2, sb.a2, sb.k0, sb.a0, sb.k2, sb.a2, rowsB, rowsA);
      if (t + 4 < ns) pstep(t + 3, sb.k0, sb.a0, sb.k1, sb.a1, sb.k0, sb.a0, rowsA, rowsB);
      if (t + 5 < ns) pstep(t + 4, sb.k1, sb.a1, sb.k2, sb.a2, sb.k1, sb.a1, rowsB, rowsA);
      if (t + 6 < ns) pstep(t + 5, sb.k2, sb.a2, sb.k0, sb.a0, sb.k2, sb.a2, rowsA, rowsB);
    }
    // the last stage (possibly partial); u holds its tile 0
    if (ns > 0) {
      const int t = ns - 1;
      const int nv0 = ncols - t * kSI;
      uint32_t s2 = tile_sum(u, nv0);
      if (nv0 > kCT) {
        // one call per buffer: the LDS arrays stay compile-time known (no generic pointers)
        f32x16 x;
        if (t % 3 == 0) x = tile_mfma_(sb.k0, sb.a0, 1);
        else if (t % 3 == 1) x = tile_mfma_(sb.k1, sb.a1, 1);
        else x = tile_mfma_(sb.k2, sb.a2, 1);
        s2 += tile_sum(x, nv0 - kCT);
      }
      store_chunk(t, s2);
    }
  } else {
  // step t issues stage t + 2 with the rows fetched at step t - 1 and fetches
  // those of stage t + 3: stage t + 2 uses rowsA when t is even
  for (int t = 0; t < ns; t += 6) {
    step(t, sb.k0, sb.a0, sb.k2, sb.a2, rowsA, rowsB);
    if (t + 1 < ns) step(t + 1, sb.k1, sb.a1, sb.k0, sb.a0, rowsB, rowsA);
    if (t + 2 < ns) step(t + 2, sb.k2, sb.a2, sb.k1, sb.a1, rowsA, rowsB);
    if (t + 3 < ns) step(t + 3, sb.k0, sb.a0, sb.k2, sb.a2, rowsB, rowsA);
    if (t + 4 < ns) step(t + 4, sb.k1, sb.a1, sb.k0, sb.a0, rowsA, rowsB);
    if (t + 5 < ns) step(t + 5, sb.k2, sb.a2, sb.k1, sb.a1, rowsB, rowsA);
  }
  }
  if constexpr (MODE == RS_CHUNK) return;
  if constexpr (MODE == RS_FIXUP) {
    fixup_finish(S64);
    return;
  }
  uint64_t tot = S64;
  tot += __shfl_xor(tot, 32, 64);
  if (!rv || h != 0) return;
  {
    int64_t *dst = MODE == RS_SURV_EV ? ws.sub : ws.sub_adm;
    atomicAdd(reinterpret_cast<unsigned long long *>(&dst[out_idx]), (unsigned long long)tot);
  }
}

template <int D, int P, int MODE, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * gram_waves<D>(), gram_waves<D>() == 4 ? 3 : 2) void k_rowsum_mfma(
    dkv_bank bank, const void *seg_k, const void *seg_v, Geom g, Prm p, Workspace ws, int64_t *out) {
  constexpr int KB = SCfg<D>::KEYB, AB = SCfg<D>::AUGB;
  __shared__ __attribute__((aligned(1024))) char k0[KB], k1[KB], k2[KB];
  __shared__ __attribute__((aligned(16))) char a0[AB], a1[AB], a2[AB];
  const StageBufs<D> sb{k0, k1, k2, a0, a1, a2, nullptr};
  rowsum_body<D, P, MODE, FOLD, KV>(bank, seg_k, seg_v, g, p, ws, out, blockIdx.x, blockIdx.y, blockIdx.z, sb);
}

// ---------------------------------------------------------------------------
// Symmetric Grams (W_xy = W_yx bit for bit, keys on the grid): each item's sum of
// weights to the other items of one list, the admitted candidates (ADM) or a
// bank's live slots.  A workgroup holds 32 W items, 32 per wave, as the A operand,
// so the lane (h, n) gets the weights of streamed item n with the wave's held
// items 8 (i / 4) + 4 h + i % 4 in register i, and both sums are cheap: the held
// items' in 16 integer accumulators per lane (half an instruction per weight,
// two tiles at a time; one reduction over the lanes per work item), the streamed
// item's as the sum of the lane's 16 weights (half an instruction each), one LDS
// add per lane and tile, and one 64-bit atomic per item and stage.  Bound by the
// VALU (the exact epilogue); each pair is evaluated once, where an epilogue that
// reduced the other side over the lanes tile by tile took 45 more instructions.
//
// Block J (items [32 W J, 32 W (J + 1))) takes its own block (both orders, each
// item's own sum only) and, in runs of several stages, the items after it.
// ---------------------------------------------------------------------------
// Stages per run: shorter runs pay the held rows' load more often, longer ones
// balance worse (sym_stages picks).
constexpr int kSymLong = 12, kSymShort = 4;

// Sum over the 16 lanes of each DPP row of the lane's 16 values: returns the row's sum of value lane % 16.
__device__ __forceinline__ uint32_t row_transpose_sum(const uint32_t (&w)[16], int l) {
  const bool b3 = (l >> 3) & 1;
  uint32_t a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t keep = b3 ? w[i + 8] : w[i], send = b3 ? w[i] : w[i + 8];
    a[i] = keep + dpp_mov<0x140>(send);  // row mirror: lane 15 - x (bit 3 flipped)
  }
  return row_transpose_tail(a, l);
}

// Work items of n list items in blocks of 32 W: block J's runs over the items after
// it, then every block's own.  A run of st stages spans S = st kSI / (32 W) blocks, so
// block J with k blocks after it has ceil(k / S) runs (a last block that is not
// full leaves that as it is), and the items of the blocks with at most k blocks
// after them are a closed form: no walk over the blocks per item (up to 74 dependent
// scalar steps at 9,360 items).
template <int W, int ST>
constexpr int kSymBlocks = ST * kSI / (32 * W);
template <int W>
__host__ __device__ constexpr int sym_before(int k, int st) {  // runs of the blocks with at most k blocks after them
  static_assert(kSymShort * kSI % (32 * W) == 0 && kSymLong % kSymShort == 0, "runs of whole blocks");
  constexpr int SL = kSymBlocks<W, kSymLong>, SS = kSymBlocks<W, kSymShort>;
  const int S = st == kSymLong ? SL : SS, q = st == kSymLong ? k / SL : k / SS;  // divisions by constants
  return S * q * (q + 1) / 2 + (k - S * q) * (q + 1);
}
template <int W>
__host__ __device__ constexpr int sym_items(int n, int st) {
  const int nb = (n + 32 * W - 1) / (32 * W);
  return nb + (nb > 0 ? sym_before<W>(nb - 1, st) : 0);
}
// Item -> block J and run (-1: the block's own).
template <int W>
__device__ __forceinline__ void sym_item(int n, int st, int item, int &J, int &run) {
  constexpr int SL = kSymBlocks<W, kSymLong>, SS = kSymBlocks<W, kSymShort>;
  const int S = st == kSymLong ? SL : SS;
  const int nb = (n + 32 * W - 1) / (32 * W), off = sym_before<W>(nb - 1, st);
  if (item >= off) {
    J = item - off;
    run = -1;
    return;
  }
  // blocks with q S + 1 .. (q + 1) S blocks after them have q + 1 runs each
  int q = (int)((__builtin_sqrtf(1.0f + (st == kSymLong ? 8.0f / SL : 8.0f / SS) * (float)item) - 1.0f) * 0.5f);
  while (S * q * (q + 1) / 2 > item) --q;
  while (S * (q + 1) * (q + 2) / 2 <= item) ++q;
  const int t = item - S * q * (q + 1) / 2, u = t / (q + 1);
  J = nb - 2 - S * q - u;
  run = t - u * (q + 1);
}

// Stages per run of B symmetric Grams of up to n items: short runs where long ones
// leave workgroup slots of the chip empty (32 banks x 999, d = 64: maintenance 512
// long items on 768 slots, update 91 us; with short ones 75 us including 10 us of
// the sort's).  Above a round the length matters little (12 x 4,680: 127 us with
// 12 stages, 126 with 8; densities of 12 x 9,360: 380 and 390).
template <int W>
inline int sym_stages(uint64_t B, int n) {
  const uint64_t items = B * (uint64_t)sym_items<W>(n, kSymLong), slots = W == kWaves ? 3 * 256 : 256;
  return items >= slots ? kSymLong : kSymShort;
}

template <int D, int P, bool FOLD, bool KV, bool ADM>
__device__ __forceinline__ void sym_body(const dkv_bank &bank, const void *seg_k, const void *seg_v, const Geom &g,
                                         const Prm &p, const Workspace &ws, int n_items, int st, int item, int b,
                                         const StageBufs<D> &sb) {
  constexpr int W = gram_waves<D>();
  int J, run;
  sym_item<W>(n_items, st, item, J, run);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, h = l >> 5, n = l & 31;
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  const Desc src = ADM ? Desc{static_cast<const uint16_t *>(seg_k), static_cast<const uint16_t *>(seg_v)}
                       : Desc{static_cast<const uint16_t *>(bank.k), static_cast<const uint16_t *>(bank.v)};
  const uint4 *aug = ADM ? ws.caug : ws.baug;
  int64_t *dst = ADM ? ws.mut_adm + nb : ws.sub + rb;
  const int64_t row0 = ADM ? (int64_t)nb : (int64_t)rb;
  auto row_of = [&](int j) -> int64_t { return ADM ? (int64_t)(nb + ws.adm_list[nb + j]) : (int64_t)(rb + j); };
  // streamed items [j0, j1)
  const bool diag = run < 0;
  const int hold0 = J * 32 * W;
  const int j0 = diag ? hold0 : hold0 + 32 * W + run * st * kSI;
  const int j1 = min(n_items, j0 + (diag ? 32 * W : st * kSI));
  const int ncols = j1 - j0, ns = (ncols + kSI - 1) / kSI;
  // stage loads: a bank's slots in order take the per-lane offsets of consecutive
  // rows; list rows are fetched one stage ahead of their use
  constexpr bool kSeq = !ADM && !KV;
  StageRows<D, W> rows;
  [[maybe_unused]] const StageOff<D, W> soff = stage_offsets<D, W>();
  auto fetch = [&](int st) __attribute__((always_inline)) {
    if constexpr (!kSeq) stage_rows<D, W>(rows, st * kSI, ncols, [&](int j) { return row_of(j0 + j); });
  };
  auto issue = [&](int st, char *kd, char *ad) __attribute__((always_inline)) {
    if constexpr (kSeq) stage_dma_seq<D, false, W>(soff, j0 + st * kSI, src.k, aug, nullptr, kd, ad, nullptr, row0, g.Mcap);
    else stage_dma<D, false, KV, W>(rows, src, aug, nullptr, kd, ad, nullptr, row0, ADM ? g.N : g.Mcap);
  };
  fetch(0);
  issue(0, sb.k0, sb.a0);
  if (ns > 1) {
    fetch(1);
    issue(1, sb.k1, sb.a1);
    if (ns > 2) fetch(2);
  }
  for (int i = threadIdx.x; i < 3 * kSI; i += 64 * W) sb.cb[i] = 0;  // before the first stage barrier
  // held items; past the list's end an item far from everything, whose weights round to 0
  RowFrag<D> rf;
  {
    const int c = hold0 + wave * 32 + n;
    const bool v = c < n_items;
    const int64_t r = row_of(min(c, n_items - 1));
    load_row_frag<D, FOLD, KV>(rf, src, r, ADM ? ws.cnorm[r] : bank.knorm[r], v, -2.0f * p.inv_sigma2, p.inv_sigma2);
    if (!v && h == 0) {
      constexpr uint32_t far = 0x4C80u;  // bf16 2^26: t > 2^24
      rf.b[TileCfg<D>::kSteps] = __builtin_bit_cast(
          bf16x8, u32x4{(uint32_t)kOne | ((uint32_t)kOne << 16), (uint32_t)kOne | (far << 16), 0u, 0u});
    }
  }
  int aoff[TileCfg<D>::kSteps];
  frag_offsets<D>(aoff);
  // t of one 32-item streamed tile: the held items as A, the streamed ones as B
  auto tile = [&](const char *kb, const char *ab, int half) __attribute__((always_inline)) -> f32x16 {
    constexpr int KS = TileCfg<D>::kSteps;
    bf16x8 y[KS + 1];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      y[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kb + 32 * half * SCfg<D>::RB + aoff[kk]));
    y[KS] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(ab + 16 * (32 * half + n)));
    f32x16 x = {};
#pragma unroll
    for (int kk = 0; kk <= KS; ++kk) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rf.b[kk], y[kk], x, 0, 0, 0);
    return x;
  };
  uint32_t acc[16], tiles = 0;  // held items' sums (raw weights: each with kMagic), tiles added
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0;
  auto raw16 = [&](const f32x16 &u, uint32_t (&w)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = weight_raw<P, FOLD>(u[i], 8388608.0f);
  };
  auto sum16 = [&](const uint32_t (&w)[16]) __attribute__((always_inline)) -> uint32_t {
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += w[i];
    return s;
  };
  constexpr int kOps = stage_ops<D, false, W>();
  constexpr uint32_t kStreamBias = 2u * W * 16u * kMagic;  // of a streamed item's sum: 2 W lanes x 16 weights
  // the sums of stage t's streamed items, complete before the barrier just passed, to the global ones
  auto flush = [&](int t) __attribute__((always_inline)) {
    if ((int)threadIdx.x < kSI) {
      uint32_t *c = sb.cb + (t % 3) * kSI + threadIdx.x;
      const uint32_t v = *c - kStreamBias;
      *c = 0;
      const int j = j0 + t * kSI + (int)threadIdx.x;
      if (j < j1) atomicAdd(reinterpret_cast<unsigned long long *>(&dst[j]), (unsigned long long)v);
    }
  };
  // one tile with masks: streamed items past j1, and in the own block an item with itself
  auto masked = [&](const f32x16 &u, int t, int half) __attribute__((always_inline)) {
    uint32_t w[16];
    raw16(u, w);
    const int j = t * kSI + 32 * half + n;  // streamed item, from j0
    const bool v = j < ncols;
    const bool own = diag && t * kSI + 32 * half == wave * 32;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      w[i] = v && !(own && n == col_of_reg(i, h)) ? w[i] : kMagic;
      acc[i] += w[i];
    }
    ++tiles;
    if (!diag) atomicAdd(&sb.cb[(t % 3) * kSI + 32 * half + n], sum16(w));
  };
  auto stage_wait = [&](bool more) __attribute__((always_inline)) {
    if (more) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kOps));
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
    stage_barrier();
  };
  if (diag || D > 128) {
    // plain loop: wait, barrier, both tiles
    auto step = [&](int t, const char *kb, const char *ab, char *kn, char *an) __attribute__((always_inline)) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      stage_barrier();
      if (t + 2 < ns) {
        issue(t + 2, kn, an);
        if (t + 3 < ns) fetch(t + 3);
      }
      if (!diag && t > 0) flush(t - 1);
      masked(tile(kb, ab, 0), t, 0);
      masked(tile(kb, ab, 1), t, 1);
    };
    for (int t = 0; t < ns; t += 3) {
      step(t, sb.k0, sb.a0, sb.k2, sb.a2);
      if (t + 1 < ns) step(t + 1, sb.k1, sb.a1, sb.k0, sb.a0);
      if (t + 2 < ns) step(t + 2, sb.k2, sb.a2, sb.k1, sb.a1);
    }
  } else if constexpr (D <= 128) {
    // tile-granular pipeline as in the score kernel; iteration t: tile 1 of stage
    // t beside the epilogue of tile 0, the barrier for stage t + 1, tile 0 of
    // stage t + 1 beside the epilogue of tile 1
    f32x16 u;
    auto pstep = [&](int t, const char *kc, const char *ac, const char *kn, const char *an, char *kd, char *ad)
        __attribute__((always_inline)) {
      uint32_t w0[16], w1[16];
      f32x16 x = tile(kc, ac, 1);
      raw16(u, w0);
      uint32_t s0 = sum16(w0);
      tile_interleave<D>();
      asm volatile("" : "+v"(s0));  // the epilogue of tile 0 stays beside the MFMAs of tile 1
      atomicAdd(&sb.cb[(t % 3) * kSI + n], s0);
      u = x;
      stage_wait(t + 2 < ns);
      if (t + 3 < ns) {
        issue(t + 3, kd, ad);
        if (t + 4 < ns) fetch(t + 4);
      }
      if (t > 0) flush(t - 1);
      x = tile(kn, an, 0);
      raw16(u, w1);
      uint32_t s1 = sum16(w1);
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] += w0[i] + w1[i];
      tile_interleave<D>();
      asm volatile("" : "+v"(s1));
      atomicAdd(&sb.cb[(t % 3) * kSI + 32 + n], s1);
      tiles += 2;
      u = x;
    };
    stage_wait(ns > 1);
    if (ns > 2) {
      issue(2, sb.k2, sb.a2);
      if (ns > 3) fetch(3);
    }
    u = tile(sb.k0, sb.a0, 0);
    for (int t = 0; t + 1 < ns; t += 3) {
      pstep(t, sb.k0, sb.a0, sb.k1, sb.a1, sb.k0, sb.a0);
      if (t + 2 < ns) pstep(t + 1, sb.k1, sb.a1, sb.k2, sb.a2, sb.k1, sb.a1);
      if (t + 3 < ns) pstep(t + 2, sb.k2, sb.a2, sb.k0, sb.a0, sb.k2, sb.a2);
    }
    const int t = ns - 1;  // u: its tile 0
    f32x16 x;
    if (t % 3 == 0) x = tile(sb.k0, sb.a0, 1);
    else if (t % 3 == 1) x = tile(sb.k1, sb.a1, 1);
    else x = tile(sb.k2, sb.a2, 1);
    masked(u, t, 0);
    masked(x, t, 1);
  }
  if (!diag) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
    stage_barrier();
    if (D <= 128 && ns > 1) flush(ns - 2);
    flush(ns - 1);
  }
  // the held items' sums over the lanes
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] -= tiles * kMagic;
  const uint32_t tot = row_transpose_sum(acc, l);
  const int c = hold0 + wave * 32 + col_of_reg(l & 15, h);
  if (c < n_items) atomicAdd(reinterpret_cast<unsigned long long *>(&dst[c]), (unsigned long long)tot);
}

// Maintenance work items (Supp. C): per bank, the (row block, column split)
// pairs of survivors x evicted (row blocks of the survivors x splits of the
// evicted) and admitted x survivors, and the items of admitted x admitted.  A
// bank that admits nothing and releases nothing has none.
struct MaintItems {
  int rows_s, rows_a, n_se, n_ab, rs;
};
// rpw: rows per workgroup of the maintenance Grams
__device__ __forceinline__ MaintItems maint_items(const Geom &g, const Workspace &ws, int b, int rpw) {
  const int ne = ws.n_ev[b], rs = ws.r_star[b / g.gs], ns = ws.m[b] - ne;
  MaintItems it;
  it.rs = rs;
  it.rows_s = (ns + rpw - 1) / rpw;
  it.rows_a = (rs + rpw - 1) / rpw;
  it.n_se = it.rows_s * ((ne + kColsPerSplit - 1) / kColsPerSplit);
  it.n_ab = it.rows_a * ((ns + kColsPerSplit - 1) / kColsPerSplit);
  return it;
}

// Workgroups that walk work items of unequal size: five rounds of the CUs' three each.
constexpr unsigned kItemWgs = 4096;

// The maintenance Grams of every bank.
template <int D, int P, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * gram_waves<D>(), gram_waves<D>() == 4 ? 3 : 2) void k_maint_mfma(
    dkv_bank bank, const void *seg_k, const void *seg_v, Geom g, Prm p, Workspace ws, int st) {
  constexpr int W = gram_waves<D>(), kRpw = 32 * W;
  constexpr int KB = SCfg<D>::KEYB, AB = SCfg<D>::AUGB;
  __shared__ __attribute__((aligned(1024))) char k0[KB], k1[KB], k2[KB];
  __shared__ __attribute__((aligned(16))) char a0[AB], a1[AB], a2[AB];
  __shared__ __attribute__((aligned(16))) uint32_t cb[3 * kSI];
  __shared__ int pre[65];
  if (!ws.crossed[0]) return;  // no bank admits or releases anything
  const StageBufs<D> sb{k0, k1, k2, a0, a1, a2, cb};
  walk_items(
      g.B, pre,
      [&](int b) {
        const MaintItems it = maint_items(g, ws, b, kRpw);
        return it.n_se + it.n_ab + sym_items<W>(it.rs, st);
      },
      [&](int b, int i) __attribute__((always_inline)) {
        const MaintItems it = maint_items(g, ws, b, kRpw);
        __syncthreads();  // the previous item's LDS stages are done with
        if (i < it.n_se) {
          rowsum_body<D, P, RS_SURV_EV, FOLD, KV>(bank, seg_k, seg_v, g, p, ws, nullptr, i % it.rows_s, i / it.rows_s, b,
                                                  sb);
        } else if (i < it.n_se + it.n_ab) {
          const int j = i - it.n_se;
          rowsum_body<D, P, RS_ADM_BASE, FOLD, KV>(bank, seg_k, seg_v, g, p, ws, nullptr, j % it.rows_a, j / it.rows_a, b,
                                                   sb);
        } else {
          sym_body<D, P, FOLD, KV, true>(bank, seg_k, seg_v, g, p, ws, it.rs, st, i - it.n_se - it.n_ab, b,
                                          sb);
        }
      });
}

// From-scratch densities of every bank (Eq. 3).
template <int D, int P, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * gram_waves<D>(), gram_waves<D>() == 4 ? 3 : 2) void k_density_mfma(dkv_bank bank, Geom g,
                                                                                                    Prm p, Workspace ws, int st) {
  constexpr int W = gram_waves<D>();
  constexpr int KB = SCfg<D>::KEYB, AB = SCfg<D>::AUGB;
  __shared__ __attribute__((aligned(1024))) char k0[KB], k1[KB], k2[KB];
  __shared__ __attribute__((aligned(16))) char a0[AB], a1[AB], a2[AB];
  __shared__ __attribute__((aligned(16))) uint32_t cb[3 * kSI];
  __shared__ int pre[65];
  const StageBufs<D> sb{k0, k1, k2, a0, a1, a2, cb};
  walk_items(
      g.B, pre, [&](int b) { return sym_items<W>(ws.m[b], st); },
      [&](int b, int i) __attribute__((always_inline)) {
        __syncthreads();  // the previous item's LDS stages are done with
        sym_body<D, P, FOLD, KV, false>(bank, nullptr, nullptr, g, p, ws, ws.m[b], st, i, b, sb);
      });
}

// ---------------------------------------------------------------------------
// First violating prefix length of every bank state (Eqs. 8-9).
//
// Chunk search: the state's group of 8 lanes holds its 64-candidate chunk
// sums, 16 per lane; a scan over the group gives every lane's prefix, and the
// lane whose 16 chunks contain the first prefix that lifts rho + P to tau b
// (2^k (rho + P) >= T b, integers) finds the chunk and how much of that
// chunk's weight is still needed.  Then the exact length inside the chunk,
// with the same binary32 weights.  States that never reach the bound within
// the tested prefixes get R + 1; states whose empty prefix already violates 0.
// ---------------------------------------------------------------------------
constexpr int kCrossLanes = 8;                      // lanes per state in the chunk search
constexpr int kCrossPerLane = 16;                   // chunk sums per lane
constexpr int kCrossStates = 64 / kCrossLanes;      // states per chunk-search pass of a wave

// v of the lane O below within a group of 8 lanes (a DPP row shift: the group
// lies in one row of 16 lanes), 0 for the group's first O lanes (q < O).  A DPP
// read from a lane that is switched off returns 0, so the shift runs with every
// lane on (the empty asm keeps it out of the branch of q >= O) and the select
// follows.
template <int O>
__device__ __forceinline__ uint64_t group_shr_u64(uint64_t v, int q) {
  static_assert(O >= 1 && O < kCrossLanes, "shift within a group");
  uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0x110 + O, 0xF, 0xF, true);
  uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), 0x110 + O, 0xF, 0xF, true);
  asm volatile("" : "+v"(lo), "+v"(hi));
  return q >= O ? ((uint64_t)hi << 32) | lo : 0ull;
}

struct CrossFind {
  bool pos;       // the bound lies above rho (else the empty prefix violates)
  bool hit;       // this lane's chunks hold the first prefix that reaches it
  int ch;         // that chunk (hit lane only)
  uint32_t need;  // the bound minus rho minus every chunk before it, in [1, 2^29] (hit lane only)
};

// Chunk search for one bank row by lane q of its group: the loads (issued
// together for several rows), then the search; nch chunks are tested.
struct CrossRow {
  int64_t base, rho;
  uint4 x[kCrossPerLane / 4];
};

__device__ __forceinline__ CrossRow cross_load(const dkv_bank &bank, const Workspace &ws, size_t row, int q, int nch) {
  CrossRow r;
  r.base = bank.base[row];
  r.rho = bank.rho[row];
  // 16-byte groups of the row (nck >= 4, a multiple of 4, at least nch); only
  // those that hold tested chunks are read (the rest may be stale), clamped
  const uint4 *ckr = reinterpret_cast<const uint4 *>(ws.ck + row * ws.nck);
  const int last = ws.nck / 4 - 1;
#pragma unroll
  for (int v4 = 0; v4 < kCrossPerLane / 4; ++v4) {
    const int grp = (kCrossPerLane * q) / 4 + v4;
    r.x[v4] = 4 * grp < nch ? ckr[min(grp, last)] : uint4{0u, 0u, 0u, 0u};
  }
  return r;
}

__device__ __forceinline__ CrossFind cross_find(const CrossRow &r, const Prm &p, int nch, int q) {
  static_assert((DKV_MAX_CANDIDATES + kCkStride - 1) / kCkStride <= kCrossLanes * kCrossPerLane,
                "every chunk sum of a state is held by its lane group");
  const int64_t lim = ((int64_t)p.tau_num * r.base + ((1ll << p.tau_shift) - 1)) >> p.tau_shift;
  const int64_t thr = lim - r.rho;
  uint32_t c[kCrossPerLane];
#pragma unroll
  for (int v4 = 0; v4 < kCrossPerLane / 4; ++v4) {
    const int c0 = kCrossPerLane * q + 4 * v4;
    c[4 * v4 + 0] = c0 + 0 < nch ? r.x[v4].x : 0u;
    c[4 * v4 + 1] = c0 + 1 < nch ? r.x[v4].y : 0u;
    c[4 * v4 + 2] = c0 + 2 < nch ? r.x[v4].z : 0u;
    c[4 * v4 + 3] = c0 + 3 < nch ? r.x[v4].w : 0u;
  }
  // a chunk sum is at most 64 x 2^23 = 2^29: seven of them fit 32 bits, eight may not
  uint32_t a7 = 0, b7 = 0;
#pragma unroll
  for (int t = 0; t < 7; ++t) {
    a7 += c[t];
    b7 += c[8 + t];
  }
  const uint64_t s8a = (uint64_t)a7 + c[7], tot = s8a + (uint64_t)b7 + c[15];
  // inclusive scan over the group (DPP row shifts: a group of 8 lies in one row of 16 lanes)
  uint64_t incl = tot;
  incl += group_shr_u64<1>(incl, q);
  incl += group_shr_u64<2>(incl, q);
  incl += group_shr_u64<4>(incl, q);
  // what this lane's chunks must still supply; the crossing lies in them iff it is in (0, tot]
  const int64_t need_l = thr - (int64_t)(incl - tot);
  CrossFind f;
  f.pos = thr > 0;
  f.hit = f.pos && need_l > 0 && need_l <= (int64_t)tot;
  // the half of the lane's chunks that holds it, and the rest in [1, 2^32] (32 bits after -1)
  const bool hi = need_l > (int64_t)s8a;
  const uint32_t nd1 = (uint32_t)((uint64_t)(hi ? need_l - (int64_t)s8a : need_l) - 1u);
  // chunks of that half before the crossing: those whose end prefix is still below the bound
  // (the half's full sum reaches it, so at most seven, whose prefixes fit 32 bits)
  uint32_t pr = 0, pre = 0;
  int cnt = 0;
#pragma unroll
  for (int t = 0; t < 7; ++t) {
    pr += hi ? c[8 + t] : c[t];
    if (pr <= nd1) {
      ++cnt;
      pre = pr;
    }
  }
  f.ch = kCrossPerLane * q + (hi ? 8 : 0) + cnt;
  f.need = nd1 - pre + 1u;
  return f;
}

// The whole crossing search over every tested prefix, for the groups that the
// first part leaves open (every group when first crossings are requested).
// A wave takes 32 states, a workgroup 128.
// The chunk search runs in four passes of eight states; each state's result then
// moves to lanes n and n + 32 (n = its index in the wave).  The exact walk: the
// workgroup's crossing chunks, in increasing order, each staged through LDS as a
// column stage of the Gram kernels (two buffers, alternating), and in every wave
// that has a state crossing there one 64 x 32 MFMA Gram with the Gram stages' own
// tiles: A = the chunk's ordered candidates (two tiles of 32) with their norm
// steps, B = the 32 states as row items, so lane (n, h) gets t of state n with
// candidates 8 k + 4 h + j (registers 4 k + j) of each tile, bit for bit the t
// that made the chunk sums; each lane keeps the Gram of its own chunk.  Then,
// once per lane, the weights summed in candidate order (the two halves exchange
// their 4-candidate group sums), and the crossing length is one plus the number
// of candidates whose inclusive prefix is still below the need.
constexpr int kCrossWaveStates = 32;

template <int D, int P, bool FOLD, bool KV>
__device__ __forceinline__ void cross_body(const dkv_bank &bank, const Geom &g, const Prm &p, const Workspace &ws,
                                           int32_t *out_first, int b, int bx) {
  static_assert(kCkStride == 64, "two 32-candidate tiles per chunk");
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int grp = l / kCrossLanes, q = l % kCrossLanes, n32 = l & 31, hw = l >> 5;
  const int i0 = (bx * kWaves + wave) * kCrossWaveStates;
  const int m = ws.m[b], R = ws.R[b];
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  const int nch = (R + kCkStride - 1) / kCkStride;
  // per state of this lane's column: whether its bound lies above rho, whether
  // it crosses within the tested prefixes, the crossing chunk and the need
  int my_ch = 0;
  uint32_t my_need = 0;
  bool my_pos = false, my_walk = false;
  constexpr int kPasses = kCrossWaveStates / kCrossStates;
  CrossRow rows[kPasses];  // every pass's loads in flight together
#pragma unroll
  for (int ps = 0; ps < kPasses; ++ps)
    rows[ps] = cross_load(bank, ws, rb + min(i0 + kCrossStates * ps + grp, m - 1), q, nch);
#pragma unroll
  for (int ps = 0; ps < kPasses; ++ps) {
    const int s = kCrossStates * ps + grp;
    const bool valid = i0 + s < m;
    const CrossFind f = cross_find(rows[ps], p, nch, q);
    const unsigned long long pos = __ballot(valid && f.pos);
    const unsigned long long hits = __ballot(valid && f.hit);
    // group g8 of this pass -> lanes n32 = 8 ps + g8
    const int g8 = (n32 - kCrossStates * ps) & (kCrossStates - 1);
    const unsigned gbits = (unsigned)(hits >> (kCrossLanes * g8)) & 0xFFu;
    const int src = kCrossLanes * g8 + (gbits ? __ffs(gbits) - 1 : 0);
    const int ch = __shfl(f.ch, src, 64);
    const uint32_t nd = __shfl(f.need, src, 64);
    if ((n32 >> 3) == ps) {
      my_ch = ch;
      my_need = nd;
      my_pos = (pos >> (kCrossLanes * g8)) & 1ull;
      my_walk = gbits != 0;
    }
  }
  int first = my_pos ? R + 1 : 0;
  // the workgroup's crossing chunks (at most 128: four words)
  __shared__ uint32_t chunk_set[4];
  if (threadIdx.x < 4) chunk_set[threadIdx.x] = 0;
  __syncthreads();
  if (my_walk && hw == 0) atomicOr(&chunk_set[my_ch >> 5], 1u << (my_ch & 31));
  __syncthreads();
  uint32_t cs[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) cs[k] = __builtin_amdgcn_readfirstlane(chunk_set[k]);
  if (cs[0] | cs[1] | cs[2] | cs[3]) {  // uniform over the workgroup
    // B operand: this lane's state as the Gram stages hold a row item (keys
    // times -2 / sigma^2 and the norm step); read for the states that walk only
    // (the others' columns of the Gram are not used)
    const int64_t srow = (int64_t)(rb + min(i0 + n32, m - 1));
    RowFrag<D> rf;
    load_row_frag<D, FOLD, KV>(rf, Desc{static_cast<const uint16_t *>(bank.k), static_cast<const uint16_t *>(bank.v)},
                               srow, my_walk ? bank.knorm[srow] : 0.0f, my_walk, -2.0f * p.inv_sigma2, p.inv_sigma2);
    int aoff[TileCfg<D>::kSteps];
    frag_offsets<D>(aoff);
    // each crossing chunk's 64 ordered candidates go through a stage buffer
    // (two, alternating) exactly as in the chunk-sum Gram, so t and every
    // weight are those of the chunk sums bit for bit; each lane keeps the
    // Gram of its own chunk
    constexpr int KB = SCfg<D>::KEYB, AB = SCfg<D>::AUGB;
    __shared__ __attribute__((aligned(1024))) char kbuf[2][KB];
    __shared__ __attribute__((aligned(16))) char abuf[2][AB];
    const Desc OK{ws.sk, nullptr};
    const StageOff<D> soff = stage_offsets<D>();
    auto issue = [&](int c, int buf) __attribute__((always_inline)) {
      stage_dma_seq<D, false>(soff, c * kCkStride, OK.k, ws.saug, nullptr, kbuf[buf], abuf[buf], nullptr, (int64_t)nb,
                              g.N);
    };
    // the chunks in increasing order (uniform over the workgroup)
    auto pop_chunk = [&]() __attribute__((always_inline)) -> int {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (cs[k]) {
          const int c = 32 * k + __builtin_ctz(cs[k]);
          cs[k] &= cs[k] - 1;
          return c;
        }
      return -1;
    };
    f32x16 mine[2] = {};
    bool partial = false;
    int c = pop_chunk(), buf = 0;
    issue(c, 0);
    while (c >= 0) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      stage_barrier();  // every wave's loads of chunk c landed; every wave is done with the other buffer
      const int cn = pop_chunk();
      if (cn >= 0) issue(cn, buf ^ 1);
      partial = partial || (c + 1) * kCkStride > R;
      const bool keep = my_walk && my_ch == c;
      if (__ballot(keep)) {  // uniform over the wave
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) {
          const f32x16 x = tile_mfma<D>(kbuf[buf], abuf[buf], tl, rf, aoff);
#pragma unroll
          for (int r = 0; r < 16; ++r) mine[tl][r] = keep ? x[r] : mine[tl][r];
        }
      }
      c = cn;
      buf ^= 1;
    }
    // weights in candidate order inside the lane (groups of four consecutive
    // candidates, k = 0..3 of each tile, the two halves alternating); candidates
    // past R weigh nothing (wave-uniform test: a chunk that ends past R)
    const int ch0 = my_ch * kCkStride;
    const int nvalid = min(kCkStride, R - ch0);
    uint32_t w[2][16], gs[2][4];
    auto weights = [&](auto mask_tag) __attribute__((always_inline)) {
      constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
      for (int tl = 0; tl < 2; ++tl) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          gs[tl][k] = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            uint32_t W = weight_raw<P, FOLD>(mine[tl][4 * k + j], 8388608.0f) - kMagic;
            if constexpr (MASK) {
              asm volatile("" : "+v"(W));  // computed for every lane, then masked
              W = 32 * tl + 8 * k + 4 * hw + j < nvalid ? W : 0u;
            }
            w[tl][4 * k + j] = W;
            gs[tl][k] += W;
          }
        }
      }
    };
    if (!__ballot(my_walk)) goto done;  // uniform over the wave
    if (partial) weights(std::integral_constant<bool, true>{});
    else weights(std::integral_constant<bool, false>{});
    // inclusive prefixes in candidate order; the crossing length is one plus the
    // number still below the need.  Candidates past R add nothing, so their
    // prefix equals the last valid one's and they are counted only if that one
    // was (cnt then reaches nvalid either way).
    uint32_t run = 0, cnt = 0;
    const uint32_t nd1 = my_need - 1u;
#pragma unroll
    for (int tl = 0; tl < 2; ++tl) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t other = __shfl_xor(gs[tl][k], 32, 64);
        uint32_t pr = run + (hw ? other : 0u);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          pr += w[tl][4 * k + j];
          cnt += pr <= nd1 ? 1u : 0u;
        }
        run += gs[tl][k] + other;
      }
    }
    cnt += __shfl_xor(cnt, 32, 64);
    if (my_walk) first = (int)cnt < nvalid ? ch0 + (int)cnt + 1 : ch0 + nvalid;  // the latter unreachable
  }
done:
  const int i = i0 + n32;
  if (hw == 0 && i < m) {
    ws.first[rb + i] = first;
    if (out_first) out_first[rb + i] = first;
  }
}

template <int D, int P, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * kWaves, D <= 128 ? 3 : 2) void k_cross_mfma(dkv_bank bank, Geom g, Prm p, Workspace ws,
                                                                            int32_t *out_first) {
  const int b = blockIdx.y;
  if (ws.more[b / g.gs] < kMoreOpen || (int)blockIdx.x * kWaves * kCrossWaveStates >= ws.m[b]) return;
  cross_body<D, P, FOLD, KV>(bank, g, p, ws, out_first, b, blockIdx.x);
}

// The first part of the crossing search in one pass: the prefix-chunk Gram of
// the workgroup's 128 bank states over the first kCrossFirst ordered
// candidates (4 waves x 32 states as row items, one 64-candidate chunk, read
// through the order, per column stage) stores each chunk sum as the chunk-sum
// Gram does, and every state whose running prefix reaches its bound within a
// chunk takes its first crossing there from the same weights, summed in
// candidate order (the two half-waves exchange their 4-candidate group sums);
// states that do not cross get R + 1, states already at their bound 0.
//
// c_r only grows with r, and the evictions a bank can make at a tested length,
// max(0, m + r - M), are at most E = max(0, m + R - M): a bank with more than E
// crossings r <= L is infeasible at every r >= L (Eqs. 9-10), so r* < L for its
// group (Eq. 11), and the crossings r <= L decide r*, the mandatory releases
// (first crossing <= r*) and the projected densities at r* (chunks before r*
// only).  ws.found counts a bank's crossings per chunk, on a line of its own:
// once they decide it after c chunks, workgroups of the bank that start later
// stop there and add nothing, and ws.more of the group drops to c, so that the
// second part leaves it out; unless every state's first crossing is wanted, when
// every workgroup walks all the chunks.
// (One counter line for all groups made its atomics and loads wait in turn: 1.4 ms.)
// Bound by the bank rows' reads where one chunk decides (360 banks of 9,280
// states at their growth bound: 547 us with four chunks, 535 with one; a workgroup's
// chain of dependent loads is what is left).
template <int D, int P, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * kWaves, D <= 128 ? 3 : 2) void k_first_part_mfma(dkv_bank bank, const void *seg_k,
                                                                                 const void *seg_v, Geom g, Prm p,
                                                                                 Workspace ws, int32_t *out_first) {
  static_assert(kCkStride == 2 * kCT, "two 32-candidate tiles per chunk");
  const int b = blockIdx.y;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, n = l & 31, hw = l >> 5;
  const int m = ws.m[b], R = ws.R[b];
  if ((int)blockIdx.x * 32 * kWaves >= m || ws.whole[b]) return;  // whole workgroup (the stages have barriers)
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  // the chunks that decide the bank, from its crossings by chunk (kMoreOpen: not decided)
  const int E = max(0, m + R - ws.M[b]);
  auto decided_at = [&](uint64_t found) {
    int sum = 0, c = 0;
    for (; c < kMoreOpen - 1; ++c) {
      sum += (int)(found >> (16 * c)) & 0xFFFF;
      if (sum > E) break;
    }
    return c + 1;
  };
  // with every state's first crossing wanted, nothing is counted: no workgroup stops early, whatever R is, and
  // `more` stays as k_begin left it
  const bool count = g.N > kCrossFirst && !out_first;
  uint64_t *found = ws.found + (size_t)b * kFoundStride;
  // as known when the workgroup starts (the same for all its waves)
  __shared__ int limit;
  if (threadIdx.x == 0)
    limit = count ? decided_at(__hip_atomic_load(found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : kMoreOpen;
  const int v = blockIdx.x * 32 * kWaves + wave * 32 + n;
  const bool rv = v < m;
  const int64_t row = (int64_t)(rb + min(v, m - 1));
  // the bound: the state violates once rho + P reaches ceil(T b / 2^k)
  const int64_t lim = ((int64_t)p.tau_num * bank.base[row] + ((1ll << p.tau_shift) - 1)) >> p.tau_shift;
  const int64_t thr = lim - bank.rho[row];
  int nch = min((R + kCkStride - 1) / kCkStride, kCrossFirst / kCkStride);
  int first = thr > 0 ? R + 1 : 0;
  bool open = thr > 0;  // not yet crossed
  uint64_t mine = 0;    // crossings of this wave by chunk, 16 bits each (lengths 0 count with the first)
  const unsigned long long at0 = __ballot(hw == 0 && rv && thr <= 0);
  mine += (uint64_t)__popcll(at0);
  if (nch > 0) {
    RowFrag<D> rf;
    load_row_frag<D, FOLD, KV>(rf, Desc{static_cast<const uint16_t *>(bank.k), static_cast<const uint16_t *>(bank.v)},
                               row, bank.knorm[row], rv, -2.0f * p.inv_sigma2, p.inv_sigma2);
    int aoff[TileCfg<D>::kSteps];
    frag_offsets<D>(aoff);
    constexpr int KB = SCfg<D>::KEYB, AB = SCfg<D>::AUGB;
    constexpr int NBUF = 2;
    __shared__ __attribute__((aligned(1024))) char kbuf[NBUF][KB];
    __shared__ __attribute__((aligned(16))) char abuf[NBUF][AB];
    const Desc SK{static_cast<const uint16_t *>(seg_k), static_cast<const uint16_t *>(seg_v)};
    StageRows<D, kWaves> rows;
    auto fetch = [&](int c) __attribute__((always_inline)) {
      stage_rows<D, kWaves>(rows, c * kCkStride, R, [&](int j) { return (int64_t)(nb + ws.order[nb + j]); });
    };
    auto issue = [&](int buf) __attribute__((always_inline)) {
      stage_dma<D, false, KV, kWaves>(rows, SK, ws.caug, nullptr, kbuf[buf], abuf[buf], nullptr, (int64_t)nb, g.N);
    };
    uint64_t run = 0;  // the state's prefix sum before chunk c
    fetch(0);
    issue(0);
    if (nch > 1) fetch(1);
    for (int c = 0; c < nch; ++c) {
      const int buf = c % NBUF;
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      stage_barrier();  // every wave's loads of chunk c landed; every wave is done with chunk c - 1's buffer
      if (c == 0) nch = min(nch, __builtin_amdgcn_readfirstlane(limit));
      if (c + 1 < nch) {
        issue(buf ^ 1);
        if (c + 2 < nch) fetch(c + 2);
      }
      const f32x16 x0 = tile_mfma<D>(kbuf[buf], abuf[buf], 0, rf, aoff);
      const f32x16 x1 = tile_mfma<D>(kbuf[buf], abuf[buf], 1, rf, aoff);
      // weights in candidate order inside the lane: tile tl, register 4 k + j is
      // candidate 32 tl + 8 k + 4 hw + j of the chunk; candidates past R weigh
      // nothing.  The weights stay raw (each with kMagic, taken off their sums), and
      // only a chunk that R cuts is masked: 6 instead of 9 instructions per weight.
      const int nvalid = min(kCkStride, R - c * kCkStride);
      uint32_t w[2][16], gsum[2][4];
#pragma unroll
      for (int tl = 0; tl < 2; ++tl)
#pragma unroll
        for (int i = 0; i < 16; ++i) w[tl][i] = weight_raw<P, FOLD>(tl ? x1[i] : x0[i], 8388608.0f);
      if (nvalid < kCkStride) {
#pragma unroll
        for (int tl = 0; tl < 2; ++tl)
#pragma unroll
          for (int i = 0; i < 16; ++i) w[tl][i] = 32 * tl + col_of_reg(i, hw) < nvalid ? w[tl][i] : kMagic;
      }
#pragma unroll
      for (int tl = 0; tl < 2; ++tl)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          gsum[tl][k] = w[tl][4 * k] + w[tl][4 * k + 1] + w[tl][4 * k + 2] + w[tl][4 * k + 3] - 4u * kMagic;
      uint32_t lane_tot = 0;
#pragma unroll
      for (int tl = 0; tl < 2; ++tl)
#pragma unroll
        for (int k = 0; k < 4; ++k) lane_tot += gsum[tl][k];
      const uint32_t tot = lane_tot + __shfl_xor(lane_tot, 32, 64);  // the chunk sum (at most 2^29)
      if (rv && hw == 0) ws.ck[(rb + v) * ws.nck + c] = tot;
      const bool hit = open && (int64_t)(run + tot) >= thr;
      if (__ballot(hit)) {  // uniform over the wave
        // inclusive prefixes in candidate order; the crossing is one plus the
        // number of candidates whose prefix is still below the need
        const uint32_t nd1 = hit ? (uint32_t)(thr - (int64_t)run) - 1u : 0u;
        uint32_t pr = 0, cnt = 0;
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t other = __shfl_xor(gsum[tl][k], 32, 64);
            uint32_t q = pr + (hw ? other : 0u);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              q += w[tl][4 * k + j] - kMagic;
              cnt += q <= nd1 ? 1u : 0u;
            }
            pr += gsum[tl][k] + other;
          }
        }
        cnt += __shfl_xor(cnt, 32, 64);
        if (hit) {
          first = c * kCkStride + (int)cnt + 1;
          open = false;
        }
        mine += (uint64_t)__popcll(__ballot(hit && hw == 0 && rv)) << (16 * c);
      }
      run += tot;
    }
  }
  if (hw == 0 && rv) {
    ws.first[rb + v] = first;
    if (out_first) out_first[rb + v] = first;
  }
  if (l == 0 && mine && count && (nch == 0 || limit > 1)) {
    const uint64_t old = atomicAdd(reinterpret_cast<unsigned long long *>(found), (unsigned long long)mine);
    const int at = decided_at(old + mine);
    if (at < kMoreOpen && at < decided_at(old)) atomicMin(&ws.more[b / g.gs], at);
  }
}

// Chunk sums of the ordered prefixes past the first part for the groups that it
// left open: one workgroup per 32 W states and split of `per` candidates.  (Over
// a fixed grid whose workgroups walked the open groups' items, this and the search
// after it kept 20 to 40 registers more and ran in lockstep: 64 full banks of 9,360
// states, d = 64: 685 us against 612 and 350 against 278; 48 of d = 128: 699
// against 635 and 402 against 369; 12 of [K; V] rows: the search 248 against 171.)
template <int D, int P, bool FOLD, bool KV>
__global__ __launch_bounds__(64 * gram_waves<D>(), gram_waves<D>() == 4 ? 3 : 2) void k_chunk_part_mfma(
    dkv_bank bank, const void *seg_k, const void *seg_v, Geom g, Prm p, Workspace ws, int per) {
  constexpr int KB = SCfg<D>::KEYB, AB = SCfg<D>::AUGB;
  if (ws.more[blockIdx.z / g.gs] < kMoreOpen) return;
  __shared__ __attribute__((aligned(1024))) char k0[KB], k1[KB], k2[KB];
  __shared__ __attribute__((aligned(16))) char a0[AB], a1[AB], a2[AB];
  const StageBufs<D> sb{k0, k1, k2, a0, a1, a2, nullptr};
  rowsum_body<D, P, RS_CHUNK, FOLD, KV>(bank, seg_k, seg_v, g, p, ws, nullptr, blockIdx.x, blockIdx.y, blockIdx.z, sb,
                                        kCrossFirst, per);
}

// Candidate keys and norm steps in score order, for the groups that the first
// part left open, so that the passes of the second stream contiguous rows: one thread per 16-byte chunk of kGatherRows key
// rows (every load and store instruction covers whole rows).
constexpr int kGatherRows = 4;

template <int D, bool KV>
__global__ __launch_bounds__(256) void k_gather_sorted(const void *seg_k, const void *seg_v, Geom g, Workspace ws) {
  constexpr int CH = D / 8;      // 16-byte chunks per bf16 row
  constexpr int RPP = 256 / CH;  // rows per workgroup pass
  static_assert(kGatherRows <= CH, "one metadata lane per row of the group");
  const Desc src{static_cast<const uint16_t *>(seg_k), static_cast<const uint16_t *>(seg_v)};
  const int c = threadIdx.x % CH;
  const int per_bank = (g.N + RPP * kGatherRows - 1) / (RPP * kGatherRows);
  __shared__ int pre[65];
  walk_items(
      g.B, pre, [&](int b) { return ws.more[b / g.gs] >= kMoreOpen ? per_bank : 0; },
      [&](int b, int i) __attribute__((always_inline)) {
        const int j0 = i * RPP * kGatherRows + threadIdx.x / CH;
        const size_t nb = (size_t)b * g.N;
        // loads from clamped (in-range) rows, unconditional so that they overlap
        int xs[kGatherRows];
#pragma unroll
        for (int u = 0; u < kGatherRows; ++u) xs[u] = ws.order[nb + min(j0 + u * RPP, g.N - 1)];
        u32x4 tmp[kGatherRows];
#pragma unroll
        for (int u = 0; u < kGatherRows; ++u)
          tmp[u] = *reinterpret_cast<const u32x4 *>(desc_chunk<D, KV>(src, (int64_t)(nb + xs[u]), c));
#pragma unroll
        for (int u = 0; u < kGatherRows; ++u)
          if (j0 + u * RPP < g.N) reinterpret_cast<u32x4 *>(ws.sk + (nb + j0 + u * RPP) * D)[c] = tmp[u];
        // lane c < kGatherRows of a row group copies the norm step of row c
        if (c < kGatherRows) {
          const int j = j0 + c * RPP;
          if (j < g.N) ws.saug[nb + j] = ws.caug[nb + ws.order[nb + j]];
        }
      });
}

inline unsigned cdiv(int a, int b) { return (unsigned)((a + b - 1) / b); }
inline unsigned grid_of(uint64_t items, unsigned most) { return (unsigned)(items < 1 ? 1 : (items < most ? items : most)); }
// Workgroups of a Gram kernel that the 256 CUs hold at once (three per CU; one
// of 8 waves at descriptor dimension 256): the grid of the exact re-scores, whose
// work items are equal.
template <int D>
constexpr unsigned kGramWgs = gram_waves<D>() == 4 ? 3 * 256 : 256;

// Workgroups that the chunk sums are split into at least, if they have the work.
constexpr uint64_t kChunkWgs = 49152;

// D is the descriptor dimension: the key dimension, or twice it for the
// [K; V] geometry (KV: the candidates' values seg_v and bank.v are read too).
template <int D, int P, bool F, bool KV>
void mfma_update_impl(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                      const dkv_update_out &out, const Workspace &ws, hipStream_t s, int stage) {
  constexpr int W = gram_waves<D>();
  const int T = 64 * W;
  const unsigned rowsM = cdiv(g.Mcap, 32 * W), rowsN = cdiv(g.N > 0 ? g.N : 1, 32 * W);
  const void *sv = seg.v;
  switch (stage) {
    case kGramScoreApprox:
      k_score_probe<D, P, F, KV><<<g.B, T, 0, s>>>(bank, seg.k, sv, g, p, ws);
      [[fallthrough]];
    case kGramScore:
      (stage == kGramScore ? k_score_mfma<D, P, F, KV, false> : k_score_mfma<D, P, F, KV, true>)
          <<<rowsN * cdiv(g.Mcap, kColsPerSplit) * (unsigned)g.B, T, 0, s>>>(bank, seg.k, sv, g, p, ws);
      break;
    case kGramOrder:
    case kGramOrderRest: {
      const int rest = stage == kGramOrderRest;
      if (!rest) k_order_mark<<<g.B, kOrderThreads, 0, s>>>(g, ws);
      k_rescore<D, P, F, KV><<<grid_of((uint64_t)rowsN * cdiv(g.Mcap, kColsPerSplit) * (unsigned)g.B, kGramWgs<D>), T, 0,
                               s>>>(bank, seg.k, sv, g, p, ws, rest);
      k_order_fix<<<g.B, kOrderThreads, 0, s>>>(g, ws, rest);
      break;
    }
    case kGramFirstPart:
    case kGramSecondPart: {
      // The crossing search in two parts: the chunk sums of the first
      // kCrossFirst ordered candidates and the crossings within them; then, for
      // the groups that this leaves open, the ordered copy and the chunk sums of
      // the rest and the whole search again.
      if (stage == kGramFirstPart) {
        k_first_part_mfma<D, P, F, KV><<<dim3(cdiv(g.Mcap, 32 * kWaves), g.B), 64 * kWaves, 0, s>>>(
            bank, seg.k, sv, g, p, ws, out.first_cross);
      } else {
        const unsigned B = (unsigned)g.B;
        k_gather_sorted<D, KV><<<grid_of((uint64_t)cdiv(g.N, 256 / (D / 8) * kGatherRows) * B, 1024), 256, 0, s>>>(
            seg.k, sv, g, ws);
        // splits of 1,024 candidates, longer ones where the workgroups are many (an empty one costs 0.3 ns: 85 us
        // for 360 decided banks in splits of 1,024)
        const unsigned rest = (unsigned)(g.N - kCrossFirst), most = cdiv((int)rest, 1024);
        const uint64_t want = (kChunkWgs + (uint64_t)rowsM * B - 1) / ((uint64_t)rowsM * B);
        const unsigned splits = want < most ? (unsigned)want : most;
        const unsigned per = cdiv(cdiv((int)rest, (int)splits), kCkStride) * kCkStride;
        k_chunk_part_mfma<D, P, F, KV><<<dim3(rowsM, cdiv((int)rest, (int)per), B), T, 0, s>>>(bank, seg.k, sv, g, p, ws,
                                                                                              (int)per);
        k_cross_mfma<D, P, F, KV><<<dim3(cdiv(g.Mcap, kWaves * kCrossWaveStates), B), 64 * kWaves, 0, s>>>(
            bank, g, p, ws, out.first_cross);
      }
      break;
    }
    case kGramFixup:
      k_rowsum_mfma<D, P, RS_FIXUP, F, KV><<<dim3(rowsM, 1, g.B), T, 0, s>>>(bank, seg.k, sv, g, p, ws, out.rho_tilde);
      break;
    case kGramMaint: {
      // at most this many items per bank, but for states that violated before the update
      const uint64_t y_ev = cdiv(g.N > 0 ? g.N : 1, kColsPerSplit), y_surv = cdiv(g.Mcap, kColsPerSplit);
      const int n_adm = g.N < g.Mcap ? g.N : g.Mcap, st = sym_stages<W>((unsigned)g.B, n_adm);
      const uint64_t items = rowsM * y_ev + (g.N > 0 ? rowsN : 0u) * y_surv + sym_items<W>(n_adm, st);
      k_maint_mfma<D, P, F, KV><<<grid_of(items * (unsigned)g.B, kItemWgs), T, 0, s>>>(bank, seg.k, sv, g, p, ws, st);
      break;
    }
    default:
      break;
  }
}

// The +1 of t = 1 + u rides in the MFMA when sigma^2 <= 2^11 (exact there).
inline bool fold_one(const Prm &p) { return p.inv_sigma2 >= 1.0f / 2048.0f; }

template <int D, bool KV>
void mfma_stage_d(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                  const dkv_update_out &out, const Workspace &ws, hipStream_t s, int stage) {
  const bool f = fold_one(p);
  if (p.p == 1) f ? mfma_update_impl<D, 1, true, KV>(bank, seg, g, p, out, ws, s, stage) : mfma_update_impl<D, 1, false, KV>(bank, seg, g, p, out, ws, s, stage);
  else if (p.p == 2) f ? mfma_update_impl<D, 2, true, KV>(bank, seg, g, p, out, ws, s, stage) : mfma_update_impl<D, 2, false, KV>(bank, seg, g, p, out, ws, s, stage);
  else f ? mfma_update_impl<D, 4, true, KV>(bank, seg, g, p, out, ws, s, stage) : mfma_update_impl<D, 4, false, KV>(bank, seg, g, p, out, ws, s, stage);
}

template <int D, int P, bool F, bool KV>
void mfma_score_impl(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                     int64_t *score_q, float *score_f, int64_t *density, const Workspace &ws, hipStream_t s) {
  constexpr int W = gram_waves<D>();
  const int T = 64 * W;
  if (g.N > 0 && (score_q || score_f)) {
    k_score_mfma<D, P, F, KV, false><<<cdiv(g.N, 32 * W) * cdiv(g.Mcap, kColsPerSplit) * (unsigned)g.B, T, 0, s>>>(
        bank, seg.k, seg.v, g, p, ws);
  }
  if (density) {
    const int st = sym_stages<W>((unsigned)g.B, g.Mcap);
    const uint64_t items = (uint64_t)sym_items<W>(g.Mcap, st) * (unsigned)g.B;
    k_density_mfma<D, P, F, KV><<<grid_of(items, kItemWgs), T, 0, s>>>(bank, g, p, ws, st);
  }
}

template <int D, bool KV>
void mfma_score_d(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p, int64_t *score_q,
                  float *score_f, int64_t *density, const Workspace &ws, hipStream_t s) {
  const bool f = fold_one(p);
  if (p.p == 1) f ? mfma_score_impl<D, 1, true, KV>(bank, seg, g, p, score_q, score_f, density, ws, s) : mfma_score_impl<D, 1, false, KV>(bank, seg, g, p, score_q, score_f, density, ws, s);
  else if (p.p == 2) f ? mfma_score_impl<D, 2, true, KV>(bank, seg, g, p, score_q, score_f, density, ws, s) : mfma_score_impl<D, 2, false, KV>(bank, seg, g, p, score_q, score_f, density, ws, s);
  else f ? mfma_score_impl<D, 4, true, KV>(bank, seg, g, p, score_q, score_f, density, ws, s) : mfma_score_impl<D, 4, false, KV>(bank, seg, g, p, score_q, score_f, density, ws, s);
}

}  // namespace

// The library compiles this file once per descriptor geometry (DKV_GRAM_DESC =
// descriptor dimension, DKV_GRAM_KV = concatenated [K; V] rows), in parallel;
// dkv_internal.hpp declares the four pairs of launchers.
#define DKV_CAT2(a, b, c) a##b##_kv##c
#define DKV_CAT(a, b, c) DKV_CAT2(a, b, c)

// Stage launchers (GramStage) used by the update sequence for bf16 banks.
void DKV_CAT(launch_gram_d, DKV_GRAM_DESC, DKV_GRAM_KV)(const dkv_bank &bank, const dkv_segment &seg, const Geom &g,
                                                        const Prm &p, const dkv_update_out &out, const Workspace &ws,
                                                        hipStream_t s, int stage) {
  mfma_stage_d<DKV_GRAM_DESC, DKV_GRAM_KV != 0>(bank, seg, g, p, out, ws, s, stage);
}

void DKV_CAT(launch_score_d, DKV_GRAM_DESC, DKV_GRAM_KV)(const dkv_bank &bank, const dkv_segment &seg, const Geom &g,
                                                         const Prm &p, int64_t *score_q, float *score_f,
                                                         int64_t *density, const Workspace &ws, hipStream_t s) {
  mfma_score_d<DKV_GRAM_DESC, DKV_GRAM_KV != 0>(bank, seg, g, p, score_q, score_f, density, ws, s);
}

}  // namespace dkv
