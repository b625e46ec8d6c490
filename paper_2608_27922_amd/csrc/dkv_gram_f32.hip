// Gram stages of the DensityKV update for fp32 banks (gfx950).
//
// The same stages as the bf16 ones (dkv_gram_mfma.hip) on
// v_mfma_f32_32x32x2_f32: fp32 products and sums, exact on the key grid.  A wave
// holds 32 row items as the B operand (lane l <-> row l % 32, dims 8 c + 4 (l /
// 32) + 0..3 of every 8, times -2) and takes tiles of 32 column items as A
// straight from global memory in the same dim order; one more K step adds the
// two norms, so the lane (h, n) gets d2 of row n with columns 8 (i / 4) + 4 h +
// i % 4 in register i.  The epilogue is the binary32 contract of pair_weight;
// sums are integers, combined over waves and workgroups with 64-bit atomics.
//
// A wave takes every fourth tile of its workgroup's kCols columns, so that the
// smallest updates (64 candidates, 256 states) spread over several workgroups:
// one thread per row walking every column took 150 us for the score there, 117
// us for the maintenance and 30 us for the crossing.  At large sizes the matrix
// cores bound it (D / 2 + 1 MFMAs of 64 cycles per 32 x 32 tile).
#include <hip/hip_runtime.h>

#include "dkv_internal.hpp"

namespace dkv {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kT = 32;               // rows, and columns, of a tile
constexpr int kGWaves = 4;
constexpr int kCols = 512;           // columns per workgroup

template <int D>
struct Frag {
  float4 k[D / 8];
};

template <int D>
__device__ __forceinline__ Frag<D> load_frag(const float *row, int h, float scale) {
  Frag<D> f;
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    const float4 x = *reinterpret_cast<const float4 *>(row + 8 * c + 4 * h);
    f.k[c] = float4{x.x * scale, x.y * scale, x.z * scale, x.w * scale};
  }
  return f;
}

// d2 of 32 columns (A: key row and norm of column lane % 32) with the wave's rows (B).
template <int D>
__device__ __forceinline__ f32x16 tile_d2(const Frag<D> &a, float anorm, const Frag<D> &b, float bnorm, int h) {
  f32x16 x = {};
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    x = __builtin_amdgcn_mfma_f32_32x32x2f32(a.k[c].x, b.k[c].x, x, 0, 0, 0);
    x = __builtin_amdgcn_mfma_f32_32x32x2f32(a.k[c].y, b.k[c].y, x, 0, 0, 0);
    x = __builtin_amdgcn_mfma_f32_32x32x2f32(a.k[c].z, b.k[c].z, x, 0, 0, 0);
    x = __builtin_amdgcn_mfma_f32_32x32x2f32(a.k[c].w, b.k[c].w, x, 0, 0, 0);
  }
  return __builtin_amdgcn_mfma_f32_32x32x2f32(h ? 1.0f : anorm, h ? bnorm : 1.0f, x, 0, 0, 0);
}

__device__ __forceinline__ int col_of_reg(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

enum Mode { SCORE, DENSITY, SURV_EV, ADM_BASE, ADM_MUT };

// Row sums of one workgroup: rows [32 bx, ..) x columns [kCols by, ..) of bank b.
template <int D, int P, int MODE>
__device__ __forceinline__ void gram_body(const dkv_bank &bank, const float *seg_k, const Geom &g, const Prm &p,
                                          const Workspace &ws, int bx, int by, int b) {
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  const float *bk = static_cast<const float *>(bank.k);
  const int m = ws.m[b];
  constexpr bool kLists = MODE == SURV_EV || MODE == ADM_BASE || MODE == ADM_MUT;
  const int n_ev = kLists ? ws.n_ev[b] : 0, rs = kLists ? ws.r_star[b / g.gs] : 0;
  int nrows, ncols;
  if constexpr (MODE == SCORE) nrows = g.N, ncols = ws.whole[b] == 2 ? 0 : m;
  else if constexpr (MODE == DENSITY) nrows = ncols = m;
  else if constexpr (MODE == SURV_EV) nrows = m - n_ev, ncols = n_ev;
  else if constexpr (MODE == ADM_BASE) nrows = rs, ncols = m - n_ev;
  else nrows = ncols = rs;
  const int c0 = by * kCols, c1 = min(ncols, c0 + kCols);
  if (bx * kT >= nrows || c0 >= c1) return;
  const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = l >> 5, n = l & 31;
  const int v = bx * kT + n, vc = min(v, nrows - 1);
  const bool rv = v < nrows;
  const float *row;
  float rnorm;
  size_t dst;
  if constexpr (MODE == SCORE) {
    row = seg_k + (nb + vc) * D, rnorm = ws.cnorm[nb + vc], dst = nb + vc;
  } else if constexpr (MODE == DENSITY) {
    row = bk + (rb + vc) * D, rnorm = bank.knorm[rb + vc], dst = rb + vc;
  } else if constexpr (MODE == SURV_EV) {
    const int s = ws.surv_list[rb + vc];
    row = bk + (rb + s) * D, rnorm = bank.knorm[rb + s], dst = rb + s;
  } else {
    const int x = ws.adm_list[nb + vc];
    row = seg_k + (nb + x) * D, rnorm = ws.cnorm[nb + x], dst = nb + vc;
  }
  const Frag<D> rf = load_frag<D>(row, h, -2.0f);
  uint64_t sum = 0;
  for (int j0 = c0 + wave * kT; j0 < c1; j0 += kGWaves * kT) {
    const int jc = min(j0 + n, c1 - 1);
    const float *col;
    float cnorm;
    if constexpr (MODE == SCORE || MODE == DENSITY) {
      col = bk + (rb + jc) * D, cnorm = bank.knorm[rb + jc];
    } else if constexpr (MODE == ADM_MUT) {
      const int x = ws.adm_list[nb + jc];
      col = seg_k + (nb + x) * D, cnorm = ws.cnorm[nb + x];
    } else {
      const int s = MODE == SURV_EV ? ws.ev_list[rb + jc] : ws.surv_list[rb + jc];
      col = bk + (rb + s) * D, cnorm = bank.knorm[rb + s];
    }
    const f32x16 d2 = tile_d2<D>(load_frag<D>(col, h, 1.0f), cnorm, rf, rnorm, h);
    uint32_t s32 = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int j = j0 + col_of_reg(i, h);
      float scale = 8388608.0f;
      if constexpr (MODE == SCORE) scale = ws.bs[rb + min(j, c1 - 1)];
      const uint32_t W = q23_round(pair_weight(d2[i], p.inv_sigma2, P), scale);
      bool ok = j < c1;
      if constexpr (MODE == DENSITY || MODE == ADM_MUT) ok = ok && j != v;  // j != i by index
      s32 += ok ? W : 0u;
    }
    sum += s32;
  }
  sum += __shfl_xor(sum, 32, 64);
  if (!rv || h != 0 || sum == 0) return;
  int64_t *out = MODE == SCORE ? ws.acol : (MODE == ADM_BASE ? ws.sub_adm : (MODE == ADM_MUT ? ws.mut_adm : ws.sub));
  atomicAdd(reinterpret_cast<unsigned long long *>(&out[dst]), (unsigned long long)sum);
}

template <int D, int P, int MODE>
__global__ __launch_bounds__(64 * kGWaves) void k_gram_f32(dkv_bank bank, const float *seg_k, Geom g, Prm p, Workspace ws) {
  gram_body<D, P, MODE>(bank, seg_k, g, p, ws, blockIdx.x, blockIdx.y, blockIdx.z);
}

// The maintenance Grams (Supp. C) in one launch: column splits [0, y_ev) are
// survivors x evicted, then y_surv of admitted x survivors, then admitted x admitted.
template <int D, int P>
__global__ __launch_bounds__(64 * kGWaves) void k_maint_f32(dkv_bank bank, const float *seg_k, Geom g, Prm p, Workspace ws,
                                                            int y_ev, int y_surv) {
  const int y = blockIdx.y;
  if (y < y_ev) gram_body<D, P, SURV_EV>(bank, seg_k, g, p, ws, blockIdx.x, y, blockIdx.z);
  else if (y < y_ev + y_surv) gram_body<D, P, ADM_BASE>(bank, seg_k, g, p, ws, blockIdx.x, y - y_ev, blockIdx.z);
  else gram_body<D, P, ADM_MUT>(bank, seg_k, g, p, ws, blockIdx.x, y - y_ev - y_surv, blockIdx.z);
}

// Weights of 64 ordered candidates (chunk c, candidates past `end` weigh 0) with
// the wave's 32 states: w[t][4 k + j] is candidate 32 t + 8 k + 4 h + j.
template <int D, int P>
__device__ __forceinline__ void chunk_weights(uint32_t (&w)[2][16], const float *seg_k, const Geom &g, const Prm &p,
                                              const Workspace &ws, size_t nb, int c, int end, const Frag<D> &rf,
                                              float rnorm, int h, int n) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int j0 = c * kCkStride + 32 * t;
    const int x = ws.order[nb + min(j0 + n, end - 1)];
    const f32x16 d2 = tile_d2<D>(load_frag<D>(seg_k + (nb + x) * D, h, 1.0f), ws.cnorm[nb + x], rf, rnorm, h);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t W = q23_round(pair_weight(d2[i], p.inv_sigma2, P), 8388608.0f);
      w[t][i] = j0 + col_of_reg(i, h) < end ? W : 0u;
    }
  }
}

__device__ __forceinline__ uint32_t chunk_total(const uint32_t (&w)[2][16]) {
  uint32_t s = 0;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) s += w[t][i];
  return s + __shfl_xor(s, 32, 64);
}

// First violating prefix of every bank state (Eqs. 8-9), one wave per 32
// states: chunk sums in order, and where a state's running prefix reaches its
// bound inside a chunk, the inclusive prefixes of that chunk's weights.
template <int D, int P>
__global__ __launch_bounds__(64) void k_cross_f32(dkv_bank bank, const float *seg_k, Geom g, Prm p, Workspace ws,
                                                  int32_t *out_first) {
  const int b = blockIdx.y, l = threadIdx.x, h = l >> 5, n = l & 31;
  const int m = ws.m[b], R = ws.R[b];
  if ((int)blockIdx.x * kT >= m || ws.whole[b]) return;
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  const int v = blockIdx.x * kT + n;
  const bool rv = v < m;
  const size_t row = rb + min(v, m - 1);
  const Frag<D> rf = load_frag<D>(static_cast<const float *>(bank.k) + row * D, h, -2.0f);
  const float rnorm = bank.knorm[row];
  const int64_t lim = ((int64_t)p.tau_num * bank.base[row] + ((1ll << p.tau_shift) - 1)) >> p.tau_shift;
  const int64_t thr = lim - bank.rho[row];
  int first = thr > 0 ? R + 1 : 0;
  bool open = thr > 0;
  int64_t run = 0;
  for (int c = 0; c * kCkStride < R; ++c) {
    uint32_t w[2][16];
    chunk_weights<D, P>(w, seg_k, g, p, ws, nb, c, R, rf, rnorm, h, n);
    const uint32_t tot = chunk_total(w);
    if (rv && h == 0) ws.ck[row * ws.nck + c] = tot;
    const bool hit = open && run + (int64_t)tot >= thr;
    if (__ballot(hit)) {  // uniform over the wave
      // candidates in groups of four, the half-waves' groups alternating
      const uint32_t nd1 = hit ? (uint32_t)(thr - run) - 1u : 0u;
      uint32_t pr = 0, cnt = 0;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t mine = w[t][4 * k] + w[t][4 * k + 1] + w[t][4 * k + 2] + w[t][4 * k + 3];
          const uint32_t other = __shfl_xor(mine, 32, 64);
          uint32_t q = pr + (h ? other : 0u);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            q += w[t][4 * k + j];
            cnt += q <= nd1 ? 1u : 0u;
          }
          pr += mine + other;
        }
      }
      cnt += __shfl_xor(cnt, 32, 64);
      if (hit) {
        first = c * kCkStride + (int)cnt + 1;
        open = false;
      }
    }
    run += tot;
  }
  if (h != 0 || !rv) return;
  ws.first[row] = first;
  if (out_first) out_first[row] = first;
}

// rho~(r*) = rho + the whole chunks before r* + the partial chunk.
template <int D, int P>
__global__ __launch_bounds__(64) void k_fixup_f32(dkv_bank bank, const float *seg_k, Geom g, Prm p, Workspace ws,
                                                  int64_t *out_rho_t) {
  const int b = blockIdx.y, l = threadIdx.x, h = l >> 5, n = l & 31;
  const int m = ws.m[b];
  if ((int)blockIdx.x * kT >= m || ws.whole[b]) return;
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  const int v = blockIdx.x * kT + n;
  const size_t row = rb + min(v, m - 1);
  const int rs = ws.r_star[b / g.gs], full = rs / kCkStride;
  if (rs == 0 && !out_rho_t) return;  // rho~ = rho: the commit reads rho itself
  int64_t P_ = 0;
  if (rs > full * kCkStride) {  // uniform
    const Frag<D> rf = load_frag<D>(static_cast<const float *>(bank.k) + row * D, h, -2.0f);
    uint32_t w[2][16];
    chunk_weights<D, P>(w, seg_k, g, p, ws, nb, full, rs, rf, bank.knorm[row], h, n);
    P_ = chunk_total(w);
  }
  if (h != 0 || v >= m) return;
  for (int t = 0; t < full; ++t) P_ += ws.ck[row * ws.nck + t];
  const int64_t rt = bank.rho[row] + P_;
  ws.rho_t[row] = rt;
  if (out_rho_t) out_rho_t[row] = rt;
}

inline unsigned cdiv(int a, int b) { return (unsigned)((a + b - 1) / b); }

template <int D, int P>
void stage_f32(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p, const dkv_update_out &out,
               const Workspace &ws, hipStream_t s, int stage) {
  const float *sk = static_cast<const float *>(seg.k);
  const unsigned B = (unsigned)g.B, T = 64 * kGWaves;
  const dim3 states(cdiv(g.Mcap, kT), B);
  switch (stage) {
    case kF32Score:
      k_gram_f32<D, P, SCORE><<<dim3(cdiv(g.N, kT), cdiv(g.Mcap, kCols), B), T, 0, s>>>(bank, sk, g, p, ws);
      break;
    case kF32Density:
      k_gram_f32<D, P, DENSITY><<<dim3(cdiv(g.Mcap, kT), cdiv(g.Mcap, kCols), B), T, 0, s>>>(bank, sk, g, p, ws);
      break;
    case kF32Cross:
      k_cross_f32<D, P><<<states, 64, 0, s>>>(bank, sk, g, p, ws, out.first_cross);
      break;
    case kF32Fixup:
      k_fixup_f32<D, P><<<states, 64, 0, s>>>(bank, sk, g, p, ws, out.rho_tilde);
      break;
    case kF32Maint: {
      // releases and survivors are up to Mcap each; workgroups past a bank's own counts return at once
      const int rows = g.Mcap > g.N ? g.Mcap : g.N;
      const unsigned y_ev = cdiv(g.Mcap, kCols), y_adm = cdiv(g.N > 0 ? g.N : 1, kCols);
      k_maint_f32<D, P><<<dim3(cdiv(rows, kT), 2 * y_ev + y_adm, B), T, 0, s>>>(bank, sk, g, p, ws, (int)y_ev, (int)y_ev);
      break;
    }
    default:
      break;
  }
}

}  // namespace

void launch_gram_f32(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                     const dkv_update_out &out, const Workspace &ws, hipStream_t s, int stage) {
  auto run = g.d == 128 ? (p.p == 1 ? stage_f32<128, 1> : (p.p == 2 ? stage_f32<128, 2> : stage_f32<128, 4>))
                        : (p.p == 1 ? stage_f32<64, 1> : (p.p == 2 ? stage_f32<64, 2> : stage_f32<64, 4>));
  run(bank, seg, g, p, out, ws, s, stage);
}

}  // namespace dkv
