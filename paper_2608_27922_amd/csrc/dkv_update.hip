// DensityKV bank update and candidate scoring on gfx950.
//
// One update of every bank from one block (Supp. C, Algorithm 1) is the kernel
// sequence below, all on the caller's stream, with r* kept on the device.  The
// Gram stages of bf16 banks run on MFMA (dkv_gram_mfma.hip: k_score_probe,
// k_score_mfma, k_order_mark, k_rescore, k_order_fix, k_first_part_mfma, k_gather_sorted,
// k_chunk_part_mfma, k_cross_mfma, k_rowsum_mfma, k_maint_mfma); fp32 banks use
// dkv_gram_f32.hip.
//
//   k_begin         clamp occupancy/budget, tested prefix R of the group (Eq. 11),
//                   score scale 1/b of every bank state (Eq. 6), |k_x|^2 of
//                   every candidate, norm steps, cleared accumulators
//   score           S_x = sum_i RNE(w_ix / b_i scaled) (Eq. 6)
//   k_order_count   stable ascending order of S_x, ties by source index (Alg. 1):
//                   ranks counted in one launch, or for more candidates
//   k_sort_chunks   512-key chunks sorted in LDS, then
//   k_sort_rank     ranked by search
//   crossing        prefix sums over the ordered candidates (64-candidate
//                   chunk sums), first violating prefix of every bank state (Eqs. 8-9)
//   k_feas          c_r for every r, the flags c_r <= e_r (Eqs. 9-10), and r* of
//                   each group (Eq. 11)
//   fix-up          projected density rho~(r*) of every bank state
//   k_select        mandatory + densest eviction (Sec. 3.4 step 3), commit plan
//   maintenance     weights to the evicted and to the co-admitted states (Supp. C)
//   k_commit        exact density maintenance of the survivors (Supp. C),
//                   admitted K/V placement, densities and baselines (Eq. 5)
//
// Arithmetic: keys on the 1/64 grid give exact fp32 inner products; weights are
// binary32 with round-to-nearest-even; every sum is an integer sum of Q23
// terms, so results do not depend on tiling or thread order.
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>

#include "dkv_internal.hpp"

namespace dkv {

namespace {

constexpr int kThreads = 256;
constexpr int kBig = 1024;       // one-workgroup-per-bank kernels
constexpr uint64_t kRhoMax = (1ull << 40) - 1;

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// ---------------------------------------------------------------------------
// Block-wide scans for kBig threads (16 waves of 64 lanes).
// ---------------------------------------------------------------------------
__device__ int block_excl_scan(int v, int *total, int *tmp /*[16]*/) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) tmp[wid] = x;
  __syncthreads();
  if (wid == 0) {
    int t = lane < nw ? tmp[lane] : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int y = __shfl_up(t, o, 64);
      if (lane >= o) t += y;
    }
    if (lane < nw) tmp[lane] = t;
  }
  __syncthreads();
  int pre = (wid > 0 ? tmp[wid - 1] : 0) + x - v;
  *total = tmp[nw - 1];
  __syncthreads();
  return pre;
}

__device__ int block_max(int v, int *tmp) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  if (lane == 0) tmp[wid] = v;
  __syncthreads();
  int r = tmp[0];
  for (int w = 1; w < nw; ++w) r = max(r, tmp[w]);
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------------------
// k_begin: grid (1 + ceil(max(N, Mcap) / 512), B).  Workgroup 0 of a bank
// clamps occupancy and budget, fixes the tested prefix R of its group (Eq. 11)
// and the score exponent E, then writes the score scale of every live state
// (Eq. 6); the other workgroups compute candidate norms, the column aug steps
// of candidates and bank states, and clear the accumulators that the Gram
// stages fill with atomic adds.
//
// whole: the group's banks are replaced whole whatever the weights are.  With
// R = M_b for every bank of the group that holds states, e_R = m + R - M_b = m:
// the longest prefix may release every state, so it is feasible (Eqs. 9-10),
// r* = R (Eq. 11), and e_{r*} = m states leave under every fill rule.  Then no
// crossing, projected density or survivor is needed (1), and with R = N not
// even the candidates' order (2): all of them enter.  This holds for budgets up
// to one block.  Such a one-layer update (12 banks, budget = block = 4,680)
// took 432 us with the score, the sort keys and the whole crossing search.
// allow: the largest value the requested outputs permit.
//
// near (n_ev, where the call may approximate its scores): more states than the
// bank can release stand so close to their bound that the first part of the
// crossing search will very likely decide the bank (k_first_part_mfma): the first
// 256 candidates, the ones of lowest score, would have to weigh less than a
// quarter of what the bank's own states weigh on average.  A guess that costs
// time when it is wrong, and nothing else.
// ---------------------------------------------------------------------------
// The candidate rows come through LDS, a wave's 64 rows in parts of 128 bytes: a
// lane that read its own row from memory took 16 bytes of 64 different lines per
// load.  Workgroup 0's chain of loads is what small calls wait for: the group's
// budgets are read side by side, eight baselines per thread are in flight (12 banks
// replaced whole: update 128.0 -> 125.5 us; scores and densities of 12 x 9,360 states
// 388 -> 383 us).
template <int DT>
constexpr int kBeginThreads = DT == DKV_BF16 ? 512 : 256;  // (the small fp32 banks gain nothing from more)

typedef __attribute__((address_space(3))) void lds_void;

// Squared norms of rows [row0, row0 + 64) of src (nrow of them, at least 1; D
// bf16), one per lane, added to s in element order.  buf: 8 KB of the wave's own.
template <int D>
__device__ __forceinline__ void add_row_norms(const uint16_t *src, int nrow, char *buf, float &s) {
  const int l = threadIdx.x & 63;
  constexpr int kAllDone = 7 << 4;  // s_waitcnt: no vector-memory and no LDS operation outstanding
  for (int part = 0; part < D / 64; ++part) {
    const uint16_t *base = src + 64 * part;
    // the buffer ends with the last row, so rows past it read as zero; row r's 16-byte chunk c lies at chunk c ^ (r % 8)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), (short)0,
                                                                        ((nrow - 1) * D + 64) * 2, 0x00020000);
    __builtin_amdgcn_s_waitcnt(kAllDone);  // the reads of the part before
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = 8 * q + (l >> 3);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(buf + 1024 * q), 16, r * D * 2 + 16 * ((l & 7) ^ (r & 7)),
                                               0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(kAllDone);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint4 x = *reinterpret_cast<const uint4 *>(buf + 128 * l + 16 * (c ^ (l & 7)));
      const uint32_t w4[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = __uint_as_float(w4[e] << 16), hi = __uint_as_float(w4[e] & 0xFFFF0000u);
        s = __builtin_fmaf(lo, lo, s);
        s = __builtin_fmaf(hi, hi, s);
      }
    }
  }
}

template <int D, int DT>
__global__ __launch_bounds__(kBeginThreads<DT>) void k_begin(dkv_bank bank, const void *seg_k, const void *seg_v, Geom g,
                                                         Workspace ws, Prm p, int norms, int allow, int approx) {
  const float inv_s2 = p.inv_sigma2;
  const int b = blockIdx.y;
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  if (blockIdx.x > 0) {
    const int j0 = (blockIdx.x - 1) * kBeginThreads<DT>, j = j0 + threadIdx.x;
    if (norms) {
      float s = 0.0f;
      if constexpr (DT == DKV_BF16) {
        // |k|^2 (then + |v|^2 for the [K; V] geometry) in element order
        __shared__ __attribute__((aligned(16))) char rows[kBeginThreads<DT> / 64][8192];
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r0 = j0 + 64 * wave;
        if (r0 < g.N) {
          add_row_norms<D>(static_cast<const uint16_t *>(seg_k) + (nb + r0) * D, min(64, g.N - r0), rows[wave], s);
          if (seg_v)
            add_row_norms<D>(static_cast<const uint16_t *>(seg_v) + (nb + r0) * D, min(64, g.N - r0), rows[wave], s);
        }
      } else if (j < g.N) {
        const float4 *src = reinterpret_cast<const float4 *>(static_cast<const float *>(seg_k) + (nb + j) * D);
#pragma unroll 8
        for (int q = 0; q < D / 4; ++q) {
          const float4 x = src[q];
          s = __builtin_fmaf(x.x, x.x, s);
          s = __builtin_fmaf(x.y, x.y, s);
          s = __builtin_fmaf(x.z, x.z, s);
          s = __builtin_fmaf(x.w, x.w, s);
        }
      }
      if (j < g.N) {
        ws.cnorm[nb + j] = s;
        ws.caug[nb + j] = column_aug(s, inv_s2);
      }
    }
    if (j < g.N) {
      ws.acol[nb + j] = 0;
      ws.sub_adm[nb + j] = 0;
      ws.mut_adm[nb + j] = 0;
    }
    if (j < g.Mcap) {
      const int mj = clampi(bank.occupancy[b], 0, clampi(bank.budget[b], 0, g.Mcap));
      if (j < mj) {
        ws.sub[rb + j] = 0;
        ws.baug[rb + j] = column_aug(bank.knorm[rb + j], inv_s2);
      }
    }
    return;
  }
  const int Mb = clampi(bank.budget[b], 0, g.Mcap);
  const int m = clampi(bank.occupancy[b], 0, Mb);
  // Tested prefix lengths 0..R: R = min(N, every budget of the group).  Each wave
  // reads the group's budgets and occupancies, one bank per lane (where a few
  // lanes hold banks, the minimum is read from them instead of reduced).
  int R = g.N;
  const int g0 = (b / g.gs) * g.gs, lane = threadIdx.x & 63;
  for (int j = lane; j < g.gs; j += 64) R = min(R, clampi(bank.budget[g0 + j], 0, g.Mcap));
  if (g.gs <= 4) {
    R = min(min(__builtin_amdgcn_readlane(R, 0), __builtin_amdgcn_readlane(R, 1)),
            min(__builtin_amdgcn_readlane(R, 2), __builtin_amdgcn_readlane(R, 3)));
  } else {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) R = min(R, __shfl_xor(R, o, 64));
  }
  bool some = false;  // a bank of the group that holds states is not replaced whole
  for (int j = lane; j < g.gs; j += 64) {
    const int Mj = clampi(bank.budget[g0 + j], 0, g.Mcap);
    some |= R != Mj && clampi(bank.occupancy[g0 + j], 0, Mj) > 0;
  }
  int whole = __any(some) ? 0 : allow;
  if (whole > 1 && R < g.N) whole = 1;
  // Score scale exponent E: binary exponent of max_i fp32(2^23 / b_i), i.e. of
  // the value at the smallest baseline (the division and rounding are monotone).
  __shared__ long long redb[kBeginThreads<DT> / 64];
  constexpr int kU = 8;  // independent loads per round trip
  long long mn = LLONG_MAX;
  for (int i0 = threadIdx.x; i0 < m; i0 += kU * kBeginThreads<DT>) {
    long long bq[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) bq[u] = bank.base[rb + min(i0 + u * kBeginThreads<DT>, m - 1)];  // clamped, unconditional
#pragma unroll
    for (int u = 0; u < kU; ++u) mn = bq[u] < mn ? bq[u] : mn;  // (a state read twice changes no minimum)
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const long long y = __shfl_xor(mn, o, 64);
    mn = y < mn ? y : mn;
  }
  if ((threadIdx.x & 63) == 0) redb[threadIdx.x >> 6] = mn;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kBeginThreads<DT> / 64; ++w) mn = redb[w] < mn ? redb[w] : mn;
  int E = 0;
  if (m > 0) {
    const long long bi = mn < 1 ? 1 : mn;
    frexpf((float)(8388608.0 / (double)bi), &E);
  }
  int close = 0;
  for (int i0 = threadIdx.x; i0 < m; i0 += kU * kBeginThreads<DT>) {
    long long bq[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) bq[u] = bank.base[rb + min(i0 + u * kBeginThreads<DT>, m - 1)];  // clamped, unconditional
    if (approx) {
      long long rq[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) rq[u] = bank.rho[rb + min(i0 + u * kBeginThreads<DT>, m - 1)];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const long long thr = ((p.tau_num * bq[u] + ((1ll << p.tau_shift) - 1)) >> p.tau_shift) - rq[u];
        close += i0 + u * kBeginThreads<DT> < m && (float)thr * (float)m <= 0.25f * kCrossFirst * (float)rq[u];
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = i0 + u * kBeginThreads<DT>;
      if (i < m) ws.bs[rb + i] = score_scale(bq[u], E);
    }
  }
  if (approx) {
    __shared__ int redc[kBeginThreads<DT> / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) close += __shfl_xor(close, o, 64);
    if ((threadIdx.x & 63) == 0) redc[threadIdx.x >> 6] = close;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < kBeginThreads<DT> / 64; ++w) close += redc[w];
      ws.n_ev[b] = close > max(0, m + R - Mb);
    }
  }
  if (threadIdx.x == 0) {
    ws.m[b] = m;
    ws.M[b] = Mb;
    ws.R[b] = R;
    ws.E[b] = E;
    ws.whole[b] = whole;
    if (b == 0) ws.crossed[0] = 0;
    if (g.N > kCrossFirst) ws.found[(size_t)b * kFoundStride] = 0;
  }
  if (b == g0) {  // the group's: whether the crossing search may go on past its first part, and k_feas's state
    if (threadIdx.x == 0) {
      ws.more[b / g.gs] = whole ? 0 : (R <= kCrossFirst ? kMoreOpen - 1 : kMoreOpen);
      ws.r_star[b / g.gs] = 0;
    }
    for (int w = threadIdx.x; w < ws.nfw; w += kBeginThreads<DT>) ws.feas[(size_t)b * ws.nfw + w] = ~0u;
  }
}

template <int D, int DT>
void launch_begin(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p, const Workspace &ws,
                  bool norms, int allow_whole, int approx, hipStream_t s) {
  const int span = g.N > g.Mcap ? g.N : g.Mcap;
  // [K; V] geometry: candidate norms over the concatenated key-value rows
  const void *seg_v = (p.flags & DKV_POLICY_KV_DESCRIPTOR) ? seg.v : nullptr;
  k_begin<D, DT><<<dim3((unsigned)(1 + (span + kBeginThreads<DT> - 1) / kBeginThreads<DT>), (unsigned)g.B), kBeginThreads<DT>, 0, s>>>(
      bank, seg.k, seg_v, g, ws, p, norms ? 1 : 0, allow_whole, approx);
}

// ---------------------------------------------------------------------------
// Candidate order: unique keys (S_x << 13) | x sorted ascending (ties of S_x
// by source index).  k_sort_chunks: a workgroup sorts a chunk of 512 keys in
// LDS with a bitonic network (one compare-exchange per thread and stage; a chunk
// of n keys needs the stages of the next power of two only, the rest is padding
// in place already).
// k_sort_rank: the rank of a key is its position in its own chunk plus the
// number of smaller keys in every other chunk, found by branch-free binary
// searches that run in lockstep over all chunks (ten dependent LDS rounds).
// ---------------------------------------------------------------------------
constexpr int kChunk = 512;
constexpr int kSortThreads = kChunk / 2;
constexpr int kMaxChunks = kSortMax / kChunk;

__global__ __launch_bounds__(kSortThreads) void k_sort_chunks(Geom g, Workspace ws, int64_t *out_score,
                                                              int source_order) {
  const int b = blockIdx.y, c = blockIdx.x, t = threadIdx.x;
  if (ws.whole[b] == 2) return;  // no order needed
  const size_t nb = (size_t)b * g.N;
  __shared__ uint64_t v[kChunk];
  // two keys per thread, clamped, unconditional loads
  int64_t A[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) A[u] = ws.acol[nb + min(c * kChunk + t + u * kSortThreads, g.N - 1)];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int idx = c * kChunk + t + u * kSortThreads;
    // ascending score, ties by source index; or source order alone (policy ablation)
    const uint64_t key = source_order ? (uint64_t)idx : (((uint64_t)A[u] << 13) | (uint64_t)idx);
    v[t + u * kSortThreads] = idx < g.N ? key : ~0ull;
    if (out_score && idx < g.N) out_score[nb + idx] = A[u];
  }
  __syncthreads();
  const int n = min(kChunk, g.N - c * kChunk);
  for (int k = 2; k < 2 * n && k <= kChunk; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      // the t-th index i with bit j clear, against i + j; ascending where bit k of i is clear
      const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
      const uint64_t x = v[i], y = v[i + j];
      const bool up = (i & k) == 0;
      if (up ? (x > y) : (x < y)) {
        v[i] = y;
        v[i + j] = x;
      }
      __syncthreads();
    }
  }
  const size_t base = (size_t)b * ws.npad + (size_t)c * kChunk;
#pragma unroll
  for (int u = 0; u < 2; ++u) ws.skeys[base + t + u * kSortThreads] = v[t + u * kSortThreads];
}

template <int NCH>  // chunk slots searched (>= the number of chunks)
__global__ __launch_bounds__(kBig) void k_sort_rank(Geom g, Workspace ws, int32_t *out_order) {
  const int b = blockIdx.y;
  if (ws.whole[b] == 2) return;  // no order needed
  __shared__ uint64_t sk[kSortMax];
  const int np = ws.npad;
  const int nch = np / kChunk;
  {
    // clamped, unconditional loads, all in flight at once
    constexpr int kPer = kSortMax / kBig;
    uint64_t t[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) t[u] = ws.skeys[(size_t)b * np + min((int)threadIdx.x + u * kBig, np - 1)];
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if ((int)threadIdx.x + u * kBig < np) sk[threadIdx.x + u * kBig] = t[u];
  }
  __syncthreads();
  const size_t nb = (size_t)b * g.N;
  for (int p = blockIdx.x * kBig + threadIdx.x; p < np; p += gridDim.x * kBig) {
    const uint64_t key = sk[p];
    if (key == ~0ull) continue;
    const int c = p / kChunk;
    // count of keys < key in every chunk: cnt grows by half while the key at
    // cnt + half - 1 is smaller (at most 511), then by one more if the key at
    // cnt is smaller; chunks past the last one read the last one and are masked
    int cnt[NCH];
#pragma unroll
    for (int c2 = 0; c2 < NCH; ++c2) cnt[c2] = 0;
#pragma unroll
    for (int half = kChunk / 2; half >= 1; half >>= 1) {
#pragma unroll
      for (int c2 = 0; c2 < NCH; ++c2) {
        const int base = min(c2, nch - 1) * kChunk;
        cnt[c2] += sk[base + cnt[c2] + half - 1] < key ? half : 0;
      }
    }
    int rank = p - c * kChunk;
#pragma unroll
    for (int c2 = 0; c2 < NCH; ++c2) {
      const int base = min(c2, nch - 1) * kChunk;
      const int n2 = cnt[c2] + (sk[base + cnt[c2]] < key ? 1 : 0);
      if (c2 < nch && c2 != c) rank += n2;
    }
    const int x = (int)(key & 0x1FFFull);
    ws.order[nb + rank] = x;
    ws.rank[nb + x] = rank;
    if (out_order) out_order[nb + rank] = x;
  }
}

// Order of few candidates in one launch: the rank of a key is the number of
// smaller keys, counted over all of them.  A workgroup ranks 64 candidates, one
// per lane; its 16 waves take a sixteenth of the keys each, read two at a time as
// broadcasts from LDS.  N^2 compares, but no dependent stages and one launch less:
// updates of 48 banks x 1,000 candidates 82.5 -> 75.7 us, 24 x 2,040 (1.0e8 compares)
// 105.5 -> 104.2, 120 x 1,000 (1.2e8) 128.6 -> 132.1, 360 x 450 (7.3e7) 161.2 -> 162.1.
constexpr int kCountMax = 2048;
constexpr double kCountPairs = 6e7;

__global__ __launch_bounds__(kBig) void k_order_count(Geom g, Workspace ws, int64_t *out_score, int32_t *out_order,
                                                      int source_order) {
  const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (ws.whole[b] == 2) return;  // no order needed
  const size_t nb = (size_t)b * g.N;
  __shared__ __attribute__((aligned(16))) uint64_t key[kCountMax];
  __shared__ int part[kBig / 64][64];
  const int seg = ((g.N + kBig / 64 - 1) / (kBig / 64) + 1) & ~1;  // keys per wave; 16 seg <= kCountMax
  for (int i = threadIdx.x; i < seg * (kBig / 64); i += kBig) {
    const int64_t A = ws.acol[nb + min(i, g.N - 1)];
    const uint64_t k = source_order ? (uint64_t)i : (((uint64_t)A << 13) | (uint64_t)i);
    key[i] = i < g.N ? k : ~0ull;
    if (out_score && blockIdx.x == 0 && i < g.N) out_score[nb + i] = A;
  }
  __syncthreads();
  const int x = blockIdx.x * 64 + lane;
  const uint64_t mine = key[min(x, g.N - 1)];
  int cnt = 0;
  for (int j = wave * seg; j < (wave + 1) * seg; j += 2) {
    const ulonglong2 k2 = *reinterpret_cast<const ulonglong2 *>(&key[j]);
    cnt += (k2.x < mine ? 1 : 0) + (k2.y < mine ? 1 : 0);
  }
  part[wave][lane] = cnt;
  __syncthreads();
  if (wave != 0 || x >= g.N) return;
#pragma unroll
  for (int w = 1; w < kBig / 64; ++w) cnt += part[w][lane];
  ws.order[nb + cnt] = x;
  ws.rank[nb + x] = cnt;
  if (out_order) out_order[nb + cnt] = x;
}

// ---------------------------------------------------------------------------
// Feasibility: c_r = #{i : first_i <= r}; feasible iff c_r <= e_r for every bank
// of the group; r* = largest feasible r.
// ---------------------------------------------------------------------------
__device__ void block_inclusive_scan_lds(int *a, int n, int *tmp) {
  const int per = (n + kBig - 1) / kBig;
  const int lo = min(n, (int)threadIdx.x * per), hi = min(n, lo + per);
  int s = 0;
  for (int i = lo; i < hi; ++i) s += a[i];
  int tot;
  int pre = block_excl_scan(s, &tot, tmp);
  for (int i = lo; i < hi; ++i) {
    pre += a[i];
    a[i] = pre;
  }
  __syncthreads();
}

// Per bank: c_r = #{i : first_i <= r} by histogram + scan, and bit r of the
// feasibility mask set iff c_r <= e_r = max(0, m + r - M) (Eqs. 9-10), ANDed into
// the group's mask.  The group's last bank to arrive (counted in r_star, which
// k_begin cleared) then takes r* = the largest r feasible for every bank
// (Eq. 11) and every bank's e_{r*}.  Masks and count go through device-scope
// atomics.  The count's release waits for its own wave's memory operations only,
// and the workgroup barrier waits for none: each wave takes its ANDs' results, so
// that they are done when it reaches the barrier, before the count.
__global__ __launch_bounds__(kBig) void k_feas(Geom g, Workspace ws, int32_t *out_rstar) {
  const int b = blockIdx.x, grp = b / g.gs, b0 = grp * g.gs;
  __shared__ int hist[kSortMax + 1];
  __shared__ int tmp[16];
  __shared__ int last;
  const int R = ws.R[b];
  const int m = ws.m[b], M = ws.M[b];
  if (ws.whole[b]) {  // a group replaced whole (of all its banks or none): r* = R, nothing to search
    if (b != b0) return;
    if (threadIdx.x == 0) {
      ws.r_star[grp] = R;
      if (out_rstar) out_rstar[grp] = R;
    }
    for (int j = threadIdx.x; j < g.gs; j += kBig) ws.e[b0 + j] = max(0, ws.m[b0 + j] + R - ws.M[b0 + j]);
    return;
  }
  for (int r = threadIdx.x; r <= R; r += kBig) hist[r] = 0;
  __syncthreads();
  // four independent (clamped, unconditional) loads per round trip
  for (int i0 = threadIdx.x; i0 < m; i0 += 4 * kBig) {
    int t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = ws.first[(size_t)b * g.Mcap + min(i0 + u * kBig, m - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i0 + u * kBig < m && t[u] <= R) atomicAdd(&hist[t[u]], 1);
  }
  __syncthreads();
  block_inclusive_scan_lds(hist, R + 1, tmp);
  // one wave per 64 values of r: the flags by ballot, two mask words per wave
  uint32_t *f = ws.feas + (size_t)b0 * ws.nfw;
  const int lane = threadIdx.x & 63;
  uint32_t seen = 0;
  for (int w2 = threadIdx.x >> 6; 2 * w2 < ws.nfw; w2 += kBig / 64) {
    const int r = 64 * w2 + lane;
    const bool ok = r <= R && hist[r <= R ? r : 0] <= max(0, m + r - M);
    const unsigned long long bits = __ballot(ok);
    const uint32_t word = lane == 0 ? (uint32_t)bits : (uint32_t)(bits >> 32);
    if (lane < 2 && 2 * w2 + lane < ws.nfw)
      seen |= __hip_atomic_fetch_and(&f[2 * w2 + lane], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  asm volatile("" ::"v"(seen) : "memory");  // every AND of this wave has returned
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(&ws.r_star[grp], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == g.gs - 1;
  __syncthreads();
  if (!last) return;
  int best = 0;
  for (int w = threadIdx.x; w < ws.nfw; w += kBig) {
    const uint32_t bits = __hip_atomic_load(&f[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (bits) best = max(best, 32 * w + 31 - __clz(bits));
  }
  best = block_max(best, tmp);
  if (threadIdx.x == 0) {
    ws.r_star[grp] = best;
    if (out_rstar) out_rstar[grp] = best;
  }
  for (int j = threadIdx.x; j < g.gs; j += kBig) ws.e[b0 + j] = max(0, ws.m[b0 + j] + best - ws.M[b0 + j]);
}

// ---------------------------------------------------------------------------
// k_select: one workgroup per bank.  Violators at r* are evicted; the fill
// takes the non-violators with the largest rho~(r*), ties by provenance, then
// slot (key (2^40-1-rho~, prov, slot) ascending, found by MSB radix select).
// Then the commit plan: evicted list, admitted list, final slot of everything.
// ---------------------------------------------------------------------------
enum : unsigned char { ST_NONE = 0, ST_CAND = 1, ST_SEL = 2, ST_VIOL = 3 };

__device__ __forceinline__ int sel_digit(const Workspace &ws, const dkv_bank &bank, size_t row, int slot,
                                         int pass) {
  if (pass < 5) {
    const uint64_t w0 = kRhoMax - (uint64_t)ws.rho_t[row];
    return (int)((w0 >> (8 * (4 - pass))) & 0xFF);
  }
  if (pass < 13) {
    const uint64_t w1 = (uint64_t)bank.prov[row];
    return (int)((w1 >> (8 * (12 - pass))) & 0xFF);
  }
  return (int)(((uint32_t)slot >> (8 * (14 - pass))) & 0xFF);
}

__global__ __launch_bounds__(kBig) void k_select(dkv_bank bank, Geom g, Workspace ws,
                                                 dkv_update_out out, uint32_t flags) {
  // policy ablations: no mandatory set, or a fill in admission order (key
  // (provenance, slot): the radix passes over rho~ are skipped)
  const bool no_mandatory = (flags & DKV_POLICY_DENSEST_ONLY) != 0;
  const int first_pass = (flags & DKV_POLICY_SOURCE_FILL) ? 5 : 0;
  const int b = blockIdx.x;
  const int m = ws.m[b];
  const int rs = ws.r_star[b / g.gs];
  const int e = ws.e[b];
  __shared__ unsigned char st[DKV_MAX_CAPACITY + 1];
  __shared__ __attribute__((aligned(16))) int hist[256];
  __shared__ int tmp[16];
  __shared__ int sh_bucket, sh_below, sh_cnt;
  const size_t rb = (size_t)b * g.Mcap;

  // this thread's candidate ranks (admitted list below), loaded up front
  const int N = g.N;
  const size_t nb = (size_t)b * N;
  constexpr int kPerN = (DKV_MAX_CANDIDATES + kBig - 1) / kBig;
  const int perN = (N + kBig - 1) / kBig;
  const int loN = min(N, (int)threadIdx.x * perN), hiN = min(N, loN + perN);
  int rk[kPerN];
  const int whole = ws.whole[b];  // 2: every candidate enters, no ranks
#pragma unroll
  for (int u = 0; u < kPerN; ++u) {
    const int r = whole != 2 && rs > 0 ? ws.rank[nb + min(loN + u, N - 1)] : INT_MAX;  // clamped
    rk[u] = loN + u < hiN ? r : INT_MAX;
  }
  if (whole) {
    // Every state leaves and R = M candidates (fewer only into a bank that held
    // none) take the slots in order: no fill, no survivors, no holes.  The lists
    // are written side by side instead of in runs per thread (12 banks of 4,680:
    // 13.7 us by the general path).
    for (int i = threadIdx.x; i < m; i += kBig) {
      ws.ev_list[rb + i] = i;
      ws.dest[rb + i] = -1;
    }
    for (int k = threadIdx.x; k < rs; k += kBig) ws.adm_dest[nb + k] = k;
    if (whole == 2) {
      for (int k = threadIdx.x; k < rs; k += kBig) ws.adm_list[nb + k] = k;
    } else {
      int ca = 0, n_adm;
#pragma unroll
      for (int u = 0; u < kPerN; ++u) ca += rk[u] < rs;
      int pa = block_excl_scan(ca, &n_adm, tmp);
#pragma unroll
      for (int u = 0; u < kPerN; ++u)
        if (rk[u] < rs) ws.adm_list[nb + pa++] = loN + u;
    }
    if (out.evicted)
      for (int j = threadIdx.x; j < g.Mcap; j += kBig) out.evicted[rb + j] = j < m ? j : -1;
    if (out.admitted) {
      __syncthreads();
      for (int j = threadIdx.x; j < N; j += kBig) out.admitted[nb + j] = j < rs ? ws.adm_list[nb + j] : -1;
    }
    if (threadIdx.x == 0) {
      ws.n_ev[b] = m;
      if (rs > 0 || m > 0) ws.crossed[0] = 1;
      bank.occupancy[b] = rs;
      if (out.n_evicted) out.n_evicted[b] = m;
      if (out.n_admitted) out.n_admitted[b] = rs;
    }
    return;
  }
  // violators and candidates for the fill (four independent loads per round trip)
  int nv_local = 0;
  for (int i0 = threadIdx.x; i0 < m; i0 += 4 * kBig) {
    int f[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) f[u] = ws.first[rb + min(i0 + u * kBig, m - 1)];  // clamped, unconditional
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * kBig;
      if (i < m) {
        const bool v = !no_mandatory && f[u] <= rs;
        st[i] = v ? ST_VIOL : ST_CAND;
        nv_local += v;
      }
    }
  }
  int nv;
  (void)block_excl_scan(nv_local, &nv, tmp);
  if (rs == 0 && nv == 0) {  // nothing enters or leaves (e_0 = 0): no lists, no destinations
    if (out.evicted)
      for (int j = threadIdx.x; j < g.Mcap; j += kBig) out.evicted[rb + j] = -1;
    if (out.admitted)
      for (int j = threadIdx.x; j < N; j += kBig) out.admitted[nb + j] = -1;
    if (threadIdx.x == 0) {
      ws.n_ev[b] = 0;
      bank.occupancy[b] = m;
      if (out.n_evicted) out.n_evicted[b] = 0;
      if (out.n_admitted) out.n_admitted[b] = 0;
    }
    return;
  }
  int need = e - nv;
  if (need > 0 && need >= m - nv) {
    // every non-violator is evicted too (e = m): no ranking needed
    for (int i = threadIdx.x; i < m; i += kBig)
      if (st[i] == ST_CAND) st[i] = ST_SEL;
    need = 0;
    __syncthreads();
  }
  if (need > 0) {
    for (int pass = first_pass; pass < 15; ++pass) {
      for (int t = threadIdx.x; t < 256; t += kBig) hist[t] = 0;
      __syncthreads();
      for (int i = threadIdx.x; i < m; i += kBig)
        if (st[i] == ST_CAND) atomicAdd(&hist[sel_digit(ws, bank, rb + i, i, pass)], 1);
      __syncthreads();
      // the first bucket whose cumulative count reaches `need` (more than `need`
      // candidates are left, so there is one): wave 0, four buckets per lane (one
      // thread adding up to 256 buckets took 2-5 us of dependent LDS reads a pass)
      if (threadIdx.x < 64) {
        const int4 c4 = reinterpret_cast<const int4 *>(hist)[threadIdx.x];
        const int own = c4.x + c4.y + c4.z + c4.w;
        int incl = own;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(incl, o, 64);
          if ((int)threadIdx.x >= o) incl += y;
        }
        int cum = incl - own;
        if (cum < need && need <= incl) {
          const int c[4] = {c4.x, c4.y, c4.z, c4.w};
          int d = 0;
          while (d < 3 && cum + c[d] < need) cum += c[d++];
          sh_bucket = 4 * (int)threadIdx.x + d;
          sh_below = cum;
          sh_cnt = c[d];
        }
      }
      __syncthreads();
      const int bk = sh_bucket, below = sh_below, cnt = sh_cnt;
      const bool finish = (need - below) == cnt;
      for (int i = threadIdx.x; i < m; i += kBig) {
        if (st[i] != ST_CAND) continue;
        const int dg = sel_digit(ws, bank, rb + i, i, pass);
        if (dg < bk || (dg == bk && finish)) st[i] = ST_SEL;
        else if (dg > bk) st[i] = ST_NONE;
      }
      need -= below;
      __syncthreads();
      if (finish) break;
    }
  }

  // evicted list (ascending slots) and rank of each evicted slot
  const int per = (m + kBig - 1) / kBig;
  const int lo = min(m, (int)threadIdx.x * per), hi = min(m, lo + per);
  int cnt_local = 0;
  for (int i = lo; i < hi; ++i) cnt_local += (st[i] == ST_VIOL || st[i] == ST_SEL);
  int n_ev;
  int pos = block_excl_scan(cnt_local, &n_ev, tmp);
  int spos = lo - pos;  // survivors before this thread's range
  for (int i = lo; i < hi; ++i) {
    if (st[i] == ST_VIOL || st[i] == ST_SEL) {
      ws.ev_list[rb + pos] = i;
      ws.dest[rb + i] = -1 - pos;  // provisional: encodes the evicted rank
      if (pos < rs) ws.adm_dest[nb + pos] = i;  // admitted entry pos fills the pos-th evicted slot
      ++pos;
    } else {
      ws.surv_list[rb + spos] = i;
      ws.dest[rb + i] = i;
      ++spos;
    }
  }
  // admitted list: source indices x with rank(x) < r*, ascending; entries
  // beyond the evicted slots are appended after the old occupancy
  int ca = 0;
#pragma unroll
  for (int u = 0; u < kPerN; ++u) ca += rk[u] < rs;
  int n_adm;
  int pa = block_excl_scan(ca, &n_adm, tmp);
  __syncthreads();
  const int m_new = m - n_ev + rs;
#pragma unroll
  for (int u = 0; u < kPerN; ++u) {
    if (rk[u] < rs) {
      ws.adm_list[nb + pa] = loN + u;
      if (pa >= n_ev) ws.adm_dest[nb + pa] = m + (pa - n_ev);
      ++pa;
    }
  }
  __syncthreads();
  if (n_ev > rs) {
    // More evicted than admitted: close the holes below m_new with the
    // occupants at or beyond m_new, both in ascending slot order.
    // occupied(s) after placement: survivor, or an evicted slot filled by an
    // admitted candidate (evicted rank < r*).
    int mv_local = 0, lh_local = 0;
    for (int i = lo; i < hi; ++i) {
      const int dsl = ws.dest[rb + i];
      const bool occ = dsl >= 0 || (-1 - dsl) < rs;
      mv_local += occ && i >= m_new;
      lh_local += !occ && i < m_new;
    }
    int n_mv, n_lh;
    int pm = block_excl_scan(mv_local, &n_mv, tmp);
    int ph = block_excl_scan(lh_local, &n_lh, tmp);
    // list of the holes below m_new, ascending
    for (int i = lo; i < hi; ++i) {
      const int dsl = ws.dest[rb + i];
      const bool occ = dsl >= 0 || (-1 - dsl) < rs;
      if (!occ && i < m_new) ws.hole_list[rb + (ph++)] = i;
    }
    __syncthreads();
    for (int i = lo; i < hi; ++i) {
      const int dsl = ws.dest[rb + i];
      const bool occ = dsl >= 0 || (-1 - dsl) < rs;
      if (occ && i >= m_new) {
        const int to = ws.hole_list[rb + pm];
        ++pm;
        if (dsl >= 0) {
          ws.dest[rb + i] = to;  // moving survivor
        } else {
          ws.adm_dest[nb + (-1 - dsl)] = to;  // admitted candidate placed in a high hole
        }
      }
    }
    __syncthreads();
  }
  // finalize dest: evicted -> -1; outputs
  for (int i = lo; i < hi; ++i)
    if (ws.dest[rb + i] < 0) ws.dest[rb + i] = -1;
  if (out.evicted) {
    for (int j = threadIdx.x; j < g.Mcap; j += kBig) out.evicted[rb + j] = j < n_ev ? ws.ev_list[rb + j] : -1;
  }
  if (out.admitted) {
    for (int j = threadIdx.x; j < N; j += kBig) out.admitted[nb + j] = j < n_adm ? ws.adm_list[nb + j] : -1;
  }
  if (threadIdx.x == 0) {
    ws.n_ev[b] = n_ev;
    if (rs > 0 || n_ev > 0) ws.crossed[0] = 1;
    bank.occupancy[b] = m_new;
    if (out.n_evicted) out.n_evicted[b] = n_ev;
    if (out.n_admitted) out.n_admitted[b] = rs;
  }
}

// ---------------------------------------------------------------------------
// Commit.  commit_surv: thread per surviving state: rho <- rho~(r*) minus its
// weights to the evicted states (Supp. C); a state that closes a hole (only when
// more states left than entered) moves with its key, value and metadata.
// commit_adm: the admitted K/V rows into their slots, four 16-byte chunks of
// one token per thread; the first lane of each token writes its density over
// the final bank, frozen baseline max(rho, delta) (Eq. 5), provenance and norm.
// ---------------------------------------------------------------------------
template <int D, int DT>
__device__ __forceinline__ void commit_surv(const dkv_bank &bank, const Geom &g, const Prm &p, const Workspace &ws,
                                            int bx) {
  using E = typename std::conditional<DT == DKV_BF16, uint16_t, float>::type;
  const int b = blockIdx.y, v = bx * kThreads + threadIdx.x;
  if (v >= ws.m[b]) return;
  const size_t rb = (size_t)b * g.Mcap;
  const int rs = ws.r_star[b / g.gs];
  const bool same = rs == 0 && ws.n_ev[b] == 0;  // nothing entered or left: every state as it is
  if (same && !(p.flags & DKV_POLICY_REFRESH_BASE)) return;
  const int to = same ? v : ws.dest[rb + v];
  if (to < 0) return;
  // r* = 0: the projected density is the density
  const int64_t rho = (rs > 0 ? ws.rho_t[rb + v] : bank.rho[rb + v]) - ws.sub[rb + v];
  if (to != v) {
    E *K = static_cast<E *>(bank.k);
    E *V = static_cast<E *>(bank.v);
    for (int j = 0; j < D; ++j) {
      K[(rb + to) * D + j] = K[(rb + v) * D + j];
      V[(rb + to) * D + j] = V[(rb + v) * D + j];
    }
    bank.base[rb + to] = bank.base[rb + v];
    bank.prov[rb + to] = bank.prov[rb + v];
    bank.knorm[rb + to] = bank.knorm[rb + v];
  }
  bank.rho[rb + to] = rho;
  // refreshed baselines (policy ablation): b = max(rho, delta) after the update
  if (p.flags & DKV_POLICY_REFRESH_BASE) bank.base[rb + to] = rho > p.delta_q ? rho : p.delta_q;
}

typedef uint32_t vu4 __attribute__((ext_vector_type(4)));
constexpr int kCommitChunks = 4;  // 16-byte chunks of one admitted token per thread (1 and 2 were slower)

// Admitted tokens per workgroup of the commit: a token's K and V rows are
// 2 * D * sizeof(E) / 16 chunks, kCommitChunks per thread.
template <int D, int DT>
__host__ __device__ constexpr int commit_tok_per_wg() {
  return kThreads / (2 * D * (DT == DKV_BF16 ? 2 : 4) / 16 / kCommitChunks);
}

template <int D, int DT>
__device__ __forceinline__ void commit_adm(const dkv_bank &bank, const dkv_segment &seg, const Geom &g,
                                           const Prm &p, const Workspace &ws, int bx) {
  using E = typename std::conditional<DT == DKV_BF16, uint16_t, float>::type;
  constexpr int kCh = D * (int)sizeof(E) / 16;  // 16-byte chunks per key (and per value) row
  constexpr int kLanes = 2 * kCh / kCommitChunks;  // lanes per token
  constexpr int kTokWG = commit_tok_per_wg<D, DT>();
  static_assert(2 * kCh % kCommitChunks == 0 && kThreads % kLanes == 0, "whole tokens per workgroup");
  const int b = blockIdx.y;
  const int j = threadIdx.x % kLanes;
  const int k = bx * kTokWG + threadIdx.x / kLanes;
  const int rs = min(ws.r_star[b / g.gs], g.N);
  const size_t rb = (size_t)b * g.Mcap, nb = (size_t)b * g.N;
  if (bx * kTokWG >= rs) return;  // whole workgroup
  // loads from a clamped (in-range) entry, unconditional so that they overlap;
  // only the stores are predicated
  const int kc = min(k, rs - 1);
  const int x = ws.adm_list[nb + kc], to = ws.adm_dest[nb + kc];
  vu4 tmp[kCommitChunks];
#pragma unroll
  for (int u = 0; u < kCommitChunks; ++u) {
    const int cc = j + kLanes * u;  // chunk of the token's [K row; V row]
    const bool isv = cc >= kCh;
    tmp[u] = reinterpret_cast<const vu4 *>(static_cast<const E *>(isv ? seg.v : seg.k) + (nb + x) * D)[cc - (isv ? kCh : 0)];
  }
  if (k >= rs) return;
#pragma unroll
  for (int u = 0; u < kCommitChunks; ++u) {
    const int cc = j + kLanes * u;
    const bool isv = cc >= kCh;
    // streaming store: the bank rows are not read again by this update
    __builtin_nontemporal_store(tmp[u], reinterpret_cast<vu4 *>(static_cast<E *>(isv ? bank.v : bank.k) + (rb + to) * D) +
                                            (cc - (isv ? kCh : 0)));
  }
  if (j == 0) {
    // density over the final bank: the survivors plus the other co-admitted candidates
    const int64_t rho = ws.sub_adm[nb + k] + ws.mut_adm[nb + k];
    bank.rho[rb + to] = rho;
    bank.base[rb + to] = rho > p.delta_q ? rho : p.delta_q;
    bank.prov[rb + to] = ((int64_t)p.block_id << 32) | (int64_t)x;
    bank.knorm[rb + to] = ws.cnorm[nb + x];
  }
}

// Commit (Eq. 12) in one launch: the first nx_surv workgroups update the
// survivors (and move the few that close holes), the rest place the admitted
// candidates.  The two write disjoint slots.
template <int D, int DT>
__global__ __launch_bounds__(kThreads) void k_commit(dkv_bank bank, dkv_segment seg, Geom g, Prm p, Workspace ws,
                                                     int nx_surv) {
  if ((int)blockIdx.x < nx_surv) commit_surv<D, DT>(bank, g, p, ws, blockIdx.x);
  else commit_adm<D, DT>(bank, seg, g, p, ws, blockIdx.x - nx_surv);
}

// Score entry point outputs from the accumulated sums.
__global__ void k_score_out(Geom g, Workspace ws, int64_t *out_q, float *out_f) {
  const int b = blockIdx.y, x = blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= g.N) return;
  const size_t o = (size_t)b * g.N + x;
  const int m = ws.m[b];
  const int64_t A = ws.acol[o];
  if (out_q) out_q[o] = A;
  if (out_f) out_f[o] = m > 0 ? (float)(ldexp((double)A, ws.E[b] - 23) / (double)m) : 0.0f;
}

__global__ void k_density_out(Geom g, Workspace ws, int64_t *out) {
  const int b = blockIdx.y, i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ws.m[b]) return;
  out[(size_t)b * g.Mcap + i] = ws.sub[(size_t)b * g.Mcap + i];
}

__global__ void k_pair_weight(const float *d2, int64_t n, Prm p, int32_t *w) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = (int32_t)q23_round(pair_weight(d2[i], p.inv_sigma2, p.p), 8388608.0f);
}

inline dim3 grid2(int n, int per, int B) { return dim3((unsigned)((n + per - 1) / per), (unsigned)B); }

constexpr double kApproxPairs = 1e10;

template <int D, int DT>
hipError_t update_impl(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                       const dkv_update_out *outp, const Workspace &ws, hipStream_t s) {
  dkv_update_out out = outp ? *outp : dkv_update_out{};
  // the Gram stages of bf16 banks (dkv_gram_mfma.hip) or of fp32 banks (dkv_gram_f32.hip)
  constexpr bool kMfma = DT == DKV_BF16;
  // the crossings and projected densities are computed in full when they are asked for; so are the scores
  // (and the order they give), which the sequential competition needs in any case
  const bool seq = (p.flags & DKV_POLICY_SEQUENTIAL) != 0;
  const int allow_whole = (seq || out.first_cross || out.rho_tilde) ? 0 : ((out.order || out.score_q) ? 1 : 2);
  // Large calls that ask for neither the scores nor the order may take
  // approximate scores first and exact ones only where the approximation leaves
  // the order open (dkv_gram_mfma.hip).  k_score_probe decides for each bank: it
  // pays where the order is needed at its head only and few neighbours are too
  // close (360 frozen banks of 9,300 states x 4,680 candidates: update 5.45 ->
  // 5.14 ms, 360 head-wise banks 4.30 -> 4.08).  The six launches cost 25 to 30 us
  // where it does not (24 banks of 9,000 states, 1.0e9 pairs: 410 -> 437 us; 96
  // growing banks, 2.1e9: 2,315 -> 2,320), so calls below 1e10 pairs (by capacity,
  // of which banks in use hold about half) score exactly from the start.
  const bool approx = kMfma && !seq && !(p.flags & DKV_POLICY_SOURCE_ORDER) && !out.order && !out.score_q &&
                      (double)g.B * g.Mcap * g.N >= kApproxPairs;
  launch_begin<D, DT>(bank, seg, g, p, ws, g.N > 0, allow_whole, approx ? 1 : 0, s);
  if (g.N > 0) {
    // in source order the scores are only reported
    if (!(p.flags & DKV_POLICY_SOURCE_ORDER) || out.score_q) {
      if (kMfma) launch_gram_mfma(bank, seg, g, p, out, ws, s, approx ? kGramScoreApprox : kGramScore);
      else launch_gram_f32(bank, seg, g, p, out, ws, s, kF32Score);
    }
    const int source_order = (p.flags & DKV_POLICY_SOURCE_ORDER) ? 1 : 0;
    // by counting up to 6e7 compares (sorting takes as long from about 8e7 on)
    if (g.N <= kCountMax && (double)g.B * g.N * g.N <= kCountPairs) {
      k_order_count<<<dim3((unsigned)((g.N + 63) / 64), (unsigned)g.B), kBig, 0, s>>>(g, ws, out.score_q, out.order,
                                                                                      source_order);
    } else {
      k_sort_chunks<<<dim3((unsigned)((g.N + kChunk - 1) / kChunk), (unsigned)g.B), kSortThreads, 0, s>>>(
          g, ws, out.score_q, source_order);
      const dim3 grid((unsigned)((ws.npad + kBig - 1) / kBig), (unsigned)g.B);
      const int nch = ws.npad / kChunk;
      auto rank = nch <= 4 ? k_sort_rank<4> : (nch <= 8 ? k_sort_rank<8> : (nch <= 12 ? k_sort_rank<12> : k_sort_rank<kMaxChunks>));
      rank<<<grid, kBig, 0, s>>>(g, ws, out.order);
    }
  }
  // within-block sequential competition: the rest is one candidate per step
  if (kMfma && (p.flags & DKV_POLICY_SEQUENTIAL)) return launch_sequential(bank, seg, g, p, out, ws, s);
  // with no candidates only states that already violate are found (prefix 0)
  if (kMfma) {
    if (approx) launch_gram_mfma(bank, seg, g, p, out, ws, s, kGramOrder);
    launch_gram_mfma(bank, seg, g, p, out, ws, s, kGramFirstPart);
    if (g.N > kCrossFirst) {
      if (approx) launch_gram_mfma(bank, seg, g, p, out, ws, s, kGramOrderRest);
      launch_gram_mfma(bank, seg, g, p, out, ws, s, kGramSecondPart);
    }
  } else {
    launch_gram_f32(bank, seg, g, p, out, ws, s, kF32Cross);
  }
  k_feas<<<g.B, kBig, 0, s>>>(g, ws, out.r_star);
  if (kMfma) launch_gram_mfma(bank, seg, g, p, out, ws, s, kGramFixup);
  else launch_gram_f32(bank, seg, g, p, out, ws, s, kF32Fixup);
  k_select<<<g.B, kBig, 0, s>>>(bank, g, ws, out, p.flags);
  if (kMfma) launch_gram_mfma(bank, seg, g, p, out, ws, s, kGramMaint);
  else launch_gram_f32(bank, seg, g, p, out, ws, s, kF32Maint);
  {
    const int nxs = (g.Mcap + kThreads - 1) / kThreads;
    const int tok_per_wg = commit_tok_per_wg<D, DT>();
    const int nxa = g.N > 0 ? (g.N + tok_per_wg - 1) / tok_per_wg : 0;
    k_commit<D, DT><<<dim3((unsigned)(nxs + nxa), (unsigned)g.B), kThreads, 0, s>>>(bank, seg, g, p, ws, nxs);
  }
  return hipGetLastError();
}

template <int D, int DT>
hipError_t score_impl(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                      int64_t *score_q, float *score_f, int64_t *density, const Workspace &ws,
                      hipStream_t s) {
  launch_begin<D, DT>(bank, seg, g, p, ws, g.N > 0 && (score_q || score_f), 0, 0, s);
  const bool scores = g.N > 0 && (score_q || score_f);
  if constexpr (DT == DKV_BF16) {
    launch_score_mfma(bank, seg, g, p, scores ? score_q : nullptr, scores ? score_f : nullptr, density, ws, s);
  } else {
    if (scores) launch_gram_f32(bank, seg, g, p, dkv_update_out{}, ws, s, kF32Score);
    if (density) launch_gram_f32(bank, seg, g, p, dkv_update_out{}, ws, s, kF32Density);
  }
  if (scores) k_score_out<<<grid2(g.N, 256, g.B), 256, 0, s>>>(g, ws, score_q, score_f);
  if (density) k_density_out<<<grid2(g.Mcap, 256, g.B), 256, 0, s>>>(g, ws, density);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_update(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                         const dkv_update_out *out, const Workspace &ws, hipStream_t s) {
  if (g.d == 128 && g.dtype == DKV_BF16) return update_impl<128, DKV_BF16>(bank, seg, g, p, out, ws, s);
  if (g.d == 128 && g.dtype == DKV_F32) return update_impl<128, DKV_F32>(bank, seg, g, p, out, ws, s);
  if (g.d == 64 && g.dtype == DKV_BF16) return update_impl<64, DKV_BF16>(bank, seg, g, p, out, ws, s);
  return update_impl<64, DKV_F32>(bank, seg, g, p, out, ws, s);
}

hipError_t launch_score(const dkv_bank &bank, const dkv_segment &seg, const Geom &g, const Prm &p,
                        int64_t *score_q, float *score_f, int64_t *density, const Workspace &ws,
                        hipStream_t s) {
  if (g.d == 128 && g.dtype == DKV_BF16) return score_impl<128, DKV_BF16>(bank, seg, g, p, score_q, score_f, density, ws, s);
  if (g.d == 128 && g.dtype == DKV_F32) return score_impl<128, DKV_F32>(bank, seg, g, p, score_q, score_f, density, ws, s);
  if (g.d == 64 && g.dtype == DKV_BF16) return score_impl<64, DKV_BF16>(bank, seg, g, p, score_q, score_f, density, ws, s);
  return score_impl<64, DKV_F32>(bank, seg, g, p, score_q, score_f, density, ws, s);
}

hipError_t launch_pair_weight(const float *d2, int64_t n, const Prm &p, int32_t *w, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  k_pair_weight<<<(unsigned)blocks, 256, 0, s>>>(d2, n, p, w);
  return hipGetLastError();
}

}  // namespace dkv
