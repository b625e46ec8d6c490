// Native attention over [retained bank; local window; sink] on gfx950.
//
// out = softmax(q K^T * scale) V with K = [bank k[0:m_b]; window k; sink k],
// the backbone's own attention reading the retained bank together with the
// local window (Sec. 1, Fig. 1; logit of Sec. 3.2) and, in the paper's
// deployment context, a first-frame sink (Supp. D, memory budget and temporal
// alignment).  Every segment is optional.  Online (streaming) softmax in
// fp32 over key tiles staged in LDS; exp2 with the scale folded into log2(e).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dkv_internal.hpp"

namespace dkv {
namespace {

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// The host sizes the splits of a call by the capacity.  Of them a bank takes as
// many as leave the first at least LEAST of its `total` tiles, one at least; the
// others end at once and leave no result.  (12 banks of capacity 18,720 that hold
// nothing yet, 64 queries, a window of 64: 15.5 us, 19.7 with every split at work,
// 10.3 without splits; 2 such fp32 banks 14.5, 39.7 and 31.8.)
template <int LEAST>
__device__ __forceinline__ int splits_used(int total, int nsplit) {
  return max(1, min(nsplit, LEAST > 1 ? (total - 1) / (LEAST - 1) : total));
}
// Tiles [t0, t1) of one split: the splits of a (bank, query block) take equal runs.
__device__ __forceinline__ void split_range(int total, int nsplit, int split, int &t0, int &t1) {
  const int per = (total + nsplit - 1) / nsplit;
  t0 = min(total, split * per);
  t1 = min(total, t0 + per);
}

// Partial results of a split attention: for split s and row (bank, query), the
// running maximum and weight sum of its keys and the unnormalised output.
struct Part {
  float *o;   // [S, rows, D]
  float2 *ml; // [S, rows] (maximum, sum); null without splits
};

// Weight sums of a row's keys (or part of them) under their maximum mx: -1 for
// keys whose scores are all -inf (the result is NaN unless other parts hold
// finite scores, whose combination multiplies this by 0), 0 without keys.
__device__ __forceinline__ float row_sum(float mx, float l, bool keys) {
  return keys && mx == -INFINITY && l == 0.0f ? -1.0f : l;
}
__device__ __forceinline__ float inv_sum(float l) { return l > 0.0f ? 1.0f / l : (l < 0.0f ? NAN : 0.0f); }

typedef float f32x16 __attribute__((ext_vector_type(16)));

// fp32 path on v_mfma_f32_32x32x2_f32 (fp32 products and sums).  A wave owns 32
// queries and walks tiles of 32 keys: S^T = K Q^T with the key rows as A and the
// query rows as B (both read 16 bytes at dims 8 c + 4 h, so K step 4 c + j takes
// dims 8 c + j and 8 c + 4 + j of both), so lane (h, n) holds query n's scores
// for keys 8 (i / 4) + 4 h + i % 4; then O^T += V^T P^T with register i's two
// keys as the K step.  Keys and values come straight from global memory: the
// four waves of a workgroup read the same tiles.  Few queries leave the chip
// idle, so the tiles are split over workgroups.  Before, one thread walked all
// keys of its query: 148 us for 64 queries over 320 keys in 2 banks (D = 64),
// 16 us now, most of it two launches.
constexpr int kRWaves = 4;
constexpr int kRQ = 32 * kRWaves;  // queries per workgroup
constexpr int kRK = 32;            // keys per tile
constexpr int kRLeast = 1;         // tiles of a split
constexpr int kFK = 64;            // bf16 path: keys per tile
constexpr int kFLeast = 4;         // and tiles of a split

template <int D>
__global__ __launch_bounds__(64 * kRWaves, 1) void k_attn_f32(dkv_bank bank, const float *__restrict__ q, int nq,
                                                              KvSeg win, KvSeg sink, float *__restrict__ out,
                                                              float scale_log2, Geom g, int nsplit, Part part) {
  constexpr int DT = D / 32, KC = D / 8;
  const int nqb = (nq + kRQ - 1) / kRQ;
  const int bs = blockIdx.x / nqb, b = bs / nsplit, split = bs % nsplit;
  const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = l >> 5, n = l & 31;
  const int q0 = (blockIdx.x % nqb) * kRQ + wave * 32, qi = q0 + n;
  if (q0 >= nq) return;  // whole wave; no barrier follows
  const bool qv = qi < nq;
  const int M = clampi(bank.budget[b], 0, g.Mcap);
  const int m = clampi(bank.occupancy[b], 0, M);
  const int nw = win.n, ns = sink.n;
  const int nt0 = (m + kRK - 1) / kRK, nt1 = nt0 + (nw + kRK - 1) / kRK;
  const int total = nt1 + (ns + kRK - 1) / kRK, used = splits_used<kRLeast>(total, nsplit);
  if (split >= used) return;
  int tb, nt;
  split_range(total, used, split, tb, nt);
  const size_t qrow = (size_t)b * nq + (qv ? qi : nq - 1);
  float4 qf[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) qf[c] = *reinterpret_cast<const float4 *>(q + qrow * D + 8 * c + 4 * h);
  f32x16 o[DT];
#pragma unroll
  for (int t2 = 0; t2 < DT; ++t2) o[t2] = f32x16{};
  float mx = -INFINITY, lsum = 0.0f;
  for (int t = tb; t < nt; ++t) {
    // tiles never straddle a segment boundary
    const float *kp, *vp;
    int nv;
    if (t < nt0) {
      const size_t r = (size_t)b * g.Mcap + (size_t)t * kRK;
      kp = static_cast<const float *>(bank.k) + r * D;
      vp = static_cast<const float *>(bank.v) + r * D;
      nv = min(kRK, m - t * kRK);
    } else if (t < nt1) {
      const size_t r = (size_t)b * nw + (size_t)(t - nt0) * kRK;
      kp = static_cast<const float *>(win.k) + r * D;
      vp = static_cast<const float *>(win.v) + r * D;
      nv = min(kRK, nw - (t - nt0) * kRK);
    } else {
      const size_t r = (size_t)b * ns + (size_t)(t - nt1) * kRK;
      kp = static_cast<const float *>(sink.k) + r * D;
      vp = static_cast<const float *>(sink.v) + r * D;
      nv = min(kRK, ns - (t - nt1) * kRK);
    }
    // rows past the tile's last key repeat it (their weights are 0)
    float4 kx[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) kx[c] = *reinterpret_cast<const float4 *>(kp + min(n, nv - 1) * D + 8 * c + 4 * h);
    float vx[DT][16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float *vr = vp + min(8 * (i >> 2) + 4 * h + (i & 3), nv - 1) * D + n;
#pragma unroll
      for (int t2 = 0; t2 < DT; ++t2) vx[t2][i] = vr[32 * t2];
    }
    f32x16 sc = {};
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kx[c].x, qf[c].x, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kx[c].y, qf[c].y, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kx[c].z, qf[c].z, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kx[c].w, qf[c].w, sc, 0, 0, 0);
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      sc[i] = 8 * (i >> 2) + 4 * h + (i & 3) < nv ? sc[i] * scale_log2 : -INFINITY;
      tmax = fmaxf(tmax, sc[i]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    const float mnew = fmaxf(mx, tmax);
    const float mref = mnew == -INFINITY ? 0.0f : mnew;  // scores of -inf alone: weights 0, not inf - inf
    const float corr = exp2f(mx - mref);
    mx = mnew;
    float p[16], ps = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = exp2f(sc[i] - mref);
      ps += p[i];
    }
    lsum = __builtin_fmaf(lsum, corr, ps);
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2) {
#pragma unroll
      for (int i = 0; i < 16; ++i) o[t2][i] *= corr;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int t2 = 0; t2 < DT; ++t2) o[t2] = __builtin_amdgcn_mfma_f32_32x32x2f32(vx[t2][i], p[i], o[t2], 0, 0, 0);
  }
  const float lt = row_sum(mx, lsum + __shfl_xor(lsum, 32, 64), tb < nt);
  if (!qv) return;
  float inv = 1.0f;
  float *dst = out + qrow * D;
  if (part.ml) {
    const size_t row = (size_t)split * g.B * nq + qrow;
    if (h == 0) part.ml[row] = float2{mx, lt};
    dst = part.o + row * D;
  } else {
    inv = inv_sum(lt);
  }
#pragma unroll
  for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
    for (int gg = 0; gg < 4; ++gg)
      *reinterpret_cast<float4 *>(dst + 32 * t2 + 8 * gg + 4 * h) =
          float4{o[t2][4 * gg] * inv, o[t2][4 * gg + 1] * inv, o[t2][4 * gg + 2] * inv, o[t2][4 * gg + 3] * inv};
}

// Rows of a split attention: the partial outputs under their common maximum
// (c: the factor of the maxima's unit to log2), divided by the common sum.
// One wave per row group: D / 4 lanes per row, 16-byte loads.
template <int D, int DT>
__global__ __launch_bounds__(256) void k_attn_combine(dkv_bank bank, Part part, int nsplit, size_t rows, int nq, int nw,
                                                      int ns, void *out, float c) {
  constexpr int LR = D / 4;
  const size_t row = (size_t)blockIdx.x * (256 / LR) + threadIdx.x / LR;
  const int j = 4 * (threadIdx.x % LR);
  if (row >= rows) return;
  // the splits that the row's bank took (few rows: a split call has at most some thousand workgroups)
  constexpr int K = DT == DKV_BF16 ? kFK : kRK;
  const uint32_t b = (uint32_t)row / (uint32_t)nq;
  const int m = clampi(bank.occupancy[b], 0, clampi(bank.budget[b], 0, bank.capacity));
  const int used = splits_used<DT == DKV_BF16 ? kFLeast : kRLeast>((m + K - 1) / K + (nw + K - 1) / K + (ns + K - 1) / K, nsplit);
  const float2 ml0 = part.ml[row];  // read while `used` is on its way
  const float4 x0 = *reinterpret_cast<const float4 *>(part.o + row * D + j);
  float M = ml0.x;
  for (int s = 1; s < used; ++s) M = fmaxf(M, part.ml[s * rows + row].x);
  const float w0 = ml0.x == M ? 1.0f : __builtin_amdgcn_exp2f((ml0.x - M) * c);
  float l = ml0.y * w0, a[4] = {x0.x * w0, x0.y * w0, x0.z * w0, x0.w * w0};
  for (int s = 1; s < used; ++s) {
    const float2 ml = part.ml[s * rows + row];
    const float4 x = *reinterpret_cast<const float4 *>(part.o + (s * rows + row) * D + j);
    const float w = ml.x == M ? 1.0f : __builtin_amdgcn_exp2f((ml.x - M) * c);
    l = __builtin_fmaf(ml.y, w, l);
    a[0] = __builtin_fmaf(x.x, w, a[0]);
    a[1] = __builtin_fmaf(x.y, w, a[1]);
    a[2] = __builtin_fmaf(x.z, w, a[2]);
    a[3] = __builtin_fmaf(x.w, w, a[3]);
  }
  const float inv = inv_sum(l);
  if constexpr (DT == DKV_BF16)
    *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(out) + row * D + j) =
        uint2{pack_bf16x2(a[0] * inv, a[1] * inv), pack_bf16x2(a[2] * inv, a[3] * inv)};
  else
    *reinterpret_cast<float4 *>(static_cast<float *>(out) + row * D + j) =
        float4{a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv};
}

// ---------------------------------------------------------------------------
// bf16 path on MFMA (v_mfma_f32_32x32x16_bf16).
//
// A workgroup of 8 waves owns 256 queries, 32 per wave.  Per tile of 64 keys:
//   S^T = K Q^T     A = K tile (LDS), B = Q^T (registers): lane l <-> query
//                   l % 32, registers <-> keys, so the softmax row statistics
//                   stay inside the lane (plus one exchange with lane l ^ 32);
//   O^T += V^T P^T  B = P straight from the S registers (bf16); A = V^T read
//                   from the row-major V tile with the transposing LDS read
//                   (ds_read_b64_tr_b16).  Inside each 16-key K step the key
//                   order is permuted identically in both operands
//                   (slot 8h + j <-> key 8 (j / 4) + 4 h + j % 4).
// K and V tiles go global -> LDS with 16-byte buffer loads to LDS (no VGPR
// staging) into a ring of three stages (two tiles in flight while one is
// used); rows are stored with an XOR swizzle of their
// 16-byte chunks so that both the K reads and the transposed V reads are free
// of LDS bank conflicts.  Within a tile the LDS fragment reads are scheduled
// ahead of the MFMAs that use them (6 MFMAs ahead for S, 4 for P V).
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kFWaves = 8;
constexpr int kFQ = 32 * kFWaves;  // queries per workgroup
constexpr int kFStages = 3;        // K/V tiles resident in LDS (2 in flight while 1 is used)
// Word 3 of a raw buffer resource: 32-bit data format, no swizzle, no
// thread-id addressing.
constexpr int kBufferRsrcWord3 = 0x00020000;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int D>
struct FCfg {
  static constexpr int kRowBytes = 2 * D;           // one K or V row
  static constexpr int kChunks = D / 8;             // 16-byte chunks per row
  static constexpr int kRowsPerLoad = 1024 / kRowBytes;   // rows per 1 KB direct load
  static constexpr int kLoadsPerTile = kFK / kRowsPerLoad;  // per tensor, per workgroup
  static constexpr int kTileBytes = kFK * kRowBytes;
};

// Physical 16-byte chunk of logical chunk c of row r (K: conflict-free 16-byte
// reads of one chunk across 16 rows; V: conflict-free transposed 8-byte reads
// of 4 chunks across 4 rows).
template <int D>
__device__ __forceinline__ int k_swz(int r, int c) { return c ^ (r % FCfg<D>::kChunks); }
template <int D>
__device__ __forceinline__ int v_swz(int r, int c) { return c ^ ((4 * (r % 4)) % FCfg<D>::kChunks); }

// The direct-to-LDS loads of one K or V tile.  Lane i of a load writes 16
// bytes at LDS offset 16 i of its 1 KB block, i.e. physical chunk pc of row r;
// it fetches logical chunk swz(r, pc) (the XOR swizzle is an involution, so
// logical chunk c lands at physical swz(r, c)).  These byte offsets within a
// tile are the same for every tile, so they are computed once per lane; the
// tile's first row is the uniform buffer base and the buffer ends after its
// nvalid rows, so the rows beyond read as zero (finite; their scores are
// masked and their weights are 0).  The loads are raw buffer loads to LDS
// rather than global loads to LDS: with a global load to LDS in flight the
// compiler counts every later LDS read as possibly out of order and waits for
// all of them before each use, which serializes the MFMAs on the LDS latency.
template <int D>
struct FTileOff {
  static constexpr int kPerWave = FCfg<D>::kLoadsPerTile / kFWaves;  // loads per wave per tensor
  int k[kPerWave], v[kPerWave];
};

template <int D>
__device__ __forceinline__ FTileOff<D> ftile_offsets() {
  constexpr int RPL = FCfg<D>::kRowsPerLoad, CH = FCfg<D>::kChunks;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int rsub = l / CH, pc = l % CH;
  FTileOff<D> o;
#pragma unroll
  for (int q = 0; q < FTileOff<D>::kPerWave; ++q) {
    const int r = (wave * FTileOff<D>::kPerWave + q) * RPL + rsub;
    o.k[q] = (r * D + 8 * k_swz<D>(r, pc)) * 2;
    o.v[q] = (r * D + 8 * v_swz<D>(r, pc)) * 2;
  }
  return o;
}

template <int D>
__device__ __forceinline__ void ftile_issue(const uint16_t *base, int nvalid, char *buf,
                                            const int *voff /*[FTileOff<D>::kPerWave]*/) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const __amdgpu_buffer_rsrc_t rs =  // base and extent are uniform
      __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, nvalid * FCfg<D>::kRowBytes, kBufferRsrcWord3);
#pragma unroll
  for (int q = 0; q < FTileOff<D>::kPerWave; ++q)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(buf + (wave * FTileOff<D>::kPerWave + q) * 1024), 16,
                                             voff[q], 0, 0, 0);
}

// Lazy softmax bound: the reference maximum is only raised when a lane's tile
// sum of exp2 terms exceeds 2^16 (or is not finite), so every P stays below
// 2^16 and the running sums stay far from overflow; the final division by l
// removes the common factor exactly.
constexpr float kLazyLimit = 65536.0f;

// s_waitcnt immediate (gfx9 encoding): at most n vector-memory operations
// outstanding and no LDS operation outstanding (expcnt left alone).
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

// Workgroup barrier for the K/V stages.  Each thread has already waited for
// its own direct-to-LDS loads of the stage about to be read (and for its LDS
// reads), so the barrier needs no memory fence; the "memory" clobber keeps
// the compiler from moving LDS accesses across it, and leaving out the fence
// keeps it from also waiting for the next stage's loads, which stay in flight.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_barrier" ::: "memory"); }

// SPLIT: the keys in nsplit splits (its index arithmetic and the partial results cost
// a call without splits 0.3 to 0.5 us, 2% of the smallest).
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kFWaves, 1) void k_attn_mfma(dkv_bank bank, const uint16_t *q, int nq,
                                                               KvSeg win, KvSeg sink,
                                                               uint16_t *out, float c, Geom g, int nsplit, Part part) {
  constexpr int KS = D / 16;   // K steps of S
  constexpr int DT = D / 32;   // dv tiles of O
  constexpr int RB = FCfg<D>::kRowBytes;
  constexpr int TB = FCfg<D>::kTileBytes;
  // direct-to-LDS loads per thread for one K + V tile
  constexpr int kTileLoads = 2 * (FCfg<D>::kLoadsPerTile / kFWaves);
  static_assert(FCfg<D>::kLoadsPerTile % kFWaves == 0, "tile loads must split evenly over the waves");
  // Workgroup L is dispatched to XCD L % 8.  Rank the workgroups XCD by XCD
  // (p = workgroups on lower XCDs + L / 8) and give rank p query block p % nqb
  // of (bank, key split) p / nqb: the query blocks that read the same keys and
  // values then run on one XCD and share its L2 for them.
  const int nqb = (nq + kFQ - 1) / kFQ;
  const int T = (int)gridDim.x, L = (int)blockIdx.x, xcd = L % 8;
  const int p = xcd * (T / 8) + min(xcd, T % 8) + L / 8;
  const int bs = p / nqb, qblk = p % nqb;
  const int b = SPLIT ? bs / nsplit : bs, split = SPLIT ? bs % nsplit : 0;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, h = l >> 5, n = l & 31;
  const int M = clampi(bank.budget[b], 0, g.Mcap);
  const int m = clampi(bank.occupancy[b], 0, M);
  const int nw = win.n, ns = sink.n;
  const size_t rb = (size_t)b * g.Mcap, wb = (size_t)b * nw, sb = (size_t)b * ns;
  const uint16_t *wk = static_cast<const uint16_t *>(win.k), *wv = static_cast<const uint16_t *>(win.v);
  const uint16_t *sk = static_cast<const uint16_t *>(sink.k), *sv = static_cast<const uint16_t *>(sink.v);
  const uint16_t *bk = static_cast<const uint16_t *>(bank.k);
  const uint16_t *bv = static_cast<const uint16_t *>(bank.v);
  // One LDS array per stage (not one indexed array): with the stage known at
  // compile time the compiler can tell that reads of one stage never wait for
  // the direct-to-LDS loads still filling the others.
  __shared__ __attribute__((aligned(1024))) char k0[TB], k1[TB], k2[TB];
  __shared__ __attribute__((aligned(1024))) char v0[TB], v1[TB], v2[TB];

  const int qi = qblk * kFQ + wave * 32 + n;
  const bool qv = qi < nq;
  bf16x8 qf[KS];
  const size_t qrow = (size_t)b * nq + (qv ? qi : 0);
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    u32x4 x = {0, 0, 0, 0};
    if (qv) x = *reinterpret_cast<const u32x4 *>(q + qrow * D + 16 * kk + 8 * h);
    qf[kk] = __builtin_bit_cast(bf16x8, x);
  }
  f32x16 o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) o[t] = f32x16{};
  float mrun = -INFINITY, lrun = 0.0f;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  // Tiles never straddle the bank/window boundary: ceil(m/64) bank tiles, then
  // ceil(nw/64) window tiles, so every tile has one (scalar) base pointer.
  const int nt0 = (m + kFK - 1) / kFK;
  const int nt1 = nt0 + (nw + kFK - 1) / kFK;
  // this split's tiles [tb, nt)
  int tb = 0, nt = nt1 + (ns + kFK - 1) / kFK;
  if constexpr (SPLIT) {
    const int used = splits_used<kFLeast>(nt, nsplit);
    if (split >= used) return;  // whole workgroup
    split_range(nt, used, split, tb, nt);
  }
  auto nvalid_of = [&](int t) {
    return t < nt0 ? min(kFK, m - t * kFK) : (t < nt1 ? min(kFK, nw - (t - nt0) * kFK) : min(kFK, ns - (t - nt1) * kFK));
  };
  const FTileOff<D> toff = ftile_offsets<D>();
  auto issue = [&](int t, char *kd, char *vd) {
    if (t >= nt) return;
    const int nv = nvalid_of(t);
    if (t < nt0) {
      ftile_issue<D>(bk + (rb + (size_t)t * kFK) * D, nv, kd, toff.k);
      ftile_issue<D>(bv + (rb + (size_t)t * kFK) * D, nv, vd, toff.v);
    } else if (t < nt1) {
      const size_t r0 = wb + (size_t)(t - nt0) * kFK;
      ftile_issue<D>(wk + r0 * D, nv, kd, toff.k);
      ftile_issue<D>(wv + r0 * D, nv, vd, toff.v);
    } else {
      const size_t r0 = sb + (size_t)(t - nt1) * kFK;
      ftile_issue<D>(sk + r0 * D, nv, kd, toff.k);
      ftile_issue<D>(sv + r0 * D, nv, vd, toff.v);
    }
  };
  // transposed V read: lane group gq = l / 16 (h = gq / 2), member cq = l % 16
  const int gq = l >> 4, cq = l & 15;

  // Tile t lives in stage t % 3.  Wait for its loads (the loads of tile t + 1
  // may stay in flight), then at the barrier every wave has finished tile
  // t - 1, so its stage receives tile t + 2.  Then S^T = K Q^T, softmax
  // update, O^T += V^T P^T.
  auto sync = [&](int t, char *kn, char *vn) __attribute__((always_inline)) {
    if (t + 1 < nt) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kTileLoads));
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
    stage_barrier();
    issue(t + 2, kn, vn);
  };
  auto step = [&](int t, const char *kt, const char *vtile, char *kn, char *vn) {
    sync(t, kn, vn);
    f32x16 sc[2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const int key = 32 * sub + n;
      bf16x8 a[KS];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        a[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kt + key * RB + 16 * k_swz<D>(key, 2 * kk + h)));
      f32x16 acc = {};
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], qf[kk], acc, 0, 0, 0);
      sc[sub] = acc;
    }
    // S block: LDS fragment reads run 6 MFMAs ahead of their use
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i + 6 < 2 * KS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    const int nvalid = nvalid_of(t);
    if (nvalid < kFK) {
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (32 * sub + 8 * (i >> 2) + 4 * h + (i & 3) >= nvalid) sc[sub][i] = -INFINITY;
    }
    uint32_t pb[2][8];
    float psum = 0.0f;
    auto exps = [&](float moff) {
      float ps[2] = {0.0f, 0.0f};
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[sub][i], c, moff));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[sub][i + 1], c, moff));
          pb[sub][i >> 1] = pack_bf16x2(p0, p1);
          // row sum of the bf16 weights actually multiplied into O
          ps[sub] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pb[sub][i >> 1]), ones, ps[sub], false);
        }
      psum = ps[0] + ps[1];
    };
    exps(-mrun * c);
    if (__any(!(psum <= kLazyLimit))) {
      float tmax = sc[0][0];
#pragma unroll
      for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, sc[0][i]);
#pragma unroll
      for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, sc[1][i]);
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      const float mnew = fmaxf(mrun, tmax);
      const float mref = mnew == -INFINITY ? 0.0f : mnew;  // scores of -inf alone: weights 0, not inf - inf
      const float corr = __builtin_amdgcn_exp2f((mrun - mref) * c);
      mrun = mnew;
      lrun *= corr;
#pragma unroll
      for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[t2][i] *= corr;
      exps(-mref * c);
    }
    lrun += psum;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int kst = 0; kst < 2; ++kst) {
        u32x4 bp = {pb[sub][4 * kst + 0], pb[sub][4 * kst + 1], pb[sub][4 * kst + 2], pb[sub][4 * kst + 3]};
        const bf16x8 bop = __builtin_bit_cast(bf16x8, bp);
        const int key0 = 32 * sub + 16 * kst + 4 * (gq >> 1) + (cq >> 2);
#pragma unroll
        for (int t2 = 0; t2 < DT; ++t2) {
          const int dvb = 8 * t2 + 4 * (gq & 1) + (cq & 3);  // 8-byte dv block
          const int ka = key0, kb = key0 + 8;
          const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_i16x4 *)(vtile + ka * RB + 16 * v_swz<D>(ka, dvb >> 1) + 8 * (dvb & 1)));
          const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_i16x4 *)(vtile + kb * RB + 16 * v_swz<D>(kb, dvb >> 1) + 8 * (dvb & 1)));
          const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
          const u32x4 av = {lo2[0], lo2[1], hi2[0], hi2[1]};
          o[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), bop, o[t2], 0, 0, 0);
        }
      }
    }
    // P V block: the two transposed reads of an MFMA run 4 MFMAs ahead of it
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
    for (int i = 0; i < 4 * DT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i + 4 < 4 * DT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
  };

  static_assert(kFStages == 3, "the loop below cycles through three stage buffers");
  issue(tb, k0, v0);
  issue(tb + 1, k1, v1);
  if (__builtin_amdgcn_readfirstlane(qblk * kFQ + wave * 32) >= nq) {  // a wave past the last query only loads
    for (int t = tb; t < nt; t += kFStages) {
      sync(t, k2, v2);
      if (t + 1 < nt) sync(t + 1, k0, v0);
      if (t + 2 < nt) sync(t + 2, k1, v1);
    }
    return;
  }
  for (int t = tb; t < nt; t += kFStages) {
    step(t, k0, v0, k2, v2);
    if (t + 1 < nt) step(t + 1, k1, v1, k0, v0);
    if (t + 2 < nt) step(t + 2, k2, v2, k1, v1);
  }
  // both half-waves hold the row's maximum (raised together) and a part of its sum
  const float ltot = row_sum(mrun, lrun + __shfl_xor(lrun, 32, 64), tb < nt);
  if (!qv) return;
  if constexpr (SPLIT) {
    const size_t row = (size_t)split * g.B * nq + qrow;
    if (h == 0) part.ml[row] = float2{mrun, ltot};
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg)
        *reinterpret_cast<float4 *>(part.o + row * D + 32 * t2 + 8 * gg + 4 * h) =
            float4{o[t2][4 * gg], o[t2][4 * gg + 1], o[t2][4 * gg + 2], o[t2][4 * gg + 3]};
    return;
  }
  const float inv = inv_sum(ltot);
#pragma unroll
  for (int t2 = 0; t2 < DT; ++t2) {
#pragma unroll
    for (int gg = 0; gg < 4; ++gg) {
      const int dv = 32 * t2 + 8 * gg + 4 * h;
      u32x2 pk = {pack_bf16x2(o[t2][4 * gg] * inv, o[t2][4 * gg + 1] * inv),
                  pack_bf16x2(o[t2][4 * gg + 2] * inv, o[t2][4 * gg + 3] * inv)};
      *reinterpret_cast<u32x2 *>(out + qrow * D + dv) = pk;
    }
  }
}

constexpr int kCUs = 256;
constexpr int kMaxSplit = 64;

// Key splits of a call whose query blocks alone do not fill the chip.  A
// workgroup of the bf16 kernel takes a whole CU (256 queries, 96 KB of tile
// stages), so the time is about rounds x (tiles per split + 6 tiles of
// prologue and epilogue), plus a second kernel that combines the partial
// results (about 4 tiles of launch and, in tiles of 1.6 us, its traffic).  With
// 84 workgroups (12 banks x 7 query blocks, 18,720 keys) this gives 3 splits (417
// -> 176 us); with 228 (12 x 19) a split cannot help, and one workgroup per query
// block stays (237 us either way).
int attn_splits_bf16(long long nwg, long long rows, int tiles, int d) {
  int best = 1;
  double best_cost = 0.0;
  for (int S = 1; S <= kMaxSplit && (S == 1 || (tiles + S - 1) / S >= kFLeast); ++S) {
    const double rounds = (double)((nwg * S + kCUs - 1) / kCUs);
    double cost = rounds * ((tiles + S - 1) / S + 6);
    if (S > 1) cost += 4.0 + (double)rows * S * (8.0 * d + 16.0) / (4e12 * 1.6e-6);
    if (S == 1 || cost < 0.95 * best_cost) best = S, best_cost = cost;
  }
  return best;
}

// fp32: a split walks at least one 32-key tile; up to two workgroups a CU.
int attn_splits_f32(long long nwg, int tiles) {
  const long long fill = 2 * kCUs / nwg;
  return (int)(fill < 1 ? 1 : (fill > tiles ? (tiles < 1 ? 1 : tiles) : fill));
}

// A split call takes a second launch and a buffer for the partial results: 14 us
// from launch to launch where an unsplit call takes 10 (eager calls from Python; a
// smaller GPU time shows in a captured graph only).  So calls whose one workgroup
// per query block ends within 14 us stay unsplit.  Its time: bf16 with 2 (8) of the
// 8 waves at work 3.0 + 0.72 (5.1 + 1.02) us per tile at d = 64, 3.7 + 0.94 (7.9 +
// 1.34) at d = 128; fp32 3.2 + 2.9 and 3.9 + 5.1.  2 banks x 64 queries, d = 64: 10
// tiles 10.2 us unsplit, 15.2 split; 16 tiles 14.7 and 14.8; 24 tiles 20.3 and 13.9.
constexpr double kSplitFrom = 14.0;
double unsplit_us(int dtype, int d, int nq, int tiles) {
  if (dtype != DKV_BF16) return d == 64 ? 3.2 + 2.9 * tiles : 3.9 + 5.1 * tiles;
  const int w = nq >= kFQ ? kFWaves : (nq + 31) / 32;  // waves at work
  return d == 64 ? 2.3 + 0.35 * w + (0.62 + 0.05 * w) * tiles : 2.3 + 0.7 * w + (0.81 + 0.066 * w) * tiles;
}

}  // namespace

// Splits the launch takes (1: none) and the bytes of its partial results.
int attention_splits(const dkv_bank &bank, int nq, int nw, int ns, size_t *bytes) {
  *bytes = 0;
  if (nq <= 0) return 1;
  const long long rows = (long long)bank.num_banks * nq;
  const int K = bank.dtype == DKV_BF16 ? kFK : kRK;
  const int tiles = (bank.capacity + K - 1) / K + (nw + K - 1) / K + (ns + K - 1) / K;
  if (unsplit_us(bank.dtype, bank.head_dim, nq, tiles) < kSplitFrom) return 1;
  int S;
  if (bank.dtype == DKV_BF16) {
    S = attn_splits_bf16((long long)((nq + kFQ - 1) / kFQ) * bank.num_banks, rows, tiles, bank.head_dim);
  } else {
    S = attn_splits_f32((long long)((nq + kRQ - 1) / kRQ) * bank.num_banks, tiles);
    if (S > kMaxSplit) S = kMaxSplit;
  }
  if (S > 1) *bytes = (size_t)rows * S * (bank.head_dim * 4 + 8);
  return S;
}

namespace {

template <int D, int DT>
hipError_t attn_impl(const dkv_bank &bank, const void *q, int nq, KvSeg win, KvSeg sink,
                     void *out, float scale, const Geom &g, void *ws, int nsplit, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  const float scale_log2 = scale * 1.4426950408889634f;
  const size_t rows = (size_t)g.B * nq;
  Part part{nullptr, nullptr};
  if (nsplit > 1) {  // the outputs first (rows of D floats), then the maxima and sums
    part.o = static_cast<float *>(ws);
    part.ml = reinterpret_cast<float2 *>(part.o + rows * nsplit * D);
  }
  const int per = DT == DKV_BF16 ? kFQ : kRQ;
  const long long nwg = (long long)((nq + per - 1) / per) * g.B * nsplit;   // one-dimensional grid
  if (nwg > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  if constexpr (DT == DKV_BF16) {
    const uint16_t *qb = static_cast<const uint16_t *>(q);
    uint16_t *ob = static_cast<uint16_t *>(out);
    const dim3 grid((unsigned)nwg);
    if (nsplit > 1) k_attn_mfma<D, true><<<grid, 64 * kFWaves, 0, s>>>(bank, qb, nq, win, sink, ob, scale_log2, g, nsplit, part);
    else k_attn_mfma<D, false><<<grid, 64 * kFWaves, 0, s>>>(bank, qb, nq, win, sink, ob, scale_log2, g, nsplit, part);
  } else {
    k_attn_f32<D><<<(unsigned)nwg, 64 * kRWaves, 0, s>>>(bank, static_cast<const float *>(q), nq, win, sink,
                                                             static_cast<float *>(out), scale_log2, g, nsplit, part);
  }
  if (nsplit > 1) {
    constexpr int kRows = 256 / (D / 4);
    // the bf16 maxima are raw scores, the fp32 ones already in log2 units
    k_attn_combine<D, DT><<<(unsigned)((rows + kRows - 1) / kRows), 256, 0, s>>>(bank, part, nsplit, rows, nq, win.n, sink.n,
                                                                                 out, DT == DKV_BF16 ? scale_log2 : 1.0f);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention(const dkv_bank &bank, const void *q, int nq, KvSeg win, KvSeg sink, void *out,
                            float scale, const Geom &g, void *ws, int nsplit, hipStream_t s) {
  auto impl = g.d == 128 ? (g.dtype == DKV_BF16 ? attn_impl<128, DKV_BF16> : attn_impl<128, DKV_F32>)
                         : (g.dtype == DKV_BF16 ? attn_impl<64, DKV_BF16> : attn_impl<64, DKV_F32>);
  return impl(bank, q, nq, win, sink, out, scale, g, ws, nsplit, s);
}

}  // namespace dkv
