// Products of the training path with bf16 weights: float32 activations times
// bf16 weights, float32 accumulation, on the bf16 matrix pipes.
//
// A float32 value of magnitude 2^-109 or more is the exact sum of three bf16
// values (split3), and a product of two bf16 values is exact in float32 short of
// underflow, so  x w = hi w + mid w + lo w  costs three bf16 MFMAs and rounds
// only in the float32 accumulator, as the float32 MFMA does.  Below 2^-109 the
// terms miss less than 2^-133 of x.  bf16 MFMA runs at 16
// times the float32 rate, so three terms are worth it (per-launch figures at
// train_gemm3_kernel).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_util.h"
#include "train_internal.h"

namespace svl {
namespace {

constexpr int G3_BM = 128, G3_BN = 256, G3_BK = 32;
constexpr int G3_NT = 512;                       // 8 waves, 2 x 4 of 64 x 64 outputs
constexpr int G3_PLANE = G3_BM * G3_BK;          // bf16 values of one A term in a stage
constexpr int G3_STAGE = 3 * G3_PLANE + G3_BN * G3_BK;

// Eight float32 values as three bf16 vectors: each term is what is left cut to 8
// bits one unit below it, so hi + mid + lo == x exactly for |x| >= 2^-109 (below,
// lo loses less than 2^-133), and none of the three is zero unless x is: times
// an infinite weight each is an infinity of the same sign, where a zero term would
// make a NaN.  An infinity has an infinite lo, a NaN is one in every term.
// x is no -0 (the saturating step would make a NaN of it) unless NEG0, which turns
// it into +0 first: free where a scale precedes it, 2% of a step elsewhere (8
// layers, 640 rows: 17.8 ms, 18.15 with it), so the step's kernels store their
// rows with + 0.0f instead.
template <bool NEG0>
__device__ __forceinline__ void split3(const float4& a, const float4& b, uint4& hi, uint4& mid,
                                       uint4& lo) {
  const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t h[8], m[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float v = NEG0 ? x[i] + 0.0f : x[i];
    h[i] = __builtin_elementwise_sub_sat(__float_as_uint(v), 1u);
    const float r = v - __uint_as_float(h[i] & 0xffff0000u);
    m[i] = __builtin_elementwise_sub_sat(__float_as_uint(r), 1u);
    l[i] = __float_as_uint(r - __uint_as_float(m[i] & 0xffff0000u));
  }
  // the upper halves of a pair of words, first value in the low half
  auto up = [](uint32_t v0, uint32_t v1) { return __builtin_amdgcn_perm(v1, v0, 0x07060302u); };
  hi = make_uint4(up(h[0], h[1]), up(h[2], h[3]), up(h[4], h[5]), up(h[6], h[7]));
  mid = make_uint4(up(m[0], m[1]), up(m[2], m[3]), up(m[4], m[5]), up(m[6], m[7]));
  lo = make_uint4(up(l[0], l[1]), up(l[2], l[3]), up(l[4], l[5]), up(l[6], l[7]));
}

__device__ __forceinline__ float4 as_f4(const uint4& v) { return __builtin_bit_cast(float4, v); }

// C = R + (s . A) op(B): BL = 0 reads B as [N][K], BL = 1 as [K][N].  NEG0: A may
// hold -0 (rows that no kernel of the step wrote).
//
// Tile: 128 rows x 256 columns over 8 waves of 64 x 64 (4 x 4 blocks of
// v_mfma_f32_16x16x32_bf16), K in steps of 32.  Per step the workgroup holds
// the three terms of A (24 KB) and B (16 KB) in LDS, in fragment order (a
// 16 x 32 block is 1 KB, lane l's 16 bytes at 16 l), free of bank conflicts (BL = 1,
// whose columns are transposed on the way in: 0.8 conflict cycles an LDS
// instruction); two such stages, one barrier each.  Next step's operands
// wait in registers: the split costs about 8 VALU operations per value, once per
// workgroup, and is done by waves 0-3 before their products and by waves 4-7
// after theirs, so the two waves of a SIMD alternate between the vector and
// the matrix pipe.
//
// Three terms make the tile compute-bound: a step is 1536 cycles of MFMA per
// SIMD against 32 KB of loads and 168 KB of LDS traffic.  At 640 rows, 7B shape
// (float32 MFMA with 64 x 64 tiles before): Q, K and V in one launch 181 us
// (three launches of 200 us), gate and up 353 (1000), output 71 + 10 for the
// slices (224), down 164 + 11 (600), the gradients of gate and up in one launch
// 321 + 8 (1100): 0.91-1.08 PFLOP/s of bf16 products without the slices, 0.80-1.07
// with them, where a library product of 8192^3 reaches 1.15 on the same card;
// the matrix pipes are 47-49% busy.  Sums in two
// levels (below) cost 4% of that and bring the error of a two-layer step against
// float64 to 0.9e-6 (hidden), 1.5e-6 (token gradients) and 1.3e-6 (gate gradients),
// medians of 700 seeds; float32 MFMA 3.2e-6, 3.7e-6 and 8.1e-6, one level 2.3e-6,
// 3.6e-6 and 6.0e-6, means of eight.
template <int BL, bool ASC, bool NEG0>
__global__ __launch_bounds__(G3_NT, 1) void train_gemm3_kernel(TGemm3Args a) {
  __shared__ __attribute__((aligned(16))) uint16_t sm[2 * G3_STAGE];
  const int tix = xcd_tile_index();
  if (tix >= a.ntiles) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  // tile order: M fastest (the M tiles of a weight slice run together on one
  // XCD), then N, then the K piece
  const int mt = tix % a.mtiles;
  const int rest = tix / a.mtiles;
  const int piece = rest / a.ntn;
  int nt = rest % a.ntn;
  int sn = 0;                                    // output segment (ksegs: always 0)
  if (!a.ksegs) {
    while (sn + 1 < a.nseg && nt >= a.seg[sn].ntn) nt -= a.seg[sn++].ntn;
  }
  const int64_t m0 = (int64_t)mt * G3_BM;
  const int n0 = nt * G3_BN;
  const int rows = (int)(a.M - m0 < G3_BM ? a.M - m0 : G3_BM);
  const int N = a.seg[sn].N;
  const int c_lo = piece * a.cpiece;             // K steps of this piece
  const int c_hi = c_lo + a.cpiece < a.nchunks ? c_lo + a.cpiece : a.nchunks;

  // A: thread -> (row, 8 k) in fragment order; B likewise (BL = 0: two pieces of 8
  // k of one column; BL = 1: 8 k of two columns)
  const int ar = 16 * (tid >> 6) + (lane & 15), ak = 8 * (lane >> 4);
  const int64_t arow = m0 + ar;
  const float* srow = nullptr;
  if constexpr (ASC) srow = a.ascale + (ar < rows ? (arow / a.S) * a.astride : 0);
  const int b1k = 8 * (wave & 3), b1n = 128 * (wave >> 2) + 2 * lane;   // BL = 1

  uint4 ra[2], rb[2];
  uint32_t rt[8];
  float sc[2];
  auto load = [&](int c) __attribute__((always_inline)) {
    int s = sn, kc = c;
    if (a.ksegs) {
      s = 0;
      while (s + 1 < a.nseg && kc >= a.seg[s].chunks) kc -= a.seg[s++].chunks;
    }
    const TSeg& g = a.seg[s];
    const int k0 = kc * G3_BK;
    const uint32_t ldA = (uint32_t)g.lda * 4u, ldB = (uint32_t)g.ldb * 2u;
    const __amdgpu_buffer_rsrc_t rsA = make_rsrc(g.A + m0 * g.lda, (uint32_t)rows * ldA);
    const uint32_t oob = 0x80000000u;            // past every range: reads zero
    const uint32_t oa = k0 + ak < g.K ? ar * ldA + (uint32_t)(k0 + ak) * 4u : oob;
    ra[0] = load16(rsA, oa, 0);
    ra[1] = load16(rsA, oa + 16u, 0);
    if constexpr (ASC) {
      const int kk = k0 + ak < g.K ? k0 + ak : 0;
      sc[0] = srow[(uint32_t)kk / (uint32_t)a.kg];
      sc[1] = srow[(uint32_t)(kk + 4) / (uint32_t)a.kg];
    }
    if constexpr (BL == 0) {
      const int ncol = N - n0 < G3_BN ? N - n0 : G3_BN;
      const __amdgpu_buffer_rsrc_t rsB =
          make_rsrc(static_cast<const uint16_t*>(g.B) + (int64_t)n0 * g.ldb, (uint32_t)ncol * ldB);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int col = 128 * h + ar;            // block 8 h + wave, column lane % 16
        rb[h] = load16(rsB, k0 + ak < g.K && col < ncol ? col * ldB + (uint32_t)(k0 + ak) * 2u : oob, 0);
      }
    } else {
      const int kr = g.K - k0 < G3_BK ? g.K - k0 : G3_BK;
      const __amdgpu_buffer_rsrc_t rsB =
          make_rsrc(static_cast<const uint16_t*>(g.B) + (int64_t)k0 * g.ldb, (uint32_t)kr * ldB);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        rt[j] = __builtin_amdgcn_raw_buffer_load_b32(
            rsB, n0 + b1n < N ? (uint32_t)(b1k + j) * ldB + (uint32_t)(n0 + b1n) * 2u : oob, 0, 0);
    }
  };
  // BL = 1: 16-byte units of column pairs; unit index inside a block XOR f(block)
  // spreads a half wave's stores over all banks
  auto swz = [](int blk) { return BL == 1 ? (blk & 1) | ((blk & 2) << 3) : 0; };
  auto store = [&](int buf) __attribute__((always_inline)) {
    uint16_t* S = sm + buf * G3_STAGE;
    float4 x0 = as_f4(ra[0]), x1 = as_f4(ra[1]);
    if constexpr (ASC) {
      x0 = make_float4(x0.x * sc[0], x0.y * sc[0], x0.z * sc[0], x0.w * sc[0]);
      x1 = make_float4(x1.x * sc[1], x1.y * sc[1], x1.z * sc[1], x1.w * sc[1]);
    }
    uint4 t[3];
    split3<ASC || NEG0>(x0, x1, t[0], t[1], t[2]);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(&S[p * G3_PLANE + tid * 8]) = t[p];
    uint16_t* SB = S + 3 * G3_PLANE;
    if constexpr (BL == 0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) *reinterpret_cast<uint4*>(&SB[(512 * h + tid) * 8]) = rb[h];
    } else {
      const int blk = b1n >> 4, u = (b1k >> 3) * 16 + (b1n & 15);
      uint4 c0, c1;
      uint32_t* p0 = reinterpret_cast<uint32_t*>(&c0);
      uint32_t* p1 = reinterpret_cast<uint32_t*>(&c1);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        p0[j] = __builtin_amdgcn_perm(rt[2 * j + 1], rt[2 * j], 0x05040100u);
        p1[j] = __builtin_amdgcn_perm(rt[2 * j + 1], rt[2 * j], 0x07060302u);
      }
      *reinterpret_cast<uint4*>(&SB[(64 * blk + (u ^ swz(blk))) * 8]) = c0;
      *reinterpret_cast<uint4*>(&SB[(64 * blk + ((u + 1) ^ swz(blk))) * 8]) = c1;
    }
  };

  // acc sums 512 columns of K at a time, total the whole piece: a sum of n terms
  // in two levels rounds at the size of the short sums
  floatx4 acc[4][4], total[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = total[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const bool live = 64 * wm < rows && n0 + 64 * wn < N;   // the wave owns outputs
  auto compute = [&](int buf) __attribute__((always_inline)) {
    const uint16_t* S = sm + buf * G3_STAGE;
    const uint16_t* SB = S + 3 * G3_PLANE;
    uint4 fb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int blk = 4 * wn + j;
      fb[j] = *reinterpret_cast<const uint4*>(&SB[(64 * blk + (lane ^ swz(blk))) * 8]);
    }
#pragma unroll
    for (int p = 2; p >= 0; --p) {
      uint4 fa[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        fa[i] = *reinterpret_cast<const uint4*>(&S[p * G3_PLANE + (64 * (4 * wm + i) + lane) * 8]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma16x16x32<false>(fa[i], fb[j], acc[i][j]);
    }
  };

  if (c_lo < c_hi) {
    load(c_lo);
    store(0);
    if (c_lo + 1 < c_hi) load(c_lo + 1);
    __syncthreads();
    for (int c = c_lo; c < c_hi; ++c) {
      const int buf = (c - c_lo) & 1;
      auto refill = [&]() __attribute__((always_inline)) {
        if (c + 1 < c_hi) store(buf ^ 1);
        if (c + 2 < c_hi) load(c + 2);
      };
      if (wave < 4) refill();
      if (live) compute(buf);
      if (wave >= 4) refill();
      if (((c - c_lo) & 15) == 15 || c + 1 == c_hi) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            total[i][j] += acc[i][j];
            acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
      }
      __syncthreads();
    }
  }

  // total[i][j][r] = C[64 wm + 16 i + 4 (lane / 16) + r][64 wn + 16 j + lane % 16]
  // (piece 0 of a split in its place in C, the others in their slices)
  float* C = piece ? a.part + (int64_t)(piece - 1) * a.M * a.ncols + (a.ksegs ? 0 : a.seg[sn].col0)
                   : a.seg[sn].C;
  const int64_t ldc = piece ? a.ncols : a.seg[sn].ldc;
  const float* R = a.ksplit > 1 ? nullptr : a.R;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int col = n0 + 64 * wn + 16 * j + (lane & 15);
    if (col >= N) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 64 * wm + 16 * i + 4 * (lane >> 4) + r;
        if (row >= rows) continue;
        float o = total[i][j][r];
        if (R) o += R[(m0 + row) * a.ldr + col];
        C[(m0 + row) * ldc + col] = o;
      }
  }
}

// C = R + the K pieces added in order (the first is in C), four columns per thread.
__global__ void train_reduce3_kernel(TGemm3Args a) {
  const int n4 = a.ncols / 4;
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= a.M * n4) return;
  const int64_t m = q / n4;
  const int c = (int)(q % n4) * 4;
  int sn = 0;
  if (!a.ksegs)
    while (sn + 1 < a.nseg && c >= a.seg[sn + 1].col0) ++sn;
  const int cc = a.ksegs ? c : c - a.seg[sn].col0;
  float4* out = reinterpret_cast<float4*>(a.seg[sn].C + m * a.seg[sn].ldc + cc);
  float4 s = *out;
  for (int z = 1; z < a.ksplit; ++z) {
    const float4 p = *reinterpret_cast<const float4*>(a.part + ((z - 1) * a.M + m) * a.ncols + c);
    s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
  }
  if (a.R) {
    const float4 r = *reinterpret_cast<const float4*>(a.R + m * a.ldr + cc);
    s.x = r.x + s.x; s.y = r.y + s.y; s.z = r.z + s.z; s.w = r.w + s.w;
  }
  *out = s;
}

}  // namespace

// K pieces of a launch: a piece is one round of a CU, so the launch costs
// (rounds of 256 workgroups) x (K steps of a piece + about 5 steps to fill and
// drain the tile), and a split adds the slices' traffic.
KPieces train_gemm3_pieces(int64_t M, int64_t mtiles_x_ntiles, int64_t ncols, int64_t nchunks,
                           int64_t slice_floats) {
  KPieces best{1, nchunks};
  double best_t = -1.0;
  for (int64_t ns = 1; ns <= 8; ++ns) {
    const int64_t cp = (nchunks + ns - 1) / ns;
    if (ns > 1 && (cp < 8 || cp * (ns - 1) >= nchunks || (ns - 1) * M * ncols > slice_floats)) break;
    const double rounds = (double)((mtiles_x_ntiles * ns + 255) / 256);
    // a step takes about 0.9 us; slices are written and read at about 4 TB/s
    double t = rounds * (double)(cp + 5) * 0.9;
    if (ns > 1) t += 4.0 + 2.0 * ns * (double)M * (double)ncols * 4.0 / 4.0e6;
    if (best_t < 0 || t < best_t) {
      best_t = t;
      best = {(int32_t)ns, cp};
    }
  }
  return best;
}

void train_gemm3_plan(TGemm3Args& a, int64_t slice_floats) {
  a.mtiles = (int32_t)((a.M + G3_BM - 1) / G3_BM);
  a.ntn = 0;
  a.ncols = 0;
  a.nchunks = 0;
  for (int s = 0; s < a.nseg; ++s) {
    TSeg& g = a.seg[s];
    g.ntn = (g.N + G3_BN - 1) / G3_BN;
    g.chunks = (g.K + G3_BK - 1) / G3_BK;
    g.col0 = a.ncols;
    if (!a.ksegs || s == 0) {
      a.ntn += g.ntn;
      a.ncols += g.N;
    }
    a.nchunks = a.ksegs ? a.nchunks + g.chunks : g.chunks;
  }
  const KPieces kp = train_gemm3_pieces(a.M, (int64_t)a.mtiles * a.ntn, a.ncols, a.nchunks,
                                        slice_floats);
  a.ksplit = kp.ns;
  a.cpiece = (int32_t)kp.chunks;
  a.ntiles = a.mtiles * a.ntn * a.ksplit;
}

hipError_t launch_train_gemm3(const TGemm3Args& a, int32_t bl, hipStream_t st) {
  if (a.M <= 0 || a.ntiles <= 0) return hipSuccess;
  if (a.ksplit > 1 && !a.part) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((a.ntiles + 7) / 8 * 8);
  if (bl == 0) {
    if (a.ascale) train_gemm3_kernel<0, true, false><<<grid, G3_NT, 0, st>>>(a);
    else if (a.neg0) return hipErrorInvalidValue;
    else train_gemm3_kernel<0, false, false><<<grid, G3_NT, 0, st>>>(a);
  } else {
    if (a.ascale) return hipErrorInvalidValue;
    if (a.neg0) train_gemm3_kernel<1, false, true><<<grid, G3_NT, 0, st>>>(a);
    else train_gemm3_kernel<1, false, false><<<grid, G3_NT, 0, st>>>(a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.ksplit <= 1) return e;
  const int64_t n = a.M * (a.ncols / 4);
  train_reduce3_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace svl
