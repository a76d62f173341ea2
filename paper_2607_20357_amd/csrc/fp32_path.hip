// Float32 kernels of the masked GEMM and of the causal attention (the
// SVL_F32 path: small decoders checked at float32 accuracy).  Same plan
// descriptors and semantics as the 16-bit kernels, on float32 MFMA.
//
// These launches are short (a few hundred rows and columns), so latency bounds
// them, not the float32 rate: the GEMM takes small tiles, splits K over the
// waves of a workgroup and loads fragments straight into registers; there is
// no barrier before the last one.  Two-layer 256-wide decoder, 48 rows, per
// launch (64 x 64 tiles of vector FMAs, K walked 16 columns per barrier pair,
// before): QKV 30 -> 8.8 us, output 25 -> 7, gate/up 30 -> 8.8, down 60 -> 12;
// attention (one query per thread of one wave before) 56 -> 10.  At 1024 rows of a
// 2048-wide layer the kernels take 3.3 instead of 8.0 ms.
#include "svl_internal.h"
#include "device_util.h"

namespace svl {
namespace {

constexpr int BM = F32_BM, BN = F32_BN;
static_assert(BM == 32 && BN == 32 && F32_SWIGLU_CH == 16, "2 x 2 MFMA blocks per tile");
constexpr int KW = 4;   // waves of a workgroup, each a quarter of the K chunks

// Tile of 32 rows x 32 weight rows (gate/up: 16 channels' gate and up rows) by
// v_mfma_f32_16x16x4_f32.  Wave w multiplies chunks w, w + 4, ... of the group;
// lane (r, q) loads 4 consecutive k of its row, k = 16 s + 4 q + [0, 4), so
// four MFMAs consume a 16-byte load of either operand (both in the same order
// of k).  The four waves' sums are added in wave order through LDS.
template <int EPI>
__global__ __launch_bounds__(64 * KW) void gemm_f32_kernel(GemmArgs a) {
  __shared__ float red[KW][16][64];
  const int t = xcd_tile_index();
  if (t >= a.ntiles) return;
  const GemmGroup g = a.groups[find_group(a.groups, a.ngroups, t)];
  constexpr int BNO = (EPI == EPI_SWIGLU) ? F32_SWIGLU_CH : BN;
  const int local = t - g.tile0;
  const int nm = (g.nrows + BM - 1) / BM;
  const int mt = local % nm, nt = local / nm;
  const int arow0 = g.arow0 + mt * BM, orow0 = g.orow0 + mt * BM;
  const int mcnt = min(BM, g.nrows - mt * BM);
  const int n0 = g.n0 + nt * BNO;
  const int ncnt = min(BNO, g.n1 - n0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int fr = lane & 15, fq = lane >> 4;
  const float* A = static_cast<const float*>(a.A);

  // Weight row of tile row c (nullptr: outside the tile).
  auto wrow = [&](int c) -> const float* {
    if constexpr (EPI == EPI_SWIGLU) {
      const int ch = c & 15;
      if (ch >= ncnt) return nullptr;
      return static_cast<const float*>(c < 16 ? a.W0 : a.W1) + (size_t)(n0 + ch) * a.ldw;
    } else {
      if (c >= ncnt) return nullptr;
      const int col = n0 + c;
      if constexpr (EPI == EPI_STORE) {
        if (n0 < a.nb1) return static_cast<const float*>(a.W0) + (size_t)col * a.ldw;
        if (n0 < a.nb2) return static_cast<const float*>(a.W1) + (size_t)(col - a.nb1) * a.ldw;
        return static_cast<const float*>(a.W2) + (size_t)(col - a.nb2) * a.ldw;
      } else {
        return static_cast<const float*>(a.W0) + (size_t)col * a.ldw;
      }
    }
  };
  const float* src[4];   // A rows of the two row blocks, weight rows of the two column blocks
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    src[i] = 16 * i + fr < mcnt ? A + (size_t)(arow0 + 16 * i + fr) * a.lda : nullptr;
    src[2 + i] = wrow(16 * i + fr);
  }
  // 16-byte loads need both row strides (and a chunk's start) in whole float4s
  const bool vec = (a.lda & 3) == 0 && (a.ldw & 3) == 0;

  float4 v[2][4][4];   // [chunk parity][16-column step][operand]
  auto load = [&](int kc, float4 (&x)[4][4]) __attribute__((always_inline)) {
    const KChunk ch = a.chunks[g.kc_off + kc];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 16 * s + 4 * fq;
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        x[s][o] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!src[o] || k >= ch.len) continue;
        const float* p = src[o] + ch.k0 + k;
        if (vec && (ch.k0 & 3) == 0 && k + 4 <= ch.len) {
          x[s][o] = *reinterpret_cast<const float4*>(p);
        } else {
          x[s][o].x = p[0];
          if (k + 1 < ch.len) x[s][o].y = p[1];
          if (k + 2 < ch.len) x[s][o].z = p[2];
          if (k + 3 < ch.len) x[s][o].w = p[3];
        }
      }
    }
  };
  floatx4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto mul = [&](const float4 (&x)[4][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        auto at = [&](int o) {
          return e == 0 ? x[s][o].x : e == 1 ? x[s][o].y : e == 2 ? x[s][o].z : x[s][o].w;
        };
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(at(i), at(2 + j), acc[i][j], 0, 0, 0);
      }
  };
  // the wave's next chunk is in flight while one multiplies
  int kc = wave;
  if (kc < g.kc_cnt) load(kc, v[0]);
  while (kc < g.kc_cnt) {
    if (kc + KW < g.kc_cnt) load(kc + KW, v[1]);
    mul(v[0]);
    kc += KW;
    if (kc >= g.kc_cnt) break;
    if (kc + KW < g.kc_cnt) load(kc + KW, v[0]);
    mul(v[1]);
    kc += KW;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][8 * i + 4 * j + r][lane] = acc[i][j][r];
  __syncthreads();
  auto sum = [&](int q) { return ((red[0][q][lane] + red[1][q][lane]) + red[2][q][lane]) + red[3][q][lane]; };
  // acc[i][j][r] is C[16 i + 4 (lane / 16) + r][16 j + lane % 16]; wave w finishes
  // block (w / 2, w % 2), gate/up: rows of block w (waves 0 and 1)
  if constexpr (EPI == EPI_SWIGLU) {
    if (wave >= 2 || fr >= ncnt) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * wave + 4 * fq + r;
      if (row >= mcnt) continue;
      const float gt = sum(8 * wave + r), up = sum(8 * wave + 4 + r);
      static_cast<float*>(a.out)[(size_t)(orow0 + row) * a.ldo + n0 + fr] =
          gt / (1.0f + expf(-gt)) * up;
    }
  } else {
    const int i = wave >> 1, j = wave & 1, col = 16 * j + fr;
    if (col >= ncnt) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * i + 4 * fq + r;
      if (row >= mcnt) continue;
      float* o = static_cast<float*>(a.out) + (size_t)(orow0 + row) * a.ldo + n0 + col;
      const float s = sum(4 * wave + r);
      *o = EPI == EPI_STORE ? s : *o + s;
    }
  }
}

// One workgroup: 64 query rows of one active head of one sample, four waves of
// 16 queries each on v_mfma_f32_16x16x4_f32, 64 keys at a time through LDS
// with an online softmax; RoPE is applied to Q and K rows while they load.
// Lane l holds rows 4 (l / 16) + r, r < 4, of every 16 x 16 block, so a
// row's statistics stay in the 16 lanes that share l / 16.
template <int D>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a) {
  constexpr int BQ = ATTN_BQ, BKV = 64, NBO = D / 16, H = D / 2, H4 = H / 4;
  static_assert(BQ == 64, "four waves of 16 queries");
  __shared__ __attribute__((aligned(16))) union {
    float xt[D][68];       // Q^T (read once into registers), then K^T of a key tile
    float pt[BKV][68];     // P^T once every wave has its scores
  } u;
  __shared__ __attribute__((aligned(16))) float vs[BKV][D + 4];
  const int t = blockIdx.x;
  if (t >= a.ntiles) return;
  const AttnGroup g = a.groups[find_group(a.groups, a.ngroups, t)];
  const int local = t - g.tile0;
  const int hs = local % g.h_cnt;
  const int qt = g.nqt - 1 - local / g.h_cnt;
  const int h = a.head_table[g.h_off + hs];
  const int kvh = h / (a.n_heads / a.n_kv_heads);
  const int S = g.S, q0 = qt * BQ, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4, qw = 16 * wave;
  const float* base = static_cast<const float*>(a.qkv) + (size_t)g.row0 * a.ldq;
  const int kcol = (a.n_heads + kvh) * D, vcol = (a.n_heads + a.n_kv_heads + kvh) * D;

  // rows [row0, row0 + 64) of a head's columns, rotated, scaled and transposed
  // into u.xt (rows past S read 0)
  auto load_rotated = [&](int row0, int col, float scale) {
    for (int idx = tid; idx < 64 * H4; idx += 256) {
      const int r = idx / H4, c = (idx % H4) * 4, row = row0 + r;
      float4 x1 = make_float4(0.f, 0.f, 0.f, 0.f), x2 = x1, w0 = x1, w1 = x1;
      if (row < S) {
        const float* p = base + (size_t)row * a.ldq + col + c;
        const float4* w = reinterpret_cast<const float4*>(a.rope + (size_t)row * H + c);
        x1 = *reinterpret_cast<const float4*>(p);
        x2 = *reinterpret_cast<const float4*>(p + H);
        w0 = w[0];
        w1 = w[1];
      }
      u.xt[c + 0][r] = (x1.x * w0.x - x2.x * w0.y) * scale;
      u.xt[c + 1][r] = (x1.y * w0.z - x2.y * w0.w) * scale;
      u.xt[c + 2][r] = (x1.z * w1.x - x2.z * w1.y) * scale;
      u.xt[c + 3][r] = (x1.w * w1.z - x2.w * w1.w) * scale;
      u.xt[H + c + 0][r] = (x2.x * w0.x + x1.x * w0.y) * scale;
      u.xt[H + c + 1][r] = (x2.y * w0.z + x1.y * w0.w) * scale;
      u.xt[H + c + 2][r] = (x2.z * w1.x + x1.z * w1.y) * scale;
      u.xt[H + c + 3][r] = (x2.w * w1.z + x1.w * w1.w) * scale;
    }
  };
  load_rotated(q0, h * D, a.scale);
  __syncthreads();
  float qf[D / 4];   // the wave's query fragments
#pragma unroll
  for (int i = 0; i < D / 4; ++i) qf[i] = u.xt[4 * i + lg][qw + lr];
  float mrow[4], lrow[4];
  floatx4 o[NBO];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    mrow[r] = -1.0e30f;
    lrow[r] = 0.f;
  }
#pragma unroll
  for (int n = 0; n < NBO; ++n) o[n] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int kv_end = min(S, q0 + BQ);
  for (int kv0 = 0; kv0 < kv_end; kv0 += BKV) {
    __syncthreads();   // the previous tile's (and the query fragments') readers are done
    load_rotated(kv0, kcol, 1.0f);
    for (int idx = tid; idx < 64 * (D / 4); idx += 256) {
      const int r = idx / (D / 4), c = (idx % (D / 4)) * 4;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (kv0 + r < S) v = *reinterpret_cast<const float4*>(base + (size_t)(kv0 + r) * a.ldq + vcol + c);
      *reinterpret_cast<float4*>(&vs[r][c]) = v;
    }
    __syncthreads();
    floatx4 sc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) sc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < D; d += 4)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        sc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[d / 4], u.xt[d + lg][16 * j + lr], sc[j], 0, 0, 0);
    float corr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qi = q0 + qw + 4 * lg + r;
      float mx = -1.0e30f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kv = kv0 + 16 * j + lr;
        sc[j][r] = kv <= qi && kv < S ? sc[j][r] : -1.0e30f;
        mx = fmaxf(mx, sc[j][r]);
      }
#pragma unroll
      for (int o2 = 1; o2 < 16; o2 <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o2, 64));
      const float mn = fmaxf(mrow[r], mx);
      corr[r] = expf(mrow[r] - mn);
      float rs = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kv = kv0 + 16 * j + lr;
        const float p = kv <= qi && kv < S ? expf(sc[j][r] - mn) : 0.f;
        sc[j][r] = p;
        rs += p;
      }
#pragma unroll
      for (int o2 = 1; o2 < 16; o2 <<= 1) rs += __shfl_xor(rs, o2, 64);
      lrow[r] = lrow[r] * corr[r] + rs;
      mrow[r] = mn;
    }
    __syncthreads();   // every wave has read K^T: P^T goes in its place
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<float4*>(&u.pt[16 * j + lr][qw + 4 * lg]) =
          make_float4(sc[j][0], sc[j][1], sc[j][2], sc[j][3]);
#pragma unroll
    for (int n = 0; n < NBO; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[n][r] *= corr[r];
    wave_lds_handoff();   // a wave reads only the P^T columns that its own lanes wrote
    // O += P V
#pragma unroll 4
    for (int k = 0; k < BKV; k += 4) {
      const float pa = u.pt[k + lg][qw + lr];
#pragma unroll
      for (int n = 0; n < NBO; ++n)
        o[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa, vs[k + lg][16 * n + lr], o[n], 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int qi = q0 + qw + 4 * lg + r;
    if (qi >= S) continue;
    const float inv = 1.0f / lrow[r];
    float* orow = static_cast<float*>(a.out) + (size_t)(g.row0 + qi) * a.ldo + h * D + lr;
#pragma unroll
    for (int n = 0; n < NBO; ++n) orow[16 * n] = o[n][r] * inv;
  }
}

}  // namespace

hipError_t launch_gemm_f32(const GemmArgs& a, int32_t epi, hipStream_t st) {
  if (a.ntiles <= 0) return hipSuccess;
  const unsigned grid = (unsigned)((a.ntiles + 7) / 8 * 8);
  switch (epi) {
    case EPI_STORE: gemm_f32_kernel<EPI_STORE><<<grid, 64 * KW, 0, st>>>(a); break;
    case EPI_RESID: gemm_f32_kernel<EPI_RESID><<<grid, 64 * KW, 0, st>>>(a); break;
    default: gemm_f32_kernel<EPI_SWIGLU><<<grid, 64 * KW, 0, st>>>(a); break;
  }
  return hipGetLastError();
}

hipError_t launch_attn_f32(const AttnArgs& a, int32_t head_dim, hipStream_t st) {
  if (a.ntiles <= 0) return hipSuccess;
  switch (head_dim) {
    case 32: attn_f32_kernel<32><<<a.ntiles, 256, 0, st>>>(a); break;
    case 64: attn_f32_kernel<64><<<a.ntiles, 256, 0, st>>>(a); break;
    case 128: attn_f32_kernel<128><<<a.ntiles, 256, 0, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace svl
