// Masked grouped GEMM of the bf16 activation mode's QKV and gate/up products:
//
//   C[rows, cols] = sum over the tile's K chunks of (A + A2)[rows, k] * W[cols, k]
//
// A and A2 are the high and low bf16 parts of the normed rows, both in the
// fragment-packed layout (plan_types.h), W a bf16 weight matrix in [out][in]
// layout; v_mfma_f32_16x16x32_bf16, float32 accumulation, the low part's
// product right after the high part's against the same weight fragments.
// Tiles, K chunk lists and outputs are those of the other 16-bit GEMMs (one
// tile record per workgroup: up to 256 rows times up to NB 16-column blocks
// times a range of K chunks of 64).
//
// Workgroup: 512 threads.  Waves 0-3 multiply, waves 4-7 bring the weights,
// one of each on every SIMD.  Vector loads complete in order, so a wave that
// loads both operands waits for its HBM weight loads (2-3 us under load)
// whenever it waits for an activation fragment that L2 had ready; apart, the
// weights run three stages ahead and the activations as far as registers
// allow.  Four multiplying waves instead of eight halve the LDS reads per
// MFMA (a weight fragment feeds up to 4 row blocks, twice), which with two
// MFMAs per fragment pair leaves the matrix pipes as the larger part of a
// stage.
//
// Against eight waves that each load and multiply (a LLaVA-7B prefill of 350
// rows, 3 of 4 groups on): eight layers 2.65 -> 2.23 ms.  Launches where that
// form is the faster one keep it (waves_apart, plan_types.h).  The single-term
// products (fp16) have half the MFMAs per byte loaded and measured 5% slower in
// this form, so they keep theirs.
#include <type_traits>
#include <utility>

#include "svl_internal.h"
#include "device_util.h"

namespace svl {
namespace {

constexpr int BM = MFMA_BM;
constexpr int KS = 4;                          // K chunks per weight stage (one barrier each)
constexpr int LDS_STRIDE = KS * MFMA_BK;       // 16-bit elements per LDS row (512 B, 32 units)
constexpr int MAX_CHUNKS = 1024;               // K chunks per tile (K <= 65536)

template <int P>
using Phase = std::integral_constant<int, P>;

template <int EPI, int NB>
__global__ __launch_bounds__(512) void gemm_lo_kernel(MmArgs a) {
  constexpr int NT = 512;
  constexpr int CW = 4;                         // multiplying waves
  // 16-row blocks per multiplying wave; tiles of 8 blocks come with up to 12 row
  // blocks in all (a fourth per wave would spill registers)
  constexpr int RB = NB == 8 ? 3 : BM / (16 * CW);
  static_assert(NB != 8 || !(waves_apart(8, 13) || waves_apart(8, 14) || waves_apart(8, 15) ||
                             waves_apart(8, 16)), "the planner's rule");
  constexpr int LT = 256;                       // threads that bring the weights
  constexpr int BN = NB * 16;                   // weight rows per tile
  // weight register stages in flight (8 NB registers each)
  constexpr int NWS = NB <= 6 ? 3 : 2;
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2 * BN * LDS_STRIDE];
  // the tile's chunk offsets (no vmcnt waits), the last repeated up to a whole stage
  __shared__ __attribute__((aligned(16))) int32_t s_k0[MAX_CHUNKS + KS];

  const int t = xcd_tile_index();
  if (t >= a.ntiles) return;
  const MmTile tl = a.tiles[t];
  const int mcnt = tl.mcnt;
  const int nblk = tl.nblk;
  const int nk = tl.kcn;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // a wave's role is uniform
  const int nkp = nk > 0 ? nk + KS : 0;
  for (int c = tid; c < nkp; c += NT) {
    const int r = min(c, nk - 1);
    s_k0[c] = tl.kdense >= 0 ? tl.kdense + MFMA_BK * r : a.chunks[tl.chunk0 + r].k0;
  }
  const int d = a.head_dim, hb = d >> 4;        // QKV: blocks per head
  __syncthreads();   // s_k0 ready

  const int last = nk - 1;
  const int nst = (nk + KS - 1) / KS;

  // ---- weights.  One stage = KS chunks: piece p = lt + LT*s (s < WLD) is
  // unit p % 32 (chunk u / 8 of the stage, 16-byte segment u % 8) of tile row
  // p / 32 (block j = row/16, column i = row%16 of the block).  Half a wave
  // loads 512 bytes of one weight row; piece s holds column half s % 2 of
  // block s / 2 (i < 8 or i >= 8), so gate and up pieces alternate.
  constexpr int RU = KS * 8;                    // 16-byte units per stage row
  constexpr int WLD = BN * RU / LT;             // BN * RU pieces / LT threads
  static_assert(KS == 4 && WLD == 2 * NB, "8 rows of 32 units per piece");
  const int lt = tid - 64 * CW;                 // loading thread
  const int wu = lt & (RU - 1), wqc = wu >> 3;  // its unit and chunk of the stage
  __amdgpu_buffer_rsrc_t rsB[2];
  uint32_t voB[WLD];
  auto setupW = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int m = EPI == EPI_QKV ? tl.wsel : h;   // gate, then up rows
      const void* base = m == 0 ? a.W[0] : (m == 1 ? a.W[1] : a.W[2]);
      const int rows = m == 0 ? a.w_rows[0] : (m == 1 ? a.w_rows[1] : a.w_rows[2]);
      rsB[h] = make_rsrc(base, (uint32_t)rows * (uint32_t)a.ldw * 2u);
    }
#pragma unroll
    for (int s = 0; s < WLD; ++s) {
      const int j = s >> 1, i = lt / RU + 8 * (s & 1);
      const int gb = tl.b0 + j;
      int row;
      if constexpr (EPI == EPI_QKV)
        row = tl.wrow0 + (gb / hb) * d + (gb % hb) * 8 + (i & 7) + ((i >> 3) ? (d >> 1) : 0);
      else
        row = tl.wrow0 + gb * 8 + (i & 7);
      // pieces past the tile's blocks read out of range (zero, no traffic); the
      // chunk offset added later (< 2^17) keeps 2^31 out of range without
      // wrapping (a weight matrix spans less than 2^31 bytes)
      voB[s] = j < nblk ? (uint32_t)row * a.ldw * 2u + (wu & 7) * 16u : 0x80000000u;
    }
  };
  // weight stage S: chunks S*KS .. S*KS + KS-1 (a chunk past the last of the
  // last stage: the last again; a stage past the last: out of range); the
  // chunk offset varies across the half wave, so it goes in the lane offset
  auto loadW = [&](int S, uint4 (&rb)[WLD]) __attribute__((always_inline)) {
    const bool past = S >= nst;
    const uint32_t ko = (uint32_t)s_k0[min(S * KS + wqc, last)] * 2u;
#pragma unroll
    for (int s = 0; s < WLD; ++s)
      rb[s] = load16w(rsB[s & 1], past ? 0x80000000u : voB[s] + ko, 0);
  };
  auto wstore = [&](int buf, const uint4 (&rb)[WLD]) __attribute__((always_inline)) {
    uint16_t* B = Bs + buf * (BN * LDS_STRIDE);
#pragma unroll
    for (int s = 0; s < WLD; ++s) {
      const int tr = (lt + LT * s) / RU;
      *reinterpret_cast<uint4*>(&B[tr * LDS_STRIDE + (wu ^ swz(tr)) * 8]) = rb[s];
    }
  };

  // ---- activations: packed blocks of this tile's rows.  Multiplying wave w
  // owns 16-row blocks w, w + 4, w + 8, w + 12 (a ragged tile's blocks spread
  // evenly over the SIMDs).
  auto rowblock = [&](int i) __attribute__((always_inline)) { return wave + CW * i; };
  const uint32_t kblocks = (uint32_t)(a.lda / 64);
  const uint32_t blk_bytes = kblocks * 2048u;   // one 16-row block over all of K
  const int rb0 = (tl.arow) / 16;
  const __amdgpu_buffer_rsrc_t rsA =
      make_rsrc(static_cast<const uint16_t*>(a.A) + (size_t)rb0 * kblocks * 1024,
                (uint32_t)((mcnt + 15) / 16) * blk_bytes);
  const __amdgpu_buffer_rsrc_t rsA2 =
      make_rsrc(static_cast<const uint16_t*>(a.A2) + (size_t)rb0 * kblocks * 1024,
                (uint32_t)((mcnt + 15) / 16) * blk_bytes);
  floatx4 acc[RB][NB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Inside a chunk, lane group q = lane / 16 holds k 16q + [0, 8) in the
  // first MFMA k-step and 16q + [8, 16) in the second, for both operands.
  // fragment unit of lane group g in chunk q, k-step ks: q*8 + 2g + ks; the
  // swizzle of rows j*16 + lane%16 depends on lane%16 only
  const int fl = (2 * (lane >> 4)) ^ swz(lane & 15);
  const uint16_t* Bl = Bs + (lane & 15) * LDS_STRIDE;

  // The multiplying waves' pipeline, instantiated for the row blocks a wave
  // has in the tile (no loads or MFMAs past it, straight-line code, so the
  // waits stay exact).  A k-step (half a chunk) is a register slot; NSK of
  // them are in flight, as many as fit beside the accumulators.  The weight
  // fragments of the next step (a k-step, or half its blocks in the widest
  // tiles) are read from LDS before the MFMAs of the current one; scheduling
  // barriers keep that order (left alone, the compiler reads a fragment right
  // before its use and sinks the A loads to the end of the stage).  The
  // stage's barrier stands before its last step's MFMAs, whose fragments are
  // in registers by then.
  auto multiply = [&](auto nrb) __attribute__((always_inline)) {
    constexpr int NRB = decltype(nrb)::value;
    constexpr int AF = 2;                       // fragments per row block and k-step: high, low
    constexpr int NG = NB == 8 ? 4 : 1;         // weight fragment groups per k-step
    constexpr int GB = NB / NG;
    // registers for the accumulators, two fragment groups and the A slots (more
    // spill at 8 blocks)
    constexpr int FREE = (NB == 8 ? 204 : 212) - 4 * NB * NRB - 8 * GB;
    constexpr int SLOT = 4 * (NRB > 0 ? NRB : 1) * AF;
    constexpr int NSK = FREE >= 8 * SLOT   ? 8
                        : FREE >= 6 * SLOT ? 6
                        : FREE >= 4 * SLOT ? 4
                        : FREE >= 3 * SLOT ? 3
                                           : 2;
    constexpr int NP = NSK == 6 || NSK == 3 ? 3 : 1;   // stages per round of slots
    constexpr int KQ = 2 * KS;                  // k-steps per stage
    uint4 sa[NSK][RB][AF], bfr[2][GB];
    uint32_t voA[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) voA[i] = (uint32_t)rowblock(i) * blk_bytes + lane * 16u;
    // chunk byte offsets (into A) of this stage and the next, in scalar registers
    uint32_t ko[2 * KS];
    auto offsets = [&](int S, uint32_t* o) __attribute__((always_inline)) {
      const int4 k4 = *reinterpret_cast<const int4*>(&s_k0[min(S, nst - 1) * KS]);
      o[0] = (uint32_t)__builtin_amdgcn_readfirstlane(k4.x) * 32u;
      o[1] = (uint32_t)__builtin_amdgcn_readfirstlane(k4.y) * 32u;
      o[2] = (uint32_t)__builtin_amdgcn_readfirstlane(k4.z) * 32u;
      o[3] = (uint32_t)__builtin_amdgcn_readfirstlane(k4.w) * 32u;
    };
    auto loadA = [&](uint32_t soA, int ks, uint4 (&ra)[RB][AF]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NRB; ++i) {
        ra[i][0] = load16(rsA, voA[i] + 1024u * ks, soA);
        ra[i][1] = load16(rsA2, voA[i] + 1024u * ks, soA);
      }
    };
    // weight fragments of k-step ks2 of a stage, group g.  Blocks past the
    // tile's nblk hold zero weights (their loads read out of range), so they
    // are multiplied unconditionally.
    auto readB = [&](int buf, int ks2, int g, uint4 (&o)[GB]) __attribute__((always_inline)) {
      const uint16_t* B = Bl + buf * (BN * LDS_STRIDE);
      const int u = (((ks2 >> 1) * 8 + (ks2 & 1)) ^ fl) * 8;
      if constexpr (NRB > 0)
#pragma unroll
        for (int j = 0; j < GB; ++j)
          o[j] = *reinterpret_cast<const uint4*>(&B[(g * GB + j) * 16 * LDS_STRIDE + u]);
    };
    auto compute = [&](int g, const uint4 (&ra)[RB][AF], const uint4 (&bf)[GB]) __attribute__((always_inline)) {
#pragma unroll
      for (int f = 0; f < AF; ++f)   // the high parts, then the low parts
#pragma unroll
        for (int i = 0; i < NRB; ++i)
#pragma unroll
          for (int j = 0; j < GB; ++j)
            acc[i][g * GB + j] = mfma16x16x32<false>(ra[i][f], bf[j], acc[i][g * GB + j]);
    };
    offsets(0, ko);
    offsets(1, ko + KS);
    [&]<int... Q>(std::integer_sequence<int, Q...>) __attribute__((always_inline)) {
      (loadA(ko[Q / 2], Q % 2, sa[Q]), ...);
    }(std::make_integer_sequence<int, NSK>{});
    __syncthreads();
    readB(0, 0, 0, bfr[0]);
    // step u = NG * k-step + g of a stage
    auto step = [&](int S, auto ph, auto qq, auto full) __attribute__((always_inline)) {
      constexpr int P = decltype(ph)::value, Q = decltype(qq)::value / NG, g = decltype(qq)::value % NG;
      constexpr bool FULL = decltype(full)::value;
      constexpr int slot = (P * KQ + Q) % NSK, cur = (Q * NG + g) & 1;
      if constexpr (Q == KQ - 1 && g == NG - 1) {
        if (FULL || S + 1 < nst) {
          __syncthreads();
          readB((S + 1) & 1, 0, 0, bfr[cur ^ 1]);
        }
      } else {
        readB(S & 1, g == NG - 1 ? Q + 1 : Q, g == NG - 1 ? 0 : g + 1, bfr[cur ^ 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (FULL || S * KS + Q / 2 < nk) {
        compute(g, sa[slot], bfr[cur]);
        if constexpr (g == NG - 1) loadA(ko[(Q + NSK) / 2], (Q + NSK) % 2, sa[slot]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto stage = [&](int S, auto ph, auto full) __attribute__((always_inline)) {
      [&]<int... Q>(std::integer_sequence<int, Q...>) __attribute__((always_inline)) {
        (step(S, ph, std::integral_constant<int, Q>{}, full), ...);
      }(std::make_integer_sequence<int, KQ * NG>{});
#pragma unroll
      for (int c = 0; c < KS; ++c) ko[c] = ko[c + KS];
      offsets(S + 2, ko + KS);
    };
    const int nmain = min(nk / KS, nst - 1);   // full stages with a successor
    int S = 0;
    for (; S + NP <= nmain; S += NP)
      [&]<int... P>(std::integer_sequence<int, P...>) __attribute__((always_inline)) {
        (stage(S + P, Phase<P>{}, std::true_type{}), ...);
      }(std::make_integer_sequence<int, NP>{});
    // at most NP + 1 stages remain
    [&]<int... P>(std::integer_sequence<int, P...>) __attribute__((always_inline)) {
      ((S + P < nst ? stage(S + P, Phase<P % NP>{}, std::false_type{}) : void()), ...);
    }(std::make_integer_sequence<int, NP + 1>{});
  };

  // The loading waves: stage S + 1 goes from registers into the LDS buffer
  // that the multiplying waves left at the last barrier, its registers are
  // refilled with stage S + 1 + NWS, one barrier per stage.  (nst barriers,
  // as in the pipeline above.)
  auto bring = [&]() __attribute__((always_inline)) {
    uint4 sw[NWS][WLD];
    setupW();
    loadW(0, sw[0]);
#pragma unroll
    for (int s = 1; s < NWS; ++s) loadW(s, sw[s]);
    wstore(0, sw[0]);
    loadW(NWS, sw[0]);
    __syncthreads();
    int S = 0;
    for (; S + NWS < nst; S += NWS)
      [&]<int... P>(std::integer_sequence<int, P...>) __attribute__((always_inline)) {
        ((wstore((S + P + 1) & 1, sw[(P + 1) % NWS]), loadW(S + P + 1 + NWS, sw[(P + 1) % NWS]),
          __syncthreads()),
         ...);
      }(std::make_integer_sequence<int, NWS>{});
    [&]<int... P>(std::integer_sequence<int, P...>) __attribute__((always_inline)) {
      ((S + P + 1 < nst ? (wstore((S + P + 1) & 1, sw[(P + 1) % NWS]), __syncthreads()) : void()),
       ...);
    }(std::make_integer_sequence<int, NWS>{});
  };

  // Every wave runs the same number of barriers, whatever its part and its
  // row blocks.
  if (nk > 0) {
    const int nrb = ((mcnt + 15) / 16 - wave + CW - 1) / CW;   // row blocks w, w + 4, .. in the tile
    if (wave >= CW) bring();
    else if (nrb >= 4 && RB >= 4) multiply(std::integral_constant<int, RB>{});
    else if (nrb >= 3) multiply(std::integral_constant<int, 3>{});
    else if (nrb == 2) multiply(std::integral_constant<int, 2>{});
    else if (nrb == 1) multiply(std::integral_constant<int, 1>{});
    else multiply(std::integral_constant<int, 0>{});
  }

  // Epilogue.  acc[i][j][r] of a multiplying wave is C[trow(i, r)][16 j +
  // lane%16] of the tile; tile row m is row m0 + m of the group.
  const bool mul = wave < CW;
  auto trow = [&](int i, int r) __attribute__((always_inline)) {
    return 16 * rowblock(i) + (lane >> 4) * 4 + r;
  };
  const int ci = lane & 15;           // column inside the block
  if (a.split > 1) {
    // split-K piece: raw float32 accumulators at the output column (QKV) or
    // at the gate / up column (SWIGLU); the finish kernel does the rest
    if (!mul) return;
    float* out = a.partial + (size_t)tl.slice * a.pslice;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = trow(i, r);
        float* orow = out + (size_t)(tl.orow + min(row, mcnt - 1)) * a.pld;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int gb = tl.b0 + j;
          int col;
          if constexpr (EPI == EPI_QKV)
            col = tl.ocol0 + (gb / hb) * d + (gb % hb) * 8 + (ci & 7) + ((ci >> 3) ? (d >> 1) : 0);
          else
            col = ((ci >> 3) ? (a.pld >> 1) : 0) + tl.ocol0 + gb * 8 + (ci & 7);
          if (j < nblk && row < mcnt) orow[col] = acc[i][j][r];
        }
      }
    return;
  }
  // 16-bit outputs go through a staging tile in the (now idle) weight
  // buffers, 256 rows x RW values: QKV, both halves of every block (16 NB
  // columns); SWIGLU, the 8 NB channels.  Each lane of the workgroup then
  // stores whole 16-byte pieces (8 consecutive columns of one row), instead
  // of one 2-byte value per row and block.
  // (SWIGLU rows are padded to an odd number of 16-byte pieces, so the
  // row-strided piece reads below hit distinct banks)
  constexpr int RW = EPI == EPI_QKV ? NB * 16 : (NB | 1) * 8;
  static_assert(BM * RW <= 2 * BN * LDS_STRIDE, "the staging tile fits the weight buffers");
  uint16_t* E = Bs;
  uint16_t* out = static_cast<uint16_t*>(a.out);
  if constexpr (EPI == EPI_QKV) {
    const int half = d >> 1;
    // table entries of a row block, read one block ahead of their use
    // (tiles of more than 5 blocks have no registers for that)
    constexpr int AHEAD = NB <= 5 ? 1 : 0;
    float2 cs[1 + AHEAD][4][NB];
    auto load_cs = [&](int i, float2 (&o)[4][NB]) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = min(trow(i, r), mcnt - 1);
        const int pos = tl.pos0 >= 0 ? tl.pos0 + rr : a.rowpos[tl.arow + rr];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int gb = tl.b0 + min(j, nblk - 1);
          o[r][j] = a.rope[(size_t)pos * half + (gb % hb) * 8 + (ci & 7)];
        }
      }
    };
    if (mul && tl.rope && AHEAD) load_cs(0, cs[0]);
    __syncthreads();   // every wave is done with the weight buffers
    if (mul) {
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        if (tl.rope && i + AHEAD < RB) load_cs(i + AHEAD, cs[(i + AHEAD) & AHEAD]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            float v = acc[i][j][r];
            const float pv = __shfl_xor(v, 8, 64);
            if (tl.rope) {
              // (x1, x2) -> (x1 cos - x2 sin, x2 cos + x1 sin); lanes ci < 8 hold x1
              const float2 c2 = cs[i & AHEAD][r][j];
              v = v * c2.x + ((ci < 8) ? -pv : pv) * c2.y;
            }
            E[trow(i, r) * RW + j * 16 + ci] = f32_to_act_bits<false>(v);
          }
      }
    }
    __syncthreads();
    // piece q: tile row q / (2 NB), block (q / 2) % NB, half q % 2
    for (int q = tid; q < mcnt * 2 * NB; q += NT) {
      const int row = q / (2 * NB), j = (q >> 1) % NB, h = q & 1;
      const uint4 v = *reinterpret_cast<const uint4*>(&E[q * 8]);
      const int gb = tl.b0 + j;
      const int col = tl.ocol0 + (gb / hb) * d + (gb % hb) * 8 + h * half;
      if (j < nblk) *reinterpret_cast<uint4*>(out + (size_t)(tl.orow + row) * a.ldo + col) = v;
    }
  } else {
    __syncthreads();   // every wave is done with the weight buffers
    if (mul) {
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const float gt = acc[i][j][r];
            const float up = __shfl_xor(gt, 8, 64);   // lanes ci < 8: gate, ci >= 8: up
            // silu(g) * u = g / (1 + exp(-g)) * u, reciprocal in hardware
            if (ci < 8)
              E[trow(i, r) * RW + j * 8 + ci] = f32_to_act_bits<false>(
                  gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up);
          }
    }
    __syncthreads();
    // piece q: tile row q % 256, block q / 256 (16 lanes store the 256
    // contiguous bytes of one 8-channel group of 16 packed rows)
#pragma unroll
    for (int it = 0; it < (BM * NB + NT - 1) / NT; ++it) {
      const int q = it * NT + tid;
      const int row = q % BM, j = q / BM;
      if (j < nblk && row < mcnt)
        *reinterpret_cast<uint4*>(out + packed_index((int64_t)tl.orow + row,
                                                     tl.ocol0 + (tl.b0 + j) * 8, a.ldo)) =
            *reinterpret_cast<const uint4*>(&E[row * RW + j * 8]);
    }
  }
}

template <int EPI, int NB>
hipError_t launch(const MmArgs& a, hipStream_t st) {
  const unsigned grid = (unsigned)((a.ntiles + 7) / 8 * 8);
  gemm_lo_kernel<EPI, NB><<<grid, 512, 0, st>>>(a);
  return hipGetLastError();
}

template <int EPI>
hipError_t by_nb(const MmArgs& a, int32_t nb, hipStream_t st) {
  switch (nb) {
    case 2: return launch<EPI, 2>(a, st);
    case 3: return launch<EPI, 3>(a, st);
    case 4: return launch<EPI, 4>(a, st);
    case 5: return launch<EPI, 5>(a, st);
    case 6: return launch<EPI, 6>(a, st);
    case 8: return launch<EPI, 8>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_gemm_lo(const MmArgs& a, int32_t epi, int32_t nb, hipStream_t st) {
  switch (epi) {
    case EPI_QKV: return by_nb<EPI_QKV>(a, nb, st);
    case EPI_SWIGLU: return by_nb<EPI_SWIGLU>(a, nb, st);
    default: return hipErrorInvalidValue;   // low parts come with the normed rows only
  }
}

}  // namespace svl
