// bf16 GEMM with fp32 accumulation on gfx950 MFMA, C = epilogue(A W^T).
//
// A [M][K] and W [N][K] are both K-contiguous (every projection of the block
// stores its weight [out][in]).  A 512-thread workgroup computes a 128 x 256
// or a 192 x 256 tile (the height picked per shape, see choose_bm); its eight
// waves own 64 x 64 or 96 x 64 pieces (2 x 4) as 4 x 4 or 6 x 4 blocks of
// v_mfma_f32_16x16x32_bf16.  K advances in steps of 64 through LDS stages
// (three for the 128-row tile, two for the 192-row one) filled by direct
// global->LDS loads (global_load_lds_dwordx4): the loads of a later step are
// in flight while step k is multiplied, and the loaded bytes never pass
// through registers.  The loads are issued from inline asm:
// the compiler's own form makes every later LDS read wait for all of them,
// which would leave no load in flight; the kernel waits on the vector-memory
// counter itself before the barrier that publishes a stage.  Each LDS row
// is 128 bytes with its eight 16-byte chunks XOR-swizzled by (row / 2) % 8,
// so the fragment reads of 16 consecutive rows spread over all banks.  The
// fragment reads run half a step ahead of the MFMAs: the second 32-wide half
// of step k is read under the first half's MFMAs and the first half of step
// k+1 under the second half's, so the LDS reads never stand alone between
// barriers (8% faster than reading a step's fragments up front).
//
// The MFMA computes C^T = W A^T: W rows feed the A operand and A rows the B
// operand, so each lane ends up owning one output row m and four
// consecutive columns n per block.  The epilogue applies bias / GELU /
// gate * y + residual in fp32, staging the tile through LDS so that the
// residual is read and C written one contiguous row at a time.
// Rows past M read a clamped row and store nothing; an N ending on a
// half tile (N % 256 == 128) clamps W rows the same way.
#include <type_traits>

#include "launch.h"

namespace ardit {

namespace {

constexpr int BN = 256, BK = 64, NT = 512;
constexpr int NWAVES = NT / 64;
constexpr int WN = 64, NB = WN / 16;
constexpr int NWN = BN / WN;
constexpr int ROW_BYTES = BK * 2;
constexpr int W_BYTES = BN * ROW_BYTES;
constexpr int W_INS = W_BYTES / 1024 / NWAVES;
constexpr int GROUP_M = 8;   // m-tiles per raster group (L2 reuse of W columns)
constexpr int CROW = BN * 4 + 16;   // epilogue: fp32 tile row in LDS, padded by 16 bytes

// Tile height BM: 128 rows with three LDS stages, or 192 rows with two (the
// waves then own 96 x 64 pieces, 6 x 4 blocks; fragment reads per MFMA fall
// by a sixth and the tile count suits other shapes).  The epilogue stages
// the fp32 tile in passes of PASS_ROWS rows that fit the stages' LDS.
template <int BM_>
struct Cfg {
  static constexpr int BM = BM_;
  static constexpr int STAGES = BM_ == 128 ? 3 : 2;
  static constexpr int WM = BM / 2, MB = WM / 16;
  static constexpr int A_BYTES = BM * ROW_BYTES;
  static constexpr int STAGE_BYTES = A_BYTES + W_BYTES;
  static constexpr int A_INS = A_BYTES / 1024 / NWAVES;   // 1 KB load instructions per wave per K step
  static constexpr int PASS_ROWS = BM * CROW <= STAGES * STAGE_BYTES ? BM : BM / 2;
  static constexpr int NPASS = BM / PASS_ROWS;
  static constexpr int RB = PASS_ROWS / (NWAVES * 2);     // rows per batch and wave, two batches a pass
  static_assert(A_INS * NWAVES * 1024 == A_BYTES && W_INS * NWAVES * 1024 == W_BYTES, "");
  static_assert(STAGES * STAGE_BYTES <= 160 * 1024, "LDS");
  static_assert(PASS_ROWS * CROW <= STAGES * STAGE_BYTES && PASS_ROWS % 16 == 0, "C tile in LDS");
  static_assert(RB * NWAVES * 2 == PASS_ROWS, "row batches");
};

__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

template <typename T>
__device__ __forceinline__ void load4(const T* p, float* f);
template <>
__device__ __forceinline__ void load4<bf16_t>(const bf16_t* p, float* f) {
  const uint2 r = *reinterpret_cast<const uint2*>(p);
  f[0] = __uint_as_float(r.x << 16);
  f[1] = __uint_as_float(r.x & 0xffff0000u);
  f[2] = __uint_as_float(r.y << 16);
  f[3] = __uint_as_float(r.y & 0xffff0000u);
}
template <>
__device__ __forceinline__ void load4<float>(const float* p, float* f) {
  const float4 r = *reinterpret_cast<const float4*>(p);
  f[0] = r.x;
  f[1] = r.y;
  f[2] = r.z;
  f[3] = r.w;
}

__device__ __forceinline__ void store4(bf16_t* p, const float* y) {
  uint2 out;
  out.x = pack_bf16x2(y[0], y[1]);
  out.y = pack_bf16x2(y[2], y[3]);
  *reinterpret_cast<uint2*>(p) = out;
}
__device__ __forceinline__ void store4(float* p, const float* y) {
  *reinterpret_cast<float4*>(p) = make_float4(y[0], y[1], y[2], y[3]);
}

// Second product of a launch: same A and shape, its own weights, bias and result.
struct GemmSecond {
  const bf16_t* W = nullptr;
  const bf16_t* bias = nullptr;
  bf16_t* C = nullptr;
};

// ResT / OutT: element type of the residual input and of C (bf16 or fp32).
// DUAL: column tiles past the first product's belong to the second.
template <int BM_, int EPI, typename ResT, typename OutT, bool DUAL>
__global__ __launch_bounds__(NT, 1) void gemm_kernel(const bf16_t* __restrict__ A, int lda,
                                                     const bf16_t* __restrict__ W, int ldw,
                                                     OutT* __restrict__ C, int ldc, int M,
                                                     int N, int K, const GemmEpiArgs ep,
                                                     int tiles_m, int tiles_n, int per_xcd,
                                                     const GemmSecond sec) {
  using G = Cfg<BM_>;
  constexpr int BM = G::BM, STAGES = G::STAGES, WM = G::WM, MB = G::MB;
  constexpr int A_BYTES = G::A_BYTES, STAGE_BYTES = G::STAGE_BYTES, A_INS = G::A_INS;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGES * STAGE_BYTES];

  // XCD-aware tile order: consecutive logical tiles land on one XCD (shared L2)
  const int p = blockIdx.x;
  const int L = (p % kNumXcd) * per_xcd + p / kNumXcd;
  if (L >= tiles_m * tiles_n) return;
  const int group = GROUP_M * tiles_n;
  const int g0 = (L / group) * GROUP_M;
  const int gm = min(tiles_m - g0, GROUP_M);
  const int tm = g0 + (L % group) % gm;
  int tn = (L % group) / gm;
  const bf16_t* bias_p = ep.bias;
  if constexpr (DUAL) {   // tiles_n counts both products' column tiles
    if (tn >= tiles_n / 2) {
      tn -= tiles_n / 2;
      W = sec.W;
      bias_p = sec.bias;
      C = sec.C;
    }
  }

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int wm = wave / NWN, wn = wave % NWN;

  // Load instruction j of this wave fills the 8 LDS rows 8 (wave * INS + j) .. + 7: lane i
  // writes slot i % 8 of row 8 (...) + i / 8, which holds chunk (i % 8) ^ swz(row).  The
  // tile's first row (scalar) plus a per-lane byte offset fixed for the whole K loop.
  const char* a_base = uniform_ptr(A + static_cast<size_t>(tm) * BM * lda);
  const char* w_base = uniform_ptr(W + static_cast<size_t>(tn) * BN * ldw);
  uint32_t a_off[A_INS], w_off[W_INS];
#pragma unroll
  for (int j = 0; j < A_INS; ++j) {
    const int r = 8 * (wave * A_INS + j) + (lane >> 3);
    const int c = (lane & 7) ^ swz(r);
    a_off[j] = static_cast<uint32_t>((min(tm * BM + r, M - 1) - tm * BM) * lda * 2 + c * 16);
  }
#pragma unroll
  for (int j = 0; j < W_INS; ++j) {
    const int r = 8 * (wave * W_INS + j) + (lane >> 3);
    const int c = (lane & 7) ^ swz(r);
    w_off[j] = static_cast<uint32_t>((min(tn * BN + r, N - 1) - tn * BN) * ldw * 2 + c * 16);
  }
  // LDS byte addresses of this wave's first 1 KB blocks of the A and W parts
  // of stage 0 (the wave index made scalar: it is the same in every lane)
  const uint32_t wave_s = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave));
  const uint32_t smem_s = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)smem))));
  const uint32_t lds_a = smem_s + wave_s * (A_INS * 1024u);
  const uint32_t lds_w = smem_s + A_BYTES + wave_s * (W_INS * 1024u);
  auto issue = [&](int kt) {
    const uint32_t so = static_cast<uint32_t>((kt % STAGES) * STAGE_BYTES);
    const int koff = kt * ROW_BYTES;
#pragma unroll
    for (int j = 0; j < A_INS; ++j) lds_dma16(a_base + koff, a_off[j], lds_a + so + 1024u * j);
#pragma unroll
    for (int j = 0; j < W_INS; ++j) lds_dma16(w_base + koff, w_off[j], lds_w + so + 1024u * j);
  };

  f32x4 acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.f;

  const int nk = K / BK;
  // fragments of one 32-wide half of a K step from a stage
  auto read_half = [&](const unsigned char* st, int kk, bf16x8 (&fa)[MB], bf16x8 (&fw)[NB])
      __attribute__((always_inline)) {
    const bf16_t* cA = reinterpret_cast<const bf16_t*>(st);
    const bf16_t* cW = reinterpret_cast<const bf16_t*>(st + A_BYTES);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int r = WN * wn + 16 * nb + l16;
      fw[nb] = *reinterpret_cast<const bf16x8*>(&cW[r * BK + 8 * ((4 * kk + g) ^ swz(r))]);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int r = WM * wm + 16 * mb + l16;
      fa[mb] = *reinterpret_cast<const bf16x8*>(&cA[r * BK + 8 * ((4 * kk + g) ^ swz(r))]);
    }
  };
  auto mma = [&](const bf16x8 (&fa)[MB], const bf16x8 (&fw)[NB]) __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[nb], fa[mb], acc[mb][nb], 0, 0, 0);
  };
  // the MB * NB MFMAs of one half issued in MB + NB groups, each followed by
  // one fragment read of the next half (groups of 3 first, then of 2)
  constexpr int NREAD = MB + NB, EXTRA = MB * NB - 2 * NREAD;
  static_assert(EXTRA >= 0 && EXTRA <= NREAD, "MFMA groups");
  auto interleave = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < EXTRA; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
#pragma unroll
    for (int i = EXTRA; i < NREAD; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  };

  // The fragment reads run one half step ahead of the MFMAs: the second half
  // of step kt is read under the first half's MFMAs, and the first half of
  // step kt+1 under the second half's, after the barrier that publishes stage
  // kt+1.  That barrier also closes every read of stage kt.  With three
  // stages, step kt+2 is requested at the top of step kt (into the slot of
  // step kt-1); with two, right after that barrier (into the slot of step kt).
  // Either way a request has one and a half or one full step to land.
  issue(0);
  if (STAGES == 3 && nk > 1) {
    issue(1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(A_INS + W_INS));
  } else {
    asm volatile("s_waitcnt vmcnt(0)");
  }
  __syncthreads();
  if (STAGES == 2 && nk > 1) issue(1);
  bf16x8 fa0[MB], fw0[NB], fa1[MB], fw1[NB];
  read_half(smem, 0, fa0, fw0);
  // one K step on stage S (a constant: the loop runs the stages in turn, so
  // every LDS address is a register plus an immediate)
  auto step = [&](int kt, auto s_c) __attribute__((always_inline)) {
    constexpr int S = decltype(s_c)::value;
    if (STAGES == 3 && kt + 2 < nk) issue(kt + 2);
    read_half(smem + S * STAGE_BYTES, 1, fa1, fw1);
    mma(fa0, fw0);
    interleave();
    if (kt + 1 < nk) {
      if (STAGES == 3 && kt + 2 < nk) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(A_INS + W_INS));
      } else {
        asm volatile("s_waitcnt vmcnt(0)");
      }
      __syncthreads();
      if (STAGES == 2 && kt + 2 < nk) issue(kt + 2);
      read_half(smem + ((S + 1) % STAGES) * STAGE_BYTES, 0, fa0, fw0);
    }
    mma(fa1, fw1);
    interleave();
  };
  static_assert(STAGES == 2 || STAGES == 3, "the K loop is unrolled over the stages");
  for (int kt = 0; kt < nk; kt += STAGES) {
    step(kt, std::integral_constant<int, 0>{});
    if (kt + 1 < nk) step(kt + 1, std::integral_constant<int, 1>{});
    if constexpr (STAGES == 3) {
      if (kt + 2 < nk) step(kt + 2, std::integral_constant<int, 2>{});
    }
  }

  // epilogue through LDS (free once every wave has read its last fragments),
  // in passes of PASS_ROWS tile rows: the waves holding a pass's rows write
  // y = acc + bias (GELU applied) for their row and four columns of every
  // block into a row-major fp32 tile, and the workgroup then walks the pass
  // one row per wave, each lane taking four consecutive columns, so the
  // residual is read and C written as whole contiguous rows.  The residual
  // and gate loads of a wave's rows go out in two batches, the first before
  // the pass is staged and the second before the first is used, so their
  // latency hides behind the staging and the stores.  Rows are padded by 16
  // bytes: the 16 lanes of one write then cover all 64 banks.
  constexpr int PASS_ROWS = G::PASS_ROWS, NPASS = G::NPASS, RB = G::RB;
  constexpr bool HAS_RES = EPI == kEpiBiasGateRes || EPI == kEpiBiasRes;
  const bool cols_in = tn * BN + WN * wn < N;   // (a tile may end on a half tile)
  const int cl = 4 * lane;
  const bool lane_in = tn * BN + cl < N;
  const int n0 = min(tn * BN + cl, N - 4);      // lanes past N load a valid column, store nothing
  float res[2][RB][4], gmod[2][RB][4];
  auto load_batch = [&](int pass, int b) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int m = min(tm * BM + PASS_ROWS * pass + wave + NWAVES * (RB * b + i), M - 1);
      if (HAS_RES)
        load4(static_cast<const ResT*>(ep.res) + static_cast<size_t>(m) * ep.ldr + n0, res[b][i]);
      if (EPI == kEpiBiasGateRes)
        load4(ep.mod + (static_cast<size_t>(m / ep.rows_per_stream) * 6 + ep.gate_row) * ep.dim + n0,
              gmod[b][i]);
    }
  };
  float gt4[4] = {0.f, 0.f, 0.f, 0.f};
  if (EPI == kEpiBiasGateRes) load4(ep.mod_table + static_cast<size_t>(ep.gate_row) * ep.dim + n0, gt4);
  float bias[NB][4];
  if (cols_in) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) load4(bias_p + tn * BN + WN * wn + 16 * nb + 4 * g, bias[nb]);
  }
#pragma unroll
  for (int pass = 0; pass < NPASS; ++pass) {
    load_batch(pass, 0);
    __syncthreads();
    if (cols_in) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int r = WM * wm + 16 * mb + l16 - PASS_ROWS * pass;
        if (NPASS > 1 && (WM * wm + 16 * mb) / PASS_ROWS != pass) continue;   // (wave-uniform)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int c = WN * wn + 16 * nb + 4 * g;
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = acc[mb][nb][e] + bias[nb][e];
          if (EPI == kEpiBiasGelu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = gelu_tanh(y[e]);
          }
          *reinterpret_cast<float4*>(smem + r * CROW + c * 4) = make_float4(y[0], y[1], y[2], y[3]);
        }
      }
    }
    __syncthreads();
    load_batch(pass, 1);
    if (lane_in) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          const int rr = wave + NWAVES * (RB * b + i);
          const int m = tm * BM + PASS_ROWS * pass + rr;
          if (m < M) {
            const float4 t = *reinterpret_cast<const float4*>(smem + rr * CROW + cl * 4);
            float y[4] = {t.x, t.y, t.z, t.w};
            if (EPI == kEpiBiasGateRes) {
#pragma unroll
              for (int e = 0; e < 4; ++e) y[e] = res[b][i][e] + (gmod[b][i][e] + gt4[e]) * y[e];
            } else if (EPI == kEpiBiasRes) {
#pragma unroll
              for (int e = 0; e < 4; ++e) y[e] = res[b][i][e] + y[e];
            }
            store4(C + static_cast<size_t>(m) * ldc + n0, y);
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------ small products
// Products of a few hundred rows leave most CUs without a 128 x 256 tile and
// run at the latency of one tile's K loop, about 0.9 us a step with two steps
// in flight (text keys and values of 589 tokens, 1536 wide: 50 us in four
// launches, now 17 us in two; the tiny block's step, 192 rows of 256: 101 -> 65
// us).  Here tiles are small (64 x 128 on eight waves, or 32 x 64 on
// four, so more CUs take part) and S - 1 steps are in flight through a ring of
// S LDS stages: at K = 256 a tile's whole operands are requested at once.  One
// barrier per step: it publishes stage kt and closes the reads of stage kt-1,
// into which step kt+S-1 is then requested.  Each output element goes through
// the same MFMA sequence as in gemm_kernel, so C does not depend on which of
// the kernels computes it.  The epilogue's operands are loaded before the K
// loop and the results stored from registers (4 columns a lane; the outputs
// are small).
//
// Up to two products of one A (text keys and values) share a launch: the
// workgroups past the first product's take W2 / bias2.  The second's result
// may go transposed per head ([H][hd][len] per stream, vt), where 16 lanes
// hold 16 consecutive tokens of a dim.
struct SmallDual {
  const bf16_t* W2 = nullptr;      // second product (null: none), same shape and A
  const bf16_t* bias2 = nullptr;
  bf16_t* C2 = nullptr;            // transposed per head and stream
  RowStreams rs;                   // streams of the rows (len, row_begin)
};

template <int WM_, int WN_, int MB, int NB, int S, int EPI, typename ResT, typename OutT, bool DUAL>
__global__ __launch_bounds__(64 * WM_ * WN_, 1) void gemm_small_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, int ldw,
    OutT* __restrict__ C, int ldc, int M, int N, int K, const GemmEpiArgs ep, int tiles_m,
    int tiles_n, const SmallDual du) {
  constexpr int NW = WM_ * WN_, BM = 16 * MB * WM_, BNS = 16 * NB * WN_;
  constexpr int AB = BM * ROW_BYTES, WB = BNS * ROW_BYTES, STAGE = AB + WB;
  constexpr int A_INS = AB / 1024 / NW, WI = WB / 1024 / NW, INS = A_INS + WI;
  static_assert(A_INS * NW * 1024 == AB && WI * NW * 1024 == WB, "whole 1 KB loads per wave");
  static_assert(S * STAGE <= 160 * 1024 && S >= 3 && S <= 6, "LDS");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S * STAGE];
  // XCD-aware order: each XCD takes a run of column tiles with all their row
  // tiles, so a W tile is fetched by one XCD only
  const int total = (DUAL ? 2 : 1) * tiles_m * tiles_n;
  const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
  int p = static_cast<int>(blockIdx.x % kNumXcd) * per_xcd + static_cast<int>(blockIdx.x / kNumXcd);
  if (p >= total) return;
  const bool second = DUAL && p >= tiles_m * tiles_n;
  if (second) p -= tiles_m * tiles_n;
  const int tm = p % tiles_m, tn = p / tiles_m;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int wm = wave / WN_, wn = wave % WN_;
  const char* a_base = uniform_ptr(A + static_cast<size_t>(tm) * BM * lda);
  const char* w_base = uniform_ptr((second ? du.W2 : W) + static_cast<size_t>(tn) * BNS * ldw);
  uint32_t a_off[A_INS], w_off[WI];
#pragma unroll
  for (int j = 0; j < A_INS; ++j) {
    const int r = 8 * (wave * A_INS + j) + (lane >> 3);
    a_off[j] = static_cast<uint32_t>((min(tm * BM + r, M - 1) - tm * BM) * lda * 2 +
                                     ((lane & 7) ^ swz(r)) * 16);
  }
#pragma unroll
  for (int j = 0; j < WI; ++j) {   // (N is a multiple of the tile width)
    const int r = 8 * (wave * WI + j) + (lane >> 3);
    w_off[j] = static_cast<uint32_t>(r * ldw * 2 + ((lane & 7) ^ swz(r)) * 16);
  }
  const uint32_t wave_s = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave));
  const uint32_t smem_s = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)smem))));
  const uint32_t lds_a = smem_s + wave_s * (A_INS * 1024u);
  const uint32_t lds_w = smem_s + AB + wave_s * (WI * 1024u);
  auto issue = [&](int kt, int slot) {
    const uint32_t so = static_cast<uint32_t>(slot * STAGE);
    const int koff = kt * ROW_BYTES;
#pragma unroll
    for (int j = 0; j < A_INS; ++j) lds_dma16(a_base + koff, a_off[j], lds_a + so + 1024u * j);
#pragma unroll
    for (int j = 0; j < WI; ++j) lds_dma16(w_base + koff, w_off[j], lds_w + so + 1024u * j);
  };

  // epilogue operands, requested first: lane owns row m of block mb, columns n .. n + 3 of nb
  constexpr bool HAS_RES = EPI == kEpiBiasGateRes || EPI == kEpiBiasRes;
  const int m0 = tm * BM + 16 * MB * wm + l16, n0 = tn * BNS + 16 * NB * wn + 4 * g;
  const bf16_t* bias = second ? du.bias2 : ep.bias;
  float bi[NB][4], res[MB][NB][4], gm[MB][NB][4], gt[NB][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    load4(bias + n0 + 16 * nb, bi[nb]);
    if (EPI == kEpiBiasGateRes) load4(ep.mod_table + static_cast<size_t>(ep.gate_row) * ep.dim + n0 + 16 * nb, gt[nb]);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = min(m0 + 16 * mb, M - 1);
      if (HAS_RES)
        load4(static_cast<const ResT*>(ep.res) + static_cast<size_t>(m) * ep.ldr + n0 + 16 * nb, res[mb][nb]);
      if (EPI == kEpiBiasGateRes)
        load4(ep.mod + (static_cast<size_t>(m / ep.rows_per_stream) * 6 + ep.gate_row) * ep.dim + n0 + 16 * nb,
              gm[mb][nb]);
    }
  }
  // the vector-memory waits below count these loads too (they are older than
  // every stage's), so they are done whenever the first stage is

  f32x4 acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.f;
  const int nk = K / BK;
#pragma unroll
  for (int i = 0; i < S - 1; ++i)
    if (i < nk) issue(i, i);
  int slot = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // stage kt has landed once at most the later requested steps are in flight
    const int rem = min(S - 2, nk - 1 - kt);
    if (rem >= 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * INS));
    else if (rem == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * INS));
    else if (rem == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * INS));
    else if (rem == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(INS));
    else asm volatile("s_waitcnt vmcnt(0)");
    __syncthreads();
    if (kt + S - 1 < nk) issue(kt + S - 1, slot == 0 ? S - 1 : slot - 1);
    const bf16_t* cA = reinterpret_cast<const bf16_t*>(smem + slot * STAGE);
    const bf16_t* cW = reinterpret_cast<const bf16_t*>(smem + slot * STAGE + AB);
    bf16x8 fa[2][MB], fw[2][NB];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int r = 16 * (NB * wn + nb) + l16;
        fw[kk][nb] = *reinterpret_cast<const bf16x8*>(&cW[r * BK + 8 * ((4 * kk + g) ^ swz(r))]);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int r = 16 * (MB * wm + mb) + l16;
        fa[kk][mb] = *reinterpret_cast<const bf16x8*>(&cA[r * BK + 8 * ((4 * kk + g) ^ swz(r))]);
      }
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[kk][nb], fa[kk][mb], acc[mb][nb], 0, 0, 0);
    slot = slot == S - 1 ? 0 : slot + 1;
  }

#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int m = m0 + 16 * mb;
    if (m >= M) continue;
    size_t vt = 0;   // transposed output: element of (head 0, dim 0, this token)
    int len = 0;
    if (second) {
      int b = 0;
      for (int i = 1; i < du.rs.n; ++i)
        if (m >= du.rs.s[i].row_begin) b = i;
      len = du.rs.s[b].len;
      vt = static_cast<size_t>(du.rs.s[b].row_begin) * N + (m - du.rs.s[b].row_begin);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int n = n0 + 16 * nb;
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = acc[mb][nb][e] + bi[nb][e];
        if (EPI == kEpiBiasGelu) y[e] = gelu_tanh(y[e]);
        if (EPI == kEpiBiasGateRes) y[e] = res[mb][nb][e] + (gm[mb][nb][e] + gt[nb][e]) * y[e];
        if (EPI == kEpiBiasRes) y[e] = res[mb][nb][e] + y[e];
      }
      if (second) {   // (column n = head n / hd, dim n % hd: row n of the stream's [H hd][len])
#pragma unroll
        for (int e = 0; e < 4; ++e) du.C2[vt + static_cast<size_t>(n + e) * len] = f2bf(y[e]);
      } else {
        store4(C + static_cast<size_t>(m) * ldc + n, y);
      }
    }
  }
}

}  // namespace

// Tile height for an M x N product.  Both heights give bit-identical C (the
// same MFMA sequence per output element), so the choice is speed only: the
// 192-row tile is taken when it needs clearly fewer rounds of 256
// workgroups, counting one of its rounds as 1.38 rounds of 128-row tiles
// (1.5 times the work at 92% of the time per unit of work).
static int choose_bm(int M, int N) {
  const long tn = (N + BN - 1) / BN;
  const long r128 = ((M + 127) / 128 * tn + 255) / 256;
  const long r192 = ((M + 191) / 192 * tn + 255) / 256;
  return 1.38 * static_cast<double>(r192) < static_cast<double>(r128) ? 192 : 128;
}

template <int BM_, int EPI, typename ResT, typename OutT>
static void launch_t(hipStream_t st, const bf16_t* A, int lda, const bf16_t* W, int ldw, void* C,
                     int ldc, int M, int N, int K, const GemmEpiArgs& ep) {
  const int tiles_m = (M + BM_ - 1) / BM_, tiles_n = (N + BN - 1) / BN;
  const int total = tiles_m * tiles_n;
  const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
  hipLaunchKernelGGL((gemm_kernel<BM_, EPI, ResT, OutT, false>), dim3(per_xcd * kNumXcd), dim3(NT), 0,
                     st, A, lda, W, ldw, static_cast<OutT*>(C), ldc, M, N, K, ep, tiles_m, tiles_n,
                     per_xcd, GemmSecond{});
}

// Which small tile, if any (0: the large tiles); N counts both products' columns
// when two share a launch.  32 x 64 tiles leave room for two workgroups on a CU,
// 64 x 128 for one, and each is taken while its workgroups fit one round of the
// chip: past that a second round costs more than the larger tile's lower share
// of CUs.  Text keys and values of 1536-wide tokens (two products, us): 64
// tokens 12 / 16 / 27 on 32-row / 64-row / 128-row tiles, 192: 14 / 17 / 28,
// 512: 21 / 17 / 29, 1560: 48 / 40 / 33; 5120-wide: 64 tokens 37 / 40 / 66,
// 192: 58 / 42 / 69, 512: 132 / 99 / 71.
static int small_tile(int M, int N) {
  if (static_cast<long>((M + 31) / 32) * (N / 64) <= 512) return 32;
  return static_cast<long>((M + 63) / 64) * (N / 128) <= 256 ? 64 : 0;
}

template <int WM_, int WN_, int MB, int NB, int EPI, typename ResT, typename OutT, bool DUAL>
static void launch_small_t(hipStream_t st, const bf16_t* A, int lda, const bf16_t* W, int ldw, void* C,
                           int ldc, int M, int N, int K, const GemmEpiArgs& ep, const SmallDual& du) {
  const int tm = (M + 16 * MB * WM_ - 1) / (16 * MB * WM_), tn = N / (16 * NB * WN_);
  const int wgs = ((DUAL ? 2 : 1) * tm * tn + kNumXcd - 1) / kNumXcd * kNumXcd;
  hipLaunchKernelGGL((gemm_small_kernel<WM_, WN_, MB, NB, 6, EPI, ResT, OutT, DUAL>), dim3(wgs),
                     dim3(64 * WM_ * WN_), 0, st, A, lda, W, ldw, static_cast<OutT*>(C), ldc, M, N, K, ep, tm,
                     tn, du);
}
template <int EPI, typename ResT, typename OutT>
static void launch_small(int tile, hipStream_t st, const bf16_t* A, int lda, const bf16_t* W, int ldw,
                         void* C, int ldc, int M, int N, int K, const GemmEpiArgs& ep) {
  if (tile == 32)
    launch_small_t<2, 2, 1, 2, EPI, ResT, OutT, false>(st, A, lda, W, ldw, C, ldc, M, N, K, ep, SmallDual{});
  else
    launch_small_t<2, 4, 2, 2, EPI, ResT, OutT, false>(st, A, lda, W, ldw, C, ldc, M, N, K, ep, SmallDual{});
}

template <int EPI, typename ResT, typename OutT>
static void launch_bm(hipStream_t st, const bf16_t* A, int lda, const bf16_t* W, int ldw, void* C,
                      int ldc, int M, int N, int K, const GemmEpiArgs& ep) {
  if (const int tile = small_tile(M, N))
    launch_small<EPI, ResT, OutT>(tile, st, A, lda, W, ldw, C, ldc, M, N, K, ep);
  else if (choose_bm(M, N) == 192)
    launch_t<192, EPI, ResT, OutT>(st, A, lda, W, ldw, C, ldc, M, N, K, ep);
  else
    launch_t<128, EPI, ResT, OutT>(st, A, lda, W, ldw, C, ldc, M, N, K, ep);
}

template <int BM_>
static void launch_dual_t(hipStream_t st, const bf16_t* A, int lda, const bf16_t* W, int ldw, bf16_t* C, int ldc,
                          int M, int N, int K, const GemmEpiArgs& ep, const GemmSecond& sec) {
  const int tiles_m = (M + BM_ - 1) / BM_, tiles_n = 2 * ((N + BN - 1) / BN);
  const int per_xcd = (tiles_m * tiles_n + kNumXcd - 1) / kNumXcd;
  hipLaunchKernelGGL((gemm_kernel<BM_, kEpiBias, bf16_t, bf16_t, true>), dim3(per_xcd * kNumXcd), dim3(NT), 0,
                     st, A, lda, W, ldw, C, ldc, M, N, K, ep, tiles_m, tiles_n, per_xcd, sec);
}

hipError_t launch_ctx_gemms(hipStream_t st, const bf16_t* ctx, int M, int D, const bf16_t* Wk,
                            const bf16_t* bk, bf16_t* ck, const bf16_t* Wv, const bf16_t* bv, bf16_t* cv,
                            bf16_t* ctx_v, const RowStreams& rs, bool* v_done) {
  *v_done = false;
  if (M == 0) return hipSuccess;
  if (D % 128 != 0) return hipErrorInvalidValue;
  GemmEpiArgs e;
  e.bias = bk;
  // the tile rule of small_tile on the workgroups of both products
  const int tile = ctx_v ? small_tile(M, 2 * D) : 0;
  if (tile) {
    SmallDual du{};
    du.W2 = Wv;
    du.bias2 = bv;
    du.C2 = ctx_v;
    du.rs = rs;
    if (tile == 32)
      launch_small_t<2, 2, 1, 2, kEpiBias, bf16_t, bf16_t, true>(st, ctx, D, Wk, D, ck, D, M, D, D, e, du);
    else
      launch_small_t<2, 4, 2, 2, kEpiBias, bf16_t, bf16_t, true>(st, ctx, D, Wk, D, ck, D, M, D, D, e, du);
    *v_done = true;
  } else {
    const GemmSecond sec{Wv, bv, cv};
    if (choose_bm(M, 2 * D) == 192) launch_dual_t<192>(st, ctx, D, Wk, D, ck, D, M, D, D, e, sec);
    else launch_dual_t<128>(st, ctx, D, Wk, D, ck, D, M, D, D, e, sec);
  }
  return hipGetLastError();
}

hipError_t launch_gemm(hipStream_t st, int epi, const bf16_t* A, int lda, const bf16_t* W,
                       int ldw, void* C, int ldc, int M, int N, int K, const GemmEpiArgs& ep) {
  if (M == 0) return hipSuccess;
  if (N % 128 != 0 || K % BK != 0 || K == 0) return hipErrorInvalidValue;
  const bool rf = ep.res_f32, of = ep.out_f32;
#define ARDIT_GEMM(E, R, O) launch_bm<E, R, O>(st, A, lda, W, ldw, C, ldc, M, N, K, ep)
  switch (epi) {
    case kEpiBias:
      if (of) ARDIT_GEMM(kEpiBias, bf16_t, float); else ARDIT_GEMM(kEpiBias, bf16_t, bf16_t);
      break;
    case kEpiBiasGelu:
      ARDIT_GEMM(kEpiBiasGelu, bf16_t, bf16_t);
      break;
    case kEpiBiasGateRes:
      if (rf && of) ARDIT_GEMM(kEpiBiasGateRes, float, float);
      else if (rf) ARDIT_GEMM(kEpiBiasGateRes, float, bf16_t);
      else if (of) ARDIT_GEMM(kEpiBiasGateRes, bf16_t, float);
      else ARDIT_GEMM(kEpiBiasGateRes, bf16_t, bf16_t);
      break;
    case kEpiBiasRes:
      if (rf && of) ARDIT_GEMM(kEpiBiasRes, float, float);
      else if (rf) ARDIT_GEMM(kEpiBiasRes, float, bf16_t);
      else if (of) ARDIT_GEMM(kEpiBiasRes, bf16_t, float);
      else ARDIT_GEMM(kEpiBiasRes, bf16_t, bf16_t);
      break;
    default:
      return hipErrorInvalidValue;
  }
#undef ARDIT_GEMM
  return hipGetLastError();
}

}  // namespace ardit
