// GEMMs of the denoiser blocks: C[M][N] = A[M][K] W[N][K]^T + b with a fused
// epilogue:
//   EPI_BIAS  : out = C                         (QKV projection)      -> bf16/fp32
//   EPI_GELU  : out = GELU_tanh(C)              (MLP first layer)     -> bf16/fp32
//   EPI_GATED : h  += (1 + gate[row]) * C       (out-proj, MLP second layer; fp32 residual)
// M = selected tokens (ragged); N and K multiples of 128 on the bf16 path.
//
// bf16 path (gfx950 MFMA): k_gemm_dma_* (described with their code).  Operand
// offsets are 32-bit: the caller guarantees M*K and N*K below 2^31 elements.
//
// fp32 path (fp32 models): k_gemm_f32, described with its code.
#include <atomic>
#include <type_traits>

#include "kernels.hpp"
#include "launch_rules.hpp"

namespace sphinx {

namespace {
// ---------------------------------------------------------------------------
// bf16 GEMM with direct global->LDS copies (global_load_lds_dwordx4).
//  * Block tile 128x128x64, 4 waves in 2x2, each a 64x64 tile of 4x4
//    v_mfma_f32_16x16x32_bf16; two workgroups per CU.  That form draws less
//    power than the 32x32x16 one at the same work (register-only loops on random
//    operands run at 2050 against 1790 TFLOP/s), and long runs are power-limited.
//    In these kernels it gives up to 4 % (M 10816, D 1152, QKV 101.4 -> 97.0 us;
//    M 23712, D 512, QKV 44.7 -> 43.2, D 640, MLP2 84.7 -> 81.4), at most sizes
//    nothing that shows.  Eight-wave tiles of small selections, bound by latency,
//    take the 32x32x16 form with its smaller number of instructions (QKV at M
//    1613: 16.5 us against 17.5).  Both add the products of a row in ascending k.
//    That they also round alike inside an instruction is measured, not given by
//    their definition: 67 million outputs of K 32 to 4096 from operands of like
//    size, of exponents over 2^+-30, with cancelling pairs, with subnormal
//    products and with overflow are the same to the bit.
//  * Operand tiles are unpadded 128-byte rows (A rows, then W rows, of one
//    64-wide K step); chunk c of row r sits at c ^ ((r >> 1) & 7), which spreads
//    the 16 rows of one ds_read_b128 pass (same chunk) over all 64 LDS banks.
//    Each wave copies 8 rows per instruction: lane i of copy q writes slot i%8
//    of row 8q + i/8 and reads the global chunk the permutation puts there, so
//    the copy needs no registers and no LDS stores; its source is a
//    wave-uniform scalar base (A or W, moved by scalar adds per K step) plus a
//    fixed per-lane byte offset, so it needs no VALU either.
//  * On gfx950 VALU work does not overlap other waves' MFMAs, so the loop is
//    kept free of it: the K loop is unrolled over the ring, making every
//    fragment address a loop-invariant base plus an immediate offset.
//  * K steps live in a 2-slot ring.  The wait for the next step's copies and
//    the workgroup barrier sit inside the last k-step (16 or 32 deep) of the current
//    one, so the next step's first fragments are read (and the following
//    copies issued) while the last MFMAs of the current step run; inside a
//    step each k-step's fragment reads are issued before the previous
//    k-step's MFMAs.  Barriers carry no memory fence: each wave waits for its
//    own copies (vmcnt) and LDS reads (lgkmcnt) first.
//  * Every output starts at its bias and accumulates its k-steps in ascending
//    k, whatever the tile shape; with the two MFMA forms rounding alike, all
//    variants give bit-identical results (every one is compared in
//    tests/test_gpu_gemm_tiles.py), so packed and separate requests do too.
//  * A 192-row variant (wave tiles 96x64, 80 KB of LDS, epilogue staged one
//    wave row at a time) is launched where its smaller tile count packs into
//    fewer rounds of two workgroups per CU; same results.
//  * Launches whose 128-, 192- or 256-row tiles all fit on the CUs at once
//    (few selected tokens) run the smallest such tile, one eight-wave
//    workgroup per CU with a ring of 3 or 4 stages; same results.
namespace dma {

// s_waitcnt immediate: vmcnt(vm) expcnt(7) lgkmcnt(0) (gfx9 encoding: vmcnt in
// bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
constexpr int wait_vm_lgkm0(int vm) { return 0x0070 | (vm & 15) | ((vm >> 4) << 14); }

// EH: the fp32 epilogue tile is staged in EH row halves (EH = 2 when the
// whole tile would need more LDS than the operand ring).  NW waves in 2 rows
// of NW/2 (4: 2x2, 8: 2x4).
template <int BM, int BN, int NS, int EH = 1, int NW = 4>
struct DmaCfg {
  static constexpr int BK = 64;
  static constexpr int NT = 64 * NW, WGN = NW / 2;  // threads; waves along N
  // MF x MF output blocks per MFMA; LG lane groups share a row, KS k-steps
  static constexpr int MF = NW == 8 ? 32 : 16, NQ = MF * MF / 256, LG = 64 / MF, KS = 8 / LG;
  using Acc = std::conditional_t<MF == 32, f32x16, f32x4>;
  static constexpr int WM = BM / 2, WN = BN / WGN, TI = WM / MF, TJ = WN / MF;
  static constexpr int STAGE = (BM + BN) * 128;     // bytes per K-step
  static constexpr int COPIES = (BM + BN) / 8 / NW; // copy instructions per wave per stage
  static constexpr int CLD = BN + 4;                // epilogue staging row (fp32)
  static constexpr int EROWS = BM / EH;             // tile rows staged at once
  static constexpr int SMEM = NS * STAGE > EROWS * CLD * 4 ? NS * STAGE : EROWS * CLD * 4;
  static_assert(EH == 1 || EH == 2, "whole tile or two halves (one per wave row)");
  static_assert(NW == 4 || NW == 8, "2x2 or 2x4 waves");
  static_assert(COPIES * 8 * NW == BM + BN && BM % 8 == 0, "each copy instruction moves 8 rows of A or of W");
};

// Tile of a one-dimensional grid of BM x BN tiles; workgroups are dealt to the
// 8 XCDs round-robin.  Wide N (more than 8 column tiles, and W at least a
// quarter of A): tiles in plain N-fastest order, so XCD x always gets the
// column tiles n = x (mod 8) and keeps that eighth of W in its L2 for the
// whole kernel.  Otherwise renumbered (xcd_tile) so that each XCD takes
// consecutive row blocks of A with all their column tiles: A is fetched into
// one L2 instead of eight, W into all eight.
template <int BM, int BN>
__device__ __forceinline__ void grid_tile(int M, int N, int& m0, int& n0) {
  const int nt = N / BN;
  if (nt > 8 && M < 4 * N) {
    m0 = ((int)blockIdx.x / nt) * BM;
    n0 = ((int)blockIdx.x % nt) * BN;
  } else {
    const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    m0 = (tile / nt) * BM;
    n0 = (tile % nt) * BN;
  }
}

template <int EPI, int BM, int BN, int NS, int EH = 1, int NW = 4>
__device__ __forceinline__ void gemm_dma_body(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                              const bf16* __restrict__ bias, int M, int N, int K, GemmEpi e,
                                              unsigned char* smem, int m0, int n0) {
  typedef DmaCfg<BM, BN, NS, EH, NW> C;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WGN, wn = wave % C::WGN;
  const int g = lane / C::MF, rf = lane % C::MF;

  // copy sources: instruction i of this wave fills rows 8q .. 8q+7 of the
  // stage (q = wave * COPIES + i; rows < BM are A rows, the rest W rows)
  // (the operand, A or W, is wave-uniform: a scalar base; the lane's byte
  // offset from it is fixed, so moving to the next K step is scalar arithmetic)
  const bf16* src[C::COPIES];
  uint32_t voff[C::COPIES];
#pragma unroll
  for (int i = 0; i < C::COPIES; ++i) {
    const int q = wave * C::COPIES + i;
    const int row = 8 * q + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    if (8 * q < BM) {
      src[i] = A;
      voff[i] = 2u * (uint32_t)(min(m0 + row, M - 1) * K + c * 8);
    } else {
      src[i] = W;
      voff[i] = 2u * (uint32_t)((n0 + row - BM) * K + c * 8);
    }
  }
  auto copy_stage = [&](int kt, int slot) {
    unsigned char* base = smem + slot * C::STAGE;
#pragma unroll
    for (int i = 0; i < C::COPIES; ++i)
      lds_dma16_at(src[i] + kt * C::BK, voff[i], base + (wave * C::COPIES + i) * 1024);
  };
  // fragment offsets inside a stage (one k-step per MFMA)
  int foff[C::KS];
#pragma unroll
  for (int ks = 0; ks < C::KS; ++ks) foff[ks] = rf * 128 + (((C::LG * ks + g) ^ ((rf >> 1) & 7)) << 4);
  const int a_row0 = wm * C::WM, b_row0 = BM + wn * C::WN;

  // acc[i][j] is the transposed output block: the MFMA takes the W fragment
  // as its A operand, so lane l holds row a_row0 + MF i + l%MF of the tile and,
  // in registers 4q .. 4q+3, its four consecutive columns wn WN + MF j + 8q +
  // 4(l/MF) .. +3.  The accumulators start at the bias of their column, so the
  // epilogue adds no bias.
  typename C::Acc acc[C::TI][C::TJ];
#pragma unroll
  for (int j = 0; j < C::TJ; ++j)
#pragma unroll
    for (int q = 0; q < C::NQ; ++q) {
      const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(bias + n0 + wn * C::WN + j * C::MF + 8 * q + 4 * g);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < C::TI; ++i) acc[i][j][4 * q + t] = (float)b4[t];
    }

  const int KT = K / C::BK;  // even (K is a multiple of 128)
  static_assert(NS >= 2 && NS <= 4, "ring of 2 to 4 stages");
  // Stage j lives in slot j % NS.  The wait for stage kt+1 and the barrier sit
  // inside the last k-step of tile kt: after it every wave has read all of
  // stage kt (so its slot can be refilled with stage kt+NS) and stage kt+1 has
  // landed (so its first fragments can be read while the last MFMAs of tile
  // kt run).  With NS > 2 every K step refills its slot, near the end with a
  // copy of the last stage into a slot that is not read again, so that at
  // each wait exactly the NS - 2 newest stages may still be in flight.
  auto sync_stage = [&]() {
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((NS - 2) * C::COPIES));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
#pragma unroll
  for (int st = 0; st < NS; ++st) copy_stage(NS == 2 ? st : min(st, KT - 1), st);
  // stage 0 must land before the first reads; the later ones may stay in flight
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((NS - 1) * C::COPIES));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  bf16x8 fa[C::KS][C::TI], fb[C::KS][C::TJ];  // one register set per k-step
  auto read = [&](const unsigned char* st, int ks, int buf) {
#pragma unroll
    for (int i = 0; i < C::TI; ++i)
      fa[buf][i] = *reinterpret_cast<const bf16x8*>(st + (a_row0 + C::MF * i) * 128 + foff[ks]);
#pragma unroll
    for (int j = 0; j < C::TJ; ++j)
      fb[buf][j] = *reinterpret_cast<const bf16x8*>(st + (b_row0 + C::MF * j) * 128 + foff[ks]);
  };
  // One K step in ring slot SLOT (a compile-time constant, so that every
  // fragment address is a loop-invariant base plus an immediate offset).
  auto step = [&](int kt, auto SLOT) {
    constexpr int slot = decltype(SLOT)::value, nslot = slot + 1 == NS ? 0 : slot + 1;
    const unsigned char* st = smem + slot * C::STAGE;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
      if (ks + 1 < C::KS) {
        read(st, ks + 1, ks + 1);
      } else if (kt + 1 < KT) {
        sync_stage();
        if constexpr (NS == 2) {
          if (kt + NS < KT) copy_stage(kt + NS, slot);
        } else {
          copy_stage(min(kt + NS, KT - 1), slot);
        }
        read(smem + nslot * C::STAGE, 0, 0);
      }
      // the next k-step's reads are issued before this k-step's MFMAs
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < C::TI; ++i)
#pragma unroll
        for (int j = 0; j < C::TJ; ++j) {
          if constexpr (C::MF == 32)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  read(smem, 0, 0);
  // whole trips over the ring, then (NS > 2) the last KT % NS stages; with two
  // slots KT is even (K is a multiple of 128, which launch_gemm checks)
  if constexpr (NS == 2) {
    for (int kt = 0; kt < KT; kt += 2) {
      step(kt, std::integral_constant<int, 0>{});
      step(kt + 1, std::integral_constant<int, 1>{});
    }
  } else {
    int kt = 0;
    for (; kt + NS <= KT; kt += NS) {
      step(kt, std::integral_constant<int, 0>{});
      step(kt + 1, std::integral_constant<int, 1>{});
      step(kt + 2, std::integral_constant<int, 2>{});
      if constexpr (NS > 3) step(kt + 3, std::integral_constant<int, 3>{});
    }
    if (kt < KT) step(kt, std::integral_constant<int, 0>{});
    if (kt + 1 < KT) step(kt + 1, std::integral_constant<int, 1>{});
    if constexpr (NS > 3)
      if (kt + 2 < KT) step(kt + 2, std::integral_constant<int, 2>{});
  }
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // epilogue: fp32 tile staged in LDS (whole, or one wave row's half at a
  // time), then 16-byte row-contiguous I/O.  Outputs and the residual are
  // addressed as a wave-uniform tile base plus the thread's 32-bit byte offset
  // (at most EROWS rows of ldo elements), which grows by a fixed stride per
  // pass; tiles wholly inside M skip the per-row checks, and the query scale
  // is a tile-uniform branch.
  float* sC = reinterpret_cast<float*>(smem);
  constexpr int TPR = BN / 4;          // threads per row (one float4 each)
  constexpr int RPP = C::NT / TPR;     // rows per pass
  constexpr int NP = C::EROWS / RPP;   // row passes per staged half
  constexpr int OSZ = EPI == EPI_GATED ? 4 : 2;  // output bytes: fp32 residual or bf16 activation
  const int c4 = (tid % TPR) * 4, rsub = tid / TPR;
  const uint32_t off0 = (uint32_t)(rsub * e.ldo + c4) * OSZ, ostep = (uint32_t)(RPP * e.ldo) * OSZ;
  auto epilogue = [&](auto FULL, auto QT) {
    constexpr bool kFull = decltype(FULL)::value, kQ = decltype(QT)::value;
#pragma unroll
    for (int h = 0; h < EH; ++h) {
      const int mh = m0 + h * C::EROWS;  // first row of this half
      char* obase = reinterpret_cast<char*>(e.out) + ((int64_t)mh * e.ldo + n0) * OSZ;
      // gated residual: every pass's residual and gate loads are issued before
      // the staging (rows past M read row M - 1 and are not stored), so their
      // latencies overlap instead of following one another pass by pass
      float4 hres[EPI == EPI_GATED ? NP : 1], gres[EPI == EPI_GATED ? NP : 1];
      if constexpr (EPI == EPI_GATED) {
        int cr[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const int m = mh + p * RPP + rsub;
          cr[p] = e.crow[kFull ? m : min(m, M - 1)];
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          // in a tile that crosses M the clamped row may lie before this half
          // (a whole half past M reads row M - 1): address it absolutely there
          if constexpr (kFull)
            hres[p] = *reinterpret_cast<const float4*>(obase + off0 + p * ostep);
          else
            hres[p] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(e.out) +
                                                       (int64_t)min(mh + p * RPP + rsub, M - 1) * e.ldo + n0 + c4);
          gres[p] = *reinterpret_cast<const float4*>(e.gate + (int64_t)cr[p] * e.ldg + n0 + c4);
        }
      }
      if (EH == 1 || wm == h) {  // four consecutive columns per 16-byte LDS store
        float* srow = sC + (a_row0 - h * C::EROWS + rf) * C::CLD + wn * C::WN + 4 * g;
#pragma unroll
        for (int i = 0; i < C::TI; ++i)
#pragma unroll
          for (int j = 0; j < C::TJ; ++j)
#pragma unroll
            for (int q = 0; q < C::NQ; ++q)
              *reinterpret_cast<float4*>(srow + i * C::MF * C::CLD + j * C::MF + 8 * q) =
                  make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
      }
      __syncthreads();
      if constexpr (EPI == EPI_GATED) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const float4 v = *reinterpret_cast<const float4*>(&sC[(p * RPP + rsub) * C::CLD + c4]);
          const float4 gv = gres[p];
          float4 hv = hres[p];
          hv.x = fmaf(1.0f + gv.x, v.x, hv.x);
          hv.y = fmaf(1.0f + gv.y, v.y, hv.y);
          hv.z = fmaf(1.0f + gv.z, v.z, hv.z);
          hv.w = fmaf(1.0f + gv.w, v.w, hv.w);
          if (kFull || mh + p * RPP + rsub < M) *reinterpret_cast<float4*>(obase + off0 + p * ostep) = hv;
        }
      } else {
#pragma unroll 4
        for (int p = 0; p < NP; ++p) {
          if (!kFull && mh + p * RPP + rsub >= M) continue;
          float4 v = *reinterpret_cast<const float4*>(&sC[(p * RPP + rsub) * C::CLD + c4]);
          if constexpr (EPI == EPI_GELU) {
            v.x = gelu_tanh(v.x);
            v.y = gelu_tanh(v.y);
            v.z = gelu_tanh(v.z);
            v.w = gelu_tanh(v.w);
          }
          if constexpr (kQ) {
            v.x *= e.qscale;
            v.y *= e.qscale;
            v.z *= e.qscale;
            v.w *= e.qscale;
          }
          bf16x4 o;
          o[0] = (bf16)v.x;
          o[1] = (bf16)v.y;
          o[2] = (bf16)v.z;
          o[3] = (bf16)v.w;
          *reinterpret_cast<bf16x4*>(obase + off0 + p * ostep) = o;
        }
      }
      if (h + 1 < EH) __syncthreads();  // the next half reuses the staging rows
    }
  };
  // a column tile is all queries or none (qcols is a multiple of 128)
  const bool qtile = EPI == EPI_BIAS && n0 < e.qcols;
  if (m0 + BM <= M) {
    if (qtile) epilogue(std::true_type{}, std::true_type{});
    else epilogue(std::true_type{}, std::false_type{});
  } else {
    if (qtile) epilogue(std::false_type{}, std::true_type{});
    else epilogue(std::false_type{}, std::false_type{});
  }
}
#define SPHINX_GEMM_DMA_KERNEL(NAME, EPI, BM, EH)                                                            \
  __global__ __launch_bounds__(256, 2) void NAME(const bf16* __restrict__ A, const bf16* __restrict__ W,          \
                                                 const bf16* __restrict__ bias, int M, int N, int K, GemmEpi e) {  \
    __shared__ __attribute__((aligned(1024))) unsigned char smem[DmaCfg<BM, 128, 2, EH>::SMEM];                   \
    int m0, n0;                                                                                                  \
    grid_tile<BM, 128>(M, N, m0, n0);                                                                               \
    gemm_dma_body<EPI, BM, 128, 2, EH>(A, W, bias, M, N, K, e, smem, m0, n0);                                    \
  }
SPHINX_GEMM_DMA_KERNEL(k_gemm_dma_bias, EPI_BIAS, 128, 1)
SPHINX_GEMM_DMA_KERNEL(k_gemm_dma_gelu, EPI_GELU, 128, 1)
SPHINX_GEMM_DMA_KERNEL(k_gemm_dma_gated, EPI_GATED, 128, 1)
// 192-row tiles (wave tiles 96x64, epilogue in two halves; 80 KB of LDS, so
// still two workgroups per CU): fewer tiles for the same M, and 5/6 of the
// LDS reads per MFMA of the 128-row tile
SPHINX_GEMM_DMA_KERNEL(k_gemm_dma192_bias, EPI_BIAS, 192, 2)
SPHINX_GEMM_DMA_KERNEL(k_gemm_dma192_gelu, EPI_GELU, 192, 2)
SPHINX_GEMM_DMA_KERNEL(k_gemm_dma192_gated, EPI_GATED, 192, 2)
#undef SPHINX_GEMM_DMA_KERNEL

// BM-row tiles (64, 128, 192 or 256) with a ring of NS stages (4 x 24 KB,
// 4 x 32 KB, 4 x 40 KB or 3 x 48 KB of LDS, so one workgroup per CU), for
// launches whose tiles all fit on the CUs at once.  A lone workgroup waits out
// the copy latency of every K step when only the next stage is in flight; here
// NS - 1 are.  Eight waves of 32x32, 64x32, 96x32 or 128x32 (two per SIMD), so
// that each SIMD has a second wave to issue while one waits.  Same results as
// the other tiles.
template <int EPI, int NS, int BM = 128>
__global__ __launch_bounds__(512, 1) void k_gemm_dma_deep(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                          const bf16* __restrict__ bias, int M, int N, int K,
                                                          GemmEpi e) {
  constexpr int EH = BM <= 128 ? 1 : 2;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DmaCfg<BM, 128, NS, EH, 8>::SMEM];
  int m0, n0;
  grid_tile<BM, 128>(M, N, m0, n0);
  gemm_dma_body<EPI, BM, 128, NS, EH, 8>(A, W, bias, M, N, K, e, smem, m0, n0);
}

// Mixed row tiles: nb 192-row and ns 128-row tiles per column tile.  Same
// results as either tile.
//  * Narrow outputs (at most 8 column tiles) that fit in one round of two
//    workgroups per CU: XCD x takes the row band [x B, (x+1) B),
//    B = 192 nb + 128 ns, with all column tiles; its first nb * nt workgroups
//    (at most one per CU) are the 192-row ones.  With only 192-row tiles a CU
//    can hold two of them (384 rows) while others hold one; here a CU holds at
//    most 192 + 128 rows.
//  * Wide outputs: column-fastest order (XCD x keeps the column tiles
//    n = x mod 8), the 192-row tiles first and the 128-row ones last, so that
//    the last round is made of the smaller tiles.
template <int EPI, bool WIDE>
__global__ __launch_bounds__(256, 2) void k_gemm_dma_mix(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                         const bf16* __restrict__ bias, int M, int N, int K,
                                                         GemmEpi e, int nb, int ns) {
  constexpr int S192 = DmaCfg<192, 128, 2, 2>::SMEM, S128 = DmaCfg<128, 128, 2, 1>::SMEM;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S192 > S128 ? S192 : S128];
  const int nt = N / 128;
  if constexpr (WIDE) {  // nb row tiles of 192 rows, then ns of 128, column-fastest
    const int k = (int)blockIdx.x;
    if (k < nb * nt) {
      gemm_dma_body<EPI, 192, 128, 2, 2>(A, W, bias, M, N, K, e, smem, (k / nt) * 192, (k % nt) * 128);
    } else {
      const int j = k - nb * nt;
      const int m0 = 192 * nb + (j / nt) * 128;
      if (m0 < M) gemm_dma_body<EPI, 128, 128, 2, 1>(A, W, bias, M, N, K, e, smem, m0, (j % nt) * 128);
    }
  } else {  // XCD bands
    const int x = (int)blockIdx.x & 7, k = (int)blockIdx.x >> 3;
    const int band = x * (192 * nb + 128 * ns);
    if (k < nb * nt) {
      const int m0 = band + (k / nt) * 192;
      if (m0 < M) gemm_dma_body<EPI, 192, 128, 2, 2>(A, W, bias, M, N, K, e, smem, m0, (k % nt) * 128);
    } else {
      const int j = k - nb * nt;
      const int m0 = band + 192 * nb + (j / nt) * 128;
      if (m0 < M) gemm_dma_body<EPI, 128, 128, 2, 1>(A, W, bias, M, N, K, e, smem, m0, (j % nt) * 128);
    }
  }
}
// ---------------------------------------------------------------------------
// Tall tiles: 32 TI rows (TI 3 .. 8) x BN columns (192 or 256), one eight-wave
// workgroup per CU.
//  * Waves in 2x4, each 16 TI x BN/4 outputs; two stages of 64-deep K steps.
//  * A tile's worth is its bytes moved per FLOP: 256x256 copies 3/5 of the bytes
//    of 192x128 from L2 to LDS and reads 9/10 of the fragment bytes.  In the
//    headline step these kernels issue MFMAs at 44 % (QKV) and 43 % (MLP1) of the
//    register-only rate at about 2.4 GHz; in streams of equal launches the clock
//    falls (1.7-1.8 GHz), and fewer bytes help there as well.
//    Rows of 128 bytes matter as well: half-line (64-byte) copies ran at half
//    the L2 rate (1256 instead of 1115 cycles per 1024 of MFMA work).
//  * Row i of a k-step (TJ MFMAs on fa[i]) is followed by the read of the next
//    k-step's fa[i - 1], so one register set of A fragments serves both
//    k-steps and only the W fragments are doubled; with both doubled the
//    256-row tile spills.
//  * The workgroup barrier stands two rows into the second k-step: by then the
//    last fragments of the stage, read one row earlier, have arrived, and the
//    copies of stage kt+2 have half a stage of MFMAs and more to land.
//  * The epilogue needs no LDS: lanes l and l^16 exchange halves of two column
//    blocks so that each stores 16 bytes, 64 contiguous bytes of a row per four
//    lanes; the fp32 residual is read and written in 16-byte pieces the same way.
// Against the two-per-CU tiles, streams of equal launches: M 9677, K 1024, N 3072
// 65 -> 58 us and N 4096 88 -> 79; M 30925, N 1024, K 4096 (gated) 301 -> 241.
// Every output starts at its bias and adds its products in ascending k, as in
// the other tiles: same results, as described there.
template <int EPI, int TI, int BN>
__device__ __forceinline__ void gemm_tall_body(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                               const bf16* __restrict__ bias, int M, int K, const GemmEpi& e,
                                               unsigned char* smem, int m0, int n0) {
  constexpr int BM = 32 * TI, TJ = BN / 64, STAGE = (BM + BN) * 128;
  constexpr int NC = (BM + BN) / 8, COPIES = (NC + 7) / 8;  // 8-row copies per stage, and per wave
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3, g = lane >> 4, r16 = lane & 15;
  // copy c of this wave fills rows 8q .. 8q+7 of the stage (A rows, then W
  // rows), q = 8c + wave; the last one only where q < NC
  const bf16* src[COPIES];
  uint32_t voff[COPIES];
#pragma unroll
  for (int c = 0; c < COPIES; ++c) {
    const int q = 8 * c + wave, row = 8 * q + (lane >> 3);
    const int ch = (lane & 7) ^ ((row >> 1) & 7);
    if (8 * q < BM) {
      src[c] = A;
      voff[c] = 2u * (uint32_t)(min(m0 + row, M - 1) * K + ch * 8);
    } else {
      src[c] = W;
      voff[c] = 2u * (uint32_t)((n0 + min(row - BM, BN - 1)) * K + ch * 8);
    }
  }
  auto copy = [&](int kt, int slot, int c) {
    if (NC % 8 == 0 || c + 1 < COPIES || wave < NC % 8)
      lds_dma16_at(src[c] + kt * 64, voff[c], smem + slot * STAGE + (8 * c + wave) * 1024);
  };
  int foff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) foff[ks] = r16 * 128 + (((4 * ks + g) ^ ((r16 >> 1) & 7)) << 4);
  const int a0 = wm * 16 * TI, b0 = wn * 16 * TJ;
  // transposed output blocks: lane l holds row a0 + 16 i + l%16 and columns
  // b0 + 16 j + 4(l/16) .. + 3
  f32x4 acc[TI][TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(bias + n0 + b0 + j * 16 + 4 * g);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < TI; ++i) acc[i][j][t] = (float)b4[t];
  }
  const int KT = K / 64;  // even (K is a multiple of 128)
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int c = 0; c < COPIES; ++c) copy(st, st, c);
  // stage 0 must land (a wave with one copy less per stage waits for one more)
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(NC % 8 == 0 ? COPIES : COPIES - 1));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  bf16x8 fa[2][TI], fb[2][TJ];
  // fragment r of a k-step: the TJ of W first, then the TI of A
  auto read = [&](int slot, int ks, int r) {
    const unsigned char* st = smem + slot * STAGE + foff[ks];
    if (r < TJ) fb[ks][r] = *reinterpret_cast<const bf16x8*>(st + (BM + b0 + 16 * r) * 128);
    else fa[ks][r - TJ] = *reinterpret_cast<const bf16x8*>(st + (a0 + 16 * (r - TJ)) * 128);
  };
  auto row = [&](int ks, int i) {
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int LAST = TJ + TI - 1;       // A fragment TI - 1, read at the start of its own k-step
  constexpr int BR = TI >= 6 ? 2 : 1;     // rows of the second k-step before the barrier
  constexpr int RR = TI - BR;             // and after it
  auto step = [&](int kt, auto SLOT) {
    constexpr int s = decltype(SLOT)::value;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      if (i == 0) read(s, 0, LAST);
      if (i < TJ) read(s, 1, i);
      if (i >= 1) read(s, 1, TJ + i - 1);
      if (TI < TJ && i + 1 == TI) read(s, 1, TJ - 1);
      row(0, i);
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      if (i == 0) read(s, 1, LAST);
      if (i == BR) {
        // stage kt+1 has landed, and every wave has read all of stage kt
        __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      if (i >= BR) {
        // copies first; the last stages are refilled with the last one, which
        // is not read again, so that the loop has no branch (one makes the
        // 256-row tile spill)
        constexpr int CR = RR > 1 ? RR - 1 : 1;
#pragma unroll
        for (int c = 0; c < COPIES; ++c)
          if (c * CR / COPIES == i - BR) copy(min(kt + 2, KT - 1), s, c);
        // the next stage's first k-step over the rows left; fa[r] not before row r + 1
#pragma unroll
        for (int r = 0; r < LAST; ++r) {
          const int even = r * RR / LAST, after = r - TJ + 1 - BR;
          if ((even > after ? even : after) == i - BR) read(s ^ 1, 0, r);
        }
      }
      row(1, i);
    }
  };
#pragma unroll
  for (int r = 0; r < LAST; ++r) read(0, 0, r);
  for (int kt = 0; kt < KT; kt += 2) {
    step(kt, std::integral_constant<int, 0>{});
    step(kt + 1, std::integral_constant<int, 1>{});
  }
  // the refills of the last stages must land while the workgroup holds its LDS
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
  const bool qtile = EPI == EPI_BIAS && n0 < e.qcols;  // a column tile is all queries or none (launch rule)
  if constexpr (EPI == EPI_GATED) {
    int cr[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i) cr[i] = e.crow[min(m0 + a0 + 16 * i + r16, M - 1)];
    const int cr0 = __builtin_amdgcn_readfirstlane(cr[0]);
    bool same = true;
#pragma unroll
    for (int i = 0; i < TI; ++i) same = same && cr[i] == cr0;
    float* hb = static_cast<float*>(e.out) + n0 + b0 + 4 * g;
    const float* gb = e.gate + n0 + b0 + 4 * g;
    // residual loads run PD rows ahead of the stores (issued row by row, each
    // would wait out a memory latency behind the previous row's stores)
    constexpr int PD = TI < 4 ? TI : 4;
    auto rows = [&](auto SAME) {
      f32x4 g0[TJ], h[PD][TJ];
      auto load = [&](int i) {
        const float* hr = hb + (int64_t)min(m0 + a0 + 16 * i + r16, M - 1) * e.ldo;
#pragma unroll
        for (int j = 0; j < TJ; ++j) h[i % PD][j] = *reinterpret_cast<const f32x4*>(hr + 16 * j);
      };
#pragma unroll
      for (int i = 0; i < PD; ++i) load(i);
      if constexpr (decltype(SAME)::value)
#pragma unroll
        for (int j = 0; j < TJ; ++j) g0[j] = *reinterpret_cast<const f32x4*>(gb + (int64_t)cr0 * e.ldg + 16 * j);
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const int m = m0 + a0 + 16 * i + r16;
        f32x4 gv[TJ];
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          if constexpr (decltype(SAME)::value) gv[j] = g0[j];
          else gv[j] = *reinterpret_cast<const f32x4*>(gb + (int64_t)cr[i] * e.ldg + 16 * j);
        }
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          f32x4 v;
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = fmaf(1.0f + gv[j][t], acc[i][j][t], h[i % PD][j][t]);
          if (m < M) *reinterpret_cast<f32x4*>(hb + (int64_t)m * e.ldo + 16 * j) = v;
        }
        if (i + PD < TI) load(i + PD);
      }
    };
    // one conditioning row for the wave's rows (frames on one timestep): its gate is read once
    if (__ballot(same) == ~0ull) rows(std::true_type{});
    else rows(std::false_type{});
  } else {
    bf16* ob = static_cast<bf16*>(e.out) + n0 + b0;
    const float qs = qtile ? e.qscale : 1.0f;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      const int m = m0 + a0 + 16 * i + r16;
      bf16* orow = ob + (int64_t)m * e.ldo;
      uint2 p[TJ];
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        bf16x4 o;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          float v = acc[i][j][t];
          if constexpr (EPI == EPI_GELU) v = gelu_tanh(v);
          if constexpr (EPI == EPI_BIAS) v = qtile ? v * qs : v;
          o[t] = (bf16)v;
        }
        p[j] = __builtin_bit_cast(uint2, o);
      }
      // columns 16 j .. 16 j + 31 in pairs of blocks: rows of 16 lanes 0, 2 end
      // up with 8 columns of block j, rows 1, 3 with 8 of block j + 1
#pragma unroll
      for (int j = 0; j + 1 < TJ; j += 2) {
        const auto x = __builtin_amdgcn_permlane16_swap(p[j].x, p[j + 1].x, false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(p[j].y, p[j + 1].y, false, false);
        const uint4 v = make_uint4(x[0], y[0], x[1], y[1]);
        if (m < M) *reinterpret_cast<uint4*>(orow + 16 * j + 16 * (g & 1) + 8 * (g >> 1)) = v;
      }
      if constexpr (TJ % 2 == 1)
        if (m < M) *reinterpret_cast<uint2*>(orow + 16 * (TJ - 1) + 4 * g) = p[TJ - 1];
    }
  }
}

// n1 row tiles of 32 t1 rows, then n2 of 32 t2 rows, each with all N / BN
// column tiles.  Each part's tiles are dealt to the XCDs in contiguous ranges
// of panels four row tiles high, column by column inside a panel, so that the
// tiles an XCD runs at a time share few rows of A and of W in its L2 (M 30925,
// N 4096, K 1024: 268 us in plain order, 227 in panels).
template <int EPI, int BN>
__global__ __launch_bounds__(512, 2) void k_gemm_tall(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                      const bf16* __restrict__ bias, int M, int N, int K, GemmEpi e,
                                                      TallPlan p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * (256 + BN) * 128];
  const int nt = N / BN, first = p.n1 * nt;
  const bool two = (int)blockIdx.x >= first;
  const int rt = two ? p.n2 : p.n1, ti = two ? p.t2 : p.t1;
  const int tile = xcd_tile((int)blockIdx.x - (two ? first : 0), rt * nt);
  const int panel = tile / (4 * nt), rem = tile - panel * 4 * nt, ph = min(4, rt - 4 * panel);
  const int m0 = (two ? 32 * p.t1 * p.n1 : 0) + (4 * panel + rem % ph) * 32 * ti, n0 = (rem / ph) * BN;
  switch (ti) {
    case 3: gemm_tall_body<EPI, 3, BN>(A, W, bias, M, K, e, smem, m0, n0); break;
    case 4: gemm_tall_body<EPI, 4, BN>(A, W, bias, M, K, e, smem, m0, n0); break;
    case 5: gemm_tall_body<EPI, 5, BN>(A, W, bias, M, K, e, smem, m0, n0); break;
    case 6: gemm_tall_body<EPI, 6, BN>(A, W, bias, M, K, e, smem, m0, n0); break;
    case 7: gemm_tall_body<EPI, 7, BN>(A, W, bias, M, K, e, smem, m0, n0); break;
    default: gemm_tall_body<EPI, 8, BN>(A, W, bias, M, K, e, smem, m0, n0); break;
  }
}
}  // namespace dma

// fp32 GEMM on v_mfma_f32_32x32x2_f32 (64 cycles for a wave's 32x32x2), N and K
// multiples of 64.  MFMA-bound, so what matters is that small selections reach
// every SIMD: workgroup tile 32x64 in four waves, two 32x32 column blocks times
// two halves of each 64-deep K step (wave kh takes chunks 8 kh .. 8 kh + 7),
// the halves added through LDS at the end.  1024 selected tokens at D 512 then
// give 256 workgroups for the narrow outputs; 64x64 tiles gave 128.
//  * Operand rows of one K step are 256 bytes, copied global->LDS directly;
//    16-byte chunk c of row r sits at c ^ (r & 15), so the 16 rows of a read
//    pass (same chunk) fall on 16 different bank groups.  A lane's chunk feeds
//    four k-steps (the contraction order is free, and the same on both sides).
//  * K steps live in a three-slot ring (72 KB of LDS, two workgroups per CU):
//    at each step the copies of the newest one stay in flight.
//  * Row bases are wave-uniform 64-bit addresses; a lane's offset spans at most
//    four rows, so activations of any size the caller accepts are addressable.
// Each output is bias + first halves + second halves in ascending K, whatever
// the launch, so packed and separate requests round alike.  Against a 64x64
// tile of scalar multiply-adds, at 1024 rows: QKV 75.7 -> 27.0 us, MLP1 75.2 ->
// 28.3, out-projection and MLP2 162 -> 23.8 on average.
constexpr int kF32BM = 32, kF32BN = 64, kF32BK = 64, kF32NS = 3;
template <int EPI>
__global__ __launch_bounds__(256, 2) void k_gemm_f32(const float* __restrict__ A, const float* __restrict__ W,
                                                     const float* __restrict__ bias, int M, int N, int K, GemmEpi e) {
  constexpr int ROWS = kF32BM + kF32BN, STAGE = ROWS * 256, COPIES = ROWS / 4 / 4, CLD = kF32BN + 4;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kF32NS * STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave & 1, kh = wave >> 1, g = lane >> 5, r32 = lane & 31;
  const int nt = N / kF32BN;
  const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
  const int m0 = (tile / nt) * kF32BM, n0 = (tile % nt) * kF32BN;
  const float* src[COPIES];
  uint32_t voff[COPIES];
#pragma unroll
  for (int i = 0; i < COPIES; ++i) {
    const int q = wave * COPIES + i, row = 4 * q + (lane >> 4);  // copy q fills rows 4q .. 4q+3 of the stage
    const int c = (lane & 15) ^ (row & 15);
    int up = lane >> 4;  // rows above the copy's base row; rows past M repeat row M - 1
    if (4 * q < kF32BM) {
      const int base = min(m0 + 4 * q, M - 1);
      up = min(up, M - 1 - base);
      src[i] = A + (int64_t)base * K;
    } else {
      src[i] = W + (int64_t)(n0 + 4 * q - kF32BM) * K;
    }
    voff[i] = 4u * (uint32_t)(up * K + c * 4);
  }
  const int KT = K / kF32BK;
  auto copy_stage = [&](int kt, int slot) {
#pragma unroll
    for (int i = 0; i < COPIES; ++i)
      lds_dma16_at(src[i] + (int64_t)kt * kF32BK, voff[i], smem + slot * STAGE + (wave * COPIES + i) * 1024);
  };
  f32x16 acc = {};
  if (kh == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + n0 + wn * 32 + 8 * q + 4 * g);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[4 * q + t] = b4[t];
    }
  }
  copy_stage(0, 0);
  copy_stage(min(1, KT - 1), 1);
  int slot = 0;
  for (int kt = 0; kt < KT; ++kt) {
    // step kt has landed (only step kt + 1 may be in flight) and every wave has
    // read step kt - 1, whose slot the copies of step kt + 2 refill (near the
    // end with the last step again, so that every wait counts the same)
    __builtin_amdgcn_s_waitcnt(dma::wait_vm_lgkm0(COPIES));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    copy_stage(min(kt + 2, KT - 1), slot == 0 ? kF32NS - 1 : slot - 1);
    const unsigned char* a = smem + slot * STAGE + r32 * 256;
    const unsigned char* b = a + (kF32BM + wn * 32) * 256;
    f32x4 fa[4], fb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = ((8 * kh + 2 * j + g) ^ (r32 & 15)) << 4;
      fa[j] = *reinterpret_cast<const f32x4*>(a + o);
      fb[j] = *reinterpret_cast<const f32x4*>(b + o);
    }
    // transposed block: lane l holds row l % 32 and, in registers 4q .. 4q+3,
    // columns 8q + 4 (l / 32) .. + 3
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j][t], fa[j][t], acc, 0, 0, 0);
    slot = slot + 1 == kF32NS ? 0 : slot + 1;
  }
  __builtin_amdgcn_s_waitcnt(dma::wait_vm_lgkm0(0));
  asm volatile("" ::: "memory");
  __syncthreads();
  float* sC = reinterpret_cast<float*>(smem);
  float* srow = sC + r32 * CLD + wn * 32 + 4 * g;
  if (kh == 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<f32x4*>(srow + 8 * q) = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
  }
  __syncthreads();
  if (kh == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v = *reinterpret_cast<const f32x4*>(srow + 8 * q);
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] += acc[4 * q + t];
      *reinterpret_cast<f32x4*>(srow + 8 * q) = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int r = 16 * p + (tid >> 4), c = (tid & 15) * 4, m = m0 + r;
    if (m >= M) continue;
    f32x4 v = *reinterpret_cast<const f32x4*>(sC + r * CLD + c);
    float* o = reinterpret_cast<float*>(e.out) + (int64_t)m * e.ldo + n0 + c;
    if constexpr (EPI == EPI_GATED) {
      const f32x4 gv = *reinterpret_cast<const f32x4*>(e.gate + (int64_t)e.crow[m] * e.ldg + n0 + c);
      const f32x4 hv = *reinterpret_cast<const f32x4*>(o);
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = fmaf(1.0f + gv[t], v[t], hv[t]);
    } else if constexpr (EPI == EPI_GELU) {
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = gelu_tanh(v[t]);
    } else if (n0 < e.qcols) {  // a column tile is all queries or none (qcols is a multiple of 64)
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] *= e.qscale;
    }
    *reinterpret_cast<f32x4*>(o) = v;
  }
}
// Calibration loop: four independent 32x32x16 bf16 MFMA chains per wave.
// MFMA calibration loop; RANDOM: operands are hashed random bf16 in [-2, 2),
// eight (A, B) pairs used in rotation.
__device__ __forceinline__ float peak_rand(unsigned x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return (float)(x & 0xffffu) * (4.0f / 65536.0f) - 2.0f;
}

template <bool RANDOM>
__global__ __launch_bounds__(256) void k_peak_mfma(int iters, float* __restrict__ out) {
  constexpr int NS = RANDOM ? 8 : 1;
  const unsigned t = blockIdx.x * 256u + threadIdx.x;
  bf16x8 a[NS], b[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      a[s][i] = RANDOM ? (bf16)peak_rand(t * 64u + s * 8u + i) : (bf16)(1e-3f * (float)((threadIdx.x + i) & 15));
      b[s][i] = RANDOM ? (bf16)peak_rand(0x9e3779b9u ^ (t * 64u + s * 8u + i)) : (bf16)(1e-3f * (float)(i + 1));
    }
  f32x16 c0 = f32x16{}, c1 = f32x16{}, c2 = f32x16{}, c3 = f32x16{};
  // one round: four MFMAs on operand pairs s..s+3 (static register indices)
  auto round = [&](auto sc) {
    constexpr int s = decltype(sc)::value;
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s % NS], b[(s + 1) % NS], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[(s + 1) % NS], b[(s + 2) % NS], c1, 0, 0, 0);
    c2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[(s + 2) % NS], b[(s + 3) % NS], c2, 0, 0, 0);
    c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[(s + 3) % NS], b[s % NS], c3, 0, 0, 0);
  };
  int it = 0;
  for (; it + 1 < iters; it += 2) {
    round(std::integral_constant<int, 0>{});
    round(std::integral_constant<int, 4>{});
  }
  if (it < iters) round(std::integral_constant<int, 0>{});
  float sum = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) sum += c0[r] + c1[r] + c2[r] + c3[r];
  sum = wave_sum(sum);
  if (threadIdx.x == 0) out[blockIdx.x] = sum;
}
}  // namespace

namespace {
// Compute units of the current device (cached per device; 256 if unknown).
int cu_count() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int c = cache[dev].load(std::memory_order_relaxed);
  if (c <= 0) {
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) c = 256;
    cache[dev].store(c, std::memory_order_relaxed);
  }
  return c;
}

void launch_tall(int epi, int bn, const TallPlan& p, const bf16* a, const bf16* w, const bf16* b, int M, int N, int K,
                 const GemmEpi& e, hipStream_t s) {
  const int grid = (p.n1 + p.n2) * (N / bn);
  auto go = [&](auto E, auto BN) {
    dma::k_gemm_tall<decltype(E)::value, decltype(BN)::value><<<grid, 512, 0, s>>>(a, w, b, M, N, K, e, p);
  };
  auto by_bn = [&](auto E) {
    if (bn == 256) go(E, std::integral_constant<int, 256>{});
    else go(E, std::integral_constant<int, 192>{});
  };
  if (epi == EPI_BIAS) by_bn(std::integral_constant<int, EPI_BIAS>{});
  else if (epi == EPI_GELU) by_bn(std::integral_constant<int, EPI_GELU>{});
  else by_bn(std::integral_constant<int, EPI_GATED>{});
}

// One eight-wave workgroup per BM-row tile with an NS-stage ring.
template <int NS, int BM>
void launch_deep(int epi, int tiles, const bf16* a, const bf16* w, const bf16* b, int M, int N, int K,
                 const GemmEpi& e, hipStream_t s) {
  if (epi == EPI_BIAS) dma::k_gemm_dma_deep<EPI_BIAS, NS, BM><<<tiles, 512, 0, s>>>(a, w, b, M, N, K, e);
  else if (epi == EPI_GELU) dma::k_gemm_dma_deep<EPI_GELU, NS, BM><<<tiles, 512, 0, s>>>(a, w, b, M, N, K, e);
  else dma::k_gemm_dma_deep<EPI_GATED, NS, BM><<<tiles, 512, 0, s>>>(a, w, b, M, N, K, e);
}

// 192- and 128-row tiles in one grid: p.nb and p.ns row tiles of each.
template <bool WIDE>
void launch_mix(int epi, int tiles, const GemmPlan& p, const bf16* a, const bf16* w, const bf16* b, int M, int N,
                int K, const GemmEpi& e, hipStream_t s) {
  if (epi == EPI_BIAS) dma::k_gemm_dma_mix<EPI_BIAS, WIDE><<<tiles, 256, 0, s>>>(a, w, b, M, N, K, e, p.nb, p.ns);
  else if (epi == EPI_GELU) dma::k_gemm_dma_mix<EPI_GELU, WIDE><<<tiles, 256, 0, s>>>(a, w, b, M, N, K, e, p.nb, p.ns);
  else dma::k_gemm_dma_mix<EPI_GATED, WIDE><<<tiles, 256, 0, s>>>(a, w, b, M, N, K, e, p.nb, p.ns);
}
}  // namespace

hipError_t launch_gemm(int epi, sphinx_dtype dt, const void* A, const void* W, const void* bias, int M, int N, int K,
                       const GemmEpi& e, hipStream_t s) {
  if (dt == SPHINX_BF16) {
    // the K loop takes two 64-deep steps at a time; the query scale is applied per 128-column tile
    if (K % 128 != 0 || N % 128 != 0 || (epi == EPI_BIAS && e.qcols % 128 != 0)) return hipErrorInvalidValue;
    const bf16 *a = (const bf16*)A, *w = (const bf16*)W, *b = (const bf16*)bias;
    const GemmPlan p = plan_gemm(epi == EPI_GATED, epi == EPI_BIAS ? e.qcols : 0, M, N, K, cu_count());
    const int nt = N / 128, t128 = nt * ((M + 127) / 128), t192 = nt * ((M + 191) / 192);
    switch (p.tiles) {
      case kDeep64: launch_deep<4, 64>(epi, nt * ((M + 63) / 64), a, w, b, M, N, K, e, s); break;
      case kDeep128: launch_deep<4, 128>(epi, t128, a, w, b, M, N, K, e, s); break;
      case kDeep192: launch_deep<4, 192>(epi, t192, a, w, b, M, N, K, e, s); break;
      case kDeep256: launch_deep<3, 256>(epi, nt * ((M + 255) / 256), a, w, b, M, N, K, e, s); break;
      case kTall: launch_tall(epi, p.bn, p.tall, a, w, b, M, N, K, e, s); break;
      case kMixWide: launch_mix<true>(epi, (p.nb + p.ns) * nt, p, a, w, b, M, N, K, e, s); break;
      case kMixNarrow: launch_mix<false>(epi, 8 * (p.nb + p.ns) * nt, p, a, w, b, M, N, K, e, s); break;
      case kPair192:
        if (epi == EPI_BIAS) dma::k_gemm_dma192_bias<<<t192, 256, 0, s>>>(a, w, b, M, N, K, e);
        else if (epi == EPI_GELU) dma::k_gemm_dma192_gelu<<<t192, 256, 0, s>>>(a, w, b, M, N, K, e);
        else dma::k_gemm_dma192_gated<<<t192, 256, 0, s>>>(a, w, b, M, N, K, e);
        break;
      default:
        if (epi == EPI_BIAS) dma::k_gemm_dma_bias<<<t128, 256, 0, s>>>(a, w, b, M, N, K, e);
        else if (epi == EPI_GELU) dma::k_gemm_dma_gelu<<<t128, 256, 0, s>>>(a, w, b, M, N, K, e);
        else dma::k_gemm_dma_gated<<<t128, 256, 0, s>>>(a, w, b, M, N, K, e);
    }
  } else {
    if (K % kF32BK != 0 || N % kF32BN != 0 || (epi == EPI_BIAS && e.qcols % kF32BN != 0)) return hipErrorInvalidValue;
    const int grid = (N / kF32BN) * ((M + kF32BM - 1) / kF32BM);
    const float *a = (const float*)A, *w = (const float*)W, *b = (const float*)bias;
    if (epi == EPI_BIAS) k_gemm_f32<EPI_BIAS><<<grid, 256, 0, s>>>(a, w, b, M, N, K, e);
    else if (epi == EPI_GELU) k_gemm_f32<EPI_GELU><<<grid, 256, 0, s>>>(a, w, b, M, N, K, e);
    else k_gemm_f32<EPI_GATED><<<grid, 256, 0, s>>>(a, w, b, M, N, K, e);
  }
  return hipGetLastError();
}

hipError_t launch_peak_mfma(int iters, bool random, float* out, int blocks, hipStream_t s) {
  if (random)
    k_peak_mfma<true><<<blocks, 256, 0, s>>>(iters, out);
  else
    k_peak_mfma<false><<<blocks, 256, 0, s>>>(iters, out);
  return hipGetLastError();
}

}  // namespace sphinx
