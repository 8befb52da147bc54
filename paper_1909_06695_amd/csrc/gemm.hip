// Dense contractions of the training step: the choice between the direct-to-LDS MFMA kernels (gemm_pp.hip, gemm_dlds.hip;
// fp32: gemm_f32.hip), a register-staged bf16 MFMA kernel (LDS double-buffered, XOR-swizzled tiles, 32x32x16 matrix
// instructions) and a plain bounds-checked tiled kernel for what those do not take.
#include "gemm_common.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <utility>

namespace ouro {

// ------------------------------------------------------------------ plain tiled kernel
template <typename T, bool TA, bool TB>
__global__ __launch_bounds__(256) void gemm_plain_kernel(GemmParams p) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Bs[BK][BN + 4];
  const T* A = reinterpret_cast<const T*>(p.A);
  const T* B = reinterpret_cast<const T*>(p.B);
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int kbeg = blockIdx.z * p.kchunk;
  const int kend = min(p.K, kbeg + p.kchunk);
  const int tx = tid % 16, ty = tid / 16;
  float acc[4][4] = {};
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int e = tid + i * 256;                 // 0..1023
      int mm, kk;
      if (TA) { mm = e % BM; kk = e / BM; } else { kk = e % BK; mm = e / BK; }
      int gm = m0 + mm, gk = k0 + kk;
      float v = 0.f;
      if (gm < p.M && gk < kend) v = to_f32(TA ? A[(size_t)gk * p.lda + gm] : A[(size_t)gm * p.lda + gk]);
      As[kk][mm] = v;
      int nn, kb;
      if (TB) { kb = e % BK; nn = e / BK; } else { nn = e % BN; kb = e / BN; }
      int gn = n0 + nn; gk = k0 + kb;
      v = 0.f;
      if (gn < p.N && gk < kend) v = to_f32(TB ? B[(size_t)gn * p.ldb + gk] : B[(size_t)gk * p.ldb + gn]);
      Bs[kb][nn] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; b[i] = Bs[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
      if (m < p.M && n < p.N) epilogue_store<T>(p, m, n, acc[i][j]);
    }
}

// ------------------------------------------------------------------------- MFMA kernel
template <int BM, int BN, int WM, int WN, bool TA, bool TB>
__global__ __launch_bounds__(WM * WN * 64) void gemm_mfma_kernel(GemmParams p) {
  constexpr int BK = 64;
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int STAGE = (BM + BN) * 8;                      // uint4 per stage
  constexpr int RA = TA ? (16 * (BM / 8) / NT) * 4 : BM * 8 / NT;
  constexpr int RB = TB ? BN * 8 / NT : (16 * (BN / 8) / NT) * 4;
  extern __shared__ uint4 smem[];
  const bf16_t* A = reinterpret_cast<const bf16_t*>(p.A);
  const bf16_t* B = reinterpret_cast<const bf16_t*>(p.B);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  // spread consecutive tiles of one matrix band over one XCD (blocks go round-robin
  // over the 8 XCDs, each with its own L2)
  int bid = blockIdx.x;
  {
    int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = bid & 7, idx = bid >> 3;
    bid = x * q + min(x, r) + idx;
  }
  const int m0 = (bid / p.tilesN) * BM, n0 = (bid % p.tilesN) * BN;
  const int kbeg = blockIdx.z * p.kchunk;
  const int kend = min(p.K, kbeg + p.kchunk);
  const int nk = (kend - kbeg + BK - 1) / BK;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  uint4 ra[RA], rb[RB];
  auto gload = [&](int kt) {
    int k0 = kbeg + kt * BK;
    if (TA) load_colform<BM, NT>(A, p.lda, m0, p.M, k0, kend, tid, ra);
    else load_rowform<BM, NT>(A, p.lda, m0, p.M, k0, kend, tid, ra);
    if (TB) load_rowform<BN, NT>(B, p.ldb, n0, p.N, k0, kend, tid, rb);
    else load_colform<BN, NT>(B, p.ldb, n0, p.N, k0, kend, tid, rb);
  };
  auto sstore = [&](int stage) {
    uint4* sa = smem + stage * STAGE;
    uint4* sb = sa + BM * 8;
    if (TA) store_colform<BM, NT>(sa, tid, ra); else store_rowform<BM, NT>(sa, tid, ra);
    if (TB) store_rowform<BN, NT>(sb, tid, rb); else store_colform<BN, NT>(sb, tid, rb);
  };

  if (nk > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    if (more) gload(kt + 1);
    const uint4* sa = smem + (kt & 1) * STAGE;
    const uint4* sb = sa + BM * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      bf16x8 af[TM], bfr[TN];
      const int c = ks * 2 + (lane >> 5);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        int row = wm * (TM * 32) + i * 32 + (lane & 31);
        uint4 t = sa[row * 8 + (c ^ swz(row))];
        af[i] = *reinterpret_cast<bf16x8*>(&t);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        int row = wn * (TN * 32) + j * 32 + (lane & 31);
        uint4 t = sb[row * 8 + (c ^ swz(row))];
        bfr[j] = *reinterpret_cast<bf16x8*>(&t);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (more) sstore((kt + 1) & 1);
    __syncthreads();
  }

  mfma_epilogue<TM, TN, false>(p, acc, smem, m0 + wm * (TM * 32), n0 + wn * (TN * 32), lane, wave);
}

// ----------------------------------------------------------------------------- launch
hipError_t launch_gemm_dlds(hipStream_t s, GemmParams& p, int transA, int transB, int splits, int cfg);
hipError_t launch_gemm_pp(hipStream_t s, GemmParams& p, int transA, int transB, int splits);
hipError_t launch_gemm_pp_group(hipStream_t s, const GemmParams* ps, int n);
bool gemm_f32_ok(const GemmDesc& g);
hipError_t launch_gemm_f32(hipStream_t s, GemmParams& p, int transA, int transB, int form);
bool gemm_f32_group_ok(const GemmParams& p);
hipError_t launch_gemm_f32_group(hipStream_t s, const GemmParams* ps, int n);
hipError_t launch_gemm_dlds_group(hipStream_t s, GemmParams* ps, int n, int transA, int transB);
static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

static inline bool direct_k_ok(int transA, int transB, int K) { return K % 64 == 0 || (transA && !transB); }

bool gemm_uses_mfma(int dtype, const GemmDesc& g) {
  if (dtype != 1) return false;
  if (!aligned16(g.A) || !aligned16(g.B)) return false;
  if ((g.lda & 7) || (g.ldb & 7)) return false;
  if (g.transA ? (g.M & 7) : (g.K & 7)) return false;
  if (g.transB ? (g.K & 7) : (g.N & 7)) return false;
  if (g.M < 32 || g.N < 32 || g.K < 32) return false;
  return true;
}

template <int BM, int BN, int WM, int WN>
static hipError_t launch_mfma_cfg(hipStream_t s, GemmParams& p, int transA, int transB, int splits) {
  constexpr size_t smem_main = 2 * (size_t)(BM + BN) * 8 * sizeof(uint4);
  constexpr size_t smem_epi = (size_t)WM * WN * epilogue_stage_floats<BN / WN / 32>() * sizeof(float);
  constexpr size_t smem = smem_main > smem_epi ? smem_main : smem_epi;
  int tilesM = (p.M + BM - 1) / BM;
  p.tilesN = (p.N + BN - 1) / BN;
  dim3 grid(tilesM * p.tilesN, 1, splits), block(WM * WN * 64);
#define OURO_LAUNCH(TA_, TB_)                                                                   \
  do {                                                                                          \
    static bool attr_done = false;                                                              \
    auto kern = gemm_mfma_kernel<BM, BN, WM, WN, TA_, TB_>;                                     \
    if (!attr_done) {                                                                           \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                   \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);\
      if (e != hipSuccess) return e;                                                            \
      attr_done = true;                                                                         \
    }                                                                                           \
    hipLaunchKernelGGL(kern, grid, block, smem, s, p);                                          \
  } while (0)
  if (!transA && !transB) OURO_LAUNCH(false, false);
  else if (!transA && transB) OURO_LAUNCH(false, true);
  else if (transA && !transB) OURO_LAUNCH(true, false);
  else OURO_LAUNCH(true, true);
#undef OURO_LAUNCH
  return hipGetLastError();
}

// Tile configuration and contraction ranges of a product (of each of `products` in a launch) on the MFMA kernels.
struct GemmPlan { int cfg, splits, kchunk; bool direct_ok; };
static bool plan_mfma(const GemmDesc& g, int force, long products, GemmPlan& plan) {
  int cfg = force >= 2 ? force : -1;
  if (cfg < 0) {
    // 128x128 tiles (8 waves, two workgroups per CU) when they fill the chip at least twice
    // over; with one tile per CU and a long contraction the register-prefetch kernel with its
    // four-stage ring; otherwise, and for the split-K weight gradients, 128x64 tiles, which
    // put more workgroups on every compute unit
    const int t128 = ((g.M + 127) / 128) * ((g.N + 127) / 128);
    const long one = (long)((g.M + 255) / 256) * ((g.N + 255) / 256);
    // the tiles of all products, unless they have more past the edges than 128x128 ones (90000 x 320 over 512 with GELU 63 us on 128-wide tiles,
    // 70 on 256x256; 131072 x 128 39 and 52; 16 products of 600 x 900 over 1024 49 and 51)
    const long t256 = 4 * one <= 1.15 * t128 ? one * products : 0;
    // 256x256 tiles (one workgroup per CU, nothing beside its epilogue) pay once there are four per CU (the logits: 8192 x
    // 32768 over 512 312 us, 4800 x 32768 over 448 190), one per CU with a long contraction (dV_o: 670 -> 592 us), or where their
    // rounds are well filled.  Alone on the chip, 128x128 and 256x256 tiles, us (plain / GELU / GELU-gradient / fp32 result with the
    // recomputed LayerNorm):
    //   one round      256 tiles over 1024 38 / 46 / 45 / 62 and 32 / 41 / 42 / 52; over 512 24 / 33 / 31 / 48 and 21 / 29 / 31 / 43;
    //                  192 over 768 27 / 33 / 32 / 40 and 24 / 32 / 33 / 39; 192 over 512 20 / 28 / 27 / 37 and 19 / 27 / 28 / 36;
    //                  190 over 448 20 / 27 / 26 / 34 and 18 / 26 / 27 / 34; 144 over 768 26 / 32 / 31 / 35 and 22 / 30 / 32 / 35
    //   1.1 to 1.3     288 over 1024 46 / 58 / 56 / 78 and 49 / 65 / 70 / 79; 320 over 1024 49 / 61 / 66 / 85 and 51 / 68 / 74 / 81
    //   1.5            384 over 1024 55 / 71 / 71 / 92 and 53 / 72 / 77 / 91; over 768 45 / 60 / 58 / 85 and 45 / 67 / 70 / 82;
    //                  plain: 384 over 448 31 and 32, over 512 34 and 35 (three whole rounds of 128x128 tiles); 392 over 448 34 and 31;
    //                  640 over 512 54 and 59 where the result is wider than high, else 56 and 54
    //   two            512 over 1024 80 / 109 / - / 126 and 60 / 79 / - / 122; over 512 44 / 76 / 71 / 102 and 42 / 61 / 72 / 102
    // and 416 over 1024 69 (GELU-gradient 82) and 63 (91), 464 over 768 75 and 57, 528 over 1024 89 (GELU-gradient) and 95.
    // The lower end, plain (the faster of the 128-wide forms and 256x256): 128 tiles over 512 / 768 / 1024 12.7 / 16.7 / 20.3 and 16.5 /
    // 20.5 / 23.8, 136 16.4 / 22.7 / 28.1 and 16.4 / 20.2 / 23.8, 144 17.2 / 22.8 / 27.7 and 16.9 / 20.8 / 24.6; 144 to 160 over 384 15.0 both,
    // over 448 16.0 both, 192 17.8 and 17.1.  What counts there is whether 128x128 tiles run in one round of 512: 9288 x 832 over 640 (148
    // tiles, 511 of 128x128) 16.9 and 19.5, 12288 x 576 over 960 19 and 24.
    // Two products of 144 tiles over 512 28.0 and 32.1 (288 in all, 1.1 rounds), four of 64 24.4 and 22.5.
    // Products of few tiles are bound by what each workgroup has in flight along its contraction: 64x64 tiles with a
    // four-stage ring, two workgroups per CU, while all of them run in one round.  Against the larger tiles: 768 x 1024
    // over 1024 11.7 -> 7.3 us, over 4096 30.5 -> 17.1; 2331 x 768 over 768 11.0 -> 9.1, over 3072 25.1 -> 21.7; 288 x 128
    // over 256 5.2 -> 4.5; beyond one round 768 x 4096 over 1024 16.7 -> 20.1, 4800 x 640 over 448 9.9 -> 10.4.
    // Not where they nearly fill the round, both sides are long and an operand is column-form: L2 is the limit then (A B, 1088 x
    // 1496 over 4096 32.8 us on the register-prefetch kernel, 35.9 on 64x64 tiles, over 8192 58 and 70; A B^T 57.9 and 57.1;
    // narrower, 448 x 4096 over 8192, 60 and 50; 198 tiles, 1348 x 528 over 7552, 56 and 30).
    const long t64 = (long)((g.M + 63) / 64) * ((g.N + 63) / 64) * products;
    const bool plain = !g.out_fp32 && g.epilogue == EPI_NONE && !g.residual && !g.res32;
    auto last = [](long t) { return (t + 255) % 256 + 1; };           // tiles of the last round
    // four per CU, one per CU over a long contraction, or a last round at least three quarters full: also where much of a tile is past the edge
    // (65536 x 160 over 4096 137 us, on 128-wide tiles 154)
    auto many = [&](long t, int k) { return t >= 1024 || (t >= 256 && g.K >= 4096) || (t >= 448 && last(t) >= 192 && g.K >= k); };
    const bool big = many(one, 768) || many(t256, plain || g.epilogue == EPI_GELU ? 512 : 768) ||
                     (t128 * products > 512 && t256 >= (plain ? 144 : 224) && t256 <= 256 && g.K >= (plain ? 448 : 512)) ||
                     (plain && t256 >= 384 && (g.K >= 768 ? last(t256) >= 128 : last(t256) > 128 && t128 * products > 1536 && g.K >= 448));
    const long t128x256 = (long)((g.M + 127) / 128) * ((g.N + 255) / 256) * products;
    const bool column = g.transA || !g.transB;
    if (!g.accumulate && t64 <= 512 && !(t64 > 384 && column && g.K >= 4096 && std::min(g.M, g.N) > 512)) cfg = GEMM_TILE_64x64;
    // One nearly full round of 128x256 tiles (64x64 a wave: a third less LDS traffic per matrix instruction than 128x128 tiles,
    // three stages) pays over a long contraction, as there is one workgroup per CU and nothing beside its epilogue.  Against
    // 128x128 tiles: 256 of them (8192 x 1024) over 4096 64.8 and 66.5 us, over 2048 35.7 and 36.2, over 1024 22.1 and 21.6; 192 over
    // 4096 54.9 and 54.1; 160 52.5 and 48.7.
    else if (!g.accumulate && g.K >= 2048 && t128x256 >= 224 && t128x256 <= 256) cfg = GEMM_TILE_128x256;
    else if (!g.accumulate && big) cfg = GEMM_TILE_256x256;
    else if (g.accumulate && t128 >= 192) cfg = GEMM_TILE_128x128;   // split-K with two workgroups per CU
    // 128x64 tiles up to three per CU, over a long contraction only up to two (320 128x128 tiles: over 4096 48.7 us, on 128x64
    // ones 55.7; over 1024 18.1 and 18.2)
    else if (g.accumulate || t128 <= (g.K >= 2048 ? 256 : 384)) cfg = (!g.accumulate && (long)t128 * products <= 256 && g.K >= 1024 && g.K <= 8192) ? GEMM_TILE_PIPE128 : GEMM_TILE_128x64;
    else cfg = GEMM_TILE_128x128;
  }
  const size_t bytesA = 2 * (size_t)(g.transA ? g.K : g.M) * g.lda, bytesB = 2 * (size_t)(g.transB ? g.N : g.K) * g.ldb;
  // direct global->LDS loads need 32-bit operand offsets, and whole 64-wide K tiles unless the contraction index is
  // the slow dimension of both operands (the k-rows past the end of an operand read as zero)
  const bool direct_ok = direct_k_ok(g.transA, g.transB, g.K) && bytesA < (1ull << 31) && bytesB < (1ull << 31);
  int splits = 1;
  bool modelled = false;
  if (g.accumulate && force < 2 && direct_ok && g.K >= 512) {
    modelled = true;
    // Split-K launch: tile shape and number of K ranges together, so that the grid fills the
    // chip in whole rounds.  Cost of a candidate in us, as in launch_gemm_group: a round of 128x128
    // tiles, two workgroups per CU, takes 1.2 per K-tile and 6 K-tiles besides (ring fill, atomic
    // adds); 128x64 tiles, three per CU, do the same work at 0.8 of that rate (more operand bytes
    // per flop).  256x256 tiles take 1.45 per K-tile, 6 for the launch, and their atomic adds in full (310 per ns):
    // nothing else runs on the CU meanwhile.  256 x 4232 over 7488 47 us on 128x128 tiles against 82, 4472 x 5312 over 3200
    // 205 against 246; 8192 x 1024 over 50304 578 on 256x256 ones against 874.
    double best = 1e30;
    for (int c = 0; c < 3; ++c) {
      const int bm = c == 2 ? 256 : 128, bn = c == 2 ? 256 : c ? 64 : 128, per_cu = c == 2 ? 1 : c ? 3 : 2;
      const long tiles = (long)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * products;
      const int max_s = std::min(16, g.K / 256);
      for (int sp = 1; sp <= max_s; ++sp) {
        const int kc = ((g.K + sp - 1) / sp + 63) / 64 * 64;
        const int real = (g.K + kc - 1) / kc;
        if (real != sp) continue;
        const long rounds = (tiles * sp + 256L * per_cu - 1) / (256L * per_cu);
        const double adds = (double)g.M * g.N * products * sp;
        const double cost = c == 2 ? rounds * 1.45 * (kc / 64) + 6 + adds / 310e3 : rounds * (c ? 1.125 : 1.2) * (kc / 64 + 6);
        if (cost < best) { best = cost; cfg = c == 2 ? GEMM_TILE_256x256 : c ? GEMM_TILE_128x64 : GEMM_TILE_128x128; splits = sp; }
      }
    }
  }
  if (!direct_ok) cfg = GEMM_TILE_STAGED128;
  if (cfg < GEMM_TILE_STAGED128 || cfg > GEMM_TILE_128x256) return false;
  const int BM = cfg == GEMM_TILE_256x256 ? 256 : cfg == GEMM_TILE_64x64 ? 64 : 128, BN = cfg == GEMM_TILE_128x64 ? 64 : cfg == GEMM_TILE_128x256 ? 256 : BM;
  long tiles = (long)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) * products;
  if (g.accumulate && !modelled && tiles < 384 && g.K >= 512) {
    splits = (int)((512 + tiles - 1) / tiles);
    int maxs = g.K / 256;
    if (splits > maxs) splits = maxs;
    if (splits < 1) splits = 1;
  }
  int kchunk = (g.K + splits - 1) / splits;
  kchunk = (kchunk + 63) / 64 * 64;
  splits = (g.K + kchunk - 1) / kchunk;
  plan = {cfg, splits, kchunk, direct_ok};
  return true;
}
// fp32 products go to the matrix cores except contractions of one K-tile of the plain kernel (16) where that has more than two
// workgroups of the small matrix-core tiles per CU to save on: 2053 x 570 over 8 6.8 us, on the matrix cores 8.6; 564 x 1197
// over 6 6.2 and 9.0; 888 x 590 over 5 6.1 and 8.9; but 1024 x 512 (512 tiles) over 16 5.6 and 4.8, 31 x 2000 5.6 and 3.7, and
// 2053 x 570 over 32 7.8 and 8.3, 564 x 1197 7.1 and 6.3.
static bool f32_on_matrix_cores(const GemmDesc& g) {
  if (!gemm_f32_ok(g)) return false;
  const long t32 = (long)((g.M + 31) / 32) * ((g.N + 31) / 32);
  return g.K > 16 || t32 <= 512;
}
int gemm_plan(int dtype, const GemmDesc& g, int* splits, long products) {
  GemmPlan plan;
  *splits = 1;
  if (dtype == 0) return f32_on_matrix_cores(g) ? 20 : 1;
  if (!gemm_uses_mfma(dtype, g)) return 1;
  if (!plan_mfma(g, 0, products, plan)) return -1;
  *splits = plan.splits;
  return plan.cfg;
}

hipError_t launch_gemm(hipStream_t s, int dtype, const GemmDesc& g, int force_generic) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  GemmParams p;
  p.A = g.A; p.B = g.B; p.C = g.C;
  p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
  p.out_fp32 = g.out_fp32; p.accumulate = g.accumulate ? ACC_ATOMIC : 0;
  p.bias = g.bias; p.residual = g.residual; p.ldr = g.ldr;
  p.res32 = g.res32; p.ldr32 = g.ldr32; p.ln_mean = g.ln_mean; p.ln_rstd = g.ln_rstd; p.ln_g = g.ln_g; p.ln_b = g.ln_b;
  if (g.res32 && (g.residual || g.accumulate || (g.ln_mean && !(g.ln_rstd && g.ln_g && g.ln_b)))) return hipErrorInvalidValue;
  p.epilogue = g.epilogue; p.Z = g.Z; p.ldz = g.ldz; p.alpha = g.alpha;
  p.drop = g.drop;
  p.kchunk = g.K; p.tilesN = 0; p.vec_epi = 0; p.kind = EPIK_GENERAL;
  // taken by the direct-load kernels only, which are not chosen for operands of 2 GiB and more
  p.bytesA = (int)operand_extent(dtype == 1 ? 2 : 4, g.transA ? g.K : g.M, g.transA ? g.M : g.K, g.lda);
  p.bytesB = (int)operand_extent(dtype == 1 ? 2 : 4, g.transB ? g.N : g.K, g.transB ? g.K : g.N, g.ldb);
  p.colsum = g.colsum; p.colsum_stride = g.colsum_stride;
  if (g.colsum && (g.accumulate || g.by > 1 || g.bz > 1 || g.C2)) return hipErrorInvalidValue;
  if (g.accumulate && (!g.out_fp32 || g.bias || g.residual || g.epilogue != EPI_NONE)) return hipErrorInvalidValue;
  // a batch of products: over the grid's y and z in the direct-to-LDS kernels, else one launch each
  const int by = std::max(1, g.by), bz = std::max(1, g.bz);
  const size_t esz = dtype == 1 ? 2 : 4, csz = g.out_fp32 ? 4 : esz;
  const int grids = g.C2 ? 2 : 1;
  if (g.C2 && (!g.A2 || !g.B2)) return hipErrorInvalidValue;
  p.by = by; p.bz = bz * grids; p.bz1 = bz;
  p.A2 = g.A2; p.B2 = g.B2; p.C2 = g.C2; p.alpha2 = g.alpha2;
  p.tri = g.tri;
  p.bAy = g.sAy * (long long)esz; p.bAz = g.sAz * (long long)esz;
  p.bBy = g.sBy * (long long)esz; p.bBz = g.sBz * (long long)esz;
  p.bCy = g.sCy * (long long)csz; p.bCz = g.sCz * (long long)csz;
  if (by * bz * grids > 1) {
    if (g.bias || g.residual || g.epilogue != EPI_NONE || g.drop.on) return hipErrorInvalidValue;
    if (g.res32 && (!g.out_fp32 || g.ln_mean || g.C2)) return hipErrorInvalidValue;
    const size_t bA = 2 * (size_t)(g.transA ? g.K : g.M) * g.lda, bB = 2 * (size_t)(g.transB ? g.N : g.K) * g.ldb;
    const bool in_grid = force_generic != 1 && gemm_uses_mfma(dtype, g) && direct_k_ok(g.transA, g.transB, g.K) && bA < (1ull << 31) && bB < (1ull << 31) &&
                         !((p.bAy | p.bAz | p.bBy | p.bBz | p.bCy | p.bCz) & 15) &&
                         (!g.C2 || (aligned16(g.A2) && aligned16(g.B2) && aligned16(g.C2) == aligned16(g.C)));
    if (!in_grid) {
      for (int w = 0; w < grids; ++w)
        for (int z = 0; z < bz; ++z)
          for (int y = 0; y < by; ++y) {
            GemmDesc h = g;
            h.by = h.bz = 0; h.A2 = h.B2 = nullptr; h.C2 = nullptr;
            h.A = (const char*)(w ? g.A2 : g.A) + y * p.bAy + z * p.bAz;
            h.B = (const char*)(w ? g.B2 : g.B) + y * p.bBy + z * p.bBz;
            h.C = (char*)(w ? g.C2 : g.C) + y * p.bCy + z * p.bCz;
            if (g.res32) h.res32 = reinterpret_cast<const float*>(reinterpret_cast<const char*>(g.res32) + y * p.bCy + z * p.bCz);
            if (w) h.alpha = g.alpha2;
            hipError_t e = launch_gemm(s, dtype, h, force_generic);
            if (e != hipSuccess) return e;
          }
      return hipSuccess;
    }
  }

  if (force_generic != 1 && gemm_uses_mfma(dtype, g)) {
    const int oe = g.out_fp32 ? 3 : 7;   // ldc granularity for 16-byte row chunks
    p.vec_epi = aligned16(g.C) && !(g.ldc & oe) && (!g.residual || (aligned16(g.residual) && !(g.ldr & 7))) &&
                (!g.res32 || (aligned16(g.res32) && !(g.ldr32 & 3))) &&
                (g.epilogue == EPI_NONE || (aligned16(g.Z) && !(g.ldz & 7)));
    p.kind = epilogue_kind(p);
    GemmPlan plan;
    if (!plan_mfma(g, force_generic, (long)by * bz * grids, plan)) return hipErrorInvalidValue;
    // 256x256 tiles run one workgroup per CU, so a launch takes whole rounds of 256 tiles.  A
    // few tile rows beyond the last full round would cost a whole round more (dV_o of a
    // 50257-word vocabulary: 788 tiles, 3.08 rounds): those rows go out as a second, split-K
    // launch that adds into the zeroed rows of the fp32 result.
    if (plan.cfg == GEMM_TILE_256x256 && force_generic == 0 && plan.direct_ok && g.out_fp32 && !g.accumulate && !g.bias && !g.residual &&
        !g.res32 && !g.colsum && g.epilogue == EPI_NONE && !g.drop.on && by * bz * grids == 1 && g.ldc == g.N && g.K >= 2048) {
      const int tn = (g.N + 255) / 256;
      if (tn <= 256 && 256 % tn == 0) {
        const int rows_round = 256 / tn * 256;
        const int main = g.M / rows_round * rows_round, tail = g.M - main;
        if (main > 0 && tail > 0 && ((tail + 255) / 256) * tn <= 64) {
          GemmDesc a = g;
          a.M = main;
          hipError_t e = launch_gemm(s, dtype, a, 0);
          if (e != hipSuccess) return e;
          GemmDesc b = g;
          b.M = tail;
          b.A = reinterpret_cast<const char*>(g.A) + 2 * (g.transA ? (size_t)main : (size_t)main * g.lda);
          b.C = reinterpret_cast<float*>(g.C) + (size_t)main * g.ldc;
          b.accumulate = 1;
          e = launch_fill_zero(s, b.C, (size_t)tail * g.ldc * 4);
          if (e != hipSuccess) return e;
          return launch_gemm(s, dtype, b, 0);
        }
      }
    }
    p.kchunk = plan.kchunk;
    const int cfg = plan.cfg, splits = plan.splits;
    if (cfg == GEMM_TILE_256x256) return launch_gemm_pp(s, p, g.transA, g.transB, splits);
    if (cfg != GEMM_TILE_STAGED128) return launch_gemm_dlds(s, p, g.transA, g.transB, splits, cfg);
    return launch_mfma_cfg<128, 128, 2, 2>(s, p, g.transA, g.transB, splits);
  }

  p.accumulate = g.accumulate;
  if (dtype == 0 && force_generic != 1 && (force_generic >= 20 ? gemm_f32_ok(g) : f32_on_matrix_cores(g))) return launch_gemm_f32(s, p, g.transA, g.transB, force_generic >= 20 ? force_generic - 20 : 0);

  dim3 grid((g.N + 63) / 64, (g.M + 63) / 64, 1), block(256);
#define OURO_PLAIN(T_)                                                                        \
  do {                                                                                        \
    if (!g.transA && !g.transB) hipLaunchKernelGGL((gemm_plain_kernel<T_, false, false>), grid, block, 0, s, p); \
    else if (!g.transA && g.transB) hipLaunchKernelGGL((gemm_plain_kernel<T_, false, true>), grid, block, 0, s, p); \
    else if (g.transA && !g.transB) hipLaunchKernelGGL((gemm_plain_kernel<T_, true, false>), grid, block, 0, s, p); \
    else hipLaunchKernelGGL((gemm_plain_kernel<T_, true, true>), grid, block, 0, s, p);       \
  } while (0)
  if (dtype == 1) OURO_PLAIN(bf16_t); else OURO_PLAIN(float);
#undef OURO_PLAIN
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && g.colsum) e = launch_colsum(s, g.out_fp32 ? 0 : dtype, g.C, g.ldc, g.colsum, g.M, g.N, g.colsum_stride);
  return e;
}

// Parameters of one accumulating product of a grouped launch.
static GemmParams group_params(const GemmDesc& d, size_t esz) {
  GemmParams p;
  memset(&p, 0, sizeof p);
  p.A = d.A; p.B = d.B; p.C = d.C;
  p.M = d.M; p.N = d.N; p.K = d.K; p.lda = d.lda; p.ldb = d.ldb; p.ldc = d.ldc;
  p.bytesA = (int)operand_extent(esz, d.K, d.M, d.lda); p.bytesB = (int)operand_extent(esz, d.K, d.N, d.ldb);
  p.out_fp32 = 1; p.epilogue = EPI_NONE; p.alpha = d.alpha; p.accumulate = d.accumulate;
  p.by = p.bz = p.bz1 = 1;
  return p;
}

// One K-range length for all products, and one of two kernels.
// Beside the error-gradient chain a compute unit that the launch leaves free is worth as much as time: the mean of its duration
// and its share of the chip's is compared.  128x128 tiles, two workgroups per CU, run in whole rounds
// of 512 and take 1.2 us per K-tile (of two side by side) plus 6 K-tiles of fixed cost (ring fill, atomic adds that the
// neighbour's matrix work covers).  256x256 tiles, one workgroup per CU, take 1.45 us per K-tile and 6 us besides; nothing
// covers their atomic adds, which all workgroups of a round reach together (310 adds per ns over the chip: 70 us for
// the 22 million of a 1024-wide layer split over 256 workgroups), but a tile whose K range is not split is stored.  128x128 and
// 256x256 tiles: 1024-wide layer, 8192 rows 255 and 185 us, 6144 rows 182 and 131 (256x256 taken); 512-wide, 8192 rows 73 and
// 80 (128x128 taken); 768-wide, 2331 rows 42 and 52 (256x256 taken: 108 compute units instead of all).
// Alone on the chip the duration counts: the makespan of dealing the products, longest range first, to the slots, and the
// atomic adds of the split ones (400 per ns), which set the time of short ranges.  128x128 tiles take 0.65 us per K-tile
// where no CU has two and 0.82 side by side, and 4 us besides.  448-wide relative-position layer, 4800 rows, ranges of 1600 / 2432 /
// 3200 / 4800 rows: 73 / 74 / 58 / 62 us (estimated 77 / 84 / 65 / 68), on 256x256 tiles 66 at best; 512-wide, 8192 rows, 2432 / 4096 /
// 8192: 83 / 71 / 89; 256-wide, 2048 rows, 320 / 640 / 960: 23 / 16 / 16 (25 with the range the other rule takes).
// The search costs host time on every call, so only ranges are looked at that change some product's number of splits (of those
// with equal numbers the shortest is the best one), and nothing is allocated: 18 x 1024-wide relative-position layers, 6144 rows,
// 86 us a layer with every range and heap-allocated intervals, 11 now.
void gemm_group_plan(const GemmDesc* g, int n, bool alone, bool* big_out, int (&kchunks)[2]) {
  int kmax = 0;
  for (int i = 0; i < n; ++i) kmax = std::max(kmax, (g[i].K + 63) / 64 * 64);
  double best[2] = {1e30, 1e30};
  kchunks[0] = kchunks[1] = kmax;
  for (int kc = std::min(256, kmax), next; kc <= kmax; kc = next) {
    int splits[GEMM_GROUP_MAX];
    next = kmax + 64;
    for (int i = 0; i < n; ++i) {
      splits[i] = (g[i].K + kc - 1) / kc;
      if (splits[i] > 1) next = std::min(next, ((g[i].K + splits[i] - 2) / (splits[i] - 1) + 63) / 64 * 64);
    }
    for (int big = 0; big < 2; ++big) {
      const int bt = big ? 256 : 128;
      const long slots = big ? 256 : 512;
      struct Part { int range; long wgs; } part[GEMM_GROUP_MAX];       // longest range first
      long wgs = 0;
      double adds = 0, cost;
      for (int i = 0; i < n; ++i) {
        const Part x = {((g[i].K + splits[i] - 1) / splits[i] + 63) / 64, (long)((g[i].M + bt - 1) / bt) * ((g[i].N + bt - 1) / bt) * splits[i]};
        wgs += x.wgs;
        if (splits[i] > 1 || g[i].accumulate != ACC_STORE) adds += (double)x.wgs * bt * bt;
        int j = i;
        for (; j > 0 && part[j - 1].range < x.range; --j) part[j] = part[j - 1];
        part[j] = x;
      }
      if (alone) {
        const double rate = big ? 1.45 : wgs <= 256 ? 0.65 : 0.82, fixed = big ? 6 : 4;
        // slots by the time from which they are free: a deal takes all slots of an entry and adds one, or ends a product
        struct Free { double at; long slots; } free_at[GEMM_GROUP_MAX + 1] = {{0.0, slots}};
        int nf = 1;
        double end = 0;
        for (int i = 0; i < n; ++i)
          for (long left = part[i].wgs; left > 0;) {
            int first = 0;
            for (int j = 1; j < nf; ++j)
              if (free_at[j].at < free_at[first].at || (free_at[j].at == free_at[first].at && free_at[j].slots < free_at[first].slots)) first = j;
            Free& f = free_at[first];
            const double t = f.at + rate * part[i].range + fixed;
            const long take = std::min(left, f.slots);
            left -= take;
            if (take == f.slots) f.at = t;
            else { f.slots -= take; free_at[nf++] = {t, take}; }
            end = std::max(end, t);
          }
        cost = end + adds / (big ? 310e3 : 400e3);
      } else {
        const double one = big ? 1.45 * (kc / 64) + 6 + adds / 310e3 : 1.2 * (kc / 64 + 6);
        cost = 0.5 * one * (std::ceil((double)wgs / slots) + (double)wgs / slots);
      }
      if (cost < best[big] - 1e-9) { best[big] = cost; kchunks[big] = kc; }
    }
  }
  *big_out = best[1] < best[0];
}

hipError_t launch_gemm_group(hipStream_t s, int dtype, const GemmDesc* g, int n, int tile, int kchunk, bool alone) {
  if (n < 1 || n > GEMM_GROUP_MAX || (tile != 0 && tile != 128 && tile != 256) || kchunk < 0 || kchunk % 64) return hipErrorInvalidValue;
  // products that do not admit the grouped kernel go by themselves
  GemmDesc in[GEMM_GROUP_MAX];
  GemmParams f32[GEMM_GROUP_MAX];
  int ni = 0, nf = 0;
  for (int i = 0; i < n; ++i) {
    const GemmDesc& d = g[i];
    const size_t bA = 2 * (size_t)d.K * d.lda, bB = 2 * (size_t)d.K * d.ldb;
    const bool form = d.transA == 1 && d.transB == 0 && d.accumulate && d.out_fp32 && !d.bias && !d.residual &&
                      !d.res32 && !d.colsum && d.epilogue == EPI_NONE && !d.drop.on && d.by <= 1 && d.bz <= 1 && !d.C2 && d.M > 0 && d.N > 0;
    if (form && dtype == 1 && gemm_uses_mfma(dtype, d) && bA < (1ull << 31) && bB < (1ull << 31)) { in[ni++] = d; continue; }
    if (form && dtype == 0 && f32_on_matrix_cores(d) && gemm_f32_group_ok(group_params(d, 4))) { f32[nf++] = group_params(d, 4); continue; }
    hipError_t e = launch_gemm(s, dtype, d, 0);
    if (e != hipSuccess) return e;
  }
  if (nf) return launch_gemm_f32_group(s, f32, nf);
  if (ni == 0) return hipSuccess;
  if (ni == 1 && !tile) return launch_gemm(s, dtype, in[0], 0);
  if (alone)                                       // longest contraction first, as planned
    for (int i = 1; i < ni; ++i)
      for (int j = i; j > 0 && in[j - 1].K < in[j].K; --j) std::swap(in[j - 1], in[j]);
  g = in; n = ni;
  bool big;
  int kchunks[2];
  gemm_group_plan(g, n, alone, &big, kchunks);
  if (tile) big = tile == 256;
  if (!tile || !kchunk) kchunk = kchunks[big];
  GemmParams ps[GEMM_GROUP_MAX];
  for (int i = 0; i < n; ++i) {
    const GemmDesc& d = g[i];
    GemmParams& p = ps[i];
    p = group_params(d, 2);
    // every product splits into ranges of the same length, rounded so that the last is not a sliver
    const int splits = (d.K + kchunk - 1) / kchunk;
    p.kchunk = ((d.K + splits - 1) / splits + 63) / 64 * 64;
    p.accumulate = splits > 1 ? ACC_ATOMIC : d.accumulate;
  }
  if (big) return launch_gemm_pp_group(s, ps, n);
  return launch_gemm_dlds_group(s, ps, n, 1, 0);
}

}  // namespace ouro
