// fp32 contraction on the matrix cores (32x32x2 instructions: fp32 products, fp32 accumulation), any size and alignment.
//
// The fp32 matrix rate is a sixteenth of the bf16 one (157 TFLOP/s), so a wave multiplies one 32x32 tile and even that keeps
// loads far from limiting: 8 KB of operands per 1024 clocks.  What a launch needs instead is enough workgroups, which the two
// forms below give over the sizes of a small model:
//   WIDE    64x64 tiles, waves 2 x 2, a ring of four K-tiles (32) shared by the workgroup;
//   !WIDE   32x32 tiles, the four waves take K-tiles in turn, each through a ring of its own, and add up through LDS at the
//           end: four times as many waves on the same product (16 against 4 per 64x64 outputs), for products of fewer than 384 64x64 tiles.
// Operands go global -> LDS by direct loads through a buffer descriptor (what lies past the operand reads as zero): 16 bytes
// per lane where leading dimensions and bases allow it (VEC = 4), else 4 bytes per lane.
//   row form (k contiguous in memory): [rows][32 k], 16-byte chunk c of a row at chunk c ^ (row & 7);
//   column form (k the slow dimension): [32 k][rows].
// The contraction index may be enumerated in any order as long as both operands agree: step s of group j takes
// k = 8 j + s from the lower half of the lanes and 8 j + 4 + s from the upper, so a row-form fragment of four steps is
// one 16-byte read.
// Against the plain tiled kernel (64x64, vector arithmetic, one synchronous K-tile of 16 at a time): 1024 x 512 x 512 80 ->
// 9 us, 1024 x 512 x 2048 300 -> 26 us (32x32 tiles); 1024 x 2048 x 512 101 -> 25 us (64x64); the products of a 2-layer
// 64-wide model on 128 tokens 22 -> 4.4 us each.
#include "gemm_common.h"

#include <algorithm>

namespace ouro {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int F32_BK = 32;

// One operand of a tile: ROWS along m (or n), NW waves share its loads.
template <int ROWS, bool COL, int VEC, int NW>
struct F32Operand {
  static constexpr int BYTES = ROWS * F32_BK * 4;
  static constexpr int EPL = 64 * VEC;                            // elements per wave-load
  static constexpr int PER = ROWS * F32_BK / EPL / NW;            // wave-loads per wave
  static_assert(ROWS * F32_BK % (EPL * NW) == 0, "loads divide over the waves");
  // (row, k) that lane `lane` fetches in wave-load j; with VEC = 4 it also fetches the next three along k (row form) or row
  __device__ static __forceinline__ void place(int j, int lane, int& row, int& k) {
    const int e = (j * 64 + lane) * VEC;                          // element index in LDS
    if (COL) { k = e / ROWS; row = e % ROWS; return; }
    row = e / F32_BK;
    const int d = e % F32_BK;
    k = (((d >> 2) ^ (row & 7)) << 2) + (d & 3);
  }
};

__device__ __forceinline__ void f32_load(const void* base, int bytes, char* dst, uint32_t voff, uint32_t soff, int vec) {
  auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
  if (vec == 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)dst, 16, voff, soff, 0, 0);
  else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)dst, 4, voff, soff, 0, 0);
}

// The fragment of four steps (group j) of a 32-row tile.
template <bool COL>
struct F32Frag {
  f32x4 v;
  float c[4];
  __device__ __forceinline__ float get(int s) const { return COL ? c[s] : v[s]; }
};
// The fragments of a K-tile of both operands, ra and rb their address registers (column form: one, k-rows ROWS floats
// apart).  Inline assembly, because the compiler cannot tell an LDS read from the target of the direct loads in flight and
// would drain those first; the reads and the wait for them are one block, so that no register of a read under way is the
// compiler's to move or use.
#define OURO_F32_A_ROW_TEXT                                                                          \
  "ds_read_b128 %[a0], %[ra0]\n\t" "ds_read_b128 %[a1], %[ra1]\n\t" "ds_read_b128 %[a2], %[ra2]\n\t" \
  "ds_read_b128 %[a3], %[ra3]\n\t"
#define OURO_F32_A_ROW_OUT                                                       \
  [a0] "=&v"(a[0].v), [a1] "=&v"(a[1].v), [a2] "=&v"(a[2].v), [a3] "=&v"(a[3].v)
#define OURO_F32_A_ROW_IN                                                \
  [ra0] "v"(ra[0]), [ra1] "v"(ra[1]), [ra2] "v"(ra[2]), [ra3] "v"(ra[3])
#define OURO_F32_A_COL_TEXT                                                                     \
  "ds_read_b32 %[a0], %[ra0] offset:%[k0]\n\t" "ds_read_b32 %[a1], %[ra0] offset:%[k1]\n\t"     \
  "ds_read_b32 %[a2], %[ra0] offset:%[k2]\n\t" "ds_read_b32 %[a3], %[ra0] offset:%[k3]\n\t"     \
  "ds_read_b32 %[a4], %[ra0] offset:%[k4]\n\t" "ds_read_b32 %[a5], %[ra0] offset:%[k5]\n\t"     \
  "ds_read_b32 %[a6], %[ra0] offset:%[k6]\n\t" "ds_read_b32 %[a7], %[ra0] offset:%[k7]\n\t"     \
  "ds_read_b32 %[a8], %[ra0] offset:%[k8]\n\t" "ds_read_b32 %[a9], %[ra0] offset:%[k9]\n\t"     \
  "ds_read_b32 %[a10], %[ra0] offset:%[k10]\n\t" "ds_read_b32 %[a11], %[ra0] offset:%[k11]\n\t" \
  "ds_read_b32 %[a12], %[ra0] offset:%[k12]\n\t" "ds_read_b32 %[a13], %[ra0] offset:%[k13]\n\t" \
  "ds_read_b32 %[a14], %[ra0] offset:%[k14]\n\t" "ds_read_b32 %[a15], %[ra0] offset:%[k15]\n\t"
#define OURO_F32_A_COL_OUT                                                                                           \
  [a0] "=&v"(a[0].c[0]), [a1] "=&v"(a[0].c[1]), [a2] "=&v"(a[0].c[2]), [a3] "=&v"(a[0].c[3]), [a4] "=&v"(a[1].c[0]), \
  [a5] "=&v"(a[1].c[1]), [a6] "=&v"(a[1].c[2]), [a7] "=&v"(a[1].c[3]), [a8] "=&v"(a[2].c[0]), [a9] "=&v"(a[2].c[1]), \
  [a10] "=&v"(a[2].c[2]), [a11] "=&v"(a[2].c[3]), [a12] "=&v"(a[3].c[0]), [a13] "=&v"(a[3].c[1]),                    \
  [a14] "=&v"(a[3].c[2]), [a15] "=&v"(a[3].c[3])
#define OURO_F32_A_COL_IN \
  [ra0] "v"(ra[0])
#define OURO_F32_B_ROW_TEXT                                                                          \
  "ds_read_b128 %[b0], %[rb0]\n\t" "ds_read_b128 %[b1], %[rb1]\n\t" "ds_read_b128 %[b2], %[rb2]\n\t" \
  "ds_read_b128 %[b3], %[rb3]\n\t"
#define OURO_F32_B_ROW_OUT                                                       \
  [b0] "=&v"(b[0].v), [b1] "=&v"(b[1].v), [b2] "=&v"(b[2].v), [b3] "=&v"(b[3].v)
#define OURO_F32_B_ROW_IN                                                \
  [rb0] "v"(rb[0]), [rb1] "v"(rb[1]), [rb2] "v"(rb[2]), [rb3] "v"(rb[3])
#define OURO_F32_B_COL_TEXT                                                                     \
  "ds_read_b32 %[b0], %[rb0] offset:%[k0]\n\t" "ds_read_b32 %[b1], %[rb0] offset:%[k1]\n\t"     \
  "ds_read_b32 %[b2], %[rb0] offset:%[k2]\n\t" "ds_read_b32 %[b3], %[rb0] offset:%[k3]\n\t"     \
  "ds_read_b32 %[b4], %[rb0] offset:%[k4]\n\t" "ds_read_b32 %[b5], %[rb0] offset:%[k5]\n\t"     \
  "ds_read_b32 %[b6], %[rb0] offset:%[k6]\n\t" "ds_read_b32 %[b7], %[rb0] offset:%[k7]\n\t"     \
  "ds_read_b32 %[b8], %[rb0] offset:%[k8]\n\t" "ds_read_b32 %[b9], %[rb0] offset:%[k9]\n\t"     \
  "ds_read_b32 %[b10], %[rb0] offset:%[k10]\n\t" "ds_read_b32 %[b11], %[rb0] offset:%[k11]\n\t" \
  "ds_read_b32 %[b12], %[rb0] offset:%[k12]\n\t" "ds_read_b32 %[b13], %[rb0] offset:%[k13]\n\t" \
  "ds_read_b32 %[b14], %[rb0] offset:%[k14]\n\t" "ds_read_b32 %[b15], %[rb0] offset:%[k15]\n\t"
#define OURO_F32_B_COL_OUT                                                                                           \
  [b0] "=&v"(b[0].c[0]), [b1] "=&v"(b[0].c[1]), [b2] "=&v"(b[0].c[2]), [b3] "=&v"(b[0].c[3]), [b4] "=&v"(b[1].c[0]), \
  [b5] "=&v"(b[1].c[1]), [b6] "=&v"(b[1].c[2]), [b7] "=&v"(b[1].c[3]), [b8] "=&v"(b[2].c[0]), [b9] "=&v"(b[2].c[1]), \
  [b10] "=&v"(b[2].c[2]), [b11] "=&v"(b[2].c[3]), [b12] "=&v"(b[3].c[0]), [b13] "=&v"(b[3].c[1]),                    \
  [b14] "=&v"(b[3].c[2]), [b15] "=&v"(b[3].c[3])
#define OURO_F32_B_COL_IN \
  [rb0] "v"(rb[0])
#define OURO_F32_KROWS                                                                                            \
  [k0] "n"(0 * ROWS), [k1] "n"(4 * ROWS), [k2] "n"(8 * ROWS), [k3] "n"(12 * ROWS), [k4] "n"(32 * ROWS),           \
  [k5] "n"(36 * ROWS), [k6] "n"(40 * ROWS), [k7] "n"(44 * ROWS), [k8] "n"(64 * ROWS), [k9] "n"(68 * ROWS),        \
  [k10] "n"(72 * ROWS), [k11] "n"(76 * ROWS), [k12] "n"(96 * ROWS), [k13] "n"(100 * ROWS), [k14] "n"(104 * ROWS), \
  [k15] "n"(108 * ROWS)
#define OURO_F32_READ(FA, FB, ...) \
  asm volatile(OURO_F32_A_##FA##_TEXT OURO_F32_B_##FB##_TEXT "s_waitcnt lgkmcnt(0)" \
               : OURO_F32_A_##FA##_OUT, OURO_F32_B_##FB##_OUT : OURO_F32_A_##FA##_IN, OURO_F32_B_##FB##_IN __VA_ARGS__ : "memory")
template <int ROWS>
__device__ __forceinline__ void f32_read(F32Frag<false> (&a)[4], const uint32_t (&ra)[4], F32Frag<false> (&b)[4], const uint32_t (&rb)[4]) { OURO_F32_READ(ROW, ROW); }
template <int ROWS>
__device__ __forceinline__ void f32_read(F32Frag<false> (&a)[4], const uint32_t (&ra)[4], F32Frag<true> (&b)[4], const uint32_t (&rb)[4]) { OURO_F32_READ(ROW, COL, , OURO_F32_KROWS); }
template <int ROWS>
__device__ __forceinline__ void f32_read(F32Frag<true> (&a)[4], const uint32_t (&ra)[4], F32Frag<false> (&b)[4], const uint32_t (&rb)[4]) { OURO_F32_READ(COL, ROW, , OURO_F32_KROWS); }
template <int ROWS>
__device__ __forceinline__ void f32_read(F32Frag<true> (&a)[4], const uint32_t (&ra)[4], F32Frag<true> (&b)[4], const uint32_t (&rb)[4]) { OURO_F32_READ(COL, COL, , OURO_F32_KROWS); }
#undef OURO_F32_READ
#undef OURO_F32_KROWS
#undef OURO_F32_A_ROW_TEXT
#undef OURO_F32_A_ROW_OUT
#undef OURO_F32_A_ROW_IN
#undef OURO_F32_A_COL_TEXT
#undef OURO_F32_A_COL_OUT
#undef OURO_F32_A_COL_IN
#undef OURO_F32_B_ROW_TEXT
#undef OURO_F32_B_ROW_OUT
#undef OURO_F32_B_ROW_IN
#undef OURO_F32_B_COL_TEXT
#undef OURO_F32_B_COL_OUT
#undef OURO_F32_B_COL_IN
// Address registers of the 32-row tile that starts at row t0: row form one per group, column form one.
template <int ROWS, bool COL>
__device__ __forceinline__ void f32_addresses(uint32_t base, int t0, int lane, uint32_t (&a)[4]) {
  const int row = t0 + (lane & 31), h = lane >> 5;
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = COL ? base + h * 4 * ROWS * 4 + row * 4 : base + row * 128 + (((2 * j + h) ^ (row & 7)) << 4);
}

// Tile `tile` of a product, contraction range `range`.
template <bool WIDE, bool TA, bool TB, int VEC>
__device__ __forceinline__ void gemm_f32_body(const GemmParams& p, int tile, int range, char* lds_all) {
  constexpr int T = WIDE ? 64 : 32, S = WIDE ? 4 : 2, NW = WIDE ? 4 : 1;
  using OA = F32Operand<T, TA, VEC, NW>;
  using OB = F32Operand<T, !TB, VEC, NW>;
  constexpr int STAGE = OA::BYTES + OB::BYTES, LPT = OA::PER + OB::PER;
  static_assert((S - 1) * LPT < 64, "vmcnt range");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  char* const lds = WIDE ? lds_all : lds_all + wave * (S * STAGE);
  const int lw = WIDE ? wave : 0;                                // wave's place among those that share the loads
  const int m0 = (tile / p.tilesN) * T, n0 = (tile % p.tilesN) * T;
  const int kbeg = range * p.kchunk, kend = min(p.K, kbeg + p.kchunk);
  const int nk_all = (kend - kbeg + F32_BK - 1) / F32_BK;
  const int k_first = WIDE ? 0 : wave, k_step = WIDE ? 1 : 4;    // K-tiles of this wave
  const int nk = nk_all > k_first ? (nk_all - k_first + k_step - 1) / k_step : 0;

  uint32_t oa[OA::PER], ob[OB::PER];                             // byte offsets without the K-tile term
  auto offset = [](bool col, int row, int k, int ld) __attribute__((always_inline)) { return 4u * (col ? (uint32_t)k * (uint32_t)ld + row : (uint32_t)row * (uint32_t)ld + k); };
#pragma unroll
  for (int i = 0; i < OA::PER; ++i) { int row, k; OA::place(lw * OA::PER + i, lane, row, k); oa[i] = offset(TA, m0 + row, k, p.lda); }
#pragma unroll
  for (int i = 0; i < OB::PER; ++i) { int row, k; OB::place(lw * OB::PER + i, lane, row, k); ob[i] = offset(!TB, n0 + row, k, p.ldb); }
  auto request = [&](int it, int st) __attribute__((always_inline)) {
    const int k0 = kbeg + (k_first + it * k_step) * F32_BK;
    const uint32_t ka = 4u * (TA ? (uint32_t)k0 * (uint32_t)p.lda : (uint32_t)k0), kb = 4u * (TB ? (uint32_t)k0 : (uint32_t)k0 * (uint32_t)p.ldb);
    char* d = lds + st * STAGE;
    // a row-form operand's last K-tile may be ragged: what lies past the row's end is sent out of range, which reads as zero
    const bool ragged = k0 + F32_BK > kend;
#pragma unroll
    for (int i = 0; i < OA::PER; ++i) {
      char* da = d + (lw * OA::PER + i) * (OA::EPL * 4);
      if (!TA && ragged) { int row, k; OA::place(lw * OA::PER + i, lane, row, k); f32_load(p.A, p.bytesA, da, k0 + k < kend ? oa[i] + ka : 0x7ffffff0u, 0, VEC); }
      else f32_load(p.A, p.bytesA, da, oa[i], ka, VEC);
    }
#pragma unroll
    for (int i = 0; i < OB::PER; ++i) {
      char* db = d + OA::BYTES + (lw * OB::PER + i) * (OB::EPL * 4);
      if (TB && ragged) { int row, k; OB::place(lw * OB::PER + i, lane, row, k); f32_load(p.B, p.bytesB, db, k0 + k < kend ? ob[i] + kb : 0x7ffffff0u, 0, VEC); }
      else f32_load(p.B, p.bytesB, db, ob[i], kb, VEC);
    }
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  uint32_t ra[4], rb[4];
  f32_addresses<T, TA>(lds0, WIDE ? 32 * (wave >> 1) : 0, lane, ra);
  f32_addresses<T, !TB>(lds0 + OA::BYTES, WIDE ? 32 * (wave & 1) : 0, lane, rb);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < nk) request(s, s);
  int rd = 0, fill = S - 1;
  for (int it = 0; it < nk; ++it) {
    // this K-tile has landed once only the younger ones are outstanding; where the stages are shared, for every wave's share
    if (it + S - 1 <= nk) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * LPT) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (WIDE) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    if (it + S - 1 < nk) request(it + S - 1, fill);              // the stage read one K-tile ago (its reads were waited for)
    F32Frag<TA> fa[4];
    F32Frag<!TB> fb[4];
    uint32_t va[4], vb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { va[j] = ra[j] + rd * STAGE; vb[j] = rb[j] + rd * STAGE; }
    f32_read<T>(fa, va, fb, vb);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j].get(s), fb[j].get(s), acc, 0, 0, 0);
    fill = rd;
    rd = rd + 1 == S ? 0 : rd + 1;
  }
  const int h = lane >> 5, l32 = lane & 31;
  if (WIDE) {
    const int mb = m0 + 32 * (wave >> 1) + 4 * h, n = n0 + 32 * (wave & 1) + l32;
    float v[16];
    int m[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) { v[r] = acc[r]; m[r] = mb + 8 * (r >> 2) + (r & 3); }
    epilogue_column<float, 16>(p, m, n, v);
    return;
  }
  // add up the four waves' parts: [wave][row][33]
  __syncthreads();                                               // every wave is past its last fragment read
  float* part = reinterpret_cast<float*>(lds_all);
#pragma unroll
  for (int r = 0; r < 16; ++r) part[(wave * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * 33 + l32] = acc[r];
  __syncthreads();
  float v[4];
  int m[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = (tid >> 5) + 8 * i, col = tid & 31;
    v[i] = part[row * 33 + col] + part[(32 + row) * 33 + col] + part[(64 + row) * 33 + col] + part[(96 + row) * 33 + col];
    m[i] = m0 + row;
  }
  epilogue_column<float, 4>(p, m, n0 + (tid & 31), v);
}

template <bool WIDE, bool TA, bool TB, int VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) char lds_all[];
  gemm_f32_body<WIDE, TA, TB, VEC>(p, blockIdx.x, blockIdx.z, lds_all);
}
// Several accumulating products A^T B (weight gradients of a layer) in one launch; product i owns the work items [first[i], first[i+1]).
struct F32GroupParams {
  int n;
  int first[GEMM_GROUP_MAX + 1];
  GemmParams p[GEMM_GROUP_MAX];
};
static_assert(sizeof(F32GroupParams) <= 4096, "kernel arguments are limited to 4 KiB");
template <bool WIDE>
__global__ __launch_bounds__(256) void gemm_f32_group_kernel(F32GroupParams g) {
  extern __shared__ __attribute__((aligned(16))) char lds_all[];
  int i = 0;
  while (i + 1 < g.n && (int)blockIdx.x >= g.first[i + 1]) ++i;
  const GemmParams& p = g.p[i];
  const int local = blockIdx.x - g.first[i];
  gemm_f32_body<WIDE, true, false, 4>(p, local % p.ntiles, local / p.ntiles, lds_all);
}

bool gemm_f32_ok(const GemmDesc& g) {
  const size_t bytesA = 4 * (size_t)(g.transA ? g.K : g.M) * g.lda, bytesB = 4 * (size_t)(g.transB ? g.N : g.K) * g.ldb;
  // offsets are 32-bit, also those of the up to 63 rows that a tile has past the operand's end: none may wrap back into it
  const size_t pastA = bytesA + 256 * (size_t)g.lda, pastB = bytesB + 256 * (size_t)g.ldb;
  return bytesA < (1ull << 31) - 64 && bytesB < (1ull << 31) - 64 && pastA < (1ull << 32) && pastB < (1ull << 32) && g.K >= 1;
}

template <bool WIDE, int VEC>
static hipError_t launch_f32(hipStream_t s, GemmParams& p, int transA, int transB, int splits) {
  constexpr int T = WIDE ? 64 : 32;
  constexpr size_t smem = WIDE ? 4 * 2 * 64 * 128 : 4 * 2 * 2 * 32 * 128;
  static_assert(smem >= 4 * 32 * 33 * 4, "the parts of the four waves fit");
  p.tilesM = (p.M + T - 1) / T;
  p.tilesN = (p.N + T - 1) / T;
  dim3 grid(p.tilesM * p.tilesN, 1, splits), block(256);
#define OURO_LAUNCH(TA_, TB_)                                                                                 \
  do {                                                                                                        \
    static bool attr_done = false;                                                                            \
    if (!attr_done) {                                                                                         \
      hipError_t e = hipFuncSetAttribute((const void*)gemm_f32_kernel<WIDE, TA_, TB_, VEC>,                   \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);              \
      if (e != hipSuccess) return e;                                                                          \
      attr_done = true;                                                                                       \
    }                                                                                                         \
    hipLaunchKernelGGL((gemm_f32_kernel<WIDE, TA_, TB_, VEC>), grid, block, smem, s, p);                      \
  } while (0)
  if (!transA && !transB) OURO_LAUNCH(false, false);
  else if (!transA && transB) OURO_LAUNCH(false, true);
  else if (transA && !transB) OURO_LAUNCH(true, false);
  else OURO_LAUNCH(true, true);
#undef OURO_LAUNCH
  return hipGetLastError();
}

// 16-byte requests: aligned bases, rows of whole quads
static bool f32_vec(const GemmParams& p, int transA, int transB) {
  return !(((uintptr_t)p.A | (uintptr_t)p.B) & 15) && !((p.lda | p.ldb) & 3) && !((transA ? p.M : p.K) & 3) && !((transB ? p.K : p.N) & 3);
}
bool gemm_f32_group_ok(const GemmParams& p) { return f32_vec(p, 1, 0); }
// ps: n products A^T B that gemm_f32_ok and gemm_f32_group_ok take, accumulate as epilogue_column takes it.  The forms as for one product
// (below), the tiles of all counted together.
// Four products of a 64-wide layer over 128 rows, 3.7 to 4.3 us each, take 4.4 us in one launch; those of a 512-wide one over 1024 rows
// (768 64x64 tiles) 87 us beside the error-gradient chain, in four launches 131.
hipError_t launch_gemm_f32_group(hipStream_t s, const GemmParams* ps, int n) {
  if (n < 1 || n > GEMM_GROUP_MAX) return hipErrorInvalidValue;
  long t64 = 0, t32 = 0;
  for (int i = 0; i < n; ++i) {
    t64 += (long)((ps[i].M + 63) / 64) * ((ps[i].N + 63) / 64);
    t32 += (long)((ps[i].M + 31) / 32) * ((ps[i].N + 31) / 32);
  }
  const bool wide = t64 >= 384;
  const int T = wide ? 64 : 32;
  F32GroupParams g;
  memset(&g, 0, sizeof g);
  g.n = n;
  for (int i = 0; i < n; ++i) {
    GemmParams p = ps[i];
    p.tilesM = (p.M + T - 1) / T;
    p.tilesN = (p.N + T - 1) / T;
    p.ntiles = p.tilesM * p.tilesN;
    int splits = 1;
    if (!wide && t32 < 512) splits = (int)std::max<long>(1, std::min<long>(512 / t32, p.K / (16 * F32_BK)));
    p.kchunk = ((p.K + splits - 1) / splits + F32_BK - 1) / F32_BK * F32_BK;
    splits = (p.K + p.kchunk - 1) / p.kchunk;
    if (splits > 1) p.accumulate = ACC_ATOMIC;
    g.p[i] = p;
    g.first[i + 1] = g.first[i] + p.ntiles * splits;
  }
  const size_t smem = wide ? 4 * 2 * 64 * 128 : 4 * 2 * 2 * 32 * 128;
  static bool attr_done[2] = {false, false};
  auto kern = wide ? gemm_f32_group_kernel<true> : gemm_f32_group_kernel<false>;
  if (!attr_done[wide]) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_done[wide] = true;
  }
  hipLaunchKernelGGL(kern, dim3(g.first[n]), dim3(256), smem, s, g);
  return hipGetLastError();
}

// form: 0 automatic, 1 64x64 tiles, 2 32x32 tiles with K-tiles dealt to the waves.
hipError_t launch_gemm_f32(hipStream_t s, GemmParams& p, int transA, int transB, int form) {
  const bool vec = f32_vec(p, transA, transB);
  const long t64 = (long)((p.M + 63) / 64) * ((p.N + 63) / 64), t32 = (long)((p.M + 31) / 32) * ((p.N + 31) / 32);
  // 512 64x64 tiles: 2048 x 1024 x 1024 takes 40 us on them against 47 us in the other form; 128 tiles (1024 x 512 x 2048)
  // 51 us against 25; in between (1024 x 1536 x 512) 23 us both
  const bool wide = form == 1 || (form == 0 && t64 >= 384);
  int splits = 1;
  // a small output with a long contraction: split it over workgroups too (512 of the small tiles fill the chip), at least
  // four K-tiles per wave
  if (p.accumulate && !wide && t32 < 512) splits = (int)std::max<long>(1, std::min<long>(512 / t32, p.K / (16 * F32_BK)));
  p.kchunk = ((p.K + splits - 1) / splits + F32_BK - 1) / F32_BK * F32_BK;
  splits = (p.K + p.kchunk - 1) / p.kchunk;
  if (splits > 1) p.accumulate = ACC_ATOMIC;
  if (wide) return vec ? launch_f32<true, 4>(s, p, transA, transB, splits) : launch_f32<true, 1>(s, p, transA, transB, splits);
  return vec ? launch_f32<false, 4>(s, p, transA, transB, splits) : launch_f32<false, 1>(s, p, transA, transB, splits);
}

}  // namespace ouro
