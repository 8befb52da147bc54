// bf16 MFMA contraction on 256x256 tiles in which the two waves of a SIMD take turns: while one runs its
// matrix instructions the other reads fragments from LDS and requests tiles from memory.
//
// What bounds it: the clock first.  With random operands the chip runs these loops at 1.54 (A B^T) and 1.69 GHz (A^T B) against
// 2.4 GHz nominal, and at that clock the matrix pipe is busy 82 and 77 % of the cycles (LDS conflicts 1 %): the rest are the
// barriers between the phases and the epilogue.  8192^3 takes 780-830 us in either form, 1.33-1.41 PFLOP/s; in the 24-layer
// 1024-wide step dh_L = G V goes 874 -> 589 us, dV_o
// 670 -> 592 us, a layer's weight gradients 255 -> 170-178 us.  The same tile with one barrier per K-tile, all eight waves in step
// (the form this one replaced), needs 895 and 912 us: fragment reads and requests then stand between the matrix
// instructions instead of beside them.  Tried on the way, same products: BK = 32 with a four-stage ring 883 / 829 us (a
// row-form request then fetches half cache lines), five stages the same (latency is not the limit), requests between the
// matrix instructions 856 / 833 us, four waves with 128x128 wave tiles and one barrier per K-tile 861 / 820 us.
//
// A workgroup has eight waves (two per SIMD).  The tile consists of two 128-row halves of A and two 128-column halves of
// B; waves 0-3 own the first 64 rows of each row half, waves 4-7 the other 64; wave % 4 owns 32 columns of each column
// half.  LDS holds two stages of the four halves (K-tile 64).  A K-tile is two phases of 16 matrix instructions:
//
//   phase  reads                 multiplies            requests
//     1    A0, B1                A0 x B0, A0 x B1      A1 of K-tile kt+1, B0 of kt+2     (both halves were last read in the phase before)
//     2    A1, B0 of kt+1        A1 x B1, A1 x B0      A0 and B1 of kt+2                 (likewise)
//
// and a phase is: read the fragments and wait for them; request; wait for the halves that the next phase reads; barrier;
// multiply; barrier (requests ahead of the reads delay them: 3 % on dV_o).  Waves 4-7 run one barrier behind waves 0-3, so one group's multiplications coincide with the other group's
// reads.  Every wave waits for its fragments before the barrier inside the phase: a wave that has begun the next phase
// knows that all eight have read what this phase reads, which is what the refill needs.  A request has two phases of both
// groups' matrix work to arrive in.
#include "gemm_common.h"

namespace ouro {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int PP_BK = 64;
constexpr int PP_HALF = 128 * PP_BK * 2;           // bytes of a half: 128 rows x 64 k
constexpr int PP_LDS = 8 * PP_HALF;                // [operand][stage][half]
// One operand half in LDS.
//   row form (k contiguous in memory): [128][64], 16-byte chunk c of a row at chunk c ^ swizzle(row): the 16 rows one
//     fragment read serves per cycle fall on 16 different 16-byte slots of the 256-byte bank window.
//   COL, column form (k the slow dimension): [64][128], chunk c of k-row k at c ^ ((k & 3) << 2), transposed at read time
//     with the LDS transpose-read (see colswz in gemm_dlds.hip).
// The swizzles depend on a row's place in its 32-row tile only, so that the fragments of a wave's tiles lie at constant
// distances: a fragment read is an address register plus an immediate offset.
template <bool COL>
struct PpOperand {
  static constexpr int CPR = COL ? 16 : 8;                       // chunks per LDS row
  __device__ static __forceinline__ int swizzle(int row) { return (row ^ ((row & 31) >> 3)) & 7; }
  // Byte offset of the 16 bytes lane `lane` fetches in the first of the wave's two 1 KiB requests for the half; the second
  // lies jump() further on.  Rows are not clamped: what lies past the operand's end reads as zero, and what a row index
  // beyond the valid extent fetches otherwise only feeds outputs that are never stored.
  __device__ static __forceinline__ uint32_t src(int wave, int lane, int row0, int ld) {
    const int lr = wave * (64 / CPR) + lane / CPR, pc = lane % CPR;
    if (!COL) return 2u * ((uint32_t)(row0 + lr) * (uint32_t)ld + 8u * (pc ^ swizzle(lr)));
    return 2u * ((uint32_t)lr * (uint32_t)ld + (uint32_t)(row0 + 8 * (pc ^ ((lr & 3) << 2))));
  }
  __device__ static __forceinline__ uint32_t jump(int ld) { return 2u * (8 * (64 / CPR)) * (uint32_t)ld; }
  __device__ static __forceinline__ uint32_t half(int ld) { return 2u * 128u * (COL ? 1u : (uint32_t)ld); }     // from half 0 to half 1
  // Address registers of a wave whose 32-row tiles (up to two) start at row t0 of the half: row form one per k step (the
  // swizzle is an XOR with the chunk index), column form one per tile.
  template <int T> static constexpr int naddr() { return COL ? T : 4; }
  template <int T>
  __device__ static __forceinline__ void addresses(uint32_t base, int t0, int lane, uint32_t* a) {
    if (!COL) {
      const int row = t0 + (lane & 31);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) a[ks] = base + row * 128 + (((2 * ks + (lane >> 5)) ^ swizzle(row)) << 4);
    } else {
      const int g4 = lane >> 4, i = lane & 15;
      const int k = 8 * (g4 >> 1) + (i >> 2);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int m = t0 + 32 * t + 16 * (g4 & 1) + 4 * (i & 3);
        a[t] = base + k * 256 + (((m >> 3) ^ ((k & 3) << 2)) << 4) + ((m & 7) << 1);
      }
    }
  }
};

// A fragment as it leaves LDS (two transposing reads in column form).
template <bool COL> struct PpFrag;
template <> struct PpFrag<false> {
  u32x4 v;
  __device__ __forceinline__ bf16x8 get() const { return __builtin_bit_cast(bf16x8, v); }
};
template <> struct PpFrag<true> {
  u32x2 lo, hi;
  __device__ __forceinline__ bf16x8 get() const { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3)); }
};
template <int N> __device__ __forceinline__ void pp_wait_mem() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// The fragments of a phase: a[ks][t], the wave's two tiles of the half of A at LDS offset BA, and b[ks][0], its tile of the
// half of B at BB, for the four k steps.  Inline assembly, because the compiler cannot tell an LDS read from the target of
// the direct loads in flight and would drain those first; the reads and the wait for them are one block, so that no
// register of a read under way is the compiler's to move or use.
#define OURO_PP_A_ROW_TEXT                                                                      \
  "ds_read_b128 %[a0], %[ra0] offset:%[oa0]\n\t" "ds_read_b128 %[a1], %[ra0] offset:%[oa1]\n\t" \
  "ds_read_b128 %[a2], %[ra1] offset:%[oa0]\n\t" "ds_read_b128 %[a3], %[ra1] offset:%[oa1]\n\t" \
  "ds_read_b128 %[a4], %[ra2] offset:%[oa0]\n\t" "ds_read_b128 %[a5], %[ra2] offset:%[oa1]\n\t" \
  "ds_read_b128 %[a6], %[ra3] offset:%[oa0]\n\t" "ds_read_b128 %[a7], %[ra3] offset:%[oa1]\n\t"
#define OURO_PP_A_ROW_OUT                                                                                            \
  [a0] "=&v"(a[0][0].v), [a1] "=&v"(a[0][1].v), [a2] "=&v"(a[1][0].v), [a3] "=&v"(a[1][1].v), [a4] "=&v"(a[2][0].v), \
  [a5] "=&v"(a[2][1].v), [a6] "=&v"(a[3][0].v), [a7] "=&v"(a[3][1].v)
#define OURO_PP_A_ROW_IN                                                                                      \
  [ra0] "v"(ra[0]), [ra1] "v"(ra[1]), [ra2] "v"(ra[2]), [ra3] "v"(ra[3]), [oa0] "n"(BA), [oa1] "n"(BA + 4096)
#define OURO_PP_A_COL_TEXT                                                                                    \
  "ds_read_b64_tr_b16 %[a0], %[ra0] offset:%[oa0]\n\t" "ds_read_b64_tr_b16 %[a1], %[ra0] offset:%[oa1]\n\t"   \
  "ds_read_b64_tr_b16 %[a2], %[ra1] offset:%[oa0]\n\t" "ds_read_b64_tr_b16 %[a3], %[ra1] offset:%[oa1]\n\t"   \
  "ds_read_b64_tr_b16 %[a4], %[ra0] offset:%[oa2]\n\t" "ds_read_b64_tr_b16 %[a5], %[ra0] offset:%[oa3]\n\t"   \
  "ds_read_b64_tr_b16 %[a6], %[ra1] offset:%[oa2]\n\t" "ds_read_b64_tr_b16 %[a7], %[ra1] offset:%[oa3]\n\t"   \
  "ds_read_b64_tr_b16 %[a8], %[ra0] offset:%[oa4]\n\t" "ds_read_b64_tr_b16 %[a9], %[ra0] offset:%[oa5]\n\t"   \
  "ds_read_b64_tr_b16 %[a10], %[ra1] offset:%[oa4]\n\t" "ds_read_b64_tr_b16 %[a11], %[ra1] offset:%[oa5]\n\t" \
  "ds_read_b64_tr_b16 %[a12], %[ra0] offset:%[oa6]\n\t" "ds_read_b64_tr_b16 %[a13], %[ra0] offset:%[oa7]\n\t" \
  "ds_read_b64_tr_b16 %[a14], %[ra1] offset:%[oa6]\n\t" "ds_read_b64_tr_b16 %[a15], %[ra1] offset:%[oa7]\n\t"
#define OURO_PP_A_COL_OUT                                                                            \
  [a0] "=&v"(a[0][0].lo), [a1] "=&v"(a[0][0].hi), [a2] "=&v"(a[0][1].lo), [a3] "=&v"(a[0][1].hi),    \
  [a4] "=&v"(a[1][0].lo), [a5] "=&v"(a[1][0].hi), [a6] "=&v"(a[1][1].lo), [a7] "=&v"(a[1][1].hi),    \
  [a8] "=&v"(a[2][0].lo), [a9] "=&v"(a[2][0].hi), [a10] "=&v"(a[2][1].lo), [a11] "=&v"(a[2][1].hi),  \
  [a12] "=&v"(a[3][0].lo), [a13] "=&v"(a[3][0].hi), [a14] "=&v"(a[3][1].lo), [a15] "=&v"(a[3][1].hi)
#define OURO_PP_A_COL_IN                                                                                         \
  [ra0] "v"(ra[0]), [ra1] "v"(ra[1]), [oa0] "n"(BA + 0), [oa1] "n"(BA + 1024), [oa2] "n"(BA + 4096),             \
  [oa3] "n"(BA + 5120), [oa4] "n"(BA + 8192), [oa5] "n"(BA + 9216), [oa6] "n"(BA + 12288), [oa7] "n"(BA + 13312)
#define OURO_PP_B_ROW_TEXT                                                                      \
  "ds_read_b128 %[b0], %[rb0] offset:%[ob0]\n\t" "ds_read_b128 %[b1], %[rb1] offset:%[ob0]\n\t" \
  "ds_read_b128 %[b2], %[rb2] offset:%[ob0]\n\t" "ds_read_b128 %[b3], %[rb3] offset:%[ob0]\n\t"
#define OURO_PP_B_ROW_OUT                                                                    \
  [b0] "=&v"(b[0][0].v), [b1] "=&v"(b[1][0].v), [b2] "=&v"(b[2][0].v), [b3] "=&v"(b[3][0].v)
#define OURO_PP_B_ROW_IN                                                                \
  [rb0] "v"(rb[0]), [rb1] "v"(rb[1]), [rb2] "v"(rb[2]), [rb3] "v"(rb[3]), [ob0] "n"(BB)
#define OURO_PP_B_COL_TEXT                                                                                  \
  "ds_read_b64_tr_b16 %[b0], %[rb0] offset:%[ob0]\n\t" "ds_read_b64_tr_b16 %[b1], %[rb0] offset:%[ob1]\n\t" \
  "ds_read_b64_tr_b16 %[b2], %[rb0] offset:%[ob2]\n\t" "ds_read_b64_tr_b16 %[b3], %[rb0] offset:%[ob3]\n\t" \
  "ds_read_b64_tr_b16 %[b4], %[rb0] offset:%[ob4]\n\t" "ds_read_b64_tr_b16 %[b5], %[rb0] offset:%[ob5]\n\t" \
  "ds_read_b64_tr_b16 %[b6], %[rb0] offset:%[ob6]\n\t" "ds_read_b64_tr_b16 %[b7], %[rb0] offset:%[ob7]\n\t"
#define OURO_PP_B_COL_OUT                                                                         \
  [b0] "=&v"(b[0][0].lo), [b1] "=&v"(b[0][0].hi), [b2] "=&v"(b[1][0].lo), [b3] "=&v"(b[1][0].hi), \
  [b4] "=&v"(b[2][0].lo), [b5] "=&v"(b[2][0].hi), [b6] "=&v"(b[3][0].lo), [b7] "=&v"(b[3][0].hi)
#define OURO_PP_B_COL_IN                                                                                 \
  [rb0] "v"(rb[0]), [ob0] "n"(BB + 0), [ob1] "n"(BB + 1024), [ob2] "n"(BB + 4096), [ob3] "n"(BB + 5120), \
  [ob4] "n"(BB + 8192), [ob5] "n"(BB + 9216), [ob6] "n"(BB + 12288), [ob7] "n"(BB + 13312)
#define OURO_PP_READ(FA, FB) \
  asm volatile(OURO_PP_A_##FA##_TEXT OURO_PP_B_##FB##_TEXT "s_waitcnt lgkmcnt(0)" \
               : OURO_PP_A_##FA##_OUT, OURO_PP_B_##FB##_OUT : OURO_PP_A_##FA##_IN, OURO_PP_B_##FB##_IN : "memory")
template <int BA, int BB>
__device__ __forceinline__ void pp_read(PpFrag<false> (&a)[4][2], const uint32_t* ra, PpFrag<false> (&b)[4][1], const uint32_t* rb) { OURO_PP_READ(ROW, ROW); }
template <int BA, int BB>
__device__ __forceinline__ void pp_read(PpFrag<false> (&a)[4][2], const uint32_t* ra, PpFrag<true> (&b)[4][1], const uint32_t* rb) { OURO_PP_READ(ROW, COL); }
template <int BA, int BB>
__device__ __forceinline__ void pp_read(PpFrag<true> (&a)[4][2], const uint32_t* ra, PpFrag<false> (&b)[4][1], const uint32_t* rb) { OURO_PP_READ(COL, ROW); }
template <int BA, int BB>
__device__ __forceinline__ void pp_read(PpFrag<true> (&a)[4][2], const uint32_t* ra, PpFrag<true> (&b)[4][1], const uint32_t* rb) { OURO_PP_READ(COL, COL); }
// B alone
template <int BB>
__device__ __forceinline__ void pp_read(PpFrag<false> (&b)[4][1], const uint32_t* rb) {
  asm volatile(OURO_PP_B_ROW_TEXT "s_waitcnt lgkmcnt(0)" : OURO_PP_B_ROW_OUT : OURO_PP_B_ROW_IN : "memory");
}
template <int BB>
__device__ __forceinline__ void pp_read(PpFrag<true> (&b)[4][1], const uint32_t* rb) {
  asm volatile(OURO_PP_B_COL_TEXT "s_waitcnt lgkmcnt(0)" : OURO_PP_B_COL_OUT : OURO_PP_B_COL_IN : "memory");
}
#undef OURO_PP_READ
#undef OURO_PP_A_ROW_TEXT
#undef OURO_PP_A_ROW_OUT
#undef OURO_PP_A_ROW_IN
#undef OURO_PP_A_COL_TEXT
#undef OURO_PP_A_COL_OUT
#undef OURO_PP_A_COL_IN
#undef OURO_PP_B_ROW_TEXT
#undef OURO_PP_B_ROW_OUT
#undef OURO_PP_B_ROW_IN
#undef OURO_PP_B_COL_TEXT
#undef OURO_PP_B_COL_OUT
#undef OURO_PP_B_COL_IN
// plain hardware barrier: a fenced one would drain the loads in flight
__device__ __forceinline__ void pp_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}
// The wave's two requests for a half: 16 bytes per lane, the K-tile's offset `k` a scalar.
// `k` and `jump` may by themselves lie past the operand's end (a ragged last K-tile, a second half past a narrow operand): the
// range check counts the scalar offset in, and such a request reads zeros (a contraction over 65 with NaN behind it).
__device__ __forceinline__ void pp_request(const void* base, int bytes, char* dst, uint32_t voff, uint32_t k, uint32_t jump) {
  auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)dst, 16, voff, k, 0, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(dst + PP_HALF / 2), 16, voff, k + jump, 0, 0);
}

// acc[2 * row half + 32-row tile][column half] = the tile at (m0, n0) over nk K-tiles from contraction index kbeg on (nk >= 1;
// where both operands are column-form the last may be ragged).  LDS is free for reuse when the call returns.
template <bool TA, bool TB>
__device__ __forceinline__ void pp_mainloop(const GemmParams& p, int m0, int n0, int kbeg, int nk, char* lds, f32x16 (&acc)[4][2]) {
  using OA = PpOperand<TA>;
  using OB = PpOperand<!TB>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const uint32_t oa = OA::src(wave, lane, m0, p.lda), ob = OB::src(wave, lane, n0, p.ldb);
  const uint32_t jumpA = OA::jump(p.lda), jumpB = OB::jump(p.ldb), halfA = OA::half(p.lda), halfB = OB::half(p.ldb);
  const uint32_t stepA = 2u * (TA ? (uint32_t)PP_BK * p.lda : (uint32_t)PP_BK), stepB = 2u * (TB ? (uint32_t)PP_BK : (uint32_t)PP_BK * p.ldb);
  uint32_t ka = 2u * (TA ? (uint32_t)kbeg * p.lda : (uint32_t)kbeg), kb = 2u * (TB ? (uint32_t)kbeg : (uint32_t)kbeg * p.ldb);   // of K-tile kt
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  uint32_t ra[OA::template naddr<2>()], rb[OB::template naddr<1>()];
  OA::template addresses<2>(lds0, wm * 64, lane, ra);
  OB::template addresses<1>(lds0 + 4 * PP_HALF, wn * 32, lane, rb);
  char* const dst = lds + wave * 1024;
  auto reqA = [&](int st, int h, uint32_t k) __attribute__((always_inline)) { pp_request(p.A, p.bytesA, dst + (2 * st + h) * PP_HALF, oa, k + h * halfA, jumpA); };
  auto reqB = [&](int st, int h, uint32_t k) __attribute__((always_inline)) { pp_request(p.B, p.bytesB, dst + (4 + 2 * st + h) * PP_HALF, ob, k + h * halfB, jumpB); };
  PpFrag<TA> fa[4][2];
  PpFrag<!TB> fb0[2][4][1], fb1[4][1];             // B0 is read one K-tile ahead, into the set of that K-tile's parity
  auto mul = [&](int h, int j, PpFrag<!TB> (&b)[4][1]) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[2 * h + t][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][t].get(), b[ks][0].get(), acc[2 * h + t][j], 0, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i >> 1][i & 1][r] = 0.f;

  reqB(0, 0, kb); reqA(0, 0, ka); reqB(0, 1, kb); reqA(0, 1, ka);
  if (nk > 1) { reqB(1, 0, kb + stepB); reqA(1, 0, ka + stepA); reqB(1, 1, kb + stepB); pp_wait_mem<8>(); }
  else pp_wait_mem<2>();                           // all but A1 (and K-tile 1)
  pp_barrier();
  pp_read<0>(fb0[0], rb);
  pp_barrier();                                    // B0 of stage 0 may be refilled
  if (wm == 1) pp_barrier();                       // the second group stays one barrier behind
#define OURO_PP_TILE(ST)                                                                                     \
  do {                                                                                                       \
    pp_read<2 * (ST) * PP_HALF, (2 * (ST) + 1) * PP_HALF>(fa, ra, fb1, rb);                                  \
    if (kt + 1 < nk) reqA(1 - (ST), 1, ka + stepA);                                                          \
    if (kt + 2 < nk) reqB(ST, 0, kb + 2 * stepB);                                                            \
    if (kt + 2 < nk) pp_wait_mem<8>();                                                                       \
    else if (kt + 1 < nk) pp_wait_mem<2>();         /* A1 of kt+1 may be under way */                        \
    else pp_wait_mem<0>();                                                                                   \
    pp_barrier();                                                                                            \
    __builtin_amdgcn_s_setprio(1);                                                                           \
    mul(0, 0, fb0[ST]); mul(0, 1, fb1);                                                                      \
    __builtin_amdgcn_s_setprio(0);                                                                           \
    pp_barrier();                                                                                            \
    /* past the last K-tile: B0 is never used */                                                             \
    pp_read<(2 * (ST) + 1) * PP_HALF, 2 * (1 - (ST)) * PP_HALF>(fa, ra, fb0[1 - (ST)], rb);                  \
    if (kt + 2 < nk) { reqA(ST, 0, ka + 2 * stepA); reqB(ST, 1, kb + 2 * stepB); }                           \
    if (kt + 2 < nk) pp_wait_mem<8>();                                                                       \
    else pp_wait_mem<0>();                                                                                   \
    pp_barrier();                                                                                            \
    __builtin_amdgcn_s_setprio(1);                                                                           \
    mul(1, 1, fb1); mul(1, 0, fb0[ST]);                                                                      \
    __builtin_amdgcn_s_setprio(0);                                                                           \
    pp_barrier();                                                                                            \
    ka += stepA; kb += stepB;                                                                                \
  } while (0)
  int kt = 0;
  for (; kt + 1 < nk; ++kt) { OURO_PP_TILE(0); ++kt; OURO_PP_TILE(1); }
  if (kt < nk) OURO_PP_TILE(0);
#undef OURO_PP_TILE
  if (wm == 0) pp_barrier();
  __syncthreads();
}

template <bool TA, bool TB>
__global__ __launch_bounds__(512, 2) void gemm_pp_kernel(GemmParams p) {
  extern __shared__ uint4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  batch_offsets(p);
  int m0, n0, kbeg;
  tile_of_block(p, 256, 256, blockIdx.x, gridDim.x, m0, n0, kbeg);
  const int nk = (min(p.K, kbeg + p.kchunk) - kbeg + PP_BK - 1) / PP_BK;
  f32x16 acc[4][2];
  pp_mainloop<TA, TB>(p, m0, n0, kbeg, nk, reinterpret_cast<char*>(smem), acc);
  const int m_w = m0 + 64 * (wave >> 2), n_w = n0 + 32 * (wave & 3);
  mfma_epilogue<4, 2, !TA && TB, 128, 128>(p, acc, smem, m_w, n_w, lane, wave);
}

// Several accumulating products in one launch (weight gradients of a layer).  Product i owns the work items
// [first[i], first[i+1]), a multiple of 8 so that the low bits of a work item still name its XCD.
struct PpGroupParams {
  int n;
  int first[GEMM_GROUP_MAX + 1];
  GemmParams p[GEMM_GROUP_MAX];
};
static_assert(sizeof(PpGroupParams) <= 4096, "kernel arguments are limited to 4 KiB");
__global__ __launch_bounds__(512, 2) void gemm_pp_group_kernel(PpGroupParams g) {
  extern __shared__ uint4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bid = blockIdx.x;
  int i = 0;
  while (i + 1 < g.n && bid >= g.first[i + 1]) ++i;
  const GemmParams& p = g.p[i];
  int m0, n0, kbeg;
  tile_of_block(p, 256, 256, bid - g.first[i], g.first[i + 1] - g.first[i], m0, n0, kbeg);
  if (kbeg >= p.K) return;                         // a work item past the last K range (the item count is rounded up)
  f32x16 acc[4][2];
  pp_mainloop<true, false>(p, m0, n0, kbeg, (min(p.K, kbeg + p.kchunk) - kbeg + PP_BK - 1) / PP_BK, reinterpret_cast<char*>(smem), acc);
  mfma_accumulate<4, 2, 128, 128>(p, acc, m0 + 64 * (wave >> 2), n0 + 32 * (wave & 3), lane);
}

static hipError_t pp_allow_lds(const void* kern, size_t smem, bool& done) {
  if (done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  done = e == hipSuccess;
  return e;
}

hipError_t launch_gemm_pp(hipStream_t s, GemmParams& p, int transA, int transB, int splits) {
  static_assert((size_t)8 * epilogue_stage_floats<2>() * sizeof(float) <= PP_LDS, "the epilogue's patches fit the ring");
  p.tilesM = (p.M + 255) / 256;
  p.tilesN = (p.N + 255) / 256;
  p.ntiles = p.tilesM * p.tilesN;
  p.mfast = splits > 1 && p.N > p.M;
  p.band = splits == 1 && p.tilesM % 8 == 0 && p.tilesN % 8 == 0 && p.tilesN > 8;
  dim3 grid(p.ntiles * splits, p.by, p.bz), block(512);
#define OURO_LAUNCH(TA_, TB_)                                                                       \
  do {                                                                                              \
    static bool allowed = false;                                                                    \
    hipError_t e = pp_allow_lds((const void*)gemm_pp_kernel<TA_, TB_>, PP_LDS, allowed);            \
    if (e != hipSuccess) return e;                                                                  \
    hipLaunchKernelGGL((gemm_pp_kernel<TA_, TB_>), grid, block, PP_LDS, s, p);                      \
  } while (0)
  if (!transA && !transB) OURO_LAUNCH(false, false);
  else if (!transA && transB) OURO_LAUNCH(false, true);
  else if (transA && !transB) OURO_LAUNCH(true, false);
  else OURO_LAUNCH(true, true);
#undef OURO_LAUNCH
  return hipGetLastError();
}

// ps: kchunk set; accumulate as mfma_accumulate takes it.
hipError_t launch_gemm_pp_group(hipStream_t s, const GemmParams* ps, int n) {
  if (n < 1 || n > GEMM_GROUP_MAX) return hipErrorInvalidValue;
  PpGroupParams g;
  memset(&g, 0, sizeof g);
  g.n = n;
  for (int i = 0; i < n; ++i) {
    GemmParams p = ps[i];
    p.tilesM = (p.M + 255) / 256;
    p.tilesN = (p.N + 255) / 256;
    p.ntiles = p.tilesM * p.tilesN;
    p.mfast = p.N > p.M;                           // neighbouring tiles share the larger operand's columns
    p.band = 0;
    g.p[i] = p;
    g.first[i + 1] = g.first[i] + (p.ntiles * ((p.K + p.kchunk - 1) / p.kchunk) + 7) / 8 * 8;
  }
  static bool allowed = false;
  hipError_t e = pp_allow_lds((const void*)gemm_pp_group_kernel, PP_LDS, allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gemm_pp_group_kernel, dim3(g.first[n]), dim3(512), PP_LDS, s, g);
  return hipGetLastError();
}

}  // namespace ouro
