// Causal attention in fp32 on the matrix cores (32x32x2 instructions), head sizes up to 64, no relative term.
//
// The fp32 matrix rate is low enough (a 32 x 32 tile of scores over 64 features: 2048 clocks) that fragments come straight
// from global memory (L2) into registers: no LDS tiles, no barriers in the loop.  What a small model lacks is parallelism,
// so a workgroup owns 32 queries (or keys) of one head and deals the 32-wide tiles of the other axis to its four waves,
// which merge through LDS at the end.  As in the bf16 kernels the softmax row stays in the lane: scores are formed
// transposed (keys x queries; queries x keys where a key owns the lane), and since an instruction's two contraction indices
// may be any pair as long as both operands agree, the accumulator register r of a tile (rows 8 (r/4) + r%4 and that + 4 in
// the two halves of the wave) is itself the operand of the next product.
// The per-row kernels (attention_plain.hip) took 90 us forward and 470 us backward at 4 x 8 heads of 64, T = 256; these
// take 21 and 50 us.
#include "common.h"
#include "tiles.h"

#include <algorithm>

namespace ouro {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct AfParams {
  int B, H, T, S, dh, Mv;
  const float *q, *k, *v, *o, *d_o;
  float *out, *lse, *dq, *dk, *dv;
  int ldq, ldk, ldv, ldo, lddo, lddq, lddk, lddv;
  float scale, scale_log2;
};

__device__ __forceinline__ int af_row(int r, int h32) { return 8 * (r >> 2) + 4 * h32 + (r & 3); }

// Row fragment: features 8 j + 4 h32 + (0..3), j < DH / 8, of the lane's row (row pointer `src`); features past dh are zero.
template <int DH, bool VEC>
__device__ __forceinline__ void af_load_row(const float* src, int dh, int h32, bool on, f32x4 (&f)[DH / 8]) {
#pragma unroll
  for (int j = 0; j < DH / 8; ++j) {
    const int c = 8 * j + 4 * h32;
    f[j] = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
      if (on && c < dh) f[j] = *reinterpret_cast<const f32x4*>(src + c);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (on && c + e < dh) f[j][e] = src[c + e];
    }
  }
}
// Column fragment: register r of tile dt holds feature 32 dt + l32 of row row0 + af_row(r, h32) (rows clamped to rmax - 1:
// what they meet in the other operand is zero, see af_check).
template <int DH>
__device__ __forceinline__ void af_load_cols(const float* base, int ld, int row0, int rmax, int dh, int h32, int l32, float (&f)[DH / 32][16]) {
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt) {
    const int c = 32 * dt + l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = min(row0 + af_row(r, h32), rmax - 1);
      f[dt][r] = c < dh ? base[(size_t)row * ld + c] : 0.f;
    }
  }
}
// acc (rows = the rows of a, columns = the rows of b) = a b^T over the features
template <int DH>
__device__ __forceinline__ f32x16 af_rows_product(const f32x4 (&a)[DH / 8], const f32x4 (&b)[DH / 8]) {
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int j = 0; j < DH / 8; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j][e], b[j][e], acc, 0, 0, 0);
  return acc;
}
// acc[dt] (rows = features) += cols^T x
template <int DH>
__device__ __forceinline__ void af_cols_product(f32x16 (&acc)[DH / 32], const float (&cols)[DH / 32][16], const f32x16& x) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(cols[dt][r], x[r], acc[dt], 0, 0, 0);
}
// The products over a tile's rows give those that a lane does not see a weight of zero, which does not keep an infinity or
// NaN out of the sum.  `bad` becomes NaN when a tile that not every lane sees whole (`part`) holds one; the workgroup then
// computes its rows once more, one at a time over the visible rows alone (af_*_rows).  The check is one instruction per
// element in the tiles on the diagonal and at the end.
template <int DH>
__device__ __forceinline__ void af_check(bool part, const float (&cols)[DH / 32][16], float& bad) {
  if (!part) return;
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) bad = fmaf(cols[dt][r], 0.f, bad);
}
// a . b over the features, in every lane
__device__ __forceinline__ float af_dot(const float* a, const float* b, int dh, int lane) { return wave_sum(lane < dh ? a[lane] * b[lane] : 0.f); }
// Four registers of one group g of a transposed tile (features 32 dt + 8 g + 4 h32 + (0..3) of the lane's row) to memory.
template <bool VEC>
__device__ __forceinline__ void af_store4(float* row, int c, int dh, f32x4 v) {
  if (VEC) {
    if (c < dh) *reinterpret_cast<f32x4*>(row + c) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < dh) row[c + e] = v[e];
  }
}

// ------------------------------------------------------------------------------ forward
__device__ __forceinline__ void af_fwd_rows(const AfParams& p, int q0, int head, int b, int wave, int lane) {
  const float* kb = p.k + (size_t)b * p.S * p.ldk + head * p.dh;
  const float* vb = p.v + (size_t)b * p.S * p.ldv + head * p.dh;
  for (int i = q0 + wave; i < min(p.T, q0 + 32); i += 4) {
    const float* q = p.q + ((size_t)b * p.T + i) * p.ldq + head * p.dh;
    const int nvis = p.Mv + i + 1;
    float mx = -INFINITY, sum = 0.f, acc = 0.f;
    for (int j = 0; j < nvis; ++j) mx = fmaxf(mx, af_dot(q, kb + (size_t)j * p.ldk, p.dh, lane) * p.scale);
    for (int j = 0; j < nvis; ++j) {
      const float e = expf(af_dot(q, kb + (size_t)j * p.ldk, p.dh, lane) * p.scale - mx);
      sum += e;
      if (lane < p.dh) acc = fmaf(e, vb[(size_t)j * p.ldv + lane], acc);
    }
    if (lane < p.dh) p.out[((size_t)b * p.T + i) * p.ldo + head * p.dh + lane] = acc / sum;
    if (lane == 0) p.lse[((size_t)b * p.H + head) * p.T + i] = mx + logf(sum);
  }
}
// (the bound on registers keeps the occupancy that the kernel has without af_check)
template <int DH, bool VEC>
__global__ __launch_bounds__(256, DH == 64 ? 2 : 3) void af_fwd_kernel(AfParams p) {
  constexpr int ND = DH / 32;
  __shared__ float so[4][ND * 16][64];
  __shared__ float sm[4][32], sl[4][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h32 = lane >> 5, l32 = lane & 31;
  const int q0 = (gridDim.x - 1 - blockIdx.x) * 32, head = blockIdx.y, b = blockIdx.z, qi = q0 + l32;   // longest rows first
  const float* qb = p.q + (size_t)b * p.T * p.ldq + head * p.dh;
  const float* kb = p.k + (size_t)b * p.S * p.ldk + head * p.dh;
  const float* vb = p.v + (size_t)b * p.S * p.ldv + head * p.dh;
  f32x4 qf[DH / 8];
  af_load_row<DH, VEC>(qb + (size_t)min(qi, p.T - 1) * p.ldq, p.dh, h32, qi < p.T, qf);
  const int nkt = (min(p.S, p.Mv + min(p.T, q0 + 32)) + 31) / 32;                  // key tiles any of the queries sees
  f32x16 oacc[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
  float m = -INFINITY, l = 0.f, bad = 0.f;
  for (int kt = wave; kt < nkt; kt += 4) {
    const int k0 = kt * 32;
    f32x4 kf[DH / 8];
    float vf[ND][16];
    af_load_row<DH, VEC>(kb + (size_t)min(k0 + l32, p.S - 1) * p.ldk, p.dh, h32, true, kf);
    af_load_cols<DH>(vb, p.ldv, k0, p.S, p.dh, h32, l32, vf);
    f32x16 s = af_rows_product<DH>(kf, qf);
    float mloc = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + af_row(r, h32);
      s[r] = key <= p.Mv + qi && key < p.S && qi < p.T ? s[r] * p.scale_log2 : -INFINITY;
      mloc = fmaxf(mloc, s[r]);
    }
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float mn = fmaxf(m, mloc), ref = mn == -INFINITY ? 0.f : mn;
    const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - ref);
    float lsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = __builtin_amdgcn_exp2f(s[r] - ref); lsum += s[r]; }
    l = l * alpha + lsum + __shfl_xor(lsum, 32, 64);
    m = mn;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
    af_check<DH>(k0 + 31 > p.Mv + q0, vf, bad);
    af_cols_product<DH>(oacc, vf, s);
  }
  if (__syncthreads_or(bad != bad)) { af_fwd_rows(p, q0, head, b, wave, lane); return; }
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) so[wave][dt * 16 + r][lane] = oacc[dt][r];
  if (h32 == 0) { sm[wave][l32] = m; sl[wave][l32] = l; }
  __syncthreads();
  if (qi >= p.T) return;
  float mm = sm[0][l32], a[4], lt = 0.f;
#pragma unroll
  for (int w = 1; w < 4; ++w) mm = fmaxf(mm, sm[w][l32]);
#pragma unroll
  for (int w = 0; w < 4; ++w) { a[w] = sm[w][l32] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sm[w][l32] - mm); lt += a[w] * sl[w][l32]; }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  float* orow = p.out + ((size_t)b * p.T + qi) * p.ldo + head * p.dh;
#pragma unroll
  for (int gg = 0; gg < ND; ++gg) {                        // groups of four registers, dealt to the waves
    const int grp = wave * ND + gg, dt = grp >> 2, g = grp & 3;
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = dt * 16 + 4 * g + e;
      v[e] = (so[0][r][lane] * a[0] + so[1][r][lane] * a[1] + so[2][r][lane] * a[2] + so[3][r][lane] * a[3]) * inv;
    }
    af_store4<VEC>(orow, 32 * dt + 8 * g + 4 * h32, p.dh, v);
  }
  if (wave == 0 && h32 == 0) p.lse[((size_t)b * p.H + head) * p.T + qi] = (mm + log2f(lt)) * 0.6931471805599453f;
}

// Sums a transposed tile set over the four waves and stores it, times `mul`, to the lane's row.
template <int DH, bool VEC>
__device__ __forceinline__ void af_reduce_store(float (&so)[4][DH / 2][64], const f32x16 (&acc)[DH / 32], float* row, int dh, float mul, bool on,
                                                int wave, int lane) {
  constexpr int ND = DH / 32;
  const int h32 = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) so[wave][dt * 16 + r][lane] = acc[dt][r];
  __syncthreads();
#pragma unroll
  for (int gg = 0; gg < ND; ++gg) {
    const int grp = wave * ND + gg, dt = grp >> 2, g = grp & 3;
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = dt * 16 + 4 * g + e;
      v[e] = (so[0][r][lane] + so[1][r][lane] + so[2][r][lane] + so[3][r][lane]) * mul;
    }
    if (on) af_store4<VEC>(row, 32 * dt + 8 * g + 4 * h32, dh, v);
  }
  __syncthreads();
}

// ------------------------------------------------------------------------------ dQ
__device__ __forceinline__ void af_dq_rows(const AfParams& p, int q0, int head, int b, int wave, int lane) {
  const float* kb = p.k + (size_t)b * p.S * p.ldk + head * p.dh;
  const float* vb = p.v + (size_t)b * p.S * p.ldv + head * p.dh;
  for (int i = q0 + wave; i < min(p.T, q0 + 32); i += 4) {
    const size_t row = (size_t)b * p.T + i, stat = ((size_t)b * p.H + head) * p.T + i;
    const float *q = p.q + row * p.ldq + head * p.dh, *dov = p.d_o + row * p.lddo + head * p.dh;
    const float D = af_dot(p.o + row * p.ldo + head * p.dh, dov, p.dh, lane), lse = p.lse[stat];
    float acc = 0.f;
    for (int j = 0; j <= p.Mv + i; ++j) {
      const float* kj = kb + (size_t)j * p.ldk;
      const float e = expf(af_dot(q, kj, p.dh, lane) * p.scale - lse);
      const float ds = e * (af_dot(dov, vb + (size_t)j * p.ldv, p.dh, lane) - D) * p.scale;
      if (lane < p.dh) acc = fmaf(ds, kj[lane], acc);
    }
    if (lane < p.dh) p.dq[row * p.lddq + head * p.dh + lane] = acc;
  }
}
// `rank` counts from the last query tile (the longest rows).
template <int DH, bool VEC>
__device__ __forceinline__ void af_bwd_dq_body(const AfParams& p, float (&so)[4][DH / 2][64], int rank, int head, int b) {
  constexpr int ND = DH / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h32 = lane >> 5, l32 = lane & 31;
  const int q0 = ((p.T + 31) / 32 - 1 - rank) * 32, qi = q0 + l32;
  const int qc = min(qi, p.T - 1);
  const float* kb = p.k + (size_t)b * p.S * p.ldk + head * p.dh;
  const float* vb = p.v + (size_t)b * p.S * p.ldv + head * p.dh;
  f32x4 qf[DH / 8], dof[DH / 8];
  af_load_row<DH, VEC>(p.q + ((size_t)b * p.T + qc) * p.ldq + head * p.dh, p.dh, h32, qi < p.T, qf);
  af_load_row<DH, VEC>(p.d_o + ((size_t)b * p.T + qc) * p.lddo + head * p.dh, p.dh, h32, qi < p.T, dof);
  const size_t stat = ((size_t)b * p.H + head) * p.T + qc;
  const float lse2 = p.lse[stat] * 1.4426950408889634f;
  float D = 0.f;
  {
    f32x4 of[DH / 8];
    af_load_row<DH, VEC>(p.o + ((size_t)b * p.T + qc) * p.ldo + head * p.dh, p.dh, h32, qi < p.T, of);
#pragma unroll
    for (int j = 0; j < DH / 8; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) D = fmaf(of[j][e], dof[j][e], D);
    D += __shfl_xor(D, 32, 64);
  }
  const int nkt = (min(p.S, p.Mv + min(p.T, q0 + 32)) + 31) / 32;
  float bad = 0.f;
  f32x16 acc[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;
  for (int kt = wave; kt < nkt; kt += 4) {
    const int k0 = kt * 32, kc = min(k0 + l32, p.S - 1);
    f32x4 kf[DH / 8], vf[DH / 8];
    float kcol[ND][16];
    af_load_row<DH, VEC>(kb + (size_t)kc * p.ldk, p.dh, h32, true, kf);
    af_load_row<DH, VEC>(vb + (size_t)kc * p.ldv, p.dh, h32, true, vf);
    af_load_cols<DH>(kb, p.ldk, k0, p.S, p.dh, h32, l32, kcol);
    f32x16 s = af_rows_product<DH>(kf, qf);
    f32x16 dp = af_rows_product<DH>(vf, dof);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + af_row(r, h32);
      const bool vis = key <= p.Mv + qi && key < p.S && qi < p.T;
      dp[r] = vis ? __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -lse2)) * (dp[r] - D) : 0.f;
    }
    af_check<DH>(k0 + 31 > p.Mv + q0, kcol, bad);
    af_cols_product<DH>(acc, kcol, dp);
  }
  if (__syncthreads_or(bad != bad)) { af_dq_rows(p, q0, head, b, wave, lane); return; }
  af_reduce_store<DH, VEC>(so, acc, p.dq + ((size_t)b * p.T + qc) * p.lddq + head * p.dh, p.dh, p.scale, qi < p.T, wave, lane);
}

// ------------------------------------------------------------------------------ dK, dV
__device__ __forceinline__ void af_dkv_rows(const AfParams& p, int k0, int head, int b, int wave, int lane) {
  const float* qb = p.q + (size_t)b * p.T * p.ldq + head * p.dh;
  const float* dob = p.d_o + (size_t)b * p.T * p.lddo + head * p.dh;
  const size_t stat = ((size_t)b * p.H + head) * p.T;
  for (int j = k0 + wave; j < min(p.S, k0 + 32); j += 4) {
    const float *kj = p.k + ((size_t)b * p.S + j) * p.ldk + head * p.dh, *vj = p.v + ((size_t)b * p.S + j) * p.ldv + head * p.dh;
    float dk = 0.f, dv = 0.f;
    for (int i = max(0, j - p.Mv); i < p.T; ++i) {
      const float *q = qb + (size_t)i * p.ldq, *dov = dob + (size_t)i * p.lddo;
      const float e = expf(af_dot(q, kj, p.dh, lane) * p.scale - p.lse[stat + i]);
      const float D = af_dot(p.o + ((size_t)b * p.T + i) * p.ldo + head * p.dh, dov, p.dh, lane);
      const float ds = e * (af_dot(dov, vj, p.dh, lane) - D) * p.scale;
      if (lane < p.dh) { dv = fmaf(e, dov[lane], dv); dk = fmaf(ds, q[lane], dk); }
    }
    if (lane < p.dh) {
      p.dk[((size_t)b * p.S + j) * p.lddk + head * p.dh + lane] = dk;
      p.dv[((size_t)b * p.S + j) * p.lddv + head * p.dh + lane] = dv;
    }
  }
}
// D = rowsum(dO * O) and the base-2 log-sum-exp of a query tile are formed by the wave that works on it: a lane holds a query's
// row of dO anyway, and the two go through LDS (`stat`) to the registers' rows.
template <int DH, bool VEC>
__device__ __forceinline__ void af_bwd_dkv_body(const AfParams& p, float (&so)[4][DH / 2][64], float (&stat)[4][64], int tile, int head, int b) {
  constexpr int ND = DH / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h32 = lane >> 5, l32 = lane & 31;
  const int k0 = tile * 32, key = k0 + l32;                // key tile 0 sees every query
  const int kc = min(key, p.S - 1);
  const float* qb = p.q + (size_t)b * p.T * p.ldq + head * p.dh;
  const float* dob = p.d_o + (size_t)b * p.T * p.lddo + head * p.dh;
  const float* lse = p.lse + ((size_t)b * p.H + head) * p.T;
  const float* ob = p.o + (size_t)b * p.T * p.ldo + head * p.dh;
  f32x4 kf[DH / 8], vf[DH / 8];
  af_load_row<DH, VEC>(p.k + ((size_t)b * p.S + kc) * p.ldk + head * p.dh, p.dh, h32, key < p.S, kf);
  af_load_row<DH, VEC>(p.v + ((size_t)b * p.S + kc) * p.ldv + head * p.dh, p.dh, h32, key < p.S, vf);
  f32x16 dk[ND], dv[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dk[dt][r] = 0.f; dv[dt][r] = 0.f; }
  const int nqt = (p.T + 31) / 32;
  float bad = 0.f;
  for (int qt = max(0, k0 - p.Mv) / 32 + wave; qt < nqt; qt += 4) {
    const int q0 = qt * 32, qc = min(q0 + l32, p.T - 1);
    f32x16 s, dp;
    {
      f32x4 f[DH / 8];
      af_load_row<DH, VEC>(qb + (size_t)qc * p.ldq, p.dh, h32, true, f);
      s = af_rows_product<DH>(f, kf);
    }
    {
      f32x4 f[DH / 8];
      af_load_row<DH, VEC>(dob + (size_t)qc * p.lddo, p.dh, h32, true, f);
      dp = af_rows_product<DH>(f, vf);
      f32x4 of[DH / 8];
      af_load_row<DH, VEC>(ob + (size_t)qc * p.ldo, p.dh, h32, true, of);
      float D = 0.f;
#pragma unroll
      for (int j = 0; j < DH / 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) D = fmaf(of[j][e], f[j][e], D);
      D += __shfl_xor(D, 32, 64);
      stat[wave][lane] = h32 ? D : lse[qc] * 1.4426950408889634f;
      __builtin_amdgcn_wave_barrier();
    }
    float l2[16], Dr[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(&stat[wave][8 * g + 4 * h32]), y = *reinterpret_cast<const f32x4*>(&stat[wave][32 + 8 * g + 4 * h32]);
#pragma unroll
      for (int e = 0; e < 4; ++e) { l2[4 * g + e] = x[e]; Dr[4 * g + e] = y[e]; }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = q0 + af_row(r, h32);
      const bool vis = key <= p.Mv + i && i < p.T && key < p.S;
      const float pv = vis ? __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -l2[r])) : 0.f;
      s[r] = pv;
      dp[r] = vis ? pv * (dp[r] - Dr[r]) : 0.f;
    }
    const bool part = k0 + 31 > p.Mv + q0 || q0 + 32 > p.T;
    float col[ND][16];
    af_load_cols<DH>(dob, p.lddo, q0, p.T, p.dh, h32, l32, col);
    af_check<DH>(part, col, bad);
    af_cols_product<DH>(dv, col, s);
    af_load_cols<DH>(qb, p.ldq, q0, p.T, p.dh, h32, l32, col);
    af_check<DH>(part, col, bad);
    af_cols_product<DH>(dk, col, dp);
  }
  if (__syncthreads_or(bad != bad)) { af_dkv_rows(p, k0, head, b, wave, lane); return; }
  af_reduce_store<DH, VEC>(so, dk, p.dk + ((size_t)b * p.S + kc) * p.lddk + head * p.dh, p.dh, p.scale, key < p.S, wave, lane);
  af_reduce_store<DH, VEC>(so, dv, p.dv + ((size_t)b * p.S + kc) * p.lddv + head * p.dh, p.dh, 1.f, key < p.S, wave, lane);
}

// dQ and dK / dV in one launch: neither waits for the other, and the light tiles of one fill in beside the heavy ones of the
// other.  Work items heaviest first: of each rank first the keys' tile, then the queries'.
// 4 x 8 heads of 64, T = 256: 61 -> 50 us (dQ 26, dK / dV 35 in two launches); 4 x 2 heads of 32, T = 32: 16.8 -> 9.3.
template <int DH, bool VEC>
__global__ __launch_bounds__(256) void af_bwd_kernel(AfParams p) {
  __shared__ __attribute__((aligned(16))) float so[4][DH / 2][64];
  __shared__ __attribute__((aligned(16))) float stat[4][64];
  const unsigned groups = p.H * p.B, nq = (p.T + 31) / 32, nk = (p.S + 31) / 32, nmin = min(nq, nk);
  // grid (nq + nk, H, B): along one axis the work items of many short streams would pass the 2^32 threads that it may have
  const unsigned i = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  unsigned rank = i / (2 * groups), r = i - rank * 2 * groups;
  bool keys = r < groups;
  if (rank >= nmin) {                                      // the longer axis' surplus
    r = i - nmin * 2 * groups;
    rank = nmin + r / groups;
    keys = nk > nq;
  }
  const unsigned g = r % groups, head = g % p.H, b = g / p.H;
  if (keys) af_bwd_dkv_body<DH, VEC>(p, so, stat, rank, head, b);
  else af_bwd_dq_body<DH, VEC>(p, so, rank, head, b);
}

// ----------------------------------------------------------------------------- dispatch
bool attn_f32_ok(int dtype, const AttnDesc& a) { return dtype == 0 && !a.rel && a.dh <= 64; }

static AfParams af_params(const AttnDesc& a) {
  AfParams p;
  p.B = a.B; p.H = a.H; p.T = a.T; p.S = a.S; p.dh = a.dh; p.Mv = a.Mv;
  p.q = (const float*)a.q; p.k = (const float*)a.k; p.v = (const float*)a.v; p.o = (const float*)a.o; p.d_o = (const float*)a.d_o;
  p.out = (float*)a.o; p.lse = a.lse; p.dq = (float*)a.dq; p.dk = (float*)a.dk; p.dv = (float*)a.dv;
  p.ldq = a.ldq; p.ldk = a.ldk; p.ldv = a.ldv; p.ldo = a.ldo; p.lddo = a.lddo; p.lddq = a.lddq; p.lddk = a.lddk; p.lddv = a.lddv;
  p.scale = a.scale; p.scale_log2 = a.scale * 1.4426950408889634f;
  return p;
}
static bool af_aligned(const AttnDesc& a, bool bwd) {
  uintptr_t ptrs = (uintptr_t)a.q | (uintptr_t)a.k | (uintptr_t)a.v | (uintptr_t)a.o;
  int lds = a.ldq | a.ldk | a.ldv | a.ldo | a.dh;
  if (bwd) { ptrs |= (uintptr_t)a.d_o | (uintptr_t)a.dq | (uintptr_t)a.dk | (uintptr_t)a.dv; lds |= a.lddo | a.lddq | a.lddk | a.lddv; }
  return !(ptrs & 15) && !(lds & 3);
}
// the narrow instances serve head sizes up to 32
#define OURO_AF(KERN, GRID, VEC)                                                                         \
  do {                                                                                                   \
    if (a.dh <= 32) {                                                                                    \
      if (VEC) hipLaunchKernelGGL((KERN<32, true>), GRID, dim3(256), 0, s, p);                           \
      else hipLaunchKernelGGL((KERN<32, false>), GRID, dim3(256), 0, s, p);                              \
    } else {                                                                                             \
      if (VEC) hipLaunchKernelGGL((KERN<64, true>), GRID, dim3(256), 0, s, p);                           \
      else hipLaunchKernelGGL((KERN<64, false>), GRID, dim3(256), 0, s, p);                              \
    }                                                                                                    \
  } while (0)
hipError_t launch_attn_fwd_f32(hipStream_t s, const AttnDesc& a) {
  AfParams p = af_params(a);
  OURO_AF(af_fwd_kernel, dim3((a.T + 31) / 32, a.H, a.B), af_aligned(a, false));
  return hipGetLastError();
}
hipError_t launch_attn_bwd_f32(hipStream_t s, const AttnDesc& a) {
  AfParams p = af_params(a);
  const bool vec = af_aligned(a, true);
  OURO_AF(af_bwd_kernel, dim3((a.T + 31) / 32 + (a.S + 31) / 32, a.H, a.B), vec);
  return hipGetLastError();
}
#undef OURO_AF

}  // namespace ouro
