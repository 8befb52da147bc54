// Parameters and epilogues shared by the contraction kernels.
#pragma once
#include "common.h"
#include "tiles.h"

namespace ouro {

struct GemmParams {
  const void* A; const void* B; void* C;
  int M, N, K, lda, ldb, ldc;
  int out_fp32, accumulate;
  const float* bias;
  const void* residual; int ldr;
  const float* res32; int ldr32;
  const float* ln_mean; const float* ln_rstd; const float* ln_g; const float* ln_b;
  int epilogue;
  void* Z; int ldz;
  float alpha;
  int bytesA, bytesB;   // operand extents, for the buffer descriptors of the direct loads (each operand is under 2 GiB)
  int kchunk;      // K range per blockIdx.z
  int tilesN;      // tiles along N (MFMA kernel)
  int tilesM, ntiles, mfast, band;   // direct-to-LDS kernels: see tile_of_block
  int vec_epi;     // 1: C, Z, residual allow 16-byte row-chunk accesses (MFMA kernel)
  int by, bz, bz1;                          // bz1: blockIdx.z from here on belongs to the second grid of products
  const void* A2; const void* B2; void* C2; float alpha2;
  long long bAy, bAz, bBy, bBz, bCy, bCz;   // byte strides of a batch of products over blockIdx.y, blockIdx.z (direct-to-LDS kernels)
  DropDesc drop;
  float* colsum; size_t colsum_stride;      // see GemmDesc
};

// Which output tile and K range a workgroup takes.  Workgroups go to the 8 XCDs round-robin, and
// each XCD has its own L2: the grid index is turned into (XCD, position in that XCD's share)
// and the XCD's share is a contiguous run of work items, ordered so that the workgroups in
// flight together share operand tiles through that L2:
//  - with split K the K range is the slowest index, so an XCD works inside one K range (or
//    few) instead of streaming every range at once; tiles are numbered along M first when B
//    is the larger operand (neighbours then share the B tile), else along N;
//  - without split K and with tilesM a multiple of 8 an XCD owns a band of tilesM/8 tile rows
//    and walks it in groups of 8 tile columns (tilesN a multiple of 8), rows fastest: the 32 to 64 tiles in flight
//    cover (band x 8 columns), so both operands' tiles are re-used from L2 instead of one
//    operand being re-streamed for every tile row.
__device__ __forceinline__ void tile_of_block(const GemmParams& p, int BM, int BN, int bid, int nb, int& m0, int& n0, int& kbeg) {
  {
    int q = nb >> 3, r = nb & 7, x = bid & 7, idx = bid >> 3;
    if (p.band) {
      const int mb = p.tilesM >> 3, per = mb * 8;            // tile rows per XCD, tiles per full group
      const int g = idx / per, w = idx - g * per;
      m0 = (x * mb + w % mb) * BM;
      n0 = (g * 8 + w / mb) * BN;
      kbeg = 0;
      return;
    }
    bid = x * q + min(x, r) + idx;
  }
  const int kz = bid / p.ntiles;
  const int tile = bid - kz * p.ntiles;
  m0 = (p.mfast ? tile % p.tilesM : tile / p.tilesN) * BM;
  n0 = (p.mfast ? tile / p.tilesM : tile % p.tilesN) * BN;
  kbeg = kz * p.kchunk;
}

// The product this workgroup belongs to, of a batch laid over blockIdx.y and blockIdx.z.
__device__ __forceinline__ void batch_offsets(GemmParams& p) {
  int z = blockIdx.z;
  if (z >= p.bz1) { z -= p.bz1; p.A = p.A2; p.B = p.B2; p.C = p.C2; p.alpha = p.alpha2; }
  p.A = reinterpret_cast<const char*>(p.A) + blockIdx.y * p.bAy + z * p.bAz;
  p.B = reinterpret_cast<const char*>(p.B) + blockIdx.y * p.bBy + z * p.bBz;
  p.C = reinterpret_cast<char*>(p.C) + blockIdx.y * p.bCy + z * p.bCz;
  if (p.res32) p.res32 = reinterpret_cast<const float*>(reinterpret_cast<const char*>(p.res32) + blockIdx.y * p.bCy + z * p.bCz);
}

// Returns the value stored.
template <typename T>
__device__ __forceinline__ float epilogue_store(const GemmParams& p, int m, int n, float acc) {
  float v = acc * p.alpha;
  if (p.accumulate) {
    unsafeAtomicAdd(reinterpret_cast<float*>(p.C) + (size_t)m * p.ldc + n, v);
    return v;
  }
  if (p.bias) v += p.bias[n];
  if (p.drop.on) v *= drop_factor(p.drop, (uint64_t)m * p.drop.ld + n);
  if (p.epilogue == EPI_GELU) {
    reinterpret_cast<T*>(p.Z)[(size_t)m * p.ldz + n] = from_f32<T>(v);
    v = gelu_f(v);
  } else if (p.epilogue == EPI_GELUGRAD) {
    v *= gelu_grad_f(to_f32(reinterpret_cast<const T*>(p.Z)[(size_t)m * p.ldz + n]));
  }
  if (p.residual) v += to_f32(reinterpret_cast<const T*>(p.residual)[(size_t)m * p.ldr + n]);
  if (p.res32) {
    float r = p.res32[(size_t)m * p.ldr32 + n];
    if (p.ln_mean) r = (r - p.ln_mean[m]) * p.ln_rstd[m] * p.ln_g[n] + p.ln_b[n];
    v += r;
  }
  if (p.out_fp32) {
    reinterpret_cast<float*>(p.C)[(size_t)m * p.ldc + n] = v;
    return v;
  }
  const T o = from_f32<T>(v);
  reinterpret_cast<T*>(p.C)[(size_t)m * p.ldc + n] = o;
  return to_f32(o);
}
// The workgroup's copy of the column sums.
__device__ __forceinline__ float* epilogue_colsum(const GemmParams& p) { return p.colsum + (blockIdx.x & 7) * p.colsum_stride; }


// The same for R rows of one column (lanes l and l + 32 of a wave own the same column): what depends on the column is read once, and the reads of a stage go out together.
template <typename T, int R>
__device__ __forceinline__ void epilogue_column(const GemmParams& p, const int (&m)[R], int n, float (&v)[R]) {
  if (n >= p.N) return;
  bool on[R];
#pragma unroll
  for (int r = 0; r < R; ++r) { on[r] = m[r] < p.M; v[r] *= p.alpha; }
  if (p.accumulate == ACC_ATOMIC) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (on[r]) unsafeAtomicAdd(reinterpret_cast<float*>(p.C) + (size_t)m[r] * p.ldc + n, v[r]);
    return;
  }
  if (p.bias) {
    const float b = p.bias[n];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] += b;
  }
  if (p.drop.on) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] *= drop_factor(p.drop, (uint64_t)m[r] * p.drop.ld + n);
  }
  if (p.epilogue == EPI_GELU) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (on[r]) reinterpret_cast<T*>(p.Z)[(size_t)m[r] * p.ldz + n] = from_f32<T>(v[r]);
      v[r] = gelu_f(v[r]);
    }
  } else if (p.epilogue == EPI_GELUGRAD) {
    float z[R];
#pragma unroll
    for (int r = 0; r < R; ++r) z[r] = on[r] ? to_f32(reinterpret_cast<const T*>(p.Z)[(size_t)m[r] * p.ldz + n]) : 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] *= gelu_grad_f(z[r]);
  }
  if (p.residual) {
    float x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = on[r] ? to_f32(reinterpret_cast<const T*>(p.residual)[(size_t)m[r] * p.ldr + n]) : 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] += x[r];
  }
  if (p.res32) {
    float x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = on[r] ? p.res32[(size_t)m[r] * p.ldr32 + n] : 0.f;
    if (p.ln_mean) {
      float mu[R], rs[R];
#pragma unroll
      for (int r = 0; r < R; ++r) { mu[r] = on[r] ? p.ln_mean[m[r]] : 0.f; rs[r] = on[r] ? p.ln_rstd[m[r]] : 0.f; }
      const float g = p.ln_g[n], b = p.ln_b[n];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = (x[r] - mu[r]) * rs[r] * g + b;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] += x[r];
  }
  float sum = 0.f;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (!on[r]) continue;
    if (p.out_fp32) { reinterpret_cast<float*>(p.C)[(size_t)m[r] * p.ldc + n] = v[r]; sum += v[r]; }
    else { const T o = from_f32<T>(v[r]); reinterpret_cast<T*>(p.C)[(size_t)m[r] * p.ldc + n] = o; sum += to_f32(o); }
  }
  if (p.colsum) {
    sum += __shfl_xor(sum, 32, 64);
    if ((threadIdx.x & 63) < 32) unsafeAtomicAdd(epilogue_colsum(p) + n, sum);
  }
}

// Eight consecutive columns n..n+7 of row m (bf16 operands), all in range and 16-byte
// addressable: the same epilogue as epilogue_store with 16-byte accesses.  v: the accumulator's values, on return those stored.
__device__ __forceinline__ void epilogue_store8(const GemmParams& p, int m, int n, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] *= p.alpha;
  if (p.bias) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += p.bias[n + e];
  }
  if (p.drop.on) {
    const uint64_t i0 = (uint64_t)m * p.drop.ld + n;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= drop_factor(p.drop, i0 + e);
  }
  if (p.epilogue == EPI_GELU) {
    union { bf16_t h[8]; uint4 u; } z;
#pragma unroll
    for (int e = 0; e < 8; ++e) { z.h[e] = (bf16_t)v[e]; v[e] = gelu_f(v[e]); }
    *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(p.Z) + (size_t)m * p.ldz + n) = z.u;
  } else if (p.epilogue == EPI_GELUGRAD) {
    union { bf16_t h[8]; uint4 u; } z;
    z.u = *reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_t*>(p.Z) + (size_t)m * p.ldz + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f((float)z.h[e]);
  }
  if (p.residual) {
    union { bf16_t h[8]; uint4 u; } r;
    r.u = *reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_t*>(p.residual) + (size_t)m * p.ldr + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += (float)r.h[e];
  }
  if (p.res32) {
    const float4* rp = reinterpret_cast<const float4*>(p.res32 + (size_t)m * p.ldr32 + n);
    const float4 lo = rp[0], hi = rp[1];
    float r[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    if (p.ln_mean) {
      const float mu = p.ln_mean[m], rs = p.ln_rstd[m];
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = (r[e] - mu) * rs * p.ln_g[n + e] + p.ln_b[n + e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += r[e];
  }
  if (p.out_fp32) {
    float4* c = reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + (size_t)m * p.ldc + n);
    c[0] = make_float4(v[0], v[1], v[2], v[3]);
    c[1] = make_float4(v[4], v[5], v[6], v[7]);
  } else {
    union { bf16_t h[8]; uint4 u; } o;
#pragma unroll
    for (int e = 0; e < 8; ++e) { o.h[e] = (bf16_t)v[e]; v[e] = (float)o.h[e]; }
    *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(p.C) + (size_t)m * p.ldc + n) = o.u;
  }
}

// Floats of LDS each wave needs for the staged epilogue (one row of TN 32x32 tiles).
template <int TN> constexpr int epilogue_stage_floats() { return TN * 32 * 36; }

// Writes a wave's TM x TN accumulator tiles (32x32 each; column = lane%32, row =
// 8*(r/4) + 4*(lane/32) + r%4) through the epilogue.  smem must be free for reuse (all
// waves past their last operand read).  m_w, n_w: first row / column of the wave's tiles.
// Split-K accumulation adds straight from the registers (128 contiguous bytes per
// instruction).  Otherwise each wave turns one row of tiles at a time through a private
// LDS patch (row stride 36 floats) so that a lane leaves with 8 consecutive columns of one
// output row: 16-byte loads of the residual / pre-activation, 16-byte stores of the result.
// Only the register dump is unrolled; the arithmetic runs in a rolled loop over the patch.
// CS: distance in columns between the tiles of a row.
// p.accumulate: ACC_ATOMIC, others may add to the same elements of C; ACC_STORE, nothing else does and C is known to be zero.
template <int TM, int TN, int CS = 32>
__device__ __forceinline__ void mfma_accumulate(const GemmParams& p, f32x16 (&acc)[TM][TN], int m_w, int n_w, int lane) {
  const int mode = p.accumulate;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n_w + j * CS + (lane & 31);
      const int mb = m_w + i * 32 + 4 * (lane >> 5);
      float* c = reinterpret_cast<float*>(p.C) + (size_t)mb * p.ldc + n;
      if (mode == ACC_ATOMIC) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dm = 8 * (r >> 2) + (r & 3);
          if (n < p.N && mb + dm < p.M) unsafeAtomicAdd(c + (size_t)dm * p.ldc, acc[i][j][r] * p.alpha);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dm = 8 * (r >> 2) + (r & 3);
          if (n < p.N && mb + dm < p.M) c[(size_t)dm * p.ldc] = acc[i][j][r] * p.alpha;
        }
      }
    }
}
// SUM: with column sums (p.colsum).
template <int TM, int TN, int CS, bool SUM>
__device__ __forceinline__ void mfma_epilogue_rows(const GemmParams& p, f32x16 (&acc)[TM][TN], uint4* smem, int m_w, int n_w,
                                                   int lane, int wave) {
  float* stage = reinterpret_cast<float*>(smem) + wave * epilogue_stage_floats<TN>();
  const int h32 = lane >> 5, l32 = lane & 31;
  const int srow = lane >> 2, scol = (lane & 3) * 8;
  float cs[SUM ? TN : 1][8];                       // the lane's share of the column sums
#pragma unroll
  for (int j = 0; j < (SUM ? TN : 1); ++j)
#pragma unroll
    for (int e = 0; e < 8; ++e) cs[j][e] = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stage[j * (32 * 36) + (8 * (r >> 2) + 4 * h32 + (r & 3)) * 36 + l32] = acc[i][j][r];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll 1
    for (int t = 0; t < 2; ++t) {
      const int row = t * 16 + srow;
      const float* src = stage + j * (32 * 36) + row * 36 + scol;
      const int m = m_w + i * 32 + row;
      const int n = n_w + j * CS + scol;
      if (m < p.M) {
        if (p.vec_epi && n + 8 <= p.N) {
          float4 lo = *reinterpret_cast<const float4*>(src);
          float4 hi = *reinterpret_cast<const float4*>(src + 4);
          float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          epilogue_store8(p, m, n, v);
          if (SUM) {
#pragma unroll
            for (int e = 0; e < 8; ++e) cs[SUM ? j : 0][e] += v[e];
          }
        } else {
#pragma unroll 1
          for (int e = 0; e < 8; ++e)
            if (n + e < p.N) {
              const float v = epilogue_store<bf16_t>(p, m, n + e, src[e]);
              if (SUM) unsafeAtomicAdd(epilogue_colsum(p) + n + e, v);
            }
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (SUM) {
    // lanes of equal lane % 4 hold the same columns
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n_w + j * CS + scol;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float t = cs[SUM ? j : 0][e];
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) t += __shfl_xor(t, o, 64);
        if (lane < 4 && p.vec_epi && n + 8 <= p.N) unsafeAtomicAdd(epilogue_colsum(p) + n + e, t);
      }
    }
  }
}

template <int TM, int TN, int CS = 32>
__device__ __forceinline__ void mfma_epilogue(const GemmParams& p, f32x16 (&acc)[TM][TN], uint4* smem, int m_w, int n_w,
                                              int lane, int wave) {
  if (p.accumulate) mfma_accumulate<TM, TN, CS>(p, acc, m_w, n_w, lane);
  else if (p.colsum) mfma_epilogue_rows<TM, TN, CS, true>(p, acc, smem, m_w, n_w, lane, wave);
  else mfma_epilogue_rows<TM, TN, CS, false>(p, acc, smem, m_w, n_w, lane, wave);
}

}  // namespace ouro
