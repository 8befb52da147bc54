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
  int kind;        // EPIK_*: the straight-line epilogue that serves this product
  int by, bz, bz1;                          // bz1: blockIdx.z from here on belongs to the second grid of products
  const void* A2; const void* B2; void* C2; float alpha2;
  int tri;         // see GemmDesc
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

// First row of tile row i relative to the wave's: pairs of 32-row tiles lie RH apart (gemm_pp.hip: the two 128-row halves).
template <int RH> __device__ __forceinline__ constexpr int epilogue_row(int i) { return (i >> 1) * RH + (i & 1) * 32; }

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
template <int TM, int TN, int CS = 32, int RH = 64>
__device__ __forceinline__ void mfma_accumulate(const GemmParams& p, f32x16 (&acc)[TM][TN], int m_w, int n_w, int lane) {
  const int mode = p.accumulate;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n_w + j * CS + (lane & 31);
      const int mb = m_w + epilogue_row<RH>(i) + 4 * (lane >> 5);
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
template <int TM, int TN, int CS, int RH, bool SUM>
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
      const int m = m_w + epilogue_row<RH>(i) + row;
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

// The combinations a training step's products need have an epilogue of their own, in straight-line code; EPIK_GENERAL, the
// rolled form below, serves every other one (and edges that cut through a lane's columns).
//
// What bounds an epilogue is its chain of memory round trips.  Memory operations of a wave complete in order, so in a loop over
// the tile a load behind a store waits for the store's acknowledgement: 16 trips of 1-2 us on a 256x256 tile, with one
// workgroup per CU and nothing to cover them.  Here what depends on the column only (bias, LayerNorm scale and shift) is read
// once, and the residual, pre-activation or sum rows are requested several 32x32 tiles ahead of the tile that is stored.
// In the steps, rolled form and this one: logits 8192 x 32768 over 512 361 -> 312 us, 6144 x 65536 over 1024 794 -> 718; feed-forward
// products 8192 x 4096 over 1024 on 256x256 tiles (with a second stream's work beside them) 192 -> 170, 6144 x 4096 over 1024 on 128x128
// tiles 83 -> 77; 2331 x 768 on 64x64 tiles 25.0 -> 21.9; 4800 x 448 on 128x64 tiles 14.4 -> 12.8, 10.6 -> 9.5.
enum { EPIK_GENERAL = 0, EPIK_BF16 = 1, EPIK_F32 = 2, EPIK_GELU = 3, EPIK_GELUGRAD = 4, EPIK_RES_BF16 = 5, EPIK_RES_F32 = 6, EPIK_RES_LN = 7,
       EPIK_RES_BF16_DROP = 8, EPIK_RES_LN_DROP = 9 };
inline int epilogue_kind(const GemmParams& p) {
  constexpr int LIM = 1 << 21;                     // byte offsets within a wave's rows fit 32 bits
  if (!p.vec_epi || p.accumulate || p.ldc >= LIM) return EPIK_GENERAL;
  if (p.epilogue != EPI_NONE) {
    if (p.drop.on || p.out_fp32 || p.residual || p.res32 || p.ldz >= LIM) return EPIK_GENERAL;
    if (p.epilogue == EPI_GELU) return p.colsum ? EPIK_GENERAL : EPIK_GELU;
    return p.bias ? EPIK_GENERAL : EPIK_GELUGRAD;
  }
  if (p.colsum) return EPIK_GENERAL;
  if (p.res32) return !p.out_fp32 || p.ldr32 >= LIM || ((p.bias || p.drop.on) && !p.ln_mean) ? EPIK_GENERAL : !p.ln_mean ? EPIK_RES_F32 : p.drop.on ? EPIK_RES_LN_DROP : EPIK_RES_LN;
  if (p.residual) return !p.out_fp32 || p.ldr >= LIM || p.bias ? EPIK_GENERAL : p.drop.on ? EPIK_RES_BF16_DROP : EPIK_RES_BF16;
  return p.drop.on ? EPIK_GENERAL : p.out_fp32 ? EPIK_F32 : EPIK_BF16;
}

constexpr unsigned EPI_OFF = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t epilogue_rows_of(const void* base, size_t esz, int row, int ld) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(base)) + esz * (size_t)row * ld, 0, 0x7fffffff, 0x00020000);
}
template <typename T> __device__ __forceinline__ T epilogue_load(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s);
template <> __device__ __forceinline__ uint4 epilogue_load<uint4>(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0));
}
template <> __device__ __forceinline__ uint2 epilogue_load<uint2>(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
}
template <> __device__ __forceinline__ uint32_t epilogue_load<uint32_t>(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0);
}
// Without a scalar offset: behind a 16-byte buffer store that has one, the compiler lets the next instruction write the stored
// registers, and the first of them was then seen to arrive with its new value in some lanes.
__device__ __forceinline__ void epilogue_store_at(__amdgpu_buffer_rsrc_t r, uint4 x, unsigned v) {
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, x), r, v, 0, 0);
}

// A tile goes through the wave's LDS patch (row pitch 36 floats) so that a lane leaves with consecutive columns of a row:
// eight of a bf16 result (64 contiguous bytes of a row per tile), four of an fp32 one (128 bytes).
template <int KIND_, int TM, int TN, int CS, int RH>
__device__ __forceinline__ void epilogue_tiles(const GemmParams& p, f32x16 (&acc)[TM][TN], float* stage, int m_w, int n_w, int lane) {
  constexpr bool DROP = KIND_ >= EPIK_RES_BF16_DROP;
  constexpr int KIND = KIND_ == EPIK_RES_BF16_DROP ? EPIK_RES_BF16 : KIND_ == EPIK_RES_LN_DROP ? EPIK_RES_LN : KIND_;
  constexpr bool OUT32 = KIND == EPIK_F32 || KIND >= EPIK_RES_BF16, LN = KIND == EPIK_RES_LN, ROWS32 = LN || KIND == EPIK_RES_F32;
  constexpr bool READS = KIND == EPIK_GELUGRAD || KIND >= EPIK_RES_BF16, SUM = KIND == EPIK_GELUGRAD;
  constexpr bool BIAS = !READS || LN, OTHER = READS || KIND == EPIK_GELU;           // OTHER: a second matrix beside C, read or written
  constexpr int W = OUT32 ? 4 : 8, LPR = 32 / W, RPI = 64 / LPR, T = 32 / RPI;       // columns of a lane, lanes of a row, rows of an access, accesses of a tile
  constexpr int NT = TM * TN, AHEAD = !READS ? 1 : NT <= 4 ? NT : LN ? 1 : 2;
  const int lr = lane / LPR, lc = (lane % LPR) * W, h32 = lane >> 5, l32 = lane & 31;
  float bias[BIAS ? TN : 1][W], lg[LN ? TN : 1][W], lb[LN ? TN : 1][W];
  int nc[TN];
  // Addresses: a buffer descriptor at the wave's first row, a lane term per column tile and a scalar row term.  A lane whose row
  // or column is not the result's gets EPI_OFF, past every descriptor's end: it reads zero and its stores are dropped.
  unsigned vc[TN], vr[OTHER ? TN : 1];
  const int ldread = SUM || KIND == EPIK_GELU ? p.ldz : ROWS32 ? p.ldr32 : p.ldr;
  const auto rc = epilogue_rows_of(p.C, OUT32 ? 4 : 2, m_w, p.ldc);
  const auto rz = epilogue_rows_of(p.Z, 2, m_w, p.ldz);
  const auto rr = KIND == EPIK_GELUGRAD ? rz : ROWS32 ? epilogue_rows_of(p.res32, 4, m_w, p.ldr32) : epilogue_rows_of(p.residual, 2, m_w, p.ldr);
  const auto rmu = epilogue_rows_of(p.ln_mean, 4, m_w, 1), rrs = epilogue_rows_of(p.ln_rstd, 4, m_w, 1);
  const int rows = p.M - m_w;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n_w + j * CS + lc;
    const bool on = n < p.N;                       // and then n + W <= N: the caller's tiles end at a multiple of W
    nc[j] = on ? n : 0;
    vc[j] = on ? (OUT32 ? 4u : 2u) * ((unsigned)lr * (unsigned)p.ldc + (unsigned)n) : EPI_OFF;
    if (OTHER) vr[OTHER ? j : 0] = on ? (ROWS32 ? 4u : 2u) * ((unsigned)lr * (unsigned)ldread + (unsigned)n) : EPI_OFF;
#pragma unroll
    for (int e = 0; e < W; ++e) {
      if (BIAS) bias[BIAS ? j : 0][e] = p.bias ? p.bias[nc[j] + e] : 0.f;
      if (LN) { lg[LN ? j : 0][e] = p.ln_g[nc[j] + e]; lb[LN ? j : 0][e] = p.ln_b[nc[j] + e]; }
    }
  }
  // what is read, AHEAD tiles of it under way
  uint4 in[AHEAD][T];
  float mu[AHEAD][T], rs[AHEAD][T];
  auto request = [&](int s) __attribute__((always_inline)) {
    const int i = s / TN, j = READS ? s % TN : 0, a = s % AHEAD;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int dm = epilogue_row<RH>(i) + t * RPI;
      const unsigned v = lr < rows - dm ? vr[j] : EPI_OFF, row = (unsigned)dm * (unsigned)ldread;
      if (KIND == EPIK_RES_BF16) { const uint2 h = epilogue_load<uint2>(rr, v, 2u * row); in[a][t].x = h.x; in[a][t].y = h.y; }
      else in[a][t] = epilogue_load<uint4>(rr, v, (ROWS32 ? 4u : 2u) * row);
      if (LN) {
        const unsigned w = lr < rows - dm ? 4u * lr : EPI_OFF;
        mu[a][t] = __uint_as_float(epilogue_load<uint32_t>(rmu, w, 4u * dm)); rs[a][t] = __uint_as_float(epilogue_load<uint32_t>(rrs, w, 4u * dm));
      }
    }
  };
  auto dump = [&](int s) __attribute__((always_inline)) {
    float* d = stage + (s % TN) * (32 * 36) + 4 * h32 * 36 + l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) d[(8 * (r >> 2) + (r & 3)) * 36] = acc[s / TN][s % TN][r];
  };
  float cs[SUM ? TN : 1][W];                       // the lane's share of the column sums
#pragma unroll
  for (int j = 0; j < (SUM ? TN : 1); ++j)
#pragma unroll
    for (int e = 0; e < W; ++e) cs[j][e] = 0.f;
  if (READS) {
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) request(s);
  }
  dump(0);
#pragma unroll
  for (int s = 0; s < NT; ++s) {
    const int i = s / TN, j = s % TN, a = s % AHEAD;
    __builtin_amdgcn_wave_barrier();
    float v[T][W];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const float* src = stage + j * (32 * 36) + (t * RPI + lr) * 36 + lc;
#pragma unroll
      for (int q = 0; q < W / 4; ++q) {
        const float4 x = *reinterpret_cast<const float4*>(src + 4 * q);
        v[t][4 * q] = x.x; v[t][4 * q + 1] = x.y; v[t][4 * q + 2] = x.z; v[t][4 * q + 3] = x.w;
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (s + 1 < NT) dump(s + 1);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int dm = epilogue_row<RH>(i) + t * RPI;
      const bool row_on = lr < rows - dm;
      const unsigned at = row_on ? vc[j] + (OUT32 ? 4u : 2u) * (unsigned)dm * (unsigned)p.ldc : EPI_OFF;
#pragma unroll
      for (int e = 0; e < W; ++e) v[t][e] = BIAS ? v[t][e] * p.alpha + bias[BIAS ? j : 0][e] : v[t][e] * p.alpha;
      if (DROP) {
        const uint64_t i0 = (uint64_t)(m_w + dm + lr) * p.drop.ld + nc[j];
#pragma unroll
        for (int e = 0; e < W; ++e) v[t][e] *= drop_factor(p.drop, i0 + e);
      }
      if (KIND == EPIK_GELU) {
        union { bf16_t h[8]; uint4 u; } z;
#pragma unroll
        for (int e = 0; e < W; ++e) { z.h[e] = (bf16_t)v[t][e]; v[t][e] = gelu_f(v[t][e]); }
        epilogue_store_at(rz, z.u, row_on ? vr[j] + 2u * (unsigned)dm * (unsigned)p.ldz : EPI_OFF);
      }
      if (KIND == EPIK_GELUGRAD) {
        union { bf16_t h[8]; uint4 u; } z;
        z.u = in[a][t];
#pragma unroll
        for (int e = 0; e < W; ++e) v[t][e] *= gelu_grad_f((float)z.h[e]);
      }
      if (KIND == EPIK_RES_BF16) {
        union { bf16_t h[4]; uint2 u; } r;
        r.u = make_uint2(in[a][t].x, in[a][t].y);
#pragma unroll
        for (int e = 0; e < W; ++e) v[t][e] += (float)r.h[e & 3];
      }
      if (ROWS32) {
        const float r[4] = {__uint_as_float(in[a][t].x), __uint_as_float(in[a][t].y), __uint_as_float(in[a][t].z), __uint_as_float(in[a][t].w)};
#pragma unroll
        for (int e = 0; e < W; ++e) v[t][e] += LN ? (r[e & 3] - mu[a][t]) * rs[a][t] * lg[LN ? j : 0][e] + lb[LN ? j : 0][e] : r[e & 3];
      }
      if (OUT32) {
        epilogue_store_at(rc, make_uint4(__float_as_uint(v[t][0]), __float_as_uint(v[t][1]), __float_as_uint(v[t][2]), __float_as_uint(v[t][3])), at);
      } else {
        union { bf16_t h[8]; uint4 u; } o;
#pragma unroll
        for (int e = 0; e < W; ++e) o.h[e & 7] = (bf16_t)v[t][e];
        epilogue_store_at(rc, o.u, at);
        if (SUM) {
          const float keep = row_on ? 1.f : 0.f;
#pragma unroll
          for (int e = 0; e < W; ++e) {
            cs[SUM ? j : 0][e] = fmaf((float)o.h[e & 7], keep, cs[SUM ? j : 0][e]);
            asm volatile("" : "+v"(cs[SUM ? j : 0][e]));        // added here: else the tiles' terms are kept to the end, in more registers than there are
          }
        }
      }
    }
    if (READS && s + AHEAD < NT) request(s + AHEAD);
    if (NT > 4) __builtin_amdgcn_sched_barrier(0);            // else the requests of all tiles are moved up, beyond the registers there are
  }
  if (SUM && p.colsum) {
    // lanes of equal lane % 4 hold the same columns
#pragma unroll
    for (int j = 0; j < (SUM ? TN : 1); ++j)
#pragma unroll
      for (int e = 0; e < W; ++e) {
        float t = cs[j][e];
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) t += __shfl_xor(t, o, 64);
        if (lane < LPR && vc[j] != EPI_OFF) unsafeAtomicAdd(epilogue_colsum(p) + nc[j] + e, t);
      }
  }
}

// FULL: the kernel serves all kinds (products of two row-form operands, as every product with a fused epilogue is); else the plain ones.
template <int TM, int TN, bool FULL, int CS = 32, int RH = 64>
__device__ __forceinline__ void mfma_epilogue(const GemmParams& p, f32x16 (&acc)[TM][TN], uint4* smem, int m_w, int n_w,
                                              int lane, int wave) {
  if (p.accumulate) { mfma_accumulate<TM, TN, CS, RH>(p, acc, m_w, n_w, lane); return; }
  if (m_w >= p.M || n_w >= p.N) return;
  const bool fast = p.kind != EPIK_GENERAL && (n_w + (TN - 1) * CS + 32 <= p.N || p.N % 8 == 0);
  float* stage = reinterpret_cast<float*>(smem) + wave * epilogue_stage_floats<TN>();
  if (fast && p.kind == EPIK_BF16) epilogue_tiles<EPIK_BF16, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (fast && p.kind == EPIK_F32) epilogue_tiles<EPIK_F32, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (FULL && fast && p.kind == EPIK_GELU) epilogue_tiles<EPIK_GELU, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (FULL && fast && p.kind == EPIK_GELUGRAD) epilogue_tiles<EPIK_GELUGRAD, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (FULL && fast && p.kind == EPIK_RES_BF16) epilogue_tiles<EPIK_RES_BF16, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (FULL && fast && p.kind == EPIK_RES_F32) epilogue_tiles<EPIK_RES_F32, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (FULL && fast && p.kind == EPIK_RES_LN) epilogue_tiles<EPIK_RES_LN, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (FULL && fast && p.kind == EPIK_RES_BF16_DROP) epilogue_tiles<EPIK_RES_BF16_DROP, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (FULL && fast && p.kind == EPIK_RES_LN_DROP) epilogue_tiles<EPIK_RES_LN_DROP, TM, TN, CS, RH>(p, acc, stage, m_w, n_w, lane);
  else if (p.colsum) mfma_epilogue_rows<TM, TN, CS, RH, true>(p, acc, smem, m_w, n_w, lane, wave);
  else mfma_epilogue_rows<TM, TN, CS, RH, false>(p, acc, smem, m_w, n_w, lane, wave);
}

}  // namespace ouro
