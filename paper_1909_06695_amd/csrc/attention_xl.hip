// Fused causal attention with the Transformer-XL relative-position term on the matrix cores
// (bf16, head size 64):  score(i, j) = (q_i + u) . k_j + (q_i + v) . r_{Mv + i - j}.
//
// The content term is the plain kernel's product with q + u in place of q.  The position term
// of a 32-query x 64-key block only involves the 95 distances Mv + i - j of the block: the
// product of those rows of r with q + v is one more matrix product, and the element the score
// (i, j) needs sits on the diagonal Mv + i - j of it.  A lane owns a query (forward and dQ
// kernels), so that diagonal runs through the lane's own column: the product goes through a
// per-wave LDS patch and comes back shifted, and dS takes the same way back for dQ.
//
// dK and dV have no attention kernel of their own: the dQ kernel, which holds the probabilities
// P and dS of every visible pair anyway, leaves P^T and dS^T (key as row) in the workspace, and
// dV = P^T dO, dK = scale dS^T (Q + u) are contractions on the contraction kernels (one product
// per (head, batch)); dr is gathered from dS^T along its diagonals by fa_xl_dr_kernel.  A kernel
// that owns keys would have to rotate the position product across lanes element by element and
// add dr atomically from every (batch, key block): that took 418 us per layer at 16 x 16 heads,
// T = M = 384.
#include "attention_tiles.h"

#include <algorithm>

namespace ouro {

// LDS of a workgroup: two stages of K and V, the rows of r, a patch per wave.  A block needs the 192 distances
// Mv + Q0 - 64 jb + 128 - [0, 192), largest first: three groups of 64; the next block needs two of them and the 64 below.  Group t
// of block jb is at place (2 - t - jb) mod 4, so that a block fetches one group (8 KB instead of 24) into the place that no one
// reads.
constexpr int XL_NSTAGE = 2;
constexpr int XL_STAGE = 2 * TILE_BYTES;             // K, V
constexpr int XL_R = XL_NSTAGE * XL_STAGE;           // where the rows of r start
constexpr int XL_PATCHES = XL_R + 4 * TILE_BYTES;
// A wave's patch: what its 32 queries have with the 64 distances of a 32 x 32 sub-tile, a query's cells next to each other.
// fp32 position terms, then in the same memory bf16 dS.  With both pitches (68 floats, 68 halves: 34 dwords) the lanes' rows
// start at different banks, also along the diagonals.
constexpr int XL8_LD = 68;
constexpr int XL8_PATCH = 32 * XL8_LD * 4;           // bytes per wave
constexpr int XL_DS_LD = 68;
constexpr int XL_PARTS_MAX = 4;
constexpr int XL_LDS_Q8 = XL_PATCHES + 8 * XL8_PATCH;
static_assert(XL8_PATCH >= 5 * 1024 && 5 * 1024 >= 32 * XL_DS_LD * 2, "clearing the dS cells takes five writes");
static_assert(XL8_PATCH >= (32 * 64 + 2 * 64) * 4, "the sums of the bias gradients use the whole patch");
// the patch holds floats and halves in turn
typedef float xl_f32 __attribute__((may_alias));
typedef float xl_f32x4 __attribute__((ext_vector_type(4), may_alias));
typedef uint32_t xl_u32x4 __attribute__((ext_vector_type(4), may_alias));
typedef uint64_t xl_u64_at2 __attribute__((may_alias, aligned(2)));
typedef uint32_t xl_u32x2 __attribute__((ext_vector_type(2), may_alias));

// One wave's share (8 rows) of a direct load of 64 rows x 64 features into an LDS tile; the row
// index is clamped to rmax-1.
__device__ __forceinline__ void dma_tile8(const bf16_t* src, int ld, int row0, int rmax, char* tile, int wave, int lane) {
  const int row = 8 * wave + (lane >> 3);
  const int c = (lane & 7) ^ swza(row);
  const int gr = min(row0 + row, rmax - 1);
  __builtin_amdgcn_global_load_lds((gbl_void*)(src + (size_t)gr * ld + 8 * c), (lds_void*)(tile + wave * 1024), 16, 0, 0);
}
// The same for the rows row0 down to row0 - 63 of r, clamped to [0, rmax-1].
__device__ __forceinline__ void dma_tile8_down(const bf16_t* src, int ld, int row0, int rmax, char* tile, int wave, int lane) {
  const int row = 8 * wave + (lane >> 3);
  const int c = (lane & 7) ^ swza(row);
  const int gr = max(0, min(row0 - row, rmax - 1));
  __builtin_amdgcn_global_load_lds((gbl_void*)(src + (size_t)gr * ld + 8 * c), (lds_void*)(tile + wave * 1024), 16, 0, 0);
}

// q + bias for the lane's fragment features (fp32 add, rounded to bf16 once)
__device__ __forceinline__ bf16x8 add_bias(bf16x8 q, bf16x8 b) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16_t)((float)q[e] + (float)b[e]);
  return r;
}

// The lane's share of 64 features of a row in operand order, zero where row >= rows; the loads are not conditional, so that
// those of several rows are under way together (row by row under a condition a workgroup began with eight round trips to memory).
__device__ __forceinline__ void xl_load_row(const bf16_t* src, int ld, int row, int rows, int h32, uint4 (&t)[4]) {
  const bf16_t* at = src + (size_t)min(row, rows - 1) * ld + 8 * h32;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) t[ks] = *reinterpret_cast<const uint4*>(at + 16 * ks);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    if (row >= rows) t[ks] = make_uint4(0, 0, 0, 0);
}

// row of the accumulator element r of the lane's half: 8*(r/4) + 4*half + r%4
__device__ __forceinline__ constexpr int acc_row(int r, int h32) { return 8 * (r >> 2) + 4 * h32 + (r & 3); }

// 32 rows of the r window from row w0 (a multiple of 32) on, at block jb
__device__ __forceinline__ const char* xl_r_rows(const char* lds, int w0, int jb) { return lds + XL_R + ((2 - (w0 >> 6) - jb) & 3) * TILE_BYTES + (w0 & 32) * 128; }

// Position term of a 32-key sub-tile for a wave whose lanes own queries: rows [rrow0, +64) of the r window times (q + v), as
// patch[query][cell].  Key kk of the sub-tile and the lane's query meet at cell 32 - lane%32 + kk (ascending with the key: four
// keys of a lane are next to each other): added to s.
__device__ __forceinline__ void xl_position_product(const char* lds, int rrow0, int jb, const bf16x8 (&qvf)[4], char* patch, int lane) {
  const int h32 = lane >> 5, l32 = lane & 31;
  f32x16 acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int t = 0; t < 2; ++t)
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows(xl_r_rows(lds, rrow0 + 32 * t, jb), 0, ks, lane), qvf[ks], acc[t], 0, 0, 0);
  xl_f32* row = reinterpret_cast<xl_f32*>(patch) + l32 * XL8_LD + 4 * h32;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      xl_f32x4 x = {acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
      *reinterpret_cast<xl_f32x4*>(row + 32 * t + 8 * g) = x;
    }
}
__device__ __forceinline__ void xl_add_position(f32x16& s, const char* patch, int lane) {
  const int h32 = lane >> 5, l32 = lane & 31;
  const xl_f32* cell = reinterpret_cast<const xl_f32*>(patch) + l32 * XL8_LD + 32 - l32 + 4 * h32;
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] += cell[8 * (r >> 2) + (r & 3)];
}

// Forward kernel: workgroup -> (query block, part of its keys, head, batch), longest rows first over the whole launch: the
// dispatcher hands out workgroups in linear id order, so all workgroups of the last query block
// (the most keys) start first and the lighter blocks fill the slots as they free up.
__device__ __forceinline__ void xl_decode_block(int parts, int& qblk, int& part, int& head, int& b) {
  const int lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const int per = gridDim.y * gridDim.z;
  const int rest = lin % per, x = lin / per;
  qblk = (int)gridDim.x / parts - 1 - x / parts;
  part = x % parts;
  head = rest % gridDim.y;
  b = rest / gridDim.y;
}

// Both kernels below: grid (ceil(T/128), H, B); 8 waves = (4 groups of 32 queries) x (the two
// 32-key halves of a 64-key block), waves w and w + 4 (one query group) on one SIMD; one
// workgroup per CU, so two waves per SIMD (four waves owning whole 64-key blocks, one per
// SIMD, were 4 and 20 % slower).  What bounds them is the chain of a block in each wave: position
// product -> patch -> scores -> exponentials -> patch -> gradient product.  16 x 16 heads, T = M = 384: forward 72 -> 69 us, dQ 209 ->
// 156; 32 x 10 heads, T = M = 150: 38 -> 37 and 138 -> 75, by the patches in query rows (16-byte writes, dS in place as bf16 without masks
// and conversions), one r group a block, the loads of the prologue together, the sums of the bias gradients through LDS.
// Without the position path the dQ kernel takes 35 us less, without its stores 30 (both at 16 x 16 heads, before those changes).

// ------------------------------------------------------------------------------ forward
// The two key halves of a query group keep their own running maximum, sum and output; the
// second half hands its state to the first through LDS at the end.
// PARTS: the keys of a query block are dealt to p.parts workgroups (grid.x = query blocks x parts), which leave their unscaled
// output, running maximum and sum for fa_xl_merge_kernel.
template <bool PARTS>
__global__ __launch_bounds__(512) void fa_xl_fwd_kernel(FaParams p) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h32 = lane >> 5, l32 = lane & 31;
  const int qg = wave & 3, kh = wave >> 2;
  int qblk, part, head, b;
  xl_decode_block(PARTS ? p.parts : 1, qblk, part, head, b);
  const int Q0 = qblk * 128, q0 = Q0 + qg * 32, qi = q0 + l32;
  const bf16_t* qb = p.q + (size_t)b * p.T * p.ldq + head * 64;
  const bf16_t* kb = p.k + (size_t)b * p.S * p.ldk + head * 64;
  const bf16_t* vb = p.v + (size_t)b * p.S * p.ldv + head * 64;
  const bf16_t* rb = p.r + head * 64;
  char* const patch = lds + XL_PATCHES + wave * XL8_PATCH;
  bf16x8 quf[4], qvf[4];
  const int wg_last_q = min(p.T, Q0 + 128) - 1;
  const int kend = min(p.S, p.Mv + wg_last_q + 1);
  const int nkb_all = (kend + 63) / 64;
  const int jb0 = PARTS ? nkb_all * part / p.parts : 0, nkb = PARTS ? nkb_all * (part + 1) / p.parts : nkb_all;
  const bool wave_on = q0 < p.T;
  const int wave_kmax = p.Mv + min(p.T - 1, q0 + 31);
  const int rrow0 = 96 - 32 * qg + 32 * kh;                 // window row of the wave's patch cell 0
  f32x16 oacc[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
  float m = -INFINITY, l = 0.f;
  auto issue = [&](int jb) __attribute__((always_inline)) {
    char* st = lds + (jb % XL_NSTAGE) * XL_STAGE;
    dma_tile8(kb, p.ldk, jb * 64, p.S, st, wave, lane);
    dma_tile8(vb, p.ldv, jb * 64, p.S, st + TILE_BYTES, wave, lane);
    const int d0 = p.Mv + Q0 - jb * 64 + 128;             // distance of window row 0
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (t == 2 || jb == jb0) dma_tile8_down(rb, p.ldr, d0 - 64 * t, p.S, lds + XL_R + ((2 - t - jb) & 3) * TILE_BYTES, wave, lane);
  };
  if (jb0 < nkb) issue(jb0);
  {
    uint4 q[4], ub[4], vb8[4];
    xl_load_row(qb, p.ldq, qi, p.T, h32, q);
    xl_load_row(p.u + head * 64, 0, 0, 1, h32, ub);
    xl_load_row(p.vb + head * 64, 0, 0, 1, h32, vb8);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      quf[ks] = add_bias(as_bf16x8(q[ks]), as_bf16x8(ub[ks]));
      qvf[ks] = add_bias(as_bf16x8(q[ks]), as_bf16x8(vb8[ks]));
    }
  }
  for (int jb = jb0; jb < nkb; ++jb) {
    fa_wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    if (jb + 1 < nkb) issue(jb + 1);
    const char* sK = lds + (jb % XL_NSTAGE) * XL_STAGE;
    const char* sV = sK + TILE_BYTES;
    const int key0 = jb * 64 + 32 * kh;                     // first key of the wave's sub-tile
    if (wave_on && key0 <= wave_kmax) {
      const bool edge = key0 + 31 > p.Mv + q0 || key0 + 31 >= p.S || q0 + 31 >= p.T;
      xl_position_product(lds, rrow0, jb, qvf, patch, lane);
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows(sK, 32 * kh, ks, lane), quf[ks], s, 0, 0, 0);
      __builtin_amdgcn_wave_barrier();
      xl_add_position(s, patch, lane);
      __builtin_amdgcn_wave_barrier();
      float mloc = -INFINITY;
      if (edge) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = key0 + acc_row(r, h32);
          const bool vis = key <= p.Mv + qi && key < p.S && qi < p.T;
          s[r] = vis ? s[r] : -INFINITY;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, s[r]);
      mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64)) * p.scale_log2;
      const bool grow = mloc > m + 8.f;                    // lazy reference maximum, as in the plain kernel
      if (__any(grow)) {
        const float m_new = grow ? mloc : m;
        const float alpha = grow ? __builtin_amdgcn_exp2f(m - m_new) : 1.f;
        l *= alpha;
        m = m_new;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
      }
      const float neg_m = (m == -INFINITY) ? 0.f : -m;
      float lsum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, neg_m));
        lsum += s[r];
      }
      lsum += __shfl_xor(lsum, 32, 64);
      l += lsum;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        bf16x8 pb = pack_acc(s, sub);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows_t(sV, 32 * dt, 32 * kh + 16 * sub, lane), pb, oacc[dt], 0, 0, 0);
      }
    }
  }
  // merge the two key halves: state of the second through its patch (34 floats per lane)
  if (kh == 1) {
    xl_f32* mine = reinterpret_cast<xl_f32*>(patch);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[(16 * dt + r) * 64 + lane] = oacc[dt][r];
    mine[32 * 64 + lane] = m;
    mine[33 * 64 + lane] = l;
  }
  __syncthreads();
  if (kh == 0 && qi < p.T) {
    const xl_f32* other = reinterpret_cast<const xl_f32*>(lds + XL_PATCHES + (wave + 4) * XL8_PATCH);
    const float m1 = other[32 * 64 + lane], l1 = other[33 * 64 + lane];
    const float mm = fmaxf(m, m1);
    const float a0 = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mm);
    const float a1 = (m1 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m1 - mm);
    l = l * a0 + l1 * a1;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[dt][r] = oacc[dt][r] * a0 + other[(16 * dt + r) * 64 + lane] * a1;
    if (PARTS) {
      const size_t row = (((size_t)part * p.B + b) * p.H + head) * p.T + qi;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4*>(p.part_o + row * 64 + 32 * dt + 8 * g + 4 * h32) = make_float4(oacc[dt][4 * g], oacc[dt][4 * g + 1], oacc[dt][4 * g + 2], oacc[dt][4 * g + 3]);
      if (h32 == 0) *reinterpret_cast<float2*>(p.part_ml + row * 2) = make_float2(mm, l);
      return;
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    store_acc_row(p.o + ((size_t)b * p.T + qi) * p.ldo + head * 64, oacc, inv, h32);
    if (h32 == 0) p.lse[((size_t)b * p.H + head) * p.T + qi] = (mm + log2f(l)) * 0.6931471805599453f;
  }
}


// The parts' outputs, each scaled to the common maximum; 16 lanes a row.
__global__ __launch_bounds__(256) void fa_xl_merge_kernel(FaParams p) {
  const size_t rows = (size_t)p.B * p.H * p.T, row = (size_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  if (row >= rows) return;
  const int c = (threadIdx.x & 15) * 4;
  float2 ml[XL_PARTS_MAX];
  float4 o[XL_PARTS_MAX];
  float mm = -INFINITY, l = 0.f;
#pragma unroll
  for (int i = 0; i < XL_PARTS_MAX; ++i) {
    const size_t at = (size_t)min(i, p.parts - 1) * rows + row;
    ml[i] = *reinterpret_cast<const float2*>(p.part_ml + at * 2);
    o[i] = *reinterpret_cast<const float4*>(p.part_o + at * 64 + c);
    if (i < p.parts) mm = fmaxf(mm, ml[i].x);
  }
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < XL_PARTS_MAX; ++i) {
    if (i >= p.parts) continue;
    // a part none of whose keys the row sees has a zero sum and output; one whose scores are all NaN has the same maximum (the
    // maximum skips NaN), and its sum and output stay NaN
    const float a = ml[i].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[i].x - mm);
    l += ml[i].y * a;
    sum.x += o[i].x * a; sum.y += o[i].y * a; sum.z += o[i].z * a; sum.w += o[i].w * a;
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;
  const size_t i = row % p.T, bh = row / p.T, head = bh % p.H, b = bh / p.H;
  union { bf16_t h[4]; uint2 u; } x;
  x.h[0] = (bf16_t)(sum.x * inv); x.h[1] = (bf16_t)(sum.y * inv); x.h[2] = (bf16_t)(sum.z * inv); x.h[3] = (bf16_t)(sum.w * inv);
  *reinterpret_cast<uint2*>(p.o + (b * p.T + i) * p.ldo + head * 64 + c) = x.u;
  if (c == 0) p.lse[row] = (mm + log2f(l)) * 0.6931471805599453f;
}

// ---------------------------------------------------------------------------- dQ kernel
// The two key halves of a query group add their dQ through LDS at the end.  Besides dQ the
// kernel produces the gradients of the two biases (du = sum over queries of the content half of
// dq, dvb = that of the position half) and leaves what the gradients of k, v and r are
// contractions of:
//   pt  [B, H, S, t_ld]   P^T, probabilities with the key as row, bf16 (dV = P^T dO)
//   dst [B, H, S, t_ld]   dS^T, likewise (dK = scale dS^T (Q + u); dr: fa_xl_dr_kernel)
//   qu, qv, dop [B, t_ld, H * 64]   q + u, q + v, dO with rows padded to t_ld
// t_ld = T rounded up to 64; a cell of pt / dst is addressed by a 32-bit byte offset within its
// (batch, head) matrix, so S * t_ld * 2 < 2^32 (attn_xl_ok).  Every (query, key) cell in a
// computed 32-key sub-tile is written (masked cells as zero); cells outside (keys no query of
// the wave sees, rows i >= T) are never written and must be zero from the caller (they are the
// same cells for the same Mv).
__global__ __launch_bounds__(512) void fa_xl_dq_kernel(FaParams p) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h32 = lane >> 5, l32 = lane & 31;
  const int qg = wave & 3, kh = wave >> 2;                  // waves w and w + 4 share a SIMD
  // (the launch-wide heaviest-first order of the forward kernel measured 10 % slower here: the three
  // query blocks of a (batch, head) then write their parts of P^T and dS^T far apart in time)
  const int qblk = gridDim.x - 1 - blockIdx.x;
  const int head = blockIdx.y, b = blockIdx.z;
  const int Q0 = qblk * 128, q0 = Q0 + qg * 32, qi = q0 + l32;
  const bf16_t* qb = p.q + (size_t)b * p.T * p.ldq + head * 64;
  const bf16_t* dob = p.d_o + (size_t)b * p.T * p.lddo + head * 64;
  const bf16_t* ob = p.o + (size_t)b * p.T * p.ldo + head * 64;
  const bf16_t* kb = p.k + (size_t)b * p.S * p.ldk + head * 64;
  const bf16_t* vb = p.v + (size_t)b * p.S * p.ldv + head * 64;
  const bf16_t* rb = p.r + head * 64;
  char* const patch = lds + XL_PATCHES + wave * XL8_PATCH;
  bf16x8 quf[4], qvf[4], dof[4];
  // this (batch, head)'s P^T and dS^T (uniform bases; a cell's offset fits 32 bits)
  bf16_t* ptb = p.pt + ((size_t)b * p.H + head) * p.S * p.t_ld;
  bf16_t* dstb = p.dst + ((size_t)b * p.H + head) * p.S * p.t_ld;
  const int wg_last_q = min(p.T, Q0 + 128) - 1;
  const int kend = min(p.S, p.Mv + wg_last_q + 1);
  const int nkb = (kend + 63) / 64;
  const bool wave_on = q0 < p.T;
  const int wave_kmax = p.Mv + min(p.T - 1, q0 + 31);
  const int rrow0 = 96 - 32 * qg + 32 * kh;                 // window row of the wave's patch cell 0
  f32x16 dqa[2], dqb[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dqa[dt][r] = 0.f; dqb[dt][r] = 0.f; }
  auto issue = [&](int jb) __attribute__((always_inline)) {
    char* st = lds + (jb % XL_NSTAGE) * XL_STAGE;
    dma_tile8(kb, p.ldk, jb * 64, p.S, st, wave, lane);
    dma_tile8(vb, p.ldv, jb * 64, p.S, st + TILE_BYTES, wave, lane);
    const int d0 = p.Mv + Q0 - jb * 64 + 128;             // distance of window row 0
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (t == 2 || jb == 0) dma_tile8_down(rb, p.ldr, d0 - 64 * t, p.S, lds + XL_R + ((2 - t - jb) & 3) * TILE_BYTES, wave, lane);
  };
  issue(0);
  float D_q = 0.f, lse_q = 0.f;
  {
    uint4 q[4], dO[4], o[4], ub[4], vb8[4];
    xl_load_row(qb, p.ldq, qi, p.T, h32, q);
    xl_load_row(dob, p.lddo, qi, p.T, h32, dO);
    xl_load_row(ob, p.ldo, qi, p.T, h32, o);
    xl_load_row(p.u + head * 64, 0, 0, 1, h32, ub);
    xl_load_row(p.vb + head * 64, 0, 0, 1, h32, vb8);
    lse_q = p.lse[((size_t)b * p.H + head) * p.T + min(qi, p.T - 1)] * 1.4426950408889634f;
    if (qi >= p.T) lse_q = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      quf[ks] = add_bias(as_bf16x8(q[ks]), as_bf16x8(ub[ks]));
      qvf[ks] = add_bias(as_bf16x8(q[ks]), as_bf16x8(vb8[ks]));
      dof[ks] = as_bf16x8(dO[ks]);
      const bf16x8 of = as_bf16x8(o[ks]);
#pragma unroll
      for (int e = 0; e < 8; ++e) D_q += (float)of[e] * (float)dof[ks][e];
    }
    D_q += __shfl_xor(D_q, 32, 64);
    if (qi < p.T && kh == 0) {
      const size_t at = ((size_t)b * p.t_ld + qi) * (p.H * 64) + head * 64 + 8 * h32;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        *reinterpret_cast<bf16x8*>(p.qu + at + 16 * ks) = quf[ks];
        *reinterpret_cast<bf16x8*>(p.qv + at + 16 * ks) = qvf[ks];
        *reinterpret_cast<bf16x8*>(p.dop + at + 16 * ks) = dof[ks];
      }
    }
  }
  for (int jb = 0; jb < nkb; ++jb) {
    fa_wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    if (jb + 1 < nkb) issue(jb + 1);
    const char* sK = lds + (jb % XL_NSTAGE) * XL_STAGE;
    const char* sV = sK + TILE_BYTES;
    const int key0 = jb * 64 + 32 * kh;                     // first key of the wave's sub-tile
    if (wave_on && key0 <= wave_kmax) {
      const bool edge = key0 + 31 > p.Mv + q0 || key0 + 31 >= p.S || q0 + 31 >= p.T;
      xl_position_product(lds, rrow0, jb, qvf, patch, lane);
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows(sK, 32 * kh, ks, lane), quf[ks], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows(sV, 32 * kh, ks, lane), dof[ks], dp, 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();
      // key kk of the sub-tile and the lane's query meet at cell 32 - l32 + kk: the lane takes its position terms from there,
      // forms P and dS, and puts dS (without its factor `scale`: the finished gradients take it once) into the same cells of
      // the cleared patch, as bf16
      xl_add_position(s, patch, lane);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < 5; ++i) reinterpret_cast<xl_u32x4*>(patch)[64 * i + lane] = xl_u32x4{0, 0, 0, 0};
      if (edge) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = key0 + acc_row(r, h32);
          const bool vis = key <= p.Mv + qi && key < p.S && qi < p.T;
          s[r] = vis ? __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -lse_q)) : 0.f;
          dp[r] = s[r] * (dp[r] - D_q);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -lse_q));
          dp[r] = s[r] * (dp[r] - D_q);
        }
      }
      // bf16 once: the rounded dS feeds dQ below and, with P, goes to the workspace
      bf16x8 pb[2], dsb[2];
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) { pb[sub] = pack_acc(s, sub); dsb[sub] = pack_acc(dp, sub); }
      union { bf16x8 v; uint64_t q[2]; uint32_t w[4]; } pw[2], dw[2];
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) { pw[sub].v = pb[sub]; dw[sub].v = dsb[sub]; }
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<xl_u64_at2*>(patch + 2 * (l32 * XL_DS_LD + 32 - l32 + 4 * h32 + 8 * g)) = dw[g >> 1].q[g & 1];
      const unsigned at0 = ((unsigned)(key0 + 4 * h32) * (unsigned)p.t_ld + (unsigned)qi) * 2u;   // byte offset
      auto put = [&](int r) __attribute__((always_inline)) {
        const unsigned at = at0 + (unsigned)(8 * (r >> 2) + (r & 3)) * (unsigned)p.t_ld * 2u;
        *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ptb) + at) = (uint16_t)(pw[r >> 3].w[(r & 7) >> 1] >> (16 * (r & 1)));
        *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(dstb) + at) = (uint16_t)(dw[r >> 3].w[(r & 7) >> 1] >> (16 * (r & 1)));
      };
      if (key0 + 31 < p.S) {
        if (qi < p.T) {
#pragma unroll
          for (int r = 0; r < 16; ++r) put(r);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (key0 + acc_row(r, h32) < p.S && qi < p.T) put(r);
      }
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
          dqa[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows_t(sK, 32 * dt, 32 * kh + 16 * sub, lane), dsb[sub], dqa[dt], 0, 0, 0);
      __builtin_amdgcn_wave_barrier();
      // position half of dQ: the cells off the lane's diagonal band are zero
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
          const char* at = patch + l32 * (2 * XL_DS_LD) + 2 * (32 * t + 16 * sub + 4 * h32);
          union { xl_u32x2 h[2]; bf16x8 v; } g;
          g.h[0] = *reinterpret_cast<const xl_u32x2*>(at);
          g.h[1] = *reinterpret_cast<const xl_u32x2*>(at + 16);
#pragma unroll
          for (int dt = 0; dt < 2; ++dt)
            dqb[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows_t(xl_r_rows(lds, rrow0 + 32 * t, jb), 32 * dt, 16 * sub, lane), g.v, dqb[dt], 0, 0, 0);
        }
      __builtin_amdgcn_wave_barrier();
    }
  }
  // Bias gradients: sums over the workgroup's queries.  A wave puts its registers (feature x query) into its patch, lane l takes
  // the sum of one feature's 32 queries (register l / 2, half l % 2; its eight reads start at different chunks, so that 16 lanes
  // fall on 16 different ones), the workgroup's waves are added and one wave a bias adds 64 consecutive floats.  With a butterfly
  // over the lanes per register and an atomic of two lanes per feature, wave by wave, this tail took a fifth of
  // the kernel: backward pass of 32 x 10 heads, T = M = 150, 200 -> 155 us, 16 x 16 heads, T = M = 384, 400 -> 373.
  {
    const f32x16* both[2] = {dqa, dqb};
    xl_f32* mine = reinterpret_cast<xl_f32*>(patch);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
#pragma unroll
      for (int i = 0; i < 32; ++i) mine[i * 64 + lane] = both[w][i >> 4][i & 15];
      __builtin_amdgcn_wave_barrier();
      float sum = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const xl_f32x4 x = *reinterpret_cast<const xl_f32x4*>(mine + 32 * lane + 4 * ((c + (lane >> 1)) & 7));
        sum += (x.x + x.y) + (x.z + x.w);
      }
      __builtin_amdgcn_wave_barrier();
      mine[2048 + 64 * w + lane] = sum;
    }
  }
  // dQ: the second key half hands its sum to the first through its (own) patch
  if (kh == 1) {
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) reinterpret_cast<xl_f32*>(patch)[(16 * dt + r) * 64 + lane] = dqa[dt][r] + dqb[dt][r];
  }
  __syncthreads();
  if (wave < 2) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) sum += reinterpret_cast<const xl_f32*>(lds + XL_PATCHES + w * XL8_PATCH)[2048 + 64 * wave + lane];
    const int reg = lane >> 1;
    unsafeAtomicAdd((wave ? p.dvb : p.du) + head * 64 + 32 * (reg >> 4) + acc_row(reg & 15, lane & 1), sum * p.scale);
  }
  if (kh == 0 && qi < p.T) {
    const xl_f32* other = reinterpret_cast<const xl_f32*>(lds + XL_PATCHES + (wave + 4) * XL8_PATCH);
    f32x16 sum[2];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[dt][r] = dqa[dt][r] + dqb[dt][r] + other[(16 * dt + r) * 64 + lane];
    store_acc_row(p.dq + ((size_t)b * p.T + qi) * p.lddq + head * 64, sum, p.scale, h32);
  }
}


// ------------------------------------------------------------------------------ dr kernel
// dr[delta, f] += scale * sum over (b, i) of dS(b, i, j = Mv + i - delta) * (q + v)(b, i, f), from
// the dS^T the dQ kernel left (key as row).  grid (ceil(S/64) distance blocks, H, batch groups);
// 4 waves: wave = (32 of the 64 distances) x (32 of the 64 features).  Per (batch, 64 queries)
// the cells that meet the block's distances lie in 127 key rows of dS^T; they are staged in LDS
// with rows of 33 dwords, so that the lanes of a fragment read, which walk a diagonal (next
// distance = previous key row, same query column), fall on 32 different banks.  Rows outside
// [0, S) are staged as zeros.  The fragment's eight contraction slots hold the queries
// 8 (e / 4) + 4 half + e % 4 of a 16-query step, the order of the transposing LDS read that
// fetches the (q + v) operand.
constexpr int DR_LD = 132;                               // bytes per staged row
constexpr int DR_STAGE = 128 * DR_LD + TILE_BYTES;       // dS^T rows + the (q + v) tile
constexpr int XL_LDS_DR = 2 * DR_STAGE;

__global__ __launch_bounds__(256) void fa_xl_dr_kernel(FaParams p, int bpw) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h32 = lane >> 5, l32 = lane & 31;
  // Neighbouring distance blocks stage the same key rows, half of theirs, at the same step: they are kept on one XCD, whose L2
  // then serves the second reader (the launch is bound by the bytes of dS^T; consecutive workgroups go to consecutive XCDs).
  // 16 heads and batches of 384 queries, 768 distances 53.8 -> 41.0 us; 10 heads, 32 batches of 150 queries, 300 distances
  // 25.4 -> 21.5 us.
  int db = blockIdx.x, grp = blockIdx.y + gridDim.y * blockIdx.z;
  if (((gridDim.y * gridDim.z) & 7) == 0) {
    const int lin = blockIdx.x + gridDim.x * grp, slot = lin >> 3;
    db = slot % gridDim.x;
    grp = (lin & 7) + 8 * (slot / gridDim.x);
  }
  const int D0 = db * 64, head = grp % gridDim.y;
  const int b0 = grp / gridDim.y * bpw, nb = min(p.B, b0 + bpw) - b0;
  const int wd = wave & 1, wf = wave >> 1;
  const int HD = p.H * 64;
  const int nib = (p.T + 63) / 64;
  const int ib_lo = max(0, D0 - p.Mv) / 64;              // first query block with a key at these distances
  const int nper = nib - ib_lo;
  const int nit = nb * nper;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  uint4 stage[4];
  auto fetch = [&](int it) __attribute__((always_inline)) {
    const int b = b0 + it / nper, i0 = (ib_lo + it % nper) * 64;
    const int jbase = p.Mv + i0 - D0 - 63;
    const bf16_t* src = p.dst + ((size_t)b * p.H + head) * p.S * p.t_ld + i0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = tid + 256 * q, r = c >> 3, cc = c & 7, j = jbase + r;
      stage[q] = make_uint4(0, 0, 0, 0);
      if (j >= 0 && j < p.S) stage[q] = *reinterpret_cast<const uint4*>(src + (size_t)j * p.t_ld + 8 * cc);
    }
    dma_tile(p.qv + (size_t)b * p.t_ld * HD + head * 64, HD, i0, p.t_ld, lds + (it & 1) * DR_STAGE + 128 * DR_LD, wave, lane);
  };
  auto put = [&](int it) __attribute__((always_inline)) {
    char* sT = lds + (it & 1) * DR_STAGE;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = tid + 256 * q, r = c >> 3, cc = c & 7;
      uint32_t* d = reinterpret_cast<uint32_t*>(sT + r * DR_LD + cc * 16);
      d[0] = stage[q].x; d[1] = stage[q].y; d[2] = stage[q].z; d[3] = stage[q].w;
    }
  };
  if (nit > 0) { fetch(0); put(0); }
  for (int it = 0; it < nit; ++it) {
    fa_wait_vmcnt<0>();                                   // this iteration's (q + v) tile has landed
    __syncthreads();                                      // ... and every wave's share of the staged rows is written
    if (it + 1 < nit) fetch(it + 1);
    const char* sT = lds + (it & 1) * DR_STAGE;
    const char* sQ = sT + 128 * DR_LD;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      union { uint16_t h[8]; bf16x8 v; } a;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int qq = 16 * ks + 8 * (e >> 2) + 4 * h32 + (e & 3);
        const int row = qq - (32 * wd + l32) + 63;
        a.h[e] = *reinterpret_cast<const uint16_t*>(sT + row * DR_LD + qq * 2);
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, read_rows_t(sQ, 32 * wf, 16 * ks, lane), acc, 0, 0, 0);
    }
    if (it + 1 < nit) put(it + 1);                         // the other buffer: last read before the barrier above
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int delta = D0 + 32 * wd + acc_row(r, h32);
    if (delta < p.S && nit > 0) unsafeAtomicAdd(p.dr + (size_t)delta * HD + head * 64 + 32 * wf + l32, acc[r] * p.scale);
  }
}

// ----------------------------------------------------------------------------- dispatch
static inline bool xl_al16(const void* x) { return (reinterpret_cast<uintptr_t>(x) & 15) == 0; }

bool attn_xl_ok(int dtype, const AttnDesc& a) {
  if (dtype != 1 || a.dh != 64 || !a.rel) return false;
  if ((a.ldq | a.ldk | a.ldv | a.ldo | a.ldr) & 7) return false;
  if (!xl_al16(a.q) || !xl_al16(a.k) || !xl_al16(a.v) || !xl_al16(a.o) || !xl_al16(a.r) || !xl_al16(a.u) || !xl_al16(a.vb)) return false;
  if (a.d_o) {
    if ((a.lddo | a.lddq | a.lddk | a.lddv) & 7) return false;
    if (!xl_al16(a.d_o) || !xl_al16(a.dq) || !xl_al16(a.dk) || !xl_al16(a.dv)) return false;
    if ((size_t)a.S * ((a.T + 63) / 64 * 64) * 2 >= ((size_t)1 << 32)) return false;   // 32-bit offsets into P^T, dS^T
  }
  return true;
}

// Parts that the keys of a query block are dealt to.  One workgroup a CU, so a launch of few of them leaves compute units idle
// for as long as the longest row takes; six blocks of keys a part in the last query block, which sees all, pay for the second launch.
// Earlier query blocks see fewer keys (without a memory the first two blocks) and are dealt to as many parts, some of which get one block or none.
// 2 x 16 heads, T = 384 on 1152 keys of memory (96 workgroups of up to 24 blocks): 40 us; in two parts 26 and 5 for the merge.  110 drawn
// shapes with two to four parts, with and without memory: 0.65 to 0.98 of the time in one part (8 x 16 heads, T = 128 on 640: 23.6 and 23.2).
static int xl_parts(int B, int H, int T, int S) {
  const long wgs = (long)((T + 127) / 128) * H * B;
  return (int)std::max<long>(1, std::min<long>({(long)XL_PARTS_MAX, 256 / wgs, (long)(S + 63) / 64 / 6}));
}
size_t attn_fwd_parts_floats(int B, int H, int T, int S) {
  const int parts = xl_parts(B, H, T, S);
  return parts > 1 ? (size_t)parts * B * H * T * 66 : 0;
}
hipError_t launch_attn_fwd_xl(hipStream_t s, const AttnDesc& a) {
  FaParams p = fa_params(a);
  const int nq = (a.T + 127) / 128;
  p.parts = a.parts ? xl_parts(a.B, a.H, a.T, a.S) : 1;
  auto kern = p.parts > 1 ? fa_xl_fwd_kernel<true> : fa_xl_fwd_kernel<false>;
  static bool attr_done[2] = {false, false};
  if (!attr_done[p.parts > 1]) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, XL_LDS_Q8);
    if (e != hipSuccess) return e;
    attr_done[p.parts > 1] = true;
  }
  const size_t rows = (size_t)a.B * a.H * a.T;
  p.part_o = a.parts;
  p.part_ml = a.parts ? a.parts + (size_t)p.parts * rows * 64 : nullptr;
  hipLaunchKernelGGL(kern, dim3(nq * p.parts, a.H, a.B), dim3(512), XL_LDS_Q8, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.parts == 1) return e;
  hipLaunchKernelGGL(fa_xl_merge_kernel, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, s, p);
  return hipGetLastError();
}

// Workspace of the backward pass in floats: two [B, H, S, t_ld] bf16 arrays (see
// fa_xl_dq_kernel) and three [B, t_ld, H * 64] ones.
size_t attn_bwd_xl_scratch_floats(int B, int H, int T, int S) {
  const size_t t_ld = (size_t)(T + 63) / 64 * 64;
  return (2 * (size_t)B * H * S * t_ld + 3 * (size_t)B * t_ld * H * 64) / 2;
}

hipError_t launch_attn_bwd_xl(hipStream_t s, const AttnDesc& a) {
  FaParams p = fa_params(a);
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fa_xl_dq_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, XL_LDS_Q8);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int t_ld = (a.T + 63) / 64 * 64, HD = a.H * 64;
  const size_t nmat = (size_t)a.B * a.H * a.S * t_ld, npad = (size_t)a.B * t_ld * HD;
  bf16_t* w = reinterpret_cast<bf16_t*>(a.scratch);
  p.t_ld = t_ld;
  p.pt = w; p.dst = w + nmat;
  p.qu = w + 2 * nmat; p.qv = p.qu + npad; p.dop = p.qv + npad;
  // cells the kernel never writes must read as zero in the contractions below
  if (!a.scratch_clean) {
    hipError_t e = launch_fill_zero(s, w, (2 * nmat + 3 * npad) * 2);
    if (e != hipSuccess) return e;
  }
  // du, dvb and dr are accumulated into (the caller zeroes them)
  hipLaunchKernelGGL(fa_xl_dq_kernel, dim3((a.T + 127) / 128, a.H, a.B), dim3(512), XL_LDS_Q8, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // dV[b, :, h] = P^T dO ; dK[b, :, h] = scale dS^T (Q + u): one product per (head, batch)
  GemmDesc g;
  memset(&g, 0, sizeof g);
  g.M = a.S; g.N = 64; g.K = t_ld; g.lda = t_ld; g.ldb = HD; g.transA = 0; g.transB = 0;
  g.by = a.H; g.bz = a.B;
  g.sAy = (long long)a.S * t_ld; g.sAz = (long long)a.H * a.S * t_ld;
  g.sBy = 64; g.sBz = (long long)t_ld * HD;
  g.sCy = 64;
  g.tri = a.Mv + 1;                // query i sees the keys up to Mv + i
  g.A = p.pt; g.B = p.dop; g.C = a.dv; g.ldc = a.lddv; g.sCz = (long long)a.S * a.lddv; g.alpha = 1.f;
  if (a.lddk == a.lddv) {          // both grids in one launch
    g.A2 = p.dst; g.B2 = p.qu; g.C2 = a.dk; g.alpha2 = a.scale;
    e = launch_gemm(s, 1, g, 0);
    if (e != hipSuccess) return e;
  } else {
    e = launch_gemm(s, 1, g, 0);
    if (e != hipSuccess) return e;
    g.A = p.dst; g.B = p.qu; g.C = a.dk; g.ldc = a.lddk; g.sCz = (long long)a.S * a.lddk; g.alpha = a.scale;
    e = launch_gemm(s, 1, g, 0);
    if (e != hipSuccess) return e;
  }
  // dr += scale sum over (b, i) of dS at distance delta times (q + v).  Batches per workgroup: 768 workgroups are resident at
  // once, and one ends with 4096 atomic adds, as long as some six of its 64-query steps.  So at least 12 steps each while 384
  // workgroups are left: 1600 units of 3 steps (10 heads, 32 batches of 150 queries, 300 distances) as 800 workgroups 21.7 us,
  // 550 21.0, 400 19.0, 350 23.1; 3072 units of 6 steps (16 heads and batches of 384 queries, 768 distances) as 768 41.3, 576 51.
  const int ndb = (a.S + 63) / 64, steps = (a.T + 63) / 64;
  const long long units = (long long)a.B * ndb * a.H;
  const int bpw = std::max(1, (int)std::max(units / 768, std::min((long long)(12 + steps - 1) / steps, units / 384)));
  hipLaunchKernelGGL(fa_xl_dr_kernel, dim3(ndb, a.H, (a.B + bpw - 1) / bpw), dim3(256), XL_LDS_DR, s, p, bpw);
  return hipGetLastError();
}

}  // namespace ouro
