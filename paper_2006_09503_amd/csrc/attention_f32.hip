// fp32 masked-softmax attention on the gfx950 matrix cores (v_mfma_f32_32x32x2_f32), forward and backward, any head
// size that is a multiple of 8 up to 128.  Operands, scores, probabilities and accumulators are fp32 throughout.
//
// What bounds it: the fp32 matrix rate (64 cycles per 32x32x2 instruction and SIMD) once there is work for every
// SIMD, and latency below that.  Microbatches of the fp32 mode are small (16 heads x 512 queries are 256 blocks of 32
// queries), so a workgroup owns only ONE block of 32 rows (queries in the forward and dQ kernels, keys in dK/dV) and
// its four waves take every fourth tile of 32 rows of the streamed side; their partial results meet in LDS once, at
// the end, in a fixed order.  Inside the loop nothing is shared: an MFMA of this shape needs one float per lane and
// operand, which a wave loads from L2 straight into its fragment registers (16 bytes per lane along the head for the
// row operands, 128-byte rows for the column operands), one step ahead of their use.  No LDS, no barrier.
// Measured at b=2 s=512 a=8 dh=64, causal, against one thread per row on the vector ALU: forward 520 -> 18 us, dQ with
// delta 423 -> 26, dK/dV 723 -> 33; the matrix instructions alone are 7, 10 and 14 us of the longest workgroup.
//
// v_mfma_f32_32x32x2_f32: lane l supplies element (l % 32, l / 32) of the first operand (32 x 2) and (l / 32, l % 32) of
// the second (2 x 32); it receives column l % 32 of the result, rows 8*(r/4) + 4*(l/32) + (r%4) in register r.  The two
// k-slots of an instruction may be any two indices as long as both operands agree:
//   * products over the head dimension: instruction 4j+i takes head columns 8j+i (lanes 0..31) and 8j+4+i (lanes
//     32..63), so a lane's four values of step j are 16 contiguous bytes of its row;
//   * products over keys (queries): instruction r takes the rows that register r of a result block holds, so scores
//     are second operands as they stand.
//
// Masks: a masked score is replaced by -inf before the exponential and its dS by zero, so what the masked positions
// hold does not matter, with one exception: the products over keys (queries) multiply a zero probability with the
// row of a position that some of the block's rows may not see.  Only tiles on the diagonal of a causal mask have such
// rows, and 0 * x is 0 unless x is infinite or NaN; there accumulate_visible keeps those out of the rows that must
// not see them.
#include "kernels.hpp"

namespace k2bw {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Waves per workgroup (NW): four, which split the streamed rows, or one where a launch has blocks enough without that (one_wave)
constexpr int kManyWaves = 4;
constexpr int kRows = 32;               // rows a workgroup owns
constexpr float kLog2e = 1.4426950408889634f;

template <int DH>
struct CfgF {
  static constexpr int NF = DH / 2;                  // fragment registers of a row operand
  static constexpr int DB = (DH + 31) / 32;          // 32-column blocks of a result
  static constexpr int LD = DB * 32 + 4;             // floats per row of a result strip in LDS
};

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

__device__ __forceinline__ int reg_row(int r, int hf) { return 8 * (r >> 2) + 4 * hf + (r & 3); }

// Row operand: this lane's row (already inside the matrix), head columns 8j + 4*hf .. +3 in f[4j ..]; columns past dh are zero.
template <int DH>
__device__ __forceinline__ void load_row(const float* __restrict__ row, int dh, int hf, float (&f)[CfgF<DH>::NF]) {
#pragma unroll
  for (int j = 0; j < DH / 8; ++j) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (8 * j < dh) v = *reinterpret_cast<const float4*>(row + 8 * j + 4 * hf);   // dh is a multiple of 8: uniform
    f[4 * j] = v.x; f[4 * j + 1] = v.y; f[4 * j + 2] = v.z; f[4 * j + 3] = v.w;
  }
}

// Column operand of the 32 rows at `tile` (uniform): f[db][r] = tile[reg_row(r)][32*db + l32]; rows from `rows` on are zero,
// columns past dh hold a copy of the last one (they only reach result columns that are never stored).  In a whole tile a
// row's address is scalar and the lane's offset the same for all rows.
template <int DH>
__device__ __forceinline__ void load_cols(const float* __restrict__ tile, int ld, int rows, int dh, int l32, int hf,
                                          float (&f)[CfgF<DH>::DB][16]) {
  constexpr int DB = CfgF<DH>::DB;
  uint32_t col[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) col[db] = (uint32_t)min(db * 32 + l32, dh - 1);
  if (rows >= 32) {
    const uint32_t half = (uint32_t)(4 * hf * ld);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* __restrict__ row = tile + (int64_t)reg_row(r, 0) * ld;
#pragma unroll
      for (int db = 0; db < DB; ++db) f[db][r] = row[half + col[db]];
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = reg_row(r, hf);
      const uint32_t at = (uint32_t)(min(row, rows - 1) * ld);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const float v = tile[at + col[db]];
        f[db][r] = row < rows ? v : 0.f;
      }
    }
  }
}

// acc (32 x 32) += A * B over the head dimension
template <int DH>
__device__ __forceinline__ void mul_rows(const float (&a)[CfgF<DH>::NF], const float (&b)[CfgF<DH>::NF], f32x16& acc) {
#pragma unroll
  for (int i = 0; i < CfgF<DH>::NF; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
}

// The operand a workgroup keeps for its own 32 rows (Q and dO in dQ, K and V in dK/dV), the same for all four waves: in
// fragment registers, or for large heads, where the accumulators and the streamed operands need those, in LDS (rows of
// DH + 4 floats: the 16-byte reads of 16 consecutive rows fall on all banks).
template <int DH, int NW, bool IN_LDS>
struct Resident {
  float f[CfgF<DH>::NF];
  __device__ __forceinline__ void load(const float* __restrict__ row, int dh, int, int hf, int, float*) { load_row<DH>(row, dh, hf, f); }
  __device__ __forceinline__ void mul(const float (&x)[CfgF<DH>::NF], f32x16& acc, const float*, int, int) const { mul_rows<DH>(x, f, acc); }
};
template <int DH, int NW>
struct Resident<DH, NW, true> {
  static constexpr int LDR = DH + 4;
  // every wave writes its share of the columns of all 32 rows; the caller synchronises
  __device__ __forceinline__ void load(const float* __restrict__ row, int dh, int l32, int hf, int wave, float* rows) {
    for (int j = wave; j < DH / 8; j += NW) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (8 * j < dh) v = *reinterpret_cast<const float4*>(row + 8 * j + 4 * hf);
      *reinterpret_cast<float4*>(rows + l32 * LDR + 8 * j + 4 * hf) = v;
    }
  }
  __device__ __forceinline__ void mul(const float (&x)[CfgF<DH>::NF], f32x16& acc, const float* rows, int l32, int hf) const {
#pragma unroll
    for (int j = 0; j < DH / 8; ++j) {
      const float4 v = *reinterpret_cast<const float4*>(rows + l32 * LDR + 8 * j + 4 * hf);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[4 * j], v.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[4 * j + 1], v.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[4 * j + 2], v.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[4 * j + 3], v.w, acc, 0, 0, 0);
    }
  }
};
template <int DH, int NW> constexpr int strip_floats() { return NW * kRows * CfgF<DH>::LD; }
template <int DH> constexpr int resident_floats() { return kRows * (DH + 4); }
template <int DH> constexpr bool kDqLds = DH >= 112;
template <int DH> constexpr bool kDkvLds = DH >= 48;

// out[db] += X^T P over the 32 rows of a tile
template <int DH>
__device__ __forceinline__ void mul_cols(const float (&x)[CfgF<DH>::DB][16], const f32x16& p, f32x16 (&out)[CfgF<DH>::DB]) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int db = 0; db < CfgF<DH>::DB; ++db) out[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[db][r], p[r], out[db], 0, 0, 0);
}

template <int DH>
__device__ __forceinline__ bool any_not_finite(const float (&x)[CfgF<DH>::DB][16]) {
  bool bad = false;
#pragma unroll
  for (int db = 0; db < CfgF<DH>::DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) bad = bad || !(fabsf(x[db][r]) < INFINITY);
  return __any(bad);
}

// mul_cols for a tile in which not every lane's row (query or key) sees every row of the tile, when the tile holds
// infinities or NaNs: row by row, added only where it is seen (sees(row)).  Rare, so it keeps few registers: the
// weights pass through `p_lds` (32 x 32 floats of this wave), the rows come from `tile` again.
template <int DH, typename Sees>
__device__ __forceinline__ void accumulate_visible(const float* __restrict__ tile, int64_t ld, int rows, int dh, const f32x16& p,
                                                   f32x16 (&out)[CfgF<DH>::DB], float* p_lds, int l32, int hf, Sees&& sees) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
  for (int r = 0; r < 16; ++r) p_lds[reg_row(r, hf) * 32 + l32] = p[r];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll 1
  for (int row = 0; row < rows; ++row) {
    const float w = p_lds[row * 32 + l32];
    const bool vis = sees(row);
    const float* x = tile + row * ld + 4 * hf;
#pragma unroll
    for (int db = 0; db < CfgF<DH>::DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (db * 32 + 8 * g >= dh) continue;   // (a multiple of 8: uniform)
        const float4 v = *reinterpret_cast<const float4*>(x + db * 32 + 8 * g);
        if (vis) {
          out[db][4 * g] = fmaf(w, v.x, out[db][4 * g]);
          out[db][4 * g + 1] = fmaf(w, v.y, out[db][4 * g + 1]);
          out[db][4 * g + 2] = fmaf(w, v.z, out[db][4 * g + 2]);
          out[db][4 * g + 3] = fmaf(w, v.w, out[db][4 * g + 3]);
        }
      }
  }
}

// This wave's 32 x DH partial result (lane % 32 = row, registers = head columns), times f, into its strip
template <int DH>
__device__ __forceinline__ void put_strip(const f32x16 (&acc)[CfgF<DH>::DB], float f, float* strip, int l32, int hf) {
#pragma unroll
  for (int db = 0; db < CfgF<DH>::DB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(strip + l32 * CfgF<DH>::LD + db * 32 + 8 * g + 4 * hf) =
          make_float4(acc[db][4 * g] * f, acc[db][4 * g + 1] * f, acc[db][4 * g + 2] * f, acc[db][4 * g + 3] * f);
}

// Sum of the waves' strips, times row_scale(row), to out[row][0 .. dh) for the first `rows` rows
template <int DH, int NW, typename Scale>
__device__ __forceinline__ void sum_strips(const float* strips, float* __restrict__ out, int64_t ld, int rows, int dh, int tid,
                                           Scale&& row_scale) {
  constexpr int kStrip = kRows * CfgF<DH>::LD;
  const int per_row = dh / 4;
  for (int e = tid; e < kRows * per_row; e += NW * 64) {
    const int row = e / per_row, c = e % per_row;
    if (row >= rows) break;
    float4 t = *reinterpret_cast<const float4*>(strips + row * CfgF<DH>::LD + 4 * c);
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float4 v = *reinterpret_cast<const float4*>(strips + w * kStrip + row * CfgF<DH>::LD + 4 * c);
      t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
    }
    const float f = row_scale(row);
    *reinterpret_cast<float4*>(out + row * ld + 4 * c) = make_float4(t.x * f, t.y * f, t.z * f, t.w * f);
  }
}

// ------------------------------------------------------------------------------------------------
// forward: lane = query, registers = keys (S^T = K Q^T, O^T = V^T P^T)
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, 1) void attn_f32_fwd_kernel(const float* __restrict__ qkv, float* __restrict__ o, float* __restrict__ lse,
                                                                    int s, int a, int dh, int mask_mode, const int32_t* __restrict__ seqlens) {
  using C = CfgF<DH>;
  extern __shared__ __attribute__((aligned(16))) float smem[];   // strips, then m[NW][32], l[NW][32]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int n = blockIdx.y, head = blockIdx.x;
  const bool causal = mask_mode == 1;
  const int blk = causal ? (int)(gridDim.z - 1 - blockIdx.z) : (int)blockIdx.z;   // the blocks with the most keys first
  const int i0 = blk * kRows, i = i0 + l32;
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const float* base = qkv + (int64_t)n * s * ld + head * dh;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;
  const float scale = 1.0f / sqrtf((float)dh), c = scale * kLog2e;

  float qf[C::NF], kf[C::NF], vc[C::DB][16];
  load_row<DH>(base + (int64_t)min(i, s - 1) * ld, dh, hf, qf);
  f32x16 oacc[C::DB];
#pragma unroll
  for (int db = 0; db < C::DB; ++db) oacc[db] = zero16();
  float m_i = -INFINITY, l_i = 0.f;
  const int jend = causal ? min(i0 + kRows, s) : kv_len;
  const int ntiles = (jend + 31) / 32;
  auto load_k = [&](int t) { load_row<DH>(base + h + (int64_t)min(t * 32 + l32, jend - 1) * ld, dh, hf, kf); };
  if (wave < ntiles) load_k(wave);
  for (int t = wave; t < ntiles; t += NW) {
    const int j0 = t * 32;
    load_cols<DH>(base + 2 * h + (int64_t)j0 * ld, (int)ld, jend - j0, dh, l32, hf, vc);
    __builtin_amdgcn_sched_barrier(0);   // V travels while the scores are computed
    f32x16 sc = zero16();
    mul_rows<DH>(kf, qf, sc);
    __builtin_amdgcn_sched_barrier(0);
    if (t + NW < ntiles) load_k(t + NW);   // the next tile's K travels under the softmax and the second product
    __builtin_amdgcn_sched_barrier(0);
    const bool diag = causal && j0 + 31 > i0;
    if (diag || j0 + 32 > jend) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = j0 + reg_row(r, hf);
        sc[r] = key < jend && (!causal || key <= i) ? sc[r] : -INFINITY;
      }
    }
    float mloc = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mloc = fmaxf(mloc, sc[r]);
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float m_new = fmaxf(m_i, mloc);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;   // nothing visible so far
    const float alpha = __builtin_amdgcn_exp2f((m_i - m_use) * c);
    float rowsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = __builtin_amdgcn_exp2f((sc[r] - m_use) * c);
      rowsum += sc[r];
    }
    l_i = l_i * alpha + rowsum;
    m_i = m_new;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
    if (diag && any_not_finite<DH>(vc)) accumulate_visible<DH>(base + 2 * h + (int64_t)j0 * ld, ld, min(jend - j0, 32), dh, sc, oacc, smem + wave * kRows * C::LD, l32, hf, [&](int row) { return j0 + row <= i; });
    else mul_cols<DH>(vc, sc, oacc);
  }
  // the waves' maxima meet, every partial result is rescaled to the common one
  float* m_lds = smem + NW * kRows * C::LD;
  float* l_lds = m_lds + NW * kRows;
  l_i += __shfl_xor(l_i, 32, 64);
  if (hf == 0) m_lds[wave * kRows + l32] = m_i;
  __syncthreads();
  float m = m_lds[l32];
#pragma unroll
  for (int w = 1; w < NW; ++w) m = fmaxf(m, m_lds[w * kRows + l32]);
  // a wave without a visible key adds nothing; one whose scores are all NaN has the same maximum, and its l, which is NaN, stays
  const float f = m_i == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_i - m) * c);
  if (hf == 0) l_lds[wave * kRows + l32] = l_i * f;
  put_strip<DH>(oacc, f, smem + wave * kRows * C::LD, l32, hf);
  __syncthreads();
  auto total = [&](int row) {
    float t = l_lds[row];
#pragma unroll
    for (int w = 1; w < NW; ++w) t += l_lds[w * kRows + row];
    return t;
  };
  sum_strips<DH, NW>(smem, o + ((int64_t)n * s + i0) * h + head * dh, h, s - i0, dh, tid, [&](int row) { return 1.0f / total(row); });
  if (wave == 0 && hf == 0 && i < s) lse[((int64_t)n * a + head) * s + i] = m * scale + logf(total(l32));
}

// ------------------------------------------------------------------------------------------------
// dQ (and delta = rowsum(dO * O), which the dK/dV kernel reads): the forward's orientation
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, 1) void attn_f32_dq_kernel(const float* __restrict__ qkv, const float* __restrict__ o,
                                                                   const float* __restrict__ d_o, const float* __restrict__ lse,
                                                                   float* __restrict__ delta, float* __restrict__ dqkv, int s, int a, int dh,
                                                                   int mask_mode, const int32_t* __restrict__ seqlens) {
  using C = CfgF<DH>;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int n = blockIdx.y, head = blockIdx.x;
  const bool causal = mask_mode == 1;
  const int blk = causal ? (int)(gridDim.z - 1 - blockIdx.z) : (int)blockIdx.z;
  const int i0 = blk * kRows, i = i0 + l32, ic = min(i, s - 1);
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const float* base = qkv + (int64_t)n * s * ld + head * dh;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;
  const float scale = 1.0f / sqrtf((float)dh), c = scale * kLog2e;

  float kf[C::NF], vf[C::NF], kc[C::DB][16];
  Resident<DH, NW, kDqLds<DH>> q, g;
  float* q_lds = smem + strip_floats<DH, NW>();
  float* g_lds = q_lds + resident_floats<DH>();
  const float* g_row = d_o + ((int64_t)n * s + ic) * h + head * dh;
  q.load(base + (int64_t)ic * ld, dh, l32, hf, wave, q_lds);
  g.load(g_row, dh, l32, hf, wave, g_lds);
  if (kDqLds<DH>) __syncthreads();
  float delta_i;
  {
    float of[C::NF], gf[C::NF];
    load_row<DH>(o + ((int64_t)n * s + ic) * h + head * dh, dh, hf, of);
    load_row<DH>(g_row, dh, hf, gf);
    float part = 0.f;
#pragma unroll
    for (int e = 0; e < C::NF; ++e) part = fmaf(gf[e], of[e], part);
    delta_i = part + __shfl_xor(part, 32, 64);
    if (wave == 0 && hf == 0 && i < s) delta[((int64_t)n * a + head) * s + i] = delta_i;
  }
  const float lse_i = lse[((int64_t)n * a + head) * s + ic];
  f32x16 dq[C::DB];
#pragma unroll
  for (int db = 0; db < C::DB; ++db) dq[db] = zero16();
  const int jend = causal ? min(i0 + kRows, s) : kv_len;
  const int ntiles = (jend + 31) / 32;
  auto load_kv = [&](int t) {
    const float* row = base + h + (int64_t)min(t * 32 + l32, jend - 1) * ld;
    load_row<DH>(row, dh, hf, kf);
    load_row<DH>(row + h, dh, hf, vf);
  };
  // large heads: rows of the next tile are not requested ahead, and the column operand only once the rows are used up
  constexpr bool kAhead = DH <= 96;
  if (kAhead && wave < ntiles) load_kv(wave);
  for (int t = wave; t < ntiles; t += NW) {
    const int j0 = t * 32;
    if (!kAhead) load_kv(t);
    auto load_k_cols = [&] { load_cols<DH>(base + h + (int64_t)j0 * ld, (int)ld, jend - j0, dh, l32, hf, kc); };
    if (kAhead) load_k_cols();
    __builtin_amdgcn_sched_barrier(0);
    f32x16 sc = zero16(), dp = zero16();
    q.mul(kf, sc, q_lds, l32, hf);
    g.mul(vf, dp, g_lds, l32, hf);
    __builtin_amdgcn_sched_barrier(0);
    if (!kAhead) load_k_cols();
    if (kAhead && t + NW < ntiles) load_kv(t + NW);
    __builtin_amdgcn_sched_barrier(0);
    const bool diag = causal && j0 + 31 > i0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = j0 + reg_row(r, hf);
      const bool vis = key < jend && (!causal || key <= i);
      const float p = __builtin_amdgcn_exp2f(fmaf(sc[r], scale, -lse_i) * kLog2e);
      sc[r] = vis ? p * (dp[r] - delta_i) : 0.f;   // dS^T (the scale is applied at the end)
    }
    if (diag && any_not_finite<DH>(kc)) accumulate_visible<DH>(base + h + (int64_t)j0 * ld, ld, min(jend - j0, 32), dh, sc, dq, smem + wave * kRows * C::LD, l32, hf, [&](int row) { return j0 + row <= i; });
    else mul_cols<DH>(kc, sc, dq);
  }
  put_strip<DH>(dq, scale, smem + wave * kRows * C::LD, l32, hf);
  __syncthreads();
  sum_strips<DH, NW>(smem, dqkv + ((int64_t)n * s + i0) * ld + head * dh, ld, s - i0, dh, tid, [](int) { return 1.0f; });
}

// ------------------------------------------------------------------------------------------------
// dK, dV: lane = key, registers = queries (S = Q K^T, dV^T = dO^T P, dK^T = Q^T dS)
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, 1) void attn_f32_dkv_kernel(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                                    const float* __restrict__ lse, const float* __restrict__ delta,
                                                                    float* __restrict__ dqkv, int s, int a, int dh, int mask_mode,
                                                                    const int32_t* __restrict__ seqlens) {
  using C = CfgF<DH>;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int n = blockIdx.y, head = blockIdx.x, blk = blockIdx.z;   // causal: the first keys are seen by the most queries
  const bool causal = mask_mode == 1;
  const int j0 = blk * kRows, j = j0 + l32, jc = min(j, s - 1);
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const float* base = qkv + (int64_t)n * s * ld + head * dh;
  const float* gbase = d_o + (int64_t)n * s * h + head * dh;
  const float* lse_row = lse + ((int64_t)n * a + head) * s;
  const float* delta_row = delta + ((int64_t)n * a + head) * s;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;
  const float scale = 1.0f / sqrtf((float)dh);

  float qf[C::NF], gf[C::NF], qc[C::DB][16], gc[C::DB][16];
  Resident<DH, NW, kDkvLds<DH>> k, v;
  float* k_lds = smem + strip_floats<DH, NW>();
  float* v_lds = k_lds + resident_floats<DH>();
  k.load(base + h + (int64_t)jc * ld, dh, l32, hf, wave, k_lds);
  v.load(base + 2 * h + (int64_t)jc * ld, dh, l32, hf, wave, v_lds);
  if (kDkvLds<DH>) __syncthreads();
  f32x16 dk[C::DB], dv[C::DB];
#pragma unroll
  for (int db = 0; db < C::DB; ++db) { dk[db] = zero16(); dv[db] = zero16(); }
  // query tiles that can see a key of the block: none if the block is padding, from the block itself on if causal
  const int t0 = causal ? blk : 0;
  const int t1 = j0 >= kv_len ? t0 : (s + 31) / 32;
  auto load_qg = [&](int t) {
    const int i = min(t * 32 + l32, s - 1);
    load_row<DH>(base + (int64_t)i * ld, dh, hf, qf);
    load_row<DH>(gbase + (int64_t)i * h, dh, hf, gf);
  };
  // the column operands travel under the first two products, and the next tile's rows under the last two, where the
  // registers allow it
  constexpr bool kColsFirst = DH <= 64, kAhead = DH <= 64;
  if (kAhead && t0 + wave < t1) load_qg(t0 + wave);
  for (int t = t0 + wave; t < t1; t += NW) {
    const int i0 = t * 32;
    if (!kAhead) load_qg(t);
    auto load_g_cols = [&] { load_cols<DH>(gbase + (int64_t)i0 * h, h, s - i0, dh, l32, hf, gc); };
    auto load_q_cols = [&] { load_cols<DH>(base + (int64_t)i0 * ld, (int)ld, s - i0, dh, l32, hf, qc); };
    if (kColsFirst) { load_g_cols(); load_q_cols(); }
    float lv[16], dl[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = min(i0 + reg_row(r, hf), s - 1);
      lv[r] = lse_row[i];
      dl[r] = delta_row[i];
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x16 sc = zero16(), dp = zero16();
    k.mul(qf, sc, k_lds, l32, hf);
    v.mul(gf, dp, v_lds, l32, hf);
    __builtin_amdgcn_sched_barrier(0);
    if (!kColsFirst) load_g_cols();
    if (kAhead && t + NW < t1) load_qg(t + NW);
    __builtin_amdgcn_sched_barrier(0);
    const bool diag = causal && i0 < j0 + 31;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = i0 + reg_row(r, hf);
      const bool vis = j < kv_len && i < s && (!causal || j <= i);
      const float p = vis ? __builtin_amdgcn_exp2f(fmaf(sc[r], scale, -lv[r]) * kLog2e) : 0.f;
      dp[r] = vis ? p * (dp[r] - dl[r]) : 0.f;
      sc[r] = p;
    }
    // a key past the sequence's length sees no query at all: its lanes must stay zero whatever the tile holds
    const bool partial = diag || j0 + 32 > kv_len;
    float* p_lds = smem + wave * kRows * C::LD;
    auto sees_len = [&](int row) { return j < kv_len && (!causal || j <= i0 + row); };
    if (partial && any_not_finite<DH>(gc)) accumulate_visible<DH>(gbase + (int64_t)i0 * h, h, min(s - i0, 32), dh, sc, dv, p_lds, l32, hf, sees_len);
    else mul_cols<DH>(gc, sc, dv);
    if (!kColsFirst) { __builtin_amdgcn_sched_barrier(0); load_q_cols(); }
    if (partial && any_not_finite<DH>(qc)) accumulate_visible<DH>(base + (int64_t)i0 * ld, ld, min(s - i0, 32), dh, dp, dk, p_lds, l32, hf, sees_len);
    else mul_cols<DH>(qc, dp, dk);
  }
  float* out = dqkv + ((int64_t)n * s + j0) * ld + h + head * dh;
  put_strip<DH>(dk, scale, smem + wave * kRows * C::LD, l32, hf);
  __syncthreads();
  sum_strips<DH, NW>(smem, out, ld, s - j0, dh, tid, [](int) { return 1.0f; });
  __syncthreads();
  put_strip<DH>(dv, 1.0f, smem + wave * kRows * C::LD, l32, hf);
  __syncthreads();
  sum_strips<DH, NW>(smem, out + h, ld, s - j0, dh, tid, [](int) { return 1.0f; });
}

template <int DH, int NW>
hipError_t fwd_launch(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) {
  constexpr size_t lds = (strip_floats<DH, NW>() + 2 * NW * kRows) * sizeof(float);
  static bool done = false;
  if (!done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_f32_fwd_kernel<DH, NW>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    done = true;
  }
  dim3 grid(d.a, d.b, ceil_div(d.s, kRows));
  hipLaunchKernelGGL((attn_f32_fwd_kernel<DH, NW>), grid, dim3(NW * 64), lds, st, static_cast<const float*>(qkv), static_cast<float*>(o), lse,
                     d.s, d.a, d.dh, d.mask_mode, d.seqlens);
  return hipGetLastError();
}

template <int DH, int NW>
hipError_t bwd_launch(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta,
                      hipStream_t st) {
  constexpr size_t lds_dq = (strip_floats<DH, NW>() + (kDqLds<DH> ? 2 * resident_floats<DH>() : 0)) * sizeof(float);
  constexpr size_t lds_dkv = (strip_floats<DH, NW>() + (kDkvLds<DH> ? 2 * resident_floats<DH>() : 0)) * sizeof(float);
  static_assert(lds_dq <= 160 * 1024 && lds_dkv <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  if (!done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_f32_dq_kernel<DH, NW>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_dq);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_f32_dkv_kernel<DH, NW>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_dkv);
    if (e != hipSuccess) return e;
    done = true;
  }
  dim3 grid(d.a, d.b, ceil_div(d.s, kRows));
  hipLaunchKernelGGL((attn_f32_dq_kernel<DH, NW>), grid, dim3(NW * 64), lds_dq, st, static_cast<const float*>(qkv), static_cast<const float*>(o),
                     static_cast<const float*>(d_o), lse, delta, static_cast<float*>(dqkv), d.s, d.a, d.dh, d.mask_mode, d.seqlens);
  hipLaunchKernelGGL((attn_f32_dkv_kernel<DH, NW>), grid, dim3(NW * 64), lds_dkv, st, static_cast<const float*>(qkv), static_cast<const float*>(d_o),
                     lse, delta, static_cast<float*>(dqkv), d.s, d.a, d.dh, d.mask_mode, d.seqlens);
  return hipGetLastError();
}

}  // namespace

namespace {
// F<DH, NW>::run for the head size, rounded up to a multiple of 16 (fragments) and 32 (result blocks; what lies past it is zero),
// and the waves of a call
template <template <int, int> class F, int NW, typename... Args>
hipError_t by_head(const AttnDesc& d, Args... args) {
  if (d.dh <= 16) return F<16, NW>::run(d, args...);   // (half of the score products of 32: b=60 s=178 a=32 dh=8 backward 560 -> 493 us)
  if (d.dh <= 32) return F<32, NW>::run(d, args...);
  if (d.dh <= 48) return F<48, NW>::run(d, args...);
  if (d.dh <= 64) return F<64, NW>::run(d, args...);
  if (d.dh <= 80) return F<80, NW>::run(d, args...);
  if (d.dh <= 96) return F<96, NW>::run(d, args...);
  if (d.dh <= 112) return F<112, NW>::run(d, args...);
  return F<128, NW>::run(d, args...);
}
template <int DH, int NW>
struct Fwd {
  static hipError_t run(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) { return fwd_launch<DH, NW>(d, qkv, o, lse, st); }
};
template <int DH, int NW>
struct Bwd {
  static hipError_t run(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta, hipStream_t st) {
    return bwd_launch<DH, NW>(d, qkv, o, lse, d_o, dqkv, delta, st);
  }
};
}  // namespace

namespace {
// A CU holds one workgroup of four waves (their registers fill it) or four of one wave (three in the backward pass of heads above 112,
// whose LDS fills it).  With t tiles of 32 rows to stream and an overhead of about 1.2 tiles, `blocks` blocks take ceil(blocks / CUs)
// rounds of ceil(t / 4) + 1.2 tiles, or ceil(blocks / 4 CUs) rounds of t + 1.2, each of those 1.2 times as long as it would be alone;
// 1.35 times more under a causal mask in a launch of one round, which ends on its longest blocks; 1.4 times more in the forward pass of
// heads up to 32, of whose four-wave workgroups a CU holds two.  One wave over four, forward | backward, dh=64: s=64 384 blocks
// 0.83 | 0.81, 640 0.62 | 0.61; s=100 512 1.15 | 1.20, 1024 0.70 | 0.71; s=300 640 0.89 | 0.92 (causal 1.24 | 1.31), 1600 causal
// 0.60 | 0.60; s=512 768 1.07 | 1.07, 1024 0.85 | 0.82; dh=32 s=160 640 causal 1.28 | 1.01; dh=128 s=300 960 0.73 | 1.35.  Over the 336
// launches behind these the choice costs 0.8 % over the better one, and none is more than 5 % behind four waves.  Where one thread
// per row had been ahead of four waves (us, one thread, four, one): b=60 s=40 a=32 dh=32 29 | 73, 30 | 148, 21 | 75; b=46 s=17 a=12
// dh=64 21 | 52, 18 | 57, 7.6 | 23.
bool one_wave(const AttnDesc& d, bool bwd) {
  const int64_t tiles = ceil_div(d.s, kRows), blocks = (int64_t)d.b * d.a * tiles, cus = gemm_compute_units();
  const int64_t at_once = cus * (bwd && d.dh > 112 ? 3 : 4);
  double one = 1.2 * ceil_div(blocks, at_once) * (tiles + 1.2);
  if (d.mask_mode == 1 && blocks <= at_once && tiles > 2) one *= 1.35;
  if (!bwd && d.dh <= 32) one *= 1.4;
  return one < ceil_div(blocks, cus) * (ceil_div(tiles, kManyWaves) + 1.2);
}
}  // namespace

hipError_t attention_fwd_f32(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) {
  return one_wave(d, false) ? by_head<Fwd, 1>(d, qkv, o, lse, st) : by_head<Fwd, kManyWaves>(d, qkv, o, lse, st);
}

hipError_t attention_bwd_f32(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta,
                             hipStream_t st) {
  return one_wave(d, true) ? by_head<Bwd, 1>(d, qkv, o, lse, d_o, dqkv, delta, st) : by_head<Bwd, kManyWaves>(d, qkv, o, lse, d_o, dqkv, delta, st);
}

}  // namespace k2bw
