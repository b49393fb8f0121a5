// fp32 masked-softmax attention on the gfx950 matrix cores (v_mfma_f32_32x32x2_f32), forward and backward, any head
// size that is a multiple of 8 up to 128.  Operands, scores, probabilities and accumulators are fp32 throughout.
//
// What bounds it: the fp32 matrix rate (64 cycles per 32x32x2 instruction and SIMD) once there is work for every
// SIMD, and latency below that.  Microbatches of the fp32 mode are small (16 heads x 512 queries are 256 blocks of 32
// queries), so a workgroup owns only ONE block of 32 rows (queries in the forward and dQ kernels, keys in dK/dV) and
// its four waves take every fourth tile of 32 rows of the streamed side; their partial results meet in LDS once, at
// the end, in a fixed order.  Inside the loop nothing is shared and there is no barrier: a wave fetches its tiles into LDS of
// its own (WaveTile), the next one under the last product of the current one.
// Measured at b=2 s=512 a=8 dh=64, causal: forward 17 us, backward 38 (41 in the plain order of blocks, see attn_f32_bwd_folded_kernel;
// 55 while every fragment came from L2 by itself and dQ and dK/dV were launches of their own; 520 and 1146 with one thread per row on
// the vector ALU); the matrix instructions alone are 7 and 14 us of the longest workgroups.
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
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void glob_void_t;

// Waves per workgroup (NW): four, which split the streamed rows, or one where a launch has blocks enough without that (fwd_one_wave, bwd_form)
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

// The 32 rows of a streamed operand that a wave works on, in LDS of its own: fetched once, 16 bytes per lane along the rows and no
// registers, and read both as rows (16 bytes per lane) and as columns (4 bytes).  Straight from L2 into fragment registers every
// operand came twice, the second time by 16 loads of two rows each per 32 columns, and a load occupies the CU's address unit for some
// 16 cycles whatever it brings: 112 of them per tile and wave in dK/dV were as much time as the matrix instructions.
// Layout: rows of LW floats (what lies past the head is zero) in blocks of kRowsPer rows, as one load instruction writes them (three for
// rows of 96), 16-byte chunks XOR-swizzled by row inside a block and kPad floats between blocks: 16 consecutive rows at one chunk then
// fall on all banks, and the addresses of a lane differ by constants but for two or four.
__device__ const float4 kZeros = {0.f, 0.f, 0.f, 0.f};
template <int DH>
struct WaveTile {
  static constexpr int LW = DH <= 16 ? 16 : DH <= 32 ? 32 : DH <= 64 ? 64 : DH <= 96 ? 96 : 128;
  static constexpr int CH = LW / 4, kLoads = LW == 96 ? 3 : 1, kRowsPer = 64 * kLoads / CH;
  static constexpr int kPad = LW == 16 ? 0 : LW == 128 ? 8 : 16;
  static constexpr int kBlock = kLoads * 256 + kPad, kFloats = 32 / kRowsPer * kBlock;
  // swizzle of a row: two bits, one for rows of 512 bytes; the same in every block
  static __device__ __forceinline__ int swz(int row) { return LW == 128 ? row & 1 : LW == 64 ? row & 3 : LW == 16 ? (row >> 2) & 3 : (row >> 1) & 3; }
  static __device__ __forceinline__ int at(int row) { return row / kRowsPer * kBlock + row % kRowsPer * LW; }
  // rows [0, rows) x [0, dh) of the matrix at src (uniform) into t; the rest is zero
  static __device__ __forceinline__ void issue(const float* __restrict__ src, int64_t ld, int rows, int dh, int lane, float* t) {
    asm volatile("" : "+s"(src));   // else the loop keeps a pointer per lane and load instruction
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int L = u * 64 + lane, row = L / CH, c = (L % CH) ^ swz(row);
      const float* from = src + row * ld + 4 * c;
      const bool in_head = 4 * c < dh;
#pragma unroll
      for (int q = 0; q < 32 / kRowsPer; ++q) {
        const float* p = in_head && row < rows - q * kRowsPer ? from + q * kRowsPer * ld : reinterpret_cast<const float*>(&kZeros);
        __builtin_amdgcn_global_load_lds((glob_void_t*)p, (lds_void_t*)(t + q * kBlock + u * 256), 16, 0, 0);
      }
    }
  }
  // head columns 8j + 4*hf .. +3 of row l32
  static __device__ __forceinline__ float4 row4(const float* t, int j, int l32, int hf) {
    return *reinterpret_cast<const float4*>(t + at(l32) + (((2 * (j & 1) + hf) ^ swz(l32)) << 2) + 16 * (j >> 1));
  }
  // f[db][r] = row reg_row(r, hf), column 32*db + l32 of NB blocks of columns (columns past DH: zero, or another's if rows have 16; they only reach result
  // columns that are never stored)
  template <int NB>
  static __device__ __forceinline__ void cols(const float* t, int l32, int hf, float (&f)[NB][16]) {
    const int col = LW == 16 ? l32 & 15 : l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = reg_row(r, hf);
      const float* x = t + at(row) + ((((col >> 2) ^ swz(row)) << 2) | (col & 3));
#pragma unroll
      for (int db = 0; db < NB; ++db) f[db][r] = x[32 * db];
    }
  }
  // acc += (this tile's rows) * f^T over the head dimension
  static __device__ __forceinline__ void mul(const float* t, const float (&f)[CfgF<DH>::NF], f32x16& acc, int l32, int hf) {
#pragma unroll
    for (int j = 0; j < DH / 8; ++j) {
      const float4 v = row4(t, j, l32, hf);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v.x, f[4 * j], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v.y, f[4 * j + 1], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v.z, f[4 * j + 2], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v.w, f[4 * j + 3], acc, 0, 0, 0);
    }
  }
};
// a wave's loads into its tiles have landed / its reads of them are done
__device__ __forceinline__ void tiles_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void tiles_read() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// LDS, in floats: every wave's two tiles (the strips of the results re-use them), then what the kernel adds
template <int DH, int NW> constexpr int strip_floats() { return NW * kRows * CfgF<DH>::LD; }
template <int DH, int NW> constexpr int tile_floats() {
  const int t = NW * 2 * WaveTile<DH>::kFloats, s = strip_floats<DH, NW>();
  return t > s ? t : s;
}
// Waves per SIMD that the registers leave room for: two up to head size 64 (one of 512 registers instead: backward at b=8 s=512 a=16
// dh=64 332 -> 364 us, forward 96 -> 110)
template <int DH> constexpr int kPerSimd = DH <= 64 ? 2 : 1;
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// out[db] += X^T P over the 32 rows of a tile
template <int NB>
__device__ __forceinline__ void mul_cols(const float (&x)[NB][16], const f32x16& p, f32x16 (&out)[NB]) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int db = 0; db < NB; ++db) out[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[db][r], p[r], out[db], 0, 0, 0);
}

template <int NB>
__device__ __forceinline__ bool any_not_finite(const float (&x)[NB][16]) {
  bool bad = false;
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) bad = bad || !(fabsf(x[db][r]) < INFINITY);
  return __any(bad);
}

// mul_cols for a tile in which not every lane's row (query or key) sees every row of the tile, when the tile holds
// infinities or NaNs: row by row, added only where it is seen (sees(row)).  Rare, so it keeps few registers: the rows
// come from `tile`, the matrix, again.
template <int NB, typename Sees>
__device__ __forceinline__ void accumulate_visible(const float* __restrict__ tile, int64_t ld, int rows, int dh, const f32x16& p,
                                                   f32x16 (&out)[NB], int hf, Sees&& sees) {
#pragma unroll 1
  for (int row = 0; row < rows; ++row) {
    const int reg = (row >> 3) * 4 + (row & 3);
    float w = p[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) w = e == reg ? p[e] : w;
    const float other = __shfl_xor(w, 32, 64);
    w = ((row >> 2) & 1) == hf ? w : other;
    const bool vis = sees(row);
    const float* x = tile + row * ld + 4 * hf;
#pragma unroll
    for (int db = 0; db < NB; ++db)
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
template <int DH, int NB>
__device__ __forceinline__ void put_strip(const f32x16 (&acc)[NB], float f, float* strip, int l32, int hf) {
#pragma unroll
  for (int db = 0; db < NB; ++db)
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
__global__ __launch_bounds__(NW * 64, (kPerSimd<DH>)) void attn_f32_fwd_kernel(const float* __restrict__ qkv, float* __restrict__ o, float* __restrict__ lse,
                                                                    int s, int a, int dh, int mask_mode, const int32_t* __restrict__ seqlens) {
  using C = CfgF<DH>;
  extern __shared__ __attribute__((aligned(16))) float smem[];   // tiles (then strips), m[NW][32], l[NW][32]
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

  float qf[C::NF], vc[C::DB][16];
  load_row<DH>(base + (int64_t)min(i, s - 1) * ld, dh, hf, qf);
  f32x16 oacc[C::DB];
#pragma unroll
  for (int db = 0; db < C::DB; ++db) oacc[db] = zero16();
  float m_i = -INFINITY, l_i = 0.f;
  const int jend = causal ? min(i0 + kRows, s) : kv_len;
  const int ntiles = (jend + 31) / 32;
  float* k_tile = smem + wave * 2 * WaveTile<DH>::kFloats;
  float* v_tile = k_tile + WaveTile<DH>::kFloats;
  auto issue = [&](int t) {
    const float* row = base + h + (int64_t)t * 32 * ld;
    WaveTile<DH>::issue(row, ld, jend - t * 32, dh, lane, k_tile);
    WaveTile<DH>::issue(row + h, ld, jend - t * 32, dh, lane, v_tile);
  };
  if (wave < ntiles) issue(wave);
  for (int t = wave; t < ntiles; t += NW) {
    const int j0 = t * 32;
    tiles_landed();
    f32x16 sc = zero16();
    WaveTile<DH>::mul(k_tile, qf, sc, l32, hf);
    WaveTile<DH>::cols(v_tile, l32, hf, vc);
    tiles_read();
    if (t + NW < ntiles) issue(t + NW);   // the next tile travels under the softmax and the second product
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
    if (diag && any_not_finite(vc)) accumulate_visible(base + 2 * h + (int64_t)j0 * ld, ld, min(jend - j0, 32), dh, sc, oacc, hf, [&](int row) { return j0 + row <= i; });
    else mul_cols(vc, sc, oacc);
  }
  // the waves' maxima meet, every partial result is rescaled to the common one
  float* m_lds = smem + tile_floats<DH, NW>();
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
__device__ __forceinline__ void attn_f32_dq(const float* __restrict__ qkv, const float* __restrict__ o, const float* __restrict__ d_o,
                                            const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dqkv, int s, int a,
                                            int dh, int mask_mode, const int32_t* __restrict__ seqlens, int blk, float* smem) {
  using C = CfgF<DH>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int n = blockIdx.y, head = blockIdx.x;
  const bool causal = mask_mode == 1;
  const int i0 = blk * kRows, i = i0 + l32, ic = min(i, s - 1);
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const float* base = qkv + (int64_t)n * s * ld + head * dh;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;
  const float scale = 1.0f / sqrtf((float)dh), c = scale * kLog2e;

  float qf[C::NF], gf[C::NF], kc[C::DB][16];
  const float* g_row = d_o + ((int64_t)n * s + ic) * h + head * dh;
  const int jend = causal ? min(i0 + kRows, s) : kv_len;
  const int ntiles = (jend + 31) / 32;
  float* k_tile = smem + wave * 2 * WaveTile<DH>::kFloats;
  float* v_tile = k_tile + WaveTile<DH>::kFloats;
  auto issue = [&](int t) {
    const float* row = base + h + (int64_t)t * 32 * ld;
    WaveTile<DH>::issue(row, ld, jend - t * 32, dh, lane, k_tile);
    WaveTile<DH>::issue(row + h, ld, jend - t * 32, dh, lane, v_tile);
  };
  if (wave < ntiles) issue(wave);
  load_row<DH>(base + (int64_t)ic * ld, dh, hf, qf);
  load_row<DH>(g_row, dh, hf, gf);
  float delta_i;
  {
    float of[C::NF];
    load_row<DH>(o + ((int64_t)n * s + ic) * h + head * dh, dh, hf, of);
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
  for (int t = wave; t < ntiles; t += NW) {
    const int j0 = t * 32;
    tiles_landed();
    f32x16 sc = zero16(), dp = zero16();
    WaveTile<DH>::mul(k_tile, qf, sc, l32, hf);
    WaveTile<DH>::mul(v_tile, gf, dp, l32, hf);
    WaveTile<DH>::cols(k_tile, l32, hf, kc);
    tiles_read();
    if (t + NW < ntiles) issue(t + NW);
    __builtin_amdgcn_sched_barrier(0);
    const bool diag = causal && j0 + 31 > i0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = j0 + reg_row(r, hf);
      const bool vis = key < jend && (!causal || key <= i);
      const float p = __builtin_amdgcn_exp2f(fmaf(sc[r], scale, -lse_i) * kLog2e);
      sc[r] = vis ? p * (dp[r] - delta_i) : 0.f;   // dS^T (the scale is applied at the end)
    }
    if (diag && any_not_finite(kc)) accumulate_visible(base + h + (int64_t)j0 * ld, ld, min(jend - j0, 32), dh, sc, dq, hf, [&](int row) { return j0 + row <= i; });
    else mul_cols(kc, sc, dq);
  }
  __syncthreads();   // every wave is done with its tiles
  put_strip<DH>(dq, scale, smem + wave * kRows * C::LD, l32, hf);
  __syncthreads();
  sum_strips<DH, NW>(smem, dqkv + ((int64_t)n * s + i0) * ld + head * dh, ld, s - i0, dh, tid, [](int) { return 1.0f; });
}

// ------------------------------------------------------------------------------------------------
// dK, dV: lane = key, registers = queries (S = Q K^T, dV^T = dO^T P, dK^T = Q^T dS)
// FUSED: delta from dO and O, as the launch that forms it for others is the same one; else it is read.
// EXACT: the second run of a workgroup that met infinities or NaNs in a tile which not all its keys see in whole (returns true for it),
// for the results' 32 columns from 32 * db0 on.  All columns at once in that run, whose row-by-row path keeps more alive, spill 92 to 302
// registers at head sizes 48, 64, 112 and 128, some of them inside the loop of the first run (backward without that 0.97 to 0.98 of the
// time at those heads and 80 and 96, over 2700 random sizes).
// In that run, too, only tiles that hold such values are added row by row (a NaN in dO of one query, b=2 s=512 a=8 dh=128 with lengths:
// 854 -> 321 us; without the NaN 93).
template <int DH, int NW, bool FUSED, bool EXACT>
__device__ __forceinline__ bool attn_f32_dkv(const float* __restrict__ qkv, const float* __restrict__ o, const float* __restrict__ d_o,
                                             const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dqkv, int s, int a, int dh, int mask_mode,
                                             const int32_t* __restrict__ seqlens, int blk, float* smem, int db0 = 0) {
  using C = CfgF<DH>;
  constexpr int NB = EXACT ? 1 : C::DB;   // blocks of 32 result columns
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int n = blockIdx.y, head = blockIdx.x;   // causal: the first keys are seen by the most queries
  const bool causal = mask_mode == 1;
  const int j0 = blk * kRows, j = j0 + l32, jc = min(j, s - 1);
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const float* base = qkv + (int64_t)n * s * ld + head * dh;
  const float* gbase = d_o + (int64_t)n * s * h + head * dh;
  const float* obase = o + (int64_t)n * s * h + head * dh;
  const float* lse_row = lse + ((int64_t)n * a + head) * s;
  const float* delta_row = delta + ((int64_t)n * a + head) * s;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;
  const float scale = 1.0f / sqrtf((float)dh);

  // query tiles that can see a key of the block: none if the block is padding, from the block itself on if causal
  const int t0 = causal ? blk : 0;
  const int t1 = j0 >= kv_len ? t0 : (s + 31) / 32;
  float* q_tile = smem + wave * 2 * WaveTile<DH>::kFloats;
  float* g_tile = q_tile + WaveTile<DH>::kFloats;
  auto issue = [&](int t) {
    int l = lane;
    if (DH > 32 && DH <= 64) asm volatile("" : "+v"(l));   // 256 registers have no room for what of the addresses stays the same
    WaveTile<DH>::issue(base + (int64_t)t * 32 * ld, ld, s - t * 32, dh, l, q_tile);
    WaveTile<DH>::issue(gbase + (int64_t)t * 32 * h, h, s - t * 32, dh, l, g_tile);
  };
  if (t0 + wave < t1) issue(t0 + wave);
  float kf[C::NF], vf[C::NF], xc[NB][16];
  constexpr bool kAgain = EXACT && C::DB > 1;   // K and V fetched for every tile rather than in registers throughout
  auto load_kv = [&] {
    const float* row = base + h + (int64_t)jc * ld;
    if (kAgain) asm volatile("" : "+v"(row));
    load_row<DH>(row, dh, hf, kf);
    load_row<DH>(row + h, dh, hf, vf);
  };
  if (!kAgain) load_kv();
  // lse and delta of the tile's queries: a lane has those of its row, the products need them by register
  float* stat = smem + tile_floats<DH, NW>() + wave * 64;
  f32x16 dk[NB], dv[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db) { dk[db] = zero16(); dv[db] = zero16(); }
  float lse_i = 0.f, delta_i = 0.f, of[FUSED ? C::NF : 1];
  bool hidden = false;
  // (O's row a tile ahead only where the registers allow it)
  constexpr bool kOAhead = DH <= 32;
  auto load_o = [&](int t) {
    if constexpr (FUSED) load_row<DH>(obase + (int64_t)min(t * 32 + l32, s - 1) * h, dh, hf, of);
  };
  auto load_stat = [&](int t) {
    const int i = min(t * 32 + l32, s - 1);
    lse_i = lse_row[i];
    if (kOAhead) load_o(t);
    if (!FUSED) delta_i = delta_row[i];
  };
  if (t0 + wave < t1) load_stat(t0 + wave);
  for (int t = t0 + wave; t < t1; t += NW) {
    const int i0 = t * 32;
    if (!kOAhead) load_o(t);
    tiles_landed();
    if constexpr (FUSED) {
      float part = 0.f;
#pragma unroll
      for (int j2 = 0; j2 < DH / 8; ++j2) {
        const float4 x = WaveTile<DH>::row4(g_tile, j2, l32, hf);
        part = fmaf(x.x, of[4 * j2], part); part = fmaf(x.y, of[4 * j2 + 1], part);
        part = fmaf(x.z, of[4 * j2 + 2], part); part = fmaf(x.w, of[4 * j2 + 3], part);
      }
      delta_i = part + __shfl_xor(part, 32, 64);
    }
    stat[lane] = hf == 0 ? lse_i : delta_i;
    wave_fence();
    f32x16 sc = zero16(), dp = zero16();
    if (kAgain) load_kv();
    WaveTile<DH>::mul(q_tile, kf, sc, l32, hf);
    __builtin_amdgcn_sched_barrier(0);   // (the fragments of both products together do not fit)
    WaveTile<DH>::mul(g_tile, vf, dp, l32, hf);
    __builtin_amdgcn_sched_barrier(0);
    const bool diag = causal && i0 < j0 + 31;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 l4 = *reinterpret_cast<const float4*>(stat + 8 * g + 4 * hf), d4 = *reinterpret_cast<const float4*>(stat + 32 + 8 * g + 4 * hf);
      const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dl[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * g + e, i = i0 + reg_row(r, hf);
        const bool vis = j < kv_len && i < s && (!causal || j <= i);
        const float p = vis ? __builtin_amdgcn_exp2f(fmaf(sc[r], scale, -lv[e]) * kLog2e) : 0.f;
        dp[r] = vis ? p * (dp[r] - dl[e]) : 0.f;
        sc[r] = p;
      }
    }
    // a key past the sequence's length sees no query at all: its lanes must stay zero whatever the tile holds
    const bool partial = diag || j0 + 32 > kv_len;
    auto sees_len = [&](int row) { return j < kv_len && (!causal || j <= i0 + row); };
    __builtin_amdgcn_sched_barrier(0);
    WaveTile<DH>::cols(g_tile + 32 * db0, l32, hf, xc);
    if (EXACT && partial && any_not_finite(xc)) {
      accumulate_visible(gbase + (int64_t)i0 * h + 32 * db0, h, min(s - i0, 32), dh - 32 * db0, sc, dv, hf, sees_len);
    } else {
      if (!EXACT && partial) hidden = hidden || any_not_finite(xc);
      mul_cols(xc, sc, dv);
    }
    __builtin_amdgcn_sched_barrier(0);
    WaveTile<DH>::cols(q_tile + 32 * db0, l32, hf, xc);
    tiles_read();
    if (t + NW < t1) { issue(t + NW); load_stat(t + NW); }   // the next tile travels under the last product
    __builtin_amdgcn_sched_barrier(0);
    if (EXACT && partial && any_not_finite(xc)) {
      accumulate_visible(base + (int64_t)i0 * ld + 32 * db0, ld, min(s - i0, 32), dh - 32 * db0, dp, dk, hf, sees_len);
    } else {
      if (!EXACT && partial) hidden = hidden || any_not_finite(xc);
      mul_cols(xc, dp, dk);
    }
  }
  if (EXACT) __syncthreads();   // every wave is done with its tiles
  else if (__syncthreads_or(hidden)) return true;
  float* out = dqkv + ((int64_t)n * s + j0) * ld + h + head * dh + 32 * db0;
  const int cols = EXACT ? min(dh - 32 * db0, 32) : dh;
  put_strip<DH>(dk, scale, smem + wave * kRows * C::LD, l32, hf);
  __syncthreads();
  sum_strips<DH, NW>(smem, out, ld, s - j0, cols, tid, [](int) { return 1.0f; });
  __syncthreads();
  put_strip<DH>(dv, 1.0f, smem + wave * kRows * C::LD, l32, hf);
  __syncthreads();
  sum_strips<DH, NW>(smem, out + h, ld, s - j0, cols, tid, [](int) { return 1.0f; });
  return false;
}
template <int DH, int NW, bool FUSED>
__device__ __forceinline__ void attn_f32_dkv_all(const float* __restrict__ qkv, const float* __restrict__ o, const float* __restrict__ d_o,
                                                 const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dqkv, int s, int a, int dh, int mask_mode,
                                                 const int32_t* __restrict__ seqlens, int blk, float* smem) {
  if (!attn_f32_dkv<DH, NW, FUSED, false>(qkv, o, d_o, lse, delta, dqkv, s, a, dh, mask_mode, seqlens, blk, smem)) return;
#pragma unroll 1
  for (int db0 = 0; db0 < CfgF<DH>::DB; ++db0) {
    attn_f32_dkv<DH, NW, FUSED, true>(qkv, o, d_o, lse, delta, dqkv, s, a, dh, mask_mode, seqlens, blk, smem, db0);
    __syncthreads();   // the strips are read, the next tiles may come
  }
}

template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, (kPerSimd<DH>)) void attn_f32_dq_kernel(const float* __restrict__ qkv, const float* __restrict__ o,
                                                                    const float* __restrict__ d_o, const float* __restrict__ lse,
                                                                    float* __restrict__ delta, float* __restrict__ dqkv, int s, int a, int dh,
                                                                    int mask_mode, const int32_t* __restrict__ seqlens) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  attn_f32_dq<DH, NW>(qkv, o, d_o, lse, delta, dqkv, s, a, dh, mask_mode, seqlens, mask_mode == 1 ? (int)(gridDim.z - 1 - blockIdx.z) : (int)blockIdx.z, smem);
}
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, (kPerSimd<DH>)) void attn_f32_dkv_kernel(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                                     const float* __restrict__ lse, const float* __restrict__ delta,
                                                                     float* __restrict__ dqkv, int s, int a, int dh, int mask_mode,
                                                                     const int32_t* __restrict__ seqlens) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  attn_f32_dkv_all<DH, NW, false>(qkv, nullptr, d_o, lse, delta, dqkv, s, a, dh, mask_mode, seqlens, blockIdx.z, smem);
}
// Both in one launch: block 2k of grid.z has the keys of block k, block 2k + 1 the queries of block k (causal: k from the end), so the
// longest workgroups of either kind go first.
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, (kPerSimd<DH>)) void attn_f32_bwd_kernel(const float* __restrict__ qkv, const float* __restrict__ o,
                                                                     const float* __restrict__ d_o, const float* __restrict__ lse,
                                                                     float* __restrict__ delta, float* __restrict__ dqkv, int s, int a, int dh,
                                                                     int mask_mode, const int32_t* __restrict__ seqlens) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int k = blockIdx.z >> 1;
  if (blockIdx.z & 1) attn_f32_dq<DH, NW>(qkv, o, d_o, lse, delta, dqkv, s, a, dh, mask_mode, seqlens, mask_mode == 1 ? (int)(gridDim.z >> 1) - 1 - k : k, smem);
  else attn_f32_dkv_all<DH, NW, true>(qkv, o, d_o, lse, delta, dqkv, s, a, dh, mask_mode, seqlens, k, smem);
}

// The same where all workgroups of a causal launch start at once, two on a CU (Fold).  A kernel of its own: two more arguments and a select
// in front of everything cost the others 0.1 us.  b=2 s=512 a=8 dh=64 41.5 -> 37.9 us, b=1 s=451 a=16 dh=48 33.6 -> 30.7.
template <int DH>
__global__ __launch_bounds__(kManyWaves * 64, (kPerSimd<DH>)) void attn_f32_bwd_folded_kernel(const float* __restrict__ qkv, const float* __restrict__ o,
                                                                     const float* __restrict__ d_o, const float* __restrict__ lse,
                                                                     float* __restrict__ delta, float* __restrict__ dqkv, int s, int a, int dh,
                                                                     int nblk, Fold fold) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int z = folded_z(fold), k = z >> 1;
  if (z & 1) attn_f32_dq<DH, kManyWaves>(qkv, o, d_o, lse, delta, dqkv, s, a, dh, 1, nullptr, nblk - 1 - k, smem);
  else attn_f32_dkv_all<DH, kManyWaves, true>(qkv, o, d_o, lse, delta, dqkv, s, a, dh, 1, nullptr, k, smem);
}

// The fold where it pays.  Where it would turn only the last two positions, the dK/dV and the dQ workgroups of the shortest block change
// places.  That gains or is level, except where blocks take more than one step of the four waves and heads x sequences divides the CUs, so that the
// two stand exactly beside the longest dK/dV and the longest dQ: the longer of the long ones gets the longer of the short ones.  Folded over
// plain, means and worst of 30 random calls each by heads x sequences: 4 1.006, 1.024; 8 1.022, 1.053; 16 1.032, 1.063; 32 1.044, 1.082
// (b=4 s=138 a=8 dh=64 19.7 -> 21.0 us); one step, 64 0.952, 0.993; no divisor 0.989, 1.024.  (300 random folded calls with this rule:
// 0.987, three positions and more 0.978, at worst 1.013.)
bool folds(const AttnDesc& d, const Fold& fold, int blocks) {
  const int turned = 2 * blocks - fold.at;
  return turned > 2 || (turned == 2 && (blocks <= kManyWaves || gemm_compute_units() % (d.a * d.b) != 0));
}

template <typename K>
hipError_t set_lds(K kern, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Long causal sequences whose blocks are more than the CUs and no more than twice: all start at once where a CU holds two workgroups of
// four waves, and the CUs that got one idle when it ends.  With one at a time the longest blocks go first and the others follow where a CU
// comes free (two over one: from 13 tiles on 1.02 to 1.23, b=2 s=700 a=8 dh=56 25.6 -> 20.9 us; 9 to 12 tiles up to 320 blocks 1.0 to
// 1.16, beyond 0.84 to 1.0; fewer 0.7 to 0.96; above 512 blocks 0.8 to 0.91).  Head sizes up to 32 are even up to 256 blocks and behind above.
template <int DH, int NW>
bool one_at_a_time(const AttnDesc& d) {
  const int64_t tiles = ceil_div(d.s, kRows), blocks = (int64_t)d.b * d.a * tiles, cus = gemm_compute_units();
  return NW > 1 && DH > 32 && DH <= 64 && d.mask_mode == 1 && blocks > cus && blocks <= 2 * cus && (tiles >= 13 || (tiles >= 9 && 4 * blocks <= 5 * cus));
}

template <int DH, int NW>
hipError_t fwd_launch(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) {
  constexpr size_t need = (tile_floats<DH, NW>() + 2 * NW * kRows) * sizeof(float), most = need > 81 * 1024 ? need : 81 * 1024;
  static_assert(need <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  if (!done) {
    hipError_t e = set_lds(attn_f32_fwd_kernel<DH, NW>, most);
    if (e != hipSuccess) return e;
    done = true;
  }
  const size_t lds = one_at_a_time<DH, NW>(d) ? most : need;
  dim3 grid(d.a, d.b, ceil_div(d.s, kRows));
  hipLaunchKernelGGL((attn_f32_fwd_kernel<DH, NW>), grid, dim3(NW * 64), lds, st, static_cast<const float*>(qkv), static_cast<float*>(o), lse,
                     d.s, d.a, d.dh, d.mask_mode, d.seqlens);
  return hipGetLastError();
}

template <int DH, int NW>
hipError_t bwd_launch(const AttnDesc& d, bool one_launch, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta,
                      hipStream_t st) {
  constexpr size_t lds_dq = tile_floats<DH, NW>() * sizeof(float);
  constexpr size_t lds = lds_dq + NW * 64 * sizeof(float);
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  constexpr bool kFolds = NW == kManyWaves && kPerSimd<DH> == 2;
  static bool done = false;
  if (!done) {
    hipError_t e = set_lds(attn_f32_bwd_kernel<DH, NW>, lds);
    if (e == hipSuccess) e = set_lds(attn_f32_dq_kernel<DH, NW>, lds_dq);
    if (e == hipSuccess) e = set_lds(attn_f32_dkv_kernel<DH, NW>, lds);
    if constexpr (kFolds) if (e == hipSuccess) e = set_lds(attn_f32_bwd_folded_kernel<DH>, lds);
    if (e != hipSuccess) return e;
    done = true;
  }
  const int blocks = ceil_div(d.s, kRows);
  const float *q = static_cast<const float*>(qkv), *out = static_cast<const float*>(o), *g = static_cast<const float*>(d_o);
  float* dst = static_cast<float*>(dqkv);
  const Fold fold = fold_of(d, 2 * blocks, kFolds ? 2 : 1);
  if (one_launch && kFolds && folds(d, fold, blocks)) {
    if constexpr (kFolds)
      hipLaunchKernelGGL((attn_f32_bwd_folded_kernel<DH>), dim3(d.a, d.b, 2 * blocks), dim3(NW * 64), lds, st, q, out, g, lse, delta, dst, d.s, d.a, d.dh, blocks,
                         fold);
  } else if (one_launch) {
    hipLaunchKernelGGL((attn_f32_bwd_kernel<DH, NW>), dim3(d.a, d.b, 2 * blocks), dim3(NW * 64), lds, st, q, out, g, lse, delta, dst, d.s, d.a, d.dh,
                       d.mask_mode, d.seqlens);
  } else {
    hipLaunchKernelGGL((attn_f32_dq_kernel<DH, NW>), dim3(d.a, d.b, blocks), dim3(NW * 64), lds_dq, st, q, out, g, lse, delta, dst, d.s, d.a, d.dh,
                       d.mask_mode, d.seqlens);
    hipLaunchKernelGGL((attn_f32_dkv_kernel<DH, NW>), dim3(d.a, d.b, blocks), dim3(NW * 64), lds, st, q, g, lse, delta, dst, d.s, d.a, d.dh,
                       d.mask_mode, d.seqlens);
  }
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
  static hipError_t run(const AttnDesc& d, bool one_launch, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta, hipStream_t st) {
    return bwd_launch<DH, NW>(d, one_launch, qkv, o, lse, d_o, dqkv, delta, st);
  }
};
}  // namespace

namespace {
// One wave per workgroup, or four that split the t tiles of 32 rows to stream?  Forward, an empirical rule: four waves cost a round of
// ceil(t / 4) + 1.2 tiles per block on each CU, one wave a round of t + 1.2 per four blocks, times 1.2; 1.35 times more under a causal
// mask in a launch of up to four blocks per CU, which ends on its longest blocks; 1.4 times more for heads up to 32.  (It counts one or
// four workgroups on a CU at every head size; up to 64 a CU holds two or eight.)  Over 2700 random sizes the choice costs 0.7 % (heads up
// to 32) and 0.3 % (above) over the better one.  Over the time before the tiles went through LDS: heads up to 32 0.90, 64 0.92, 96 0.98,
// 128 0.96, at worst 1.07 to 1.09 (b=3 s=685 a=12 dh=80 92 -> 97 us: one wave, four workgroups on every CU).
bool fwd_one_wave(const AttnDesc& d) {
  const int64_t tiles = ceil_div(d.s, kRows), blocks = (int64_t)d.b * d.a * tiles, cus = gemm_compute_units();
  double one = 1.2 * ceil_div(blocks, 4 * cus) * (tiles + 1.2);
  if (d.mask_mode == 1 && tiles > 2 && blocks <= 4 * cus) one *= 1.35;
  if (d.dh <= 32) one *= 1.4;
  return one < ceil_div(blocks, cus) * (ceil_div(tiles, kManyWaves) + 1.2);
}

// Backward: one wave or four, and dQ and dK/dV in one launch or in two.  One launch has twice the workgroups, of both lengths, and spares
// a launch and its tail; in two dK/dV reads the delta that dQ has left and needs no row of O.
// Heads up to 64: a CU holds two workgroups of four waves or eight of one.  One launch over two, four waves: up to 128 blocks 0.6, to
// 256 0.7 to 1.0, to 1024 0.9, above 1.0; one wave: up to 512 blocks 0.65, to 2048 0.65 to 0.8 under a causal mask, 0.9 with lengths,
// 1.0 without, beyond 0.9 with a mask.  The constants of one wave against four are fitted to 500 random sizes with each form forced.
// Longer heads: one of four or four of one, so where the workgroups of one launch are not all there at once, what counts is whole rounds.
// One launch over two, no mask, by blocks over what the CUs hold: up to 0.5 0.65, to 1 1.0 to 1.2 (sequences of up to 3 tiles 0.8 to
// 1.0), to 1.5 0.72 to 0.93, to 2 0.92 to 1.16, to 2.5 0.82 to 0.95, to 3 0.97 to 1.1; under a causal mask 0.65 as long as the longest
// blocks fit side by side.  The constants below, which weigh the four forms in units of a tile, are fitted to 5568 random sizes with each
// form forced.
// Over the least time of the forms: up to 64 1.008, above 1.006.  (The folded order, later than the fit, makes four waves faster where it applies;
// 500 random causal calls of up to 700 blocks with heads up to 64, one wave and four forced: 1.004, 15 calls more than 1.03, all of them of 480 to
// 672 blocks of short sequences, where nothing is folded, the worst b=7 s=96 a=24 dh=48 23.7 | 28.8.)  Over the time before the tiles went through LDS and the two halves into
// one launch: up to 64 0.61, above 0.68, of 5568 calls 13 more than 1.03, the worst b=7 s=88 a=12 dh=80 causal, 28.6 -> 32.0 us.  (With
// the rule of the shorter heads above 64, too: 1.05 over the least, 235 calls more than 1.03 over that time, at worst 1.26.)
struct BwdForm { int waves; bool one_launch; };
BwdForm bwd_form(const AttnDesc& d) {
  const int64_t tiles = ceil_div(d.s, kRows), blocks = (int64_t)d.b * d.a * tiles, cus = gemm_compute_units();
  const bool causal = d.mask_mode == 1;
  if (d.dh <= 64) {
    const bool few = blocks <= 4 * cus, l1 = few || d.mask_mode != 0;
    const int64_t wgs1 = l1 ? 2 * blocks : blocks, wgs4 = few ? 2 * blocks : blocks;
    double one = 0.93 * (l1 ? 1 : 2) * ceil_div(wgs1, 8 * cus) * (tiles + 0.34);
    if (causal && tiles > 2 && wgs1 <= 8 * cus) one *= 1.56;
    const double four = (few ? 1 : 2) * ceil_div(wgs4, 2 * cus) * (ceil_div(tiles, kManyWaves) + 0.34);
    return one < four ? BwdForm{1, l1} : BwdForm{kManyWaves, few};
  }
  BwdForm best = {0, false};
  double least = 0;
  for (int waves : {1, kManyWaves})
    for (bool one : {false, true}) {
      const int64_t wgs = one ? 2 * blocks : blocks, slots = (waves == 1 ? 4 : 1) * cus;
      const int64_t steps = ceil_div(tiles, waves), whole = tiles / waves;
      const double x = (double)wgs / slots, over = waves == 1 ? 0.14 : 0.46;   // what a workgroup costs beside its steps
      double rounds;
      if (causal) {   // blocks of all lengths, the longest first
        const double mean = (waves * whole * (whole + 1) / 2 + (tiles - waves * whole) * steps) / (double)tiles;
        rounds = x * (mean + over) / (steps + over) + (x > 0.5 ? 0.3 : 0.0);
      } else {   // in one launch the last round starts as the shorter half of the one before ends
        const double part = !one ? 0.0 : tiles <= 3 ? 1.0 : d.mask_mode == 2 ? 0.4 : 0.3;
        rounds = (1 - part) * ceil_div(wgs, slots) + part * x;
      }
      if (rounds < 1) rounds = 1;
      const double length = (waves == 1 ? 0.91 : 1.0) * (steps + over);   // of dQ and dK/dV together
      const double time = one ? 0.14 + length * (0.16 + 0.51 * rounds) : 0.28 + length * rounds;
      if (best.waves == 0 || time < least) { best = {waves, one}; least = time; }
    }
  return best;
}
}  // namespace

hipError_t attention_fwd_f32(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) {
  return fwd_one_wave(d) ? by_head<Fwd, 1>(d, qkv, o, lse, st) : by_head<Fwd, kManyWaves>(d, qkv, o, lse, st);
}

hipError_t attention_bwd_f32(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta,
                             hipStream_t st) {
  const BwdForm f = bwd_form(d);
  return f.waves == 1 ? by_head<Bwd, 1>(d, f.one_launch, qkv, o, lse, d_o, dqkv, delta, st) : by_head<Bwd, kManyWaves>(d, f.one_launch, qkv, o, lse, d_o, dqkv, delta, st);
}

}  // namespace k2bw
