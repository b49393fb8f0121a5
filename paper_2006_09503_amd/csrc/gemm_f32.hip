// fp32 GEMM on the gfx950 matrix cores for the fp32 mode of the stage: v_mfma_f32_32x32x2_f32, fp32
// operands and accumulation throughout (fp32 MFMA peak of the part: 157.3 TFLOP/s).
//
// A 256-thread workgroup (2 x 2 waves) computes a 128 x 128 tile of C in K steps of 16 through two LDS
// stages; a wave owns 64 x 64 (2 x 2 MFMA blocks, 64 accumulator registers).  Both operand tiles sit in
// LDS k-major, [16 k][128 rows + 32 pad] floats: an MFMA fragment is then one 4-byte read per lane of 32
// consecutive rows at k (lanes 0..31) and at k+1 (lanes 32..63), and the pad of 32 puts the two halves
// on disjoint banks.  Global loads are 16-byte vectors along whichever index is contiguous in HBM (the
// tile of step kt+1 is in flight in registers while step kt runs its MFMAs); one barrier per K step.
// Any M, N, K: what lies outside the matrices is loaded as zero and never stored; operands whose leading
// dimension or base address do not allow 16-byte loads take guarded 4-byte loads instead.
//
// Products whose 128 x 128 tiles do not fill the chip run on gemm_f32_split_kernel (further down): tiles of 64 x 64 or 32 x 32 whose reduction range
// is split over the workgroup's waves; the smallest ones on gemm_f32_narrow_kernel, tiles of 16 x 16.
//
// Lane layout of v_mfma_f32_32x32x2_f32: lane l supplies element (l % 32, l / 32) of the first operand
// (32 x 2) and (l / 32, l % 32) of the second (2 x 32); it receives column l % 32 of D, rows
// 8*(r/4) + 4*(l/32) + (r % 4) for accumulator register r.  As in the bf16 kernels the B tile is fed as the
// first operand and the A tile as the second, so a lane owns one row m of C and four consecutive columns
// per register quad: the epilogue's accesses are 16-byte vectors.
#include <cmath>
#include <cstdio>
#include <type_traits>

#include "kernels.hpp"

namespace k2bw {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 128, BK = 16, LDT = 128 + 32;   // LDT: floats per k row of a staged tile
constexpr int kThreads = 256;

struct F32Params {
  const float* A; const float* B; float* C;
  int M, N, K, lda, ldb, ldc;
  const float* bias; const float* aux; float* aux_out;
  int accumulate;
  int vec_a, vec_b, vec_c;   // 16-byte accesses allowed on A, on B, on C / aux / aux_out / bias
};

// One operand's 128 x 16 tile on its way from HBM to LDS.  ROW_CONTIG: element (row, k) at X[k*ld + row],
// else at X[row*ld + k].  Two 16-byte pieces per thread.
template <bool ROW_CONTIG>
struct TileMover {
  float4 v[2];
  __device__ __forceinline__ void load(const float* __restrict__ X, int ld, int row0, int rows, int k0, int K, bool vec,
                                       int tid) {
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      int r, k;
      if (ROW_CONTIG) { k = tid / 32 + 8 * it; r = (tid % 32) * 4; }
      else { r = tid / 4 + 64 * it; k = (tid % 4) * 4; }
      const int gr = row0 + r, gk = k0 + k;
      float e[4] = {0.f, 0.f, 0.f, 0.f};
      if (ROW_CONTIG) {
        if (gk < K) {
          const float* p = X + (int64_t)gk * ld + gr;
          if (vec && gr + 3 < rows) {
            const float4 q = *reinterpret_cast<const float4*>(p);
            e[0] = q.x; e[1] = q.y; e[2] = q.z; e[3] = q.w;
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) if (gr + i < rows) e[i] = p[i];
          }
        }
      } else {
        if (gr < rows) {
          const float* p = X + (int64_t)gr * ld + gk;
          if (vec && gk + 3 < K) {
            const float4 q = *reinterpret_cast<const float4*>(p);
            e[0] = q.x; e[1] = q.y; e[2] = q.z; e[3] = q.w;
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) if (gk + i < K) e[i] = p[i];
          }
        }
      }
      v[it] = make_float4(e[0], e[1], e[2], e[3]);
    }
  }
  __device__ __forceinline__ void store(float* __restrict__ tile, int tid) const {
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      if (ROW_CONTIG) {
        const int k = tid / 32 + 8 * it, r = (tid % 32) * 4;
        *reinterpret_cast<float4*>(tile + k * LDT + r) = v[it];
      } else {
        const int r = tid / 4 + 64 * it, k = (tid % 4) * 4;
        tile[(k + 0) * LDT + r] = v[it].x; tile[(k + 1) * LDT + r] = v[it].y;
        tile[(k + 2) * LDT + r] = v[it].z; tile[(k + 3) * LDT + r] = v[it].w;
      }
    }
  }
};

// Epilogue of four consecutive columns gn .. gn+3 of row gm (gm < M, gn < N)
template <int EPI>
__device__ __forceinline__ void finish4(const F32Params& p, int gm, int gn, const float (&acc)[4]) {
  const int64_t idx = (int64_t)gm * p.ldc + gn;
  float v[4] = {acc[0], acc[1], acc[2], acc[3]};
  const bool whole = p.vec_c && gn + 3 < p.N;
  auto rd4 = [&](const float* src, float (&o)[4]) {
    if (whole) { const float4 q = *reinterpret_cast<const float4*>(src); o[0] = q.x; o[1] = q.y; o[2] = q.z; o[3] = q.w; }
    else {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = gn + i < p.N ? src[i] : 0.f;
    }
  };
  auto wr4 = [&](float* dst, const float (&o)[4]) {
    if (whole) *reinterpret_cast<float4*>(dst) = make_float4(o[0], o[1], o[2], o[3]);
    else {
#pragma unroll
      for (int i = 0; i < 4; ++i) if (gn + i < p.N) dst[i] = o[i];
    }
  };
  if (EPI == kEpiStore) {
    if (p.bias) { float b[4]; rd4(p.bias + gn, b);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] += b[i]; }
    if (p.aux) { float r[4]; rd4(p.aux + idx, r);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] += r[i]; }
    wr4(p.C + idx, v);
  } else if (EPI == kEpiGelu) {
    float b[4]; rd4(p.bias + gn, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] += b[i];
    wr4(p.C + idx, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = gelu_f(v[i]);
    wr4(p.aux_out + idx, v);
  } else if (EPI == kEpiGeluGrad) {
    float u[4]; rd4(p.aux + idx, u);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] *= gelu_grad_f(u[i]);
    wr4(p.C + idx, v);
  } else {
    if (p.accumulate) { float c[4]; rd4(p.C + idx, c);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = c[i] + v[i]; }
    wr4(p.C + idx, v);
  }
}

template <bool TA, bool TB, int EPI>
__global__ __launch_bounds__(kThreads) void gemm_f32_mfma_kernel(F32Params p) {
  __shared__ __attribute__((aligned(16))) float sA[2][BK * LDT];
  __shared__ __attribute__((aligned(16))) float sB[2][BK * LDT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;

  f32x16 acc[2][2];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  TileMover<TA> mv_a;     // A(m,k): m contiguous iff trans_a
  TileMover<!TB> mv_b;    // B(k,n): n contiguous iff not trans_b
  const int nk = (p.K + BK - 1) / BK;
  mv_a.load(p.A, p.lda, m0, p.M, 0, p.K, p.vec_a != 0, tid);
  mv_b.load(p.B, p.ldb, n0, p.N, 0, p.K, p.vec_b != 0, tid);
  mv_a.store(sA[0], tid);
  mv_b.store(sB[0], tid);
  __syncthreads();

  const int half = lane >> 5, l32 = lane & 31;
  for (int kt = 0; kt < nk; ++kt) {
    const float* a_t = sA[kt & 1];
    const float* b_t = sB[kt & 1];
    if (kt + 1 < nk) {   // uniform: the next tile travels in registers while this one is multiplied
      mv_a.load(p.A, p.lda, m0, p.M, (kt + 1) * BK, p.K, p.vec_a != 0, tid);
      mv_b.load(p.B, p.ldb, n0, p.N, (kt + 1) * BK, p.K, p.vec_b != 0, tid);
    }
#pragma unroll
    for (int kk = 0; kk < BK; kk += 2) {
      float af[2], bf[2];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi) af[mi] = a_t[(kk + half) * LDT + wm * 64 + mi * 32 + l32];
#pragma unroll
      for (int ni = 0; ni < 2; ++ni) bf[ni] = b_t[(kk + half) * LDT + wn * 64 + ni * 32 + l32];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(bf[ni], af[mi], acc[mi][ni], 0, 0, 0);
    }
    if (kt + 1 < nk) {
      mv_a.store(sA[(kt + 1) & 1], tid);
      mv_b.store(sB[(kt + 1) & 1], tid);
    }
    __syncthreads();
  }

  // Epilogue: lane owns row m and, per register quad g, columns n .. n+3.
#pragma unroll
  for (int mi = 0; mi < 2; ++mi) {
    const int gm = m0 + wm * 64 + mi * 32 + l32;
    if (gm >= p.M) continue;
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int gn = n0 + wn * 64 + ni * 32 + 8 * g + 4 * half;
        if (gn >= p.N) continue;
        const float v[4] = {acc[mi][ni][4 * g], acc[mi][ni][4 * g + 1], acc[mi][ni][4 * g + 2], acc[mi][ni][4 * g + 3]};
        finish4<EPI>(p, gm, gn, v);
      }
  }
}

// ------------------------------------------------------------------------------------------------
// Small products.  128 x 128 tiles leave most CUs without work when M or N is a few hundred (the tiny parity stage: 1 to 4
// workgroups), and each of them then walks the whole reduction range alone.  Here a workgroup owns a tile of 32*MB x 32*NB and
// its kSplit waves take every kSplit-th chunk of 16 k, each for the whole tile; the partial sums meet in LDS once, in a fixed
// order.  Nothing is shared inside the loop, so there is no LDS and no barrier in it: operands come straight into the
// fragment registers (16 bytes per lane where k is contiguous, 128-byte rows otherwise), one chunk ahead of their use.
// k-slots: instruction i of group j (8 k) takes k = 8j + i in lanes 0..31 and 8j + 4 + i in lanes 32..63, in both operands.
constexpr int kChunk = 16;

template <int NBLK, bool ROW_CONTIG>
struct FragLoader {   // fragments of 32*NBLK rows x kChunk k: f[block][k-instruction]
  const float* base[NBLK];
  int ld;
  __device__ __forceinline__ void init(const float* X, int ld_, int row0, int rows, int l32, int hf) {
    ld = ld_;
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
      const int r = min(row0 + 32 * b + l32, rows - 1);   // rows past the matrix: a copy, never stored
      base[b] = ROW_CONTIG ? X + r + (int64_t)(4 * hf) * ld : X + (int64_t)r * ld + 4 * hf;
    }
  }
  __device__ __forceinline__ void load(int k0, float (&f)[NBLK][kChunk / 2]) const {
#pragma unroll
    for (int b = 0; b < NBLK; ++b)
#pragma unroll
      for (int j = 0; j < kChunk / 8; ++j) {
        if (ROW_CONTIG) {
#pragma unroll
          for (int i = 0; i < 4; ++i) f[b][4 * j + i] = base[b][(int64_t)(k0 + 8 * j + i) * ld];
        } else {
          const float4 v = *reinterpret_cast<const float4*>(base[b] + k0 + 8 * j);
          f[b][4 * j] = v.x; f[b][4 * j + 1] = v.y; f[b][4 * j + 2] = v.z; f[b][4 * j + 3] = v.w;
        }
      }
  }
  // the last, partial chunk: what lies past K is zero
  __device__ __forceinline__ void load_tail(int k0, int K, int hf, float (&f)[NBLK][kChunk / 2]) const {
#pragma unroll
    for (int b = 0; b < NBLK; ++b)
#pragma unroll
      for (int e = 0; e < kChunk / 2; ++e) {
        const int k = k0 + 8 * (e / 4) + (e % 4);   // (base holds the 4*hf)
        f[b][e] = 0.f;
        if (k + 4 * hf < K) f[b][e] = ROW_CONTIG ? base[b][(int64_t)k * ld] : base[b][k];
      }
  }
};

constexpr int kGroupF32 = 24;   // products of one form that may share a launch
template <int CAP>
struct GroupOfF32 {
  F32Params p[CAP];
  int tile_start[CAP + 1];
  int count;
};
using GroupF32 = GroupOfF32<kGroupF32>;   // on the host
// What a launch carries (its arguments are copied on the host's time): only weight-gradient products share launches
template <int EPI>
constexpr int kLaunchCap = EPI == kEpiAccum ? kGroupF32 : 1;

template <int MB, int NB, int kSplit, bool TA, bool TB, int EPI, int CAP>
__device__ __forceinline__ void split_tile(const GroupOfF32<CAP>& gp, float* part) {   // part: [kSplit][TM][TN + 4]
  constexpr int TM = 32 * MB, TN = 32 * NB, LDS_LD = TN + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  int g = 0;
  if (CAP > 1)
    for (int q = 1; q < gp.count; ++q) g = (int)blockIdx.x >= gp.tile_start[q] ? q : g;
  const F32Params& p = gp.p[g];
  const int t = (int)blockIdx.x - gp.tile_start[g], tiles_n = (p.N + TN - 1) / TN;
  const int m0 = t / tiles_n * TM, n0 = t % tiles_n * TN;

  FragLoader<MB, TA> la;
  FragLoader<NB, !TB> lb;
  la.init(p.A, p.lda, m0, p.M, l32, hf);
  lb.init(p.B, p.ldb, n0, p.N, l32, hf);
  f32x16 acc[MB][NB];
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int ni = 0; ni < NB; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
  float a[2][MB][kChunk / 2], b[2][NB][kChunk / 2];
  auto multiply = [&](int s) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < kChunk / 2; ++e)
#pragma unroll
      for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[s][ni][e], a[s][mi][e], acc[mi][ni], 0, 0, 0);
  };
  const int full = p.K / kChunk;
  int c = wave;
  if (c < full) { la.load(c * kChunk, a[0]); lb.load(c * kChunk, b[0]); }
  for (; c < full; c += 2 * kSplit) {
    if (c + kSplit < full) { la.load((c + kSplit) * kChunk, a[1]); lb.load((c + kSplit) * kChunk, b[1]); }
    __builtin_amdgcn_sched_barrier(0);
    multiply(0);
    if (c + kSplit >= full) break;
    if (c + 2 * kSplit < full) { la.load((c + 2 * kSplit) * kChunk, a[0]); lb.load((c + 2 * kSplit) * kChunk, b[0]); }
    __builtin_amdgcn_sched_barrier(0);
    multiply(1);
  }
  if (full * kChunk < p.K && full % kSplit == wave) {
    la.load_tail(full * kChunk, p.K, hf, a[0]);
    lb.load_tail(full * kChunk, p.K, hf, b[0]);
    multiply(0);
  }
  // a lane owns row m and four consecutive columns per register quad
  float* mine = part + wave * TM * LDS_LD;
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int ni = 0; ni < NB; ++ni)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(mine + (mi * 32 + l32) * LDS_LD + ni * 32 + 8 * q + 4 * hf) =
            make_float4(acc[mi][ni][4 * q], acc[mi][ni][4 * q + 1], acc[mi][ni][4 * q + 2], acc[mi][ni][4 * q + 3]);
  __syncthreads();
  for (int e = tid; e < TM * TN / 4; e += kSplit * 64) {
    const int row = e / (TN / 4), col = e % (TN / 4) * 4;
    if (m0 + row >= p.M || n0 + col >= p.N) continue;
    float4 s = *reinterpret_cast<const float4*>(part + row * LDS_LD + col);
#pragma unroll
    for (int w = 1; w < kSplit; ++w) {
      const float4 v = *reinterpret_cast<const float4*>(part + (w * TM + row) * LDS_LD + col);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    const float v[4] = {s.x, s.y, s.z, s.w};
    finish4<EPI>(p, m0 + row, n0 + col, v);
  }
}
template <int MB, int NB, int kSplit, bool TA, bool TB, int EPI>
__global__ __launch_bounds__(kSplit * 64) void gemm_f32_split_kernel(GroupOfF32<kLaunchCap<EPI>> gp) {
  extern __shared__ __attribute__((aligned(16))) float part[];
  split_tile<MB, NB, kSplit, TA, TB, EPI>(gp, part);
}

// Weight gradients in 32 x 32 tiles and, in the workgroups behind theirs, sums over the rows of matrices (the bias, gain and shift gradients of
// the same pass: colsum_finalize_grouped), which have nothing to do with them but to be due at the same time: one launch less per pass of a
// stage that is bound by its launches (two layers of 128 tokens, h = 128: 23.3 -> 22.3 per microbatch; a launch of few products also carries
// 2 instead of 4.3 KB of arguments).  A workgroup owns 64 columns: 16 threads x 16 bytes along a row, 32 such groups walk the rows.
constexpr int kSumProducts = 16, kSumItems = 24;
struct SumItems {
  const float* in[kSumItems];
  float* out[kSumItems];
  int rows[kSumItems], n[kSumItems], ld[kSumItems], block0[kSumItems];
  int count, accumulate;
};
__global__ __launch_bounds__(512) void gemm_f32_wgrad_sums_kernel(GroupOfF32<kSumProducts> gp, SumItems g) {
  extern __shared__ __attribute__((aligned(16))) float part[];
  const int block = (int)blockIdx.x - gp.tile_start[kSumProducts];
  if (block < 0) {
    split_tile<1, 1, 8, true, false, kEpiAccum>(gp, part);
    return;
  }
  float4 (*red)[17] = reinterpret_cast<float4 (*)[17]>(part);   // [32][17]
  int q = 0;
  for (int i = 1; i < g.count; ++i) q = block >= g.block0[i] ? i : q;
  const float* in = g.in[q];
  const int rows = g.rows[q], n = g.n[q], ld = g.ld[q];
  const int c = threadIdx.x & 15, pl = threadIdx.x >> 4, col = ((block - g.block0[q]) * 16 + c) * 4;
  auto add = [](float4& a, const float4& b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; };
  auto at = [&](int r) { return *reinterpret_cast<const float4*>(in + (int64_t)r * ld + col); };
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (col < n) {
    int r = pl;
    for (; r + 3 * 32 < rows; r += 4 * 32) {   // four rows in flight, added as a tree
      float4 v[4] = {at(r), at(r + 32), at(r + 64), at(r + 96)};
      add(v[0], v[2]); add(v[1], v[3]); add(v[0], v[1]); add(s, v[0]);
    }
    for (; r < rows; r += 32) add(s, at(r));
  }
  red[pl][c] = s;
  __syncthreads();
  if (pl == 0 && col < n) {
    float4 v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = red[i][c];
#pragma unroll
    for (int w = 16; w > 0; w /= 2)
#pragma unroll
      for (int i = 0; i < w; ++i) add(v[i], v[i + w]);
    float4* out = reinterpret_cast<float4*>(g.out[q] + col);
    if (g.accumulate) add(v[0], *out);
    *out = v[0];
  }
}

// ------------------------------------------------------------------------------------------------
// The smallest products (at most one tile of 16 x 16 per CU): v_mfma_f32_16x16x4_f32, so that four times as many CUs as with 32 x 32 share
// the operands' way in and the products themselves (a 32 x 32 tile with K = 1024 is 3.5 us of one CU's matrix cores).
// The eight waves take every eighth chunk of 16 k, two chunks of a wave in flight at once.  With more of them a wave asks for chunks that
// it has not got whenever its share is no multiple, and starts on its first one later.  2 | 4 | 8 chunks in us, means over 650 random
// sizes by K: 256 to 384 3.1 | 3.3 | 4.1; 1200 to 1700 5.3 | 6.0 | 7.3; 4800 to 6800 15.0 | 16.6 | 19.5; operands from memory instead of L2,
// 256 to 360 3.8 | 3.9 | 4.5, 2048 to 2900 11.4 | 11.4 | 12.5.
// Lane layout: lane l supplies row l % 16 of either operand at k = l / 16 and receives column l % 16, rows 4 * (l / 16) + r.
// k-slots: instruction i of a chunk takes k = 4 * (l / 16) + i in lane l.
template <bool ROW_CONTIG>
struct NarrowLoader {
  const float* base;
  int ld;
  __device__ __forceinline__ void init(const float* X, int ld_, int row0, int rows, int l16, int quarter) {
    ld = ld_;
    const int r = min(row0 + l16, rows - 1);   // rows past the matrix: a copy, never stored
    base = ROW_CONTIG ? X + r + (int64_t)(4 * quarter) * ld : X + (int64_t)r * ld + 4 * quarter;
  }
  __device__ __forceinline__ void load(int k0, float (&f)[4]) const {
    if (ROW_CONTIG) {
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = base[(int64_t)(k0 + i) * ld];
    } else {
      const float4 v = *reinterpret_cast<const float4*>(base + k0);
      f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
  }
};
constexpr int kNarrow = 16, kNarrowWaves = 8, kNarrowChunks = 2;

// The waves' partial sums of a 16 x 16 tile (a lane owns row l16 and four consecutive columns) to the epilogue
template <int EPI>
__device__ __forceinline__ void finish_narrow(const F32Params& p, const f32x4& acc, float* part, int m0, int n0, int tid, int wave) {
  constexpr int T = kNarrow, LDS_LD = T + 4;
  const int lane = tid & 63;
  *reinterpret_cast<float4*>(part + (wave * T + (lane & 15)) * LDS_LD + 4 * (lane >> 4)) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  if (tid < T * T / 4) {
    const int row = tid / (T / 4), col = tid % (T / 4) * 4;
    if (m0 + row >= p.M || n0 + col >= p.N) return;
    float4 s = *reinterpret_cast<const float4*>(part + row * LDS_LD + col);
#pragma unroll
    for (int w = 1; w < kNarrowWaves; ++w) {
      const float4 v = *reinterpret_cast<const float4*>(part + (w * T + row) * LDS_LD + col);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    const float v[4] = {s.x, s.y, s.z, s.w};
    finish4<EPI>(p, m0 + row, n0 + col, v);
  }
}

template <bool TB, int EPI>
__global__ __launch_bounds__(kNarrowWaves * 64) void gemm_f32_narrow_kernel(F32Params p) {
  constexpr int W = kNarrowWaves, T = kNarrow, NC = kNarrowChunks;
  __shared__ __attribute__((aligned(16))) float part[W * T * (T + 4)];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, quarter = lane >> 4;
  const int tiles_n = (p.N + T - 1) / T, m0 = (int)blockIdx.x / tiles_n * T, n0 = (int)blockIdx.x % tiles_n * T;
  NarrowLoader<false> la;
  NarrowLoader<!TB> lb;
  la.init(p.A, p.lda, m0, p.M, l16, quarter);
  lb.init(p.B, p.ldb, n0, p.N, l16, quarter);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int chunks = p.K / kChunk;
  for (int c0 = wave; c0 < chunks; c0 += NC * W) {
    float a[NC][4], b[NC][4];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = min(c0 + i * W, chunks - 1);   // past the end: the last one again, not multiplied
      la.load(c * kChunk, a[i]);
      lb.load(c * kChunk, b[i]);
    }
    __builtin_amdgcn_sched_barrier(0);   // (else the loads sink to their uses)
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      if (c0 + i * W >= chunks) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(b[i][e], a[i][e], acc, 0, 0, 0);
    }
  }
  const int rem = p.K % kChunk;   // a multiple of 4: whole quarters of a chunk
  if (rem > 0 && chunks % W == wave) {
    float a[4], b[4];
    const bool in = 4 * quarter < rem;
    const int k0 = chunks * kChunk - (in ? 0 : 4 * quarter);   // (the chunk's first quarter in place of one that is not there)
    la.load(k0, a);
    lb.load(k0, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? b[e] : 0.f, in ? a[e] : 0.f, acc, 0, 0, 0);
  }
  finish_narrow<EPI>(p, acc, part, m0, n0, tid, wave);
}

// ------------------------------------------------------------------------------------------------
// A LayerNorm and the product that reads its result, in one launch: 16 x 16 tiles as above, the A operand made on the way from the rows
// the LayerNorm reads.  A wave's chunks of A are pieces of all the tile's 16 rows, so each wave adds up its part of the rows' sums, the
// parts meet in LDS, and the wave turns its fragments into the normalised ones (BWD: into the LayerNorm's input gradient) in
// registers.  What the LayerNorm leaves behind for later launches is written by the workgroup whose columns of C have the same numbers:
// its 16 columns of the result, of the copies and of the column sums over its 16 rows.  A stage of few tokens is bound by the number of
// its launches: 3 to 5 us each for LayerNorms of 128 x 128, whatever they compute (lines at ln_fits).
struct LnArgs {
  const float *x, *gain;
  float *mean, *rstd, *y;      // y: the LayerNorm's result, BWD: its input gradient
  float* keep;                 // a copy of x (BWD: of dres), or null
  const float* shift;          // forward
  float eps;
  const int32_t* n_in; int32_t* n_out; int n;   // integers to copy
  const float *dy, *dres; float* partial;       // BWD; partial: [ceil(M / 16)][3 K]
};
constexpr int kLnMaxChunks = 4;   // chunks per wave

// sum over the 16 lanes of a DPP row
__device__ __forceinline__ float row16_sum(float v) {
  auto dpp_add = [](float x, auto ctrl) {
    const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, false);
    return x + __builtin_bit_cast(float, y);
  };
  v = dpp_add(v, std::integral_constant<int, 0xB1>{});      // quad_perm [1,0,3,2]
  v = dpp_add(v, std::integral_constant<int, 0x4E>{});      // quad_perm [2,3,0,1]
  v = dpp_add(v, std::integral_constant<int, 0x141>{});     // row_half_mirror
  return dpp_add(v, std::integral_constant<int, 0x140>{});  // row_mirror
}

template <bool BWD, int NC, bool TB, int EPI>
__global__ __launch_bounds__(kNarrowWaves * 64) void gemm_f32_ln_kernel(F32Params p, LnArgs q) {
  constexpr int W = kNarrowWaves, T = kNarrow;
  __shared__ __attribute__((aligned(16))) float part[W * T * (T + 4)];
  __shared__ float row_part[2][W][T];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, quarter = lane >> 4;
  const int tiles_n = (p.N + T - 1) / T, mt = (int)blockIdx.x / tiles_n, nt = (int)blockIdx.x % tiles_n;
  const int m0 = mt * T, n0 = nt * T;
  const bool row_ok = m0 + l16 < p.M;
  const int row = min(m0 + l16, p.M - 1);   // rows past the matrix: a copy, never stored
  const int chunks = p.K / kChunk;
  if (blockIdx.x == 0)
    for (int i = tid; i < q.n; i += W * 64) q.n_out[i] = q.n_in[i];

  NarrowLoader<!TB> lb;
  lb.init(p.B, p.ldb, n0, p.N, l16, quarter);
  float x[NC][4], a[NC][4], g[NC][4], r[NC][4], b[NC][4];   // a: dy (BWD); r: shift (BWD: dres)
  auto load = [&](const float* from, float (&f)[4]) __attribute__((always_inline)) {
    const float4 v = *reinterpret_cast<const float4*>(from);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  };
  auto store = [&](float* to, const float (&f)[4]) __attribute__((always_inline)) { *reinterpret_cast<float4*>(to) = make_float4(f[0], f[1], f[2], f[3]); };
  float s1 = 0.f, s2 = 0.f, mean = 0.f, rstd = 0.f;
  if (BWD) { mean = q.mean[row]; rstd = q.rstd[row]; }
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = wave + i * W;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[i][e] = a[i][e] = g[i][e] = r[i][e] = b[i][e] = 0.f;
    if (c >= chunks) continue;   // wave-uniform
    const int col = c * kChunk + 4 * quarter;
    const int64_t at = (int64_t)row * p.K + col;
    load(q.x + at, x[i]);
    load(q.gain + col, g[i]);
    if (BWD) {
      load(q.dy + at, a[i]);
      load(q.dres + at, r[i]);
    } else {
      load(q.shift + col, r[i]);
    }
    lb.load(c * kChunk, b[i]);
  }
  // sums over the rows: own pieces, the wave's other quarters, the other waves
  auto row_sum = [&](float v, int slot) __attribute__((always_inline)) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (quarter == 0) row_part[slot][wave][l16] = v;
  };
  auto total = [&](int slot) __attribute__((always_inline)) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) t += row_part[slot][w][l16];
    return t;
  };
  if constexpr (!BWD) {
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) s1 += x[i][e];
    row_sum(s1, 0);
    __syncthreads();
    mean = total(0) / (float)p.K;
#pragma unroll
    for (int i = 0; i < NC; ++i)
      if (wave + i * W < chunks)
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float d = x[i][e] - mean; s2 += d * d; }
    row_sum(s2, 1);
    __syncthreads();
    rstd = 1.0f / sqrtf(total(1) / (float)p.K + q.eps);
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) a[i][e] = g[i][e] * ((x[i][e] - mean) * rstd) + r[i][e];
    if (nt == 0 && wave == 0 && quarter == 0 && row_ok) { q.mean[row] = mean; q.rstd[row] = rstd; }
  } else {
    // x becomes xhat, g the gradient dy * gain of xhat; dy stays for the sums
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[i][e] = wave + i * W < chunks ? (x[i][e] - mean) * rstd : 0.f;
        g[i][e] *= a[i][e];
        s1 += g[i][e];
        s2 += g[i][e] * x[i][e];
      }
    row_sum(s1, 0);
    row_sum(s2, 1);
    __syncthreads();
    const float c1 = total(0) / (float)p.K, c2 = total(1) / (float)p.K;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      if (wave + i * W == nt && nt < chunks && row_ok && q.keep) store(q.keep + (int64_t)row * p.K + nt * kChunk + 4 * quarter, r[i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) r[i][e] += rstd * (g[i][e] - c1 - x[i][e] * c2);
    }
  }
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    if (wave + i * W >= chunks) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(b[i][e], BWD ? r[i][e] : a[i][e], acc, 0, 0, 0);
  }
  // what the LayerNorm leaves behind in the columns nt * 16 .. + 15, from the wave that has them
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    if (wave + i * W != nt || nt >= chunks) continue;   // wave-uniform
    const int col = nt * kChunk + 4 * quarter;
    const int64_t at = (int64_t)row * p.K + col;
    if (row_ok) store(q.y + at, BWD ? r[i] : a[i]);
    if constexpr (!BWD) {
      if (row_ok && q.keep) store(q.keep + at, x[i]);
    } else {
      float v[3][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float dy = row_ok ? a[i][e] : 0.f;
        v[0][e] = row16_sum(row_ok ? dy * x[i][e] : 0.f);
        v[1][e] = row16_sum(dy);
        v[2][e] = row16_sum(row_ok ? r[i][e] : 0.f);
      }
      if (l16 == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) store(q.partial + ((int64_t)mt * 3 + k) * p.K + col, v[k]);
    }
  }
  finish_narrow<EPI>(p, acc, part, m0, n0, tid, wave);
}

// ------------------------------------------------------------------------------------------------
template <int MB, int NB, int kSplit, bool TA, bool TB, int EPI>
hipError_t launch_split(GroupF32& gp, hipStream_t s) {
  constexpr size_t lds = (size_t)kSplit * 32 * MB * (32 * NB + 4) * sizeof(float);
  static bool done = false;
  if (!done && lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_f32_split_kernel<MB, NB, kSplit, TA, TB, EPI>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    done = true;
  }
  int total = 0;
  for (int g = 0; g < gp.count; ++g) {
    gp.tile_start[g] = total;
    total += ceil_div(gp.p[g].M, 32 * MB) * ceil_div(gp.p[g].N, 32 * NB);
  }
  gp.tile_start[gp.count] = total;
  GroupOfF32<kLaunchCap<EPI>> l;
  l.count = gp.count;
  for (int g = 0; g < gp.count; ++g) { l.p[g] = gp.p[g]; l.tile_start[g] = gp.tile_start[g]; }
  l.tile_start[gp.count] = total;
  hipLaunchKernelGGL((gemm_f32_split_kernel<MB, NB, kSplit, TA, TB, EPI>), dim3(total), dim3(kSplit * 64), lds, s, l);
  return hipGetLastError();
}

// The split kernels load a K-contiguous operand 16 bytes at a time
bool split_ok(const F32Params& p, bool ta, bool tb) { return (ta || p.vec_a) && (!tb || p.vec_b); }

int64_t narrow_tiles(const F32Params& p) { return (int64_t)ceil_div(p.M, kNarrow) * ceil_div(p.N, kNarrow); }
template <bool TB, int EPI>
hipError_t launch_narrow(const F32Params& p, hipStream_t s) {
  hipLaunchKernelGGL((gemm_f32_narrow_kernel<TB, EPI>), dim3((int)narrow_tiles(p)), dim3(kNarrowWaves * 64), 0, s, p);
  return hipGetLastError();
}

// Tile edge for `count` products of one form (128: one product per launch on the staged kernel): the one with the least estimated
// time.  In microseconds, with R tiles per CU, C = ceil(R) rounds and K in thousands: a launch has a fixed part, a part per tile of a
// CU (its first loads, its sums and its trip through C) and a part per k, which the split kernels pay by whole rounds; so does the
// staged kernel up to two workgroups per CU, where the part per tile also shrinks with what of a tile exists (`fill`).  Fitted to
// launches of 260 random sizes (M, N, K of 8 to 8192) with each edge forced: 6 to 12 % off each time, and the choice costs 0.4 % over
// the best edge on average.  What keeps short reduction ranges on 128 x 128 tiles is the part per tile.  Edge 128, 64, 32 in us:
// forward 4620 x 5408 x 8 37, 83, 63; 1438 x 5208 x 16 16, 30, 22; 2702 x 5584 x 216 82, 119, -; weight gradient 4620 x 5408 x 8
// 53, 119, 100; 4036 x 1920 x 48 25, 46, 38; 4278 x 7992 x 181 165, 273, -.  Small products, forward | data gradient | weight
// gradient (tokens, in, out): (128,512,128) 54|18|19, 14|7.3|7.7, 6.4|4.1|4.4; (512,1024,3072) 102|289|57, 50|63|46, 47|47|51;
// (2048,1024,1024) 103|102|180, 52|57|48, 59|62|68; (4096,1024,4096) 307|389|357, 371|317|333, 425|464|462.
struct EdgeCost { double few0, few_tile, few_k, many0, many_tile, many_k, t64_0, t64_tile, t64_k, t32_0, t32_tile, t32_k; };
int choose_f32(const F32Params* p, int count, bool ta, bool tb) {
  static constexpr EdgeCost kCost[3] = {
      {2.75, 3.4, 92.0, 6.8, 3.9, 72.0, 3.6, 2.9, 18.6, 3.3, 0.50, 6.1},   // rows of B along N (forward)
      {2.75, 3.7, 87.6, 6.3, 4.0, 69.3, 3.6, 1.5, 17.6, 3.3, 0.42, 5.5},   // both along K (data gradient)
      {3.25, 6.5, 95.6, 7.0, 7.3, 67.2, 5.0, 4.3, 19.2, 3.6, 0.91, 6.7}};  // A along M (weight gradient: C is read and written)
  const EdgeCost& q = kCost[ta ? 2 : tb ? 1 : 0];
  const double cus = gemm_compute_units();
  double c128 = 0, r64 = 0, k64 = 0, r32 = 0, k32 = 0;
  for (int g = 0; g < count; ++g) {
    if (!split_ok(p[g], ta, tb)) return 128;
    auto per_cu = [&](int edge) { return (double)ceil_div(p[g].M, edge) * ceil_div(p[g].N, edge) / cus; };
    const double r = per_cu(128), k = p[g].K * 1e-3;
    const double fill = (p[g].M < 128 ? p[g].M / 128.0 : 1.0) * (p[g].N < 128 ? p[g].N / 128.0 : 1.0);
    c128 += r <= 2 ? q.few0 + std::ceil(r) * (q.few_tile * fill + q.few_k * k) : q.many0 + r * (q.many_tile + q.many_k * k);
    r64 += per_cu(64); k64 += per_cu(64) * k;
    r32 += per_cu(32); k32 += per_cu(32) * k;
  }
  const double c64 = q.t64_0 + q.t64_tile * r64 + q.t64_k * std::ceil(r64) * (k64 / r64);
  const double c32 = q.t32_0 + q.t32_tile * r32 + q.t32_k * std::ceil(r32) * (k32 / r32);
  if (c128 <= c64 && c128 <= c32) return 128;
  if (c64 <= c32) return 64;
  // 16 x 16 tiles take 0.4 to 0.7 of the time as long as every CU has one tile at most; a second one takes as long again, and each brings
  // twice the bytes of a 32 x 32 tile's share.  Tiles of 16 per CU, 32 x 32 | 16 x 16 in us: (tokens, in, out) forward (128,256,256) 0.5
  // 4.1 | 2.8; (128,1024,256) 0.5 9.2 | 4.5; (100,2048,128) 0.22 15.9 | 6.6; (128,4096,512) 1.0 29.8 | 11.7; (16,1024,4096) 1.0 8.6 | 5.5;
  // (16,4096,4096) 1.0 30.4 | 22.7, one token 28.3 | 21.2; (51,2320,1352) 1.33 20.0 | 19.8; data gradient 16 x 4096, K = 4096 1.0 26.5 | 17.0;
  // 15 x 672, K = 288 0.16 4.1 | 3.2; 925 x 80, K = 712 1.13 7.3 | 5.7; 926 x 120, K = 1416 1.81 11.2 | 11.2.  1200 random sizes below the line:
  // 0.60 of the time of 32 x 32, at worst 1.02 (14 x 72, K = 128).
  return !ta && count == 1 && p[0].K % 4 == 0 && narrow_tiles(p[0]) <= cus ? 16 : 32;
}

template <bool TA, bool TB, int EPI>
hipError_t launch_form(GroupF32& gp, hipStream_t s) {
  if (gp.count > kLaunchCap<EPI>) return hipErrorInvalidValue;
  switch (choose_f32(gp.p, gp.count, TA, TB)) {
    case 64: return launch_split<2, 2, 4, TA, TB, EPI>(gp, s);
    case 32: return launch_split<1, 1, 8, TA, TB, EPI>(gp, s);
    case 16:
      if constexpr (!TA) return launch_narrow<TB, EPI>(gp.p[0], s);
      return hipErrorInvalidValue;
  }
  for (int g = 0; g < gp.count; ++g) {
    const F32Params& p = gp.p[g];
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<TA, TB, EPI>), dim3(ceil_div(p.N, BN), ceil_div(p.M, BM)), dim3(kThreads), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool TA, bool TB>
hipError_t launch_epi(GroupF32& gp, int epi, hipStream_t s) {
  switch (epi) {
    case kEpiStore: return launch_form<TA, TB, kEpiStore>(gp, s);
    case kEpiGelu: return launch_form<TA, TB, kEpiGelu>(gp, s);
    case kEpiGeluGrad: return launch_form<TA, TB, kEpiGeluGrad>(gp, s);
    case kEpiAccum: return launch_form<TA, TB, kEpiAccum>(gp, s);
    default: return hipErrorInvalidValue;
  }
}

bool vec16(const void* ptr, int ld) { return (reinterpret_cast<uintptr_t>(ptr) & 15) == 0 && ld % 4 == 0; }

F32Params to_params(const GemmDesc& d) {
  F32Params p{static_cast<const float*>(d.A), static_cast<const float*>(d.B), static_cast<float*>(d.C),
              d.M, d.N, d.K, d.lda, d.ldb, d.ldc, static_cast<const float*>(d.bias), static_cast<const float*>(d.aux),
              static_cast<float*>(d.aux_out), d.accumulate ? 1 : 0, 0, 0, 0};
  p.vec_a = vec16(d.A, d.lda);
  p.vec_b = vec16(d.B, d.ldb);
  p.vec_c = vec16(d.C, d.ldc) && (!d.aux || vec16(d.aux, d.ldc)) && (!d.aux_out || vec16(d.aux_out, d.ldc)) &&
            (!d.bias || vec16(d.bias, 4));
  return p;
}

bool aligned16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) == 0; }

// Whether the LayerNorm in front of product d goes into its launch: small products only, since every workgroup makes the LayerNorm of its
// rows again.  Three batches of 4 microbatches of an fp32 stage with and without, us (tokens x h, f = 4 h): 128 x 128 1800 -> 1499, 300 x 128
// 1822 -> 1486, 1024 x 128 1205 -> 1109 (one layer), 180 x 192 2205 -> 2014, 1000 x 64 2054 -> 1845, 128 x 256 1805 -> 1494, 128 x 512 1812 ->
// 1781; with the output projection's data gradient too (64 x 16 tiles of K = 256) 1024 x 256 3370 -> 3435, so the line is below that.
// (Above K = 256 the products alone have become faster since, two chunks in flight: 60 random stages of two layers with h = 256 to 512 and up to
// 500 tokens 0.90 of the time of the separate launches, at worst 1.01.)
bool ln_fits(const GemmDesc& d) {
  if (d.dtype != kF32 || d.trans_a || d.n_seg != 1 || d.K % kChunk || d.K > kLnMaxChunks * kNarrowWaves * kChunk || d.N < d.K) return false;
  const F32Params p = to_params(d);
  return p.vec_b && choose_f32(&p, 1, false, d.trans_b) <= 32 && narrow_tiles(p) * d.K <= 200000;
}

int ln_chunks(int K) {   // of a wave
  const int c = ceil_div(K, kNarrowWaves * kChunk);
  return c <= 2 ? c : kLnMaxChunks;
}
template <bool BWD, bool TB, int EPI>
hipError_t launch_ln(const F32Params& p, const LnArgs& q, hipStream_t s) {
  const dim3 grid((int)narrow_tiles(p)), block(kNarrowWaves * 64);
  switch (ln_chunks(p.K)) {
    case 1: hipLaunchKernelGGL((gemm_f32_ln_kernel<BWD, 1, TB, EPI>), grid, block, 0, s, p, q); break;
    case 2: hipLaunchKernelGGL((gemm_f32_ln_kernel<BWD, 2, TB, EPI>), grid, block, 0, s, p, q); break;
    default: hipLaunchKernelGGL((gemm_f32_ln_kernel<BWD, kLnMaxChunks, TB, EPI>), grid, block, 0, s, p, q); break;
  }
  return hipGetLastError();
}

}  // namespace

// `count` products of the same form and epilogue (1..kGemmMaxGroup); small ones share a launch
hipError_t gemm_f32_grouped(const GemmDesc* d, int count, hipStream_t stream) {
  static_assert(kGemmMaxGroup <= kGroupF32, "");
  if (count < 1 || count > kGroupF32) return hipErrorInvalidValue;
  GroupF32 gp;
  gp.count = count;
  for (int g = 0; g < count; ++g) {
    if (d[g].trans_a != d[0].trans_a || d[g].trans_b != d[0].trans_b || d[g].epilogue != d[0].epilogue) return hipErrorInvalidValue;
    gp.p[g] = to_params(d[g]);
  }
  if (d[0].trans_a) return d[0].trans_b ? launch_epi<true, true>(gp, d[0].epilogue, stream) : launch_epi<true, false>(gp, d[0].epilogue, stream);
  return d[0].trans_b ? launch_epi<false, true>(gp, d[0].epilogue, stream) : launch_epi<false, false>(gp, d[0].epilogue, stream);
}

bool gemm_ln_fwd_fits(const GemmDesc& d) { return !d.trans_b && (d.epilogue == kEpiStore || d.epilogue == kEpiGelu) && ln_fits(d); }
bool gemm_ln_bwd_fits(const GemmDesc& d) { return d.trans_b && d.M <= kNarrow * ln_bwd_max_parts() && (d.epilogue == kEpiStore || d.epilogue == kEpiGeluGrad) && ln_fits(d); }

hipError_t gemm_ln_fwd(const GemmDesc& d, const LnForward& ln, hipStream_t stream) {
  if (!gemm_ln_fwd_fits(d)) return hipErrorInvalidValue;
  LnArgs q{};
  q.x = static_cast<const float*>(ln.x); q.gain = static_cast<const float*>(ln.gain); q.shift = static_cast<const float*>(ln.shift);
  q.y = static_cast<float*>(ln.y); q.mean = ln.mean; q.rstd = ln.rstd; q.eps = ln.eps;
  if (ln.keep) { q.keep = static_cast<float*>(ln.keep->x); q.n_in = ln.keep->n_in; q.n_out = ln.keep->n_out; q.n = ln.keep->n; }
  const F32Params p = to_params(d);
  return d.epilogue == kEpiGelu ? launch_ln<false, false, kEpiGelu>(p, q, stream) : launch_ln<false, false, kEpiStore>(p, q, stream);
}

hipError_t gemm_ln_bwd(const GemmDesc& d, const LnBackward& ln, hipStream_t stream) {
  if (!gemm_ln_bwd_fits(d)) return hipErrorInvalidValue;
  LnArgs q{};
  q.x = static_cast<const float*>(ln.x); q.gain = static_cast<const float*>(ln.gain); q.mean = const_cast<float*>(ln.mean);
  q.rstd = const_cast<float*>(ln.rstd); q.y = static_cast<float*>(ln.dx); q.keep = static_cast<float*>(ln.dres_keep);
  q.dy = static_cast<const float*>(ln.dy); q.dres = static_cast<const float*>(ln.dres); q.partial = ln.partial;
  const F32Params p = to_params(d);
  return d.epilogue == kEpiGeluGrad ? launch_ln<true, true, kEpiGeluGrad>(p, q, stream) : launch_ln<true, true, kEpiStore>(p, q, stream);
}

void gemm_ln_kernel_name(const GemmDesc& d, char* out, size_t cap) {
  const char* tb = d.trans_b ? "true" : "false";
  snprintf(out, cap, "gemm_f32_ln_kernel<%s, %d, %s, %d>", tb, ln_chunks(d.K), tb, d.epilogue);
}

bool gemm_sums_fit(const GemmDesc* d, int count, const FinalizeItem* items, int n) {
  if (count < 1 || count > kSumProducts || n < 1 || n > kSumItems) return false;
  F32Params p[kSumProducts];
  for (int g = 0; g < count; ++g) {
    if (d[g].dtype != kF32 || !d[g].trans_a || d[g].trans_b || d[g].epilogue != kEpiAccum || d[g].n_seg != 1) return false;
    p[g] = to_params(d[g]);
  }
  for (int i = 0; i < n; ++i)
    if (items[i].parts <= 0 || items[i].n <= 0 || items[i].n % 4 || items[i].ld % 4 || items[i].ld < items[i].n || !aligned16(items[i].partial) || !aligned16(items[i].out))
      return false;
  return choose_f32(p, count, true, false) == 32;
}

hipError_t gemm_with_sums(const GemmDesc* d, int count, const FinalizeItem* items, int n, bool accumulate, hipStream_t stream) {
  if (!gemm_sums_fit(d, count, items, n)) return hipErrorInvalidValue;
  GroupOfF32<kSumProducts> gp;
  gp.count = count;
  int total = 0;
  for (int g = 0; g <= kSumProducts; ++g) {
    gp.tile_start[g] = total;
    if (g >= count) continue;
    gp.p[g] = to_params(d[g]);
    total += ceil_div(d[g].M, 32) * ceil_div(d[g].N, 32);
  }
  SumItems s;
  s.count = n;
  s.accumulate = accumulate ? 1 : 0;
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    s.in[i] = items[i].partial; s.out[i] = items[i].out; s.rows[i] = items[i].parts; s.n[i] = items[i].n; s.ld[i] = items[i].ld;
    s.block0[i] = blocks;
    blocks += ceil_div(items[i].n, 64);
  }
  constexpr size_t lds = 8 * 32 * (32 + 4) * sizeof(float);
  static_assert(lds >= 32 * 17 * sizeof(float4) && lds <= 64 * 1024, "");
  hipLaunchKernelGGL(gemm_f32_wgrad_sums_kernel, dim3(total + blocks), dim3(512), lds, stream, gp, s);
  return hipGetLastError();
}

void gemm_f32_kernel_name(const GemmDesc* d, int count, char* out, size_t cap) {
  F32Params p[kGroupF32];
  const int n = count < kGroupF32 ? count : kGroupF32;
  for (int g = 0; g < n; ++g) p[g] = to_params(d[g]);
  const char* ta = d[0].trans_a ? "true" : "false";
  const char* tb = d[0].trans_b ? "true" : "false";
  switch (choose_f32(p, n, d[0].trans_a, d[0].trans_b)) {
    case 64: snprintf(out, cap, "gemm_f32_split_kernel<2, 2, 4, %s, %s, %d>", ta, tb, d[0].epilogue); break;
    case 32: snprintf(out, cap, "gemm_f32_split_kernel<1, 1, 8, %s, %s, %d>", ta, tb, d[0].epilogue); break;
    case 16: snprintf(out, cap, "gemm_f32_narrow_kernel<%s, %d>", tb, d[0].epilogue); break;
    default: snprintf(out, cap, "gemm_f32_mfma_kernel<%s, %s, %d>", ta, tb, d[0].epilogue); break;
  }
}

}  // namespace k2bw
