// LayerNorm forward / backward and column-sum kernels (HBM-bound).
//
// A row of length h is handled by R threads (R = 64: one wavefront, 128 or 256: two or four
// wavefronts of the 256-thread workgroup), each owning CPT chunks of 8 consecutive elements,
// chunk index = sub + c*R, so that the R threads' 16-byte accesses are contiguous.  The row
// stays in registers between the statistics and the normalisation: one read, one write.
// Statistics are fp32: mean first, then the centred sum of squares (biased variance).
#include "kernels.hpp"

namespace k2bw {
namespace {

constexpr int kWg = 256;

struct ColsumGroup {
  const void* y[4];
  int n[4], ld[4], block0[4], col0[4];
  int count, rows, rows_per_part, total_cols;
  float* partial;
};
struct FinalizeGroup {
  const float* partial[kFinalizeMaxItems];
  float* out[kFinalizeMaxItems];
  int parts[kFinalizeMaxItems], n[kFinalizeMaxItems], ld[kFinalizeMaxItems], block0[kFinalizeMaxItems];
  int count, accumulate;
};

// sum over the R threads that share a row; R == 64 needs no LDS
template <int R>
__device__ __forceinline__ float group_sum(float v, float* red, int tid) {
  v = wave_sum(v);
  if (R == 64) return v;
  constexpr int W = R / 64;           // waves per row
  const int wave = tid >> 6;
  __syncthreads();                    // red may still be read from the previous call
  if ((tid & 63) == 0) red[wave] = v;
  __syncthreads();
  float s = 0.f;
  const int first = (wave / W) * W;
#pragma unroll
  for (int i = 0; i < W; ++i) s += red[first + i];
  return s;
}

// Eight consecutive elements as they lie in memory
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> { uint4 a; };
template <> struct Raw8<float> { float4 a, b; };
__device__ __forceinline__ void load_raw(const bf16_t* p, Raw8<bf16_t>& r) { r.a = *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void load_raw(const float* p, Raw8<float>& r) {
  r.a = *reinterpret_cast<const float4*>(p);
  r.b = *reinterpret_cast<const float4*>(p + 4);
}
__device__ __forceinline__ void store_raw(bf16_t* p, const Raw8<bf16_t>& r) { *reinterpret_cast<uint4*>(p) = r.a; }
__device__ __forceinline__ void store_raw(float* p, const Raw8<float>& r) {
  *reinterpret_cast<float4*>(p) = r.a;
  *reinterpret_cast<float4*>(p + 4) = r.b;
}
__device__ __forceinline__ void unpack_raw(const Raw8<bf16_t>& r, float (&v)[8]) {
  v[0] = __uint_as_float(r.a.x << 16); v[1] = __uint_as_float(r.a.x & 0xffff0000u);
  v[2] = __uint_as_float(r.a.y << 16); v[3] = __uint_as_float(r.a.y & 0xffff0000u);
  v[4] = __uint_as_float(r.a.z << 16); v[5] = __uint_as_float(r.a.z & 0xffff0000u);
  v[6] = __uint_as_float(r.a.w << 16); v[7] = __uint_as_float(r.a.w & 0xffff0000u);
}
__device__ __forceinline__ void unpack_raw(const Raw8<float>& r, float (&v)[8]) {
  v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w;
  v[4] = r.b.x; v[5] = r.b.y; v[6] = r.b.z; v[7] = r.b.w;
}

// KEEP: also writes the rows as they came to keep.x, and keep.n integers from keep.n_in to keep.n_out (a stage stashes its input
// and the key lengths: with copy launches and a memcpy of their own, here and for the output gradient, three batches of 4
// microbatches took 2387 us instead of 2157 in a 2-layer fp32 stage of 128 tokens, h=128, and 1.5 % longer in a bf16 layer of 4096
// tokens, h=1024)
template <typename T, int R, int CPT, bool KEEP>
__global__ __launch_bounds__(kWg) void ln_fwd_kernel(const T* __restrict__ x, const T* __restrict__ gain,
                                                      const T* __restrict__ shift, T* __restrict__ y,
                                                      float* __restrict__ mean_out, float* __restrict__ rstd_out,
                                                      int rows, int h, float eps, LnKeep keep) {
  constexpr int ROWS = kWg / R;
  __shared__ float red[4];
  const int tid = threadIdx.x;
  const int sub = tid % R;
  const int row = blockIdx.x * ROWS + tid / R;
  const bool row_ok = row < rows;
  if (KEEP && blockIdx.x == 0)
    for (int i = tid; i < keep.n; i += kWg) keep.n_out[i] = keep.n_in[i];
  float v[CPT][8];
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int col = (sub + c * R) * 8;
    if (row_ok && col < h) {
      if (KEEP) {
        Raw8<T> raw;
        load_raw(x + (int64_t)row * h + col, raw);
        store_raw(static_cast<T*>(keep.x) + (int64_t)row * h + col, raw);
        unpack_raw(raw, v[c]);
      } else {
        load8(x + (int64_t)row * h + col, v[c]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) s += v[c][i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[c][i] = 0.f;
    }
  }
  const float mean = group_sum<R>(s, red, tid) / (float)h;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int col = (sub + c * R) * 8;
    if (col < h) {
#pragma unroll
      for (int i = 0; i < 8; ++i) { const float d = v[c][i] - mean; q += d * d; }
    }
  }
  const float var = group_sum<R>(q, red, tid) / (float)h;
  const float rstd = 1.0f / sqrtf(var + eps);
  if (!row_ok) return;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int col = (sub + c * R) * 8;
    if (col < h) {
      float g[8], b[8], o[8];
      load8(gain + col, g);
      load8(shift + col, b);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = g[i] * ((v[c][i] - mean) * rstd) + b[i];
      store8(y + (int64_t)row * h + col, o);
    }
  }
  if (sub == 0) { mean_out[row] = mean; rstd_out[row] = rstd; }
}

// The end of a backward workgroup: the column sums of its ROWS sub-rows (R threads each, chunks of 8 columns at (sub + c * R) * 8) added in
// the order of the rows and stored to row = [3][h].  The matrices go through LDS as 16-byte pieces [which][CPT][2][thread] and every thread
// takes its share of the adding and storing; all three at once, unless two workgroups would no longer fit into a CU's LDS.
// (One matrix after the other, added and stored by the threads of the first sub-row alone: bf16 4096 x 1024 12.0 -> 11.3 us, 1024 x 512 4.9 -> 4.6,
// fp32 1428 x 1920 14.2 -> 12.9, 476 x 1920 8.6 -> 7.6; rows of 2048 columns and more, 4096 x 2560 21.4, are level.  All three at once for
// fp32 1428 x 1920, one workgroup per CU, 16.9.)
// IN_LDS: the third matrix is there already.
constexpr int row_sums_at_once(int cpt) { return cpt < 4 ? 3 : 1; }
template <int R, int ROWS, int CPT, bool IN_LDS = false>
__device__ __forceinline__ void store_row_sums(float4* sums, const float (&gsum)[CPT][8], const float (&bsum)[CPT][8],
                                               const float (&osum)[CPT][8], float* __restrict__ row, int h) {
  constexpr int kThreads = R * ROWS;
  const int tid = threadIdx.x;
  if constexpr (ROWS == 1) {
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int col = (tid + c * R) * 8;
      if (col < h) {
        store8(row + col, gsum[c]);
        store8(row + h + col, bsum[c]);
        store8(row + 2 * h + col, osum[c]);
      }
    }
  } else {
    constexpr int kTurn = row_sums_at_once(CPT), kPieces = kTurn * CPT * 2 * R;   // pieces of a turn, in the order of their addresses within a matrix
    static_assert(!IN_LDS || kTurn == 3, "the third matrix lies behind the first two");
#pragma unroll
    for (int w0 = 0; w0 < 3; w0 += kTurn) {
      if (w0 > 0) __syncthreads();   // the last turn's pieces are read
#pragma unroll
      for (int w = 0; w < kTurn; ++w) {
        if (IN_LDS && w == 2) break;
        const float (&v)[CPT][8] = w0 + w == 0 ? gsum : w0 + w == 1 ? bsum : osum;
#pragma unroll
        for (int c = 0; c < CPT; ++c)
#pragma unroll
          for (int q = 0; q < 2; ++q)
            sums[((w * CPT + c) * 2 + q) * kThreads + tid] = make_float4(v[c][4 * q], v[c][4 * q + 1], v[c][4 * q + 2], v[c][4 * q + 3]);
      }
      __syncthreads();
#pragma unroll
      for (int k0 = 0; k0 < kPieces; k0 += kThreads) {
        const int k = k0 + tid;
        if (kPieces % kThreads != 0 && k >= kPieces) break;
        const int q = k & 1, sub = (k >> 1) % R, wc = (k >> 1) / R, col = (sub + (wc % CPT) * R) * 8 + 4 * q;
        if (col >= h) continue;
        const float4* at = sums + (wc * 2 + q) * kThreads + sub;
        float4 t = at[0];
#pragma unroll
        for (int rr = 1; rr < ROWS; ++rr) { const float4 v = at[rr * R]; t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w; }
        *reinterpret_cast<float4*>(row + (w0 + wc / CPT) * h + col) = t;
      }
    }
  }
}

// Backward.  Workgroups stride over row groups and keep per-column sums of dy*xhat, dy and of the
// result dx in registers; each workgroup writes one row of partial[parts][3h] (dy*xhat | dy | dx).
// The third block is the bias gradient of the projection that produced this kernel's residual
// operand (its output gradient is exactly dx), so no separate pass over dx is needed for it.
// KEEP: also writes the rows of dres as they came to dres_keep (see the forward kernel).
template <typename T, int CPT, bool KEEP>
__global__ __launch_bounds__(kWg) void ln_bwd_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                      const float* __restrict__ mean_in, const float* __restrict__ rstd_in,
                                                      const T* __restrict__ gain, const T* __restrict__ dres,
                                                      T* __restrict__ dx, float* __restrict__ partial, int rows, int h, T* __restrict__ dres_keep) {
  constexpr int R = 64, ROWS = kWg / R;   // a wave to a row
  __shared__ float4 sums[row_sums_at_once(CPT) * 2 * CPT * kWg];
  const int tid = threadIdx.x;
  const int sub = tid % R, rsub = tid / R;
  float gsum[CPT][8], bsum[CPT][8], osum[CPT][8], gn[CPT][8];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int col = (sub + c * R) * 8;
    if (col < h) load8(gain + col, gn[c]);
#pragma unroll
    for (int i = 0; i < 8; ++i) { gsum[c][i] = 0.f; bsum[c][i] = 0.f; osum[c][i] = 0.f; if (col >= h) gn[c][i] = 0.f; }
  }
  // Two row groups per trip, all loads of both issued before any arithmetic: the kernel is bound
  // by memory latency, not bandwidth, at the sizes a stage gives it.
  constexpr int U = CPT <= 2 ? 2 : 1;   // (longer rows already keep enough loads in flight, and registers are short)
  const int n_groups = (rows + ROWS - 1) / ROWS;
  for (int grp0 = blockIdx.x; grp0 < n_groups; grp0 += U * gridDim.x) {
    int row[U];
    bool row_ok[U];
    float mean[U], rstd[U];
    float xh[U][CPT][8], dxh[U][CPT][8], res[U][CPT][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int grp = grp0 + u * gridDim.x;
      row[u] = grp * ROWS + rsub;
      row_ok[u] = grp < n_groups && row[u] < rows;
      mean[u] = row_ok[u] ? mean_in[row[u]] : 0.f;
      rstd[u] = row_ok[u] ? rstd_in[row[u]] : 0.f;
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int col = (sub + c * R) * 8;
        if (row_ok[u] && col < h) {
          load8(x + (int64_t)row[u] * h + col, xh[u][c]);
          load8(dy + (int64_t)row[u] * h + col, dxh[u][c]);
          if (KEEP) {
            Raw8<T> raw;
            load_raw(dres + (int64_t)row[u] * h + col, raw);
            store_raw(dres_keep + (int64_t)row[u] * h + col, raw);
            unpack_raw(raw, res[u][c]);
          } else if (dres) {
            load8(dres + (int64_t)row[u] * h + col, res[u][c]);
          }
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) { xh[u][c][i] = 0.f; dxh[u][c][i] = 0.f; }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int col = (sub + c * R) * 8;
        if (row_ok[u] && col < h) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float dv = dxh[u][c][i];
            xh[u][c][i] = (xh[u][c][i] - mean[u]) * rstd[u];
            dxh[u][c][i] = dv * gn[c][i];
            s1 += dxh[u][c][i];
            s2 += dxh[u][c][i] * xh[u][c][i];
            gsum[c][i] += dv * xh[u][c][i];
            bsum[c][i] += dv;
          }
        }
      }
      const float c1 = wave_sum(s1) / (float)h;
      const float c2 = wave_sum(s2) / (float)h;
      if (row_ok[u]) {
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          const int col = (sub + c * R) * 8;
          if (col < h) {
            float o[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = rstd[u] * (dxh[u][c][i] - c1 - xh[u][c][i] * c2);
            if (dres) {
#pragma unroll
              for (int i = 0; i < 8; ++i) o[i] += res[u][c][i];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) osum[c][i] += o[i];
            store8(dx + (int64_t)row[u] * h + col, o);
          }
        }
      }
    }
  }
  // one partial row per workgroup: the sums of its ROWS sub-rows
  store_row_sums<R, ROWS, CPT>(sums, gsum, bsum, osum, partial + (int64_t)blockIdx.x * 3 * h, h);
}

// Backward for long rows (h >= 2048).  With 256 threads the per-column sums of a row of 8192 take 96
// registers per thread next to the row itself, one wave per SIMD fits, and a CU has too few loads in
// flight to keep HBM busy.  Here a workgroup has 768 to 1024 threads, R = 256 to 1024 of them share a row
// with one or two 16-byte chunks each, so the sums are 24 or 48 registers and twelve to sixteen waves stay
// resident per CU.  A workgroup is alone on its CU, so nothing else hides its trips to HBM: the U rows per thread
// of the next step are requested (and held as loaded, 16 bytes per chunk) before the arithmetic of the
// current step starts, and the row sums of all U rows share one barrier (the exchange buffer alternates
// between steps, so a wave that runs ahead cannot overwrite sums that a slower one still reads).
// Same partial-row layout as the kernel above; the grid is one workgroup per CU at most.
template <typename T, int R, int ROWS, int CPT, int U, bool KEEP>
__global__ __launch_bounds__(R* ROWS) void ln_bwd_wide_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                              const float* __restrict__ mean_in,
                                                              const float* __restrict__ rstd_in, const T* __restrict__ gain,
                                                              const T* __restrict__ dres, T* __restrict__ dx,
                                                              float* __restrict__ partial, int rows, int h, T* __restrict__ dres_keep) {
  constexpr int kThreads = R * ROWS;
  constexpr int W = R / 64;   // waves per row
  // Requesting a step ahead costs 12 registers per chunk next to the 24 of the column sums; the budget of a
  // workgroup of more than 768 threads is 128, so it is done for 2-byte elements with one chunk per thread; with one chunk
  // per thread the sums of the results live in LDS (one 16-byte slot per thread and column quad, touched by
  // its owner only).
  constexpr bool kAhead = sizeof(T) == 2 && CPT == 1;
  constexpr bool kLdsSums = CPT == 1;
  __shared__ float red[2][2 * U][16];
  __shared__ float4 sums[ROWS > 1 ? 6 * kThreads : kLdsSums ? 2 * kThreads : 1];   // of gain, shift and results, [3][2][thread]; with one row the last only
  float4* osum_lds = sums + (ROWS > 1 ? 4 * kThreads : 0);
  static_assert(ROWS == 1 || kLdsSums, "store_row_sums takes the sums of the results from LDS");
  const int tid = threadIdx.x;
  const int sub = tid % R, rsub = tid / R;
  const int wave = tid >> 6, first_wave = (wave / W) * W;
  float gsum[CPT][8], bsum[CPT][8], osum[CPT][8], gn[CPT][8];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int col = (sub + c * R) * 8;
    if (col < h) load8(gain + col, gn[c]);
#pragma unroll
    for (int i = 0; i < 8; ++i) { gsum[c][i] = 0.f; bsum[c][i] = 0.f; osum[c][i] = 0.f; if (col >= h) gn[c][i] = 0.f; }
  }
  const int n_groups = (rows + ROWS - 1) / ROWS;
  const int stride = U * gridDim.x;
  // the rows of the step after the one being worked on, as loaded
  Raw8<T> nx[U][CPT], ndy[U][CPT], nres[U][CPT];
  float nmean[U], nrstd[U];
  auto fetch = [&](int grp0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int grp = grp0 + u * gridDim.x;
      const int row = grp * ROWS + rsub;
      const bool ok = grp < n_groups && row < rows;
      nmean[u] = ok ? mean_in[row] : 0.f;
      nrstd[u] = ok ? rstd_in[row] : 0.f;
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int col = (sub + c * R) * 8;
        if (ok && col < h) {
          load_raw(x + (int64_t)row * h + col, nx[u][c]);
          load_raw(dy + (int64_t)row * h + col, ndy[u][c]);
          if (dres) load_raw(dres + (int64_t)row * h + col, nres[u][c]);
          else nres[u][c] = Raw8<T>{};
        } else {
          nx[u][c] = Raw8<T>{}; ndy[u][c] = Raw8<T>{}; nres[u][c] = Raw8<T>{};
        }
      }
    }
  };
  if (kLdsSums) {
    osum_lds[tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    osum_lds[kThreads + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (kAhead && (int)blockIdx.x < n_groups) fetch(blockIdx.x);
  int parity = 0;
  for (int grp0 = blockIdx.x; grp0 < n_groups; grp0 += stride) {
    if (!kAhead) fetch(grp0);
    int row[U];
    bool row_ok[U];
    float mean[U], rstd[U];
    float xh[U][CPT][8], dxh[U][CPT][8];
    Raw8<T> res[U][CPT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int grp = grp0 + u * gridDim.x;
      row[u] = grp * ROWS + rsub;
      row_ok[u] = grp < n_groups && row[u] < rows;
      mean[u] = nmean[u];
      rstd[u] = nrstd[u];
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int col = (sub + c * R) * 8;
        if (row_ok[u] && col < h) {
          unpack_raw(nx[u][c], xh[u][c]);
          unpack_raw(ndy[u][c], dxh[u][c]);
          res[u][c] = nres[u][c];
          if (KEEP) store_raw(dres_keep + (int64_t)row[u] * h + col, res[u][c]);
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) { xh[u][c][i] = 0.f; dxh[u][c][i] = 0.f; }
        }
      }
    }
    if (kAhead && grp0 + stride < n_groups) fetch(grp0 + stride);
    float s1[U], s2[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s1[u] = 0.f; s2[u] = 0.f;
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int col = (sub + c * R) * 8;
        if (row_ok[u] && col < h) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float dv = dxh[u][c][i];
            xh[u][c][i] = (xh[u][c][i] - mean[u]) * rstd[u];
            dxh[u][c][i] = dv * gn[c][i];
            s1[u] += dxh[u][c][i];
            s2[u] += dxh[u][c][i] * xh[u][c][i];
            gsum[c][i] += dv * xh[u][c][i];
            bsum[c][i] += dv;
          }
        }
      }
      s1[u] = wave_sum(s1[u]);
      s2[u] = wave_sum(s2[u]);
    }
    if ((tid & 63) == 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) { red[parity][2 * u][wave] = s1[u]; red[parity][2 * u + 1][wave] = s2[u]; }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float a = 0.f, b = 0.f;
#pragma unroll
      for (int i = 0; i < W; ++i) { a += red[parity][2 * u][first_wave + i]; b += red[parity][2 * u + 1][first_wave + i]; }
      const float c1 = a / (float)h, c2 = b / (float)h;
      if (row_ok[u]) {
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          const int col = (sub + c * R) * 8;
          if (col < h) {
            float o[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = rstd[u] * (dxh[u][c][i] - c1 - xh[u][c][i] * c2);
            if (dres) {
              float rv[8];
              unpack_raw(res[u][c], rv);
#pragma unroll
              for (int i = 0; i < 8; ++i) o[i] += rv[i];
            }
            if (kLdsSums) {
              float4 lo = osum_lds[tid], hi = osum_lds[kThreads + tid];
              lo.x += o[0]; lo.y += o[1]; lo.z += o[2]; lo.w += o[3];
              hi.x += o[4]; hi.y += o[5]; hi.z += o[6]; hi.w += o[7];
              osum_lds[tid] = lo; osum_lds[kThreads + tid] = hi;
            } else {
#pragma unroll
              for (int i = 0; i < 8; ++i) osum[c][i] += o[i];
            }
            store8(dx + (int64_t)row[u] * h + col, o);
          }
        }
      }
    }
    parity ^= 1;
  }
  float* row = partial + (int64_t)blockIdx.x * 3 * h;
  if constexpr (ROWS > 1) {
    store_row_sums<R, ROWS, CPT, true>(sums, gsum, bsum, osum, row, h);
  } else {
    if (kLdsSums) {
      const float4 lo = osum_lds[tid], hi = osum_lds[kThreads + tid];
      osum[0][0] = lo.x; osum[0][1] = lo.y; osum[0][2] = lo.z; osum[0][3] = lo.w;
      osum[0][4] = hi.x; osum[0][5] = hi.y; osum[0][6] = hi.z; osum[0][7] = hi.w;
    }
    store_row_sums<R, 1, CPT>(sums, gsum, bsum, osum, row, h);
  }
}

template <typename T>
__global__ __launch_bounds__(kWg) void colsum_partial_kernel(const T* __restrict__ y, int rows, int n, int ld,
                                                              float* __restrict__ partial, int rows_per_part) {
  __shared__ float comb[7][8][32];
  const int tid = threadIdx.x;
  const int cc = tid % 32, rl = tid / 32;      // column chunk, row lane
  const int col = (blockIdx.x * 32 + cc) * 8;
  const int r0 = blockIdx.y * rows_per_part;
  const int r1 = min(rows, r0 + rows_per_part);
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (col < n) {
    for (int r = r0 + rl; r < r1; r += 8) {
      float v[8];
      load8(y + (int64_t)r * ld + col, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) s[i] += v[i];
    }
  }
  if (rl > 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) comb[rl - 1][i][cc] = s[i];
  }
  __syncthreads();
  if (rl == 0 && col < n) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int rr = 0; rr < 7; ++rr) s[i] += comb[rr][i][cc];
    store8(partial + (int64_t)blockIdx.y * n + col, s);
  }
}

// Column sums of 32 columns over all rows by one workgroup of 512 threads (4 threads to a row, 8 columns each), four rows of a
// thread in flight at a time.  ACC: added to what is there, which is asked for ahead of the rows (0.5 to 1 % of calls of 2 to 3 us; behind a
// condition on an argument it cost those that overwrite 1.4 %, 2.0 -> 2.07 us).
template <typename T, bool ACC>
__global__ __launch_bounds__(512) void colsum_direct_kernel(const T* __restrict__ y, int rows, int n, float* __restrict__ out) {
  __shared__ float part[128][33], part2[16][32];
  const int tid = threadIdx.x, cc = tid & 3, rl = tid >> 2;
  const int col = blockIdx.x * 32 + cc * 8;
  const int oc = blockIdx.x * 32 + tid;
  float before = 0.f;
  if (ACC && tid < 32 && oc < n) before = out[oc];
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (col < n) {
    int r = rl;
    for (; r + 3 * 128 < rows; r += 4 * 128) {
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) load8(y + (int64_t)(r + u * 128) * n + col, v[u]);
#pragma unroll
      for (int i = 0; i < 8; ++i) s[i] += (v[0][i] + v[2][i]) + (v[1][i] + v[3][i]);
    }
    for (; r < rows; r += 128) {
      float v[8];
      load8(y + (int64_t)r * n + col, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) s[i] += v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) part[rl][cc * 8 + i] = s[i];
  __syncthreads();
  // the 128 partial sums of a column as a tree: 7 roundings deep (one after the other, eight and then sixteen, they left 6 % more
  // error in fp32 than the two-launch form)
  const int c = tid & 31, g = tid >> 5;
  float t[16];
#pragma unroll
  for (int k = 0; k < 8; ++k) t[k] = part[g * 8 + k][c];
#pragma unroll
  for (int w = 4; w > 0; w /= 2)
#pragma unroll
    for (int k = 0; k < w; ++k) t[k] += t[k + w];
  part2[g][c] = t[0];
  __syncthreads();
  if (tid < 32 && oc < n) {
#pragma unroll
    for (int k = 0; k < 16; ++k) t[k] = part2[k][tid];
#pragma unroll
    for (int w = 8; w > 0; w /= 2)
#pragma unroll
      for (int k = 0; k < w; ++k) t[k] += t[k + w];
    out[oc] = ACC ? before + t[0] : t[0];
  }
}

__device__ __forceinline__ void plus(float& a, float b) { a += b; }
__device__ __forceinline__ void plus(float4& a, const float4& b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; }
// Sum of N numbers (a power of two) as a tree: log2 N roundings deep
template <int N, typename T>
__device__ __forceinline__ T pairwise(T (&v)[N]) {
#pragma unroll
  for (int w = N / 2; w > 0; w /= 2)
#pragma unroll
    for (int i = 0; i < w; ++i) plus(v[i], v[i + w]);
  return v[0];
}

// s += rows p, p + 16, .. below `parts` (ld apart): 8, 4, 2 and 1 of them in flight at a time.  One after the other, the last seven
// cost as many trips to memory (119 rows of 3 x 1920 fp32 columns 6.0 -> 5.0 us); all of them at once behind conditions is code that every
// short call has to fetch (22 rows 3.7 -> 4.2).
template <int N, typename T>
__device__ __forceinline__ void add_rows(T& s, const float* __restrict__ at, int64_t step) {
  T v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = *reinterpret_cast<const T*>(at + i * step);
  plus(s, pairwise(v));
}
template <typename T>
__device__ __forceinline__ T sum_rows(const float* __restrict__ partial, int p, int parts, int64_t ld) {
  T s = T{};
  for (; p + 7 * 16 < parts; p += 8 * 16) add_rows<8>(s, partial + p * ld, 16 * ld);
  if (p + 3 * 16 < parts) { add_rows<4>(s, partial + p * ld, 16 * ld); p += 4 * 16; }
  if (p + 16 < parts) { add_rows<2>(s, partial + p * ld, 16 * ld); p += 2 * 16; }
  if (p < parts) add_rows<1>(s, partial + p * ld, 16 * ld);
  return s;
}

// 16 columns x 16 part-lanes per workgroup: 64-byte segments per part row, then an LDS tree over the part-lanes.
__global__ __launch_bounds__(kWg) void colsum_finalize_kernel(const float* __restrict__ partial, int parts, int n,
                                                               int ld, float* __restrict__ out, int accumulate) {
  __shared__ float red[16][17];
  const int c = threadIdx.x & 15, pl = threadIdx.x >> 4;
  const int col = blockIdx.x * 16 + c;
  red[pl][c] = col < n ? sum_rows<float>(partial + col, pl, parts, ld) : 0.f;
  __syncthreads();
  if (pl == 0 && col < n) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = red[i][c];
    const float t = pairwise(v);
    out[col] = accumulate ? out[col] + t : t;
  }
}

// Column sums of up to 4 matrices with the same row count in one launch: blockIdx.x walks the
// 256-column blocks of all segments, blockIdx.y the row slabs.  partial is [parts][total_cols]:
// segment s owns columns [col0_s, col0_s + n_s).
template <typename T>
__global__ __launch_bounds__(kWg) void colsum_partial_grouped_kernel(ColsumGroup g) {
  __shared__ float comb[7][8][32];
  int sidx = 0;
#pragma unroll
  for (int q = 1; q < 4; ++q)
    if (q < g.count && (int)blockIdx.x >= g.block0[q]) sidx = q;
  const T* y = static_cast<const T*>(g.y[sidx]);
  const int n = g.n[sidx], ld = g.ld[sidx];
  const int tid = threadIdx.x;
  const int cc = tid % 32, rl = tid / 32;
  const int col = ((blockIdx.x - g.block0[sidx]) * 32 + cc) * 8;
  const int r0 = blockIdx.y * g.rows_per_part;
  const int r1 = min(g.rows, r0 + g.rows_per_part);
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (col < n) {
    for (int r = r0 + rl; r < r1; r += 8) {
      float v[8];
      load8(y + (int64_t)r * ld + col, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) s[i] += v[i];
    }
  }
  if (rl > 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) comb[rl - 1][i][cc] = s[i];
  }
  __syncthreads();
  if (rl == 0 && col < n) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int rr = 0; rr < 7; ++rr) s[i] += comb[rr][i][cc];
    store8(g.partial + (int64_t)blockIdx.y * g.total_cols + g.col0[sidx] + col, s);
  }
}

// out_s[n_s] (+)= sum over parts_s rows of partial_s, for up to kFinalizeMaxItems segments in one launch.
// A workgroup owns 64 columns: 16 threads x 16 bytes cover 256 contiguous bytes of a row (whole cache lines; with
// one float per thread a workgroup used half of every line it touched), 16 such groups walk the rows.  (32 columns and 32 groups, twice
// the workgroups: 256 rows x 19512 columns 6.7 -> 7.9 us; 64 columns and 32 groups 7.4.)
__global__ __launch_bounds__(kWg) void colsum_finalize_grouped_kernel(FinalizeGroup g) {
  __shared__ float4 red[16][17];
  int sidx = 0;
  for (int q = 1; q < g.count; ++q)
    if ((int)blockIdx.x >= g.block0[q]) sidx = q;
  const float* partial = g.partial[sidx];
  const int parts = g.parts[sidx], n = g.n[sidx], ld = g.ld[sidx];
  const int c = threadIdx.x & 15, pl = threadIdx.x >> 4;
  const int col = ((blockIdx.x - g.block0[sidx]) * 16 + c) * 4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (col < n) s = sum_rows<float4>(partial + col, pl, parts, ld);
  red[pl][c] = s;
  __syncthreads();
  if (pl == 0 && col < n) {
    float4 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = red[i][c];
    float4 t = pairwise(v);
    float4* out = reinterpret_cast<float4*>(g.out[sidx] + col);
    if (g.accumulate) plus(t, *out);   // (asked for ahead of the rows, its branch holds them up: 22 rows 3.5 -> 4.0 us)
    *out = t;
  }
}

// R, CPT for a row length: the fewest threads per row that keep CPT <= 4, else up to 8.
struct RowShape { int R, CPT; };
RowShape row_shape(int h) {
  const int chunks = h / 8;
  for (int R : {64, 128, 256}) {
    const int cpt = (chunks + R - 1) / R;
    if (cpt <= 4) return {R, cpt};
  }
  return {256, (chunks + 255) / 256};
}

#define LN_DISPATCH(KERNEL_CALL)                                             \
  switch (rs.R * 16 + rs.CPT) {                                              \
    case 64 * 16 + 1: KERNEL_CALL(64, 1); break;                             \
    case 64 * 16 + 2: KERNEL_CALL(64, 2); break;                             \
    case 64 * 16 + 3: KERNEL_CALL(64, 3); break;                             \
    case 64 * 16 + 4: KERNEL_CALL(64, 4); break;                             \
    case 128 * 16 + 3: KERNEL_CALL(128, 3); break;                           \
    case 128 * 16 + 4: KERNEL_CALL(128, 4); break;                           \
    case 256 * 16 + 3: KERNEL_CALL(256, 3); break;                           \
    case 256 * 16 + 4: KERNEL_CALL(256, 4); break;                           \
    case 256 * 16 + 5: KERNEL_CALL(256, 5); break;                           \
    case 256 * 16 + 6: KERNEL_CALL(256, 6); break;                           \
    case 256 * 16 + 7: KERNEL_CALL(256, 7); break;                           \
    case 256 * 16 + 8: KERNEL_CALL(256, 8); break;                           \
    default: return hipErrorInvalidValue;                                    \
  }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

hipError_t layernorm_fwd(const void* x, const void* gain, const void* shift, void* y, float* mean,
                         float* rstd, int rows, int h, float eps, int dtype, hipStream_t stream, const LnKeep* keep) {
  if (rows <= 0 || h <= 0 || h % 8 || h > 16384 || !x || !y || !gain || !shift || !mean || !rstd)
    return hipErrorInvalidValue;
  if (!aligned16(x) || !aligned16(y) || !aligned16(gain) || !aligned16(shift)) return hipErrorInvalidValue;
  if (keep && (!keep->x || !aligned16(keep->x))) return hipErrorInvalidValue;
  const LnKeep kp = keep ? *keep : LnKeep{};
  const RowShape rs = row_shape(h);
  const int grid = ceil_div(rows, kWg / rs.R);
#define CALL_FWD_AS(T_, R_, C_, K_)                                                                       \
  hipLaunchKernelGGL((ln_fwd_kernel<T_, R_, C_, K_>), dim3(grid), dim3(kWg), 0, stream,                   \
                     static_cast<const T_*>(x), static_cast<const T_*>(gain),                             \
                     static_cast<const T_*>(shift), static_cast<T_*>(y), mean, rstd, rows, h, eps, kp)
#define CALL_FWD(R_, C_)                                                                                  \
  if (dtype == kBF16 && keep) CALL_FWD_AS(bf16_t, R_, C_, true);                                          \
  else if (dtype == kBF16) CALL_FWD_AS(bf16_t, R_, C_, false);                                            \
  else if (keep) CALL_FWD_AS(float, R_, C_, true);                                                        \
  else CALL_FWD_AS(float, R_, C_, false)
  LN_DISPATCH(CALL_FWD)
#undef CALL_FWD
#undef CALL_FWD_AS
  return hipGetLastError();
}

int ln_bwd_max_parts() { return 512; }

hipError_t layernorm_bwd(const void* dy, const void* x, const float* mean, const float* rstd,
                         const void* gain, const void* dres, void* dx, float* partial, int* parts_out,
                         int rows, int h, int dtype, hipStream_t stream, void* dres_keep) {
  if (rows <= 0 || h <= 0 || h % 8 || h > 16384 || !dy || !x || !mean || !rstd || !gain || !dx || !partial ||
      !parts_out)
    return hipErrorInvalidValue;
  if (!aligned16(dy) || !aligned16(x) || !aligned16(dx) || !aligned16(gain) || !aligned16(partial) ||
      (dres && !aligned16(dres)) || (dres_keep && (!dres || !aligned16(dres_keep))))
    return hipErrorInvalidValue;
  if (h >= 2048) {
    // Long rows: one workgroup per CU at most (256 partial rows); threads per row, rows per workgroup and rows of a step per thread
    // by the length of a row.  What counts is the rows a CU has in flight.  With 512 threads to a row of 257 to 320 chunks three
    // to four of the eight waves have none of it and a workgroup takes two rows; 320 threads leave room for three (4096 x 2560 in
    // bf16 with its finalize launch 29.1 -> 26.4 us, 12000 rows 72.9 -> 59.6; 2056 columns 27.6 -> 24.7; 384 to 600 rows 0.83 to 0.95
    // of the time, 700 to 1024 rows 0.93 to 1.02, below 384 up to 1.09).  fp32 rows arrive in the step that uses them and gain nothing from a
    // third row beside the two (0.96 to 1.11); with 384 threads, twelve waves, the registers suffice for three rows per thread and
    // step instead: 0.86 to 1.00 of the time at every count of 257 to 384 chunks (4096 x 3072 53.1 -> 51.4 us, 1300 rows 25.6 -> 22.0).
    // That form is within 4 % on either side in bf16, and one row per workgroup on 640 or 768 threads with three per step is 2 to
    // 28 % behind 1024 threads with two at 513 to 768 chunks.
    const int chunks = h / 8;
#define CALL_WIDE_AS(T_, R_, N_, C_, U_, K_)                                                                 \
  hipLaunchKernelGGL((ln_bwd_wide_kernel<T_, R_, N_, C_, U_, K_>), dim3(grid), dim3(R_ * N_), 0, stream,     \
                     static_cast<const T_*>(dy), static_cast<const T_*>(x), mean, rstd,                      \
                     static_cast<const T_*>(gain), static_cast<const T_*>(dres), static_cast<T_*>(dx),       \
                     partial, rows, h, static_cast<T_*>(dres_keep))
#define CALL_WIDE(T_, R_, N_, C_, U_)                                                                        \
  do {                                                                                                       \
    const int groups = ceil_div(rows, N_);                                                                   \
    grid = groups < 256 ? groups : 256;                                                                      \
    if (dres_keep) CALL_WIDE_AS(T_, R_, N_, C_, U_, true);                                                   \
    else CALL_WIDE_AS(T_, R_, N_, C_, U_, false);                                                            \
  } while (0)
    int grid = 0;
    if (dtype == kBF16) {
      if (chunks <= 256) CALL_WIDE(bf16_t, 256, 4, 1, 2);
      else if (chunks <= 320 && rows >= 384) CALL_WIDE(bf16_t, 320, 3, 1, 2);
      else if (chunks <= 512) CALL_WIDE(bf16_t, 512, 2, 1, 2);
      else if (chunks <= 1024) CALL_WIDE(bf16_t, 1024, 1, 1, 2);
      else CALL_WIDE(bf16_t, 1024, 1, 2, 1);
    } else {
      if (chunks <= 256) CALL_WIDE(float, 256, 4, 1, 2);
      else if (chunks <= 384) CALL_WIDE(float, 384, 2, 1, 3);
      else if (chunks <= 512) CALL_WIDE(float, 512, 2, 1, 2);
      else if (chunks <= 1024) CALL_WIDE(float, 1024, 1, 1, 2);
      else CALL_WIDE(float, 1024, 1, 2, 1);
    }
#undef CALL_WIDE
#undef CALL_WIDE_AS
    *parts_out = grid;
    return hipGetLastError();
  }
  const int cpt = ceil_div(h, 64 * 8);   // 1 to 4
  const int groups = ceil_div(rows, kWg / 64);   // rows of a workgroup: one per wave
  const int grid = groups < ln_bwd_max_parts() ? groups : ln_bwd_max_parts();
#define CALL_BWD_AS(T_, C_, K_)                                                                         \
  hipLaunchKernelGGL((ln_bwd_kernel<T_, C_, K_>), dim3(grid), dim3(kWg), 0, stream,                     \
                     static_cast<const T_*>(dy), static_cast<const T_*>(x), mean, rstd,                     \
                     static_cast<const T_*>(gain), static_cast<const T_*>(dres), static_cast<T_*>(dx),      \
                     partial, rows, h, static_cast<T_*>(dres_keep))
#define CALL_BWD(C_)                                                                                    \
  if (dtype == kBF16 && dres_keep) CALL_BWD_AS(bf16_t, C_, true);                                       \
  else if (dtype == kBF16) CALL_BWD_AS(bf16_t, C_, false);                                              \
  else if (dres_keep) CALL_BWD_AS(float, C_, true);                                                     \
  else CALL_BWD_AS(float, C_, false)
  switch (cpt) {
    case 1: CALL_BWD(1); break;
    case 2: CALL_BWD(2); break;
    case 3: CALL_BWD(3); break;
    default: CALL_BWD(4); break;
  }
#undef CALL_BWD
#undef CALL_BWD_AS
  *parts_out = grid;
  return hipGetLastError();
}

int colsum_max_parts() { return 64; }

hipError_t colsum_partial(const void* y, int rows, int n, int ldy, float* partial, int* parts_out, int dtype,
                          hipStream_t stream) {
  if (rows <= 0 || n <= 0 || n % 8 || ldy % 8 || ldy < n || !y || !partial || !parts_out) return hipErrorInvalidValue;
  if (!aligned16(y) || !aligned16(partial)) return hipErrorInvalidValue;
  int parts = ceil_div(rows, 64);
  if (parts > colsum_max_parts()) parts = colsum_max_parts();
  const int rows_per_part = ceil_div(rows, parts);
  parts = ceil_div(rows, rows_per_part);
  dim3 grid(ceil_div(n, 256), parts);
  if (dtype == kBF16)
    hipLaunchKernelGGL((colsum_partial_kernel<bf16_t>), grid, dim3(kWg), 0, stream, static_cast<const bf16_t*>(y),
                       rows, n, ldy, partial, rows_per_part);
  else
    hipLaunchKernelGGL((colsum_partial_kernel<float>), grid, dim3(kWg), 0, stream, static_cast<const float*>(y),
                       rows, n, ldy, partial, rows_per_part);
  *parts_out = parts;
  return hipGetLastError();
}

// Column sums in one launch where a workgroup of 32 columns can take all rows: two launches of a small matrix cost more in
// fixed parts than the sums themselves.  A workgroup reads 64 (bf16) or 128 bytes of each row, so it stays ahead while the caches
// serve the other half of a line: up to 16 MiB, 14 where the rows do not start on lines of 128 bytes; fp32 rows that do are read in
// whole lines and have no such limit.  Two launches | one, us: bf16 128 x 3072 6.2 | 3.8, 1024 x 8192 (16 MiB) 5.8 | 3.3, 768 x 12288
// 5.8 | 7.2, 256 x 32768 (16 MiB) 6.3 | 3.8, 384 x 32768 6.4 | 9.1, 520 x 13912 (13.8) 6.5 | 6.3, 640 x 13912 (17) 7.1 | 8.4, 1000 x 22184
// 12 | 18; fp32 1024 x 4104 (16) 6.6 | 3.9, 1500 x 4104 (23.5) 7.2 | 8.1, 640 x 28256 13.9 | 11.4, 640 x 28232 (off the lines) 15.1 | 18.5.
// By rows: bf16 2048 x 512 6.1 | 4.2, 2000 x 3000 7.6 | 7.3, 4096 x 1024 6.4 | 10.1, 4096 x 8192 15.5 | 20.7; fp32 2000 x 3000 8.3 | 8.5.
hipError_t column_sums(const void* y, int rows, int n, float* partial, float* out, bool accumulate, int dtype, hipStream_t stream) {
  if (rows <= 0 || n <= 0 || n % 8 || !y || !partial || !out || !aligned16(y) || !aligned16(partial)) return hipErrorInvalidValue;
  const int64_t row_bytes = (int64_t)n * (dtype == kBF16 ? 2 : 4);
  const bool on_lines = row_bytes % 128 == 0;
  if ((rows <= 1024 || (rows <= 2048 && n <= 4096)) && ((on_lines && dtype == kF32) || rows * row_bytes <= (on_lines ? 16ll : 14ll) << 20)) {
    auto launch = [&](auto kernel, auto* rows_of) { hipLaunchKernelGGL(kernel, dim3(ceil_div(n, 32)), dim3(512), 0, stream, rows_of, rows, n, out); };
    const bf16_t* y16 = static_cast<const bf16_t*>(y);
    const float* y32 = static_cast<const float*>(y);
    if (dtype == kBF16) accumulate ? launch(colsum_direct_kernel<bf16_t, true>, y16) : launch(colsum_direct_kernel<bf16_t, false>, y16);
    else accumulate ? launch(colsum_direct_kernel<float, true>, y32) : launch(colsum_direct_kernel<float, false>, y32);
    return hipGetLastError();
  }
  int parts = 0;
  hipError_t e = colsum_partial(y, rows, n, n, partial, &parts, dtype, stream);
  return e != hipSuccess ? e : colsum_finalize(partial, parts, n, out, accumulate, stream);
}

hipError_t colsum_finalize(const float* partial, int parts, int n, float* out, bool accumulate,
                           hipStream_t stream) {
  if (parts <= 0 || n <= 0 || !partial || !out) return hipErrorInvalidValue;
  hipLaunchKernelGGL(colsum_finalize_kernel, dim3(ceil_div(n, 16)), dim3(kWg), 0, stream, partial, parts, n, n, out,
                     accumulate ? 1 : 0);
  return hipGetLastError();
}

hipError_t colsum_partial_grouped(const ColsumItem* items, int count, int rows, float* partial, int* parts_out,
                                  int* total_cols_out, int dtype, hipStream_t stream) {
  if (!items || count < 1 || count > 4 || rows <= 0 || !partial || !parts_out || !total_cols_out || !aligned16(partial))
    return hipErrorInvalidValue;
  ColsumGroup g{};
  g.count = count;
  int blocks = 0, cols = 0;
  for (int i = 0; i < count; ++i) {
    const ColsumItem& it = items[i];
    if (!it.y || it.n <= 0 || it.n % 8 || it.ld % 8 || it.ld < it.n || !aligned16(it.y)) return hipErrorInvalidValue;
    g.y[i] = it.y; g.n[i] = it.n; g.ld[i] = it.ld; g.block0[i] = blocks; g.col0[i] = cols;
    blocks += ceil_div(it.n, 256);
    cols += it.n;
  }
  int parts = ceil_div(rows, 64);
  if (parts > colsum_max_parts()) parts = colsum_max_parts();
  g.rows = rows;
  g.rows_per_part = ceil_div(rows, parts);
  parts = ceil_div(rows, g.rows_per_part);
  g.total_cols = cols;
  g.partial = partial;
  dim3 grid(blocks, parts);
  if (dtype == kBF16)
    hipLaunchKernelGGL((colsum_partial_grouped_kernel<bf16_t>), grid, dim3(kWg), 0, stream, g);
  else
    hipLaunchKernelGGL((colsum_partial_grouped_kernel<float>), grid, dim3(kWg), 0, stream, g);
  *parts_out = parts;
  *total_cols_out = cols;
  return hipGetLastError();
}

hipError_t colsum_finalize_grouped(const FinalizeItem* items, int count, bool accumulate, hipStream_t stream) {
  if (!items || count < 1 || count > kFinalizeMaxItems) return hipErrorInvalidValue;
  FinalizeGroup g{};
  g.count = count;
  g.accumulate = accumulate ? 1 : 0;
  int blocks = 0;
  for (int i = 0; i < count; ++i) {
    const FinalizeItem& it = items[i];
    if (!it.partial || !it.out || it.parts <= 0 || it.n <= 0 || it.ld < it.n) return hipErrorInvalidValue;
    if (it.n % 4 || it.ld % 4 || !aligned16(it.partial) || !aligned16(it.out)) return hipErrorInvalidValue;   // 16-byte accesses
    g.partial[i] = it.partial; g.parts[i] = it.parts; g.n[i] = it.n; g.ld[i] = it.ld; g.out[i] = it.out;
    g.block0[i] = blocks;
    blocks += ceil_div(it.n, 64);
  }
  hipLaunchKernelGGL(colsum_finalize_grouped_kernel, dim3(blocks), dim3(kWg), 0, stream, g);
  return hipGetLastError();
}

}  // namespace k2bw
