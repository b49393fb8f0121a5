// Launch shape of the bf16 attention kernels (attention_mfma.hpp).
#include "kernels.hpp"

namespace k2bw {

hipError_t attention_fwd_mfma_8x1(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st);
hipError_t attention_bwd_mfma_8x1(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                                  float* delta, hipStream_t st);
hipError_t attention_fwd_mfma_8x2(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st);
hipError_t attention_bwd_mfma_8x2(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                                  float* delta, hipStream_t st);
hipError_t attention_fwd_mfma_4x2(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st);
hipError_t attention_bwd_mfma_4x2(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                                  float* delta, hipStream_t st);

// How many rows a workgroup owns, and how often the rows it streams are split between its waves (see the three kernels):
//   8 x 1  256 rows: each streamed tile and barrier is shared among the most rows
//   8 x 2  128 rows, two halves of 4 waves
//   4 x 2   64 rows, two halves of 2 waves
// The smaller ones are two and four times as many workgroups with half the steps each.  Forward | backward in us, 8 x 1, 8 x 2,
// 4 x 2; W: workgroups of 128 rows, on 256 CUs that hold one workgroup of 8 waves each:
//   b=1 s=1024 a=8  dh=64          W 64    23.8 | 59.6   14.8 | 34.8   11.4 | 28.2
//   b=2 s=512  a=16 dh=64 padding    128   14.3 | 41.8   10.0 | 27.2    8.1 | 23.8
//   b=3 s=512  a=16 dh=64 padding    192   14.6 | 42.8   10.2 | 29.3   11.0 | 31.0
//   b=2 s=1024 a=16 dh=64            256   25.6 | 62.4   16.3 | 42.9   17.4 | 45.7
//   b=5 s=512  a=16 dh=64 padding    320   16.2 | 46.0   17.0 | 54.6   17.5 | 48.2
//   b=3 s=1024 a=16 dh=128 causal    384   35.8 | 101    27.6 | 92.5   36.1 | 130
//   b=4 s=1024 a=16 dh=64 causal     512   26.4 | 64.1   19.8 | 54.7   21.3 | 57.0
//   b=4 s=1024 a=16 dh=128 causal    512   36.9 | 103    32.3 | 114    47.8 | 168
//   b=8 s=368  a=16 dh=64 causal     384        | 36.9        | 43.1        | 40.5
//   b=31 s=444 a=4  dh=80 causal     496   19.0          22.6
//   b=12 s=152 a=12 dh=80 causal     288    9.4 | 29.3   12.9 | 39.0   11.1 | 37.1
//   b=34 s=147 a=4  dh=128 causal    272   10.5 | 37.4   15.6 | 51.9   13.0 | 52.1
//   b=16 s=99  a=12 dh=128 causal    192        | 31.6        | 36.7
//   b=18 s=16  a=16 dh=64            288        | 23.8        | 25.8        | 16.8
// So the halves pay off in a launch of one round, but without a mask only up to half a block of 256 rows per CU: above, 8 x 1 is even
// and has the simpler kernel.  A second round costs what the halves save, except under a causal mask, where the blocks' work differs
// and a launch ends on its longest: there from 257 rows on, in the backward pass and for heads above 64 from 513 unless a quarter of
// the CUs has no block of 256 rows.  At head size 128 the backward's dK and dV are workgroups of their own in these shapes, so two
// rounds begin at half as many rows.  4 x 2 while 8 x 2 would not fill half of the CUs.  Sequences of one tile have nothing to split:
// 4 x 2 there only packs more workgroups into a CU, where the registers allow it (backward; forward up to head size 64: at 80
// b=36 s=52 a=12 8.7 -> 9.6 us).  Over 700 random sizes of all masks the choice costs 3 % over the best shape, and no call of 491 with a fixed
// head size that takes more than 6 us is slower than on 8 x 1 by more than 2 %.  Under a causal mask alone, where the lines are coarsest,
// the forward pass is 9 % over the best shape (600 random calls of 60 to 1100 workgroups of 256 rows, every shape forced: 1.094, at worst 1.7;
// in the plain order of blocks 1.099, so the folded order has not moved the lines): mostly 4 x 2 where 8 x 2 is taken, or, for
// heads up to 48, 8 x 1.
namespace {
enum Shape { k8x1, k8x2, k4x2 };
Shape shape_for(const AttnDesc& d, bool bwd) {
  const int64_t heads = (int64_t)d.b * d.a, blocks = heads * ceil_div(d.s, 256), w = heads * ceil_div(d.s, 128), cus = gemm_compute_units();
  const bool causal = d.mask_mode == 1, apart = bwd && d.dh == 128;
  if (d.s <= 64) {   // one streamed tile
    if (bwd) return apart && 2 * blocks > cus ? k8x1 : k4x2;
    return blocks > cus && d.dh <= 64 ? k4x2 : k8x1;
  }
  bool split;
  if (w <= cus) split = (causal || 2 * blocks <= cus) && !(apart && 2 * w > cus && d.s <= 256);
  else split = causal && blocks <= cus && d.s > 256 && ((!bwd && d.dh <= 64) || 4 * blocks <= 3 * cus || (d.s > 512 && !apart)) && !(apart && d.s <= 512);
  if (!split) return k8x1;
  return 2 * w > cus ? k8x2 : k4x2;
}
int rows_of(Shape sh) { return sh == k8x1 ? 256 : sh == k8x2 ? 128 : 64; }
}  // namespace

int attention_colsum_rows(const AttnDesc& d) { return d.b * ceil_div(d.s, rows_of(shape_for(d, true))); }
int attention_colsum_max_rows(int b, int s) { return b * ceil_div(s, 64); }

bool attention_emits_colsum(const AttnDesc& d) {
  return d.dtype == kBF16 && (d.dh == 32 || d.dh == 64 || d.dh == 80 || d.dh == 128);
}

hipError_t attention_fwd_mfma(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) {
  switch (shape_for(d, false)) {
    case k8x1: return attention_fwd_mfma_8x1(d, qkv, o, lse, st);
    case k8x2: return attention_fwd_mfma_8x2(d, qkv, o, lse, st);
    default: return attention_fwd_mfma_4x2(d, qkv, o, lse, st);
  }
}

hipError_t attention_bwd_mfma(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta,
                              hipStream_t st) {
  switch (shape_for(d, true)) {
    case k8x1: return attention_bwd_mfma_8x1(d, qkv, o, lse, d_o, dqkv, delta, st);
    case k8x2: return attention_bwd_mfma_8x2(d, qkv, o, lse, d_o, dqkv, delta, st);
    default: return attention_bwd_mfma_4x2(d, qkv, o, lse, d_o, dqkv, delta, st);
  }
}

}  // namespace k2bw
