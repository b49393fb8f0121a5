// bf16 masked-softmax attention on the gfx950 matrix cores, forward and backward, for every head size that is a
// multiple of 8 up to 128.  fp32 scores, statistics and accumulators; no s x s matrix in HBM.
//
// Two sets of instances.  Head sizes 32, 64, 80 and 128 have one each (ANY = false).  The others run on the next larger
// of 32, 48, 64, 80, 96, 112, 128 with the true size at run time (ANY = true): tile columns past the head are fetched from
// a zeroed chunk, rows past the sequence too.  These keep their probabilities (and dS) in 32 bits, as the kernels did that these
// sizes used to run on (one thread per row in fp32 on the vector ALU): a value enters the second product as the sum of three bf16
// numbers that hold its 24 bits, three MFMAs instead of one; and a position that some rows of a tile may not see cannot reach them
// even if it holds infinities or NaNs (accumulate_visible).  Measured at b=3 s=1000 a=16 dh=96 causal against those kernels:
// forward 2892 -> 36 us, backward 16480 -> 118.  (With two numbers, 16 bits, 32 and 107 us; but a sum whose terms cancel to a
// thousandth then shows it: 1 % off instead of bf16's rounding.)
//
// All three kernels keep one query (forward, dQ) or one key (dK/dV) per lane of a 32-wide MFMA
// column, so softmax statistics, lse and delta are per-lane scalars or short in-lane loops:
//
//   forward   S^T = K Q^T  (keys x queries): lane = query, registers = keys.  Row maximum and
//             sum are in-lane plus one exchange between the two 32-lane halves.  P^T in that
//             layout is directly the second MFMA operand of O^T = V^T P^T.
//   dQ        same orientation: dP^T = V dO^T, dS^T = P^T (dP^T - delta), dQ^T = K^T dS^T.
//   dK, dV    S = Q K^T (queries x keys): lane = key, registers = queries; P and dS in that
//             layout are the second operands of dV^T = dO^T P and dK^T = Q^T dS.
//
// v_mfma_f32_32x32x16_bf16: lane l gives row l%32 of the first operand and column l%32 of the
// second, k-slots 8*(l/32)..+7; it gets column l%32 of the result, rows 8*(r/4)+4*(l/32)+(r%4)
// in register r.  Re-using a result as a second operand therefore fixes which actual index
// sits in which k-slot (slot t of half hf <-> index 16*kk + 4*hf + t for t < 4, 16*kk + 8 +
// 4*hf + t - 4 otherwise); the transposing LDS reads deliver the first operand in that order.
//
// LDS tiles are row-major [64 rows][dh] copies of K, V, Q or dO rows, filled straight from HBM by
// global_load_lds (16 bytes per lane, no registers, no LDS store instructions), two stages deep:
// the loads of tile t+1 are in flight while tile t is consumed, one barrier per tile.  A tile
// serves both operand forms: rows as MFMA rows (16-byte reads along dh) and, through
// ds_read_b64_tr_b16, columns as MFMA rows (the transposed operands K^T, V^T, Q^T, dO^T), so no
// transposed copy is ever built.  16-byte chunks are XOR-swizzled by row so that both read
// patterns are bank-conflict free.  Masked keys get probability exactly zero.
#pragma once
#include <type_traits>

#include "kernels.hpp"

namespace k2bw {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16_t;
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) char lds_char_t;
typedef __attribute__((address_space(1))) const void glob_void_t;

// Waves per workgroup (NW), 32 rows (queries or keys) each.  Measured on MI355X with 2 / 4 / 8 waves
// (one split, s = 512, dh = 64: forward 27.9 / 20.7 / 19.5 us, backward 66.7 / 58.8 / 57.1 us; s = 2048,
// dh = 128 causal: forward 270 / 258 / 152 us): more waves share each K/V tile and each barrier.
// That is with a workgroup for every CU; see shape_for for smaller launches.
constexpr int kTile = 64;         // rows streamed through LDS per step
constexpr int kMaxDeltas = 2048;  // longest sequence whose deltas a workgroup holds in LDS
constexpr float kLog2e = 1.4426950408889634f;

template <int DH, bool ANY = false>
struct Cfg {
  static constexpr int KS = DH / 16;               // MFMA k-steps over the head dimension
  static constexpr int DHP = (DH + 31) / 32 * 32;  // head dimension padded to whole 32-row blocks
  static constexpr int DB = DHP / 32;
  static constexpr int CH = DH / 8;                // 16-byte chunks per tile row
  static constexpr int kTileU4 = kTile * CH;       // uint4 per tile
  static constexpr int kPadU4 = 4;                 // transposing reads of the padded head columns run past a row
  static constexpr bool kDkvParts = ANY && DH >= 80;   // dK and dV always in workgroups of their own
  static constexpr bool kDkvVInLds = DH == 128 && !ANY;   // dK/dV kernel: V fragments of the wave's keys in LDS, not registers
};

// Chunk swizzle per head size (rows are 64 / 96 / 128 / 160 / 192 / 224 / 256 bytes; the LDS has 64 banks of 4 bytes).
// Checked against a bank model for both read patterns: 16-byte reads of 16 consecutive rows at one
// logical chunk, and the transposing 8-byte reads (4 consecutive rows x 32 or 64 contiguous bytes).
template <int DH>
__device__ __forceinline__ int swz(int r) {
  if (DH == 32) return (r >> 2) & 3;
  if (DH == 64) { const int u = (r >> 1) & 7; return ((u & 1) << 2) | (u >> 1); }
  if (DH == 48 || DH == 80 || DH == 112) return (r >> 3) & 1;   // 8 rows start on 8 different even chunks of a bank line
  if (DH == 96) return (r >> 2) & 3;                            // 4 rows start on every fourth chunk
  return ((r & 3) << 2) | ((r >> 2) & 3);
}

// s_waitcnt immediate for "at most n vector-memory operations outstanding" (gfx9 encoding)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// Rows [row0, row0 + 64) x DH of a [*, ld] matrix -> LDS tile; lane i of a load instruction owns
// LDS slot L0 + i and fetches the chunk that belongs there.  Rows >= row_end are fetched from row
// row_end - 1 (finite data; whatever they produce is masked or never stored).  ANY: those rows and the
// columns past the head come from a chunk of zeros.
__device__ const uint4 kZeroChunk = {0, 0, 0, 0};
template <int DH, bool ANY, int NW>
struct TileLoader {
  static constexpr int CH = DH / 8;
  static constexpr int kInstr = kTile * CH / 64;            // wave-instructions per tile
  static constexpr int NI = (kInstr + NW - 1) / NW;  // per wave
  int row[NI], coff[NI];
  int wave_;
  __device__ __forceinline__ void init(int wave, int lane, int dh) {
    wave_ = wave;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int L = (j * NW + wave) * 64 + lane;
      const int r = L / CH, pc = L % CH;
      row[j] = r < kTile ? r : kTile - 1;
      coff[j] = (pc ^ swz<DH>(r)) * 8;
      if (ANY && coff[j] >= dh) coff[j] = -1;
    }
  }
  __device__ __forceinline__ void issue(const bf16_t* __restrict__ src, int64_t ld, int row0, int row_end, uint4* tile) const {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      if ((j * NW + wave_) < kInstr) {   // wave-uniform
        const int r = min(row0 + row[j], row_end - 1);
        const bf16_t* from = src + (int64_t)r * ld + (ANY ? max(coff[j], 0) : coff[j]);
        if (ANY && (coff[j] < 0 || row0 + row[j] >= row_end)) from = reinterpret_cast<const bf16_t*>(&kZeroChunk);
        __builtin_amdgcn_global_load_lds((glob_void_t*)from, (lds_void_t*)(tile + (j * NW + wave_) * 64), 16, 0, 0);
      }
    }
  }
};

// 16-byte k-fragment of a row of a [*, ld] matrix straight from HBM (second MFMA operand)
template <int DH, bool ANY>
__device__ __forceinline__ void load_frags(const bf16_t* __restrict__ row_ptr, bool ok, int hf, int dh, bf16x8 (&f)[Cfg<DH>::KS]) {
#pragma unroll
  for (int ks = 0; ks < Cfg<DH>::KS; ++ks) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (ok && (!ANY || ks * 16 + hf * 8 < dh)) v = *reinterpret_cast<const uint4*>(row_ptr + ks * 16 + hf * 8);
    f[ks] = __builtin_bit_cast(bf16x8, v);
  }
}

// first operand, rows of the tile as MFMA rows: row `row`, head columns 16*ks + 8*hf .. +7
template <int DH>
__device__ __forceinline__ bf16x8 read_rows(const uint4* tile, int row, int ks, int hf) {
  return __builtin_bit_cast(bf16x8, tile[row * Cfg<DH>::CH + ((ks * 2 + hf) ^ swz<DH>(row))]);
}

// registers 8*half .. 8*half+7 of a result block -> second operand of the next MFMA
__device__ __forceinline__ bf16x8 pack_half(const f32x16& v, int half) {
  uint4 w;
  const int b = 8 * half;
  w.x = pack_bf16x2(v[b + 0], v[b + 1]); w.y = pack_bf16x2(v[b + 2], v[b + 3]);
  w.z = pack_bf16x2(v[b + 4], v[b + 5]); w.w = pack_bf16x2(v[b + 6], v[b + 7]);
  return __builtin_bit_cast(bf16x8, w);
}

// The same as the sum of three operands that together hold all 24 bits of the values: what rounding to bf16 gives, the rounding
// of what that left, and the rest (the differences are exact, and the rest has at most 6 bits)
struct Exact8 { bf16x8 part[3]; };
__device__ __forceinline__ Exact8 pack_half_exact(const f32x16& v, int half) {
  uint32_t w[3][4];
  const int b = 8 * half;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float x = v[b + 2 * i], y = v[b + 2 * i + 1];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      w[p][i] = pack_bf16x2(x, y);
      x -= __uint_as_float(w[p][i] << 16);
      y -= __uint_as_float(w[p][i] & 0xffff0000u);
    }
  }
  Exact8 e;
#pragma unroll
  for (int p = 0; p < 3; ++p) e.part[p] = __builtin_bit_cast(bf16x8, make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]));
  return e;
}
// acc += X P for such a P
__device__ __forceinline__ void mul_exact(const bf16x8& x, const Exact8& p, f32x16& acc) {
#pragma unroll
  for (int i = 0; i < 3; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, p.part[i], acc, 0, 0, 0);
}

// First operand, head columns of the tile as MFMA rows: this lane's row is head column
// d0 + lane % 32, its k-slots are tile rows 16*kk + 4*hf + 0..3 and 16*kk + 8 + 4*hf + 0..3 (the
// order in which a 32x32 result block, re-used as second operand, holds them).
// ds_read_b64_tr_b16, measured on gfx950: within each group of 16 lanes, lane a + 4t supplies the
// address of 4 consecutive columns of row t, and lane 4a + j receives rows 0..3 of column 4a + j.
template <int DH>
__device__ __forceinline__ bf16x8 read_cols(const uint4* tile, int d0, int kk, int lane) {
  const int r16 = lane & 15, a = r16 & 3, t = r16 >> 2, hf = lane >> 5;
  const int col = d0 + ((lane >> 4) & 1) * 16 + 4 * a;
  const int r0 = 16 * kk + 4 * hf + t, r1 = r0 + 8;
  const int b0 = r0 * (DH * 2) + (((col >> 3) ^ swz<DH>(r0)) << 4) + ((col >> 2) & 1) * 8;
  const int b1 = r1 * (DH * 2) + (((col >> 3) ^ swz<DH>(r1)) << 4) + ((col >> 2) & 1) * 8;
  const lds_char_t* base = (const lds_char_t*)tile;
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(base + b0));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(base + b1));
  const v8i16 w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, w);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

// A wave's result blocks through LDS (64 lanes x 16*DB floats, a lane's own), from one half of a workgroup to the other
template <int DB>
__device__ __forceinline__ void give(const f32x16 (&acc)[DB], float* buf, int lane) {
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) buf[(db * 16 + r) * 64 + lane] = acc[db][r];
}
template <int DB>
__device__ __forceinline__ void take(f32x16 (&acc)[DB], const float* buf, int lane) {
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] += buf[(db * 16 + r) * 64 + lane];
}
template <int DB>
__device__ __forceinline__ void clear(f32x16 (&acc)[DB]) {
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = zero16();
}

__device__ __forceinline__ uint2 pack4f(float a, float b, float c, float d) {
  return make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
}

// Does the 64-row tile hold an infinity or a NaN? (the same answer in every lane)
template <int DH>
__device__ __forceinline__ bool tile_not_finite(const uint4* tile, int lane) {
  uint32_t top = 0;   // adding 1 to an exponent of all ones carries into the sign's place
#pragma unroll 4
  for (int i = 0; i < Cfg<DH>::CH; ++i) {
    const uint4 v = tile[i * 64 + lane];
    top |= ((v.x & 0x7f807f80u) + 0x00800080u) | ((v.y & 0x7f807f80u) + 0x00800080u) | ((v.z & 0x7f807f80u) + 0x00800080u) |
           ((v.w & 0x7f807f80u) + 0x00800080u);
  }
  return __any((top & 0x80008000u) != 0);
}

// out += X^T P over the tile rows [row0, row0 + 32), row by row and only into the lanes whose query (key) sees the row: for
// a tile that holds infinities or NaNs and is not visible as a whole (0 * inf would reach rows that must not see it).
// Rare: the kernels only look for such tiles in their loop, and a workgroup that met one starts over in the EXACT form
// (inside the one loop this path cost the dK/dV kernel hundreds of spilled registers: 299 us instead of 100 at head size 96, b=3 s=1000 a=16).
template <int DH, typename Sees>
__device__ __forceinline__ void accumulate_visible(const uint4* tile, int row0, const f32x16& p, f32x16 (&out)[Cfg<DH>::DB], int lane, Sees&& sees) {
  const int hf = lane >> 5;
#pragma unroll 1
  for (int rr = 0; rr < 32; ++rr) {
    const int reg = (rr >> 3) * 4 + (rr & 3), row = row0 + rr;
    float w = p[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) w = e == reg ? p[e] : w;
    const float other = __shfl_xor(w, 32, 64);
    w = ((rr >> 2) & 1) == hf ? w : other;
    if (!sees(row)) continue;
    const lds_char_t* x = (const lds_char_t*)(tile + row * Cfg<DH>::CH) + hf * 8;
    const int sw = swz<DH>(row);
#pragma unroll
    for (int chunk = 0; chunk < Cfg<DH>::CH; ++chunk) {
      const u32x2 v = *(const __attribute__((address_space(3))) u32x2*)(x + ((chunk ^ sw) << 4));
      f32x16& o = out[chunk >> 2];
      const int g = 4 * (chunk & 3);
      o[g] = fmaf(w, __uint_as_float(v.x << 16), o[g]);
      o[g + 1] = fmaf(w, __uint_as_float(v.x & 0xffff0000u), o[g + 1]);
      o[g + 2] = fmaf(w, __uint_as_float(v.y << 16), o[g + 2]);
      o[g + 3] = fmaf(w, __uint_as_float(v.y & 0xffff0000u), o[g + 3]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Sum of v over the 16 lanes of a DPP row, left in every lane of the row: two quad permutes, then
// the half-row and full-row mirrors (each step adds a lane that holds the other group's sum).
__device__ __forceinline__ float row16_sum(float v) {
  auto dpp_add = [](float x, auto ctrl) {
    const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, false);
    return x + __builtin_bit_cast(float, y);
  };
  v = dpp_add(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
  v = dpp_add(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
  v = dpp_add(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
  v = dpp_add(v, std::integral_constant<int, 0x140>{});   // row_mirror
  return v;
}

// ... and over the 8 lanes of half a row
__device__ __forceinline__ float row8_sum(float v) {
  auto dpp_add = [](float x, auto ctrl) {
    const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, false);
    return x + __builtin_bit_cast(float, y);
  };
  v = dpp_add(v, std::integral_constant<int, 0xB1>{});
  v = dpp_add(v, std::integral_constant<int, 0x4E>{});
  return dpp_add(v, std::integral_constant<int, 0x141>{});
}

// Column sums over the workgroup's rows of a result held as acc[db][r] (lane = row, registers =
// head columns db*32 + 8*(r/4) + 4*hf + r%4), scaled by `scale`, written to out[0 .. DH).
// red: 2 * NW * DHP floats of LDS that no wave still reads (one partial row per 16 lanes).
template <int DH, int NW>
__device__ __forceinline__ void block_column_sums(const f32x16 (&acc)[Cfg<DH>::DB], float scale, float* red, float* out,
                                                  int tid, int lane, int wave) {
  using C = Cfg<DH>;
  const int hf = lane >> 5;
  float* mine = red + (wave * 2 + ((lane >> 4) & 1)) * C::DHP + 4 * hf;
#pragma unroll
  for (int db = 0; db < C::DB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float4 v;
      v.x = row16_sum(acc[db][4 * g]);
      v.y = row16_sum(acc[db][4 * g + 1]);
      v.z = row16_sum(acc[db][4 * g + 2]);
      v.w = row16_sum(acc[db][4 * g + 3]);
      if ((lane & 15) == 0) *reinterpret_cast<float4*>(mine + db * 32 + 8 * g) = v;
    }
  __syncthreads();
  for (int d = tid; d < DH; d += NW * 64) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 2 * NW; ++w) t += red[w * C::DHP + d];
    out[d] = t * scale;
  }
}

// Rows of a result held as acc[db][r] (lane % 32 = row, registers = head columns db*32 + 8*(r/4) + 4*hf + r%4),
// times `scale`, to out[row][0 .. DH) (bf16, `ld` elements between rows; `out` is row 0 of this wave's 32 rows, of
// which the first rows_valid exist).  Stored as they lie in the registers, a lane writes 8-byte pieces and one store
// instruction touches 32 rows with 16 bytes each: measured, those stores were two thirds of what the dK/dV kernel costs
// beyond its loop (8.5 of 12.5 us per workgroup at head size 128).  So the rows pass through a wave-private piece
// of LDS (rows 16 bytes apart from a multiple of 256: the 8-byte writes of 32 rows spread over the banks) and
// leave with 16 bytes per lane along a row.  No barrier: the piece belongs to the wave, whose LDS operations
// complete in order.  `strip`: 32 * (2 * DH + 16) bytes.
template <int DH>
constexpr int out_strip_u4() { return 32 * (2 * DH + 16) / 16; }
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <int DH>
__device__ __forceinline__ void store_rows(const f32x16 (&acc)[Cfg<DH>::DB], float scale, uint4* strip, bf16_t* out, int64_t ld,
                                           int rows_valid, int dh, int lane) {
  using C = Cfg<DH>;
  constexpr int STRIDE = 2 * DH + 16;   // bytes
  char* w = reinterpret_cast<char*>(strip);
  const int l32 = lane & 31, hf = lane >> 5;
#pragma unroll
  for (int db = 0; db < C::DB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int d = db * 32 + 8 * g + 4 * hf;
      if (d < DH)
        *reinterpret_cast<uint2*>(w + l32 * STRIDE + d * 2) =
            pack4f(acc[db][4 * g] * scale, acc[db][4 * g + 1] * scale, acc[db][4 * g + 2] * scale, acc[db][4 * g + 3] * scale);
    }
  wave_lds_sync();
  constexpr int TOTAL = 32 * C::CH;   // 16-byte chunks of the 32 rows
#pragma unroll
  for (int it = 0; it < (TOTAL + 63) / 64; ++it) {
    const int L = it * 64 + lane;
    const int row = L / C::CH, ch = L % C::CH;
    if (L < TOTAL && row < rows_valid && ch * 8 < dh)
      *reinterpret_cast<uint4*>(out + row * ld + ch * 8) = *reinterpret_cast<const uint4*>(w + row * STRIDE + ch * 16);
  }
  wave_lds_sync();   // the strip may be written again
}

// ------------------------------------------------------------------------------------------------
// forward
// (all kernels: two waves per SIMD, which 8-wave workgroups imply, cap a lane at 256 registers; the compiler then keeps
// MFMA results in ordinary VGPRs.  With 512 available it parks them in the accumulator file and copies every score to a
// VGPR and back around the softmax arithmetic, which costs more than the MFMAs.)
template <int DH, int NW, int KSPL, bool ANY, bool EXACT>
__device__ __forceinline__ bool attn_fwd(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o, float* __restrict__ lse, int s, int a, int mask_mode, const int32_t* __restrict__ seqlens, int dh_, int blk) {
  using C = Cfg<DH>;
  extern __shared__ uint4 smem[];   // stage st: K tile at st * 2 * kTileU4, V tile behind it

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  // wave = (part of the streamed rows, group of own rows): with KSPL = 2 each half of the waves takes every second tile,
  // through tiles of its own in LDS, and the halves' results meet at the end
  constexpr int RW = NW / KSPL;
  const int kg = KSPL == 1 ? 0 : wave / RW, rw = KSPL == 1 ? wave : wave % RW;
  // grid = (heads, sequences, row blocks): the row block varies slowest, so all heads' copies of a block are
  // dispatched together, and under a causal mask the blocks with the most keys to visit (the last queries) go
  // first: the workgroups that take longest start earliest and the launch does not end on one of them (where all start at once: Fold)
  const int n = blockIdx.y, head = blockIdx.x;
  const int i0 = blk * RW * 32;
  const int dh = ANY ? dh_ : DH;
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const bf16_t* base = qkv + (int64_t)n * s * ld + head * dh;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;   // lengths outside [1, s] are clamped: no read past the sequence, no empty row
  const bool causal = mask_mode == 1;
  const int iw0 = i0 + rw * 32;
  const int i = iw0 + l32;
  const float scale = 1.0f / sqrtf((float)dh);
  const float c = scale * kLog2e;

  bf16x8 qf[C::KS];
  load_frags<DH, ANY>(base + (int64_t)i * ld, i < s, hf, dh, qf);
  f32x16 oacc[C::DB];
  float m_i = -INFINITY, l_i = 0.f;
  bool hidden = false;   // ANY: a tile that not every row sees holds infinities or NaNs

  const int jend = causal ? min(i0 + RW * 32, s) : kv_len;
  const int ntiles = (jend + kTile - 1) / kTile;
  TileLoader<DH, ANY, RW> loader;
  loader.init(rw, lane, dh);
#pragma unroll
  for (int db = 0; db < C::DB; ++db) oacc[db] = zero16();
  uint4* const tiles = smem + kg * (4 * C::kTileU4 + C::kPadU4);
  if (kg < ntiles) {
    loader.issue(base + h, ld, kg * kTile, jend, tiles);
    loader.issue(base + 2 * h, ld, kg * kTile, jend, tiles + C::kTileU4);
  }
  for (int st = 0; st * KSPL < ntiles; ++st) {
    const int t = st * KSPL + kg, j0 = t * kTile;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // this wave's share of tile t has landed
    __syncthreads();                            // ... and everyone's; all waves are done with the tile before
    if (t + KSPL < ntiles) {
      uint4* nxt = tiles + ((st + 1) & 1) * 2 * C::kTileU4;
      loader.issue(base + h, ld, j0 + KSPL * kTile, jend, nxt);
      loader.issue(base + 2 * h, ld, j0 + KSPL * kTile, jend, nxt + C::kTileU4);
    }
    if (KSPL > 1 && t >= ntiles) continue;   // (the last step of an odd number of tiles)
    if (causal && j0 > iw0 + 31) continue;   // every key of the tile lies after this wave's queries
    const uint4* k_lds = tiles + (st & 1) * 2 * C::kTileU4;
    const uint4* v_lds = k_lds + C::kTileU4;

    f32x16 sacc[2] = {zero16(), zero16()};
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
      sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows<DH>(k_lds, l32, ks, hf), qf[ks], sacc[0], 0, 0, 0);
      sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows<DH>(k_lds, 32 + l32, ks, hf), qf[ks], sacc[1], 0, 0, 0);
    }
    // masks (only tiles that touch a boundary need them) and the running maximum
    const bool need_mask = (j0 + kTile > kv_len) || (causal && j0 + kTile - 1 > iw0);
    if (need_mask) {
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = j0 + nb * 32 + 8 * (r >> 2) + 4 * hf + (r & 3);
          const bool vis = key < kv_len && (!causal || key <= i);
          sacc[nb][r] = vis ? sacc[nb][r] : -INFINITY;
        }
    }
    float mloc = -INFINITY;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, sacc[nb][r]);
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float m_new = fmaxf(m_i, mloc);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;   // row with nothing visible yet
    const float alpha = __builtin_amdgcn_exp2f((m_i - m_use) * c);
    const float mc = m_use * c;
    float rowsum = 0.f;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float pv = __builtin_amdgcn_exp2f(ANY ? (sacc[nb][r] - m_use) * c : fmaf(sacc[nb][r], c, -mc));
        sacc[nb][r] = pv;
        rowsum += pv;
      }
    l_i = l_i * alpha + rowsum;
    m_i = m_new;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
    if constexpr (ANY) {
      if (causal && j0 + kTile - 1 > iw0) {
        if (EXACT) {
#pragma unroll
          for (int nb = 0; nb < 2; ++nb) accumulate_visible<DH>(v_lds, nb * 32, sacc[nb], oacc, lane, [&](int row) { return j0 + row <= i; });
          continue;
        }
        hidden = hidden || tile_not_finite<DH>(v_lds, lane);
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const Exact8 pe = pack_half_exact(sacc[kk >> 1], kk & 1);
#pragma unroll
        for (int db = 0; db < C::DB; ++db) mul_exact(read_cols<DH>(v_lds, db * 32, kk, lane), pe, oacc[db]);
      }
    } else {
      bf16x8 pb[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) pb[kk] = pack_half(sacc[kk >> 1], kk & 1);
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_cols<DH>(v_lds, db * 32, kk, lane), pb[kk], oacc[db], 0, 0, 0);
    }
  }
  if constexpr (ANY && !EXACT)
    if (__syncthreads_or(hidden)) return true;

  __syncthreads();   // every wave is done with the K / V tiles, whose LDS is used again below
  if constexpr (KSPL == 2) {
    float* buf = reinterpret_cast<float*>(smem) + rw * ((C::DB * 16 + 2) * 64);
    if (kg == 1) {
      give<C::DB>(oacc, buf, lane);
      buf[C::DB * 16 * 64 + lane] = m_i;
      buf[(C::DB * 16 + 1) * 64 + lane] = l_i;
    }
    __syncthreads();
    if (kg == 0) {   // both halves to the larger of the two maxima (a half without a visible key adds nothing)
      const float m1 = buf[C::DB * 16 * 64 + lane], l1 = buf[(C::DB * 16 + 1) * 64 + lane];
      const float m = fmaxf(m_i, m1);
      const float f0 = m_i == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_i - m) * c), f1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m1 - m) * c);
      l_i = l_i * f0 + l1 * f1;
      m_i = m;
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = oacc[db][r] * f0 + buf[(db * 16 + r) * 64 + lane] * f1;
    }
    __syncthreads();
  }
  const float l_tot = l_i + __shfl_xor(l_i, 32, 64);
  const float inv = 1.0f / l_tot;   // (rows past the sequence: never stored)
  store_rows<DH>(oacc, inv, smem + wave * out_strip_u4<DH>(), o + ((int64_t)n * s + iw0) * h + head * dh, h, kg == 0 ? s - iw0 : 0, dh, lane);
  if (i < s && hf == 0 && kg == 0) lse[((int64_t)n * a + head) * s + i] = m_i * scale + logf(l_tot);
  return false;
}
template <int DH, int NW, int KSPL, bool ANY>
__global__ __launch_bounds__(NW * 64, 2) void attn_fwd_mfma_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o, float* __restrict__ lse, int s, int a, int mask_mode, const int32_t* __restrict__ seqlens, int dh_, Fold fold) {
  const int z = folded_z(fold), blk = mask_mode == 1 ? (int)gridDim.z - 1 - z : z;
  if (attn_fwd<DH, NW, KSPL, ANY, false>(qkv, o, lse, s, a, mask_mode, seqlens, dh_, blk))
    if constexpr (ANY) attn_fwd<DH, NW, KSPL, ANY, true>(qkv, o, lse, s, a, mask_mode, seqlens, dh_, blk);
}

// ------------------------------------------------------------------------------------------------
// dQ (and, if SAVE, delta = rowsum(dO * O), which the dK/dV kernel reads afterwards)
template <int DH, int NW, int KSPL, bool ANY, bool EXACT, bool SAVE>
__device__ __forceinline__ bool attn_dq(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o, const float* __restrict__ lse, float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int a, int mask_mode, const int32_t* __restrict__ seqlens, float* __restrict__ colsum, int dh_, int blk, int nblk) {
  using C = Cfg<DH>;
  extern __shared__ uint4 smem[];   // stage st: K tile at st * 2 * kTileU4, V tile behind it

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  // wave = (part of the streamed rows, group of own rows): with KSPL = 2 each half of the waves takes every second tile,
  // through tiles of its own in LDS, and the halves' results meet at the end
  constexpr int RW = NW / KSPL;
  const int kg = KSPL == 1 ? 0 : wave / RW, rw = KSPL == 1 ? wave : wave % RW;
  // grid = (heads, sequences, row blocks): the row block varies slowest, so all heads' copies of a block are
  // dispatched together, and under a causal mask the blocks with the most keys to visit (the last queries) go
  // first: the workgroups that take longest start earliest and the launch does not end on one of them
  const int n = blockIdx.y, head = blockIdx.x;
  const int i0 = blk * RW * 32;
  const int dh = ANY ? dh_ : DH;
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const bf16_t* base = qkv + (int64_t)n * s * ld + head * dh;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;   // lengths outside [1, s] are clamped: no read past the sequence, no empty row
  const bool causal = mask_mode == 1;
  const int iw0 = i0 + rw * 32;
  const int i = iw0 + l32;
  const bool row_ok = i < s;
  const float scale = 1.0f / sqrtf((float)dh);
  const float c = scale * kLog2e;

  const int jend = causal ? min(i0 + RW * 32, s) : kv_len;
  const int ntiles = (jend + kTile - 1) / kTile;
  TileLoader<DH, ANY, RW> loader;
  loader.init(rw, lane, dh);
  uint4* const tiles = smem + kg * (4 * C::kTileU4 + C::kPadU4);
  if (kg < ntiles) {
    loader.issue(base + h, ld, kg * kTile, jend, tiles);
    loader.issue(base + 2 * h, ld, kg * kTile, jend, tiles + C::kTileU4);
  }

  bf16x8 qf[C::KS], dof[C::KS];
  load_frags<DH, ANY>(base + (int64_t)i * ld, row_ok, hf, dh, qf);
  load_frags<DH, ANY>(d_o + ((int64_t)n * s + i) * h + head * dh, row_ok, hf, dh, dof);
  float delta_i;
  {
    bf16x8 of[C::KS];
    load_frags<DH, ANY>(o + ((int64_t)n * s + i) * h + head * dh, row_ok, hf, dh, of);
    float part = 0.f;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) part = fmaf((float)dof[ks][e], (float)of[ks][e], part);
    delta_i = part + __shfl_xor(part, 32, 64);
    if (SAVE && row_ok && hf == 0 && kg == 0) delta[((int64_t)n * a + head) * s + i] = delta_i;
  }
  const float lse_i = row_ok ? lse[((int64_t)n * a + head) * s + i] * (ANY ? 1.f : kLog2e) : INFINITY;
  // dP - delta comes out of the product, whose accumulators start at -delta; at head size 32 delta is subtracted afterwards: the
  // 16 registers are what keeps that kernel under 128, so that a CU holds two workgroups (141 registers: backward at b=17 s=390
  // a=32 causal 97 us instead of 82)
  constexpr bool kDeltaFirst = DH > 32 || ANY;
  f32x16 dp_start = zero16();
  if (kDeltaFirst) {
#pragma unroll
    for (int r = 0; r < 16; ++r) dp_start[r] = -delta_i;
  }
  f32x16 dq[C::DB];
  bool hidden = false;
#pragma unroll
  for (int db = 0; db < C::DB; ++db) dq[db] = zero16();
  for (int st = 0; st * KSPL < ntiles; ++st) {
    const int t = st * KSPL + kg, j0 = t * kTile;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    if (t + KSPL < ntiles) {
      uint4* nxt = tiles + ((st + 1) & 1) * 2 * C::kTileU4;
      loader.issue(base + h, ld, j0 + KSPL * kTile, jend, nxt);
      loader.issue(base + 2 * h, ld, j0 + KSPL * kTile, jend, nxt + C::kTileU4);
    }
    if (KSPL > 1 && t >= ntiles) continue;   // (the last step of an odd number of tiles)
    if (causal && j0 > iw0 + 31) continue;
    const uint4* k_lds = tiles + (st & 1) * 2 * C::kTileU4;
    const uint4* v_lds = k_lds + C::kTileU4;

    f32x16 sacc[2] = {zero16(), zero16()}, dp[2] = {dp_start, dp_start};
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        sacc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows<DH>(k_lds, nb * 32 + l32, ks, hf), qf[ks], sacc[nb], 0, 0, 0);
        dp[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows<DH>(v_lds, nb * 32 + l32, ks, hf), dof[ks], dp[nb], 0, 0, 0);
      }
    }
    const bool need_mask = (j0 + kTile > kv_len) || (causal && j0 + kTile - 1 > iw0);
    if (need_mask) {   // a masked score of -inf gives probability exactly 0
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = j0 + nb * 32 + 8 * (r >> 2) + 4 * hf + (r & 3);
          const bool vis = key < kv_len && (!causal || key <= i);
          sacc[nb][r] = vis ? sacc[nb][r] : -INFINITY;
          if (ANY) dp[nb][r] = vis ? dp[nb][r] : 0.f;   // dS is zero then, whatever the masked V holds
        }
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float pv = __builtin_amdgcn_exp2f(ANY ? fmaf(sacc[nb][r], scale, -lse_i) * kLog2e : fmaf(sacc[nb][r], c, -lse_i));
        sacc[nb][r] = pv * (kDeltaFirst ? dp[nb][r] : dp[nb][r] - delta_i);   // dS^T (the 1/sqrt(dh) factor is applied at the end)
      }
    if constexpr (ANY) {
      if (causal && j0 + kTile - 1 > iw0) {
        if (EXACT) {
#pragma unroll
          for (int nb = 0; nb < 2; ++nb) accumulate_visible<DH>(k_lds, nb * 32, sacc[nb], dq, lane, [&](int row) { return j0 + row <= i; });
          continue;
        }
        hidden = hidden || tile_not_finite<DH>(k_lds, lane);
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const Exact8 dse = pack_half_exact(sacc[kk >> 1], kk & 1);
#pragma unroll
        for (int db = 0; db < C::DB; ++db) mul_exact(read_cols<DH>(k_lds, db * 32, kk, lane), dse, dq[db]);
      }
    } else {
      bf16x8 dsb[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) dsb[kk] = pack_half(sacc[kk >> 1], kk & 1);
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_cols<DH>(k_lds, db * 32, kk, lane), dsb[kk], dq[db], 0, 0, 0);
    }
  }
  if constexpr (ANY && !EXACT)
    if (__syncthreads_or(hidden)) return true;
  __syncthreads();   // every wave is done with the K / V tiles
  if constexpr (KSPL == 2) {
    float* buf = reinterpret_cast<float*>(smem) + rw * (C::DB * 16 * 64);
    if (kg == 1) { give<C::DB>(dq, buf, lane); clear<C::DB>(dq); }
    __syncthreads();
    if (kg == 0) take<C::DB>(dq, buf, lane);
    __syncthreads();
  }
  if (!ANY && colsum) {   // rows past the end of the sequence hold zeros
    float* row = colsum + ((int64_t)n * nblk + blk) * ld + head * dh;
    block_column_sums<DH, NW>(dq, scale, reinterpret_cast<float*>(smem), row, tid, lane, wave);
    __syncthreads();   // ... and with the partial rows of the sums
  }
  store_rows<DH>(dq, scale, smem + wave * out_strip_u4<DH>(), dqkv + ((int64_t)n * s + iw0) * ld + head * dh, ld, kg == 0 ? s - iw0 : 0, dh, lane);
  return false;
}
template <int DH, int NW, int KSPL, bool ANY>
__global__ __launch_bounds__(NW * 64, 2) void attn_dq_mfma_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o, const float* __restrict__ lse, float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int a, int mask_mode, const int32_t* __restrict__ seqlens, float* __restrict__ colsum, int dh_) {
  const int nblk = gridDim.z, blk = mask_mode == 1 ? nblk - 1 - (int)blockIdx.z : (int)blockIdx.z;
  if (attn_dq<DH, NW, KSPL, ANY, false, true>(qkv, o, d_o, lse, delta, dqkv, s, a, mask_mode, seqlens, colsum, dh_, blk, nblk))
    if constexpr (ANY) attn_dq<DH, NW, KSPL, ANY, true, true>(qkv, o, d_o, lse, delta, dqkv, s, a, mask_mode, seqlens, colsum, dh_, blk, nblk);
}

// ------------------------------------------------------------------------------------------------
// dK, dV
// PART: 0 both results; 1 only dV, 2 only dK: a workgroup makes one of the two, at the price of the scores twice.  For heads of
// the ANY set from 72 on both accumulators, the split operands and the fragments do not fit in the registers (and a spill in the
// loop waits for the next tile's loads: backward at b=3 s=1000 a=16 causal, head size 96 119 -> 100 us, 72 145 -> 91); and launches
// that leave half of the CUs idle gain the second half's work (backward, 64-row blocks: b=1 s=1024 a=8 dh=64 30.2 -> 28.2 us,
// b=1 s=2048 a=4 causal 51.3 -> 47.4).
// OWN: delta comes from own_delta, LDS for as many floats as the sequence has rows, which the workgroup fills from dO and O while its
// first tile travels (a workgroup that only makes dV has no use for it); else from what the dQ kernel left in memory.
template <int DH, int NW, int KSPL, bool ANY, bool EXACT, int PART, bool OWN>
__device__ __forceinline__ bool attn_dkv(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o, const float* __restrict__ lse, const float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int a, int mask_mode, const int32_t* __restrict__ seqlens, float* __restrict__ colsum, int dh_, int blk, int nblk, float* own_delta) {
  using C = Cfg<DH>;
  extern __shared__ uint4 smem[];
  // stage st: Q tile, dO tile, 64 lse, 64 delta
  constexpr int kStageU4 = 2 * C::kTileU4 + 2 * kTile / 4;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  // grid = (heads, sequences, key blocks), key block slowest: under a causal mask the first keys are seen by
  // the most queries, and those workgroups are dispatched first (see the forward kernel)
  // (halves of the waves: see the forward kernel)
  constexpr int RW = NW / KSPL;
  const int kg = KSPL == 1 ? 0 : wave / RW, rw = KSPL == 1 ? wave : wave % RW;
  const int n = blockIdx.y, head = blockIdx.x;
  constexpr bool DV = PART != 2, DK = PART != 1;
  const int j0 = blk * RW * 32;
  const int dh = ANY ? dh_ : DH;
  const int h = a * dh;
  const int64_t ld = 3 * (int64_t)h;
  const bf16_t* base = qkv + (int64_t)n * s * ld + head * dh;
  const bf16_t* dobase = d_o + (int64_t)n * s * h + head * dh;
  const float* lse_row = lse + ((int64_t)n * a + head) * s;
  const float* delta_row = OWN ? nullptr : delta + ((int64_t)n * a + head) * s;
  const int kv_len = mask_mode == 2 ? min(max(seqlens[n], 1), s) : s;   // lengths outside [1, s] are clamped: no read past the sequence, no empty row
  const bool causal = mask_mode == 1;
  const int jw0 = j0 + rw * 32;
  const int j = jw0 + l32;
  const bool row_ok = j < s;
  const float scale = 1.0f / sqrtf((float)dh);
  const float c = scale * kLog2e;

  bf16x8 kf[C::KS], vf[C::KS];
  load_frags<DH, ANY>(base + h + (int64_t)j * ld, row_ok, hf, dh, kf);
  load_frags<DH, ANY>(base + 2 * h + (int64_t)j * ld, row_ok, hf, dh, vf);
  // At head size 128 the two accumulators are 128 registers and the K and V fragments of the wave's keys 64 more: with
  // the scores on top the kernel spilled.  There the V fragments wait in a wave-private piece of LDS (16 bytes per
  // lane and k-step, read back in the order written: no bank conflicts, no barrier) and are fetched per use.
  constexpr bool kVInLds = Cfg<DH, ANY>::kDkvVInLds && PART == 0;
  uint4* vstore = smem + 2 * kStageU4 + C::kPadU4 + wave * (C::KS * 64);
  if (kVInLds) {
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) vstore[ks * 64 + lane] = __builtin_bit_cast(uint4, vf[ks]);
  }
  f32x16 dk[C::DB], dv[C::DB];

  const bool wg_dead = j0 >= kv_len;                       // every key of the workgroup is padding
  const int istart = causal ? (j0 / kTile) * kTile : 0;    // earlier queries see none of these keys
  const int ntiles = wg_dead ? 0 : (s - istart + kTile - 1) / kTile;
  TileLoader<DH, ANY, RW> loader;
  loader.init(rw, lane, dh);
  auto issue_tile = [&](int i0, uint4* stage) {
    loader.issue(base, ld, i0, s, stage);
    loader.issue(dobase, (int64_t)h, i0, s, stage + C::kTileU4);
  };
  // lse and delta of the tile's queries travel through a register of two waves, which lets them enter LDS in the form the
  // loop uses: -lse * log2(e) (ANY: -lse), and -delta, the starting value of the accumulators of dP
  float stat = 0.f;
  auto load_stat = [&](int i0) {
    const int i = min(i0 + lane, s - 1);
    if constexpr (!OWN) {
      if (rw < 2) stat = (rw == 0 ? lse_row : delta_row)[i];
    } else if (rw == 0) {
      stat = lse_row[i];
    } else if (DK && rw == 1) {
      stat = own_delta[i];
    }
  };
  bool hidden = false;
#pragma unroll
  for (int db = 0; db < C::DB; ++db) { dk[db] = zero16(); dv[db] = zero16(); }
  uint4* const tiles = smem + kg * (2 * kStageU4 + C::kPadU4);
  if (kg < ntiles) issue_tile(istart + kg * kTile, tiles);
  if (OWN && DK && ntiles > 0) {   // (uniform) eight lanes per row, U rows in flight
    constexpr int NC = (C::CH + 7) / 8, U = NC == 1 ? 8 : 4;
    for (int r0 = istart + wave * 8; r0 < s; r0 += U * NW * 8) {
      bf16x8 x[U][NC], y[U][NC];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t at = ((int64_t)n * s + min(r0 + u * NW * 8 + (lane >> 3), s - 1)) * h + head * dh;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const int c8 = min(((lane & 7) + q * 8) * 8, dh - 8);   // (past the head: the last chunk, not counted below)
          x[u][q] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(d_o + at + c8));
          y[u][q] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(o + at + c8));
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int row = r0 + u * NW * 8 + (lane >> 3);
        float part = 0.f;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          float t = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) t = fmaf((float)x[u][q][e], (float)y[u][q][e], t);
          part += ((lane & 7) + q * 8) * 8 < dh ? t : 0.f;
        }
        part = row8_sum(part);
        if ((lane & 7) == 0 && row < s) own_delta[row] = part;
      }
    }
    __syncthreads();
  }
  if (kg < ntiles) load_stat(istart + kg * kTile);
  for (int st = 0; st * KSPL < ntiles; ++st) {
    const int t = st * KSPL + kg, i0 = istart + t * kTile;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    if (rw < 2) {
      float* f = reinterpret_cast<float*>(tiles + (st & 1) * kStageU4 + 2 * C::kTileU4);
      f[rw * kTile + lane] = rw == 0 && !ANY ? -kLog2e * stat : -stat;   // (the stage's readers were done before the last barrier)
    }
    __syncthreads();
    if (t + KSPL < ntiles) { load_stat(i0 + KSPL * kTile); issue_tile(i0 + KSPL * kTile, tiles + ((st + 1) & 1) * kStageU4); }
    if (KSPL > 1 && t >= ntiles) continue;
    const uint4* q_lds = tiles + (st & 1) * kStageU4;
    const uint4* do_lds = q_lds + C::kTileU4;
    const float* lse_lds = reinterpret_cast<const float*>(q_lds + 2 * C::kTileU4);
    const float* delta_lds = lse_lds + kTile;
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      const int ib = i0 + qb * 32;
      if (causal && ib + 31 < jw0) continue;   // all 32 queries lie before this wave's keys
      if (ib >= s) continue;                   // no query of the block exists
      f32x16 sacc = zero16(), dp;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 d4 = *reinterpret_cast<const float4*>(delta_lds + qb * 32 + 8 * g + 4 * hf);
        dp[4 * g] = d4.x; dp[4 * g + 1] = d4.y; dp[4 * g + 2] = d4.z; dp[4 * g + 3] = d4.w;
      }
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks) {
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows<DH>(q_lds, qb * 32 + l32, ks, hf), kf[ks], sacc, 0, 0, 0);
        const bf16x8 vfr = kVInLds ? __builtin_bit_cast(bf16x8, vstore[ks * 64 + lane]) : vf[ks];
        if (DK) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_rows<DH>(do_lds, qb * 32 + l32, ks, hf), vfr, dp, 0, 0, 0);
      }
      const bool need_mask = (jw0 + 32 > kv_len) || (causal && jw0 + 31 > ib) || (ib + 32 > s);
      uint32_t seen = 0;   // ANY: per register, whether the key sees the query
      if (need_mask) {   // a masked score of -inf gives probability exactly 0
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int iq = ib + 8 * (r >> 2) + 4 * hf + (r & 3);
          const bool vis = j < kv_len && (!causal || j <= iq) && iq < s;
          sacc[r] = vis ? sacc[r] : -INFINITY;
          if (ANY) seen |= vis ? 1u << r : 0u;
        }
      }
      f32x16 pv16, ds16;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 l4 = *reinterpret_cast<const float4*>(lse_lds + qb * 32 + 8 * g + 4 * hf);
        const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
          const int r = 4 * g + t4;
          const float pv = __builtin_amdgcn_exp2f(ANY ? fmaf(sacc[r], scale, lv[t4]) * kLog2e : fmaf(sacc[r], c, lv[t4]));
          pv16[r] = pv;
          ds16[r] = pv * dp[r];
        }
      }
      if constexpr (ANY) {
        if (need_mask) {   // P and dS of unseen pairs are zero whatever lse, delta, dO and V hold there
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            pv16[r] = (seen >> r) & 1 ? pv16[r] : 0.f;
            ds16[r] = (seen >> r) & 1 ? ds16[r] : 0.f;
          }
        }
        // (a key past the length sees no query at all: its lanes stay zero whatever the tile holds)
        if (need_mask) {
          if (EXACT) {
            auto sees = [&](int row) { return j < kv_len && i0 + row < s && (!causal || j <= i0 + row); };
            if (DV) accumulate_visible<DH>(do_lds, qb * 32, pv16, dv, lane, sees);
            if (DK) accumulate_visible<DH>(q_lds, qb * 32, ds16, dk, lane, sees);
            continue;
          }
          hidden = hidden || (DK && tile_not_finite<DH>(q_lds, lane)) || (DV && tile_not_finite<DH>(do_lds, lane));
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int kk = qb * 2 + half;
          if (DV) {
            const Exact8 pe = pack_half_exact(pv16, half);
#pragma unroll
            for (int db = 0; db < C::DB; ++db) mul_exact(read_cols<DH>(do_lds, db * 32, kk, lane), pe, dv[db]);
          }
          if (DK) {
            const Exact8 dse = pack_half_exact(ds16, half);
#pragma unroll
            for (int db = 0; db < C::DB; ++db) mul_exact(read_cols<DH>(q_lds, db * 32, kk, lane), dse, dk[db]);
          }
        }
      } else {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const bf16x8 pb = pack_half(pv16, half), dsb = pack_half(ds16, half);
          const int kk = qb * 2 + half;
#pragma unroll
          for (int db = 0; db < C::DB; ++db) {
            if (DV) dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_cols<DH>(do_lds, db * 32, kk, lane), pb, dv[db], 0, 0, 0);
            if (DK) dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_cols<DH>(q_lds, db * 32, kk, lane), dsb, dk[db], 0, 0, 0);
          }
        }
      }
    }
  }
  if constexpr (ANY && !EXACT)
    if (__syncthreads_or(hidden)) return true;
  __syncthreads();   // every wave is done with the Q / dO tiles
  if constexpr (KSPL == 2) {
    constexpr int kSlots = (DK + DV) * C::DB * 16;
    float* buf = reinterpret_cast<float*>(smem) + rw * (kSlots * 64);
    float* buf_v = buf + (DK ? C::DB * 16 * 64 : 0);
    if (kg == 1) {
      if (DK) { give<C::DB>(dk, buf, lane); clear<C::DB>(dk); }
      if (DV) { give<C::DB>(dv, buf_v, lane); clear<C::DB>(dv); }
    }
    __syncthreads();
    if (kg == 0) {
      if (DK) take<C::DB>(dk, buf, lane);
      if (DV) take<C::DB>(dv, buf_v, lane);
    }
    __syncthreads();
  }
  if (!ANY && colsum) {   // masked and non-existent keys hold zeros
    float* row = colsum + ((int64_t)n * nblk + blk) * ld + head * dh;
    float* red = reinterpret_cast<float*>(smem);
    if (DK) {
      block_column_sums<DH, NW>(dk, scale, red, row + h, tid, lane, wave);
      __syncthreads();
    }
    if (DV) {
      block_column_sums<DH, NW>(dv, 1.0f, red, row + 2 * h, tid, lane, wave);
      __syncthreads();
    }
  }
  bf16_t* outk = dqkv + ((int64_t)n * s + jw0) * ld + h + head * dh;
  uint4* strip = smem + wave * out_strip_u4<DH>();
  if (DK) store_rows<DH>(dk, scale, strip, outk, ld, kg == 0 ? s - jw0 : 0, dh, lane);
  if (DV) store_rows<DH>(dv, 1.0f, strip, outk + h, ld, kg == 0 ? s - jw0 : 0, dh, lane);
  return false;
}
template <int DH, int NW, int KSPL, bool ANY, bool PARTS>
__global__ __launch_bounds__(NW * 64, 2) void attn_dkv_mfma_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ d_o, const float* __restrict__ lse, const float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int a, int mask_mode, const int32_t* __restrict__ seqlens, float* __restrict__ colsum, int dh_) {
  const int nblk = gridDim.z >> (PARTS ? 1 : 0), blk = blockIdx.z >> (PARTS ? 1 : 0);
  auto run = [&](auto part) __attribute__((always_inline)) {
    constexpr int PART = decltype(part)::value;
    if (attn_dkv<DH, NW, KSPL, ANY, false, PART, false>(qkv, nullptr, d_o, lse, delta, dqkv, s, a, mask_mode, seqlens, colsum, dh_, blk, nblk, nullptr))
      if constexpr (ANY) attn_dkv<DH, NW, KSPL, ANY, true, PART, false>(qkv, nullptr, d_o, lse, delta, dqkv, s, a, mask_mode, seqlens, colsum, dh_, blk, nblk, nullptr);
  };
  if constexpr (!PARTS) run(std::integral_constant<int, 0>{});
  else if (blockIdx.z & 1) run(std::integral_constant<int, 1>{});
  else run(std::integral_constant<int, 2>{});
}

// The whole backward pass in one launch.  Of every kRoles consecutive block numbers one has queries (causal: the blocks with the most
// keys first), the others keys, so the longest workgroups of every kind go first.  Nothing is handed from one to another: dK/dV form
// their deltas themselves, in LDS at delta_at.
template <int DH, int NW, int KSPL, bool ANY, bool PARTS>
__global__ __launch_bounds__(NW * 64, 2) void attn_bwd_mfma_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o, const float* __restrict__ lse, bf16_t* __restrict__ dqkv, int s, int a, int mask_mode, const int32_t* __restrict__ seqlens, float* __restrict__ colsum, int dh_, int delta_at) {
  extern __shared__ uint4 smem[];
  constexpr int kRoles = PARTS ? 3 : 2;
  const int nblk = gridDim.z / kRoles, k = blockIdx.z / kRoles, role = blockIdx.z % kRoles;
  float* own_delta = reinterpret_cast<float*>(smem + delta_at);
  auto run = [&](auto part) __attribute__((always_inline)) {
    constexpr int PART = decltype(part)::value;
    if (attn_dkv<DH, NW, KSPL, ANY, false, PART, true>(qkv, o, d_o, lse, nullptr, dqkv, s, a, mask_mode, seqlens, colsum, dh_, k, nblk, own_delta))
      if constexpr (ANY) attn_dkv<DH, NW, KSPL, ANY, true, PART, true>(qkv, o, d_o, lse, nullptr, dqkv, s, a, mask_mode, seqlens, colsum, dh_, k, nblk, own_delta);
  };
  if (role == kRoles - 1) {
    const int blk = mask_mode == 1 ? nblk - 1 - k : k;
    if (attn_dq<DH, NW, KSPL, ANY, false, false>(qkv, o, d_o, lse, nullptr, dqkv, s, a, mask_mode, seqlens, colsum, dh_, blk, nblk))
      if constexpr (ANY) attn_dq<DH, NW, KSPL, ANY, true, false>(qkv, o, d_o, lse, nullptr, dqkv, s, a, mask_mode, seqlens, colsum, dh_, blk, nblk);
  } else if constexpr (!PARTS) {
    run(std::integral_constant<int, 0>{});
  } else if (role == 1) {
    run(std::integral_constant<int, 1>{});
  } else {
    run(std::integral_constant<int, 2>{});
  }
}

template <typename K>
hipError_t set_lds(K kern, size_t bytes, bool* done) {
  if (*done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)bytes);
  if (e == hipSuccess) *done = true;
  return e;
}

constexpr size_t max_of(size_t a, size_t b) { return a > b ? a : b; }

// LDS of the two kernels, in bytes
template <int DH, int NW, int KSPL>
constexpr size_t dq_lds() {
  using C = Cfg<DH>;
  constexpr size_t out = (size_t)NW * out_strip_u4<DH>() * sizeof(uint4);   // the output strips re-use the tiles' LDS
  constexpr size_t merge = KSPL == 1 ? 0 : NW / KSPL * C::DB * 16 * 64 * sizeof(float);   // ... and so do the halves' results
  return max_of(max_of(KSPL * (4 * C::kTileU4 + C::kPadU4) * sizeof(uint4), out), merge);
}
template <int DH, int NW, int KSPL, bool ANY, bool PARTS>
constexpr size_t dkv_lds() {
  using C = Cfg<DH>;
  constexpr size_t out = (size_t)NW * out_strip_u4<DH>() * sizeof(uint4);
  constexpr size_t merge = KSPL == 1 ? 0 : NW / KSPL * (PARTS ? 1 : 2) * C::DB * 16 * 64 * sizeof(float);
  constexpr size_t tiles = (KSPL * (2 * (2 * C::kTileU4 + 2 * kTile / 4) + C::kPadU4) + (!PARTS && Cfg<DH, ANY>::kDkvVInLds ? NW * C::KS * 64 : 0)) * sizeof(uint4);
  return max_of(max_of(tiles, out), merge);
}

template <int DH, int NW, int KSPL, bool ANY>
hipError_t fwd_launch(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) {
  using C = Cfg<DH>;
  constexpr size_t lds_out = (size_t)NW * out_strip_u4<DH>() * sizeof(uint4);   // the output strips re-use the tiles' LDS
  constexpr size_t lds_merge = KSPL == 1 ? 0 : NW / KSPL * (C::DB * 16 + 2) * 64 * sizeof(float);   // ... and so do the halves' results
  constexpr size_t lds = max_of(max_of(KSPL * (4 * C::kTileU4 + C::kPadU4) * sizeof(uint4), lds_out), lds_merge);
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  constexpr int kPerCu = NW == 4 ? (DH <= 32 ? 4 : DH <= 64 ? 2 : 1) : DH <= (ANY ? 32 : 64) ? 2 : 1;   // workgroups, by registers and LDS
  static bool done = false;
  hipError_t e = set_lds(attn_fwd_mfma_kernel<DH, NW, KSPL, ANY>, lds, &done);
  if (e != hipSuccess) return e;
  dim3 grid(d.a, d.b, ceil_div(d.s, NW / KSPL * 32));
  hipLaunchKernelGGL((attn_fwd_mfma_kernel<DH, NW, KSPL, ANY>), grid, dim3(NW * 64), lds, st, static_cast<const bf16_t*>(qkv),
                     static_cast<bf16_t*>(o), lse, d.s, d.a, d.mask_mode, d.seqlens, d.dh,
                     fold_of(d, grid.z, kPerCu));
  return hipGetLastError();
}

template <int DH, int NW, int KSPL, bool ANY, bool PARTS>
hipError_t dkv_launch(const AttnDesc& d, const void* qkv, const float* lse, const void* d_o, void* dqkv, const float* delta, hipStream_t st) {
  constexpr size_t lds = dkv_lds<DH, NW, KSPL, ANY, PARTS>();
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  hipError_t e = set_lds(attn_dkv_mfma_kernel<DH, NW, KSPL, ANY, PARTS>, lds, &done);
  if (e != hipSuccess) return e;
  dim3 grid(d.a, d.b, ceil_div(d.s, NW / KSPL * 32) * (PARTS ? 2 : 1));
  hipLaunchKernelGGL((attn_dkv_mfma_kernel<DH, NW, KSPL, ANY, PARTS>), grid, dim3(NW * 64), lds, st, static_cast<const bf16_t*>(qkv),
                     static_cast<const bf16_t*>(d_o), lse, delta, static_cast<bf16_t*>(dqkv), d.s, d.a, d.mask_mode,
                     d.seqlens, d.colsum_partial, d.dh);
  return hipGetLastError();
}

// Whether `wgs` workgroups of both halves together go out in one launch, which spares a launch and its tail but makes dK/dV's
// workgroups form the deltas they need (their rows of dO and O: some 3 us at 600 rows): where they all run at once, or under a causal
// mask, whose blocks differ, one and a half times as many.  One over two launches by wgs over what the CUs hold at once, no mask |
// causal | lengths: up to 0.5 0.65 | 0.64 | 0.65, to 1 0.69 | 0.66 | 0.68, to 1.25 0.84 (at worst 1.04) | 0.82 | 0.91 (1.33), to 1.5
// 1.05 (1.37) | 0.79 | 0.96 (1.23), to 3 0.92 (1.2) | 0.91 (1.08) | 0.95 (1.29).  By this rule 600 random calls take 0.715 of the time
// with two launches always, none more than 1.03.
template <int DH, int NW, bool ANY>
bool one_launch(const AttnDesc& d, int64_t wgs) {
  constexpr bool kSmall = DH == 32 && !ANY;                                        // 128 registers
  constexpr int kPerCu = NW == 4 ? (kSmall ? 4 : DH <= 64 ? 2 : 1) : (kSmall ? 2 : 1);   // by registers and LDS
  return d.s <= kMaxDeltas && 2 * wgs <= (d.mask_mode == 1 ? 3 : 2) * kPerCu * (int64_t)gemm_compute_units();
}

// Both halves of the backward pass in one launch
template <int DH, int NW, int KSPL, bool ANY, bool PARTS>
hipError_t both_launch(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, hipStream_t st) {
  constexpr size_t base = max_of(dq_lds<DH, NW, KSPL>(), dkv_lds<DH, NW, KSPL, ANY, PARTS>());
  const size_t lds = base + ceil_div(d.s, 4) * sizeof(uint4);
  static bool done = false;
  hipError_t e = set_lds(attn_bwd_mfma_kernel<DH, NW, KSPL, ANY, PARTS>, base + kMaxDeltas * sizeof(float), &done);
  if (e != hipSuccess) return e;
  static_assert(base + kMaxDeltas * sizeof(float) <= 160 * 1024, "LDS of a CU");
  dim3 grid(d.a, d.b, ceil_div(d.s, NW / KSPL * 32) * (PARTS ? 3 : 2));
  hipLaunchKernelGGL((attn_bwd_mfma_kernel<DH, NW, KSPL, ANY, PARTS>), grid, dim3(NW * 64), lds, st, static_cast<const bf16_t*>(qkv), static_cast<const bf16_t*>(o),
                     static_cast<const bf16_t*>(d_o), lse, static_cast<bf16_t*>(dqkv), d.s, d.a, d.mask_mode, d.seqlens, d.colsum_partial, d.dh,
                     (int)(base / sizeof(uint4)));
  return hipGetLastError();
}

template <int DH, int NW, int KSPL, bool ANY>
hipError_t bwd_launch(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                      float* delta, hipStream_t st) {
  // (two sets of tiles and the V fragments of head size 128 do not fit in LDS together)
  constexpr bool kAlways = Cfg<DH, ANY>::kDkvParts || (KSPL == 2 && Cfg<DH, ANY>::kDkvVInLds), kMay = kAlways || (NW == 4 && KSPL == 2);
  // few blocks: dK and dV in workgroups of their own (see attn_dkv)
  const int64_t blocks = (int64_t)d.a * d.b * ceil_div(d.s, NW / KSPL * 32);
  const bool parts = kAlways || (kMay && 2 * blocks <= gemm_compute_units());
  if (one_launch<DH, NW, ANY>(d, blocks * (parts ? 3 : 2)))
    return parts ? both_launch<DH, NW, KSPL, ANY, kMay>(d, qkv, o, lse, d_o, dqkv, st) : both_launch<DH, NW, KSPL, ANY, kAlways>(d, qkv, o, lse, d_o, dqkv, st);
  constexpr size_t lds = dq_lds<DH, NW, KSPL>();
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  hipError_t e = set_lds(attn_dq_mfma_kernel<DH, NW, KSPL, ANY>, lds, &done);
  if (e != hipSuccess) return e;
  dim3 grid(d.a, d.b, ceil_div(d.s, NW / KSPL * 32));
  hipLaunchKernelGGL((attn_dq_mfma_kernel<DH, NW, KSPL, ANY>), grid, dim3(NW * 64), lds, st, static_cast<const bf16_t*>(qkv),
                     static_cast<const bf16_t*>(o), static_cast<const bf16_t*>(d_o), lse, delta,
                     static_cast<bf16_t*>(dqkv), d.s, d.a, d.mask_mode, d.seqlens, d.colsum_partial, d.dh);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return parts ? dkv_launch<DH, NW, KSPL, ANY, kMay>(d, qkv, lse, d_o, dqkv, delta, st) : dkv_launch<DH, NW, KSPL, ANY, kAlways>(d, qkv, lse, d_o, dqkv, delta, st);
}

// F<DH, NW, KSPL, ANY>::run for the head size of a call
template <template <int, int, int, bool> class F, int NW, int KSPL, typename... Args>
hipError_t by_head(const AttnDesc& d, Args... args) {
  switch (d.dh) {
    case 32: return F<32, NW, KSPL, false>::run(d, args...);
    case 64: return F<64, NW, KSPL, false>::run(d, args...);
    case 80: return F<80, NW, KSPL, false>::run(d, args...);
    case 128: return F<128, NW, KSPL, false>::run(d, args...);
  }
  if (d.dh < 32) return F<32, NW, KSPL, true>::run(d, args...);
  if (d.dh <= 48) return F<48, NW, KSPL, true>::run(d, args...);
  if (d.dh < 64) return F<64, NW, KSPL, true>::run(d, args...);
  if (d.dh < 80) return F<80, NW, KSPL, true>::run(d, args...);
  if (d.dh <= 96) return F<96, NW, KSPL, true>::run(d, args...);
  if (d.dh <= 112) return F<112, NW, KSPL, true>::run(d, args...);
  return F<128, NW, KSPL, true>::run(d, args...);
}
template <int DH, int NW, int KSPL, bool ANY>
struct Fwd {
  static hipError_t run(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) { return fwd_launch<DH, NW, KSPL, ANY>(d, qkv, o, lse, st); }
};
template <int DH, int NW, int KSPL, bool ANY>
struct Bwd {
  static hipError_t run(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta, hipStream_t st) {
    return bwd_launch<DH, NW, KSPL, ANY>(d, qkv, o, lse, d_o, dqkv, delta, st);
  }
};
}  // namespace
}  // namespace k2bw
