// Pieces shared by the GSTA kernels that give a workgroup 1 to 16 pairs (gsta_tiled.hip forward, gsta_backward_tile.hip): rows
// of H' in registers, reductions over the lane groups of a wave, and the products of a tile of 16 pairs with a wave's 16
// columns of a matrix.
#pragma once

#include "laser_internal.h"
#include "sta_mfma_tile.h"

namespace laser {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Row8;
template <> struct Row8<unsigned short> {
  u32x4 x;
  __device__ __forceinline__ void load(const unsigned short* p) { x = *reinterpret_cast<const u32x4*>(p); }
  // keeps the compiler from unpacking a block once for all layers, ahead of the first product: twice the registers, and a
  // wait for the whole block where the chain of products could already run
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(x)); }
  __device__ __forceinline__ float get(int e) const {   // (e is a constant after unrolling)
    return __uint_as_float((e & 1) ? (x[e >> 1] & 0xffff0000u) : (x[e >> 1] << 16));
  }
};
template <> struct Row8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4*>(p);
    b = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ void pin() {}
  __device__ __forceinline__ float get(int e) const { return e < 4 ? a[e] : b[e - 4]; }
};

// sum (or maximum) over the 64 / LPR lane groups of a wave, in every lane
template <int LPR, bool MAX>
__device__ __forceinline__ float over_groups(float x) {
  auto both = [](float a, float b) { return MAX ? fmaxf(a, b) : a + b; };
  if (LPR == 8) x = both(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false)));  // row_ror:8
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = both(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return both(__uint_as_float(s[0]), __uint_as_float(s[1]));
}

// What an online softmax subtracts from its scores when the largest so far is m: scores of -inf alone (or none) then have
// weight zero without a difference of infinities, and one of NaN or +inf gives NaN.
__device__ __forceinline__ float softmax_ref(float m) { return m == -INFINITY ? 0.0f : m; }

// Per storage type: the left operand's tile in LDS (16 pairs x D values of fp32 meaning), a wave's share of a matrix, and
// the product of the two.
template <typename T, int D> struct Prod;

template <int D> struct Prod<float, D> {
  static constexpr int PITCH = D + 4;                       // 16 bytes past a multiple of 256: conflict-free row reads
  struct Act { float v[16 * PITCH]; };
  static constexpr int NCOL = D / 16;                       // 16-byte pieces of a wave's 16 columns per lane
  struct Cols { f32x4 x[NCOL]; };                           // rows 16 it + lane / 4, columns n0 + 4 (lane % 4) ..
  struct Operand { f32x4 x[D / 16]; };                      // column n of the product, k = 16 j + 4 g ..
  static constexpr int PATCH = D * 16 * 4;
  static __device__ __forceinline__ float ex(float x) { return expf(x); }
  static constexpr float LOG = 1.0f;                        // scores enter ex() in this base's units
  static __device__ __forceinline__ void put(Act& a, int pair, int col, float x) { a.v[pair * PITCH + col] = x; }
  static __device__ __forceinline__ void load_cols(Cols& c, const float* W, int n0, int lane) {
#pragma unroll
    for (int it = 0; it < NCOL; ++it)
      c.x[it] = *reinterpret_cast<const f32x4*>(W + (size_t)(it * 16 + (lane >> 2)) * D + n0 + (lane & 3) * 4);
  }
  static __device__ __forceinline__ void load_rows(Operand& r, const float* W, int n0, int lane) {
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
      r.x[j] = *reinterpret_cast<const f32x4*>(W + (size_t)(n0 + (lane & 15)) * D + j * 16 + (lane >> 4) * 4);
  }
  static __device__ __forceinline__ Operand transposed(const Cols& c, unsigned char* patch, int lane) {
    float* p = reinterpret_cast<float*>(patch);             // [D][16]
#pragma unroll
    for (int it = 0; it < NCOL; ++it) *reinterpret_cast<f32x4*>(p + it * 256 + lane * 4) = c.x[it];
    __builtin_amdgcn_wave_barrier();                        // (LDS operations of a wave execute in order)
    Operand o;
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
      for (int m = 0; m < 4; ++m) o.x[j][m] = p[(j * 16 + (lane >> 4) * 4 + m) * 16 + (lane & 15)];
    __builtin_amdgcn_wave_barrier();
    return o;
  }
  static __device__ __forceinline__ f32x4 product(const Act& a, const Operand& w, int lane) {
    f32x4 s[4];                                             // independent sums: the chain is a fourth as long
#pragma unroll
    for (int m = 0; m < 4; ++m) s[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < D / 16; ++j) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(a.v + (lane & 15) * PITCH + j * 16 + (lane >> 4) * 4);
#pragma unroll
      for (int m = 0; m < 4; ++m) s[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[m], w.x[j][m], s[m], 0, 0, 0);
    }
    return (s[0] + s[1]) + (s[2] + s[3]);
  }
};

template <int D> struct Prod<unsigned short, D> {
  static constexpr int PITCH = D + 8;
  struct Act { unsigned short v[3][16 * PITCH]; };          // head, remainder, remainder of that
  static constexpr int NCOL = D / 32;
  struct Cols { u32x4 x[NCOL]; };                           // rows 32 it + lane / 2, columns n0 + 8 (lane % 2) ..
  struct Operand { bf16x8 x[D / 32]; };                     // column n of the product, k = 32 s + 8 g ..
  static constexpr int PATCH = D * 16 * 2;
  static __device__ __forceinline__ float ex(float x) { return __builtin_amdgcn_exp2f(x); }
  static constexpr float LOG = 1.4426950408889634f;
  static __device__ __forceinline__ void put(Act& a, int pair, int col, float x) {
    const unsigned short h0 = f32_to_bf16_bits(x);
    const float r1 = x - bf16_bits_to_f32(h0);
    const unsigned short h1 = f32_to_bf16_bits(r1);
    a.v[0][pair * PITCH + col] = h0;
    a.v[1][pair * PITCH + col] = h1;
    a.v[2][pair * PITCH + col] = f32_to_bf16_bits(r1 - bf16_bits_to_f32(h1));
  }
  static __device__ __forceinline__ void load_cols(Cols& c, const unsigned short* W, int n0, int lane) {
#pragma unroll
    for (int it = 0; it < NCOL; ++it)
      c.x[it] = *reinterpret_cast<const u32x4*>(W + (size_t)(it * 32 + (lane >> 1)) * D + n0 + (lane & 1) * 8);
  }
  static __device__ __forceinline__ void load_rows(Operand& r, const unsigned short* W, int n0, int lane) {
#pragma unroll
    for (int s = 0; s < D / 32; ++s)
      r.x[s] = *reinterpret_cast<const bf16x8*>(W + (size_t)(n0 + (lane & 15)) * D + s * 32 + (lane >> 4) * 8);
  }
  static __device__ __forceinline__ Operand transposed(const Cols& c, unsigned char* patch, int lane) {
#pragma unroll
    for (int it = 0; it < NCOL; ++it) *reinterpret_cast<u32x4*>(patch + it * 1024 + lane * 16) = c.x[it];   // [D][16]
    __builtin_amdgcn_wave_barrier();
    Operand o;
#pragma unroll
    for (int k = 0; k < D / 32; ++k) {
      // transpose load: lane i of a 16-lane group supplies the address of row i / 4, columns 4 (i % 4) .. and receives
      // column i of four rows
      const unsigned char* src = patch + (k * 32 + (lane >> 4) * 8 + ((lane & 15) >> 2)) * 32 + (lane & 3) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src + 128));
      o.x[k] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
    __builtin_amdgcn_wave_barrier();
    return o;
  }
  static __device__ __forceinline__ f32x4 product(const Act& a, const Operand& w, int lane) {
    f32x4 s[3];                                             // independent sums: the chain is a third as long
#pragma unroll
    for (int p = 0; p < 3; ++p) s[p] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < D / 32; ++k)
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(a.v[p] + (lane & 15) * PITCH + k * 32 + (lane >> 4) * 8);
        s[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, w.x[k], s[p], 0, 0, 0);
      }
    return (s[2] + s[1]) + s[0];
  }
};

}  // namespace laser
