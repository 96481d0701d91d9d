// Pieces shared by the GSTA kernels that give a workgroup 1 to 16 pairs (gsta_tiled.hip forward, gsta_backward_tile.hip): rows
// of H' in registers, reductions over the lane groups of a wave, and the products of a tile of 16 pairs with a wave's 16
// columns of a matrix.
#pragma once

#include <type_traits>

#include "laser_internal.h"
#include "sta_mfma_tile.h"

namespace laser {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

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

// Sums of eight values over the 64 / LPR lane groups of a wave, dealt out over the groups: lane group `grp` ends with x[0 ..
// 8 LPR / 64 - 1] = the sums of elements group_first(lane) .. (7 exchanges where every lane getting every sum takes 24)
template <int LPR>
__device__ __forceinline__ int group_first(int lane) {
  return LPR == 16 ? ((lane >> 5) * 4 + ((lane >> 4) & 1) * 2) : ((lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1));
}
template <int LPR>
__device__ __forceinline__ void scatter_over_groups(float (&x)[8], int lane) {
  static_assert(LPR == 8 || LPR == 16, "8 elements a lane, d = 64 or 128");
#pragma unroll
  for (int e = 0; e < 4; ++e) {   // the lower half of the wave keeps element e, the upper e + 4
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[e]), __float_as_uint(x[e + 4]), false, false);
    x[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {   // rows of 16 lanes in pairs
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[e]), __float_as_uint(x[e + 2]), false, false);
    x[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  if (LPR == 8) {
    const bool odd = lane & 8;
    const float keep = odd ? x[1] : x[0], send = odd ? x[0] : x[1];
    x[0] = keep + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0x128, 0xf, 0xf, false));  // row_ror:8
  }
}

// sum (or maximum) over the lanes l, l + PW, l + 2 PW .. below N (4 or 8) of 16, for l below PW; what other lanes hold is not read
template <int PW, int N, bool MAX>
__device__ __forceinline__ float over_waves(float x) {
  auto step = [](float v, auto ctrl) {
    const float o = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, false));
    return MAX ? fmaxf(v, o) : v + o;
  };
  if (PW <= 1) x = step(x, std::integral_constant<int, 0xB1>{});              // quad_perm [1,0,3,2]
  if (PW <= 2) x = step(x, std::integral_constant<int, 0x4E>{});              // quad_perm [2,3,0,1]
  if (PW <= 4 && N == 8) x = step(x, std::integral_constant<int, 0x12C>{});   // row_ror:12: lane + 4
  return x;
}

// What an online softmax subtracts from its scores when the largest so far is m: scores of -inf alone (or none) then have
// weight zero without a difference of infinities, and one of NaN or +inf gives NaN.
__device__ __forceinline__ float softmax_ref(float m) { return m == -INFINITY ? 0.0f : m; }

// Per storage type: the tile's vectors in LDS (16 pairs x D values of fp32 meaning), a wave's share of a matrix (16 columns),
// and the product of the two, with the matrix as the left operand: lane (l16, g) gets columns n0 + 4 g .. + 3 of pair l16,
// which go to LDS, and to and from memory, as one piece (the other way round, four pairs of one column, every vector took twelve
// two-byte writes where three of eight bytes do). Matrices and rows are addressed by a uniform base and an unsigned 32-bit lane
// offset: 64-bit lane addresses, kept over the layers, spilled at d = 128 in fp32.
template <typename T, int D> struct Prod;

template <int D> struct Prod<float, D> {
  static constexpr int PITCH = D + 4;                       // 16 bytes past a multiple of 256
  struct Act { float v[16 * PITCH]; };
  template <int PW> static constexpr bool turned() { return false; }
  static constexpr int NCOL = D / 16;                       // 16-byte pieces of a wave's 16 columns per lane
  struct Cols { f32x4 x[NCOL]; };                           // rows 16 it + lane / 4, columns n0 + 4 (lane % 4) ..
  struct Operand { f32x4 x[D / 16]; };                      // column n of the product, k = 16 j + 4 g ..
  static constexpr int PATCH = D * 16 * 4;
  static __device__ __forceinline__ float ex(float x) { return expf(x); }
  static constexpr float LOG = 1.0f;                        // scores enter ex() in this base's units
  template <int PW, bool TURN = false> static __device__ __forceinline__ void put(Act& a, int pair, int col, float x) {   // (<>: see below)
    a.v[pair * PITCH + col] = x;
  }
  template <int PW, bool TURN = false> static __device__ __forceinline__ void put4(Act& a, int pair, int col, const f32x4& x) {
    *reinterpret_cast<f32x4*>(a.v + pair * PITCH + col) = x;
  }
  typedef f32x4 Raw4;                                       // four stored values
  static __device__ __forceinline__ f32x4 wide4(const Raw4& x) { return x; }
  static __device__ __forceinline__ void load_cols(Cols& c, const float* W, int n0, int lane) {
#pragma unroll
    for (int it = 0; it < NCOL; ++it)
      c.x[it] = *reinterpret_cast<const f32x4*>(W + it * 16 * D + n0 + (unsigned)((lane >> 2) * D + (lane & 3) * 4));
  }
  static __device__ __forceinline__ void load_rows(Operand& r, const float* W, int n0, int lane) {
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
      r.x[j] = *reinterpret_cast<const f32x4*>(W + n0 * D + j * 16 + (unsigned)((lane & 15) * D + (lane >> 4) * 4));
  }
  static __device__ __forceinline__ Operand transposed(const Cols& c, unsigned char* patch, int lane) {
    // [D][16], row r of 64 bytes at place (r + r / 4) % 4 of its four rows: the four rows of a piece written at once, and the
    // rows r, r + 4, r + 8, r + 12 read at once, are in different banks
    float* p = reinterpret_cast<float*>(patch);
    const int place = ((lane >> 4) * 4 + (((lane >> 2) + (lane >> 4)) & 3)) * 16 + (lane & 3) * 4;
#pragma unroll
    for (int it = 0; it < NCOL; ++it) *reinterpret_cast<f32x4*>(p + it * 256 + place) = c.x[it];
    __builtin_amdgcn_wave_barrier();                        // (LDS operations of a wave execute in order)
    Operand o;
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
      for (int m = 0; m < 4; ++m) o.x[j][m] = p[j * 256 + ((lane >> 4) * 4 + ((m + (lane >> 4)) & 3)) * 16 + (lane & 15)];
    __builtin_amdgcn_wave_barrier();
    return o;
  }
  template <int PW, bool TURN = false>
  static __device__ __forceinline__ f32x4 product(const Act& a, const Operand& w, int lane) {
    f32x4 s[4];                                             // independent sums: the chain is a fourth as long
#pragma unroll
    for (int m = 0; m < 4; ++m) s[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < D / 16; ++j) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(a.v + (lane & 15) * PITCH + j * 16 + (lane >> 4) * 4);
#pragma unroll
      for (int m = 0; m < 4; ++m) s[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x[j][m], x[m], s[m], 0, 0, 0);
    }
    return (s[0] + s[1]) + (s[2] + s[3]);
  }
};

template <int D> struct Prod<unsigned short, D> {
  // pairs whose parts a product reads side by side (see there)
  template <int PW> static constexpr int side_by_side() { return PW <= 4 ? 4 : (PW <= 8 ? 8 : 16); }
  // whether a piece's number is turned over by its row (see `at`)
  template <int PW> static constexpr bool turned() { return PW > 4 && D == 128; }
  // Place of a part (head, remainder, remainder of that) of a pair's column; <PW>: of the product that will read it, whose lanes'
  // rows are N part + pair. With few pairs (TURN false) the parts are 128 and 320 bytes past a multiple of 256 from each other,
  // rows padded: four rows of three parts read at once are in different banks. From eight on, d = 128, rows have no padding and a
  // 16-byte piece sits at its own number with bits turned over by its row: a read of 16 bytes a lane is served for rows 0 - 3 and
  // 12 - 15 of one lane group together with rows 4 - 11 of the next, which reads the next piece, and whatever the row pitch, two
  // of them met in a bank (4096 pairs, S = 16, d = 128 8.48 -> 8.20 us, 1450 packed pairs, S = 31 10.41 -> 10.13, the backward
  // pass of 2048 pairs 38.5 -> 38.1; one to four pairs were 1.5 % slower with it for the longer addresses, fp32 1 %, d = 64 the
  // same).
  static constexpr int PITCH = D + 8;
  static constexpr int PART[3] = {0, 16 * PITCH + 64, 32 * PITCH + 160};
  struct Act { unsigned short v[48 * PITCH + 160]; };
  template <int PW, bool TURN = turned<PW>()> static constexpr __device__ __forceinline__ int at(int part, int pair, int col) {
    if constexpr (!TURN) return PART[part] + pair * PITCH + col;
    const int row = (pair + part * side_by_side<PW>()) & 15;
    return (part * 16 + pair) * D + (((col >> 3) ^ row) << 3) + (col & 7);
  }
  // shorts that an array needs to hold the first `parts` parts of 16 pairs: one more than their largest place
  template <int PW, bool TURN = turned<PW>()> static constexpr __device__ int extent(int parts) {
    int last = 0;
    for (int part = 0; part < parts; ++part)
      for (int pair = 0; pair < 16; ++pair)
        for (int col = 0; col < D; ++col) last = at<PW, TURN>(part, pair, col) > last ? at<PW, TURN>(part, pair, col) : last;
    return last + 1;
  }
  static constexpr int NCOL = D / 32;
  struct Cols { u32x4 x[NCOL]; };                           // rows 32 it + lane / 2, columns n0 + 8 (lane % 2) ..
  struct Operand { bf16x8 x[D / 32]; };                     // column n of the product, k = 32 s + 8 g ..
  static constexpr int PATCH = D * 16 * 2;
  static __device__ __forceinline__ float ex(float x) { return __builtin_amdgcn_exp2f(x); }
  static constexpr float LOG = 1.4426950408889634f;
  template <int PW, bool TURN = turned<PW>()> static __device__ __forceinline__ void put(Act& a, int pair, int col, float x) {
    const unsigned short h0 = f32_to_bf16_bits(x);
    const float r1 = x - bf16_bits_to_f32(h0);
    const unsigned short h1 = f32_to_bf16_bits(r1);
    a.v[at<PW, TURN>(0, pair, col)] = h0;
    a.v[at<PW, TURN>(1, pair, col)] = h1;
    a.v[at<PW, TURN>(2, pair, col)] = f32_to_bf16_bits(r1 - bf16_bits_to_f32(h1));
  }
  template <int PW, bool TURN = turned<PW>()> static __device__ __forceinline__ void put4(Act& a, int pair, int col, f32x4 x) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const bf16x4 b = {(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
      *reinterpret_cast<bf16x4*>(a.v + at<PW, TURN>(p, pair, col)) = b;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] -= (float)b[e];
    }
  }
  typedef u32x2 Raw4;                                       // four stored values
  static __device__ __forceinline__ f32x4 wide4(const Raw4& x) {
    const bf16x4 b = __builtin_bit_cast(bf16x4, x);
    return f32x4{(float)b[0], (float)b[1], (float)b[2], (float)b[3]};
  }
  static __device__ __forceinline__ void load_cols(Cols& c, const unsigned short* W, int n0, int lane) {
#pragma unroll
    for (int it = 0; it < NCOL; ++it)
      c.x[it] = *reinterpret_cast<const u32x4*>(W + it * 32 * D + n0 + (unsigned)((lane >> 1) * D + (lane & 1) * 8));
  }
  static __device__ __forceinline__ void load_rows(Operand& r, const unsigned short* W, int n0, int lane) {
#pragma unroll
    for (int s = 0; s < D / 32; ++s)
      r.x[s] = *reinterpret_cast<const bf16x8*>(W + n0 * D + s * 32 + (unsigned)((lane & 15) * D + (lane >> 4) * 8));
  }
  static __device__ __forceinline__ Operand transposed(const Cols& c, unsigned char* patch, int lane) {
    // [D][16], the halves of every second eight rows swapped: lane groups 0 and 1, and 2 and 3, read from different banks
#pragma unroll
    for (int it = 0; it < NCOL; ++it) *reinterpret_cast<u32x4*>(patch + it * 1024 + ((lane * 16) ^ ((lane & 16) << 3))) = c.x[it];
    __builtin_amdgcn_wave_barrier();
    Operand o;
#pragma unroll
    for (int k = 0; k < D / 32; ++k) {
      // transpose load: lane i of a 16-lane group supplies the address of row i / 4, columns 4 (i % 4) .. and receives
      // column i of four rows
      const unsigned char* src = patch + (k * 32 + (lane >> 4) * 8 + ((lane & 15) >> 2)) * 32 + (lane & 3) * 8;
      const int swap = (lane & 16) << 3;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src + swap));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src + (128 ^ swap)));
      o.x[k] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
    __builtin_amdgcn_wave_barrier();
    return o;
  }
  // With few pairs their parts share an operand's 16 columns: up to four pairs column 4 part + pair of one operand instead of three,
  // up to eight the first two parts at 8 part + pair. Every wave of the workgroup reads the whole tile, at d = 128 a product is
  // bound by these LDS reads (12, 8 or 4 of 16 bytes a lane; PW = 1 6.6 -> 5.9 us a layer). The parts meet by lane rotations;
  // lanes of pairs past PW hold no result.
  template <int PW, bool TURN = turned<PW>()>
  static __device__ __forceinline__ f32x4 product(const Act& a, const Operand& w, int lane) {
    auto from = [](float v, auto ctrl) {
      return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, false));
    };
    typedef std::integral_constant<int, 0x12C> From4;       // row_ror:12: lane + 4
    typedef std::integral_constant<int, 0x128> From8;       // row_ror:8
    if constexpr (PW <= 8) {
      constexpr int N = side_by_side<PW>();
      const int part = (lane & 15) / N;                     // (the fourth of N = 4: the third again)
      const unsigned short* own = a.v + (part == 0 ? PART[0] : (part == 1 ? PART[1] : PART[2]));
      f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f}, s2 = s;
#pragma unroll
      for (int k = 0; k < D / 32; ++k) {
        const int row = lane & (N - 1), col = k * 32 + (lane >> 4) * 8, plain = row * PITCH + k * 32 + (lane >> 4) * 8;
        const unsigned short* x = TURN ? a.v + at<PW, TURN>(part, row, col) : own + plain;
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.x[k], *reinterpret_cast<const bf16x8*>(x), s, 0, 0, 0);
        const unsigned short* x2 = TURN ? a.v + at<PW, TURN>(2, row, col) : a.v + PART[2] + plain;
        if (N == 8) s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.x[k], *reinterpret_cast<const bf16x8*>(x2), s2, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        s[r] += N == 4 ? from(s[r], From4{}) + from(s[r], From8{}) : from(s[r], From8{}) + s2[r];
      return s;
    }
    f32x4 s[3];                                             // independent sums: the chain is a third as long
#pragma unroll
    for (int p = 0; p < 3; ++p) s[p] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < D / 32; ++k)
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(a.v + at<PW, TURN>(p, lane & 15, k * 32 + (lane >> 4) * 8));
        s[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.x[k], x, s[p], 0, 0, 0);
      }
    return (s[2] + s[1]) + s[0];
  }
};

// every place of a vector's parts is inside Act, whichever product will read it
template <int D, bool TURN> constexpr bool act_holds() {
  typedef Prod<unsigned short, D> X;
  const int n = sizeof(X::Act::v) / sizeof(unsigned short);
  return X::template extent<4, TURN>(3) <= n && X::template extent<8, TURN>(3) <= n && X::template extent<16, TURN>(3) <= n;
}
static_assert(act_holds<64, false>() && act_holds<128, false>() && act_holds<128, true>(), "a part lies outside Act");

}  // namespace laser
