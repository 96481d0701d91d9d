// GSTA with fp32 arithmetic for either storage type, any number of layers and segments, d in {64, 128}: the form behind
// the generic variant at these widths. A workgroup owns PW pairs through all layers.
//
// Per layer a pair needs three d x d matrix-vector products and one pass over its S x d block of H' (re-associated as
// everywhere: r = W_k (t W_q)^T, e = H' r / sqrt(d), p = softmax(e) H', t += p W_v). The one-workgroup-per-pair kernel this
// replaces was a chain of dependent loads: every product walked its matrix row by row from L2. Here
//   - a layer's three matrices lie in registers, spread over the workgroup (a thread holds 8 columns of d / 32 rows), are
//     requested a layer ahead and serve all PW pairs; a column product is reduced over the row slices of a wave by lane
//     permutes and over the waves through LDS, a row product over the 16 (or 8) lanes of a row;
//   - H' is read once per layer with one row per d / 8 lanes (8 elements a lane), an online softmax per lane group merged
//     at the end; when the block fits (R row loads per lane) it stays in registers over the layers.
// All sums have a fixed order.
//
// Bound by the chain of products and barriers of one layer (about 2 us) for small batches, by the vector ALUs beyond: 3 d^2
// + 2 S d multiply-adds per pair and layer. Before / after: 100 pairs, S = 100, d = 128, two layers, bf16 77 -> 9.7 us; 1200
// pairs, S = 15, d = 64, two layers, fp32 34 -> 13.7 us; 16 pairs, S = 16, d = 64, one layer, fp32 13.5 -> 4.9 us.
#include "laser_internal.h"

namespace laser {

typedef unsigned int u32x4r __attribute__((ext_vector_type(4)));
typedef float f32x4r __attribute__((ext_vector_type(4)));

template <typename T> struct Row8;
template <> struct Row8<unsigned short> {
  u32x4r x;
  __device__ __forceinline__ void load(const unsigned short* p) { x = *reinterpret_cast<const u32x4r*>(p); }
  __device__ __forceinline__ void zero() { x = u32x4r{0u, 0u, 0u, 0u}; }
  __device__ __forceinline__ float get(int e) const {   // (e is a constant after unrolling)
    return __uint_as_float((e & 1) ? (x[e >> 1] & 0xffff0000u) : (x[e >> 1] << 16));
  }
};
template <> struct Row8<float> {
  f32x4r a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4r*>(p);
    b = *reinterpret_cast<const f32x4r*>(p + 4);
  }
  __device__ __forceinline__ void zero() { a = b = f32x4r{0.0f, 0.0f, 0.0f, 0.0f}; }
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

// PW: pairs per workgroup; R: row loads per lane and round; RES: one round holds every row (H' stays in registers)
template <typename T, int D, int PW, int R, bool RES>
__global__ __launch_bounds__(4 * D) void gsta_rows_kernel(const T* __restrict__ seg, const T* __restrict__ t0,
                                                          const T* __restrict__ wq, const T* __restrict__ wk,
                                                          const T* __restrict__ wv, const int32_t* __restrict__ lens,
                                                          const int32_t* __restrict__ cand_off, int U, int P, int C,
                                                          int L, int w, int S, int M, float* __restrict__ z) {
  constexpr int NT = 4 * D, NW = NT / 64, LPR = D / 8, RPW = 64 / LPR, XR = D / 32, WPP = NW / PW;
  static_assert(PW <= NW, "a wave serves one pair of H'");
  __shared__ float ts[PW][D], qp[PW][D], rr[PW][D], pp[PW][D];   // t, t W_q, r / sqrt(d), p
  __shared__ float part[NW][PW][D];                               // row slices of a column product, by wave
  __shared__ float pml[NW][2];
  const int tid = threadIdx.x, lane = tid & 63, gl = lane % LPR, grp = lane / LPR;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pbase = blockIdx.x * PW;
  const int x0 = (wave * RPW + grp) * XR;                         // this thread's rows of a matrix, columns 8 gl ..
  // the pair whose H' this wave works on (a pair past the last one is worked on again, and not stored)
  const int pj = wave / WPP, wp = wave % WPP;
  const int pr = pbase + pj < P ? pbase + pj : P - 1;
  const int nv = __builtin_amdgcn_readfirstlane((valid_len(lens, pair_user(cand_off, U, C, pr), L) + w - 1) / w);
  const T* H = seg + (size_t)pr * S * D + gl * 8;
  const float scale = 1.0f / sqrtf((float)D);

  auto load_w = [&](Row8<T> (&wr)[XR], const T* W) {
#pragma unroll
    for (int i = 0; i < XR; ++i) wr[i].load(W + (size_t)(x0 + i) * D + gl * 8);
  };
  auto load_h = [&](Row8<T> (&h)[R], int k0) {                    // rows at or past nv: the last valid one, weight zero
#pragma unroll
    for (int k = 0; k < R; ++k) {
      int row = ((k0 + k) * WPP + wp) * RPW + grp;
      row = row < nv ? row : nv - 1;
      h[k].load(H + (size_t)row * D);
    }
  };
  Row8<T> rq[XR], rk[XR], rv[XR], h[R];
  load_w(rq, wq);
  load_w(rk, wk);
#pragma unroll
  for (int k = 0; k < R; ++k) h[k].zero();                        // no valid segment: nothing is read
  if (nv > 0) load_h(h, 0);
  load_w(rv, wv);
  for (int e = tid; e < PW * D; e += NT) {
    const int j = e / D, y = e % D;
    ts[j][y] = load_as_f32(t0, (size_t)(pbase + j < P ? pbase + j : P - 1) * D + y);
  }
  __syncthreads();

  // part[wave][j][y] = sum over the wave's row slices of in[j][x] W[x][y]
  auto col_product = [&](const float (&in)[PW][D], const Row8<T> (&wr)[XR]) {
#pragma unroll 1
    for (int j = 0; j < PW; ++j) {
      float acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        const float x = in[j][x0 + i];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(x, wr[i].get(e), acc[e]);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = over_groups<LPR, false>(acc[e]);
      if (grp == 0) {
        *reinterpret_cast<f32x4r*>(&part[wave][j][gl * 8]) = f32x4r{acc[0], acc[1], acc[2], acc[3]};
        *reinterpret_cast<f32x4r*>(&part[wave][j][gl * 8 + 4]) = f32x4r{acc[4], acc[5], acc[6], acc[7]};
      }
    }
  };
  auto part_sum = [&](int j, int y) {
    float s = part[0][j][y];
#pragma unroll
    for (int o = 1; o < NW; ++o) s += part[o][j][y];
    return s;
  };

  for (int l = 0; l < M; ++l) {
    const size_t next = (size_t)(l + 1 < M ? l + 1 : l) * D * D;
    col_product(ts, rq);                                          // q' = t W_q
    load_w(rq, wq + next);
    __syncthreads();
    for (int e = tid; e < PW * D; e += NT) qp[e / D][e % D] = part_sum(e / D, e % D);
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j < PW; ++j) {                                // r = W_k q'
      float in[8], acc[XR];
#pragma unroll
      for (int e = 0; e < 8; ++e) in[e] = qp[j][gl * 8 + e];
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        acc[i] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[i] = fmaf(rk[i].get(e), in[e], acc[i]);
        acc[i] = row_sum<LPR>(acc[i]) * scale;
      }
      if (gl == 0)
#pragma unroll
        for (int i = 0; i < XR; ++i) rr[j][x0 + i] = acc[i];
    }
    load_w(rk, wk + next);
    __syncthreads();
    {                                                             // one pass over the rows of H'
      constexpr float NEG = -3.0e38f;
      float r8[8], acc[8], m = NEG, den = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        r8[e] = rr[pj][gl * 8 + e];
        acc[e] = 0.0f;
      }
      for (int k0 = 0; k0 * WPP * RPW < nv; k0 += R) {
        if (!RES && (k0 > 0 || l > 0)) load_h(h, k0);
        float s[R], mx = m;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          s[k] = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) s[k] = fmaf(h[k].get(e), r8[e], s[k]);
          s[k] = row_sum<LPR>(s[k]);
          if (((k0 + k) * WPP + wp) * RPW + grp < nv) mx = fmaxf(mx, s[k]);
        }
        const float corr = expf(m - mx);
        m = mx;
        den *= corr;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= corr;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const float p = ((k0 + k) * WPP + wp) * RPW + grp < nv ? expf(s[k] - m) : 0.0f;
          den += p;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = fmaf(p, h[k].get(e), acc[e]);
        }
        if (RES) break;
      }
      const float mw = over_groups<LPR, true>(m), f = expf(m - mw);
      den = over_groups<LPR, false>(den * f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = over_groups<LPR, false>(acc[e] * f);
      if (grp == 0) {
        *reinterpret_cast<f32x4r*>(&part[wave][0][gl * 8]) = f32x4r{acc[0], acc[1], acc[2], acc[3]};
        *reinterpret_cast<f32x4r*>(&part[wave][0][gl * 8 + 4]) = f32x4r{acc[4], acc[5], acc[6], acc[7]};
      }
      if (lane == 0) {
        pml[wave][0] = mw;
        pml[wave][1] = den;
      }
    }
    __syncthreads();
    for (int e = tid; e < PW * D; e += NT) {                      // p, over the waves of a pair; zero without a valid segment
      const int j = e / D, y = e % D;
      float m = pml[j * WPP][0], num = 0.0f, den = 0.0f;
#pragma unroll
      for (int o = 1; o < WPP; ++o) m = fmaxf(m, pml[j * WPP + o][0]);
#pragma unroll
      for (int o = 0; o < WPP; ++o) {
        const float f = expf(pml[j * WPP + o][0] - m);
        den = fmaf(pml[j * WPP + o][1], f, den);
        num = fmaf(part[j * WPP + o][0][y], f, num);
      }
      pp[j][y] = den > 0.0f ? num / den : 0.0f;
    }
    __syncthreads();
    col_product(pp, rv);                                          // t += p W_v
    load_w(rv, wv + next);
    __syncthreads();
    for (int e = tid; e < PW * D; e += NT) ts[e / D][e % D] += part_sum(e / D, e % D);
    __syncthreads();
  }
  for (int e = tid; e < PW * D; e += NT)
    if (pbase + e / D < P) z[(size_t)pbase * D + e] = ts[e / D][e % D];
}

bool gsta_rows_supports(const GstaArgs& a) { return a.d == 64 || a.d == 128; }

template <typename T, int D, int PW>
static void launch_pw(const GstaArgs& a, int P) {
  constexpr int R = 4;                                            // rows of H' in flight per lane
  const int held = R * (D / 16 / PW) * (512 / D);                 // rows a pair's waves hold in one round
#define LASER_ROWS(RES)                                                                                             \
  hipLaunchKernelGGL((gsta_rows_kernel<T, D, PW, R, RES>), dim3((unsigned)((P + PW - 1) / PW)), dim3(4 * D), 0,    \
                     a.stream, (const T*)a.seg, (const T*)a.t0, (const T*)a.wq, (const T*)a.wk, (const T*)a.wv,    \
                     a.lens, a.cand_off, a.U, P, a.C, a.L, a.w < a.L ? a.w : a.L, a.S, a.M, a.z_out)
  if (a.S <= held) LASER_ROWS(true);
  else LASER_ROWS(false);
#undef LASER_ROWS
}

template <typename T, int D>
static void launch_t(const GstaArgs& a) {
  const int P = gsta_pairs(a);
  const int per = P / 512;                                        // pairs per workgroup that still give two to a compute unit
  if (per >= 8 && D == 128) launch_pw<T, D, D / 16>(a, P);
  else if (per >= 4) launch_pw<T, D, 4>(a, P);
  else if (per >= 2) launch_pw<T, D, 2>(a, P);
  else launch_pw<T, D, 1>(a, P);
}

laser_status gsta_rows_launch(const GstaArgs& a) {
  if (!gsta_rows_supports(a)) return LASER_ERR_UNSUPPORTED;
  if (gsta_pairs(a) == 0) return LASER_OK;
  if (a.dt == LASER_F32) {
    if (a.d == 64) launch_t<float, 64>(a);
    else launch_t<float, 128>(a);
  } else {
    if (a.d == 64) launch_t<unsigned short, 64>(a);
    else launch_t<unsigned short, 128>(a);
  }
  return launch_status();
}

}  // namespace laser
