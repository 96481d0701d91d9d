// Backward pass of GSTA in tiles of 1 to 16 pairs (d in {64, 128}, either storage type, any number of layers): the equations
// stand at the top of gsta_backward.hip. The forward kernel's frame (gsta_tiled.hip): d / 16 waves, each with 16 columns of
// every d x d product, the products on the matrix cores with 24-bit factors, t and its gradient in the accumulator layout,
// several waves to a pair's rows when there are fewer pairs than waves.
//
// A layer takes two passes over H', one in the forward sweep (scores and p) and one in the backward sweep, where
//   D = sum_k a_k da_k = dp . p   is known before the pass (dp = do W_v^T needs no row of H'), so da_i = dp . H'_i,
//   de_i = a_i (da_i - D) and dr = sum_i de_i H'_i / sqrt(d) come from one reading of the row.
// The gradient of H' is not accumulated anywhere: with a layer's a_i, de_i, dp and r kept in LDS,
//   dH'_i = sum over layers of a_i dp + de_i r / sqrt(d)
// is formed and stored once, in the last pass. The six vectors per pair and layer whose outer products are the weight
// gradients go to the caller's scratch (gsta_bwd_w_kernel sums them).
//
// Bound by the chain of five products and two passes per workgroup (one round of workgroups) and by H' read twice and dH'
// written: 2048 pairs, S = 100, d = 128 (132 MB at most, 84 MB valid) 33 us, one workgroup per pair with its rows in LDS
// 131 us; 4096 pairs, S = 16, d = 64 15 us (18 us before the vectors of the tile crossed LDS and memory four columns at a time).
#include "gsta_tile.h"
#include "laser_internal.h"

namespace laser {

template <typename T>
__device__ __forceinline__ void store_row8(T* p, const float (&x)[8]);
template <>
__device__ __forceinline__ void store_row8<float>(float* p, const float (&x)[8]) {
  *reinterpret_cast<f32x4*>(p) = f32x4{x[0], x[1], x[2], x[3]};
  *reinterpret_cast<f32x4*>(p + 4) = f32x4{x[4], x[5], x[6], x[7]};
}
template <>
__device__ __forceinline__ void store_row8<unsigned short>(unsigned short* p, const float (&x)[8]) {
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    o[e] = (unsigned)f32_to_bf16_bits(x[2 * e]) | ((unsigned)f32_to_bf16_bits(x[2 * e + 1]) << 16);
  *reinterpret_cast<u32x4*>(p) = o;
}

__device__ __forceinline__ void lds_row8(float (&x)[8], const float* p) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = e < 4 ? a[e & 3] : b[e & 3];
}

// LDS of a workgroup, in bytes: two left operands, the waves' patches, the waves' partial sums, and per pair and layer
// r, dp, p (rows of D + 4), the softmax statistics and the rows' e / a and de
template <typename T, int D>
static constexpr size_t tile_bytes() {
  return 2 * sizeof(typename Prod<T, D>::Act) + (D / 16) * (Prod<T, D>::PATCH + (D + 4) * 4 + 16);
}
static size_t pair_layer_bytes(int D, int S) { return (3 * (D + 4) + 4 + 2 * (((size_t)S + 3) / 4 * 4)) * 4; }

template <typename T, int D, int PW>
__global__ __launch_bounds__(4 * D) void gsta_bwd_tile_kernel(const T* __restrict__ seg, const T* __restrict__ t0,
                                                              const T* __restrict__ wq, const T* __restrict__ wk,
                                                              const T* __restrict__ wv,
                                                              const int32_t* __restrict__ lens,
                                                              const float* __restrict__ dz, int P, int C, int L, int w,
                                                              int S, int M, T* __restrict__ dseg,
                                                              float* __restrict__ dt0, float* __restrict__ pv) {
  typedef Prod<T, D> X;
  constexpr int NW = D / 16, LPR = D / 8, RPW = 64 / LPR;
  constexpr int WPP = PW < NW ? NW / PW : 1;                      // waves that share a pair's rows
  constexpr int PPW = PW > NW ? PW / NW : 1;                      // pairs of a wave
  constexpr int RP = D + 4;
  constexpr int R = 16 / (int)sizeof(T) / 2;                      // rows of H' in flight per lane: 4 or 2
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ int some_of[16];                                     // the pair has a valid segment
  typename X::Act& ba = *reinterpret_cast<typename X::Act*>(lds);
  typename X::Act& bb = *reinterpret_cast<typename X::Act*>(lds + sizeof(typename X::Act));
  unsigned char* at = lds + 2 * sizeof(typename X::Act);
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* patch = at + wave * X::PATCH;
  at += NW * X::PATCH;
  float* part = reinterpret_cast<float*>(at);                     // [NW][RP] and, after it, [NW][4]: maximum, denominator
  float* pml = part + NW * RP;
  const int S4 = (S + 3) / 4 * 4;
  const size_t stride = 3 * RP + 4 + 2 * S4;                      // floats per (pair, layer)
  float* pl = pml + NW * 4;
  auto rr_of = [&](int j, int l) { return pl + (j * M + l) * stride; };   // r / sqrt(d), in the units of X::ex
  // dp_of = rr_of + RP, p_of = rr_of + 2 RP, statistics (maximum, 1 / denominator) = rr_of + 3 RP, then e (later a), de
  const int pbase = blockIdx.x * PW, n0 = wave * 16, c4 = n0 + 4 * (lane >> 4);
  const int gl = lane % LPR, grp = lane / LPR, wp = PW < NW ? wave % WPP : 0;
  const float scale = 1.0f / sqrtf((float)D);

  typename X::Cols cq, cx;                                        // columns of W_q; of W_v (forward) and W_k (backward)
  typename X::Operand rk, rv, rq;
  X::load_cols(cq, wq, n0, lane);
  auto at4 = [&] { return (size_t)(pbase + l16 < P ? pbase + l16 : P - 1) * D + c4; };   // pair l16, columns c4 ..
  const bool mine4 = l16 < PW && pbase + l16 < P;
  const typename X::Raw4 traw = *reinterpret_cast<const typename X::Raw4*>(t0 + at4());
  f32x4 g = *reinterpret_cast<const f32x4*>(dz + at4());
  X::load_rows(rk, wk, n0, lane);
  // (lengths without a branch on `lens`, in which one load would wait for the other)
  auto pair_of = [&](int i) {
    const int pr = pbase + (PW < NW ? wave / WPP : wave * PPW + i);
    return pr < P ? pr : P - 1;
  };
  int nl[PPW];
#pragma unroll
  for (int i = 0; i < PPW; ++i) nl[i] = *(lens != nullptr ? lens + pair_of(i) / C : reinterpret_cast<const int32_t*>(wq));
  int nv[PPW];
  const T* H[PPW];
  Row8<T> h[R];
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    const int pj = PW < NW ? wave / WPP : wave * PPW + i;
    nv[i] = __builtin_amdgcn_readfirstlane(((lens == nullptr || nl[i] > L ? L : (nl[i] < 0 ? 0 : nl[i])) + w - 1) / w);
    H[i] = seg + (size_t)pair_of(i) * S * D;
    if (lane == 0) some_of[pj] = nv[i] > 0;
  }
  auto load_h = [&](Row8<T> (&x)[R], int i, int k0) {             // rows at or past nv: the last valid one, weight zero
    const int last = nv[i] > 0 ? nv[i] - 1 : 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      int row = ((k0 + k) * WPP + wp) * RPW + grp;
      row = row < last ? row : last;
      x[k].load(H[i] + (unsigned)(row * D + gl * 8));
    }
  };
  load_h(h, 0, 0);                                                // (the first rows of the first pass, ahead of the products)
  __builtin_assume(M > 0);                                        // (or the loads move behind a branch on it)
  __builtin_amdgcn_sched_barrier(0);                              // (widened any earlier, t waits for its load ahead of the others)
  f32x4 t = X::wide4(traw);
  auto put_tile = [&](typename X::Act& b, const f32x4& x) { X::template put4<PW>(b, l16, c4, x); };
  auto put_scratch = [&](int l, int slot, const f32x4& x) {       // one of the six vectors of a pair and layer
    if (mine4) *reinterpret_cast<f32x4*>(pv + (((size_t)(pbase + l16) * M + l) * 6 + slot) * D + c4) = x;
  };
  auto put_rows = [&](int l, int off, const f32x4& x, float f) {  // into the (pair, layer) block
    if (l16 < PW) *reinterpret_cast<f32x4*>(rr_of(l16, l) + off + c4) = x * f;
  };
  // A vector summed over a wave's rows, `acc` still apart by lane group: handed to `take(pair, element, value)` by one lane per
  // element, or left for over_waves() where several waves share the pair.
  auto gather = [&](int i, float (&acc)[8], float f, auto take) {
    const int pj = PW < NW ? wave / WPP : wave * PPW + i;
    scatter_over_groups<LPR>(acc, lane);
    const int y0 = gl * 8 + group_first<LPR>(lane);
#pragma unroll
    for (int e = 0; e < LPR / 8; ++e) {
      if constexpr (WPP == 1) take(pj, y0 + e, acc[e] * f);
      else part[wave * RP + y0 + e] = acc[e];
    }
  };
  auto over_waves = [&](float f, auto take) {
    if constexpr (WPP > 1) {
      for (int e = tid; e < PW * D; e += 4 * D) {
        const int j = e / D, y = e % D;
        float s = part[(j * WPP) * RP + y];
#pragma unroll
        for (int o = 1; o < WPP; ++o) s += part[(j * WPP + o) * RP + y];
        take(j, y, s * f);
      }
      __syncthreads();
    }
  };

  // ---------------------------------------------------------------- forward sweep
  for (int l = 0; l < M; ++l) {
    const bool more = l + 1 < M;
    const size_t here = (size_t)l * D * D, next = (size_t)(l + 1) * D * D;
    put_tile(ba, t);
    put_scratch(l, 4, t);
    const typename X::Operand oq = X::transposed(cq, patch, lane);
    __syncthreads();
    const f32x4 q = X::template product<PW>(ba, oq, lane);                     // q' = t W_q
    if (more) {
      X::load_cols(cq, wq + next, n0, lane);
      X::load_cols(cx, wv + here, n0, lane);
    } else {
      X::load_rows(rv, wv + here, n0, lane);                      // the first operand of the backward sweep
    }
    put_tile(bb, q);
    put_scratch(l, 3, q);
    __syncthreads();
    const f32x4 r = X::template product<PW>(bb, rk, lane);                     // r = W_k q'
    if (more) X::load_rows(rk, wk + next, n0, lane);
    put_rows(l, 0, r, scale * X::LOG);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
      const int pj = PW < NW ? wave / WPP : wave * PPW + i;
      float* blk = rr_of(pj, l);
      float r8[8], acc[8], m = -INFINITY, den = 0.0f;
      lds_row8(r8, blk + gl * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
      if (i > 0 || l > 0) load_h(h, i, 0);
      for (int k0 = 0; k0 * WPP * RPW < nv[i]; k0 += R) {
        Row8<T> ahead[R];
        const bool on = (k0 + R) * WPP * RPW < nv[i];
        if (on) load_h(ahead, i, k0 + R);
        float s[R], mx = m;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          s[k] = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) s[k] = fmaf(h[k].get(e), r8[e], s[k]);
          s[k] = row_sum<LPR>(s[k]);
          const int row = ((k0 + k) * WPP + wp) * RPW + grp;
          if (row < nv[i]) {
            mx = fmaxf(mx, s[k]);
            if (gl == 0) blk[3 * RP + 4 + row] = s[k];
          }
        }
        const float ref = softmax_ref(mx), corr = X::ex(m - ref);
        den *= corr;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= corr;
        m = mx;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const float p = ((k0 + k) * WPP + wp) * RPW + grp < nv[i] ? X::ex(s[k] - ref) : 0.0f;
          den += p;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = fmaf(p, h[k].get(e), acc[e]);
        }
        if (on)
#pragma unroll
          for (int k = 0; k < R; ++k) h[k] = ahead[k];
      }
      const float mw = over_groups<LPR, true>(m), f = X::ex(m - softmax_ref(mw));
      den = over_groups<LPR, false>(den * f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] *= f;
      // no valid segment: p = 0 (by their number, as in the forward kernel)
      const float inv = nv[i] > 0 ? 1.0f / den : 0.0f;
      if (WPP == 1) {
        if (lane == 0) {
          blk[3 * RP] = softmax_ref(mw);
          blk[3 * RP + 1] = inv;
        }
      } else if (lane == 0) {
        pml[wave * 4] = nv[i] > 0 ? mw : 0.0f;
        pml[wave * 4 + 1] = nv[i] > 0 ? den : 1.0f;
      }
      gather(i, acc, inv, [&](int j, int y, float x) { rr_of(j, l)[2 * RP + y] = x; });
    }
    __syncthreads();
    if constexpr (WPP > 1) {                                      // p over the waves of a pair
      for (int e = tid; e < PW * D; e += 4 * D) {
        const int j = e / D, y = e % D;
        float m = pml[j * WPP * 4], num = 0.0f, den = 0.0f;
#pragma unroll
        for (int o = 1; o < WPP; ++o) m = fmaxf(m, pml[(j * WPP + o) * 4]);
        m = softmax_ref(m);
#pragma unroll
        for (int o = 0; o < WPP; ++o) {
          const float f = X::ex(pml[(j * WPP + o) * 4] - m);
          den = fmaf(pml[(j * WPP + o) * 4 + 1], f, den);
          num = fmaf(part[(j * WPP + o) * RP + y], f, num);
        }
        const float inv = 1.0f / den;
        float* blk = rr_of(j, l);
        blk[2 * RP + y] = num * inv;
        if (y == 0) {
          blk[3 * RP] = m;
          blk[3 * RP + 1] = inv;
        }
      }
      __syncthreads();
    }
    for (int e = tid; e < PW * D; e += 4 * D) {                   // p: to the scratch, and as an operand where t goes on
      const int j = e / D, y = e % D;
      const float x = rr_of(j, l)[2 * RP + y];
      if (more) X::template put<PW>(ba, j, y, x);
      if (pbase + j < P) pv[(((size_t)(pbase + j) * M + l) * 6) * D + y] = x;
    }
    if (more) {
      const typename X::Operand ov = X::transposed(cx, patch, lane);
      __syncthreads();
      t += X::template product<PW>(ba, ov, lane);                              // t += p W_v
      __syncthreads();
    }
  }

  // ---------------------------------------------------------------- backward sweep
  for (int l = M - 1; l >= 0; --l) {
    const size_t here = (size_t)l * D * D;
    put_tile(ba, g);
    put_scratch(l, 1, g);
    __syncthreads();
    const f32x4 dp = X::template product<PW>(ba, rv, lane);                    // dp = do W_v^T, do = g
    X::load_cols(cx, wk + here, n0, lane);
    put_rows(l, RP, dp, 1.0f);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
      const int pj = PW < NW ? wave / WPP : wave * PPW + i;
      float* blk = rr_of(pj, l);
      float* ea = blk + 3 * RP + 4;
      float dp8[8], p8[8], r8[8], acc[8], D0 = 0.0f;
      lds_row8(dp8, blk + RP + gl * 8);
      lds_row8(p8, blk + 2 * RP + gl * 8);
      lds_row8(r8, blk + gl * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        D0 = fmaf(dp8[e], p8[e], D0);
        r8[e] *= 1.0f / X::LOG;                                   // r / sqrt(d)
        acc[e] = 0.0f;
      }
      D0 = row_sum<LPR>(D0);
      const float m = blk[3 * RP], inv = blk[3 * RP + 1];
      T* dH = dseg + (size_t)(pbase + pj) * S * D + gl * 8;
      const bool mine = pbase + pj < P;
      load_h(h, i, 0);
      const int end = l == 0 ? S : nv[i];                         // the last pass writes every row, zeros past nv
      for (int k0 = 0; k0 * WPP * RPW < end; k0 += R) {
        Row8<T> ahead[R];
        const bool on = (k0 + R) * WPP * RPW < nv[i];
        if (on) load_h(ahead, i, k0 + R);
        float da[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
          da[k] = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) da[k] = fmaf(h[k].get(e), dp8[e], da[k]);
          da[k] = row_sum<LPR>(da[k]);
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int row = ((k0 + k) * WPP + wp) * RPW + grp;
          const bool ok = row < nv[i];
          const float a = ok ? X::ex(ea[row] - m) * inv : 0.0f, de = ok ? a * (da[k] - D0) : 0.0f;
          if (ok)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = fmaf(de, h[k].get(e), acc[e]);
          if (l > 0) {
            if (ok && gl == 0) {
              ea[row] = a;
              ea[S4 + row] = de;
            }
          } else if (row < S && mine) {
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = ok ? fmaf(a, dp8[e], de * r8[e]) : 0.0f;
            for (int o2 = 1; o2 < M && ok; ++o2) {
              const float* b2 = blk + o2 * stride;
              float x8[8], y8[8];
              lds_row8(x8, b2 + RP + gl * 8);
              lds_row8(y8, b2 + gl * 8);
              const float a2 = b2[3 * RP + 4 + row], d2 = b2[3 * RP + 4 + S4 + row] * (1.0f / X::LOG);
#pragma unroll
              for (int e = 0; e < 8; ++e) o[e] = fmaf(a2, x8[e], fmaf(d2, y8[e], o[e]));
            }
            store_row8<T>(dH + (size_t)row * D, o);
          }
        }
        if (on)
#pragma unroll
          for (int k = 0; k < R; ++k) h[k] = ahead[k];
      }
      gather(i, acc, scale, [&](int j, int y, float x) {
        X::template put<PW>(bb, j, y, x);
        if (pbase + j < P) pv[(((size_t)(pbase + j) * M + l) * 6 + 2) * D + y] = x;
      });
    }
    const typename X::Operand ok_ = X::transposed(cx, patch, lane);
    X::load_rows(rq, wq + here, n0, lane);
    if (l > 0) X::load_rows(rv, wv + here - (size_t)D * D, n0, lane);
    __syncthreads();
    over_waves(scale, [&](int j, int y, float x) {
      X::template put<PW>(bb, j, y, x);
      if (pbase + j < P) pv[(((size_t)(pbase + j) * M + l) * 6 + 2) * D + y] = x;
    });
    const f32x4 dq = X::template product<PW>(bb, ok_, lane);                   // dq' = dr W_k
    put_tile(ba, dq);
    put_scratch(l, 5, dq);
    __syncthreads();
    g += X::template product<PW>(ba, rq, lane);                                // g += dq' W_q^T (the residual path keeps g)
    __syncthreads();
  }
  if (mine4) *reinterpret_cast<f32x4*>(dt0 + at4()) = g;
  // A pair without a valid segment adds nothing to the weight gradients, whatever its target and dz hold: its vectors, of which p
  // and dr are zeros already, are overwritten with zeros (zero times a value that is not finite is NaN).
  for (unsigned long long m = __ballot(lane < PW && pbase + lane < P && some_of[lane & 15] == 0); m != 0; m &= m - 1)
    for (int e = tid; e < M * 6 * D; e += 4 * D) pv[(size_t)(pbase + __builtin_ctzll(m)) * M * 6 * D + e] = 0.0f;
}

template <typename T, int D>
static size_t lds_for(const GstaBwdArgs& a, int pw) {
  return tile_bytes<T, D>() + (size_t)pw * a.M * pair_layer_bytes(D, a.S);
}

template <typename T, int D, int PW>
static laser_status launch_pairs(const GstaBwdArgs& a, int P) {
  auto kern = gsta_bwd_tile_kernel<T, D, PW>;
  const size_t lds = lds_for<T, D>(a, PW);
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, DYNAMIC_LDS_MOST) != hipSuccess)
    return LASER_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, dim3((unsigned)((P + PW - 1) / PW)), dim3(4 * D), lds, a.stream, (const T*)a.seg,
                     (const T*)a.t0, (const T*)a.wq, (const T*)a.wk, (const T*)a.wv, a.lens, a.dz, P, a.C, a.L,
                     a.w < a.L ? a.w : a.L, a.S, a.M, (T*)a.dseg, a.dt0, a.work);
  return launch_status();
}

template <typename T, int D>
static laser_status launch_t(const GstaBwdArgs& a) {
  const int P = a.U * a.C, per = D == 128 || sizeof(T) == 4 ? P : (P + 1) / 2;
  // pairs per workgroup: as in the forward kernel (gsta_tiled.hip), halved while their rows' scores do not fit in LDS
  int pw = per <= 256 ? 1 : per <= 512 ? 2 : per <= 1024 ? 4 : per <= 2048 ? 8 : 16;
  while (pw > 1 && lds_for<T, D>(a, pw) > DYNAMIC_LDS_MOST) pw /= 2;
  switch (pw) {
    case 1: return launch_pairs<T, D, 1>(a, P);
    case 2: return launch_pairs<T, D, 2>(a, P);
    case 4: return launch_pairs<T, D, 4>(a, P);
    case 8: return launch_pairs<T, D, 8>(a, P);
    default: return launch_pairs<T, D, 16>(a, P);
  }
}

bool gsta_bwd_tile_supports(const GstaBwdArgs& a) {
  if (a.d != 64 && a.d != 128) return false;
  const size_t lds = a.dt == LASER_BF16 ? (a.d == 64 ? lds_for<unsigned short, 64>(a, 1) : lds_for<unsigned short, 128>(a, 1))
                                        : (a.d == 64 ? lds_for<float, 64>(a, 1) : lds_for<float, 128>(a, 1));
  return lds <= DYNAMIC_LDS_MOST;
}

laser_status gsta_bwd_tile_launch(const GstaBwdArgs& a) {
  if (!gsta_bwd_tile_supports(a)) return LASER_ERR_UNSUPPORTED;
  if (a.dt == LASER_BF16) return a.d == 64 ? launch_t<unsigned short, 64>(a) : launch_t<unsigned short, 128>(a);
  return a.d == 64 ? launch_t<float, 64>(a) : launch_t<float, 128>(a);
}

}  // namespace laser
