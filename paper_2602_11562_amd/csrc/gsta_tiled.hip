// GSTA for a tile of 1 to 16 pairs per workgroup with the matrices of a layer in registers: either storage type, any
// number of layers and segments, d in {64, 128}.
//
// Per layer a pair needs three d x d matrix-vector products and one pass over its S x d block of H' (re-associated as
// everywhere: r = W_k (t W_q)^T, e = H' r / sqrt(d), p = softmax(e) H', t += p W_v). The products of the tile are MFMAs of 16
// pairs (rows past the tile's pairs are not read back) x 16 columns: a workgroup has d / 16 waves and each owns 16 columns of
// every product, so a product is complete in the wave that computes it, and t never leaves the accumulator layout.
//   fp32 storage  v_mfma_f32_16x16x4_f32: fp32 products and sums.
//   bf16 storage  v_mfma_f32_16x16x32_bf16 with the fp32 factor (t, q', p) as three bf16 parts (24 bits), split where it is
//                 produced.
// A wave's share of W_q and W_v (its 16 columns of every row) is requested a layer ahead in 16-byte pieces and crosses a
// wave-private LDS patch into operand order when it is used; its share of W_k (16 rows) is an operand as loaded. H' is read
// once per layer, one row per d / 8 lanes (8 elements a lane), with an online softmax per lane group merged at the end; a
// block that fits (R row loads per lane) stays in registers over the layers, others stream with the next R rows in
// flight. With fewer pairs than waves several waves share a pair's rows. All sums have a fixed order.
//
// Bound by the chain of a layer (three products, the pass over H', four or five barriers: 3 us for d = 128, 1.7 us for
// d = 64) until the machine is full, by the stream of H' and of the matrices (96 KB a workgroup at d = 128) beyond. bf16, two
// layers, d = 128: 100 pairs, S = 100 10.1 us (77 us on one workgroup per pair that walked the matrices row by row); 2048
// pairs, S = 40 13.5 us, 4096 pairs, S = 32 17.8 us (16.3 and 31.2 us in the form with 32-pair tiles this one replaced);
// fp32, 1200 pairs, S = 15, d = 64, two layers 8.2 us (34 us). Parts and patches laid out so that what is read at once is in
// different banks, the next layer's W_q across its patch behind the pass, and the waves of a pair met behind the last product:
// another layer of 100 pairs, d = 128, S = 8 2.65 -> 2.45 us (fp32 6.3 -> 5.95); 120 drawn calls 0.979 of the time.
#include "gsta_tile.h"
#include "laser_internal.h"

namespace laser {

// PW: pairs per workgroup; R: row loads per lane and round; RES: one round holds every row (H' stays in registers); POOL: the
// maxima of the pooled view from the pass over the rows (one layer, bf16, a wave's pairs its own)
template <typename T, int D, int PW, int R, bool RES, bool POOL>
__global__ __launch_bounds__(4 * D, (RES && R < 4 && sizeof(T) == 2 ? 4 : 1)) void gsta_tiled_kernel(const T* __restrict__ seg, const T* __restrict__ t0,
                                                          const T* __restrict__ wq, const T* __restrict__ wk,
                                                          const T* __restrict__ wv, const int32_t* __restrict__ lens,
                                                          const int32_t* __restrict__ cand_off, int U, int P, int C,
                                                          int L, int w, int S, int M, float* __restrict__ z,
                                                          T* __restrict__ pool, T* __restrict__ recent, int recent_n) {
  typedef Prod<T, D> X;
  constexpr int NW = D / 16, LPR = D / 8, RPW = 64 / LPR;
  constexpr int WPP = PW < NW ? NW / PW : 1;                      // waves that share a pair's rows
  constexpr int PPW = PW > NW ? PW / NW : 1;                      // pairs of a wave
  constexpr int RP = D + 4;
  // The turned layout of the vectors in LDS, but for the instances of two workgroups a compute unit (R < 4) whose 128 registers
  // do not hold its longer addresses beside the rest: spilled, 2002 pairs, S = 2 took 8.5 us for 5.6, 9321 pairs, S = 11 17.9 for
  // 15.6. One and two rows a lane of sixteen pairs fit, 0.96 of the time without it.
  constexpr bool TURN = X::template turned<PW>() && !(RES && (PW == 8 ? R < 4 : R == 3));
  __shared__ __attribute__((aligned(16))) typename X::Act bt, bq; // t; q', then p
  __shared__ __attribute__((aligned(16))) float rr[PW * RP];      // r / sqrt(d)
  __shared__ __attribute__((aligned(16))) unsigned char patches[NW][X::PATCH];
  __shared__ __attribute__((aligned(16))) float part[WPP > 1 && sizeof(T) == 2 ? NW : 1][D];   // (the views)
  __shared__ __attribute__((aligned(8))) f32x2 pml[NW];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pbase = blockIdx.x * PW, n0 = wave * 16, c4 = n0 + 4 * g;
  unsigned char* patch = patches[wave];
  // rows of H': lane group `grp` of the wave, elements 8 gl ..
  const int gl = lane % LPR, grp = lane / LPR, wp = PW < NW ? wave % WPP : 0;

  typename X::Cols cq, cv;
  typename X::Operand rk;
  X::load_cols(cq, wq, n0, lane);
  const int pt = pbase + l16 < P ? pbase + l16 : P - 1;           // (rows of the tile past its pairs are not read back)
  const typename X::Raw4 traw = *reinterpret_cast<const typename X::Raw4*>(t0 + (size_t)pt * D + c4);
  // The oldest wave is served first: without a barrier here it has all of its requests in before the youngest has asked for what the
  // first product waits for. d = 128, bf16, up to eight pairs (us): 100 pairs, S = 100, two layers 8.82 -> 8.62, 2048 x 40
  // 13.75 -> 13.45, 4096 x 16, one layer 8.67 -> 8.53; sixteen pairs 10.26 -> 10.34, d = 64 and fp32 the same.
  if constexpr (D == 128 && sizeof(T) == 2 && PW <= 8) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }
  X::load_rows(rk, wk, n0, lane);
  // the pairs whose H' this wave works on (a pair past the last one is worked on again, and not stored); their lengths without a
  // branch on `lens`, in which one load would wait for the other
  auto pair_of = [&](int i) {
    const int pr = pbase + (PW < NW ? wave / WPP : wave * PPW + i);
    return pr < P ? pr : P - 1;
  };
  int nl[PPW];
#pragma unroll
  for (int i = 0; i < PPW; ++i)
    nl[i] = *(lens != nullptr ? lens + pair_user(cand_off, U, C, pair_of(i)) : reinterpret_cast<const int32_t*>(wq));
  int nv[PPW];
  const T* H[PPW];
  Row8<T> h[RES ? PPW : 1][R];
  auto load_h = [&](Row8<T> (&x)[R], int i, int k0) {             // rows at or past nv: the last valid one, weight zero
    const int last = nv[i] > 0 ? nv[i] - 1 : 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      int row = ((k0 + k) * WPP + wp) * RPW + grp;
      row = row < last ? row : last;
      x[k].load(H[i] + (unsigned)(row * D + gl * 8));
    }
  };
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    nv[i] = __builtin_amdgcn_readfirstlane(((lens == nullptr || nl[i] > L ? L : (nl[i] < 0 ? 0 : nl[i])) + w - 1) / w);
    H[i] = seg + (size_t)pair_of(i) * S * D;
    // (without a valid segment row 0 is requested and not used: a branch here makes the compiler wait for the loads)
    if (RES || i == 0) load_h(h[RES ? i : 0], i, 0);              // (streamed: the first rows of the first pass)
  }
  // the pooled maxima of pair i of a wave with pairs of its own, from the lane groups' (stored values: exact)
  auto store_pool = [&](int i, float (&top)[8]) __attribute__((always_inline)) {
    const int pr = pbase + wave * PPW + i;
#pragma unroll
    for (int e = 0; e < 8; ++e) top[e] = over_groups<LPR, true>(top[e]);
    if (grp == 0 && pr < P)
#pragma unroll
      for (int e = 0; e < 8; ++e) store_from_f32(pool, (size_t)pr * D + gl * 8 + e, nv[i] > 0 ? top[e] : 0.0f);
  };
  // (a share of a matrix takes 32 registers in fp32 at d = 128: beside eight rows a lane there is room for two)
  constexpr bool LATE = sizeof(T) == 4 && D == 128 && R == 8;
  // the next layer's share of W_q crosses the patch in the shadow of the barrier behind the pass, not when it is wanted (unless that
  // takes registers which are not there)
  constexpr bool EAGER = sizeof(T) == 2 && !(PW == 16 && D == 128 && RES && R < 4);
  if (!LATE) X::load_cols(cv, wv, n0, lane);
  const float scale = X::LOG / sqrtf((float)D);
  // (with M = 0 thinkable the compiler moves every load that only the loop wants behind a branch, and the wait for t before it)
  __builtin_assume(M > 0);
  if (sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);          // (widened any earlier, t waits for its load ahead of the others)
  f32x4 t = X::wide4(traw);                                       // pair l16, columns c4 ..
  typename X::Operand oq;

  for (int l = 0; l < M; ++l) {
    const bool more_layers = l + 1 < M;
    const size_t next = (size_t)(l + 1) * D * D;
    X::template put4<PW, TURN>(bt, l16, c4, t);
    if (EAGER ? l == 0 : true) oq = X::transposed(cq, patch, lane);
    __syncthreads();
    const f32x4 q = X::template product<PW, TURN>(bt, oq, lane);               // q' = t W_q
    if (more_layers) X::load_cols(cq, wq + next, n0, lane);
    X::template put4<PW, TURN>(bq, l16, c4, q);
    __syncthreads();
    const f32x4 rv = X::template product<PW, TURN>(bq, rk, lane);              // r = W_k q'
    if (LATE) X::load_cols(cv, wv + next - D * D, n0, lane);
    if (more_layers) X::load_rows(rk, wk + next, n0, lane);
    if (l16 < PW) *reinterpret_cast<f32x4*>(rr + l16 * RP + c4) = rv * scale;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPW; ++i) {                               // one pass over the rows of H'
      const int pj = PW < NW ? wave / WPP : wave * PPW + i;
      float r8[8], acc[8], top[8], m = -INFINITY, den = 0.0f;
      {
        const f32x4 a = *reinterpret_cast<const f32x4*>(rr + pj * RP + gl * 8);
        const f32x4 b = *reinterpret_cast<const f32x4*>(rr + pj * RP + gl * 8 + 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          r8[e] = e < 4 ? a[e & 3] : b[e & 3];
          acc[e] = 0.0f;
          top[e] = -INFINITY;
        }
      }
      Row8<T> (&hi)[R] = h[RES ? i : 0];
      Row8<T> ahead[R];
      if (!RES && i > 0) load_h(hi, i, 0);
      for (int k0 = 0; k0 * WPP * RPW < nv[i]; k0 += R) {
#pragma unroll
        for (int k = 0; k < R; ++k) hi[k].pin();
        const bool more = !RES && (k0 + R) * WPP * RPW < nv[i];
        if (more) load_h(ahead, i, k0 + R);
        float s[R], mx = m;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          s[k] = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) s[k] = fmaf(hi[k].get(e), r8[e], s[k]);
          s[k] = row_sum<LPR>(s[k]);
          if (((k0 + k) * WPP + wp) * RPW + grp < nv[i]) mx = fmaxf(mx, s[k]);
        }
        const float ref = softmax_ref(mx);
        if (!RES) {
          const float corr = X::ex(m - ref);
          den *= corr;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] *= corr;
        }
        m = mx;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          hi[k].pin();
          const float p = ((k0 + k) * WPP + wp) * RPW + grp < nv[i] ? X::ex(s[k] - ref) : 0.0f;
          den += p;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            acc[e] = fmaf(p, hi[k].get(e), acc[e]);
            if (POOL) top[e] = fmaxf(top[e], hi[k].get(e));       // (rows past the last valid one are copies of it)
          }
        }
        if (RES) break;
        if (more)
#pragma unroll
          for (int k = 0; k < R; ++k) hi[k] = ahead[k];
      }
      const float mw = over_groups<LPR, true>(m), f = X::ex(m - softmax_ref(mw));
      den = over_groups<LPR, false>(den * f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] *= f;
      scatter_over_groups<LPR>(acc, lane);
      const int y0 = gl * 8 + group_first<LPR>(lane);             // the elements this lane hands on
      // p, zero without a valid segment (by their number: a denominator of NaN, or of zero where every score is -inf, has to
      // reach the result)
      const float inv = WPP > 1 ? 1.0f : (nv[i] > 0 ? 1.0f / den : 0.0f);
#pragma unroll
      for (int e = 0; e < LPR / 8; ++e) X::template put<(WPP > 1 ? NW : PW), TURN>(bq, WPP > 1 ? wp * PW + pj : pj, y0 + e, acc[e] * inv);
      if (WPP > 1 && lane == 0) pml[wp * PW + pj] = nv[i] > 0 ? f32x2{mw, den} : f32x2{0.0f, 1.0f};
      if constexpr (POOL) store_pool(i, top);
    }
    if (!RES && more_layers) load_h(h[0], 0, 0);                  // the first rows of the next layer's pass
    const typename X::Operand ov = X::transposed(cv, patch, lane);
    if (EAGER && more_layers) oq = X::transposed(cq, patch, lane);
    __syncthreads();
    if constexpr (WPP == 1) {
      t += X::template product<PW, TURN>(bq, ov, lane);                          // t += p W_v
    } else {
      // The waves of a pair meet behind the product: column o PW + pair is the sum of wave o, relative to its own maximum (merged
      // before the product they took a barrier more, and an exponential per wave and element)
      const f32x2 ml = pml[lane & (NW - 1)];
      f32x4 y = X::template product<NW, TURN>(bq, ov, lane);
      const float f = X::ex(ml[0] - softmax_ref(over_waves<PW, NW, true>(ml[0])));
      const float scale = f / over_waves<PW, NW, false>(ml[1] * f);
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = over_waves<PW, NW, false>(y[r] * scale);
      t += y;
    }
    if (more_layers && !LATE) X::load_cols(cv, wv + next, n0, lane);
  }
  if (l16 < PW && pbase + l16 < P) *reinterpret_cast<f32x4*>(z + (size_t)(pbase + l16) * D + c4) = t;

  // the other two views (Sec. 3.4.4), bf16 only: the component-wise maximum over the valid rows and the first rows as
  // stored. The rows are read once more (they were last read a moment ago); maxima of stored values are exact.
  if constexpr (sizeof(T) == 2) {
    if ((POOL || pool == nullptr) && recent == nullptr) return;
    if constexpr (!POOL) __syncthreads();   // (orders nothing, but without it log-uniform lengths took up to 3.5 % longer)
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
      const int pj = PW < NW ? wave / WPP : wave * PPW + i, pr = pbase + pj;
      if (recent != nullptr && pr < P)
        for (int row = wp * RPW + grp; row < recent_n; row += WPP * RPW)
          *reinterpret_cast<u32x4*>(recent + ((size_t)pr * recent_n + row) * D + gl * 8) =
              *reinterpret_cast<const u32x4*>(H[i] + (unsigned)(row * D + gl * 8));
      if (POOL || pool == nullptr) continue;
      float best[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) best[e] = -INFINITY;
      for (int row = wp * RPW + grp; row < nv[i]; row += WPP * RPW) {
        Row8<T> x;
        x.load(H[i] + (unsigned)(row * D + gl * 8));
#pragma unroll
        for (int e = 0; e < 8; ++e) best[e] = fmaxf(best[e], x.get(e));
      }
      if constexpr (WPP == 1) {
        store_pool(i, best);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) best[e] = over_groups<LPR, true>(best[e]);
        if (grp == 0)
#pragma unroll
          for (int e = 0; e < 8; ++e) part[wave][gl * 8 + e] = nv[i] > 0 ? best[e] : 0.0f;
      }
    }
    if constexpr (WPP > 1) {
      if (POOL || pool == nullptr) return;
      __syncthreads();
      for (int e = tid; e < PW * D; e += 4 * D) {
        const int j = e / D, y = e % D;
        float m = part[j * WPP][y];
#pragma unroll
        for (int o = 1; o < WPP; ++o) m = fmaxf(m, part[j * WPP + o][y]);
        if (pbase + j < P) store_from_f32(pool, (size_t)(pbase + j) * D + y, m);
      }
    }
  }
}

template <typename T, int D, int PW>
static void launch_pairs(const GstaArgs& a, int P) {
  constexpr int WPP = PW < D / 16 ? D / 16 / PW : 1, HELD = WPP * (512 / D);   // rows a pair's waves hold per row load
#define LASER_TILED_FORM(R, RES, POOL)                                                                              \
  hipLaunchKernelGGL((gsta_tiled_kernel<T, D, PW, R, RES, POOL>), dim3((unsigned)((P + PW - 1) / PW)), dim3(4 * D), 0,   \
                     a.stream, (const T*)a.seg, (const T*)a.t0, (const T*)a.wq, (const T*)a.wk, (const T*)a.wv,    \
                     a.lens, a.cand_off, a.U, P, a.C, a.L, a.w < a.L ? a.w : a.L, a.S, a.M, a.z_out,               \
                     (T*)a.pool_out, (T*)a.recent_out, a.r)
#define LASER_TILED(R, RES) LASER_TILED_FORM(R, RES, false)
  // rows in flight when the block does not stay
  constexpr int STREAM = 8 / (int)sizeof(T);
  // eight rows a lane fit the registers beside the matrices up to eight pairs (sixteen where a wave has two of them and
  // rows are bf16; otherwise they spill or leave one wave per SIMD), twelve for eight pairs of bf16 rows
  constexpr bool EIGHT = PW == 4 || PW == 8 || (sizeof(T) == 2 && (PW <= 2 || (PW == 16 && D == 128)));
  // Sixteen pairs of few rows, d = 128: with up to three rows a lane the registers suffice for two workgroups on a compute
  // unit, which hide each other's chains (two layers, four rows a lane -> the fewest: S = 4 8192 pairs 23.2 -> 17.1 us, 65536 pairs
  // 165 -> 102; S = 12 23.4 -> 19.8 and 169 -> 119; three rows for 4096 pairs, one workgroup a compute unit, were slower:
  // 13.4 -> 15.1)
  constexpr bool FEW = PW == 16 && D == 128 && sizeof(T) == 2;
  // One or two rows a lane where that is all there is: with four, the rows past the last one are worked on too (4096 pairs,
  // S = 16, d = 64, bf16: 6.5 -> 5.8 us, the pass 3700 -> 1900 cycles of a workgroup's 14000)
  auto streamed = [&]() {
    if constexpr (PW == 16 && sizeof(T) == 2) {
      // The pooled maxima from the pass itself: read once more, the rows of many pairs with long blocks come from memory again
      // (d = 64, lengths full: 35621 pairs x 229 473 -> 230 us, 17520 x 110 118 -> 67; without the views 0.92 .. 1.0 of the split
      // form's times)
      if (a.M == 1 && a.pool_out != nullptr) {
        LASER_TILED_FORM(STREAM, false, true);
        return;
      }
    }
    LASER_TILED(STREAM, false);
  };
  if (a.S <= HELD) LASER_TILED(1, true);
  else if (a.S <= 2 * HELD) LASER_TILED(2, true);
  else if (FEW && a.S <= 3 * HELD && P > 256 * PW) LASER_TILED((FEW ? 3 : 4), true);
  else if (a.S <= 4 * HELD) LASER_TILED(4, true);
  else if constexpr (EIGHT) {
    if (a.S <= 8 * HELD) LASER_TILED(8, true);
    else if constexpr (PW == 8 && D == 128 && sizeof(T) == 2) {
      if (a.S <= 12 * HELD) LASER_TILED(12, true);
      else streamed();
    } else streamed();
  } else streamed();
#undef LASER_TILED
#undef LASER_TILED_FORM
}

// Pairs per workgroup: the fewest that leave the launch one round of workgroups (256 of eight waves for d = 128 and for
// fp32, whose products fill the matrix pipe; twice as many of four waves for d = 64 in bf16), since a layer's chain costs
// about the same for 1 and for 16 pairs. Two layers, bf16,
// d = 128, S = 32, PW = 1 / 2 / 4 / 8 / 16: 100 pairs 9.2 / 9.1 / 9.8 / 11.0 / 14.8 us, 512 pairs 14.8 / 9.6 / 10.0 / 11.0 / 15.0,
// 2048 pairs 45 / 26 / 16 / 11.8 / 15.5, 8192 pairs 157 / 82 / 48 / 41 / 34.
template <typename T, int D>
static void launch_t(const GstaArgs& a) {
  const int P = gsta_pairs(a), per = D == 128 || sizeof(T) == 4 ? P : (P + 1) / 2;
  if (per <= 256) launch_pairs<T, D, 1>(a, P);
  else if (per <= 512) launch_pairs<T, D, 2>(a, P);
  else if (per <= 1024) launch_pairs<T, D, 4>(a, P);
  // (d = 64 with 33 to 64 rows: eight rows a lane, for which sixteen pairs have no room: 8192 pairs, S = 50, two layers 21.9
  // against 23.7 us; one layer either way 17.5)
  else if (per <= 2048 || (D == 64 && a.S > 32 && a.S <= 64)) launch_pairs<T, D, 8>(a, P);
  else launch_pairs<T, D, 16>(a, P);
}

laser_status gsta_tile_launch(const GstaArgs& a) {
  if (!gsta_tile_supports(a)) return LASER_ERR_UNSUPPORTED;
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

bool gsta_tile_supports(const GstaArgs& a) { return a.d == 64 || a.d == 128; }

// Whether a one-layer bf16 batch runs on this kernel and not on the forms written for full machines (us, this kernel / the other,
// lengths full). At d = 64 it does: S = 2 65536 pairs 0.54 of the time, S = 16 8192 pairs 7.7 / 11.0, 32768 0.67, S = 32 65536
// 0.66, S = 64 8192 0.86, 65536 0.76; against the split form (longer blocks, up to 256) 37 calls past 16384 pairs, most with the
// views, lengths full 0.92 .. 1.05, uniform 0.83 .. 1.04, log-uniform 0.49 .. 0.88. At d = 128 it does for blocks of up to three
// rows a lane, S = 2 .. 12 with 3000 to 65536 pairs 0.58 .. 0.92. Up to 32 segments the one-kernel form is the better one once it
// fills a round of 256 workgroups of 32 pairs with more than half, and again a little into its second round.
// 500 calls at d = 128, 13 to 128 segments, 2500 to 50000 pairs without the views, this kernel's time over the other's, lengths full
// and with lengths, mean (range): on this side of the lines 0.79 (0.59 .. 1.09), 0.74 (0.57 .. 0.95). On the other side S <= 32 4097
// to 8192 pairs 1.14 (1.07 .. 1.24), 1.06 (0.94 .. 1.11), past 11264 1.04 (0.91 .. 1.20), 0.96 (0.81 .. 1.08); S = 33 .. 64 up to
// 16384 pairs 1.02 (0.95 .. 1.09), 0.91 (0.73 .. 1.07), more 1.16 (1.00 .. 1.31), 1.11 (0.87 .. 1.36); S = 65 .. 128 1.05
// (0.99 .. 1.18), 0.87 (0.59 .. 1.18). So past 8192 pairs with lengths given the lines, drawn for full ones and an earlier form of both
// kernels, leave calls there that would be faster here.
bool gsta_tile_preferred(const GstaArgs& a) {
  const int P = gsta_pairs(a);
  if (a.d == 64 || a.S <= 12) return true;
  if (!gsta_one_supports(a)) return P <= 8192;
  return P <= 4096 || (P > 8192 && P <= 11264);
}

}  // namespace laser
