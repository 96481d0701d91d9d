// The two projections around a pass over H' of its own (one layer, bf16 storage; the split form of GSTA in gsta_one.hip, FFN + GSTA
// in ffn_gsta.hip). The fp32 rows of z are what the three launches hand on:
//   gsta_r_kernel     r = (t0 W_q) W_k^T / sqrt(d)   -> z rows
//   (the pass)        p = softmax_i(H'_i . r) H'     z rows -> z rows
//   gsta_out_kernel   z = t0 + p W_v                 z rows -> z rows
// Products as in gsta_tiled.hip: a workgroup of d / 16 waves walks tiles of 16 pairs, a wave owns 16 columns of every product and
// keeps its share of the matrices in registers over the tiles; fp32 factors (q', p) enter as three bf16 parts (24 bits), t0 is
// bf16 as it is. The next tile's rows are on their way while one is multiplied.
//
// Bound by the start (launch, 64 or 32 KB of matrices a workgroup) and the chain of a tile. With FFN + GSTA between them,
// d = 128, against a tile of 32 pairs a workgroup, W_q fetched by 64 two-byte loads a lane and the factors in two parts: 192
// pairs 31.7 -> 27.9 us, 3000 46.5 -> 42.6, 16384 141.6 -> 138.6, 27000 106.4 -> 95.5 (20 segments).
#include "gsta_tile.h"
#include "laser_internal.h"

namespace laser {

// rows of 16 pairs from memory, whole rows of consecutive lanes: thread tid holds four values of row tid / (D / 4)
template <int D> __device__ __forceinline__ int flat_row(int tid) { return tid / (D / 4); }
template <int D> __device__ __forceinline__ int flat_col(int tid) { return tid % (D / 4) * 4; }

template <int D>
__global__ __launch_bounds__(4 * D, 4) void gsta_r_kernel(const unsigned short* __restrict__ t0, const unsigned short* __restrict__ wq,
                                                          const unsigned short* __restrict__ wk, int P, int tiles,
                                                          float* __restrict__ z) {
  typedef Prod<unsigned short, D> X;
  constexpr int NW = D / 16;
  __shared__ __attribute__((aligned(16))) unsigned short bt[X::template extent<16>(1)];   // (t0 is its own head)
  __shared__ __attribute__((aligned(16))) typename X::Act bq;
  __shared__ __attribute__((aligned(16))) unsigned char patches[NW][X::PATCH];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = wave * 16, c4 = n0 + 4 * g, row = flat_row<D>(tid), col = flat_col<D>(tid);
  auto rows_of = [&](int tile) {   // (rows past the last pair repeat it, and are not stored)
    const int p = tile * 16 + row < P ? tile * 16 + row : P - 1;
    return *reinterpret_cast<const u32x2*>(t0 + (size_t)p * D + col);
  };
  typename X::Cols cq;
  typename X::Operand rk;
  int tile = blockIdx.x;
  X::load_cols(cq, wq, n0, lane);
  u32x2 raw = rows_of(tile);
  X::load_rows(rk, wk, n0, lane);
  const typename X::Operand oq = X::transposed(cq, patches[wave], lane);
  const float scale = 1.0f / sqrtf((float)D);
  for (; tile < tiles; tile += gridDim.x) {
    *reinterpret_cast<u32x2*>(bt + X::template at<16>(0, row, col)) = raw;
    if (tile + (int)gridDim.x < tiles) raw = rows_of(tile + gridDim.x);
    __syncthreads();
    f32x4 q = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < D / 32; ++k)
      q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(oq.x[k], *reinterpret_cast<const bf16x8*>(bt + X::template at<16>(0, l16, k * 32 + g * 8)), q, 0, 0, 0);
    X::template put4<16>(bq, l16, c4, q);
    __syncthreads();   // (ahead of it every wave has read bt, ahead of the next tile's first one bq)
    const f32x4 r = X::template product<16>(bq, rk, lane) * scale;
    if (tile * 16 + l16 < P) *reinterpret_cast<f32x4*>(z + (size_t)(tile * 16 + l16) * D + c4) = r;
  }
}

template <int D>
__global__ __launch_bounds__(4 * D, 4) void gsta_out_kernel(const unsigned short* __restrict__ t0, const unsigned short* __restrict__ wv,
                                                            int P, int tiles, float* z) {
  typedef Prod<unsigned short, D> X;
  constexpr int NW = D / 16;
  __shared__ __attribute__((aligned(16))) typename X::Act bp[2];
  __shared__ __attribute__((aligned(16))) unsigned char patches[NW][X::PATCH];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = wave * 16, c4 = n0 + 4 * g, row = flat_row<D>(tid), col = flat_col<D>(tid);
  auto clamped = [&](int p) { return (size_t)(p < P ? p : P - 1) * D; };   // (rows past the last pair repeat it, and are not stored)
  typename X::Cols cv;
  int tile = blockIdx.x;
  X::load_cols(cv, wv, n0, lane);
  f32x4 p = *reinterpret_cast<const f32x4*>(z + clamped(tile * 16 + row) + col);
  typename X::Raw4 t = *reinterpret_cast<const typename X::Raw4*>(t0 + clamped(tile * 16 + l16) + c4);
  const typename X::Operand ov = X::transposed(cv, patches[wave], lane);
  for (int buf = 0; tile < tiles; tile += gridDim.x, buf ^= 1) {
    X::template put4<16>(bp[buf], row, col, p);
    const f32x4 base = X::wide4(t);
    if (const int next = tile + gridDim.x; next < tiles) {
      p = *reinterpret_cast<const f32x4*>(z + clamped(next * 16 + row) + col);
      t = *reinterpret_cast<const typename X::Raw4*>(t0 + clamped(next * 16 + l16) + c4);
    }
    __syncthreads();   // (one a tile: the other buffer was last read ahead of it)
    const f32x4 y = base + X::template product<16>(bp[buf], ov, lane);
    if (tile * 16 + l16 < P) *reinterpret_cast<f32x4*>(z + (size_t)(tile * 16 + l16) * D + c4) = y;
  }
}

// Two workgroups on a compute unit (four of four waves at d = 64), each walking its share of the tiles (one: 27000 pairs
// 95.5 -> 97.0; twice as many: 98.5, 16384 pairs 138.6 -> 144.1)
template <int D>
static void launch_r(const GstaArgs& a) {
  const int P = gsta_pairs(a), tiles = (P + 15) / 16, most = 512 * 128 / D;
  hipLaunchKernelGGL((gsta_r_kernel<D>), dim3((unsigned)(tiles < most ? tiles : most)), dim3(4 * D), 0, a.stream,
                     (const unsigned short*)a.t0, (const unsigned short*)a.wq, (const unsigned short*)a.wk, P, tiles, a.z_out);
}
template <int D>
static void launch_out(const GstaArgs& a) {
  const int P = gsta_pairs(a), tiles = (P + 15) / 16, most = 512 * 128 / D;
  hipLaunchKernelGGL((gsta_out_kernel<D>), dim3((unsigned)(tiles < most ? tiles : most)), dim3(4 * D), 0, a.stream,
                     (const unsigned short*)a.t0, (const unsigned short*)a.wv, P, tiles, a.z_out);
}

laser_status gsta_r_launch(const GstaArgs& a) {
  if (a.dt != LASER_BF16 || !(a.d == 64 || a.d == 128)) return LASER_ERR_UNSUPPORTED;
  if (a.d == 64) launch_r<64>(a);
  else launch_r<128>(a);
  return launch_status();
}

laser_status gsta_out_launch(const GstaArgs& a) {
  if (a.dt != LASER_BF16 || !(a.d == 64 || a.d == 128)) return LASER_ERR_UNSUPPORTED;
  if (a.d == 64) launch_out<64>(a);
  else launch_out<128>(a);
  return launch_status();
}

}  // namespace laser
