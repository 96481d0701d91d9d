// STA for fp32 storage on the fp32 matrix instructions (the usual widths, sigmoid gates, one head): the generic
// kernel's arithmetic (fp32 products, sums and gates), with the two contractions of Sec. 3.5.1 as MFMAs.
//
// v_mfma_f32_16x16x4_f32: a tile is 16 items x 16 candidates, four k-slots to an instruction. Both products are computed
// transposed, as in the bf16 kernels: Sc^T[item, cand] = K Q^T leaves lane (g, l) with candidate l and items 4g .. 4g+3 in
// its four registers, and register r of all four lane groups is, as it sits, the operand of acc^T[dcol, cand] += V^T P^T
// for the items {r, 4 + r, 8 + r, 12 + r}; the V operand of that step is row 4g + r at column l of a 16-column block. The
// k-slots of the scores are columns 16 j + 4g + m (m = 0..3 of one 16-byte load), the same for K and Q.
// Nothing goes through LDS on the way in: a wave loads the rows of its tile straight into operand registers (64-byte
// runs), which K and V traffic from L2 allows because every element meets 16 or 32 candidates.
//
// Split: a workgroup owns a user, 16 or 32 candidates and a segment (a few segments when they are short); its four waves
// take alternate item tiles of a segment, so that a single request still spreads over the chip, and their sums meet in LDS
// in a fixed order. Items past the end of a segment have a gate of exactly zero and zeros for values.
//
// Bound by the load - score - gate - sum chain of a tile, whose loads are not ahead of it (24 users x 50 candidates: waves wait
// 45 % of their cycles, the matrix pipe is busy 21 %; a 16 x 16 tile with d = d_q = 64 is 1024 cycles of it). Against the generic kernel (one candidate a wave, a score per
// lane): 24 users x 50 candidates, L = 1500, w = 100, 64 / 64: 217 -> 13.8 us; 1 x 16, L = 1024, w = 64: 23.7 -> 4.8 us.
#include "laser_internal.h"

namespace laser {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// NCT: candidate tiles of 16 per wave
template <int DQ, int D, int NCT>
__global__ __launch_bounds__(256) void sta_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                      const float* __restrict__ v, const int32_t* __restrict__ lens,
                                                      const int32_t* __restrict__ cand_off, int P, int C_all, int L,
                                                      int w, int S, int wi, int nsb, int ctiles, float inv_gamma,
                                                      float* __restrict__ seg_out, int32_t* __restrict__ seg_cnt) {
  constexpr int KJ = DQ / 16, DB = D / 16;
  __shared__ f32x4 red[3][NCT * DB][64];
  int b = blockIdx.x;
  const int sb = b % nsb;
  b /= nsb;
  const int ct = b % ctiles, u = b / ctiles;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = __builtin_amdgcn_readfirstlane(valid_len(lens, u, L));
  if (sb == 0 && ct == 0) write_seg_cnt(seg_cnt, u, n, L, w, S, tid, 256);
  const CandRange cr = cand_range(cand_off, u, C_all, P);
  const int cbase = ct * 16 * NCT;
  if (cbase >= cr.count) return;             // past this user's candidates (the whole workgroup leaves)
  const int part = wave % wi;                // which share of the segment's item tiles
  const int seg = sb * (4 / wi) + wave / wi;
  const int lo = seg * w;                    // (w <= L; a segment past S has no items)
  int hi = lo + w < L ? lo + w : L;
  if (hi > n) hi = n;
  if (seg >= S) hi = lo;

  f32x4 acc[NCT][DB];
#pragma unroll
  for (int c = 0; c < NCT; ++c)
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[c][db] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  if (lo + part * 16 < hi) {
    f32x4 qf[NCT][KJ];
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
      int cand = cbase + c * 16 + l16;       // (rows past the last candidate are not stored)
      cand = cand < cr.count ? cand : cr.count - 1;
#pragma unroll
      for (int j = 0; j < KJ; ++j)
        qf[c][j] = *reinterpret_cast<const f32x4*>(q + ((size_t)cr.first + cand) * DQ + j * 16 + g * 4);
    }
    const float* kU = k + (size_t)u * L * DQ + g * 4;
    // Values through a buffer descriptor of the tile's valid rows: rows past them read zeros (an infinity in a repeated valid row
    // would make their zero gates NaN), and one offset serves every load.
    const float* vU = v + (size_t)u * L * D;
    int v_off = (g * 4 * D + l16) * 4;
    for (int t0 = lo + part * 16; t0 < hi; t0 += wi * 16) {
      f32x4 kf[KJ];
      float vf[4][DB];
      const __amdgpu_buffer_rsrc_t v_rows = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(vU + (size_t)t0 * D), 0, (hi - t0 < 16 ? hi - t0 : 16) * D * 4, 0x00027000);   // (32-bit elements)
      asm volatile("" : "+v"(v_off));   // (keeps the sums with constants here, where they are the loads' immediate offsets)
      const int krow = t0 + l16 < hi ? t0 + l16 : hi - 1;
#pragma unroll
      for (int j = 0; j < KJ; ++j) kf[j] = *reinterpret_cast<const f32x4*>(kU + (size_t)krow * DQ + j * 16);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          vf[r][db] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(v_rows, v_off + (r * D + db * 16) * 4, 0, 0));
#pragma unroll
      for (int c = 0; c < NCT; ++c) {
        f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
          for (int m = 0; m < 4; ++m) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][m], qf[c][j][m], s, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = t0 + g * 4 + r < hi ? 1.0f / (1.0f + expf(-s[r] * inv_gamma)) : 0.0f;
#pragma unroll
          for (int db = 0; db < DB; ++db) acc[c][db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][db], p, acc[c][db], 0, 0, 0);
        }
      }
    }
  }
  // shares of one segment, in a fixed order
  if (wi > 1) {
    if (part > 0)
#pragma unroll
      for (int c = 0; c < NCT; ++c)
#pragma unroll
        for (int db = 0; db < DB; ++db) red[wave - wave / wi - 1][c * DB + db][lane] = acc[c][db];
    __syncthreads();
    if (part > 0) return;
    for (int o = 1; o < wi; ++o)
#pragma unroll
      for (int c = 0; c < NCT; ++c)
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[c][db] += red[wave + o - wave / wi - 1][c * DB + db][lane];
  }
  if (seg >= S) return;
#pragma unroll
  for (int c = 0; c < NCT; ++c) {
    const int cand = cbase + c * 16 + l16;
    if (cand < cr.count) {
      float* o = seg_out + (((size_t)cr.first + cand) * S + seg) * D + g * 4;
#pragma unroll
      for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(o + db * 16) = acc[c][db];
    }
  }
}

bool sta_f32_supports(const StaArgs& a) {
  return a.dt == LASER_F32 && a.heads == 1 && !a.softmax && (a.d_q == 32 || a.d_q == 64 || a.d_q == 128) &&
         (a.d == 64 || a.d == 128);
}

template <int DQ, int D>
static laser_status launch_widths(const StaArgs& a) {
  const int w = a.w < a.L ? a.w : a.L, tiles = (w + 15) / 16;
  const int wi = tiles >= 3 ? 4 : tiles;             // waves that share a segment
  const int nsb = (int)(((long long)a.S * wi + 3) / 4);
  // two candidate tiles a wave halve the reads of K and V; one tile where that would leave compute units without work
  const int c32 = (a.C + 31) / 32;
  const bool two = a.C > 16 && (long long)a.U * c32 * nsb >= 1024;
  const int ctiles = two ? c32 : (a.C + 15) / 16;
  const long long blocks = (long long)a.U * ctiles * nsb;
  if (blocks > 0x7fffffffLL) return LASER_ERR_SHAPE;
  const dim3 grid((unsigned)blocks), block(256);
  const float ig = 1.0f / a.gamma;
#define LASER_STA_F32(N)                                                                                            \
  hipLaunchKernelGGL((sta_f32_kernel<DQ, D, N>), grid, block, 0, a.stream, (const float*)a.q, (const float*)a.k,   \
                     (const float*)a.v, a.lens, a.cand_off, a.P, a.C, a.L, w, a.S, wi, nsb, ctiles, ig,            \
                     (float*)a.seg_out, a.seg_cnt)
  if (two) LASER_STA_F32(2);
  else LASER_STA_F32(1);
#undef LASER_STA_F32
  return launch_status();
}

laser_status sta_f32_launch(const StaArgs& a) {
  if (!sta_f32_supports(a)) return LASER_ERR_UNSUPPORTED;
  switch (a.d_q * 1000 + a.d) {
    case 32064: return launch_widths<32, 64>(a);
    case 32128: return launch_widths<32, 128>(a);
    case 64064: return launch_widths<64, 64>(a);
    case 64128: return launch_widths<64, 128>(a);
    case 128064: return launch_widths<128, 64>(a);
    default: return launch_widths<128, 128>(a);
  }
}

}  // namespace laser
