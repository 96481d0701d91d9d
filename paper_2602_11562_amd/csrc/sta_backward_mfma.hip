// Backward pass of STA on the bf16 matrix cores, for more than a few candidates per user (the equations stand at the
// top of sta_backward.hip). With C candidates sharing a history all five products are dense contractions:
//   S = Q K^T,  D = dH'_i V^T  (exact bf16 products, fp32 sums),  g = sigmoid(S / gamma),  ds = D g (1 - g) / gamma,
//   dV_i = G^T dH'_i,  dK_i = dS^T Q   (contracted over the candidates),   dQ = dS K   (contracted over the items).
// g and ds are fp32 and stay so: each enters its product as three bf16 parts (head, remainder, remainder of that: 24
// bits), three MFMAs on the same other operand, so the pass keeps fp32 precision at a third of the bf16 rate, still
// five times the rate of the fp32 matrix instructions.
//
// Two kinds of workgroup in one launch, because the two contractions want the scores the other way round:
//   items   a wave owns 32 items of one segment (their K and V rows are operands in registers, dK and dV accumulators)
//           and walks the candidates in blocks of 32 (rows of Q and dH'_i in LDS). S and D come out with lane = item and
//           candidates along the registers, which is, per 16 candidates, the left operand of dV and dK; the right
//           operand is the transpose load of the same LDS rows.
//   queries a wave owns 32 candidates (Q, and dH'_i of the segment in work, in registers) and walks the items of a run
//           of segments (rows of K and V in LDS); S and D are computed once more with lane = candidate, ds is the left
//           operand of dQ and the transpose load of the K rows the right one.
// Computing S and D twice costs 2 (d_q + d) of 3 (d_q + d) + 9 d_q + 3 d multiply-adds and replaces a transposition of ds
// through LDS; neither kind waits for the other and nothing but Q's partial sums crosses workgroups.
// A workgroup's four waves split over segments when a segment has few item tiles (or a user few candidate tiles):
// short segments and small candidate sets leave no wave idle. Rows past the end of a segment or past the last candidate
// are zeros in LDS, so they add nothing to any finite sum (padding of the history is never read); a wave whose sums come out
// not finite forms them again over the valid rows alone.
//
// What bounds it: waiting (36 % of the waves' cycles, 47 % before the rows of the next block were requested while the current one is
// worked on) and issue (29 %); the matrix pipe is busy 15 %. The rows go to LDS directly, two sets of them where the workgroups that
// registers allow on a compute unit still fit: 16 users x 64 candidates, L = 2000, w = 256, 128 / 128 41.6 -> 30 us, 1024 x 16, w = 10,
// 64 / 128 553 -> 398 us, 64 users x 64 candidates, L = 2048, w = 128, 64 / 64 (lengths 410 .. 2048) 32 -> 30 us for 128 MB, 20 us at
// the card's rate. The second set costs registers: 2 spill at 64 / 64 (none before), 3 at 64 / 128 (none), 43 at 128 / 128 (33), and
// loads return in order, so a reload in the block loop waits for the rows that were to overlap the products.
#include "laser_internal.h"
#include "sta_mfma_tile.h"

namespace laser {

// Position of 16-byte chunk c of row r in an LDS tile with rows of D bf16 values and no padding. Both access patterns
// stay free of bank conflicts: 16 consecutive rows at one chunk (operand reads, 16 bytes a lane) and four consecutive
// rows at four neighbouring chunks (transpose loads, 8 bytes a lane).
template <int D>
__device__ __forceinline__ int swz_key(int r) {
  return D == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : (D == 64 ? (((r >> 1) & 1) << 2) | ((r >> 2) & 3) : (r >> 2) & 3);
}
template <int D>
__device__ __forceinline__ int swz(int r, int c) { return r * (D * 2) + ((c ^ swz_key<D>(r)) << 4); }

// operand whose lanes are the rows of a tile: row l32, k-slots 16 ks + 8 h ..
template <int D>
__device__ __forceinline__ bf16x8 tile_rows(const unsigned char* t, int l32, int h, int ks) {
  return *reinterpret_cast<const bf16x8*>(t + swz<D>(l32, 2 * ks + h));
}
// operand whose lanes are the columns of a tile: column 32 db + l32, k-slots rows 16 s + {4h..4h+3, 8+4h..8+4h+3}
// (lane i of a 16-lane group supplies the address of row i / 4, columns 4 (i % 4) .. and receives column i of four rows)
template <int D>
__device__ __forceinline__ bf16x8 tile_cols(const unsigned char* t, int lane, int s, int db) {
  const int h = lane >> 5, i16 = lane & 15, col = db * 32 + (lane & 16) + 4 * (i16 & 3);
  const int r = s * 16 + h * 4 + (i16 >> 2);
  const int sub = (col & 4) * 2;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(t + swz<D>(r, col >> 3) + sub));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(t + swz<D>(r + 8, col >> 3) + sub));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// eight fp32 values as the sum of three bf16 operands (each remainder is exact)
struct Split3 { bf16x8 p[3]; };
__device__ __forceinline__ Split3 split3(const f32x16& x, int s) {
  Split3 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float a = x[s * 8 + e];
    const __bf16 h0 = (__bf16)a;
    const float r1 = a - (float)h0;
    const __bf16 h1 = (__bf16)r1;
    o.p[0][e] = h0;
    o.p[1][e] = h1;
    o.p[2][e] = (__bf16)(r1 - (float)h1);
  }
  return o;
}

// rows [0, rows) of a matrix with row pitch `pitch` elements (uniform, 32 rows below 4 GB) into a 32-row tile, zeros after them;
// `waves` waves share it. The rows go to LDS directly and are awaited by the caller.
template <int D>
__device__ __forceinline__ void stage_rows(unsigned char* t, const unsigned short* src, size_t pitch, int rows, int wave,
                                           int waves, int lane) {
  constexpr int CH = D / 8;
  const unsigned at = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)t);
  for (int g = wave; g < 32 * CH / 64; g += waves) {
    const int e = g * 64 + lane, r = e / CH, c = (e % CH) ^ swz_key<D>(r);
    if (r < rows) dma16(src, (unsigned)r * (unsigned)(pitch * 2) + c * 16, at + g * 1024);
    else *reinterpret_cast<u32x4*>(t + e * 16) = u32x4{0u, 0u, 0u, 0u};
  }
}
__device__ __forceinline__ void staged() { __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); }

// Whether any score gradient of a wave was not finite, from one of its column blocks of dK or dQ: every column of an item's
// or a query's row is a sum over all of its score gradients, and not finite if one of them is (zero times it is NaN).
__device__ __forceinline__ bool any_not_finite(const f32x16& x) {
  float zero = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero = fmaf(x[r], 0.0f, zero);
  return __any(!(zero == 0.0f));
}

// A row in the layout of the plain sums: lane l holds elements l, l + 64, ..
template <int D>
struct PlainRow {
  static constexpr int T = (D + 63) / 64;
  float x[T];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int t = 0; t < T; ++t) x[t] = 0.0f;
  }
  __device__ __forceinline__ void load(const unsigned short* p, int lane) {
#pragma unroll
    for (int t = 0; t < T; ++t) x[t] = lane + 64 * t < D ? bf16_bits_to_f32(p[lane + 64 * t]) : 0.0f;
  }
  __device__ __forceinline__ void store(float* p, int lane) const {
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (lane + 64 * t < D) p[lane + 64 * t] = x[t];
  }
  __device__ __forceinline__ float dot(const PlainRow& o) const {
    float s = 0.0f;
#pragma unroll
    for (int t = 0; t < T; ++t) s = fmaf(x[t], o.x[t], s);
    return wave_sum_rows(s);
  }
  __device__ __forceinline__ void add(float f, const PlainRow& o) {
#pragma unroll
    for (int t = 0; t < T; ++t) x[t] = fmaf(f, o.x[t], x[t]);
  }
};

struct StaBwdMfmaShape {
  int wi, ws_i;        // items: waves per segment, segments per workgroup (wi * ws_i = 4)
  int nsb, ntb;        // segment blocks, blocks of wi item tiles per segment
  int wc, ws_q;        // queries: candidate tiles and segments in work per workgroup (wc * ws_q = 4)
  int nct, groups, spg;
};

// PRE: two sets of tiles, the next block's rows on their way into one while the other is worked on (one barrier a block);
// half_lds: bytes of a set
template <int DQ, int D, bool PRE>
__global__ __launch_bounds__(256, DQ + D <= 128 ? 3 : 2) void sta_bwd_mfma_kernel(const unsigned short* __restrict__ q,
                                                              const unsigned short* __restrict__ k,
                                                              const unsigned short* __restrict__ v,
                                                              const unsigned short* __restrict__ dhp,
                                                              const int32_t* __restrict__ lens, int C, int L, int w,
                                                              int S, StaBwdMfmaShape sh, int query_blocks, int half_lds,
                                                              float neg_scale_log2e, float inv_gamma,
                                                              float* __restrict__ dk, float* __restrict__ dv,
                                                              float* __restrict__ dq_part) {
  constexpr int KQ = DQ / 16, KV = D / 16, QB = DQ / 32, VB = D / 32;
  constexpr int QBYTES = 32 * DQ * 2, VBYTES = 32 * D * 2;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ds in the place of D, g in the place of S
  auto gates = [&](f32x16& s, f32x16& dd) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float g = gate(s[r], neg_scale_log2e);
      s[r] = g;
      dd[r] = dd[r] * g * (1.0f - g) * inv_gamma;
    }
  };
  f32x16 zero16;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero16[r] = 0.0f;

  if ((int)blockIdx.x >= query_blocks) {
    // ------------------------------------------------------------------ items: dK and dV
    int b = blockIdx.x - query_blocks;
    const int tb = b % sh.ntb;
    b /= sh.ntb;
    const int sb = b % sh.nsb, u = b / sh.nsb;
    const int si = wave / sh.wi, ti = tb * sh.wi + wave % sh.wi;
    const int seg = sb * sh.ws_i + si;
    const int n = __builtin_amdgcn_readfirstlane(valid_len(lens, u, L));
    const int lo = seg * w + ti * 32;                    // (seg may be past S: then lo >= hi_all)
    int seg_end = seg < S ? seg * w + w : 0;
    if (seg_end > L) seg_end = L;
    const int rows_all = seg_end - lo < 32 ? seg_end - lo : 32;           // rows of the tile to write (<= 0: none)
    const int rows = (seg_end < n ? seg_end : n) - lo < 32 ? (seg_end < n ? seg_end : n) - lo : 32;
    const bool work_here = rows > 0;                     // wave-uniform
    // the first segment of the workgroup starts earliest: past the valid length there, nobody computes
    const bool any = sb * sh.ws_i * w + tb * sh.wi * 32 < n;

    bf16x8 kf[KQ], vf[KV];
    f32x16 dka[QB], dva[VB];
#pragma unroll
    for (int i = 0; i < QB; ++i) dka[i] = zero16;
#pragma unroll
    for (int i = 0; i < VB; ++i) dva[i] = zero16;
    if (any) {
      if (work_here) {
        const size_t row = (size_t)u * L + lo + (l32 < rows ? l32 : rows - 1);
#pragma unroll
        for (int ks = 0; ks < KQ; ++ks) kf[ks] = *reinterpret_cast<const bf16x8*>(k + row * DQ + ks * 16 + h * 8);
#pragma unroll
        for (int ks = 0; ks < KV; ++ks) vf[ks] = *reinterpret_cast<const bf16x8*>(v + row * D + ks * 16 + h * 8);
      }
      const int hseg = seg < S ? seg : S - 1;
      auto stage = [&](int c0, int buf) {
        const int nc = C - c0 < 32 ? C - c0 : 32;
        unsigned char* set = lds + (PRE ? buf * half_lds : 0);
        stage_rows<DQ>(set, q + ((size_t)u * C + c0) * DQ, DQ, nc, wave, 4, lane);
        stage_rows<D>(set + QBYTES + si * VBYTES, dhp + (((size_t)u * C + c0) * S + hseg) * D, (size_t)S * D, nc, wave % sh.wi, sh.wi, lane);
      };
      if (PRE) stage(0, 0);
      for (int c0 = 0, buf = 0; c0 < C; c0 += 32, buf ^= 1) {
        if (PRE) {
          staged();
          __syncthreads();
          if (c0 + 32 < C) stage(c0 + 32, buf ^ 1);
        } else {
          __syncthreads();
          stage(c0, 0);
          staged();
          __syncthreads();
        }
        const unsigned char* Qs = lds + (PRE ? buf * half_lds : 0);
        const unsigned char* Hs = Qs + QBYTES + si * VBYTES;
        if (work_here) {
          f32x16 s = zero16, dd = zero16;
#pragma unroll
          for (int ks = 0; ks < KQ; ++ks)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_rows<DQ>(Qs, l32, h, ks), kf[ks], s, 0, 0, 0);
#pragma unroll
          for (int ks = 0; ks < KV; ++ks)
            dd = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_rows<D>(Hs, l32, h, ks), vf[ks], dd, 0, 0, 0);
          gates(s, dd);
#pragma unroll
          for (int st = 0; st < 2; ++st) {
            const Split3 gs = split3(s, st);
#pragma unroll
            for (int db = 0; db < VB; ++db) {
              const bf16x8 x = tile_cols<D>(Hs, lane, st, db);
#pragma unroll
              for (int p = 2; p >= 0; --p) dva[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gs.p[p], x, dva[db], 0, 0, 0);
            }
            const Split3 ds = split3(dd, st);
#pragma unroll
            for (int db = 0; db < QB; ++db) {
              const bf16x8 x = tile_cols<DQ>(Qs, lane, st, db);
#pragma unroll
              for (int p = 2; p >= 0; --p) dka[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ds.p[p], x, dka[db], 0, 0, 0);
            }
          }
        }
      }
    }
    // Sums over score gradients that are not finite once more without the tiles: there a zero row that pads the candidates
    // meets an infinite key or value, and the zero parts of a split gate an infinite dH', and give NaN where the sum has none.
    const bool plain = work_here && any_not_finite(dka[0]);
    if (__builtin_expect(plain, 0)) {
      for (int row = 0; row < rows; ++row) {
        const size_t j = (size_t)u * L + lo + row;
        PlainRow<DQ> kr, qr, dkr;
        PlainRow<D> vr, hr, dvr;
        kr.load(k + j * DQ, lane);
        vr.load(v + j * D, lane);
        dkr.zero();
        dvr.zero();
        for (int c = 0; c < C; ++c) {
          qr.load(q + ((size_t)u * C + c) * DQ, lane);
          hr.load(dhp + (((size_t)u * C + c) * S + seg) * D, lane);
          const float gt = gate(kr.dot(qr), neg_scale_log2e);
          dvr.add(gt, hr);
          dkr.add(vr.dot(hr) * gt * (1.0f - gt) * inv_gamma, qr);
        }
        dkr.store(dk + j * DQ, lane);
        dvr.store(dv + j * D, lane);
      }
    }
    // lane = column, registers = items: whole 128-byte pieces of a row per store; rows past the valid length get zeros
    float* dkr = dk + ((size_t)u * L + lo) * DQ + l32;
    float* dvr = dv + ((size_t)u * L + lo) * D + l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 8 * (r >> 2) + 4 * h + (r & 3);
      if (row < rows_all && !(plain && row < rows)) {
        const bool ok = row < rows;
#pragma unroll
        for (int db = 0; db < QB; ++db) __builtin_nontemporal_store(ok ? dka[db][r] : 0.0f, dkr + (size_t)row * DQ + db * 32);
#pragma unroll
        for (int db = 0; db < VB; ++db) __builtin_nontemporal_store(ok ? dva[db][r] : 0.0f, dvr + (size_t)row * D + db * 32);
      }
    }
  } else {
    // ------------------------------------------------------------------ queries: dQ over a run of segments
    int b = blockIdx.x;
    const int grp = b % sh.groups;
    b /= sh.groups;
    const int ct = b % sh.nct, u = b / sh.nct;
    const int sq = wave / sh.wc;                                       // which of the segments in work
    const int cbase = (ct * sh.wc + wave % sh.wc) * 32;
    const bool mine = cbase < C;
    const int n = __builtin_amdgcn_readfirstlane(valid_len(lens, u, L));
    const int i_beg = grp * sh.spg;
    int i_end = i_beg + sh.spg < S ? i_beg + sh.spg : S;
    const int valid_segs = (n + w - 1) / w;
    if (i_end > valid_segs) i_end = valid_segs;
    const int tiles = (w + 31) / 32;                                   // (w <= L)
    const int crow = cbase + l32 < C ? cbase + l32 : C - 1;            // (rows past the last candidate are not stored)

    bf16x8 qf[KQ], hf[KV];
    f32x16 dqa[QB];
#pragma unroll
    for (int i = 0; i < QB; ++i) dqa[i] = zero16;
#pragma unroll
    for (int ks = 0; ks < KQ; ++ks)
      qf[ks] = *reinterpret_cast<const bf16x8*>(q + ((size_t)u * C + crow) * DQ + ks * 16 + h * 8);
    // item tile t of segment i0 + sq, for every wave at once; with one segment in work the history's end ends the walk
    struct At { int i0, t; };
    auto more = [&](const At& a) { return a.i0 < i_end && !(sh.ws_q == 1 && a.i0 * w + a.t * 32 >= n); };
    auto after = [&](const At& a) { return a.t + 1 < tiles ? At{a.i0, a.t + 1} : At{a.i0 + sh.ws_q, 0}; };
    auto items_of = [&](const At& a) {                                 // valid items of the tile (0: none)
      const int i = a.i0 + sq, end = i * w + w < n ? i * w + w : n, left = end - (i * w + a.t * 32);
      return i < i_end ? (left < 0 ? 0 : (left < 32 ? left : 32)) : 0;
    };
    auto stage = [&](const At& a, int buf) {
      const int rows = items_of(a);
      const size_t r0 = (size_t)u * L + (rows > 0 ? (a.i0 + sq) * w + a.t * 32 : 0);
      unsigned char* set = lds + (PRE ? buf * half_lds : 0) + sq * (QBYTES + VBYTES);
      stage_rows<DQ>(set, k + r0 * DQ, DQ, rows, wave % sh.wc, sh.wc, lane);
      stage_rows<D>(set + QBYTES, v + r0 * D, D, rows, wave % sh.wc, sh.wc, lane);
    };
    At cur = {i_beg, 0};
    if (PRE && more(cur)) stage(cur, 0);
    for (int buf = 0; more(cur); cur = after(cur), buf ^= 1) {
      {
        const int i = cur.i0 + sq, rows = items_of(cur);
        if (cur.t == 0 && i < i_end) {
#pragma unroll
          for (int ks = 0; ks < KV; ++ks)
            hf[ks] = *reinterpret_cast<const bf16x8*>(dhp + (((size_t)u * C + crow) * S + i) * D + ks * 16 + h * 8);
        }
        if (PRE) {
          staged();
          __syncthreads();
          const At nxt = after(cur);
          if (more(nxt)) stage(nxt, buf ^ 1);
        } else {
          __syncthreads();
          stage(cur, 0);
          staged();
          __syncthreads();
        }
        const unsigned char* Ks = lds + (PRE ? buf * half_lds : 0) + sq * (QBYTES + VBYTES);
        const unsigned char* Vs = Ks + QBYTES;
        if (rows > 0 && mine) {
          f32x16 s = zero16, dd = zero16;
#pragma unroll
          for (int ks = 0; ks < KQ; ++ks)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_rows<DQ>(Ks, l32, h, ks), qf[ks], s, 0, 0, 0);
#pragma unroll
          for (int ks = 0; ks < KV; ++ks)
            dd = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_rows<D>(Vs, l32, h, ks), hf[ks], dd, 0, 0, 0);
          gates(s, dd);
#pragma unroll
          for (int st = 0; st < 2; ++st) {
            const Split3 ds = split3(dd, st);
#pragma unroll
            for (int db = 0; db < QB; ++db) {
              const bf16x8 x = tile_cols<DQ>(Ks, lane, st, db);
#pragma unroll
              for (int p = 2; p >= 0; --p) dqa[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ds.p[p], x, dqa[db], 0, 0, 0);
            }
          }
        }
      }
    }
    // the waves that shared these candidates add up in a fixed order
    if (sh.ws_q > 1) {
      __syncthreads();
      float* red = reinterpret_cast<float*>(lds);
      if (sq > 0) {
        float* o = red + ((size_t)((sq - 1) * sh.wc + wave % sh.wc) * QB * 16) * 64 + lane;
#pragma unroll
        for (int db = 0; db < QB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[(db * 16 + r) * 64] = dqa[db][r];
      }
      __syncthreads();
      if (sq > 0) return;
      for (int o = 1; o < sh.ws_q; ++o) {
        const float* src = red + ((size_t)((o - 1) * sh.wc + wave) * QB * 16) * 64 + lane;
#pragma unroll
        for (int db = 0; db < QB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) dqa[db][r] += src[(db * 16 + r) * 64];
      }
    }
    if (__builtin_expect(any_not_finite(dqa[0]), 0)) {   // as for the items: padding rows of a tile meet an infinite dH'
      for (int c = cbase; c < C && c < cbase + 32; ++c) {
        PlainRow<DQ> qr, kr, dqr;
        PlainRow<D> hr, vr;
        qr.load(q + ((size_t)u * C + c) * DQ, lane);
        dqr.zero();
        for (int i = i_beg; i < i_end; ++i) {
          hr.load(dhp + (((size_t)u * C + c) * S + i) * D, lane);
          const int hi = i * w + w < n ? i * w + w : n;
          for (int j = i * w; j < hi; ++j) {
            kr.load(k + ((size_t)u * L + j) * DQ, lane);
            vr.load(v + ((size_t)u * L + j) * D, lane);
            const float gt = gate(qr.dot(kr), neg_scale_log2e);
            dqr.add(vr.dot(hr) * gt * (1.0f - gt) * inv_gamma, kr);
          }
        }
        dqr.store(dq_part + (((size_t)u * sh.groups + grp) * C + c) * DQ, lane);
      }
      return;
    }
    float* out = dq_part + (((size_t)u * sh.groups + grp) * C) * DQ + l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int c = cbase + 8 * (r >> 2) + 4 * h + (r & 3);
      if (c < C)
#pragma unroll
        for (int db = 0; db < QB; ++db) out[(size_t)c * DQ + db * 32] = dqa[db][r];
    }
  }
}

static int waves_for(int tiles) { return tiles >= 3 ? 4 : tiles; }   // 1, 2 or 4 waves share the tiles

static StaBwdMfmaShape sta_bwd_mfma_shape(const StaBwdArgs& a, int max_groups) {
  StaBwdMfmaShape s;
  const int seg = a.w < a.L ? a.w : a.L, tiles = (seg + 31) / 32, ct = (a.C + 31) / 32;
  s.wi = waves_for(tiles);
  s.ws_i = 4 / s.wi;
  s.nsb = (a.S + s.ws_i - 1) / s.ws_i;
  s.ntb = (tiles + s.wi - 1) / s.wi;
  s.wc = waves_for(ct);
  s.ws_q = 4 / s.wc;
  s.nct = (ct + s.wc - 1) / s.wc;
  // runs of segments: two workgroups per compute unit (as many as fit at once, three at d_q + d <= 128), each run a multiple of the
  // segments in work; every further run costs a partial sum of dQ in memory
  const long long users = (long long)a.U * s.nct;
  long long g = (512 + users - 1) / users;
  if (g > max_groups) g = max_groups;
  long long spg = (a.S + g - 1) / g;
  spg = (spg + s.ws_q - 1) / s.ws_q * s.ws_q;
  if (spg > a.S) spg = a.S;
  s.spg = (int)spg;
  s.groups = (a.S + s.spg - 1) / s.spg;
  return s;
}

// From five candidates on (us, the other kernel / here, full histories). Up to four the several-items-per-wave kernel streams the
// history once and is the faster one for short segments (2048 users x 4, L = 1000, w = 10: 32 / 128 561 / 860, 64 / 64 399 / 579); for
// long ones the two are about even (512 x 4, L = 2000, w = 64: 128 / 128 398 / 397, 64 / 64 195 / 178), which is left on the one line.
// Beyond four the alternative is one item per wave, eight candidates a pass: 512 x 5, L = 1000, w = 10, 32 / 128 318 / 200, 512 x 8,
// L = 2000, w = 64, 128 / 128 918 / 405. Not for segments so short that their tiles of 32 items x 32 candidates are nearly empty,
// where there are enough of them to fill the machine (L = 300): 1024 users x 5, w = 1, 128 / 64 453 / 1111, 512 x 8, w = 3, 64 / 128
// 172 / 197, 512 x 5, w = 5, 128 / 128 142 / 188 (w = 6, on this side of the line: 147 / 166); the second pass that nine candidates
// cost there moves the line to 18 products of a segment (512 x 9, w = 2, 64 / 128, on this side of 18: 312 / 284), and from 13 on this kernel
// is the better one for any segment (12, w = 1: 567 / 569).
bool sta_bwd_mfma_supports(const StaBwdArgs& a) {
  if ((long long)a.U * a.S >= 6144 && (long long)a.C * a.w <= (a.C <= 8 ? 25 : a.C <= 12 ? 18 : 0)) return false;
  return a.dt == LASER_BF16 && !a.grads_bf16 && a.C > 4 && (a.d_q == 32 || a.d_q == 64 || a.d_q == 128) &&
         (a.d == 64 || a.d == 128);
}

template <int DQ, int D>
static laser_status launch_shape(const StaBwdArgs& a, const StaBwdMfmaShape& s, float* part) {
  const long long qb = (long long)a.U * s.nct * s.groups, ib = (long long)a.U * s.nsb * s.ntb;
  if (qb + ib > 0x7fffffffLL) return LASER_ERR_SHAPE;
  const int items = 32 * DQ * 2 + s.ws_i * 32 * D * 2, queries = s.ws_q * (32 * DQ * 2 + 32 * D * 2);
  const int reduce = (s.ws_q - 1) * s.wc * DQ * 32 * 4;
  const int set = items > queries ? items : queries;
  // two sets of tiles while as many workgroups as registers allow still fit a compute unit, and more than one block to walk
  const bool pre = 2 * (DQ + D <= 128 ? 3 : 2) * set <= 160 * 1024 && (a.C > 32 || s.spg > s.ws_q || a.w > 32);
  int lds = pre ? 2 * set : set;
  if (reduce > lds) lds = reduce;
  const float inv_gamma = 1.0f / a.gamma;
  auto kern = pre ? sta_bwd_mfma_kernel<DQ, D, true> : sta_bwd_mfma_kernel<DQ, D, false>;
  // (the same limit whatever the call, half a compute unit's LDS at most is asked for: threads do not lower each other's)
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024) != hipSuccess)
    return LASER_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, dim3((unsigned)(qb + ib)), dim3(256), lds, a.stream,
                     (const unsigned short*)a.q, (const unsigned short*)a.k, (const unsigned short*)a.v,
                     (const unsigned short*)a.dhp, a.lens, a.C, a.L, a.w < a.L ? a.w : a.L, a.S, s, (int)qb, set,
                     -1.4426950408889634f * inv_gamma, inv_gamma, static_cast<float*>(a.dk), static_cast<float*>(a.dv),
                     part);
  return launch_status();
}

// groups: in, the partial sums of dQ that a.work holds per user; out, how many were written (1: straight into a.dq)
laser_status sta_bwd_mfma_launch(const StaBwdArgs& a, int* groups) {
  if (!sta_bwd_mfma_supports(a)) return LASER_ERR_UNSUPPORTED;
  const StaBwdMfmaShape s = sta_bwd_mfma_shape(a, *groups);
  *groups = s.groups;
  float* part = s.groups == 1 ? a.dq : a.work;
  switch (a.d_q * 1000 + a.d) {
    case 32064: return launch_shape<32, 64>(a, s, part);
    case 32128: return launch_shape<32, 128>(a, s, part);
    case 64064: return launch_shape<64, 64>(a, s, part);
    case 64128: return launch_shape<64, 128>(a, s, part);
    case 128064: return launch_shape<128, 64>(a, s, part);
    default: return launch_shape<128, 128>(a, s, part);
  }
}

}  // namespace laser
