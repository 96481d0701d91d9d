// Segment FFN + LayerNorm (paper Sec. 3.4.2, s <- LN(FFN(s) + s)) feeding the GSTA layer (Sec. 3.4.3) from one pass
// over H': the normalised segment vectors of a pair are scored against r = W_k (t0 W_q)^T / sqrt(d) and pooled with
// their softmax weights while they are still on chip, so the transformed H' is neither written nor read back
// (it is written as well when the caller wants it). One layer, bf16, d = 128, d_ff in {64, 128}.
//
// Three launches, the outer two shared with the split form of GSTA (gsta_project.hip):
//   gsta_r_kernel     r = (t0 W_q) W_k^T / sqrt(d)   tiles of 16 pairs, MFMA                       -> z rows
//   ffn_pool_kernel   below: a wave walks pairs       H' rows -> s rows (on chip), z rows (r) -> z rows (p)
//   gsta_out_kernel   z = t0 + p W_v                  tiles of 16 pairs, MFMA             z rows -> z rows
// with p = sum_i a_i s_i, a = softmax over the segments that hold a valid item of r . s_i (the attention equation
// with its products re-associated, which is exact).
//
// ffn_pool_kernel: the FFN tile of segment_ffn_tile.h on the valid rows (the first nv segments, the ones that hold a
// valid item) of the pairs a wave is dealt, one pair after the other, cut into tiles of 32 as one
// stream: a tile holds rows of one pair, or the last rows of one followed by the first of the next, so that only the
// wave's last tile is padded (with copies of its last row, which count as empty). The rows of the remaining segments
// are never read (whatever H' holds there is not trusted): they, and the results of a pair without any valid
// segment, are written by a pass of their own before the first tile. The rows of the wave's next tile and r of the
// pairs that start in it are in flight while it multiplies. After LayerNorm a lane holds, in the accumulator layout,
// 64 of the 128 components of row l32, rounded (what a stored s would hold): per 16 components a valid B operand, so
// the scores are one more product, r times the rows, and p = sum_i a_i s_i is another over the rows parked in the
// wave's LDS patch (transpose loads). r and the weights a are fp32 and stay so: both enter as three bf16 parts, which
// hold all 24 bits, in three rows of the A operand that are added afterwards. A tile holds rows of at most two pairs;
// they have a slot each, by the parity of their number: half h of the wave owns slot h, its scores, running maximum
// and sum (online softmax over a pair's tiles) and running p, and a row's weight is zero in the other slot.
//
// Vector issue and the matrix pipe of the two waves per SIMD bound the tile: 12.2 thousand cycles (the products 4.8, the
// normalised rows and their scores 3.1, softmax and sum 1.6, addresses and requests 1.4). Scores as four vector
// operations per word and the weighted sum row by row (a word, a weight from v_readlane, five to seven operations) were 350
// of 1100 vector instructions, another hundred where two pairs met; the two products take 16 MFMAs. With the launches before
// and behind it, 16384 pairs of 60 valid rows, d_ff = 128, rows not stored: 137.3 -> 127.2 us, with the views 145.5 -> 142.0.
// With waves a fixed 2048 pairs apart, all waves of 32 workgroups see the same eight users of 64, and the longest histories
// decide: where that matters a workgroup takes every 256th pair, which sees every user, and deals them to its waves by their
// valid rows (lengths uniform in [200, 1000], w = 10, 64 x 256 pairs, with the views and the launches around it 154 -> 141 us; by
// an LDS counter, which would make the sums of a pair depend on the run, 145).
#include "segment_ffn_tile.h"

namespace laser {

// Request a tile that holds rows of two pairs: rows a0 .. a0 + na - 1 of the pair whose row 0 is at `rowsA`, then rows
// 0 .. nb - 1 of the pair whose row 0 lies dB bytes further (nb >= 1); tile rows past the last one repeat it.
__device__ __forceinline__ void ffn_fetch_rows_two(const unsigned short* rowsA, int a0, int na, unsigned dB, int nb,
                                                   unsigned land, int lane) {
  asm volatile("" : "+v"(lane));   // (as in ffn_fetch_rows)
  const int q = lane >> 4, pos = lane & 15;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  const int last = na + nb - 1;
#pragma unroll
  for (int j = 0; j < FM_ROWS / 4; ++j) {
    const int row = 4 * j + q;
    const int src = row < last ? row : last;
    const unsigned off = src < na ? (unsigned)(a0 + src) * FM_ROWB : dB + (unsigned)(src - na) * FM_ROWB;
    ffn_dma16(rowsA, off + ((pos ^ (row & 15)) << 4), land + j * 1024);
  }
}

// x as three bf16 parts in the upper halves of hi, mid and lo (24 bits by truncation: the sum is x)
__device__ __forceinline__ void ffn_three_parts(float x, unsigned& hi, unsigned& mid, unsigned& lo) {
  hi = __float_as_uint(x) & 0xffff0000u;
  const float r1 = x - __uint_as_float(hi);
  mid = __float_as_uint(r1) & 0xffff0000u;
  lo = __float_as_uint(r1 - __uint_as_float(mid));
}

// Component-wise maximum of two words of bf16 values below 2^120: below 2^121 their bits are ordered as fp16's are. NaN
// words lose, as in fmaxf; -infinity (0xff80) is a NaN here, so it is a start value that every value replaces.
__device__ __forceinline__ unsigned ffn_word_max(unsigned a, unsigned b) {
  unsigned m;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
  return m;
}
constexpr unsigned FG_NONE = 0xff80ff80u;   // a word of bf16 -infinities

// Sum and maximum over the 32 lanes of a half of the wave, in all of them (lane permutations, no LDS)
__device__ __forceinline__ float ffn_half_sum(float v) {
  const unsigned x = __float_as_uint(row_sum<16>(v));
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float ffn_half_max(float v) {
  const unsigned x = __float_as_uint(ffn_row_max(v));
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

constexpr int FG_DECKS = 16;

// MR: also the two other views of Sec. 3.4.4 of the transformed rows: pool [P, D] bf16, the component-wise maximum
// over the segments that hold a valid item (zeros when there is none), taken from the parked rows (tile rows past the
// last one are copies of it, so they leave the maximum alone); recent [P, r, D] bf16, the first r rows as they would
// be stored. Either may be null.
// DEAL: a workgroup takes every (number of workgroups)-th pair and deals them to its waves by their valid rows (at most 64 FG_DECKS
// pairs a workgroup); without it a wave takes every (number of waves)-th pair.
template <int DFF, bool MR, bool DEAL>
__global__ __launch_bounds__(FM_THREADS) void ffn_pool_kernel(
    const unsigned short* seg, const int32_t* __restrict__ lens, const unsigned short* __restrict__ w1,
    const float* __restrict__ b1, const unsigned short* __restrict__ w2, const float* __restrict__ b2,
    const float* __restrict__ ln_g, const float* __restrict__ ln_b, const int32_t* __restrict__ cand_off, int U, int P,
    int C, int L, int w, int S, float eps,
    unsigned short* out,   // s rows [P, S, D], may be null (not wanted), may be seg
    float* z,              // [P, D]: r on entry, p on exit
    unsigned* pool, unsigned short* recent, int r) {
  constexpr int D = FM_D, KSTEPS = D / 16, DB = D / 32, OP = FM_OP;
  // per wave: r of the pairs that start in the next tile, by slot (fp32, as it lands), and the three parts of r of the pairs in
  // work, rows 3 slot + part of pitch RPP (16 rows read at once start in different banks)
  constexpr int RVB = 512, RPP = D * 2 + 16, RPB = 6 * RPP;
  constexpr int WPO = FM_ROWS * OP;        // the weights' parts: six rows of 64 bytes behind the patch's rows
  constexpr int NO_PAIR = 255;
  static_assert(WPO + 6 * 64 <= FM_PATCH, "the weights' parts fit behind the patch's rows");
  __shared__ __attribute__((aligned(1024))) unsigned char W1L[FM_W1B];
  __shared__ __attribute__((aligned(1024))) unsigned char W2L[DFF * FM_ROWB];
  __shared__ __attribute__((aligned(1024))) unsigned char patch[FM_WAVES * FM_PATCH];
  __shared__ __attribute__((aligned(1024))) unsigned char rvec[FM_WAVES * 2 * RVB];
  __shared__ __attribute__((aligned(16))) unsigned char rparts[FM_WAVES * RPB];
  __shared__ __attribute__((aligned(16))) float vecs[DFF + 3 * D];                    // b1, b2, ln_g, ln_b
  __shared__ unsigned char dealt[DEAL ? FG_DECKS : 1][64];   // the waves' pairs, 64 at a time, eight a wave

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* opatch = patch + wave * FM_PATCH;
  const unsigned land = __builtin_amdgcn_readfirstlane(ffn_lds_addr(opatch));
  unsigned char* rmine = rvec + wave * 2 * RVB;
  const unsigned rland = __builtin_amdgcn_readfirstlane(ffn_lds_addr(rmine));
  // pairs pr0 + k * stride: the workgroup's, or the wave's
  const int stride = DEAL ? gridDim.x : gridDim.x * FM_WAVES;
  const int pr0 = DEAL ? blockIdx.x : blockIdx.x * FM_WAVES + wave;
  // segments of pair p that hold a valid item (the first ones)
  auto valid_segments = [&](int p) {
    const int n = (valid_len(lens, pair_user(cand_off, U, C, p), L) + w - 1) / w;
    return __builtin_amdgcn_readfirstlane(n < S ? n : S);
  };
  constexpr int LPR = D / 8, RPI = 64 / LPR;
  const int nr = (MR && recent) ? (r < S ? r : S) : 0;
  ffn_park_weights<DFF>(__builtin_amdgcn_readfirstlane(ffn_lds_addr(W1L)), __builtin_amdgcn_readfirstlane(ffn_lds_addr(W2L)),
                        vecs, w1, w2, b1, b2, ln_g, ln_b, tid);
  // The workgroup's pairs, 64 at a time, are dealt to its waves by their valid segments: in that order (by number among equals)
  // to waves 0 .. 7, 7 .. 0, 0 .. 7 and so on. Wave i works this out for the i-th 64 of every 512 and leaves each wave's pairs, by
  // number, in LDS.
  if constexpr (DEAL) {
    for (int c = wave; c < FG_DECKS; c += FM_WAVES) {
      dealt[c][lane] = NO_PAIR;
      if (pr0 + 64 * c * stride >= P) continue;
      const int p = pr0 + (64 * c + lane) * stride;
      int key = 63 - lane;
      if (p < P) {
        const int n = (valid_len(lens, pair_user(cand_off, U, C, p), L) + w - 1) / w;
        key += (n < S ? n : S) * 64;
      }
      int rank = 0;
#pragma unroll
      for (int j = 0; j < 64; ++j) rank += __builtin_amdgcn_readlane(key, j) > key ? 1 : 0;
      const int lap = rank & (2 * FM_WAVES - 1), to = lap < FM_WAVES ? lap : 2 * FM_WAVES - 1 - lap;
      int at = 0;
#pragma unroll
      for (int i = 0; i < FM_WAVES; ++i) {
        const unsigned long long deck = __ballot(p < P && to == i);
        const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(deck >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)deck, 0));
        at = to == i ? before : at;
      }
      if (p < P) dealt[c][to * FM_WAVES + at] = (unsigned char)lane;
    }
    __syncthreads();
  }
  int turn = 0;   // pairs of this wave so far
  // The wave's next pair that has a valid segment (nvk > 0), else nvk = 0. Every pair of the
  // wave is looked at here exactly once, in order, and gets what the tiles never touch: the rows of its segments
  // without a valid item leave as zeros, and a pair without any has p = 0 and a pooled maximum of zeros.
  auto next_pair = [&](int& nvk) {
    nvk = 0;
    int k = 0;
    while (true) {
      if constexpr (DEAL) {
        if (turn == FG_DECKS * FM_WAVES) break;
        const int b = __builtin_amdgcn_readfirstlane(dealt[turn / FM_WAVES][wave * FM_WAVES + turn % FM_WAVES]);
        if (b == NO_PAIR) break;
        k = 64 * (turn / FM_WAVES) + b;
      } else {
        k = turn;
        if (pr0 + k * stride >= P) break;
      }
      ++turn;
      const int p = pr0 + k * stride;
      nvk = valid_segments(p);
      if (out)
        for (int i = nvk + lane / LPR; i < S; i += RPI)
          *reinterpret_cast<u32x4*>(out + ((size_t)p * S + i) * D + (lane % LPR) * 8) = u32x4{0u, 0u, 0u, 0u};
      if (MR && recent)
        for (int i = nvk + lane / LPR; i < nr; i += RPI)
          *reinterpret_cast<u32x4*>(recent + ((size_t)p * r + i) * D + (lane % LPR) * 8) = u32x4{0u, 0u, 0u, 0u};
      if (nvk > 0) break;
      if (MR && pool) pool[(size_t)p * (D / 2) + lane] = 0u;
      *reinterpret_cast<f32x2*>(z + (size_t)p * D + 2 * lane) = f32x2{0.0f, 0.0f};
    }
    return k;
  };
  // The valid rows of the wave's pairs, one pair after the other, are cut into tiles of 32: a tile holds rows
  // a0 .. a0 + na - 1 of pair A and, when A ends inside it and there is room, the first nb rows of the next pair
  // with a valid segment, B (which may end inside the tile too). ord counts the pairs with a valid segment.
  struct Tile {
    bool some;
    int kA, nvA, a0, na;
    int kB, nvB, nb;   // with A ending in the tile: the next pair (nvB == 0: there is none) and its rows in the tile
    int ord;
  };
  auto make_tile = [&](int k, int nvk, int off, int ord) {
    Tile t;
    t.some = nvk > 0;
    t.kA = k; t.nvA = nvk; t.a0 = off; t.ord = ord;
    t.na = nvk - off < FM_ROWS ? nvk - off : FM_ROWS;
    t.kB = k; t.nvB = 0; t.nb = 0;
    if (t.some && off + t.na == nvk) {
      t.kB = next_pair(t.nvB);
      const int room = FM_ROWS - t.na;
      t.nb = t.nvB < room ? t.nvB : room;
    }
    return t;
  };
  auto tile_after = [&](const Tile& t) {
    if (t.a0 + t.na < t.nvA) return make_tile(t.kA, t.nvA, t.a0 + t.na, t.ord);   // A goes on
    if (t.nb < t.nvB) return make_tile(t.kB, t.nvB, t.nb, t.ord + 1);             // B goes on (or starts)
    int nvn = 0, kn = t.kB;
    if (t.nvB > 0) kn = next_pair(nvn);                                  // B ended here as well
    return make_tile(kn, nvn, 0, t.ord + 2);
  };
  auto fetch_r = [&](int p, int slot) {   // 512 bytes: 16 per lane of the lower half of the wave
    if (lane < 32) ffn_dma16(z + (size_t)p * D, (unsigned)(lane << 4), rland + (slot & 1) * RVB);
  };
  // r of the pairs that start in tile t (landed) in its parts, behind the last use of the parts before. The product wants a
  // 16-group's components in the order 0..3, 8..11, 4..7, 12..15: word w (components 2 w, 2 w + 1) at 4 (w / 2 & 1) + 2
  // (w / 4) + w % 2.
  unsigned char* rpmine = rparts + wave * RPB;
  // (Offsets of lanes that are used once per tile are worked out where they are used, from a lane number the compiler cannot tell
  // from a fresh value: kept across the products they are spilled, and a reload waits for the fetches before it.)
  auto lane_again = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  auto park_r = [&](const Tile& t) {
    const int l = lane_again();
    unsigned char* rpword = rpmine + (l >> 3) * 32 + (4 * ((l >> 1) & 1) + 2 * ((l >> 2) & 1) + (l & 1)) * 4;
    auto park = [&](int slot) {
      const f32x2 rv = *reinterpret_cast<const f32x2*>(rmine + slot * RVB + l * 8);
      unsigned a[3], b[3];
      ffn_three_parts(rv[0], a[0], a[1], a[2]);
      ffn_three_parts(rv[1], b[0], b[1], b[2]);
#pragma unroll
      for (int part = 0; part < 3; ++part)
        *reinterpret_cast<unsigned*>(rpword + (3 * slot + part) * RPP) = (a[part] >> 16) | (b[part] & 0xffff0000u);
    };
    if (t.a0 == 0) park(t.ord & 1);
    if (t.nb > 0) park((t.ord + 1) & 1);
  };
  // the rows of tile t into the landing area, and r of the pairs that start in it
  auto fetch_tile = [&](const Tile& t) {
    const int pA = pr0 + t.kA * stride;
    const unsigned short* rowsA = seg + (size_t)pA * S * D;
    if (t.nb == 0) {
      ffn_fetch_rows(rowsA + (size_t)t.a0 * D, t.na - 1, land, lane);
    } else {
      const unsigned dB = (unsigned)(t.kB - t.kA) * (unsigned)stride * (unsigned)S * (unsigned)(D * 2);
      ffn_fetch_rows_two(rowsA, t.a0, t.na, dB, t.nb, land, lane);
      fetch_r(pr0 + t.kB * stride, t.ord + 1);
    }
    if (t.a0 == 0) fetch_r(pA, t.ord);
  };

  int nv0 = 0;
  const int k0 = next_pair(nv0);
  Tile cur = make_tile(k0, nv0, 0, 0);
  if (cur.some) fetch_tile(cur);

  ffn_wait_fetches();
  __syncthreads();
  const float* b1s = vecs;
  const float* b2s = vecs + DFF;
  const float* gs = vecs + DFF + D;
  const float* bs = vecs + DFF + 2 * D;
  FfnLane ln;
  ln.init(lane);
  const unsigned char* opr = opatch + (lane / LPR) * OP + (lane % LPR) * 16;
  const unsigned char* pcol = opatch + lane * 4;   // components 2 lane, 2 lane + 1 of row 0

  // gamma and beta are of a size that keeps rows plain (see below)
  bool gb_ok;
  {
    const f32x2 g2 = *reinterpret_cast<const f32x2*>(gs + 2 * lane), b2v = *reinterpret_cast<const f32x2*>(bs + 2 * lane);
    const float lim = 0x1p60f;
    gb_ok = __all(fabsf(g2[0]) < lim && fabsf(g2[1]) < lim && fabsf(b2v[0]) < lim && fabsf(b2v[1]) < lim);
  }

  bf16x8 xreg[KSTEPS];
  if (cur.some) ffn_read_rows(opatch, l32, h, xreg);
  if (cur.some) park_r(cur);
  // of the half's slot, over the pair's tiles: running maximum, sum of weights and p (components 16 b + i16, in both groups of 16)
  float m = -INFINITY, den = 0.0f, psum[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) psum[b] = 0.0f;
  unsigned mx = FG_NONE;       // pooled maximum of pair A, components 2 lane and 2 lane + 1
  bool rough = !gb_ok;         // a row's values may be large or not finite (from the tile where that was seen on)
  while (cur.some) {
    const Tile nxt = tile_after(cur);
    if (nxt.some) fetch_tile(nxt);
    const int na = cur.na, nb = cur.nb, ntot = na + nb;
    const int pA = pr0 + cur.kA * stride, pB = pr0 + cur.kB * stride;
    const bool slotA = h == (cur.ord & 1);                      // this half owns pair A's slot
    const bool mine = l32 < ntot && (l32 >= na) != slotA;       // row l32 belongs to this half's pair
    const bool fresh = !slotA || cur.a0 == 0;                   // ... which starts in this tile
    f32x16 acc[DB];
    __builtin_amdgcn_s_setprio(2);   // the other wave of the SIMD has vector work for the matrix instructions' shadow: 1.5 % of the pass
    ffn_tile_products<DFF>(xreg, ln, W1L, W2L, b1s, b2s, l32, h, acc);
    __builtin_amdgcn_s_setprio(0);
    if (nxt.some) {   // the next tile's rows move into the registers of this one's before the patch is written
      ffn_wait_fetches();
      ffn_read_rows(opatch, l32, h, xreg);
    }
    float rstd, nmr;
    ffn_row_stats(acc, eps, rstd, nmr);
    // The fast forms below add rows of two pairs with weights of zero and compare bits as fp16. A row is plain when its mean is
    // finite and moderate (nmr = -mean rstd): its normalised values are then below 12 (1 + |nmr|) < 2^45, and with gamma and beta
    // below 2^60 all of them below 2^106.
    rough = rough || !__all(fabsf(nmr) <= 0x1p40f * fminf(1.0f, rstd));
    // normalise, round (the value a stored s holds), park; the rows' scores against r of both slots from the rounded
    // values. Tile rows past the last one hold copies of it: finite like it, with weight zero below.
    // A operands: rows 0..2 of the scores' (32 rows) and 0..2 of the sums' (16) are the parts of slot 0, rows 4..6 and 8..10
    // those of slot 1; the others repeat some part, and what they give is not looked at. A row of the scores' result is thus
    // in half `slot` of the wave, and so is one of the sums'.
    f32x16 sacc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sacc[e] = 0.0f;
    const int la = lane_again();
    const unsigned char* rop = rpmine + (3 * ((la >> 2) & 1) + ((la & 3) < 2 ? (la & 3) : 2)) * RPP + (la >> 5) * 16;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      __builtin_amdgcn_sched_barrier(0);   // a column block at a time: hoisted together, the LDS reads of all four spill
      u32x4 ops[2];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c0 = db * 32 + 8 * g + 4 * h;
        const f32x4 gg = *reinterpret_cast<const f32x4*>(gs + c0);
        const f32x4 bb = *reinterpret_cast<const f32x4*>(bs + c0);
        u32x2 bits;
#pragma unroll
        for (int e2 = 0; e2 < 2; ++e2) {
          const bf16x2 o = {(__bf16)fmaf(fmaf(acc[db][4 * g + 2 * e2], rstd, nmr), gg[2 * e2], bb[2 * e2]),
                            (__bf16)fmaf(fmaf(acc[db][4 * g + 2 * e2 + 1], rstd, nmr), gg[2 * e2 + 1], bb[2 * e2 + 1])};
          bits[e2] = __builtin_bit_cast(unsigned, o);
          ops[g >> 1][2 * (g & 1) + e2] = bits[e2];
        }
        *reinterpret_cast<u32x2*>(opatch + l32 * OP + c0 * 2) = bits;
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const bf16x8 ra = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(rop + (2 * db + s2) * 32));
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ra, __builtin_bit_cast(bf16x8, ops[s2]), sacc, 0, 0, 0);
      }
    }
    // softmax over the tile's rows, merged into the running sums of the half's pair; the weights' parts go to LDS as the A
    // operand of the sum (operations of a wave on LDS execute in order: no barrier needed)
    // Contraction index 8 kg + 4 s + j of the sums is row 8 kg + 2 j + s: sixteen rows that one transpose load reads, all even or
    // all odd, start eight banks apart (row pitch 68 words).
    const int lb = lane_again(), kg = lb >> 4;
    const unsigned char* wop = opatch + WPO + (3 * ((lb >> 3) & 1) + ((lb & 3) < 2 ? (lb & 3) : 2)) * 64 + kg * 16;
    const unsigned char* sop = opatch + (8 * kg + 2 * ((lb >> 2) & 3)) * OP + (lb & 3) * 8;
    float scale;   // of what has been added up so far
    {
      unsigned char* wput = opatch + WPO + 3 * 64 * (lb >> 5) + ((lb >> 3) & 3) * 16 + (4 * (lb & 1) + ((lb >> 1) & 3)) * 2;
      const float sdot = sacc[0] + (sacc[1] + sacc[2]);
      const float m_old = fresh ? -INFINITY : m;
      m = fmaxf(m_old, ffn_half_max(mine ? sdot : -INFINITY));
      scale = __expf(m_old - m);   // 0 for the pair's first tile
      const float a = mine ? __expf(sdot - m) : 0.0f;
      unsigned part[3];
      ffn_three_parts(a, part[0], part[1], part[2]);
#pragma unroll
      for (int e = 0; e < 3; ++e) *reinterpret_cast<unsigned short*>(wput + e * 64) = (unsigned short)(part[e] >> 16);
      den = fmaf(fresh ? 0.0f : den, scale, ffn_half_sum(a));
    }
    asm volatile("" ::: "memory");
    const bf16x8 wa = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(wop));
    auto row_words = [&](int b) {   // 16 components of the 32 rows
      const s16x4 e4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(ffn_lds4(sop + b * 32));
      const s16x4 o4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(ffn_lds4(sop + b * 32 + OP));
      return __builtin_bit_cast(u32x4, (s16x8)__builtin_shufflevector(e4, o4, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    const f32x4 none = {0.0f, 0.0f, 0.0f, 0.0f};
    if (!(rough && nb > 0)) {
#pragma unroll
      for (int b = 0; b < D / 16; ++b) {
        const f32x4 t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, __builtin_bit_cast(bf16x8, row_words(b)), none, 0, 0, 0);
        psum[b] = fmaf(fresh ? 0.0f : psum[b], scale, t[0] + (t[1] + t[2]));
      }
    } else {   // zero times a value of the other pair that is not finite would be NaN: each pair's rows alone
      u32x4 inA;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 8 * kg + 4 * (e & 1) + (e >> 1);        // of the word's lower half, the upper one's is row + 2
        inA[e] = (row < na ? 0xffffu : 0u) | (row + 2 < na ? 0xffff0000u : 0u);
      }
#pragma unroll
      for (int b = 0; b < D / 16; ++b) {
        const u32x4 rows = row_words(b);
        const f32x4 tA = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, __builtin_bit_cast(bf16x8, rows & inA), none, 0, 0, 0);
        const f32x4 tB = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, __builtin_bit_cast(bf16x8, rows & ~inA), none, 0, 0, 0);
        psum[b] = fmaf(fresh ? 0.0f : psum[b], scale, slotA ? tA[0] + (tA[1] + tA[2]) : tB[0] + (tB[1] + tB[2]));
      }
    }
    // the pooled maxima, a word of two components per row: eight rows at a time where a group is one pair's
    unsigned mxB = FG_NONE;
    if (MR && pool) {
      if (!rough) {
#pragma unroll
        for (int r0 = 0; r0 < FM_ROWS; r0 += 8) {
          unsigned wd[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) wd[j] = *reinterpret_cast<const unsigned*>(pcol + (r0 + j) * OP);
          if (nb == 0 || na >= r0 + 8) {
#pragma unroll
            for (int j = 0; j < 8; ++j) mx = ffn_word_max(mx, wd[j]);
          } else if (na <= r0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) mxB = ffn_word_max(mxB, wd[j]);
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              mx = ffn_word_max(mx, r0 + j < na ? wd[j] : FG_NONE);
              mxB = ffn_word_max(mxB, r0 + j < na ? FG_NONE : wd[j]);
            }
          }
        }
      } else {
        float lo[2], hi[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          lo[e] = __uint_as_float((e ? mxB : mx) << 16);
          hi[e] = __uint_as_float((e ? mxB : mx) & 0xffff0000u);
        }
#pragma unroll 1
        for (int row = 0; row < ntot; ++row) {
          const unsigned wd = *reinterpret_cast<const unsigned*>(pcol + row * OP);
          const float vl = __uint_as_float(wd << 16), vh = __uint_as_float(wd & 0xffff0000u);
          if (row < na) { lo[0] = fmaxf(lo[0], vl); hi[0] = fmaxf(hi[0], vh); }
          else { lo[1] = fmaxf(lo[1], vl); hi[1] = fmaxf(hi[1], vh); }
        }
        mx = (__float_as_uint(lo[0]) >> 16) | (__float_as_uint(hi[0]) & 0xffff0000u);
        mxB = (__float_as_uint(lo[1]) >> 16) | (__float_as_uint(hi[1]) & 0xffff0000u);
      }
    }
    // rows on their way out, as whole 256-byte rows: tile row j is row a0 + j of A or row j - na of B. Without the
    // transformed rows wanted, only the tile rows that belong to the first r of their pair leave (jr: one past the
    // last of them), four at a time.
    {
      const unsigned dBpairs = (unsigned)(cur.kB - cur.kA) * (unsigned)stride;   // pairs between A and B
      auto rows_out = [&](int b) {
        const int j = b * RPI + lane / LPR;
        const u32x4 val = *reinterpret_cast<const u32x4*>(opr + b * RPI * OP);
        const bool jb = j >= na;
        const int i = jb ? j - na : cur.a0 + j;              // segment index inside its pair
        const unsigned pj = jb ? dBpairs : 0u;               // pair, counted from A
        if (j < ntot) {
          if (out) *reinterpret_cast<u32x4*>(out + ((size_t)pA * S + (size_t)pj * S + i) * D + (lane % LPR) * 8) = val;
          if (MR && i < nr)
            *reinterpret_cast<u32x4*>(recent + ((size_t)pA * r + (size_t)pj * r + i) * D + (lane % LPR) * 8) = val;
        }
      };
      if (out) {
#pragma unroll
        for (int b = 0; b < FM_ROWS / RPI; ++b) rows_out(b);
      } else if (MR) {
        int jr = nr == 0 ? 0 : (nb > 0 ? na + nr : nr - cur.a0);
        jr = jr < ntot ? jr : ntot;
#pragma unroll 1
        for (int b = 0; b * RPI < jr; ++b) rows_out(b);
      }
    }
    if (cur.a0 + na == cur.nvA) {   // A ended, and B too where it has no more rows: p / sum of weights in place of r
      const bool endB = nb > 0 && nb == cur.nvB;
      if (slotA || endB) {
        const float inv = 1.0f / den;
        float* zo = z + (size_t)(slotA ? pA : pB) * D + (kg & 1) * (D / 2) + (lb & 15);
#pragma unroll
        for (int b = 0; b < D / 32; ++b) {
          const float p_lo = psum[b], p_hi = psum[b + D / 32];   // (values: a choice of array elements would go through memory)
          zo[16 * b] = ((kg & 1) ? p_hi : p_lo) * inv;
        }
      }
      if (MR && pool) {
        pool[(size_t)pA * (D / 2) + lane] = mx;
        if (endB) pool[(size_t)pB * (D / 2) + lane] = mxB;
      }
      mx = endB ? FG_NONE : mxB;
    }
    if (nxt.some) park_r(nxt);
    cur = nxt;
  }
}

// (the views come from the same pass: g.pool_out, g.recent_out and g.r as for the GSTA launchers)
bool ffn_gsta_fused_supports(const FfnArgs& f, const GstaArgs& g) {
  if (f.dt != LASER_BF16 || g.dt != LASER_BF16) return false;
  if (f.d != 128 || g.d != 128 || !(f.d_ff == 64 || f.d_ff == 128)) return false;
  // a tile's rows are addressed by 32-bit byte offsets from the row 0 of its first pair
  const long long P = f.cand_off ? f.P : (long long)f.U * f.C;
  if (P * f.S * f.d * 2 >= (1LL << 32)) return false;
  return g.M == 1;
}

laser_status ffn_gsta_fused_launch(const FfnArgs& f, const GstaArgs& g) {
  if (!ffn_gsta_fused_supports(f, g)) return LASER_ERR_UNSUPPORTED;
  laser_status s = gsta_r_launch(g);
  if (s != LASER_OK) return s;
  const int P = f.cand_off ? f.P : f.U * f.C;
  long long blocks = ((long long)P + FM_WAVES - 1) / FM_WAVES;
  if (blocks > 256) blocks = 256;   // one workgroup per compute unit (LDS), each wave walking several pairs
  const bool views = g.pool_out != nullptr || g.recent_out != nullptr;
  // Pairs are dealt where lengths differ and a pair fills most of a tile or more: lengths uniform, w = 10, d_ff = 128, with the
  // views and the launches around it, in turn and dealt: S = 100 64 x 256 pairs 154 and 141 us, S = 48 94 x 200 115 and 110,
  // S = 28 91.5 and 90.6; S = 20 82.1 and 82.8, S = 8 69.5 and 71.5 (two pairs share a tile however long they are); equal
  // lengths, S = 100 201 either way.
  const bool deal = f.lens != nullptr && f.S > 24 && P > FM_WAVES * blocks && P <= 64 * FG_DECKS * blocks;
#define LASER_FFN_POOL(FF, MRF, DEAL)                                                                                       \
  hipLaunchKernelGGL((ffn_pool_kernel<FF, MRF, DEAL>), dim3((unsigned)blocks), dim3(FM_THREADS), 0, f.stream,               \
                     (const unsigned short*)f.seg, f.lens, (const unsigned short*)f.w1, f.b1,                        \
                     (const unsigned short*)f.w2, f.b2, f.ln_g, f.ln_b, f.cand_off, f.U, P, f.C, f.L, f.w, f.S, f.eps, \
                     (unsigned short*)f.seg_out, g.z_out, (unsigned*)g.pool_out, (unsigned short*)g.recent_out, g.r)
#define LASER_FFN_POOL_AS(FF, MRF)                                                                                    \
  do {                                                                                                                \
    if (deal) LASER_FFN_POOL(FF, MRF, true);                                                                          \
    else LASER_FFN_POOL(FF, MRF, false);                                                                              \
  } while (0)
  if (f.d_ff == 64) { if (views) LASER_FFN_POOL_AS(64, true); else LASER_FFN_POOL_AS(64, false); }
  else { if (views) LASER_FFN_POOL_AS(128, true); else LASER_FFN_POOL_AS(128, false); }
#undef LASER_FFN_POOL_AS
#undef LASER_FFN_POOL
  s = launch_status();
  if (s != LASER_OK) return s;
  return gsta_out_launch(g);
}

}  // namespace laser
