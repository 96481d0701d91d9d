// STA for few query rows per user (at most eight) on the matrix cores, streaming the history once; and the folded form
// (Sec. 3.5.1 re-associated: raw items are keys and values, one query row per candidate and head) with the value
// projection of the finished sums in the same kernel.
//
// With w = 10 a segment is a fraction of any tile, and the vector-ALU kernel (sta_stream_short_kernel) spends its time on
// unpacking, rows past the segment's end and a cross-lane reduction per segment. Here a wave walks a run of items in tiles
// of 32 whatever the segments are: the 16 columns of v_mfma_f32_16x16x32_bf16 are (segment, query row) pairs, 16 / CP
// segments of CP = 1, 2, 4 or 8 query rows at a time (a block). The queries are repeated over the segments' columns, so
// the score product Sc = K Q^T delivers every column's score where it is wanted; the gate of a column is kept for the items
// of its segment and set to zero for all others; and the accumulator layout of Sc is, for the two halves of a tile together,
// the right operand of acc^T += V^T P^T as it sits (k-slots = items {4g..4g+3, 16+4g..16+4g+3} of lane group g, fetched in
// that order by the transpose load). A tile that crosses the end of a block is multiplied once per block. The gates are
// fp32 and stay so: they enter the product as three bf16 parts (24 bits), three MFMAs on the same V operand.
// Accumulator rows are dealt so that a lane ends with eight consecutive columns of every 32 of its (segment, query row), which leave
// as 16-byte stores, 64 bytes of a row from four lanes; in the folded form the same registers, rounded to bf16, are the operand
// of the product with W_v (in LDS in operand order, once per workgroup), and H' leaves with the sums.
// A zero gate times an item that is not finite would spread over the block's other segments. When a finished block holds a
// value that is not finite, the block is computed again, item by item over each column's own segment.
//
// What bounds it: HBM (tables of both forms at the end of the file). Every wave has a ring of its own in LDS, two tiles
// requested with global_load_lds, and no barrier; fetches alone run at 5.8 TB/s. Stores count in the same counter as
// fetches, so a wave waits for the next tile before it stores a finished block.
#include "laser_internal.h"
#include "sta_mfma_tile.h"

namespace laser {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int FEW_TI = 32;             // items per tile
constexpr int FEW_LDS = 160 * 1024;    // of a compute unit

// 16-byte chunk c of row r of a tile with CH chunks per row sits at chunk c ^ few_swz<CH>(r) of that row: 16 rows at one
// chunk (operand reads, which the hardware serves for rows 0 - 3, 12 - 15 of one lane group with rows 4 - 11 of the next) and
// four rows at four chunks in a row (transpose loads) both spread over all banks
template <int CH>
__device__ __forceinline__ int few_swz(int r) {
  const int lo = r & 3, hi = (r >> 2) & 3;
  return (((lo * CH) >> 4) << 2) | (((hi ^ (hi >> 1)) & 1) << 1) | (hi >> 1);
}

// FE = 0: keys and values as given. FE > 0: the folded form, keys = values = raw items (DQ = D), FE output columns.
// DEAL: a workgroup's waves take its units by ticket (see few_launch)
template <int DQ, int D, int FE, bool DEAL>
struct FewShape {
  static constexpr bool FOLD = FE > 0;
  static constexpr int CMAX = FOLD ? 4 : 8;                  // query rows per user
  static constexpr int QF = DQ * CMAX > 512 ? 2 : 1;         // fetches of 64 chunks: a unit's queries,
  static constexpr int KF = FOLD ? 0 : DQ / 16, VF = D / 16, F = KF + VF;         // and a tile's items
  static constexpr int KB = KF * 1024, QOFF = F * 1024, BUF = QOFF + QF * 1024;   // ring buffer: K, V, Q
  static constexpr int WVB = FOLD ? D * FE * 2 : 0;
  static constexpr int WAVE = 2 * BUF, FIT = (FEW_LDS - WVB) / WAVE;
  static constexpr int NW = FIT < 8 ? FIT : 8;               // waves per workgroup, one workgroup per compute unit
  // the tickets' counter: behind the rings, or, where these fill the LDS (folded, FE = 64: 16 KB of W_v and eight rings of 18),
  // in the place of the first word of W_v's last fragment, lane 63, which every wave then keeps in a register (with seven waves
  // instead 150 calls, most of them dealt, took 0.98 of their time in turn, so 0.965; 514 users x 2 rows, L = 776, w = 20, full
  // 28.3, 29.7 and 28.1 us)
  static constexpr bool FULL = DEAL && WVB + NW * WAVE + 16 > FEW_LDS;
  static constexpr int NT = 64 * NW, TICKET = FULL ? WVB - 16 : WVB + NW * WAVE, LDS = WVB + NW * WAVE + (DEAL && !FULL ? 16 : 0);
  static_assert(LDS <= FEW_LDS && (!FULL || FOLD), "the counter takes the place of a piece of W_v");
};

struct FewFold {
  const unsigned short* wv;    // [D, FE]
  unsigned short* y;           // [pairs, S, FE]: H'
  int hs;                      // log2 of the heads
};

template <int DQ, int D, int FE, bool DEAL>
__global__ __launch_bounds__((FewShape<DQ, D, FE, DEAL>::NT)) void sta_few_kernel(
    const unsigned short* __restrict__ q, const unsigned short* __restrict__ k, const unsigned short* __restrict__ v,
    const int32_t* __restrict__ lens, const int32_t* __restrict__ cand_off, int P, int C_all, int L, int w, int S,
    int cps, int run_segs, unsigned runs, unsigned units, MulDiv dv, float neg_scale_log2e, unsigned short* __restrict__ seg_out,
    int32_t* __restrict__ seg_cnt, FewFold fold) {
  using Sh = FewShape<DQ, D, FE, DEAL>;
  constexpr bool FOLD = Sh::FOLD;
  constexpr int KCH = DQ / 8, VCH = D / 8, KS = DQ / 32, VT = D / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hs = FOLD ? fold.hs : 0;

  if constexpr (FOLD) {   // W_v in operand order: fragment (et, ks), lane (m, g), eight k = 32 ks + 8 g + j of column
    for (int e = tid; e < D * FE / 8; e += Sh::NT) {   // FE/4 (m / 4) + 4 et + m % 4
      const int kk = e / (FE / 8), n0 = (e % (FE / 8)) * 8;
      const u32x4 raw = *reinterpret_cast<const u32x4*>(fold.wv + (size_t)kk * FE + n0);
      const int fg = (kk >> 3) & 3, fks = kk >> 5, fj = kk & 7;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int col = n0 + j, m = (col / (FE / 4)) * 4 + (col & 3), et = (col % (FE / 4)) >> 2;
        *reinterpret_cast<unsigned short*>(smem + ((et * (D / 32) + fks) * 64 + fg * 16 + m) * 16 + fj * 2) =
            (unsigned short)((raw[j >> 1] >> ((j & 1) * 16)) & 0xffffu);
      }
    }
  }
  unsigned under_ticket = 0;   // the word of W_v that the counter takes the place of
  if constexpr (Sh::FULL) {
    __syncthreads();
    under_ticket = *reinterpret_cast<const unsigned*>(smem + Sh::TICKET);
    __syncthreads();
  }
  if (DEAL && tid == 0) *reinterpret_cast<unsigned*>(smem + Sh::TICKET) = Sh::NW;
  if (FOLD || DEAL) __syncthreads();
  const unsigned ring = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem + Sh::WVB +
                        (unsigned)wave * Sh::WAVE;
  // the folded form's sums are not read back here: with the hint they leave the cache to H'
  auto put_sums = [&](unsigned short* at, const u32x4& x) {
    if constexpr (FOLD) __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(at));
    else *reinterpret_cast<u32x4*>(at) = x;
  };
  const unsigned char* ringp = smem + Sh::WVB + wave * Sh::WAVE;

  const int CP = 1 << cps, spb = 16 >> cps;   // query rows and segments of a block
  const int col_s = l16 >> cps, col_p = l16 & (CP - 1);

  // LDS offsets that do not change. Operand read of K: row l16, chunk 4 ks + g. Transpose load of V: rows 4 g + l16 / 4
  // (and 16 further down), columns 32 (vt / 2) + 8 (l16 % 4) + 4 (vt % 2) ..
  const int krow = l16 * DQ * 2;
  const int vr = 4 * g + (l16 >> 2);
  auto koff = [&](int ks) { return krow + (((4 * ks + g) ^ few_swz<KCH>(l16)) << 4); };
  auto voff = [&](int vt) {
    const int col = 32 * (vt >> 1) + 8 * (l16 & 3) + 4 * (vt & 1);
    return vr * D * 2 + (((col >> 3) ^ few_swz<VCH>(vr)) << 4) + (col & 4) * 2;
  };

  // A unit of work is one run of a user's segments; a workgroup takes every (number of workgroups)-th one and its waves share
  // them, in turn or by ticket, so that the waves in flight sweep the arrays front to back, with the runs of a user rotated so
  // that no wave meets one run only. The fetches are two tiles ahead of the arithmetic across units, and every unit counts at
  // least two tiles, so that this reaches into the next unit and no further.
  struct Unit {
    int C, i_beg, i_ne, t_beg, t_end, ntile;
    size_t pb;
    const unsigned short *k, *v;
  };
  // (read with the arguments: read where it is first wanted, it is another trip to memory ahead of the first unit, 0.2 us of
  // every call)
  const unsigned blocks = gridDim.x;
  auto len_of = [&](unsigned it) { return it < units && lens != nullptr ? lens[dv.div(it)] : L; };
  // unit `it` of a user of (unclamped) length n: its counts, its empty segments; false: nothing to compute
  auto open_unit = [&](unsigned it, int n, Unit& x) {
    const int u = (int)dv.div(it);
    const unsigned rot = it + (((unsigned)u * 0x9E3779B1u) >> 16);
    const unsigned run = rot - dv.div(rot) * runs;
    n = n < 0 ? 0 : (n > L ? L : n);
    if (run == 0) write_seg_cnt(seg_cnt, u, n, L, w, S, lane, 64);
    const CandRange cr = cand_range(cand_off, u, C_all, P);
    x.C = __builtin_amdgcn_readfirstlane(cr.count);
    x.pb = (size_t)__builtin_amdgcn_readfirstlane(cr.first);
    x.i_beg = (int)run * run_segs;
    const int i_end = S - x.i_beg > run_segs ? x.i_beg + run_segs : S;
    const int ne = (n + w - 1) / w;   // non-empty segments are a prefix
    x.i_ne = ne < x.i_beg ? x.i_beg : (ne > i_end ? i_end : ne);
    if (x.i_ne < i_end) {   // empty segments: exact zeros
      const u32x4 z = {0u, 0u, 0u, 0u};
      const int len16 = (i_end - x.i_ne) * VCH;
      for (int c = 0; c < x.C; ++c)
        for (int e = lane; e < len16; e += 64)
          put_sums(seg_out + ((x.pb + c) * S + x.i_ne) * D + e * 8, z);
      if constexpr (FOLD) {
        const int ylen = (i_end - x.i_ne) * (FE / 8), pairs = x.C >> hs;
        for (int c = 0; c < pairs; ++c)
          for (int e = lane; e < ylen; e += 64)
            *reinterpret_cast<u32x4*>(fold.y + (((x.pb >> hs) + c) * S + x.i_ne) * FE + e * 8) = z;
      }
    }
    x.t_beg = x.i_beg * w;
    x.t_end = x.i_ne * w < n ? x.i_ne * w : n;
    const int nt = (x.t_end - x.t_beg + FEW_TI - 1) / FEW_TI;
    x.ntile = nt < 2 ? 2 : nt;
    x.k = k + (size_t)u * L * DQ;
    x.v = v + (size_t)u * L * D;
    return x.i_ne > x.i_beg && x.C > 0;
  };
  // row and byte offset of a lane's chunk of fetch f
  auto krow_of = [&](int f) { return f * (64 / KCH) + lane / KCH; };
  auto vrow_of = [&](int f) { return f * (64 / VCH) + lane / VCH; };
  unsigned kfo[FOLD ? 1 : Sh::KF], vfo[Sh::VF];
#pragma unroll
  for (int f = 0; f < Sh::KF; ++f) kfo[f] = (krow_of(f) * DQ + ((lane % KCH) ^ few_swz<KCH>(krow_of(f))) * 8) * 2;
#pragma unroll
  for (int f = 0; f < Sh::VF; ++f) vfo[f] = (vrow_of(f) * D + ((lane % VCH) ^ few_swz<VCH>(vrow_of(f))) * 8) * 2;
  // 16 bytes per lane to LDS dst + 16 * lane; items of a large history with the non-temporal hint
  auto dma = [&](unsigned dst, unsigned off, const void* src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n" ::"s"(dst), "v"(off), "s"(src) : "memory");
  };
  auto dma_nt = [&](unsigned dst, unsigned off, const void* src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt\n" ::"s"(dst), "v"(off), "s"(src) : "memory");
  };
  const bool nt = __builtin_amdgcn_readfirstlane(past_cache(lens, (int)(units / runs), L, FOLD || k == v ? D * 2 : (DQ + D) * 2, lane));
  // requests tile t of a unit into ring buffer b (with the unit's queries when it is the first) and returns how many
  // fetches that were. Rows past the end repeat the last valid one (their gates are zero).
  auto fetch = [&](const Unit& x, int t, int b) {
    int t0 = x.t_beg + t * FEW_TI;
    t0 = t0 < x.t_end ? t0 : x.t_end - 1;
    const int last = x.t_end - 1 - t0;
    const unsigned base = ring + (unsigned)b * Sh::BUF;
    if (t == 0) {
#pragma unroll
      for (int f = 0; f < Sh::QF; ++f) {
        const int e = f * 64 + lane, r = e / KCH, rr = r < x.C ? r : x.C - 1;
        dma(base + Sh::QOFF + f * 1024, (unsigned)(rr * DQ + (e % KCH) * 8) * 2, q + x.pb * DQ);
      }
    }
    const unsigned short* kt = x.k + (size_t)t0 * DQ;
    const unsigned short* vt = x.v + (size_t)t0 * D;
    if (last >= FEW_TI - 1 && nt) {
#pragma unroll
      for (int f = 0; f < Sh::KF; ++f) dma_nt(base + f * 1024, kfo[f], kt);
#pragma unroll
      for (int f = 0; f < Sh::VF; ++f) dma_nt(base + Sh::KB + f * 1024, vfo[f], vt);
    } else if (last >= FEW_TI - 1) {
#pragma unroll
      for (int f = 0; f < Sh::KF; ++f) dma(base + f * 1024, kfo[f], kt);
#pragma unroll
      for (int f = 0; f < Sh::VF; ++f) dma(base + Sh::KB + f * 1024, vfo[f], vt);
    } else {
#pragma unroll
      for (int f = 0; f < Sh::KF; ++f) {
        const int r = krow_of(f);
        dma(base + f * 1024, kfo[f] - (unsigned)((r > last ? r - last : 0) * DQ * 2), kt);
      }
#pragma unroll
      for (int f = 0; f < Sh::VF; ++f) {
        const int r = vrow_of(f);
        dma(base + Sh::KB + f * 1024, vfo[f] - (unsigned)((r > last ? r - last : 0) * D * 2), vt);
      }
    }
    return t == 0 ? Sh::F + Sh::QF : Sh::F;
  };
  // Waits until at most the youngest group of fetches is outstanding. Loads retire in order among themselves, so every
  // older one has landed; stores in flight can only make the wait longer.
  auto wait_older = [&](int young) {
    if (young == Sh::F) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(Sh::F) : "memory");
    else if (young != 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(Sh::F + Sh::QF) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };

  unsigned it = (unsigned)wave * blocks + blockIdx.x;
  int n_ahead = len_of(it);
  auto next_unit = [&](Unit& x) {   // the next unit with something to compute (its successor's length is loaded ahead)
    while (it < units) {
      const unsigned now = it;
      const int n = __builtin_amdgcn_readfirstlane(n_ahead);
      if constexpr (DEAL) {
        unsigned ticket = 0;
        if (lane == 0) ticket = atomicAdd(reinterpret_cast<unsigned*>(smem + Sh::TICKET), 1u);
        it = __builtin_amdgcn_readfirstlane(ticket) * blocks + blockIdx.x;
      } else {
        it += blocks * Sh::NW;
      }
      n_ahead = len_of(it);
      if (open_unit(now, n, x)) return true;
    }
    return false;
  };
  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  const bf16x8 zero8 = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  Unit cur, nxt;
  bool have = next_unit(cur);
  int young = 0, buf = 0;      // fetches of the youngest group; ring buffer of the tile in work
  bool landed = false;         // the tile about to be worked on has been waited for
  if (have) {
    fetch(cur, 0, 0);
    young = fetch(cur, 1, 1);
  }
  while (have) {
    const bool more = next_unit(nxt);
    const bool live = col_p < cur.C;   // this lane's query row exists
    f32x4 acc[VT];   // rows: column 32 (vt / 2) + 8 g + 4 (vt % 2) + i of the sums; columns: (segment, query row)
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) acc[vt] = zero4;
    int blk = cur.i_beg;   // first segment of the block in work
    bf16x8 qf[KS];         // right operand of the scores: column l16 holds query row col_p

    auto finish = [&]() {
      const int seg = blk + col_s;
      const bool mine = live && seg < cur.i_ne;
      bf16x8 o[VT / 2];
      auto round_acc = [&]() {
#pragma unroll
        for (int x = 0; x < VT / 2; ++x)
#pragma unroll
          for (int i = 0; i < 8; ++i) o[x][i] = (__bf16)acc[2 * x + (i >> 2)][i & 3];
      };
      round_acc();
      f32x4 bad = zero4;   // zero times the column's values: zero, or NaN unless all are finite
#pragma unroll
      for (int x = 0; x < VT / 2; ++x) bad = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zero8, o[x], bad, 0, 0, 0);
      if (__builtin_expect(__any(mine && !(bad[0] == 0.0f)), 0)) {   // once more, each column over its own segment only
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) acc[vt] = zero4;
        if (mine) {
          const int hi = (seg + 1) * w < cur.t_end ? (seg + 1) * w : cur.t_end;
          for (int j = seg * w; j < hi; ++j) {
            float s = 0.0f;
            for (int x = 0; x < DQ; ++x)
              s = fmaf(bf16_bits_to_f32(cur.k[(size_t)j * DQ + x]), bf16_bits_to_f32(q[(cur.pb + col_p) * DQ + x]), s);
            const float gt = gate(s, neg_scale_log2e);
#pragma unroll
            for (int vt = 0; vt < VT; ++vt)
#pragma unroll
              for (int i = 0; i < 4; ++i)
                acc[vt][i] = fmaf(gt, bf16_bits_to_f32(cur.v[(size_t)j * D + 32 * (vt >> 1) + 8 * g + 4 * (vt & 1) + i]), acc[vt][i]);
          }
        }
        round_acc();
      }
      constexpr int ET = FOLD ? FE / 16 : 2, LE = FE / 4;
      bf16x8 y[ET / 2];
      if constexpr (FOLD) {   // H' = sums . W_v
#pragma unroll
        for (int et = 0; et < ET; ++et) {
          f32x4 r = zero4;
#pragma unroll
          for (int ks = 0; ks < D / 32; ++ks) {
            u32x4 raw = *reinterpret_cast<const u32x4*>(smem + ((et * (D / 32) + ks) * 64 + lane) * 16);
            if (Sh::FULL && et == ET - 1 && ks == D / 32 - 1) raw[0] = lane == 63 ? under_ticket : raw[0];
            const bf16x8 a = __builtin_bit_cast(bf16x8, raw);
            r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, o[ks], r, 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) y[et / 2][4 * (et & 1) + i] = (__bf16)r[i];
        }
      }
      if (!landed) {   // the next tile is awaited ahead of the stores, which then have a whole step to retire
        wait_older(young);
        landed = true;
      }
      if (mine) {
        unsigned short* dst = seg_out + ((cur.pb + col_p) * S + seg) * D + 8 * g;
#pragma unroll
        for (int x = 0; x < VT / 2; ++x) put_sums(dst + 32 * x, __builtin_bit_cast(u32x4, o[x]));
        if constexpr (FOLD) {   // each head's columns (runs of 32 and more) from its own sums, chosen ahead of the stores
          if ((LE * g) / (FE >> hs) == (col_p & ((1 << hs) - 1))) {
            unsigned short* ydst = fold.y + (((cur.pb + col_p) >> hs) * S + seg) * FE + LE * g;
#pragma unroll
            for (int x = 0; x < ET / 2; ++x) *reinterpret_cast<bf16x8*>(ydst + 8 * x) = y[x];
          }
        }
      }
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) acc[vt] = zero4;
    };

    for (int t = 0; t < cur.ntile; ++t) {
      if (!landed) wait_older(young);
      landed = false;
      const unsigned char* base = ringp + buf * Sh::BUF;
      const unsigned char* Vs = base + Sh::KB;
      const unsigned char* Ks = FOLD ? Vs : base;
      if (t == 0) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          qf[ks] = *reinterpret_cast<const bf16x8*>(base + Sh::QOFF + (live ? col_p : 0) * DQ * 2 + ks * 64 + g * 16);
      }
      bf16x8 kf[2][KS], vf[VT];
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          kf[half][ks] = *reinterpret_cast<const bf16x8*>(Ks + half * 16 * DQ * 2 + koff(ks));
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        const unsigned char* src = Vs + voff(vt);
        const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src));
        const s16x4 hi4 =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src + 16 * D * 2));
        vf[vt] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the tile is in registers: its buffer is free
      if (t + 2 < cur.ntile) young = fetch(cur, t + 2, buf);
      else if (more) young = fetch(nxt, t + 2 - cur.ntile, buf);
      else young = 0;
      buf ^= 1;

      float gt[8];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        f32x4 sc = zero4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[half][ks], qf[ks], sc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) gt[4 * half + i] = gate(sc[i], neg_scale_log2e);
      }
      const int j0 = cur.t_beg + t * FEW_TI;
      const int j1 = j0 + FEW_TI < cur.t_end ? j0 + FEW_TI : cur.t_end;
      while (blk < cur.i_ne) {
        const int lo = (blk + col_s) * w;             // the column's segment
        const int hi = lo + w < cur.t_end ? lo + w : cur.t_end;
        const unsigned span = hi > lo ? (unsigned)(hi - lo) : 0u;
        bf16x8 p[3];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int j = j0 + 4 * g + (e >> 2) * 16 + (e & 3);
          const float x = (unsigned)(j - lo) < span ? gt[e] : 0.0f;
          const __bf16 h0 = (__bf16)x;
          const float r1 = x - (float)h0;
          const __bf16 h1 = (__bf16)r1;
          p[0][e] = h0;
          p[1][e] = h1;
          p[2][e] = (__bf16)(r1 - (float)h1);
        }
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
          for (int vt = 0; vt < VT; ++vt)
            acc[vt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[vt], p[part], acc[vt], 0, 0, 0);
        const int blk_end = (blk + spb) * w;
        if (blk_end > j1 && j1 < cur.t_end) break;    // the block goes on in the next tile
        finish();
        blk += spb;
        if (blk_end >= j1) break;                     // (the next block starts with the next tile, or nothing is left)
      }
    }
    cur = nxt;
    have = more;
  }
}

// ------------------------------------------------------------------------------------------ host side
template <int DQ, int D, int FE>
static laser_status few_launch(const StaArgs& a, const FewFold& fold) {
  using Sh = FewShape<DQ, D, FE, false>;
  int cps = 0;
  while ((1 << cps) < a.C) ++cps;
  const int w = a.w < a.L ? a.w : a.L;     // (one segment either way; keeps index arithmetic in range)
  // Runs of about 64 items (several for every wave; the waves in flight then sweep a narrower window, see the kernel),
  // fewer where that leaves waves without work
  const long long waves = 256 * Sh::NW;
  long long run = tuning_int("LASER_FEW_RUN", 64) / w;
  const long long share = (long long)a.U * a.S / waves;
  if (run > share) run = share;
  if (run < 1) run = 1;
  const unsigned runs = (unsigned)((a.S + run - 1) / run);
  const unsigned units = (unsigned)a.U * runs;   // <= U S, which fits an int
  const unsigned blocks = units < 256 ? units : 256u;
  const MulDiv dv = mul_div(runs);
  // Units of short histories hold little or nothing. Dealt out in turn, the fullest wave has half as much again as the mean, by
  // ticket (an LDS counter) a workgroup's waves end together; with few units a wave the counter costs more than it evens out, and
  // with full lengths there is less to even out. 400 calls of 3 to 8 rows, mean (and worst) time by ticket over that in turn: 3 to 4
  // units a wave 0.99 (1.09), 4 to 6 0.95 (1.05), with full lengths 0.99 (1.04), 6 to 10 0.92 (1.00), full 0.98 (1.03), more 0.93
  // (1.01), full 0.97 (1.01). d_in = 128, two rows, w = 10, 2048 users, uniform lengths 93 -> 84 us, full 118 -> 112.
  const bool deal = units > (unsigned)tuning_int("LASER_FEW_DEAL", a.lens != nullptr ? 4 : 6) * blocks * Sh::NW;
  auto launch = [&](auto shape, auto kern) {
    using X = decltype(shape);
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, X::LDS) != hipSuccess)
      return LASER_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(X::NT), X::LDS, a.stream, (const unsigned short*)a.q,
                       (const unsigned short*)a.k, (const unsigned short*)a.v, a.lens, a.cand_off, a.P, a.C, a.L, w, a.S, cps,
                       (int)run, runs, units, dv, -1.4426950408889634f / a.gamma, (unsigned short*)a.seg_out, a.seg_cnt, fold);
    return launch_status();
  };
  return deal ? launch(FewShape<DQ, D, FE, true>{}, sta_few_kernel<DQ, D, FE, true>)
              : launch(FewShape<DQ, D, FE, false>{}, sta_few_kernel<DQ, D, FE, false>);
}

// From three query rows per user on the vector-ALU kernels are bound by their arithmetic and this one by HBM; with one or two
// rows both are near HBM, and in launches that the cache holds the vector-ALU kernels, with four times the waves in flight, are
// the better ones, except for two rows of 64-wide keys and values (past the cache: few_preferred_large). Lengths uniform in
// [L / 5, L], us there and here:
//   U, C, L, w             d_q = 32, d = 128    64, 64          128, 128        64, 128
//   1500, 3, 1000, 25        96 -> 56          119 -> 44        200 -> 86       119 -> 64
//   1500, 4, 1000, 10       124 -> 96          146 -> 54        176 -> 128      131 -> 95
//   256, 4, 1000, 50         18 -> 16           20 -> 11         30 -> 21        20 -> 17
//   1000, 8, 2048, 256      250 -> 81          143 -> 67        230 -> 121      336 -> 96
//   256, 8, 8000, 512       267 -> 82          153 -> 64        277 -> 125      383 -> 94
// The table's calls fill the machine. In one that does not, the time is the chain of tiles of one run (two at least, and a
// segment is one run however long it is), and up to six rows the vector-ALU kernels, whose four waves share a long segment
// and which start faster, are the better ones: 1 user x 2, L = 2000, w = 512, 64 / 64 6.6 us there, 14.7 here; 16 x 3,
// L = 2048, w = 256, 32 / 64 6.0 and 8.5; 64 x 3, L = 200, w = 5, 128 / 128 6.0 and 7.0; 4 x 2, L = 2000, w = 2, 64 / 64 5.1 and
// 7.4. The lines lie where the times of 3000 such calls (1 to 1500 users, 2 to 8 rows, every width, w = 1 to 1000) cross: 35
// of those left here are more than 5 % slower than there, by 16 % at most.
static bool few_fills(const StaArgs& a) {
  const long long items = (long long)a.U * a.L, segs = (long long)a.U * a.S;
  const bool narrow = a.d == 64;
  if (a.C >= 7 || (a.w > 32 && a.w <= 100)) return true;
  if (a.w > 100) return a.C >= (a.w <= 128 ? 4 : 6) || segs >= (a.C == 2 ? 1024 : 512);
  if (a.w <= 4 && narrow) return items >= (a.C <= 4 ? 65536 >> a.C : 0);
  if (a.w <= 4) return items >= (a.C <= 4 ? 32768 : 524288 >> a.C);
  if (a.C == 2) return items >= (a.w <= 10 ? 65536 : 131072);
  if (narrow || a.C == 6) return true;
  if (a.C == 3) return items >= 65536;
  return a.w > 10 || items >= (a.C == 4 ? 32768 : 8192);
}

// One or two rows in a launch past the cache, whose units are dealt by ticket, against the vector-ALU kernels. With lengths given
// the histories may hold a fraction of their arrays, which the cache then keeps, and a launch needs more to be the better one
// here; segments longer than a tile that fill less than three quarters of their tiles (33 to 47 items, 65 to 71) are multiplied
// with too much of nothing; with 400 items and more a wave is left with too few units. 1950 calls of 60 to 8000 users and items,
// lengths full, uniform from nothing or a fifth on, or spread over the logarithm, mean (and worst) time here over that there:
//   one row, 64 / 64: w 10 .. 127 full from 256 MB 0.83 (1.04), with lengths from 400 MB 0.77 (1.15), below 0.88 (1.19)
//     128 / 128: w 16 .. 32 full from 256 MB 0.92 (1.01), with lengths from 1 GB 0.89 (1.06), from 600 MB 0.89 (1.30); w 48 .. 63
//       full 0.88 (1.01), with lengths from 600 MB 0.80 (1.12), below 0.93 (1.46)
//     64 / 128: w 24 .. 32 and 48 .. 64 full from 300 MB 0.93 (1.04); with lengths w 48 .. 64 from 1 GB 0.87 (1.05), below 0.97
//       (1.56), w 24 .. 32 0.97 (1.40)
//     32 / 128, w 24 .. 50 full 0.95 (1.10), with lengths 0.98 (1.57), stays there, as do 128 / 64 and 32 / 64 (1500, 1000, 40,
//       32 / 64, lengths over the logarithm 18 us and 25)
//   two rows, 32 / 64: w 8 .. 32 from 150 MB 0.66 (0.94); w 48 .. 399 full from 300 MB 0.88 (0.95), with lengths from 600 MB 0.79
//       (0.98), below 0.96 (1.29)
//     128 / 64: w 8 .. 200 from 150 MB 0.78 (1.08); w 201 .. 399 full from 300 MB 0.91 (0.94), with lengths from 600 MB 0.79 (0.88),
//       below 0.91 (1.48)
//     d = 128: w 8 (d_q = 32: 16) .. 399 full from 300 MB 0.91 (1.12), with lengths from 600 MB 0.81 (1.19), below 0.93 (1.45)
//     w 400 and more, every width 1.02 (2.01)
static bool few_preferred_large(const StaArgs& a) {
  if (a.k == a.v) return false;   // (read once by the vector-ALU kernels)
  if (a.w > 32 && 4 * a.w < 3 * ((a.w + 31) / 32 * 32)) return false;   // 33 to 47, 65 to 71
  // (a packed call's users without a row are not read; at least P / C have one: 500 calls of none to C rows a user, counted like dense
  // ones, had 17 more than 2 % slower, by 24 % at most)
  const long long mb = (long long)(a.cand_off != nullptr ? a.P / a.C : a.U) * a.L * (a.d_q + a.d) * 2 / 1000000;
  const bool full = a.lens == nullptr;
  if (a.C == 2) {
    if (a.w < (a.d_q == 32 && a.d == 128 ? 16 : 8) || a.w >= 400) return false;
    if (a.d == 64 && a.w <= (a.d_q == 128 ? 200 : 32)) return mb >= 150;
    return mb >= (full ? 300 : 600);
  }
  if (a.C != 1) return false;
  switch (a.d_q * 1000 + a.d) {
    case 64064: return a.w >= 10 && a.w < 128 && mb >= (full ? 256 : 400);
    case 128128: return a.w >= 16 && a.w < 64 && mb >= (full ? 256 : (a.w <= 32 ? 1000 : 600));
    case 64128: return a.w <= 64 && (full ? a.w >= 24 && mb >= 300 : a.w >= 48 && mb >= 1000);
    default: return false;
  }
}

bool sta_few_supports(const StaArgs& a) {
  if (a.dt != LASER_BF16 || a.C > 8 || a.heads != 1 || a.softmax) return false;
  if (!(a.d_q == 32 || a.d_q == 64 || a.d_q == 128) || !(a.d == 64 || a.d == 128)) return false;
  return (a.C > 2 || (a.C == 2 && a.d_q == 64 && a.d == 64) || few_preferred_large(a)) && few_fills(a);
}

laser_status sta_few_launch(const StaArgs& a) {
  if (!sta_few_supports(a)) return LASER_ERR_UNSUPPORTED;
  const FewFold none{nullptr, nullptr, 0};
  switch (a.d_q * 1000 + a.d) {
    case 32064: return few_launch<32, 64, 0>(a, none);
    case 32128: return few_launch<32, 128, 0>(a, none);
    case 64064: return few_launch<64, 64, 0>(a, none);
    case 64128: return few_launch<64, 128, 0>(a, none);
    case 128064: return few_launch<128, 64, 0>(a, none);
    default: return few_launch<128, 128, 0>(a, none);
  }
}

// The folded form: a is STA over the raw items (C query rows per user, heads of each candidate next to each other), p the
// projection of its sums
// 2048 users x 1 candidate x 2 heads, L = 1000, w = 10, lengths uniform in [200, 1000]: 83 us repeated on one batch (106 with a
// fixed share of units for every wave, the sums through the cache and in 16-byte pieces); the vector-ALU kernel over the raw
// items and the projection of its stored sums took 101 + 33 us. More than four query rows do not fit the ring. With one or two
// rows, long segments and few of them the separate launches are the better ones, as above (whole chain, L = 1000, w = 1000: 16
// users x 1 row 21 us, 35 here; 64 x 2 rows 32 and 36; 64 x 1, L = 4000, w = 500 the same time).
bool sta_few_folded_supports(const StaArgs& a, const ProjHeadsArgs& p) {
  if (a.dt != LASER_BF16 || a.C > 4 || a.k != a.v || a.d_q != 128 || a.d != 128) return false;
  if (a.C <= 2 && a.w > 128 * a.C && (long long)a.U * a.S < 512) return false;
  return (p.d == 64 || p.d == 128) && p.d % p.heads == 0 && (p.d / p.heads) % 32 == 0;
}

laser_status sta_few_folded_launch(const StaArgs& a, const ProjHeadsArgs& p) {
  if (!sta_few_folded_supports(a, p)) return LASER_ERR_UNSUPPORTED;
  const FewFold fold{(const unsigned short*)p.wv, (unsigned short*)p.y, p.heads == 4 ? 2 : p.heads - 1};
  return p.d == 64 ? few_launch<128, 128, 64>(a, fold) : few_launch<128, 128, 128>(a, fold);
}

}  // namespace laser
