// STA with sigmoid gates on the bf16 matrix cores, 32 or 64 candidates per workgroup: one wave fetches, the others compute.
//
// Products, operand layouts and rounding are those of sta_mfma.hip (32 candidates per wave, both products transposed, the gates
// never leave the registers), and so are the bits of H'. What differs is how the history reaches the waves. Staged through
// registers 64 rows at a time, whatever the segment holds, every tile costs two barriers with the trip to memory between them (and
// the rows past a segment of ten items five loads out of six). Here a workgroup has one more wave, the loader, which requests chunks of up to 32 rows straight into a ring in
// LDS (global_load_lds) as soon as a slot is free, waits for them and meets the others at one barrier per chunk. Loads and
// stores of a wave share one counter, so a wave that stores rows can wait for its loads only together with its stores; the
// loader stores nothing while it fetches, and the computing waves wait for no memory at all. A chunk is as many whole segments
// as fit 32 rows, or up to 32 rows of one segment, so a segment of ten items costs the fetch and the products of ten to sixteen,
// not of 64.
//
// Rows of a block past the segment's end (rows of the next segment, copies of the last row, or what the slot held before) have
// their gates cleared, and their lanes fetch the value row from a row of zeros: whatever those rows hold, 0 * 0 enters the sum.
//
// Bound by the stores of H' where segments are short, by the issue of the gates (72 vector instructions a block) and the chain of a
// block (reads, scores, gates, sums: 0.6 us) where they are long; several workgroups on a compute unit fill each other's gaps. Against
// staging through registers, us: 64 users x 256 candidates, 100 segments of 10 items, two heads of 16 / 64, lengths uniform 99.7 -> 81
// (450 MB: 5.6 TB/s); 64 x 64, 16 of 128, 64 / 64 11.3 -> 8.5; 1 x 100, 100 of 10, 32 / 128 4.8 -> 3.5; 505 x 16, 190 of 2, 64 / 64
// 171 -> 60; 32 x 256, 32 of 128, 64 / 64 (there eight waves and a second tile) 20.8 -> 18.4. 700 drawn calls (1 to 256 users, 9 to 512
// candidates, w = 1 to 700, every width, up to four heads, full to log-uniform lengths, equal and own counts), direct-to-LDS ones of both
// sides among them: 0.72 on average, six more than 3 % above, the worst 6 x 211, 48 segments of 64 items, 64 / 128, four heads 11.3 -> 12.9.
#include <type_traits>

#include "laser_internal.h"
#include "sta_mfma_tile.h"

namespace laser {

constexpr int NB = 2;   // slots of the ring: with three or four, fewer workgroups fit a compute unit, and every call tried was slower

// Waves that the registers of a form (as the compiler counts them) let a SIMD hold. The launch bounds ask for less: asked for these, forms
// of one computing wave took accumulation registers beside and held fewer.
template <int DQ, int D, int HEADS, bool SHORT, int NW>
constexpr int ring_simd_waves() {
  if (D == 64) return DQ == 128 ? 3 : (HEADS == 1 && (DQ == 32 || SHORT) ? 5 : 4);
  if (DQ == 128) return SHORT && HEADS < 4 && NW == 2 ? 3 : 2;
  return DQ == 64 && HEADS == 4 && !SHORT && NW < 3 ? 2 : 3;
}

template <int DQ, int D, int NW, int HEADS, bool SHORT>
struct RingShape {
  static constexpr int KROW = DQ * 2, VROW = D * 2, KB = 32 * KROW, CB = KB + 32 * VROW;   // bytes of a row, a chunk's keys, a chunk
  static constexpr int ZERO = NB * CB, PATCH = ZERO + 256, OP = OPitch<D>::v;
  static constexpr int LDS = PATCH + NW * CW * OP;
  static constexpr int NT = 64 * (NW + 1);
  static constexpr int BY_LDS = 160 * 1024 / LDS, BY_WAVES = 4 * ring_simd_waves<DQ, D, HEADS, SHORT, NW>() / (NW + 1);
  static constexpr int BOUND = DQ == 128 || BY_LDS * (NW + 1) < 12 ? 2 : 3;   // waves of a SIMD, at least: what the LDS allows for
  static constexpr int PER_CU = BY_WAVES < BY_LDS ? BY_WAVES : BY_LDS;   // workgroups of a compute unit
};

// 16-byte chunk c of key row r sits at c ^ ring_kswz(r) of that row, of value row r at c ^ 4 ring_vswz(r): 16 rows at one chunk
// (operand reads) and four rows at four chunks (transpose loads) spread over all banks
template <int CH> __device__ __forceinline__ int ring_kswz(int r) { return ((r * CH) >> 4) & (CH - 1); }
template <int CH> __device__ __forceinline__ int ring_vswz(int r) { return ((r * CH) >> 4) & (CH / 4 - 1); }

template <int DQ, int D, int NW, int HEADS, bool SHORT>
__global__ __launch_bounds__(64 * (NW + 1), (RingShape<DQ, D, NW, HEADS, SHORT>::BOUND)) void sta_ring_kernel(
    const unsigned short* __restrict__ q, const unsigned short* __restrict__ k, const unsigned short* __restrict__ v,
    const int32_t* __restrict__ lens, const int32_t* __restrict__ cand_off, int P, int C_all, int L, int w, int S, int spw,
    int chunk_segs, MulDiv by_runs, int sruns, MulDiv by_tiles, int ctiles, int xcd_ranges, float neg_scale_log2e,
    unsigned short* __restrict__ seg_out, int32_t* __restrict__ seg_cnt) {
  using Sh = RingShape<DQ, D, NW, HEADS, SHORT>;
  constexpr int KROW = Sh::KROW, VROW = Sh::VROW, KCH = DQ / 8, VCH = D / 8;
  constexpr int KSTEPS = DQ / 16, DB = D / 32, KH = KSTEPS / HEADS, DBH = DB / HEADS;
  static_assert(KSTEPS % HEADS == 0 && DB % HEADS == 0, "heads must own whole k-steps and whole column blocks");
  static_assert((31 + 31 + 1) * KROW <= Sh::CB + 256 + NW * CW * Sh::OP, "key reads past a chunk stay inside the LDS");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[Sh::LDS];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem);

  // Workgroups are dealt to the eight XCDs round-robin by index; renumbered so that each XCD has a contiguous range, the candidate
  // tiles of a user's run meet its items in one L2 (RING_FEW_USERS has the exception)
  int bid = blockIdx.x;
  if (xcd_ranges) {
    const int x = blockIdx.x & 7, more = gridDim.x & 7;
    bid = x * (int)(gridDim.x >> 3) + (x < more ? x : more) + (int)(blockIdx.x >> 3);
  }
  const int ut = (int)by_runs.div(bid), srun = bid - ut * sruns;
  const int u = (int)by_tiles.div(ut), ct = ut - u * ctiles;
  const int seg_lo = srun * spw, seg_hi = seg_lo + spw < S ? seg_lo + spw : S;
  const int t_lo = seg_lo * w;

  // a chunk: rows t0 .. of segment `seg` (SHORT: of chunk_segs segments from there), at most 32, up to `hi`
  struct Cur { int seg, t0, hi; };
  const bool loader = wave == NW;
  const unsigned char* kU = reinterpret_cast<const unsigned char*>(k + (size_t)u * L * DQ);
  const unsigned char* vU = reinterpret_cast<const unsigned char*>(v + (size_t)u * L * D);
  // requests rows t0 .. t0 + rows - 1 into a slot, 1 KB of keys or values a time (rows past the last repeat it); how many requests
  constexpr int KPR = 1024 / KROW, VPR = 1024 / VROW;
  auto requests = [&](int rows) { return (rows + KPR - 1) / KPR + (rows + VPR - 1) / VPR; };
  unsigned kofs[32 / KPR], vofs[32 / VPR];   // this lane's 16 bytes of each: row and swizzled chunk
#pragma unroll
  for (int g = 0; g < 32 / KPR; ++g) {
    const int r = g * KPR + lane / KCH;
    kofs[g] = r * KROW + (((lane % KCH) ^ ring_kswz<KCH>(r)) << 4);
  }
#pragma unroll
  for (int g = 0; g < 32 / VPR; ++g) {
    const int r = g * VPR + lane / VCH;
    vofs[g] = r * VROW + (((lane % VCH) ^ (4 * ring_vswz<VCH>(r))) << 4);
  }
  auto fetch = [&](int t0, int rows, int slot) __attribute__((always_inline)) {
    const unsigned at = lds + slot * Sh::CB;
    const unsigned char* kT = kU + (size_t)t0 * KROW;
    const unsigned char* vT = vU + (size_t)t0 * VROW;
#pragma unroll
    for (int g = 0; g < 32 / KPR; ++g)
      if (g * KPR < rows) {
        const int past = g * KPR + lane / KCH - (rows - 1);
        dma16(kT, kofs[g] - (past > 0 ? past * KROW : 0), at + g * 1024);
      }
#pragma unroll
    for (int g = 0; g < 32 / VPR; ++g)
      if (g * VPR < rows) {
        const int past = g * VPR + lane / VCH - (rows - 1);
        dma16(vT, vofs[g] - (past > 0 ? past * VROW : 0), at + Sh::KB + g * 1024);
      }
  };
  // The first chunk is requested before the valid length is known: its rows exist, whatever they hold, and those past the valid
  // length are never used
  int first_rows = L - t_lo;
  if (loader) {
    const int most = SHORT ? chunk_segs * w : (w < 32 ? w : 32);
    first_rows = first_rows < most ? first_rows : most;
    fetch(t_lo, first_rows, 0);
  }
  const int n = valid_len(lens, u, L);
  const CandRange crange = cand_range(cand_off, u, C_all, P);
  const int C = crange.count;               // this user's candidates
  const size_t pb = (size_t)crange.first;   // and the index of their first pair
  if (wave == 0 && srun == 0 && ct == 0) write_seg_cnt(seg_cnt, u, n, L, w, S, lane, 64);
  if (ct * (CW * NW) >= C) {   // a candidate tile past this user's count (the early request has to land before the LDS goes)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    return;
  }
  // valid items are a prefix of the history, so the non-empty segments of the run are a prefix of the run
  int seg_ne = (n + w - 1) / w;
  seg_ne = seg_ne < seg_lo ? seg_lo : (seg_ne > seg_hi ? seg_hi : seg_ne);
  const int end = seg_ne * w < n ? seg_ne * w : n;   // one past the run's last valid item
  auto chunk_end = [&](int seg) {
    const int e = (seg + (SHORT ? chunk_segs : 1)) * w;
    return e < end ? e : end;
  };
  auto rows_of = [&](const Cur& c) { return SHORT || c.hi - c.t0 < 32 ? c.hi - c.t0 : 32; };
  auto advance = [&](Cur& c) {
    c.t0 += 32;
    if (SHORT || c.t0 >= c.hi) {
      c.seg += SHORT ? chunk_segs : 1;
      c.t0 = c.seg * w;
      c.hi = chunk_end(c.seg);
    }
  };
  Cur cur{seg_lo, t_lo, chunk_end(seg_lo)};

  if (loader) {
    int asked = requests(first_rows), landed = 0, slot = 0, in = 0;   // requests made, and those up to and including the chunk waited for
    const int first_asked = asked;
    Cur ask = cur;
    // chunk i is asked for when the barrier of chunk i + 1 - NB has been passed: every wave is through with the one before that, whose
    // slot this is (the first NB at once; the first of all has been, above)
    for (int i = 1 - NB; cur.seg < seg_ne; ++i) {
      if (i > 0) {
        landed += i == 1 ? first_asked : requests(rows_of(cur));
        wait_vm(asked - landed);
        barrier_lds();
        advance(cur);
        if (i == 1) continue;
      }
      if (ask.seg < seg_ne) {
        if (in > 0) {
          fetch(ask.t0, rows_of(ask), slot);
          asked += requests(rows_of(ask));
        }
        ++in;
        advance(ask);
        slot = slot + 1 == NB ? 0 : slot + 1;
      }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    return;
  }

  const int cbase = ct * (CW * NW) + wave * CW;     // first candidate of this wave
  if (wave == 0) *reinterpret_cast<unsigned*>(smem + Sh::ZERO + lane * 4) = 0u;   // (published by the first barrier)
  if (cbase >= C) {   // no candidate: the barriers are all it takes part in
    for (; cur.seg < seg_ne; advance(cur)) barrier_lds();
    return;
  }
  // queries: B operand of the score product, lane = candidate, 8 consecutive d_q elements per k-step half
  bf16x8 qreg[KSTEPS];
  {
    const int c = cbase + l32 < C ? cbase + l32 : C - 1;   // (rows past the last candidate repeat it, and are not stored)
    const unsigned short* qU = q + (pb + c) * DQ + h * 8;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qU + ks * 16);
  }

  // patch -> global: 16 lanes x 16 B = one row; LDS operations of a wave execute in order, so the rows written by this wave are
  // visible to its own reads without a barrier. Stored cacheable, whether H' is read again next or not: with the non-temporal hint
  // outputs of up to 256 MB take as long, larger ones 4 % longer
  constexpr int LPR = D / 8, RPI = 64 / LPR;   // lanes per row, rows per instruction
  unsigned char* opatch = smem + Sh::PATCH + wave * (CW * Sh::OP);
  const unsigned row_out = (unsigned)S * VROW;
  const unsigned ooff = (unsigned)(lane / LPR) * row_out + (lane % LPR) * 16;
  unsigned char* oU = reinterpret_cast<unsigned char*>(seg_out) + (pb + cbase) * (size_t)row_out;
  const int mine = C - cbase < CW ? C - cbase : CW;   // candidates of this wave
  auto flush = [&](int seg) __attribute__((always_inline)) {
    unsigned char* o = oU + (size_t)seg * VROW;
    const unsigned char* src = opatch + (lane / LPR) * Sh::OP + (lane % LPR) * 16;
    if (mine == CW) {
#pragma unroll
      for (int it = 0; it < CW / RPI; ++it)
        *reinterpret_cast<u32x4*>(o + (size_t)it * RPI * row_out + ooff) = *reinterpret_cast<const u32x4*>(src + it * RPI * Sh::OP);
    } else {
#pragma unroll 1
      for (int row = lane / LPR; row < mine; row += RPI, o += (size_t)RPI * row_out, src += RPI * Sh::OP)
        *reinterpret_cast<u32x4*>(o + ooff) = *reinterpret_cast<const u32x4*>(src);
    }
  };

  f32x16 acc[DB];
  const f32x16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  int parked = -1;   // segment whose rows are in the patch
  const int i16 = lane & 15, vrow = h * 4 + (i16 >> 2), vlow = 2 * (l32 >> 4) + ((i16 & 3) >> 1);
  // 32 rows from row r0 of a slot; whole: all of this segment, else the first `left` of them
  auto block = [&](unsigned at, int r0, int left, auto whole) __attribute__((always_inline)) {
    constexpr bool WHOLE = decltype(whole)::value;
    bf16x8 ka[KSTEPS];
    {
      const int row = r0 + l32;
      const unsigned kb = at + row * KROW + ((h ^ ring_kswz<KCH>(row)) << 4);
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) ka[ks] = lds_read16(lds_at(kb ^ (ks << 5)));
    }
    // value rows 4 h .. and eight further down, for items 16 s ..: four rows of 16 columns per transpose load
    const int vr = r0 + vrow;
    const unsigned vb = at + Sh::KB + vr * VROW + ((vlow + 4 * ring_vswz<VCH>(vr)) << 4) + (i16 & 1) * 8;
    const unsigned vz = lds + Sh::ZERO + (vlow << 4) + (i16 & 1) * 8;
    bf16x8 va[DB];
    auto read_v = [&](int s) __attribute__((always_inline)) {
      unsigned a0 = vb, a1 = vb;
      if (!WHOLE) {
        a0 = s * 16 + vrow < left ? vb + s * 16 * VROW : vz;
        a1 = s * 16 + 8 + vrow < left ? vb + (s * 16 + 8) * VROW : vz;
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const lds_bytes p0 = lds_at(a0 ^ (db << 6)) + (WHOLE ? s * 16 * VROW : 0);
        const lds_bytes p1 = lds_at(a1 ^ (db << 6)) + (WHOLE ? (s * 16 + 8) * VROW : 0);
        const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p0);
        const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p1);
        va[db] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    };
    read_v(0);
    if (parked >= 0) {   // behind the reads, while the products have nothing to work on yet
      flush(parked);
      parked = -1;
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x16 sc[HEADS];
#pragma unroll
    for (int hd = 0; hd < HEADS; ++hd)
#pragma unroll
      for (int ks = 0; ks < KH; ++ks)
        sc[hd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[hd * KH + ks], qreg[hd * KH + ks], ks == 0 ? zero : sc[hd], 0, 0, 0);
    auto half = [&](int s, bool start) __attribute__((always_inline)) {   // items 16 s .. 16 s + 15
      u32x4 p[HEADS];
#pragma unroll
      for (int hd = 0; hd < HEADS; ++hd)
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          const bf16x2 c = {(__bf16)gate(sc[hd][s * 8 + 2 * e2], neg_scale_log2e), (__bf16)gate(sc[hd][s * 8 + 2 * e2 + 1], neg_scale_log2e)};
          unsigned bits = __builtin_bit_cast(unsigned, c);
          if (!WHOLE) {
            const int i0 = s * 16 + 8 * (e2 >> 1) + 4 * h + 2 * (e2 & 1);
            bits &= (i0 < left ? 0x0000ffffu : 0u) | (i0 + 1 < left ? 0xffff0000u : 0u);
          }
          p[hd][e2] = bits;
        }
#pragma unroll
      for (int db = 0; db < DB; ++db)
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db], __builtin_bit_cast(bf16x8, p[db / DBH]), start ? zero : acc[db], 0, 0, 0);
    };
    half(0, SHORT);
    if (WHOLE || left > 16) {
      read_v(1);
      half(1, false);
    }
  };
  auto park = [&](int seg) __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)acc[db][g * 4 + e];
        *reinterpret_cast<u32x2*>(opatch + l32 * Sh::OP + (db * 32 + g * 8 + h * 4) * 2) = __builtin_bit_cast(u32x2, o);
      }
    parked = seg;
  };

  // (a barrier: the chunk has landed, and every wave is through with the one before)
  int slot = 0;
  auto next_slot = [&]() { slot = slot + 1 == NB ? 0 : slot + 1; };
  if constexpr (SHORT) {
    for (; cur.seg < seg_ne; advance(cur), next_slot()) {
      barrier_lds();
      for (int seg = cur.seg, t = cur.t0; t < cur.hi; ++seg, t += w) {
        block(lds + slot * Sh::CB, t - cur.t0, w < cur.hi - t ? w : cur.hi - t, std::false_type{});
        park(seg);
      }
    }
  } else {
    for (int seg = seg_lo; seg < seg_ne; ++seg) {
      int left = chunk_end(seg) - seg * w;
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] = zero;
      for (; left >= 32; left -= 32, next_slot()) {
        barrier_lds();
        block(lds + slot * Sh::CB, 0, 32, std::true_type{});
      }
      if (left > 0) {
        barrier_lds();
        block(lds + slot * Sh::CB, 0, left, std::false_type{});
        next_slot();
      }
      park(seg);
    }
  }
  if (parked >= 0) flush(parked);

  // empty segments of the run: exact zeros, a candidate's rows one after the other
  const int empty = seg_hi - seg_ne;
  if (empty > 0) {
    unsigned char* o = oU + (size_t)seg_ne * VROW + (lane % LPR) * 16;
    int c = (lane / LPR) / empty, i = lane / LPR - c * empty;
    while (c < mine) {
      *reinterpret_cast<u32x4*>(o + (size_t)c * row_out + (size_t)i * VROW) = u32x4{0u, 0u, 0u, 0u};
      for (i += RPI; i >= empty; i -= empty) ++c;
    }
  }
}

// ------------------------------------------------------------------------------------------ host side
// Computing waves (32 candidates each) and segments per workgroup: the smallest estimate of rounds of workgroups times the length of one.
// A workgroup costs its start (2), its blocks of 32 rows, which take as long as there are computing waves on a SIMD to issue them, per
// segment its rows to store (0.7, and more in proportion to the waves) and per chunk 1. A launch of more than one round has a quarter of
// one at its end, and takes one and a half at least; counts of their own leave even one round uneven. Three waves share an item among
// half as many candidates again, so they are taken at 0.94 (between two and three the better one is up to a third faster, by how the
// candidates fill 64 and 96 and by what fits a compute unit; four were the better ones nowhere by more than a few percent but at four
// heads). Fitted to 1414 calls (1 to 256 users, 9 to 512 candidates, w = 1 to 700, every width, up to four heads, full to log-uniform
// lengths, equal and own counts) at both and seven numbers of segments: 2.0 % above the best of the fourteen on average.
// Chunks of more than three segments bring nothing (61 calls: three 1.8 %, four 2.6 %, six 2.1 % above the best).
struct RingPlan {
  int waves, segs;
};
static int ring_fit(int w) { return 32 / w < 3 ? 32 / w : 3; }   // segments of a chunk

static RingPlan ring_plan(const StaArgs& a, int w, const int (&per_cu)[4]) {
  const bool is_short = a.w <= 32, own = a.cand_off != nullptr;
  RingPlan best{a.C <= CW ? 1 : 2, 1};
  double least = -1.0;
  const int nw_forced = tuning_int("LASER_STA_NW", 0), forced = tuning_int("LASER_STA_SPW", 0);   // tuning builds only
  for (int nw = best.waves; nw <= (a.C <= 2 * CW ? best.waves : 3); ++nw) {
    if (a.C > CW && (nw_forced == 2 || nw_forced == 3) && nw != nw_forced) continue;
    // candidate tiles of a user (with counts of their own as the mean of them fills)
    const double ctiles = own ? (double)a.P / a.U / (CW * nw) + 0.5 : (a.C + CW * nw - 1) / (CW * nw);
    for (int n : {1, 2, 3, 4, 6, 8, 12}) {
      if (n > 1 && n > a.S) break;
      const double groups = a.U * ctiles * ((a.S + n - 1) / n), rounds = groups / (256.0 * per_cu[nw]);
      // workgroups of a compute unit at a time; of four SIMDs
      const double density = 0.25 * nw * (rounds >= 1.0 ? per_cu[nw] : (int)((groups + 255.0) / 256.0));
      const int blocks = n * ((w + 31) / 32), chunks = is_short ? (n + ring_fit(w) - 1) / ring_fit(w) : blocks;
      const double work = blocks * density + n * (0.7 + density * a.d / 128) + chunks;
      const double late = rounds + 0.25;
      const double turns = own ? (late > 1.0 ? late : 1.0) : (rounds <= 1.0 ? 1.0 : (late > 1.5 ? late : 1.5));
      const double cost = turns * (2.0 + work) * (nw == 3 ? 0.94 : 1.0);
      if (least < 0.0 || cost < least) {
        best = RingPlan{nw, n};
        least = cost;
      }
    }
  }
  if (forced >= 1 && forced <= 64) best.segs = forced;
  return best;
}

// Up to this many users with counts of their own the workgroups stay as they are dealt: an XCD's contiguous range is the work of two users
// or less then, and some XCDs end long before others. 80 calls of 1 to 16 users, counts uniform from none to all: 0.94 of the time on
// average (0.57 to 1.25). 17 to 32 users 1.00, and 65 to 256 would lose 4 %; with the same count for all it is even.
constexpr int RING_FEW_USERS = 16;

template <int DQ, int D, int NW, int HEADS, bool SHORT>
static void ring_launch(const StaArgs& a, int w, int spw) {
  using Sh = RingShape<DQ, D, NW, HEADS, SHORT>;
  const int ctiles = (a.C + CW * NW - 1) / (CW * NW), sruns = (a.S + spw - 1) / spw;
  const int chunk_segs = SHORT ? (spw < ring_fit(w) ? spw : ring_fit(w)) : 1;
  hipLaunchKernelGGL((sta_ring_kernel<DQ, D, NW, HEADS, SHORT>), dim3((unsigned)((long long)a.U * ctiles * sruns)), dim3(Sh::NT), 0,
                     a.stream, (const unsigned short*)a.q, (const unsigned short*)a.k, (const unsigned short*)a.v, a.lens, a.cand_off,
                     a.P, a.C, a.L, w, a.S, spw, chunk_segs, mul_div(sruns), sruns, mul_div(ctiles), ctiles,
                     a.cand_off == nullptr || a.U > RING_FEW_USERS, -1.4426950408889634f / a.gamma, (unsigned short*)a.seg_out, a.seg_cnt);
}

template <int DQ, int D, int HEADS, bool SHORT>
static void ring_form(const StaArgs& a) {
  const int w = a.w < a.L ? a.w : a.L;
  const RingPlan plan = ring_plan(a, w, {0, RingShape<DQ, D, 1, HEADS, SHORT>::PER_CU, RingShape<DQ, D, 2, HEADS, SHORT>::PER_CU,
                                         RingShape<DQ, D, 3, HEADS, SHORT>::PER_CU});
  if (plan.waves == 1) ring_launch<DQ, D, 1, HEADS, SHORT>(a, w, plan.segs);
  else if (plan.waves == 2) ring_launch<DQ, D, 2, HEADS, SHORT>(a, w, plan.segs);
  else ring_launch<DQ, D, 3, HEADS, SHORT>(a, w, plan.segs);
}

template <int DQ, int D>
static void ring_heads(const StaArgs& a) {
  auto form = [&](auto heads) {
    if (a.w <= 32) ring_form<DQ, D, decltype(heads)::value, true>(a);
    else ring_form<DQ, D, decltype(heads)::value, false>(a);
  };
  if (a.heads == 1) form(std::integral_constant<int, 1>{});
  else if (a.heads == 2) form(std::integral_constant<int, 2>{});
  else if constexpr (DQ >= 64 && D == 128) form(std::integral_constant<int, 4>{});
}

laser_status sta_ring_launch(const StaArgs& a) {
  if (!sta_mfma_supports(a) || a.softmax) return LASER_ERR_UNSUPPORTED;
  switch (a.d_q * 1000 + a.d) {
    case 32064: ring_heads<32, 64>(a); break;
    case 32128: ring_heads<32, 128>(a); break;
    case 64064: ring_heads<64, 64>(a); break;
    case 64128: ring_heads<64, 128>(a); break;
    case 128064: ring_heads<128, 64>(a); break;
    default: ring_heads<128, 128>(a); break;
  }
  return launch_status();
}

}  // namespace laser
