// Fused CLM-head scoring GEMM for gfx950 (MI355X): the LoRA-off and LoRA-on
// logits z_off = h W^T and z_on = z_off + s (h A^T) B^T of the CLM head are
// reduced to per-row (max, sum exp) partials and the sampled token's logit
// without ever being written to memory (Sec. 3, the CLM head of pi^hydra;
// App. A, Alg. 1 / Alg. 2, reference and actor log-probabilities).
//
// The vocabulary dimension gives thousands of output tiles, so this GEMM uses
// large tiles, which move the least data per MFMA through L2 and LDS (the
// matrix cores run power-limited, and data movement costs power):
//  * one 256 x 256 output tile per 512-thread workgroup (two waves per SIMD, so
//    that one wave's copies, LDS reads or row statistics run beside the other's
//    MFMAs); each wave owns a 128 x 64 sub-tile = 4 x 2
//    v_mfma_f32_32x32x16_bf16 tiles.  Four waves of 128 x 128 read less from
//    LDS but leave each SIMD one wave: 512 x 4096 x 32000 takes 159 us against
//    147 here, 2000 x 2048 x 50272 490 against 472, 2048 x 4096 x 32000, where
//    the clock gives way to the power limit, 463 against 461.  For few rows
//    tiles of 128 or 64 rows (score_tile below);
//  * K slabs of 32 (64 on the smaller tiles) go through an LDS ring of 3 or 4
//    stages (16-byte chunks XOR-swizzled by the row).  The copies
//    (buffer_load ... lds) are issued by the MFMA waves themselves, a share in
//    every 16-wide k-step;
//  * one barrier per slab: before it every wave has read the slab's last
//    fragments and waited for its copies of the next slab, after it the freed
//    stage is refilled;
//  * the rank-r product T = h A^T is the same for every column tile of a row
//    block, so it is computed once by the pre-pass of lora_tpre.hip (bf16 hi + lo parts of
//    s*T in the workspace, with B zero padded to the padded rank RP next to
//    it) instead of in the main loop;
//  * the LoRA update s*T*B^T is then a GEMM with 2 RP more k values ([hi | lo]
//    against [B | B]); it runs as more slabs through the same ring,
//    right after the per-row (max, sum exp) of the LoRA-off logits have been
//    taken from the accumulators, and the same statistics of the LoRA-on
//    logits follow.  The lane holding the sampled token's column records its
//    logit.  One float4 (max_off, sum_off, max_on, sum_on) per (row, column
//    tile) goes to the workspace for score_combine_kernel.
// With B = 0 or s = 0 the LoRA update adds exact zeros, so the on and off
// statistics (computed by the same code) are bit-identical and KL == 0.
//
// Two inputs (the actor pass and the LoRA-off pass each with their own final
// hidden states, App. A, Alg. 2): the grid holds twice the row tiles, the
// LoRA-off tile and the actor tile of each row block next to each other in
// the tile order (so both read a column block of W while it is in L2).  A
// LoRA-off tile takes only the LoRA-off statistics and runs no LoRA slabs;
// an actor tile runs the LoRA slabs over its own T and takes only the LoRA-on
// statistics.  Each writes its half of the (row, column tile) partial.
#include "hydra_device.h"
#include "hydra_internal.h"

namespace hydra {
namespace {

constexpr int BN = 256;        // tile columns (vocabulary entries)
constexpr int GROUP_M = 8;     // row tiles walked together (L2 reuse of W)

// 2 x (256 / WN) waves of WM x WN each, BK wide K slabs, NS ring stages.
template <int WM_, int WN_, int BK_, int NS_>
struct ScoreTile {
  static constexpr int WM = WM_, WN = WN_, BK = BK_, NS = NS_, BM = 2 * WM;
  static constexpr int NWC = BN / WN, NW = 2 * NWC, NT = NW * 64;
  static constexpr int MT = WM / 32, NTL = WN / 32;  // 32-row x and W tiles per wave
  static constexpr int CPR = BK / 8;                 // 16-byte chunks per LDS row
  static constexpr int RPB = 64 / CPR;               // rows per copy instruction
  static constexpr int SPS = BK / 16;                // 16-wide k-steps per slab
  static constexpr int STAGE = (BM + BN) * CPR;      // uint4 per stage
  static constexpr int XOFF = 0, WOFF = BM * CPR;
  static constexpr int XJ = BM / RPB / NW, WJ = BN / RPB / NW;  // copies per wave and slab
  static constexpr int DPW = XJ + WJ;
  static constexpr int dbeg(int p) { return p * DPW / SPS; }  // first copy of the p-th k-step from the barrier
  static_assert(XJ * RPB * NW == BM && WJ * RPB * NW == BN, "copies split evenly over the waves");
  static_assert(NS >= 2 && NS * STAGE * 16 <= 160 * 1024, "the ring fits in LDS");
  static_assert(2 * 8 * BM * 8 <= STAGE * 16, "the epilogue's row statistics fit in one stage");
  // LDS chunk index of (row, 16-byte chunk c) in a stage: the chunk is XOR-ed
  // with bits of the row so that the 16 lanes of one read phase (16
  // consecutive rows, one chunk) cover all banks.
  __device__ static __forceinline__ int swz(int row) { return CPR == 4 ? (row >> 2) & 3 : (row >> 1) & 7; }
  __device__ static __forceinline__ int sidx(int row, int c) { return row * CPR + (c ^ swz(row)); }
};
using Tile256 = ScoreTile<128, 64, 32, 4>;
using Tile128 = ScoreTile<64, 64, 64, 3>;
using Tile64 = ScoreTile<32, 64, 64, 4>;

static_assert(kScoreTileN == BN, "one partial per GEMM column tile");
static_assert(kScoreTileM == Tile256::BM, "launch shape known to the host checks");

// Workgroup id -> (row tile, column tile): consecutive workgroups go to
// consecutive XCDs; each XCD takes a contiguous range of the logical order,
// which walks GROUP_M row tiles per column tile (the tiles that share rows of W
// run together on one L2).  Contiguous ranges only where the count divides by
// eight cost 289 -> 215 us for 400 rows x 2 inputs at 4096 x 32000 (500 tiles),
// 226 -> 174 for 513 rows of one input (128-row tiles; the 256-row ones
// 190 either way).
__device__ __forceinline__ void tile_of(int bid, int ntm, int ntn, int& tm, int& tn) {
  const int total = ntm * ntn, q = total >> 3, rem = total & 7, xcd = bid & 7;
  const int lid = xcd * q + min(xcd, rem) + (bid >> 3);
  const int per_group = GROUP_M * ntn;
  const int group = lid / per_group;
  const int first_m = group * GROUP_M;
  const int gsize = min(ntm - first_m, GROUP_M);
  const int in = lid - group * per_group;
  tm = first_m + in % gsize;
  tn = in / gsize;
}

template <int N>
__device__ __forceinline__ void wait_vm_lds_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | (((N >> 4) & 3) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int V>
struct IC {
  static constexpr int value = V;
};

// RAGGED: the vocabulary is not a multiple of the column tile, so the last
// column tile masks the columns past N.
template <class T, bool RAGGED, bool DUAL>
__global__ __launch_bounds__(T::NT, T::NT / 256) void score_gemm_kernel(ScoreGemmArgs g) {
  constexpr int NS = T::NS, STAGE = T::STAGE, BM = T::BM, WM = T::WM, MT = T::MT, XOFF = T::XOFF, WOFF = T::WOFF;
  constexpr int XJ = T::XJ, DPW = T::DPW, BK = T::BK, CPR = T::CPR, RPB = T::RPB, SPS = T::SPS;
  constexpr int WN = T::WN, NTL = T::NTL, NWC = T::NWC, NW = T::NW;
  __shared__ uint4 sm[NS][STAGE];
  const int rp = g.rp;  // padded rank (0: no adapter)

  const LinearArgs& a = g.lin;
  const int M = a.M, N = a.N, K = a.K;
  const int t = threadIdx.x;
  const int lane = t & 63;
  // wave-uniform (SGPR) wave index: MFMAs never sit under divergent control flow
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wr = wave / NWC;
  const int wc = wave % NWC;
  const int l32 = lane & 31;
  const int lh = lane >> 5;

  constexpr bool dual = DUAL;
  int tmi, tni;
  const int bid = blockIdx.y * gridDim.x + blockIdx.x;
  if (bid >= (dual ? 2 : 1) * g.ntm * g.ntn) return;  // (the surplus of a split grid)
  tile_of(bid, dual ? 2 * g.ntm : g.ntm, g.ntn, tmi, tni);
  // two inputs: row tile 2 i is the LoRA-off tile of row block i, 2 i + 1 its actor tile
  const bool is_act = dual && (tmi & 1) != 0;
  if (dual) tmi >>= 1;
  const bool do_off = !dual || !is_act;  // this tile takes the LoRA-off statistics
  const bool do_on = !dual || is_act;    // ... and / or the LoRA-on ones
  // (tile coordinates are made provably wave-uniform, so that everything
  // derived from them -- buffer descriptors, LDS bases -- lives in SGPRs)
  const int m0 = __builtin_amdgcn_readfirstlane(tmi * BM);
  const int n0 = __builtin_amdgcn_readfirstlane(tni * BN);
  const int nkt = (K + BK - 1) / BK;
  if (nkt < 1) __builtin_unreachable();  // K >= 8 is validated by the caller
  // The LoRA update s*T*B^T is a GEMM with 2 RP more k values: the rows of
  // [hi | lo] (s*T in bf16 hi and lo parts) against the rows of [Bp | Bp]
  // (B zero padded to RP).  Those run as LS more slabs of the same ring,
  // after the LoRA-off statistics have been taken from the accumulators.
  const int LS = (2 * rp + BK - 1) / BK;
  const int nsl = nkt + (do_on ? LS : 0);  // (LoRA slabs only where they are wanted)

  // the sampled tokens of this lane's four rows, fetched early
  int tk[MT];
#pragma unroll
  for (int mi = 0; mi < MT; ++mi) {
    const int row = m0 + wr * WM + mi * 32 + l32;
    tk[mi] = row < M ? g.tokens[row] : -1;
  }

  // ---- copies.  One copy instruction moves 16 rows x 64 bytes (64 lanes x
  // 16 bytes) into 1 KB of LDS; lane i fills LDS chunk i of it, so it fetches
  // the global chunk that the swizzle maps there.  Buffer resources cover
  // exactly the tile's valid rows (rows past M or N read as zeros); a chunk
  // past K gets an out-of-range offset (zeros as well), and so do all copies
  // of the slabs past the last one, which land in stages that are not read
  // again.  Wave w copies row blocks w, w + NW, ... of the x side (j < XJ) and
  // of the W side (j >= XJ) of every slab.
  const i32x4_t xr = make_rsrc_raw((is_act ? g.x_act : a.x) + (size_t)m0 * K, (uint32_t)min(BM, M - m0) * K * 2u);
  const i32x4_t wrs = make_rsrc_raw(a.W + (size_t)n0 * K, (uint32_t)min(BN, N - n0) * K * 2u);
  const i32x4_t tsr = make_rsrc_raw(g.ts + (size_t)m0 * 2 * rp, (uint32_t)min(BM, M - m0) * 2 * rp * 2u);
  const i32x4_t bpr = make_rsrc_raw(g.bp + (size_t)n0 * rp, (uint32_t)min(BN, N - n0) * rp * 2u);
  const int row_bytes = K * 2;
  const int rl = lane / CPR;  // row within the copy
  // Copy j of slab kt.  MAIN: kt is known to be a slab of h and W (the
  // steady state); otherwise kt may also be a LoRA slab or past the end, and
  // source and offset are selected without branches.
  auto dma_one = [&](auto MAIN, uint4* st, int kt, int j) __attribute__((always_inline)) {
    const int ci = wave + NW * (j < XJ ? j : j - XJ);
    const int row = ci * RPB + rl;
    const int cg = (lane % CPR) ^ T::swz(row);  // global chunk fetched by this lane
    uint4* dst = st + (j < XJ ? XOFF : WOFF) + ci * 64;
    const int k0 = kt * BK;
    const int off_main = k0 + cg * 8 < K ? row * row_bytes + k0 * 2 + cg * 16 : kOutOfRange;
    if constexpr (decltype(MAIN)::value) {
      dma16(j < XJ ? xr : wrs, dst, off_main);
    } else {
      const bool is_main = kt < nkt, is_lora = LS > 0 && kt >= nkt && kt < nsl;
      const int k = (kt - nkt) * BK + cg * 8;  // k within [0, 2 rp) in a LoRA slab (past it: zeros)
      const int off_lora = j < XJ ? (row * 2 * rp + k) * 2 : (row * rp + (k & (rp > 0 ? rp - 1 : 0))) * 2;
      const int off = is_main ? off_main : (is_lora && k < 2 * rp ? off_lora : kOutOfRange);
      dma16(is_main ? (j < XJ ? xr : wrs) : (j < XJ ? tsr : bpr), dst, off);
    }
  };

  f32x16_t acc[MT][NTL];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NTL; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Fragments of one 16-wide k-step: W rows (A operand) and h rows (B
  // operand), double buffered across k-steps.
  struct Frag {
    uint4 w[NTL];
    uint4 x[MT];
  };
  Frag F0, F1;
  auto read_one = [&](Frag& F, const uint4* st, int s, int r) __attribute__((always_inline)) {
    const int ch = 2 * s + lh;
    if (r < NTL)
      F.w[r] = st[WOFF + T::sidx(wc * WN + r * 32 + l32, ch)];
    else
      F.x[r - NTL] = st[XOFF + T::sidx(wr * WM + (r - NTL) * 32 + l32, ch)];
  };

  // k-step S: MFMAs on Fc, reads of k-step RS of the slab in `rs` into Fn, and
  // share P of the copies of slab dkt into `ddst`.
  auto kstep = [&](auto RS, auto P, auto MAIN, const Frag& Fc, Frag& Fn, const uint4* rs, uint4* ddst, int dkt)
      __attribute__((always_inline)) {
    constexpr int NM = MT * NTL, NR = NTL + MT;
    constexpr int D0 = T::dbeg(decltype(P)::value), ND = T::dbeg(decltype(P)::value + 1) - D0;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int mi = m / NTL, ni = m % NTL;
      acc[mi][ni] = mfma32(Fc.w[ni], Fc.x[mi], acc[mi][ni]);
      // the reads spread over the MFMAs, the copies in their first half (reads
      // first and copies last: 1% slower at 4096 x 32000 over two inputs)
#pragma unroll
      for (int r = m * NR / NM; r < (m + 1) * NR / NM; ++r) read_one(Fn, rs, decltype(RS)::value, r);
#pragma unroll
      for (int d = m * 2 * ND / NM; d < (m + 1) * 2 * ND / NM; ++d)
        if (d < ND) dma_one(MAIN, ddst, dkt, D0 + d);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Slab kt (stage `cur`): k-steps 0 .. SPS - 2, which issue the rest of the
  // copies of slab kt + NS - 1 (into the stage of slab kt - 1); the barrier
  // (slab kt + 1 has landed: only the copies of slabs kt + 2 .. kt + NS - 1
  // may still be in flight); the last k-step, which reads slab kt + 1 and
  // issues the first copies of slab kt + NS (into `cur`, now free).
  auto slab = [&](auto MAIN, uint4* cur, uint4* nxt, uint4* prev, int kt) __attribute__((always_inline)) {
    kstep(IC<1>{}, IC<1>{}, MAIN, F0, F1, cur, prev, kt + NS - 1);
    if constexpr (SPS == 4) {
      kstep(IC<2>{}, IC<2>{}, MAIN, F1, F0, cur, prev, kt + NS - 1);
      kstep(IC<3>{}, IC<3>{}, MAIN, F0, F1, cur, prev, kt + NS - 1);
    }
    static_assert(SPS == 2 || SPS == 4, "k-steps listed above");
    wait_vm_lds_barrier<(NS - 2) * DPW>();
    kstep(IC<0>{}, IC<0>{}, MAIN, F1, F0, nxt, cur, kt + NS);
  };

  // prologue: slabs 0 .. NS - 2 and the first copies of slab NS - 1
#pragma unroll
  for (int q = 0; q < NS - 1; ++q)
#pragma unroll
    for (int j = 0; j < DPW; ++j) dma_one(IC<0>{}, sm[q], q, j);
#pragma unroll
  for (int j = 0; j < T::dbeg(1); ++j) dma_one(IC<0>{}, sm[NS - 1], NS - 1, j);
  wait_vm_lds_barrier<(NS - 2) * DPW + T::dbeg(1)>();
#pragma unroll
  for (int r = 0; r < NTL + MT; ++r) read_one(F0, sm[0], 0, r);
  // steady state: every copy issued by slabs kt .. kt + NS - 1 (slabs up to
  // kt + 2 NS - 1) is a copy of h and W
  int kt = 0;
  for (; kt + 2 * NS <= nkt; kt += NS) {
#pragma unroll
    for (int q = 0; q < NS; ++q) slab(IC<1>{}, sm[q], sm[(q + 1) % NS], sm[(q + NS - 1) % NS], kt + q);
  }
  for (; kt < nkt; kt += NS) {
#pragma unroll
    for (int q = 0; q < NS; ++q)
      if (q == 0 || kt + q < nkt) slab(IC<0>{}, sm[q], sm[(q + 1) % NS], sm[(q + NS - 1) % NS], kt + q);
  }

  // ---------------------------------------------------------------- epilogue
  // acc[mi][ni][4 i + e] holds z[m0 + wr*WM + mi*32 + l32][n0 + wc*WN + ni*32 + 8 i + 4 lh + e].
  // Per row block mi and 64-column block: (max, sum exp) over this lane's 32
  // logits.  Those eight partials of a row meet in LDS at the end (per lane
  // merges with the other half of the row, a shuffle each, took 1% of the
  // kernel); they are the same ones, added in the same order, on every tile
  // shape.  For a ragged vocabulary the logits of columns past N are taken as
  // -inf (branch-free).  The lane holding the sampled token's column records
  // its logit.
  constexpr int NB = NTL / 2;  // 64-column blocks per wave
  struct Stat {
    float m, s;
  };
  const int wcol0 = n0 + wc * WN;
  auto row_stats = [&](int mi, int pass, Stat (&st)[NB]) __attribute__((always_inline)) {
    float z[NTL * 16];
#pragma unroll
    for (int ni = 0; ni < NTL; ++ni)
#pragma unroll
      for (int k = 0; k < 16; ++k) z[ni * 16 + k] = acc[mi][ni][k];
    if constexpr (RAGGED) {
      const int lim = N - wcol0 - 4 * lh;  // offsets at or past lim are past N
#pragma unroll
      for (int q = 0; q < NTL * 16; ++q)
        z[q] = (q >> 4) * 32 + 8 * ((q & 15) >> 2) + (q & 3) < lim ? z[q] : -INFINITY;
    }
    const int rel = tk[mi] - wcol0 - 4 * lh;  // column offset within this lane's half
    if (rel >= 0 && rel < WN && ((rel >> 2) & 1) == 0) {
      float v = 0.f;
#pragma unroll
      for (int q = 0; q < NTL * 16; ++q) v = ((q >> 4) * 32 + 8 * ((q & 15) >> 2) + (q & 3) == rel) ? z[q] : v;
      g.zt[(size_t)(m0 + wr * WM + mi * 32 + l32) * 2 + pass] = v;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float mx = -INFINITY;
#pragma unroll
      for (int q = 0; q < 32; ++q) mx = fmaxf(mx, z[b * 32 + q]);
      float s0 = 0.f, s1 = 0.f;
      if (mx != -INFINITY) {
        // e^(z - mx) = 2^(z log2 e - mx log2 e)
        const float mxs = mx * kLog2e;
#pragma unroll
        for (int q = 0; q < 32; q += 2) {
          s0 += __builtin_amdgcn_exp2f(fmaf(z[b * 32 + q], kLog2e, -mxs));
          s1 += __builtin_amdgcn_exp2f(fmaf(z[b * 32 + q + 1], kLog2e, -mxs));
        }
      } else {
        // No column of the vocabulary (-inf: sum 0), or NaN among them, which a
        // maximum passes over.  (The sum of e^z, without the branch, makes the
        // compiler spill 94 registers: 4096 rows at 512 x 60000 345 -> 476 us.)
#pragma unroll
        for (int q = 0; q < 32; ++q) s0 += z[b * 32 + q];
        s0 = s0 != s0 ? s0 : 0.f;
      }
      st[b] = Stat{mx, s0 + s1};
    }
    static_assert(NTL == 2 || NTL == 4, "one or two 64-column blocks");
  };

  Stat st_off[MT][NB], st_on[MT][NB];
  if constexpr (DUAL) {
    // two inputs: an actor tile runs the LoRA slabs, then every tile takes
    // one kind of statistics through a single call site (so that the
    // accumulators are read in one place)
    // (the loop's bound and not a branch: behind a branch on the kind of tile
    // the compiler makes two copies of the statistics and spills a third of
    // the accumulators on the way to them)
    for (int kq = nkt; kq < nsl; ++kq) slab(IC<0>{}, sm[kq % NS], sm[(kq + 1) % NS], sm[(kq + NS - 1) % NS], kq);
    const int pass = is_act ? 1 : 0;
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
      __builtin_amdgcn_sched_barrier(0);
      row_stats(mi, pass, st_off[mi]);
    }
  } else if (do_off) {
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
      __builtin_amdgcn_sched_barrier(0);
      row_stats(mi, 0, st_off[mi]);  // LoRA off
    }
  }
  if constexpr (DUAL) {
    // done above
  } else if (rp > 0) {
    // The LoRA slabs nkt .. nkt + LS - 1 (stage (nkt + q) % NS; the last main
    // slab already read the first k-step of slab nkt into F0).
    for (int q = 0; q < LS; ++q) {
      const int kq = nkt + q;
      slab(IC<0>{}, sm[kq % NS], sm[(kq + 1) % NS], sm[(kq + NS - 1) % NS], kq);
    }
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
      __builtin_amdgcn_sched_barrier(0);
      row_stats(mi, 1, st_on[mi]);  // LoRA on
    }
  } else {
    // no adapter: the LoRA-on logits are the LoRA-off logits
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
#pragma unroll
      for (int b = 0; b < NB; ++b) st_on[mi][b] = st_off[mi][b];
      const int rel = tk[mi] - wcol0 - 4 * lh;
      if (rel >= 0 && rel < WN && ((rel >> 2) & 1) == 0) {
        const size_t zi = (size_t)(m0 + wr * WM + mi * 32 + l32) * 2;
        g.zt[zi + 1] = g.zt[zi];
      }
    }
  }
  wait_vm_lds_barrier<0>();  // every copy has landed and every wave is done with the ring

  // The row's partials (blocks in column order, two lane halves each), in LDS;
  // then one thread per row and pass takes their maximum and the sum rescaled
  // to it.  (A tile of two inputs fills only its own pass.)
  float2* red = reinterpret_cast<float2*>(sm[0]);  // [2 passes][8 partials][BM]
#pragma unroll
  for (int mi = 0; mi < MT; ++mi)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int at = ((wc * NB + b) * 2 + lh) * BM + wr * WM + mi * 32 + l32;
      if constexpr (DUAL) {
        red[(is_act ? 8 * BM : 0) + at] = make_float2(st_off[mi][b].m, st_off[mi][b].s);
      } else {
        red[at] = make_float2(st_off[mi][b].m, st_off[mi][b].s);
        red[8 * BM + at] = make_float2(st_on[mi][b].m, st_on[mi][b].s);
      }
    }
  __syncthreads();
  for (int e = t; e < 2 * BM; e += T::NT) {
    const int rl = e % BM, pass = e / BM, row = m0 + rl;
    if (row >= M || (pass == 0 ? !do_off : !do_on)) continue;
    float2 p[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) p[q] = red[(pass * 8 + q) * BM + rl];
    float mx = p[0].x;
#pragma unroll
    for (int q = 1; q < 8; ++q) mx = fmaxf(mx, p[q].x);
    // (a partial without a finite logit has weight e^-inf = 0 and sum 0, or NaN,
    // which stays)
    float sum = 0.f;
    const float base = mx == -INFINITY ? 0.f : mx;
#pragma unroll
    for (int q = 0; q < 8; ++q) sum = fmaf(p[q].y, exp_e(p[q].x - base), sum);
    reinterpret_cast<float2*>(g.part + (size_t)row * g.ntn + tni)[pass] = make_float2(mx, sum);
  }
}

// The tile (0: 256, 1: 128, 2: 64 rows) by a model of its time in us: rounds of
// 256 tiles (one workgroup per CU) x (fixed + K / 64 x step).  Chosen over M =
// 1 ... 2048, five (K, V) from 512 x 60000 to 4096 x 32000, one and two inputs:
// 0.4% slower than the best tile on average, 8% at most.  M = 100, K = 2048,
// V = 50272: 65 -> 59 us against the 256-row tile; M = 64, K = 4096, V = 32000:
// 92 -> 65; M = 250, K = 3000, V = 20000: 126 -> 79.  All three sum in the same
// order: the choice does not enter the results.
int score_tile(const ScoreGemmArgs& s) {
  constexpr struct {
    int rows;
    float fixed, step;
  } kTiles[3] = {{Tile256::BM, 10.f, 1.30f}, {Tile128::BM, 7.f, 0.82f}, {Tile64::BM, 5.f, 0.65f}};
  int best = 0;
  float cost = 0.f;
  for (int i = 0; i < 3; ++i) {
    const int64_t tiles = (int64_t)((s.lin.M + kTiles[i].rows - 1) / kTiles[i].rows) * s.ntn * (s.x_act ? 2 : 1);
    const float c = (float)((tiles + 255) / 256) * (kTiles[i].fixed + (float)((s.lin.K + 63) / 64) * kTiles[i].step);
    if (i == 0 || c < cost) {
      cost = c;
      best = i;
    }
  }
  return best;
}

template <class T, bool RAGGED>
void launch_tile(ScoreGemmArgs& s, hipStream_t stream) {
  s.ntm = (s.lin.M + T::BM - 1) / T::BM;
  // a dispatch counts the work-items of a dimension in 32 bits: the largest
  // grids are split over y
  const int64_t total = (int64_t)(s.x_act ? 2 : 1) * s.ntm * s.ntn;
  const int64_t gx = total < (int64_t(1) << 22) ? total : int64_t(1) << 22;
  const dim3 grid((uint32_t)gx, (uint32_t)((total + gx - 1) / gx));
  if (s.x_act)
    hipLaunchKernelGGL((score_gemm_kernel<T, RAGGED, true>), grid, dim3(T::NT), 0, stream, s);
  else
    hipLaunchKernelGGL((score_gemm_kernel<T, RAGGED, false>), grid, dim3(T::NT), 0, stream, s);
}

}  // namespace

// The T = h A^T pre-pass (its result the same for every column tile of a row
// block, so formed once), then the GEMM.
hipError_t launch_score_gemm(const ScoreGemmArgs& s_in, hipStream_t stream) {
  ScoreGemmArgs s = s_in;
  s.rp = padded_rank(s.lin.r);
  if (s.rp > 0) {
    TpreArgs t{};
    t.x = s.x_act ? s.x_act : s.lin.x;
    t.A = s.lin.A;
    t.B = s.lin.B;
    t.s = s.lin.s;
    t.M = s.lin.M;
    t.N = s.lin.N;
    t.K = s.lin.K;
    t.r = s.lin.r;
    t.ts = s.ts;
    t.bp = s.bp_buf;
    t.part = s.tpart;
    const hipError_t e = launch_lora_tpre(t, s.rp, &s.bp, stream);
    if (e != hipSuccess) return e;
  }
  const int tile = score_tile(s);
  if (tile == 2)
    launch_tile<Tile64, true>(s, stream);
  else if (tile == 1)
    launch_tile<Tile128, true>(s, stream);
  else if (s.lin.N % BN != 0)
    launch_tile<Tile256, true>(s, stream);
  else
    launch_tile<Tile256, false>(s, stream);
  return hipGetLastError();
}

}  // namespace hydra
