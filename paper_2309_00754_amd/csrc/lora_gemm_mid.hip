// Dual-path LoRA GEMM for row counts whose 128 x 256 tiles would leave most of
// the 256 CUs idle (prompts, mini-batches, generation batches above 8 rows).
// Same function as lora_gemm_kernel on smaller tiles (GemmMid below): the
// LoRA-off output x W^T and the LoRA-on output x W^T + s (x A^T) B^T from one
// pass over W (Sec. 3, "Dynamic LoRA" and "Stage 2: Hydra-PPO").
//
// What bounds a small tile is the copy of its operands into LDS (about
// 64 B/clk per CU) and the latency of each K slab, not the matrix cores.  So:
//  * one workgroup of 8 waves (4 up to 32 x 64) per tile; the waves that share a
//    sub-tile split every K slab among them (KS ways), which keeps the sub-tile
//    of a wave, and with it the number of MFMAs per LDS byte, large on a small
//    tile;
//  * every wave issues its share of the copies (buffer_load ... lds) for the
//    slab NS ahead, reads the fragments of the next slab from LDS into a second
//    register set, and runs the MFMAs of the current one between them; one
//    barrier per slab;
//  * after the main loop the KS partial sums of a sub-tile meet in LDS by a
//    reduce-scatter (a fixed tree, deterministic), so each of the waves ends
//    with a part of the sub-tile and the epilogue uses all of them;
//  * LoRA: either T = x A^T is accumulated in the main loop
//    (v_mfma_f32_16x16x32_bf16, the rows of A in the slab next to those of W)
//    and s T meets B in the epilogue as bf16 parts, or (PRE) the hi and lo
//    parts of s T and the padded rows of B are read from the pre-pass's
//    workspace.
// The K order of every output depends on the tile shape alone, and the shape
// on M, N and K alone (up to 16 rows on the rank and the members too, among
// shapes of one K order), so an output has the same bits whatever the entry
// point that comes here.
#include "hydra_device.h"
#include "hydra_internal.h"

namespace hydra {
namespace {

// Up to kFewRows rows tiles of kFewRows rows serve, and the sums run in short
// chains: a decode step's outputs keep the error that sums spread over many
// waves give.
constexpr int kFewRows = 16;
constexpr int kFoldSlabs = 4;

struct MidArgs {
  GroupArgs ga;                   // the members' operands; A null: no adapter
  const uint16_t* ts[kMaxGroup];  // PRE: [M x 2 rp] bf16 hi | lo parts of s x A^T (null: no adapter)
  const uint16_t* bp[kMaxGroup];  // PRE: [N x rp] bf16
  int rp;                         // PRE: padded rank
  int kall[kMaxGroup];            // PART: K of member i, cut into nkc[i] chunks of kch[i] (ga.K unused)
  int kch[kMaxGroup];
  int nkc[kMaxGroup];
  int ntm, ntn;                   // tiles of one member
  int total;                      // workgroups
  int vec4;                       // outputs may be written with 16-byte stores
};

// s_waitcnt for at most N vector-memory operations and no LDS operation in
// flight, then the workgroup barrier.
template <int N>
__device__ __forceinline__ void mid_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | (((N >> 4) & 3) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

constexpr size_t cmax(size_t a, size_t b) { return a > b ? a : b; }

// TM x TN output tile, WM x WN sub-tile per wave, KS waves per sub-tile, BK
// wide K slabs in a ring of NS stages, RA rows of A in every slab (the padded
// rank, 0: none).  A tile of 16 rows or columns lies in a sub-tile of 32 whose
// second half repeats the first and is not written.
template <int TM_, int TN_, int WM_, int WN_, int KS_, int BK_, int NS_, int WPC_, int RA_>
struct GemmMid {
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, KS = KS_, BK = BK_, RA = RA_;
  static constexpr int NWM = TM < WM ? 1 : TM / WM, NWN = TN < WN ? 1 : TN / WN, NW = NWM * NWN * KS, NT = NW * 64;
  static constexpr int XMASK = TM < 32 ? TM - 1 : -1, WMASK = TN < 32 ? TN - 1 : -1;  // row of a tile from that of a sub-tile
  static constexpr int TROWS = TM < WM ? TM : WM;  // rows of T of a row block
  static constexpr int MT = WM / 32, NTL = WN / 32, NQ = MT * NTL;
  static constexpr int CPR = BK / 8;               // 16-byte chunks per LDS row
  static constexpr int RPB = 64 / CPR;             // rows per copy instruction
  static constexpr int XB = TM / RPB, WB = TN / RPB, AB = (RA + RPB - 1) / RPB;
  static constexpr int DPW = (XB + WB + AB + NW - 1) / NW;  // copies per wave per slab
  static constexpr int ROWS = TM + TN + AB * RPB;
  static constexpr int PAD = (XB + WB + AB) % NW ? 64 : 0;  // uint4 that the surplus copies fill
  static constexpr int STAGE = ROWS * CPR;         // uint4 per stage
  static constexpr int SPW = BK / 16 / KS;         // 16-wide k-steps per wave and slab
  static constexpr int HS = SPW >= 2 ? SPW / 2 : 1;         // 32-wide k-steps of T per wave and slab
  static constexpr int TSPLIT = SPW >= 2 ? 1 : 2;           // waves that share one of them
  static constexpr int TKS = KS / TSPLIT;                   // partial sums of T
  static constexpr int TPW = RA > 0 ? TROWS / 16 / NWN / TSPLIT : 1;  // 16-row T tiles per wave
  // The partial sums of the KS waves meet in steps (reduce-scatter), or, on the
  // 16-row tiles, all at once: there the epilogue is a fifth of a small call, and
  // the fewer barriers take 0.25 us off it.
  static constexpr bool AT_ONCE = TM < 32;
  static constexpr int EXB = KS > 1 ? NW * NQ * (AT_ONCE ? 4 : 2) * 1024 : 0;  // exchange buffer
  static constexpr int TRB = RA > 0 ? TKS * TM * RA * 4 : 0;                   // partial T
  static constexpr size_t RED = AT_ONCE ? EXB + TRB : cmax(EXB, TRB);
  // s T as bf16 parts, each the rounding error of the ones before: three of
  // them hold all 24 bits (error of y_on against 64 bits 4e-7, with two 2.2e-6)
  static constexpr int BSB = TN * RA * 2;                          // bytes of B's LDS copy
  static constexpr int NP = BSB + TM * 3 * RA * 2 + RED <= 160 * 1024 ? 3 : 2;
  static constexpr int TSB = TM * NP * RA * 2;                     // ... and of s T's
  // Where all parts count, the second and third meet B without its infinities
  // (FIN): the first part decides those outputs, as T itself would, and a part of
  // the other sign, or none, would make them NaN.
  static constexpr bool FIN = RA > 0 && TM < 32;
  static constexpr int B2SB = FIN ? BSB : 0;
  static constexpr size_t EPI = BSB + TSB + B2SB + RED;
  static constexpr size_t kLds = 160 * 1024 / WPC_;
  // fewer stages where they do not fit with the rows of A; an even number where
  // a slab is one k-step (its two fragment sets then alternate with the stages)
  static constexpr int FIT = int((kLds / 16 - PAD) / STAGE);
  static constexpr int NS = SPW == 1 ? (FIT < NS_ ? FIT : NS_) & ~1 : FIT < NS_ ? FIT : NS_;
  static constexpr size_t LDS = cmax((NS * size_t(STAGE) + PAD) * 16, EPI);
  static constexpr int NU = NQ * 4;                // 4-register units of a sub-tile
  static_assert(NS >= 2 && (SPW == 1 || SPW % 2 == 0), "ring and k-steps");
  static_assert(LDS <= kLds, "fits in LDS");
  static_assert(NU % KS == 0, "the reduce-scatter ends with whole units");
  static_assert(!AT_ONCE || (KS == 4 && NWM * NWN == 1), "four partial sums of one sub-tile");
  static_assert(RA == 0 || TM > kFewRows || NP == 3, "every bit of s T on the tiles that serve few rows");
  static_assert(RA == 0 || TPW * NWN * TSPLIT * 16 == TROWS, "T rows split over the waves of a row block");
  static_assert((TM >= 32 || TM == 16) && (TN >= 32 || TN == 16), "whole 16-row fragments of T, whole units of a block");
};

template <int V>
struct IC {
  static constexpr int value = V;
};

// PLAIN: T in the tile (or no adapter); PRE: the update from the pre-pass;
// PART: the pre-pass's own product T = x A^T, one K chunk per workgroup: W is
// A ([r x K], rows past r read as zeros), N the padded rank and y_off the
// partial sums [chunk][M][N].
enum MidMode { PLAIN, PRE, PART };

// FOLD: see the main loop.
template <class G, MidMode MODE, bool FOLD>
__global__ __launch_bounds__(G::NT, G::NT / 256) void lora_gemm_mid_kernel(MidArgs g) {
  constexpr int TM = G::TM, TN = G::TN, WM = G::WM, WN = G::WN, KS = G::KS, BK = G::BK, RA = G::RA;
  constexpr int NW = G::NW, NT = G::NT, MT = G::MT, NTL = G::NTL, NQ = G::NQ, CPR = G::CPR, RPB = G::RPB;
  constexpr int NS = G::NS, STAGE = G::STAGE, SPW = G::SPW, DPW = G::DPW, NU = G::NU, NP = G::NP;
  constexpr int TJ = RA / 16, TJ1 = TJ > 0 ? TJ : 1, TPW = G::TPW, HS = G::HS;
  constexpr int XROW = 0, WROW = TM, AROW = TM + TN;
  __shared__ uint4 sm[G::LDS / 16];

  const int M = g.ga.M, N = g.ga.N, r = g.ga.r;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int kg = wave % KS;            // this wave's share of every slab
  const int wt = wave / KS;            // sub-tile
  const int wr = wt / G::NWN, wc = wt % G::NWN;
  const int l16 = lane & 15, lg = lane >> 4, l32 = lane & 31, lh = lane >> 5;

  // Consecutive workgroups go to consecutive XCDs; each XCD takes a contiguous
  // range of the logical order, which walks the members and, within one, up to
  // 8 row tiles per column tile (the tiles that share rows of W run together
  // on one L2).
  int gi, tmi, tni, kc = 0;
  {
    const int tiles = g.ntm * g.ntn, total = g.total, bid = blockIdx.x;
    const int q = total >> 3, rem = total & 7, xcd = bid & 7;
    int lid = xcd * q + min(xcd, rem) + (bid >> 3);
    gi = lid / tiles;
    lid -= gi * tiles;
    if constexpr (MODE == PART) {  // gi counts (member, chunk) pairs
      kc = gi;
      gi = 0;
      while (kc >= g.nkc[gi]) kc -= g.nkc[gi++];
    }
    const int per_group = 8 * g.ntn;
    const int group = lid / per_group, first_m = group * 8, gsize = min(g.ntm - first_m, 8);
    const int in = lid - group * per_group;
    tmi = first_m + in % gsize;
    tni = in / gsize;
  }
  gi = __builtin_amdgcn_readfirstlane(gi);
  kc = __builtin_amdgcn_readfirstlane(kc);
  // LDK values per row in memory, K of them from column kbeg on for this workgroup
  const int LDK = MODE == PART ? g.kall[gi] : g.ga.K;
  const int kbeg = MODE == PART ? kc * g.kch[gi] : 0;
  const int K = MODE == PART ? min(g.kch[gi], LDK - kbeg) : LDK;
  const uint16_t* const X = g.ga.x[gi] + kbeg;
  const uint16_t* const Wt = g.ga.W[gi] + kbeg;
  const uint16_t* const At = g.ga.A[gi];
  const uint16_t* const Bt = g.ga.B[gi];
  float* const y_off = g.ga.y_off[gi] + (MODE == PART ? (size_t)kc * M * N : 0);
  float* const y_on = MODE == PART ? nullptr : g.ga.y_on[gi];
  const int m0 = __builtin_amdgcn_readfirstlane(tmi * TM);
  const int n0 = __builtin_amdgcn_readfirstlane(tni * TN);
  const int nkt = (K + BK - 1) / BK;
  const bool lora = y_on != nullptr && (MODE == PRE ? g.ts[gi] != nullptr : RA > 0 && At != nullptr && Bt != nullptr);

  // LDS chunk index of (row, 16-byte chunk c): the chunk is XOR-ed with bits of
  // the row so that the 16 lanes of a read phase (16 consecutive rows, one
  // chunk) cover all banks once.
  auto swz = [](int row) __attribute__((always_inline)) { return CPR == 8 ? (row >> 1) & 7 : row & 15; };
  static_assert(CPR == 8 || CPR == 16, "rows of 128 or 256 bytes");
  auto lds_idx = [&](int row, int c) __attribute__((always_inline)) { return row * CPR + (c ^ swz(row)); };

  // ---- copies: one instruction moves RPB rows x BK values (64 lanes x 16
  // bytes); the slab's row blocks (x, W, A) are dealt round-robin to the waves.
  // Every wave issues DPW copies (surplus ones write zeros past the stages), so
  // that the waits below count the same in every wave.
  static_assert(G::XB % NW == 0 && G::WB % NW == 0, "copy j of every wave is of one operand");
  constexpr int XJ = G::XB / NW, WJ = G::WB / NW;
  const int rl = lane / CPR, pc = lane % CPR;
  const int row_bytes = LDK * 2;
  const int wrows = MODE == PART ? max(0, min(TN, r - n0)) : min(TN, N - n0);
  const i32x4_t xr = make_rsrc_raw(X + (size_t)m0 * LDK, ((uint32_t)min(TM, M - m0) * LDK - kbeg) * 2u);
  const i32x4_t wrs =
      make_rsrc_raw(Wt + (size_t)(wrows > 0 ? n0 : 0) * LDK, wrows > 0 ? ((uint32_t)wrows * LDK - kbeg) * 2u : 0u);
  const bool t_on = RA > 0 && lora;
  const i32x4_t ars = make_rsrc_raw(t_on ? At : nullptr, t_on ? (uint32_t)min(r, RA) * K * 2u : 0u);
  auto dma = [&](int stage, int kt, int j) __attribute__((always_inline)) {
    const bool is_a = j >= XJ + WJ;
    const int b = wave + (j < XJ ? j : j < XJ + WJ ? j - XJ : j - XJ - WJ) * NW;  // row block of its operand
    const int lrow = (j < XJ ? XROW : j < XJ + WJ ? WROW : AROW) + b * RPB;       // its first LDS row
    const bool real = !is_a || b < G::AB;
    const int c = pc ^ swz(lrow + rl);
    const int k = kt * BK + c * 8;
    dma16(j < XJ ? xr : j < XJ + WJ ? wrs : ars, real ? sm + stage * STAGE + lrow * CPR : sm + NS * STAGE,
          real && k < K ? (b * RPB + rl) * row_bytes + k * 2 : kOutOfRange);
  };

  f32x16_t acc[MT][NTL];
  f32x4_t accT[TPW][TJ1];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NTL; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
#pragma unroll
  for (int q = 0; q < TPW; ++q)
#pragma unroll
    for (int j = 0; j < TJ1; ++j) accT[q][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Fragments of one 16-wide k-step (W rows as the A operand, x rows as the B
  // operand), double buffered across the wave's k-steps, and of T: this wave's
  // x rows and the rows of A for its 32-wide part of a slab (16x16x32 layout),
  // read and used a slab ahead.
  struct Frag {
    uint4 w[NTL], x[MT];
  };
  constexpr int NRM = NTL + MT, NRT = TJ > 0 ? HS * (TPW + TJ) : 0;
  Frag F[2];
  uint4 tx[HS][TPW], ta[HS][TJ1];
  const int trow = wr * WM + (G::TSPLIT == 1 ? wc : (kg & 1) * G::NWN + wc) * TPW * 16;  // first T row of this wave
  const int tchunk = (G::TSPLIT == 1 ? kg * HS : kg >> 1) * 4 + lg;
  auto read_main = [&](Frag& f, int stage, int st, int q) __attribute__((always_inline)) {
    const uint4* s = sm + stage * STAGE;
    const int ch = 2 * (kg * SPW + st) + lh;
    if (q < NTL)
      f.w[q] = s[lds_idx(WROW + wc * WN + ((q * 32 + l32) & G::WMASK), ch)];
    else
      f.x[q - NTL] = s[lds_idx(XROW + wr * WM + (((q - NTL) * 32 + l32) & G::XMASK), ch)];
  };
  auto read_t = [&](int stage, int r) __attribute__((always_inline)) {
    const uint4* s = sm + stage * STAGE;
    const int hs = r / (TPW + TJ1), q = r % (TPW + TJ1);
    const int ch = tchunk + 4 * hs;
    if (q < TPW)
      tx[hs][q] = s[lds_idx(XROW + trow + q * 16 + l16, ch)];
    else
      ta[hs][q - TPW] = s[lds_idx(AROW + (q - TPW) * 16 + l16, ch)];
  };
  auto mfma_t = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int hs = 0; hs < HS; ++hs)
#pragma unroll
      for (int q = 0; q < TPW; ++q)
#pragma unroll
        for (int j = 0; j < TJ; ++j) accT[q][j] = mfma16(tx[hs][q], ta[hs][j], accT[q][j]);
  };
  // k-step S of slab kt in stage ST: the MFMAs of its fragments, between them
  // the reads of the next k-step; the slab's last k-step comes after the
  // barrier and also copies slab kt + NS into this stage and takes T of slab
  // kt + 1.
  auto kstep = [&](auto S, auto ST, auto PAR, int kt) __attribute__((always_inline)) {
    constexpr int sp = decltype(S)::value, st = decltype(ST)::value, par = decltype(PAR)::value;
    constexpr bool last = sp == SPW - 1;
    constexpr int rst = last ? (st + 1) % NS : st, rsp = last ? 0 : sp + 1;
    if constexpr (last) mid_barrier<(NS - 2) * DPW>();  // slab kt + 1 has landed, slab kt is in registers everywhere
    const Frag& fc = F[par];
    Frag& fn = F[par ^ 1];
    constexpr int NR = NRM + (last ? NRT : 0), ND = last ? DPW : 0;
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      acc[m / NTL][m % NTL] = mfma32(fc.w[m % NTL], fc.x[m / NTL], acc[m / NTL][m % NTL]);
#pragma unroll
      for (int r = m * NR / NQ; r < (m + 1) * NR / NQ; ++r) {
        if (r < NRM)
          read_main(fn, rst, rsp, r);
        else
          read_t(rst, r - NRM);
      }
#pragma unroll
      for (int j = m * ND / NQ; j < (m + 1) * ND / NQ; ++j) dma(st, kt + NS, j);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (last && TJ > 0) mfma_t();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto slab = [&](auto ST, auto PAR, int kt) __attribute__((always_inline)) {
    constexpr int par = decltype(PAR)::value;
    kstep(IC<0>{}, ST, IC<par>{}, kt);
    if constexpr (SPW > 1) kstep(IC<(SPW > 1 ? 1 : 0)>{}, ST, IC<par ^ 1>{}, kt);
    if constexpr (SPW > 2) {
      kstep(IC<(SPW > 2 ? 2 : 0)>{}, ST, IC<par>{}, kt);
      kstep(IC<(SPW > 2 ? 3 : 0)>{}, ST, IC<par ^ 1>{}, kt);
    }
  };

  // B's rows of this tile, zero padded to RA, requested first and put in LDS
  // after the main loop (2-byte loads: B has rows of r values at any even address).
  constexpr int BPT = RA > 0 ? (TN * RA + NT - 1) / NT : 1;
  uint32_t bv[BPT];
  if constexpr (RA > 0) {
    const __amdgpu_buffer_rsrc_t brs =
        make_rsrc(lora ? Bt + (size_t)n0 * r : nullptr, lora ? (uint32_t)min(TN, N - n0) * r * 2u : 0u);
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int e = t + i * NT, n = e / RA, j = e % RA;
      bv[i] = __builtin_amdgcn_raw_buffer_load_b16(brs, e < TN * RA && j < r ? (n * r + j) * 2 : kOutOfRange, 0, 0);
    }
  }

  // prologue: slabs 0 .. NS - 1 (those past the last read zeros)
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int j = 0; j < DPW; ++j) dma(s, s, j);
  mid_barrier<(NS - 1) * DPW>();
#pragma unroll
  for (int r = 0; r < NRM; ++r) read_main(F[0], 0, 0, r);
  if constexpr (TJ > 0) {
#pragma unroll
    for (int r = 0; r < NRT; ++r) read_t(0, r);
    mfma_t();
  }
  // The slabs, unrolled over the ring.  FOLD (up to 16 rows and more than
  // kFoldSlabs slabs): the sums of every kFoldSlabs slabs go to a total, so that
  // no chain of additions has K / (16 KS) links.  Error of y_off and y_on (rank
  // 8) against 64 bits at K = 4096: 1.9e-7 and 1.9e-7 in one chain, 0.9e-7 and
  // 1.0e-7 so; the kernel of 16 waves that served these rows had 1.2e-7 and
  // 1.3e-7.  (Counted in slabs and not in passes over the ring, whose stages
  // depend on the rank: y_off has the same bits at every rank.)
  f32x16_t tot[FOLD ? MT : 1][FOLD ? NTL : 1];
  f32x4_t totT[FOLD ? TPW : 1][TJ1];
  if constexpr (FOLD) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) tot[q / NTL][q % NTL] = acc[q / NTL][q % NTL];
#pragma unroll
    for (int q = 0; q < TPW * TJ; ++q) totT[q / TJ1][q % TJ1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        tot[q / NTL][q % NTL][e] += acc[q / NTL][q % NTL][e];
        acc[q / NTL][q % NTL][e] = 0.f;
      }
#pragma unroll
    for (int q = 0; q < TPW * TJ; ++q) {
      totT[q / TJ1][q % TJ1] += accT[q / TJ1][q % TJ1];
      accT[q / TJ1][q % TJ1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  };
  constexpr int PS = SPW == 1 ? 1 : 0;
  constexpr int UN = NS;
  static_assert(UN <= 8, "slabs listed below");
  for (int kt = 0; kt < nkt; kt += UN) {
#define HYDRA_MID_SLAB(u)                 \
  if constexpr ((u) < UN)                 \
    if ((u) == 0 || kt + (u) < nkt) {     \
      slab(IC<(u) % NS>{}, IC<((u) & PS)>{}, kt + (u)); \
      if constexpr (FOLD)                 \
        if ((kt + (u) + 1) % kFoldSlabs == 0) fold(); \
    }
    HYDRA_MID_SLAB(0)
    HYDRA_MID_SLAB(1)
    HYDRA_MID_SLAB(2)
    HYDRA_MID_SLAB(3)
    HYDRA_MID_SLAB(4)
    HYDRA_MID_SLAB(5)
    HYDRA_MID_SLAB(6)
    HYDRA_MID_SLAB(7)
#undef HYDRA_MID_SLAB
  }
  if constexpr (FOLD) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[q / NTL][q % NTL][e] += tot[q / NTL][q % NTL][e];
#pragma unroll
    for (int q = 0; q < TPW * TJ; ++q) accT[q / TJ1][q % TJ1] += totT[q / TJ1][q % TJ1];
  }
  mid_barrier<0>();  // every copy has landed, every wave is done with the ring

  // ---------------------------------------------------------------- epilogue
  char* const lds = reinterpret_cast<char*>(sm);
  uint16_t* const Bs = reinterpret_cast<uint16_t*>(lds);
  uint16_t* const Ts = reinterpret_cast<uint16_t*>(lds + G::BSB);
  uint16_t* const Bfin = reinterpret_cast<uint16_t*>(lds + G::BSB + G::TSB);  // FIN: B, 0 for infinite and NaN
  char* scratch = lds + G::BSB + G::TSB + G::B2SB;
  // PRE: the tile's rows of ts ([hi | lo], 2 rp values) and of bp (rp values)
  // go to LDS, swizzled like the slabs.  Read from memory per 32 x 32 block
  // they cost 576 KB a workgroup at rank 128 on 128 x 192, here 112 KB.  The
  // copies run during the reduce-scatter where both fit.
  const int rp = MODE == PRE ? g.rp : 16;
  const int lrp = 31 - __builtin_clz(rp);  // rp = 16, 32, 64 or 128
  const int tcl = lrp - 2, bcl = lrp - 3;  // log2 of the 16-byte chunks per row of ts and bp
  const int bs_at = TM << tcl;             // chunk of the first row of bp
  auto up_swz = [](int row, int cl) __attribute__((always_inline)) {
    return (row >> max(0, 4 - cl)) & ((1 << min(cl, 4)) - 1);
  };
  auto stage_update = [&]() __attribute__((always_inline)) {
    const i32x4_t tr = make_rsrc_raw(g.ts[gi] + (size_t)m0 * 2 * rp, (uint32_t)min(TM, M - m0) * 4u * rp);
    const i32x4_t br = make_rsrc_raw(g.bp[gi] + (size_t)n0 * rp, (uint32_t)min(TN, N - n0) * 2u * rp);
    const int tb = (TM << tcl) / 64, bb = (TN << bcl) / 64;  // copies of 64 chunks
    for (int b = wave; b < tb + bb; b += NW) {
      const bool is_t = b < tb;
      const int cl = is_t ? tcl : bcl;
      const int at = (is_t ? b : b - tb) * 64 + lane;
      const int row = at >> cl, c = (at & ((1 << cl) - 1)) ^ up_swz(row, cl);
      dma16(is_t ? tr : br, sm + b * 64, ((row << cl) + c) * 16);
    }
  };
  const bool staged = MODE == PRE && lora;
  bool early = false;
  if constexpr (MODE == PRE) {
    const size_t bytes = (size_t)(bs_at + (TN << bcl)) * 16;
    early = staged && bytes + G::EXB <= G::LDS;
    if (early) {
      scratch = lds + bytes;
      stage_update();
    }
  }
  // The KS partial sub-tiles, in units of four registers (unit u = 4 (mi NTL + ni)
  // + i), are summed over the waves in the order (0 + 1) + (2 + 3); afterwards
  // this wave holds the NU / KS units from u0.
  int u0 = 0;
  f32x4_t un[NU];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      un[q * 4 + i] = f32x4_t{acc[q / NTL][q % NTL][4 * i], acc[q / NTL][q % NTL][4 * i + 1],
                              acc[q / NTL][q % NTL][4 * i + 2], acc[q / NTL][q % NTL][4 * i + 3]};
  f32x4_t* const ex = reinterpret_cast<f32x4_t*>(scratch);
  if constexpr (G::AT_ONCE) {
#pragma unroll
    for (int u = 0; u < NU; ++u) ex[(u * KS + kg) * 64 + lane] = un[u];
  }
  auto sum_at_once = [&]() __attribute__((always_inline)) {
    u0 = kg * (NU / KS);
#pragma unroll
    for (int u = 0; u < NU / KS; ++u) {
      const f32x4_t* p = ex + (u0 + u) * KS * 64 + lane;
      un[u] = (p[0] + p[64]) + (p[128] + p[192]);
    }
  };
  if constexpr (G::AT_ONCE && RA == 0) {
    __syncthreads();
    sum_at_once();
  }
  if constexpr (RA > 0) {
#pragma unroll
    for (int i = 0; i < BPT; ++i)
      if (t + i * NT < TN * RA) {
        Bs[t + i * NT] = (uint16_t)bv[i];
        if constexpr (G::FIN) Bfin[t + i * NT] = (bv[i] & 0x7F80) == 0x7F80 ? 0 : (uint16_t)bv[i];
      }
    // accT[q][j] holds T[trow + 16 q + 4 lg + e][16 j + l16] over this wave's k values
    float* tp = reinterpret_cast<float*>(scratch + (G::AT_ONCE ? G::EXB : 0));
#pragma unroll
    for (int q = 0; q < TPW; ++q)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tp[((kg / G::TSPLIT) * TM + trow + q * 16 + 4 * lg + e) * RA + 16 * j + l16] = accT[q][j][e];
    __syncthreads();
    if constexpr (G::AT_ONCE) sum_at_once();
    for (int e = t; e < TM * RA; e += NT) {
      float v = tp[e];
#pragma unroll
      for (int k2 = 1; k2 < G::TKS; ++k2) v += tp[k2 * TM * RA + e];
      v *= g.ga.s[gi];
      const int row = e / RA, j = e % RA;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const uint32_t part = f32_to_bf16_rne(v);
        Ts[(row * NP + p) * RA + j] = (uint16_t)part;
        v = (part & 0x7FFF) < 0x7F80 ? v - bf16_to_f32(part) : 0.f;  // (an infinity has no rounding error)
      }
    }
    __syncthreads();
  }

  // Reduce-scatter: at step 2^b the waves kg and kg ^ 2^b exchange halves of the
  // units they still hold.
  if constexpr (!G::AT_ONCE && KS > 1) {
    constexpr int HALF = NU / 2;
    auto step = [&](auto BIT, auto CNT) __attribute__((always_inline)) {
      constexpr int bit = decltype(BIT)::value, cnt = decltype(CNT)::value;
      const bool up = (kg & bit) != 0;  // wave-uniform: this wave keeps the upper half
      if constexpr (bit > 1) __syncthreads();  // the previous step's values have been read
#pragma unroll
      for (int u = 0; u < cnt; ++u) {
        ex[(wave * HALF + u) * 64 + lane] = up ? un[u] : un[u + cnt];
        un[u] = up ? un[u + cnt] : un[u];
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < cnt; ++u) un[u] += ex[((wave ^ bit) * HALF + u) * 64 + lane];
      u0 += up ? cnt : 0;
    };
    step(IC<1>{}, IC<NU / 2>{});
    if constexpr (KS > 2) step(IC<2>{}, IC<NU / 4>{});
    if constexpr (KS > 4) step(IC<4>{}, IC<NU / 8>{});
    static_assert(KS <= 8, "steps listed above");
  }
  if (staged) {
    if (!early) {
      __syncthreads();  // every wave is done with the exchange buffer
      stage_update();
    }
    mid_barrier<0>();
  }
  constexpr int MYU = NU / KS;             // units held
  constexpr int MYQ = MYU >= 4 ? MYU / 4 : 1;  // sub-tile blocks they lie in
  constexpr int UPQ = MYU / MYQ;           // units per block
  u0 = __builtin_amdgcn_readfirstlane(u0);
  auto finish = [&](auto BI) __attribute__((always_inline)) {
    constexpr int b = decltype(BI)::value;
    const int q = (u0 >> 2) + b, i0 = MYU >= 4 ? 0 : (u0 & 3);  // (wave-uniform)
    const int mi = q / NTL, ni = q % NTL;
    const int row = m0 + wr * WM + mi * 32 + l32;
    const int colb = n0 + wc * WN + ni * 32 + 4 * lh;
    auto store = [&](float* y, const f32x4_t (&v)[UPQ]) __attribute__((always_inline)) {
      if (row >= M || (TM < 32 && l32 >= TM)) return;
      float* yr = y + (size_t)row * N;
#pragma unroll
      for (int k = 0; k < UPQ; ++k) {
        const int col = colb + 8 * (i0 + k);
        if (TN < 32 && col >= n0 + TN) continue;
        if (g.vec4 && col + 3 < N) {
          *reinterpret_cast<f32x4_t*>(yr + col) = v[k];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < N) yr[col + e] = v[k][e];
        }
      }
    };
    f32x4_t v[UPQ];
#pragma unroll
    for (int k = 0; k < UPQ; ++k) v[k] = un[b * UPQ + k];
    if (MODE == PART || y_off) store(y_off, v);
    if (!y_on) return;
    if (lora) {
      // s T B^T of the whole 32 x 32 block; this wave adds the units it holds.
      // A operand: rows of [B | B], B operand: rows of [hi | lo] of s T.
      f32x16_t L;
#pragma unroll
      for (int e = 0; e < 16; ++e) L[e] = 0.f;
      if constexpr (MODE == PRE) {
        const int trow = wr * WM + mi * 32 + l32, brow = wc * WN + ni * 32 + l32;
        const int tsw = up_swz(trow, tcl), bsw = up_swz(brow, bcl);
        const int bmask = (1 << bcl) - 1;
        for (int k0 = 0; k0 < (1 << tcl); k0 += 4) {  // chunks of 8 values: two 16-wide k-steps
          uint4 tf[2], bf[2];
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            const int ch = k0 + 2 * ks + lh;
            tf[ks] = sm[(trow << tcl) + (ch ^ tsw)];
            bf[ks] = sm[bs_at + (brow << bcl) + ((ch & bmask) ^ bsw)];
          }
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) L = mfma32(bf[ks], tf[ks], L);
        }
      } else {
        constexpr int RA1 = RA > 0 ? RA : 1;
#pragma unroll
        for (int ks = 0; ks < NP * RA / 16; ++ks) {
          const int k = ks * 16 + lh * 8;
          const uint16_t* const bsrc = G::FIN && ks >= RA / 16 ? Bfin : Bs;
          const uint4 bf =
              *reinterpret_cast<const uint4*>(bsrc + (wc * WN + ((ni * 32 + l32) & G::WMASK)) * RA + k % RA1);
          const uint4 tf =
              *reinterpret_cast<const uint4*>(Ts + (wr * WM + ((mi * 32 + l32) & G::XMASK)) * NP * RA + k);
          L = mfma32(bf, tf, L);
        }
      }
#pragma unroll
      for (int k = 0; k < UPQ; ++k) {
        f32x4_t l;
        if constexpr (MYU >= 4) {
          l = f32x4_t{L[4 * k], L[4 * k + 1], L[4 * k + 2], L[4 * k + 3]};
        } else {
          l = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i == i0 + k) l = f32x4_t{L[4 * i], L[4 * i + 1], L[4 * i + 2], L[4 * i + 3]};
        }
        v[k] += l;
      }
    }
    store(y_on, v);
  };
  static_assert(MYQ <= 4 && UPQ * MYQ == MYU && (MYU >= 4 || 4 % MYU == 0), "blocks listed below");
  finish(IC<0>{});
  if constexpr (MYQ > 1) finish(IC<1>{});
  if constexpr (MYQ > 2) finish(IC<2>{});
  if constexpr (MYQ > 3) finish(IC<3>{});
}

// The tiles, smallest first, with the model that chooses among them (us, at the
// end of a tile's last round): base + rounds x (fixed + slabs x step), rounds
// of 256 tiles (one workgroup per CU) and slabs of 64 k values.  The numbers
// are fits to kernel times over M = 17 ... 4096 and eight (K, N) from 700 to
// 11008 at rank 16 (rms error 11-18%).  What they say: a 64-wide slab of a tile
// costs its bytes at 66 to 74 GB/s per CU whatever the tile, so a larger one is
// cheaper per output as long as it still gives 256 tiles.
// Checked at ranks 0, 16, 32, 64 and 128 over 32 row counts from 17 to 4096 and 13
// (K, N), against the best tile: 0.2, 0.05, 0.03, 0.7 and 0.2% slower on average;
// against the 128 x 256 tile alone 0.46 to 0.55 of its time on average, in no case
// longer at ranks 32 and 64, in 18 of 1248 at the others by 1 to 7%.  Those take
// 128 x 192 tiles, either in one nearly full round with all operands in the
// last-level cache (1400 x 4096 x 4096 rank 0 46.9 -> 49.2 us; weights from memory
// 58.6 -> 53.0) or in several rounds, where at K = 1504 to 4096 the two tiles
// differ by 11% either way in an order that counts of tiles, rounds and bytes do
// not explain (rank 16, 2560 x 1504 x 7000 110 -> 122, 2560 x 4096 x 4096 115 ->
// 119, 1816 x 3000 x 6000 143 -> 127).  Members of a group, whose rounds run
// together, gain up to 18% there (four 1400 x 3000 x 6000 rank 128 535 -> 440),
// and a member's outputs have the bits of its own call: the rule is one for both.
// M x K x N, us: 48 x 4096 x 4096 41.4 -> 11.6, 333 x 4096 x 11008 72 -> 58,
// 512 x 4096 x 4096 47.6 -> 29.9, 1000 x 11008 x 4096 157 -> 121, 500 x 2048 x
// 2048 30.2 -> 13.6 (128 x 256 tile -> here, rank 16).
struct MidTile {
  int tm, tn;
  float base, fixed, step;
};
constexpr MidTile kMidTiles[] = {{32, 32, 1.7f, 2.3f, 0.123f},   {32, 64, 1.5f, 3.0f, 0.176f},
                                 {64, 64, 0.9f, 4.2f, 0.221f},   {64, 128, 0.f, 6.1f, 0.354f},
                                 {128, 128, 0.f, 6.6f, 0.482f},  {128, 192, 0.f, 8.4f, 0.613f}};
constexpr MidTile kBigTile = {kGemmTileM, kGemmTileN, 0.f, 9.0f, 0.720f};  // lora_gemm_kernel
constexpr int kMidTileCount = sizeof(kMidTiles) / sizeof(kMidTiles[0]);

float tile_cost(const MidTile& c, int M, int N, int K) {
  const int64_t tiles = (int64_t)((M + c.tm - 1) / c.tm) * ((N + c.tn - 1) / c.tn);
  return c.base + (float)((tiles + 255) / 256) * (c.fixed + (float)((K + 63) / 64) * c.step);
}

template <class G, MidMode MODE, bool FOLD = false>
hipError_t launch_tile(MidArgs& g, hipStream_t stream) {
  int members = g.ga.G;  // (member, chunk) pairs of the pre-pass
  if constexpr (MODE == PART) {
    members = 0;
    for (int i = 0; i < g.ga.G; ++i) members += g.nkc[i];
  }
  g.ntm = (g.ga.M + G::TM - 1) / G::TM;
  g.ntn = (g.ga.N + G::TN - 1) / G::TN;
  // A dispatch counts its work-items in 32 bits.  The rule gives these tiles at
  // most about 2^19 workgroups, 8 members or jobs (larger outputs take 128 x 256).
  const int64_t total = (int64_t)g.ntm * g.ntn * members;
  if (total * G::NT >= (int64_t(1) << 32)) return hipErrorInvalidValue;
  g.total = (int)total;
  hipLaunchKernelGGL((lora_gemm_mid_kernel<G, MODE, FOLD>), dim3(g.total), dim3(G::NT), 0, stream, g);
  return hipGetLastError();
}

template <class G>
hipError_t launch_plain(MidArgs& g, hipStream_t stream) {
  if constexpr (G::TM == kFewRows)
    if (g.ga.K > kFoldSlabs * G::BK) return launch_tile<G, PLAIN, true>(g, stream);
  return launch_tile<G, PLAIN>(g, stream);
}

// Workgroups per CU that the ring leaves room for: two on the 16-row tiles
// wherever half of the LDS holds three slabs (a ring of 8 and one workgroup
// otherwise: with two slabs a long K waits for every copy).
constexpr int per_cu(int tm, int tn, int ra) {
  return tm == kFewRows && tn > 16 && 80 * 1024 / ((tm + tn + ra) * 256) >= 3 ? 2 : 1;
}

template <int TM, int TN, int WM, int WN, int KS, int BK, int NS>
hipError_t launch_mid(MidArgs& g, int ra, hipStream_t stream) {
  if constexpr ((TM == 64 && TN == 64) || (TM == 128 && TN == 128))  // the pre-pass's own tiles
    if (g.nkc[0] > 0) return launch_tile<GemmMid<TM, TN, WM, WN, KS, BK, NS, 1, 0>, PART>(g, stream);
  if constexpr (TM != kFewRows)
    if (g.rp > 0) return launch_tile<GemmMid<TM, TN, WM, WN, KS, BK, NS, 1, 0>, PRE>(g, stream);
  switch (ra) {
    case 0: return launch_plain<GemmMid<TM, TN, WM, WN, KS, BK, NS, per_cu(TM, TN, 0), 0>>(g, stream);
    case 16: return launch_plain<GemmMid<TM, TN, WM, WN, KS, BK, NS, per_cu(TM, TN, 16), 16>>(g, stream);
    case 32: return launch_plain<GemmMid<TM, TN, WM, WN, KS, BK, NS, per_cu(TM, TN, 32), 32>>(g, stream);
    case 64: return launch_plain<GemmMid<TM, TN, WM, WN, KS, BK, NS, per_cu(TM, TN, 64), 64>>(g, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_any(MidArgs& g, int ra, int tile, hipStream_t stream) {
  switch (tile) {
    case 0: return launch_mid<32, 32, 32, 32, 4, 128, 5>(g, ra, stream);
    case 1: return launch_mid<32, 64, 32, 64, 4, 128, 5>(g, ra, stream);
    case 2: return launch_mid<64, 64, 32, 64, 4, 128, 4>(g, ra, stream);
    case 3: return launch_mid<64, 128, 64, 64, 4, 64, 6>(g, ra, stream);
    case 4: return launch_mid<128, 128, 64, 64, 2, 64, 5>(g, ra, stream);
    case 5: return launch_mid<128, 192, 64, 96, 2, 64, 4>(g, ra, stream);
    default: return hipErrorInvalidValue;
  }
}

// Up to 16 rows without the pre-pass: 16 x 16, 16 x 32 and 16 x 64 tiles.  All
// three sum in the same order (KS, BK and the folds are theirs in common), so
// that this choice, unlike gemm_mid_tile's, may look at the rank and at the
// members of the launch and an output still has the same bits in every call.
// Model as kMidTiles', slabs of 128 k values: with two workgroups per CU a pair
// takes `pair` per slab.  Fits over 9 and 16 rows, 1 to 8 members, 17 (K, N) from
// 512 x 512 to 4096 x 32000 (rms error 6-20%; the choice is 3% slower than the
// best of six forms on average, and at most 5% slower than the 32-row tiles).
// What they say: few workgroups wait for each slab's latency, so narrow tiles and
// a deep ring win; many are bound by the copies of x and A's rows, which a wider
// tile shares among more outputs.
// us, 9 rows, the 16-wave kernel that split K over 16 to 64 columns -> 32-row
// tiles chosen without rank and members -> here: 4096 x 4096 rank 8 11.7 -> 14.2
// -> 10.6; 8192 x 2048 rank 0 14.6 -> 17.9 -> 12.0; 4096 x 1024 rank 8 11.3 ->
// 14.2 -> 9.7; four 2048 x 8192 rank 64 54 -> 68 -> 39; eight 1000 x 3000 rank 32
// 20 -> 24 -> 19.  Left slower than that first kernel, by 2 to 8%: 520 x 1000 and
// smaller.
struct FewCost {
  float base, fixed, step, pair;
};
constexpr FewCost kFewCosts[3][4] = {
    // rank 0, 16, 32, 64
    {{2.40f, 0.83f, 0.162f, 0.f}, {1.51f, 2.66f, 0.186f, 0.f}, {1.23f, 3.54f, 0.263f, 0.f}, {1.08f, 4.85f, 0.389f, 0.f}},
    {{1.78f, 1.64f, 0.238f, 0.689f}, {1.24f, 2.98f, 0.279f, 0.715f}, {1.13f, 3.34f, 0.268f, 0.818f}, {0.26f, 5.56f, 0.488f, 0.f}},
    {{0.56f, 2.91f, 0.314f, 1.327f}, {0.f, 4.39f, 0.415f, 1.386f}, {0.f, 5.28f, 0.521f, 0.f}, {0.f, 6.07f, 0.566f, 0.f}}};

hipError_t launch_few(MidArgs& g, int ra, hipStream_t stream) {
  int best = 0;
  float cost = 0.f;
  for (int i = 0; i < 3; ++i) {
    const int tn = 16 << i;
    const FewCost& c = kFewCosts[i][ra == 0 ? 0 : ra == 16 ? 1 : ra == 32 ? 2 : 3];
    const int per = ((g.ga.N + tn - 1) / tn * g.ga.G + 255) / 256;  // workgroups for every CU
    const float slabs = (float)((g.ga.K + 127) / 128);
    const int pairs = c.pair > 0.f ? per / 2 : 0, ones = per - 2 * pairs;
    const float t = c.base + (float)pairs * (c.fixed + slabs * c.pair) + (float)ones * (c.fixed + slabs * c.step);
    if (i == 0 || t < cost) {
      cost = t;
      best = i;
    }
  }
  switch (best) {
    case 0: return launch_mid<16, 16, 32, 32, 4, 128, 8>(g, ra, stream);
    case 1: return launch_mid<16, 32, 32, 32, 4, 128, 8>(g, ra, stream);
    default: return launch_mid<16, 64, 32, 64, 4, 128, 8>(g, ra, stream);
  }
}

}  // namespace

int gemm_mid_tile(int M, int N, int K) {
  // Up to 16 rows always a small tile: launch_few's, which carry s T in all its
  // 24 bits and sum in short chains, or with the pre-pass (the backward's dx) one
  // of the two of 32 rows.
  const bool few = M <= kFewRows;
  int best = few ? 0 : -1;
  float cost = tile_cost(few ? kMidTiles[0] : kBigTile, M, N, K);
  for (int i = 0; i < kMidTileCount; ++i) {
    if (few && i > 1) break;
    const float c = tile_cost(kMidTiles[i], M, N, K);
    if (c < cost) {
      cost = c;
      best = i;
    }
  }
  return best;
}

// On the smaller tiles T in the tile costs less than the pre-pass's launches
// (10-14 us): 333 x 2048 x 2000 at rank 64 takes 16.6 us in one launch against
// 11.7 + 12.  Not where 128 x 192 tiles of padded rank 64 run more than one
// round: A adds a fifth to every slab of each round, and the pre-pass pays once
// (in the tile -> pre-pass, us: 2692 x 4096 x 4096 132 -> 122, 2300 x 11008 x 4096
// 300 -> 266, 2796 x 3000 x 6000 224 -> 203; 0.94 on average, 1.04 at most).
bool gemm_mid_in_tile(int M, int N, int K, int rp) {
  const int tile = gemm_mid_tile(M, N, K);
  if (tile < 0 || rp > 64) return false;
  const MidTile& c = kMidTiles[tile];
  const int64_t tiles = (int64_t)((M + c.tm - 1) / c.tm) * ((N + c.tn - 1) / c.tn);
  return !(rp == 64 && tile == kMidTileCount - 1 && tiles > 256);
}

hipError_t launch_lora_gemm_mid(const GroupArgs& ga, const uint16_t* const* ts, const uint16_t* const* bp, int rp_pre,
                                int tile, hipStream_t stream) {
  MidArgs g{};
  g.ga = ga;
  g.rp = rp_pre;
  g.vec4 = ga.N % 4 == 0;
  bool any_on = false;
  for (int i = 0; i < ga.G; ++i) {
    g.ts[i] = ts ? ts[i] : nullptr;
    g.bp[i] = bp ? bp[i] : nullptr;
    g.vec4 = g.vec4 && (reinterpret_cast<uintptr_t>(ga.y_off[i]) & 15) == 0 &&
             (reinterpret_cast<uintptr_t>(ga.y_on[i]) & 15) == 0;
    any_on = any_on || (ga.y_on[i] && ga.A[i] && ga.B[i]);
  }
  const int ra = any_on ? padded_rank(ga.r) : 0;
  return ga.M <= kFewRows && rp_pre == 0 ? launch_few(g, ra, stream) : launch_any(g, ra, tile, stream);
}

hipError_t launch_t_part_mid(const TpreArgs* as, int n, int rp, int* nkc, hipStream_t stream) {
  MidArgs g{};
  g.ga.G = n;
  g.ga.M = as[0].M;
  g.ga.N = rp;
  g.ga.r = as[0].r;
  g.vec4 = 1;  // rows of rp fp32 in a 16-byte aligned workspace
  // Tile (64 x 64, at rank 128 also 128 x 128) and chunk length by the model of
  // kMidTiles, plus the partial sums written and read again at 5 TB/s.  Whole
  // linear with pre-pass, us: M = 4096, K = N = 2048, rank 128 56.3 with 2
  // chunks, 60.6 with 4, 69 with 8, 61.6 for 128 x 128 in 8 chunks; 3000 x 4096
  // x 4096, rank 64 126 with 4 chunks against 130; 1024 x 4096 x 4096, rank 128
  // 63.3 with 8 chunks against 64.0 with 4.  The backward's two jobs share a
  // launch and count together: 2900 rows of 8192 and 2048 values, rank 128, 193 us
  // a backward call against 214 with each counted alone.  Tile and length depend
  // on M, Kform, Kall and rp alone, so that T has the same bits in every group.
  const int M = as[0].M;
  const int klong = as[0].Kform > 0 ? as[0].Kform : as[0].K;
  const int kshort = as[0].Kall > 0 ? as[0].Kall - klong : 0;
  int tile = 2, len = 0;
  float cost = 0.f;
  for (int i = 2; i <= (rp == 128 ? 4 : 2); i += 2) {
    const MidTile& c = kMidTiles[i];
    const int64_t tiles = (int64_t)((M + c.tm - 1) / c.tm) * ((rp + c.tn - 1) / c.tn);
    for (int n_long = 1; n_long <= kTpreMaxChunks; ++n_long) {
      const int l = ((klong + n_long - 1) / n_long + 127) / 128 * 128;
      if (n_long > 1 && l < 256) break;
      const int64_t chunks = (klong + l - 1) / l + (kshort + l - 1) / l;
      const float t = c.base + (float)((tiles * chunks + 255) / 256) * (c.fixed + (float)(l / 64) * c.step) +
                      (float)(chunks * M * rp) * 8.f / 5e6f;
      if (len == 0 || t < cost) {
        cost = t;
        tile = i;
        len = l;
      }
    }
  }
  for (int j = 0; j < n; ++j) {
    if (as[j].M != as[0].M || as[j].r != as[0].r) return hipErrorInvalidValue;
    g.ga.x[j] = as[j].x;
    g.ga.W[j] = as[j].A;
    g.ga.y_off[j] = as[j].part;
    g.kall[j] = as[j].K;
    g.kch[j] = len;
    nkc[j] = g.nkc[j] = (as[j].K + len - 1) / len;
    if (nkc[j] > kTpreMaxChunks) return hipErrorInvalidValue;
  }
  return launch_any(g, 0, tile, stream);
}

}  // namespace hydra
