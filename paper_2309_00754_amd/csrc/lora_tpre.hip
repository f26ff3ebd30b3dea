// Pre-pass of the LoRA update of the MFMA GEMMs (the dual-output linear with
// a workspace, and the fused CLM-head scoring GEMM).  T = x A^T is the same
// for every column tile of a row block, so it is computed once here instead
// of inside every tile (at rank 128 against 256-column tiles the in-tile
// product would add half of the base MFMA work):
//  * lora_t_part_kernel (padded ranks 16, 32): one workgroup per 16 rows and
//    K chunk (K split into up to 8 chunks of at least 1024, so that many
//    workgroups share the work), 8 waves taking 32-wide k-steps in turn
//    (v_mfma_f32_16x16x32_bf16, fp32 accumulation), their partial tiles
//    summed in LDS in wave order and written to the workspace;
//  * padded ranks 64, 128: a GEMM of RP columns per K chunk on the smaller
//    tiles of lora_gemm_mid.hip (launch_t_part_mid);
//  * lora_t_finish_kernel: the chunk partials added in chunk order, s * T
//    split into a bf16 hi part and a bf16 lo part (the rounding error of hi),
//    so that the GEMM's bf16 MFMAs add s T B^T to within ~2^-16 relative;
//    extra workgroups pad B to the padded rank when B's own rows cannot be
//    read as they are (r not 16, 32, 64 or 128, or B not 16-byte aligned).
// Both GEMMs then add s T B^T as 2 RP more k values of their main loop:
// rows of [hi | lo] against rows of [Bp | Bp].  Both kernels can also run two
// such pre-passes over the same rows in one launch (the backward's s dy B and
// s x A^T).
#include "hydra_device.h"
#include "hydra_internal.h"

namespace hydra {
namespace {

constexpr int T_WAVES = 8;
constexpr int T_UNROLL = 4;

// Partial T over K chunk kc for the 16 rows of blockIdx.x: the 8 waves take
// the chunk's 32-wide k-steps in turn, T_UNROLL at a time (all their loads in
// flight before the first MFMA); their partial tiles are summed in LDS in
// wave order.
template <int RP>
__device__ __forceinline__ void t_part(const TpreArgs& a, int kch, int kc) {
  constexpr int TJ = RP / 16;
  __shared__ f32x4_t red[T_WAVES][TJ][64];
  const int M = a.M, K = a.K;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l16 = lane & 15;
  const int lg = lane >> 4;
  const int m0 = blockIdx.x * 16;
  const __amdgpu_buffer_rsrc_t hrs = make_rsrc(a.x + (size_t)m0 * K, (uint32_t)min(16, M - m0) * K * 2u);
  const __amdgpu_buffer_rsrc_t ars = make_rsrc(a.A, (uint32_t)min(a.r, RP) * K * 2u);
  f32x4_t acc[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int ks0 = kc * (kch / 32);
  const int ks1 = min((K + 31) / 32, ks0 + kch / 32);
  for (int k0 = ks0 + wave; k0 < ks1; k0 += T_WAVES * T_UNROLL) {
    uint4 hf[T_UNROLL], af[T_UNROLL][TJ];
#pragma unroll
    for (int u = 0; u < T_UNROLL; ++u) {
      const int k = (k0 + u * T_WAVES) * 32 + lg * 8;
      const bool kv = k0 + u * T_WAVES < ks1 && k < K;
      hf[u] = buf_load16(hrs, kv ? (l16 * K + k) * 2 : kOutOfRange);
#pragma unroll
      for (int j = 0; j < TJ; ++j) af[u][j] = buf_load16(ars, kv ? ((j * 16 + l16) * K + k) * 2 : kOutOfRange);
    }
#pragma unroll
    for (int u = 0; u < T_UNROLL; ++u)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[j] = mfma16(hf[u], af[u][j], acc[j]);
  }
  // acc[j] lane l holds T[m0 + 4 (l / 16) + i][16 j + l % 16]
#pragma unroll
  for (int j = 0; j < TJ; ++j) red[wave][j][lane] = acc[j];
  __syncthreads();
  for (int e = t; e < 16 * RP; e += T_WAVES * 64) {
    const int rl = e / RP, j = e % RP;
    const int row = m0 + rl;
    if (row >= M) continue;
    const int src = (rl >> 2) * 16 + (j & 15);
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < T_WAVES; ++w) v += red[w][j >> 4][src][rl & 3];
    a.part[((size_t)kc * M + row) * RP + j] = v;
  }
}

// Up to kMaxGroup pre-passes over the same number of rows in one launch
// (the backward runs s dy B and s x A^T together, a group of linears one
// per member): job j has K chunks ybeg[j] .. ybeg[j + 1] - 1 of blockIdx.y
// and finish blocks bbeg[j] .. bbeg[j + 1] - 1.
struct TpreJobs {
  TpreArgs a[kMaxGroup];
  int kch[kMaxGroup];
  int nkc[kMaxGroup];
  int ybeg[kMaxGroup + 1];
  int bbeg[kMaxGroup + 1];
  int n;
};
// The job that owns item v of a prefix table (wave-uniform).
__device__ __forceinline__ int job_of(const int* beg, int n, int v) {
  int j = 0;
  for (int i = 1; i < n; ++i) j = v >= beg[i] ? i : j;
  return __builtin_amdgcn_readfirstlane(j);
}

template <int RP>
__global__ __launch_bounds__(T_WAVES * 64) void lora_t_part_kernel(TpreJobs jobs) {
  const int y = blockIdx.y;
  const int j = job_of(jobs.ybeg, jobs.n, y);
  t_part<RP>(jobs.a[j], jobs.kch[j], y - jobs.ybeg[j]);
}

// B zero padded to RP columns, by `blocks` workgroups of `threads` threads.
template <int RP>
__device__ __forceinline__ void pad_b(const TpreArgs& a, size_t block, size_t blocks, int threads) {
  const size_t total = (size_t)a.N * RP;
  for (size_t e = block * threads + threadIdx.x; e < total; e += blocks * threads) {
    const int n = (int)(e / RP), j = (int)(e % RP);
    a.bp[e] = j < a.r ? a.B[(size_t)n * a.r + j] : (uint16_t)0;
  }
}

// hi and lo bf16 parts of s * T[row][j], written row-major (ts) and / or
// transposed (tT, whose rows M..Mp are written as zeros: v = 0 there).
__device__ __forceinline__ void t_store(const TpreArgs& a, int rp, size_t row, size_t j, float v) {
  v *= a.s;
  const uint32_t hi = f32_to_bf16_rne(v);
  const uint32_t lo = f32_to_bf16_rne(v - bf16_to_f32(hi));
  if (a.ts && row < (size_t)a.M) {
    a.ts[row * 2 * rp + j] = (uint16_t)hi;
    a.ts[row * 2 * rp + rp + j] = (uint16_t)lo;
  }
  if (a.tT) {
    a.tT[j * a.Mp + row] = (uint16_t)hi;
    a.tT[(rp + j) * a.Mp + row] = (uint16_t)lo;
  }
}

// s * T of element e = row * RP + j from the chunk partials (added in chunk
// order).
template <int RP>
__device__ __forceinline__ void t_finish(const TpreArgs& a, int nkc, size_t e) {
  const int rows = a.tT ? a.Mp : a.M;
  if (e >= (size_t)rows * RP) return;
  const size_t row = e / RP, j = e % RP;
  float v = 0.f;
  if (row < (size_t)a.M) {
    // all chunk loads in flight (nkc <= kTpreMaxChunks), then added in chunk order
    float p[kTpreMaxChunks];
#pragma unroll
    for (int c = 0; c < kTpreMaxChunks; ++c) p[c] = c < nkc ? a.part[((size_t)c * a.M + row) * RP + j] : 0.f;
#pragma unroll
    for (int c = 0; c < kTpreMaxChunks; ++c)
      if (c < nkc) v += p[c];
  }
  t_store(a, RP, row, j, v);
}

// The whole pre-pass in one launch, without partial sums in memory, where K is
// short (use_small below).  A workgroup of 16 waves owns 16 rows and JT * 16 of
// the RP columns; the waves take the 32-wide k-steps in turn, S_UNROLL at a
// time, and their tiles are summed in LDS in wave order.
constexpr int S_WAVES = 16;
constexpr int S_UNROLL = 8;
constexpr int small_jt(int rp) { return rp >= 32 ? 2 : 1; }

template <int RP>
__global__ __launch_bounds__(S_WAVES * 64) void lora_t_small_kernel(TpreJobs jobs) {
  constexpr int JT = small_jt(RP), JG = RP / 16 / JT;  // column groups
  __shared__ f32x4_t red[S_WAVES][JT][64];
  const int nb = jobs.bbeg[jobs.n];
  if ((int)blockIdx.x >= nb) {
    pad_b<RP>(jobs.a[0], blockIdx.x - nb, gridDim.x - nb, S_WAVES * 64);
    return;
  }
  const int jb = job_of(jobs.bbeg, jobs.n, blockIdx.x);
  const TpreArgs& a = jobs.a[jb];
  const int b = blockIdx.x - jobs.bbeg[jb];
  const int M = a.M, K = a.K;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int m0 = b / JG * 16, j0 = b % JG * JT * 16;
  const int rows = max(0, min(16, M - m0));
  const __amdgpu_buffer_rsrc_t hrs = make_rsrc(a.x + (size_t)min(m0, M) * K, (uint32_t)rows * K * 2u);
  const int arows = max(0, min(a.r - j0, JT * 16));
  const __amdgpu_buffer_rsrc_t ars = make_rsrc(a.A + (size_t)min(j0, a.r) * K, (uint32_t)arows * K * 2u);
  f32x4_t acc[JT];
#pragma unroll
  for (int j = 0; j < JT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int nks = (K + 31) / 32;
  for (int k0 = wave; k0 < nks; k0 += S_WAVES * S_UNROLL) {
    uint4 hf[S_UNROLL], af[S_UNROLL][JT];
#pragma unroll
    for (int u = 0; u < S_UNROLL; ++u) {
      const int k = (k0 + u * S_WAVES) * 32 + lg * 8;
      hf[u] = buf_load16(hrs, k < K ? (l16 * K + k) * 2 : kOutOfRange);
#pragma unroll
      for (int j = 0; j < JT; ++j) af[u][j] = buf_load16(ars, k < K ? ((j * 16 + l16) * K + k) * 2 : kOutOfRange);
    }
#pragma unroll
    for (int u = 0; u < S_UNROLL; ++u)
#pragma unroll
      for (int j = 0; j < JT; ++j) acc[j] = mfma16(hf[u], af[u][j], acc[j]);
  }
  // acc[j] lane l holds T[m0 + 4 (l / 16) + i][j0 + 16 j + l % 16]
#pragma unroll
  for (int j = 0; j < JT; ++j) red[wave][j][lane] = acc[j];
  __syncthreads();
  if (t >= 16 * JT * 16) return;
  const int rl = t / (JT * 16), j = t % (JT * 16);
  const int src = (rl >> 2) * 16 + (j & 15);
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < S_WAVES; ++w) v += red[w][j >> 4][src][rl & 3];
  const int row = m0 + rl;
  if (row < (a.tT ? a.Mp : M)) t_store(a, RP, row, j0 + j, v);
}

// Where the one launch is faster than partial sums + finish (and the gap of
// about 1.5 us between them): K short enough that one workgroup's walk over it
// takes no longer than the two launches, or (up to K = 4096 at ranks 16 and 32,
// in the backward up to 2048 at 64 and 128) so many rows that the partial sums
// fill the chip more than once.  Only while its workgroups are
// at most 256, one round (M = 2048, rank 128: 18.1 against 7 + 5; the backward's
// two jobs at M = 2510, K = 4096, rank 16: 16.9 against 11.4 + 4.8).  us a whole
// call, one launch against two, by (rank, K, workgroups): scoring (16, 1000, 64)
// -1.8, (32, 1000, 64) -1.1, (64, 1000, 64) -2.1, (128, 1000, 64) -2.3; linears and
// backward (16, 3000, 64) -0.1, (16, 4096, 64) +2.0, (16, 4096, 128) 0, (16, 4096,
// 176) -1.2, (16, 4096, 256) -3 to -5, (32, 2048, 64) +1.0, (32, 2048, 176) -1.5,
// (32, 4096, 64) +4.5, (32, 4096, 256) -4, (64, 2048, 84) +0.4, (64, 2048,
// 256) in the backward -1.3, (128, 2048, 84) +0.4; members of a group count one by one, for the bits of T, and take +3 to
// +13 where they are more than 256 together.
bool use_small(const TpreArgs& a, int rp) {
  const int K = a.Kform > 0 ? a.Kform : a.K;
  const int64_t groups = (int64_t)((a.M + 15) / 16) * (rp / 16 / small_jt(rp)) * (a.Kall > 0 ? 2 : 1);
  if (groups > 256) return false;
  const int kmany = rp <= 32 ? 4096 : a.Kall > 0 ? 2048 : 0;
  return K <= (rp == 16 ? 3072 : 1024) || (K <= kmany && groups >= 160);
}

// Workgroups [bbeg[j], bbeg[j + 1]) finish job j; those past the last job's
// write job 0's B zero padded to RP when the GEMM cannot read B itself (a
// single job only).
template <int RP>
__global__ __launch_bounds__(256) void lora_t_finish_kernel(TpreJobs jobs) {
  const int b = blockIdx.x;
  const int nb_fin = jobs.bbeg[jobs.n];
  if (b < nb_fin) {
    const int j = job_of(jobs.bbeg, jobs.n, b);
    t_finish<RP>(jobs.a[j], jobs.nkc[j], (size_t)(b - jobs.bbeg[j]) * 256 + threadIdx.x);
    return;
  }
  pad_b<RP>(jobs.a[0], b - nb_fin, gridDim.x - nb_fin, 256);
}

template <int RP>
hipError_t launch_rp(const TpreArgs* as, int n, const uint16_t** bp_used, hipStream_t stream) {
  constexpr bool wide = RP >= 64;
  TpreJobs jobs{};
  jobs.n = n;
  // B serves as its own padded copy when its rows already are RP bf16, 16-byte
  // aligned; no B at all (B null): nothing to pad.  Only a single job pads.
  const TpreArgs& a0 = as[0];
  const bool direct = n > 1 || a0.B == nullptr || (a0.r == RP && (reinterpret_cast<uintptr_t>(a0.B) & 15) == 0);
  if (bp_used) *bp_used = a0.B == nullptr ? nullptr : direct ? a0.B : a0.bp;
  const int M = a0.M;  // (every job has the same rows)
  const size_t pads = ((size_t)a0.N * RP + 255) / 256;
  const int pad_blocks = direct ? 0 : (int)(pads < 2048 ? pads : 2048);
  if (use_small(a0, RP)) {
    for (int j = 0; j < n; ++j) {
      jobs.a[j] = as[j];
      jobs.bbeg[j + 1] = jobs.bbeg[j] + ((as[j].tT ? as[j].Mp : M) + 15) / 16 * (RP / 16 / small_jt(RP));
    }
    hipLaunchKernelGGL((lora_t_small_kernel<RP>), dim3(jobs.bbeg[n] + (pad_blocks + 3) / 4), dim3(S_WAVES * 64), 0,
                       stream, jobs);
    return hipGetLastError();
  }
  for (int j = 0; j < n; ++j) {
    jobs.a[j] = as[j];
    if (!wide) tpre_chunks(as[j].K, jobs.nkc[j], jobs.kch[j]);
    jobs.ybeg[j + 1] = jobs.ybeg[j] + jobs.nkc[j];
    jobs.bbeg[j + 1] = jobs.bbeg[j] + (int)(((size_t)(as[j].tT ? as[j].Mp : as[j].M) * RP + 255) / 256);
  }
  hipError_t e;
  if constexpr (wide) {
    e = launch_t_part_mid(as, n, RP, jobs.nkc, stream);
  } else {
    hipLaunchKernelGGL((lora_t_part_kernel<RP>), dim3((M + 15) / 16, jobs.ybeg[n]), dim3(T_WAVES * 64), 0, stream,
                       jobs);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((lora_t_finish_kernel<RP>), dim3(jobs.bbeg[n] + pad_blocks), dim3(256), 0, stream, jobs);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_lora_tpre(const TpreArgs& a, int rp, const uint16_t** bp_used, hipStream_t stream) {
  switch (rp) {
    case 16: return launch_rp<16>(&a, 1, bp_used, stream);
    case 32: return launch_rp<32>(&a, 1, bp_used, stream);
    case 64: return launch_rp<64>(&a, 1, bp_used, stream);
    case 128: return launch_rp<128>(&a, 1, bp_used, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_lora_tpre_multi(const TpreArgs* as, int n, int rp, hipStream_t stream) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  for (int j = 0; j < n; ++j) {
    if (as[j].M != as[0].M) return hipErrorInvalidValue;
    // no job may need its B padded: B absent, or rows of exactly rp bf16, 16-byte aligned
    if (as[j].B && (as[j].r != rp || (reinterpret_cast<uintptr_t>(as[j].B) & 15) != 0)) return hipErrorInvalidValue;
  }
  switch (rp) {
    case 16: return launch_rp<16>(as, n, nullptr, stream);
    case 32: return launch_rp<32>(as, n, nullptr, stream);
    case 64: return launch_rp<64>(as, n, nullptr, stream);
    case 128: return launch_rp<128>(as, n, nullptr, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_lora_tpre2(const TpreArgs& a0, const TpreArgs& a1, int rp, hipStream_t stream) {
  if (a0.B || a1.B) return hipErrorInvalidValue;
  const TpreArgs as[2] = {a0, a1};
  return launch_lora_tpre_multi(as, 2, rp, stream);
}

}  // namespace hydra
