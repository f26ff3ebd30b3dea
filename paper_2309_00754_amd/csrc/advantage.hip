// PPO advantage step for gfx950: the critic's per-token values from its
// scalar head, the per-token PPO reward, and generalized advantage estimation
// (Sec. 2, "Stage 3: PPO": GAE builds the advantage estimates from the reward
// using V; App. A, Alg. 2: critic values on the generated sequence, then the
// advantages from the reward and reference log-probabilities; App. B: KL
// weight beta, GAE gamma and lambda).
//
//  * value_head_kernel: V[m] = <h[m], w_v>.  Each wave takes two rows, which
//    share every chunk of w_v it loads; lane l takes 8 consecutive k of every
//    512-wide chunk (whole 1 KB lines), a batch of 8 chunks is requested
//    before the first is used, and the dot products run on v_dot2c_f32_bf16
//    with fp32 accumulation; the lanes are summed by a fixed butterfly.
//  * gae_kernel: one workgroup (1, 4 or 16 waves by length) per sequence.  r_t = -beta KL_t on response tokens
//    (t >= start), plus the sequence reward on its last token; delta_t = r_t +
//    gamma V_{t+1} - V_t (V_T = 0); A_t = delta_t + gamma lambda A_{t+1}
//    (A_T = 0); returns A_t + V_t; positions before start are written as 0.
//    The recursion is a linear one, evaluated as a reverse scan: thread j owns
//    a contiguous chunk of positions, folds it into (F_j, B_j) = ((gamma
//    lambda)^len, the chunk's advantage at its first position with a zero
//    advantage after it), a Kogge-Stone suffix scan over the lanes and a fold
//    over the waves combine (F, B) pairs, and each thread then runs its chunk
//    backwards from the advantage that follows it.  Chunks of up to 16 positions keep their
//    residuals in registers (all their loads issued up front); longer ones
//    are recomputed in the second pass.  Fixed order throughout:
//    deterministic.
//  * ppo_loss_kernel: the update stage's losses (Sec. 2, "Stage 3: PPO"): the
//    clipped surrogate on the ratio rho = exp(lp_new - lp_old) and the
//    critic's squared-error loss on the returns, means over the response
//    tokens, with their per-token gradients.  One workgroup per loss: thread t
//    takes the groups of four tokens t, t + 1024, ..., and the partial sums meet
//    in a fixed tree; further workgroups write the gradients.
#include "hydra_device.h"
#include "hydra_internal.h"

namespace hydra {
namespace {

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;

__device__ __forceinline__ float dot8(const uint4& a, const uint4& b, float acc) {
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.x), __builtin_bit_cast(bf16x2_t, b.x), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.y), __builtin_bit_cast(bf16x2_t, b.y), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.z), __builtin_bit_cast(bf16x2_t, b.z), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.w), __builtin_bit_cast(bf16x2_t, b.w), acc, false);
  return acc;
}

constexpr int VH_WAVES = 4;  // waves per workgroup
constexpr int VH_ROWS = 2;   // rows per wave (sharing each w_v chunk)
constexpr int VH_BATCH = 8;  // 512-wide chunks requested before use

__global__ __launch_bounds__(VH_WAVES * 64) void value_head_kernel(ValueHeadArgs a) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = (blockIdx.x * VH_WAVES + wave) * VH_ROWS;
  if (row0 >= a.M) return;  // wave-uniform
  const int K = a.K;
  const int nrows = min(VH_ROWS, a.M - row0);
  // rows past M read as zeros through the descriptor
  const __amdgpu_buffer_rsrc_t hrs = make_rsrc(a.h + (size_t)row0 * K, (uint32_t)nrows * K * 2u);
  const __amdgpu_buffer_rsrc_t wrs = make_rsrc(a.w, (uint32_t)K * 2u);
  const int nch = (K + 511) / 512;
  float acc[VH_ROWS];
#pragma unroll
  for (int i = 0; i < VH_ROWS; ++i) acc[i] = 0.f;
  for (int c0 = 0; c0 < nch; c0 += VH_BATCH) {
    uint4 hv[VH_BATCH][VH_ROWS], wv[VH_BATCH];
#pragma unroll
    for (int u = 0; u < VH_BATCH; ++u) {
      const int k = (c0 + u) * 512 + lane * 8;
      const bool kv = c0 + u < nch && k < K;
      wv[u] = buf_load16(wrs, kv ? k * 2 : kOutOfRange);
#pragma unroll
      for (int i = 0; i < VH_ROWS; ++i) hv[u][i] = buf_load16(hrs, kv ? (i * K + k) * 2 : kOutOfRange);
    }
#pragma unroll
    for (int u = 0; u < VH_BATCH; ++u)
#pragma unroll
      for (int i = 0; i < VH_ROWS; ++i) acc[i] = dot8(hv[u][i], wv[u], acc[i]);
  }
#pragma unroll
  for (int i = 0; i < VH_ROWS; ++i) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc[i] += __shfl_xor(acc[i], o);
  }
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < VH_ROWS; ++i)
      if (i < nrows) a.values[row0 + i] = acc[i];
  }
}

constexpr int GAE_REG = 16;  // chunk length held in registers

// NT threads per sequence, a contiguous chunk of positions each.
template <int NT>
__global__ __launch_bounds__(NT) void gae_kernel(GaeArgs a) {
  constexpr int NW = NT / 64;
  __shared__ float wf[NW], wb[NW];
  const int b = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int T = a.seq_len;
  const int C = (T + NT - 1) / NT;  // positions per thread
  const int t0 = t * C;
  const int t1 = min(T, t0 + C);
  const size_t base = (size_t)b * T;
  const float c = a.gamma * a.lam;
  const float rew = a.reward[b];

  auto reward_at = [&](int p, float kl) __attribute__((always_inline)) {
    float r = p >= a.start ? -a.beta * kl : 0.f;
    if (p == T - 1) r += rew;
    return r;
  };
  auto delta_at = [&](int p) __attribute__((always_inline)) {
    const float v1 = p + 1 < T ? a.values[base + p + 1] : 0.f;
    return fmaf(a.gamma, v1, reward_at(p, a.kl[base + p])) - a.values[base + p];
  };

  // this thread's chunk folded with a zero advantage after it
  float F = 1.f, Bv = 0.f;
  float dl[GAE_REG], vl[GAE_REG], rl[GAE_REG];
  const bool in_regs = C <= GAE_REG;
  if (in_regs) {
    float kv[GAE_REG];
#pragma unroll
    for (int i = 0; i < GAE_REG; ++i) {
      const int p = t0 + i;
      kv[i] = i < C && p < T ? a.kl[base + p] : 0.f;
      vl[i] = i < C && p < T ? a.values[base + p] : 0.f;
    }
    const float vn = t1 < T && t0 < T ? a.values[base + t1] : 0.f;  // the value after the chunk
#pragma unroll
    for (int i = 0; i < GAE_REG; ++i) {
      const int p = t0 + i;
      const float v1 = p + 1 < t1 ? vl[i + 1 < GAE_REG ? i + 1 : i] : vn;
      rl[i] = reward_at(p, kv[i]);
      dl[i] = fmaf(a.gamma, v1, rl[i]) - vl[i];
    }
#pragma unroll
    for (int i = GAE_REG - 1; i >= 0; --i) {
      if (t0 + i < t1) {
        Bv = fmaf(c, Bv, dl[i]);
        F *= c;
      }
    }
  } else {
    for (int p = t1 - 1; p >= t0; --p) {
      Bv = fmaf(c, Bv, delta_at(p));
      F *= c;
    }
  }
  // suffix scan over lanes: (F, B)_j <- (F_j F_{j+o}, B_j + F_j B_{j+o})
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float Fo = __shfl_down(F, o);
    const float Bo = __shfl_down(Bv, o);
    if (lane + o < 64) {
      Bv = fmaf(F, Bo, Bv);
      F *= Fo;
    }
  }
  // advantage right after this thread's chunk: the suffix of lane + 1 over the
  // suffix of the waves after this one
  float A = __shfl_down(Bv, 1), Fn = __shfl_down(F, 1);
  if (lane == 63) {
    A = 0.f;
    Fn = 1.f;
  }
  if constexpr (NW > 1) {
    if (lane == 0) {
      wf[wave] = F;
      wb[wave] = Bv;
    }
    __syncthreads();
    float after = 0.f;
    for (int w = NW - 1; w > wave; --w) after = fmaf(wf[w], after, wb[w]);
    A = fmaf(Fn, after, A);
  }
  if (in_regs) {
#pragma unroll
    for (int i = GAE_REG - 1; i >= 0; --i) {
      const int p = t0 + i;
      if (p < t1) {
        A = fmaf(c, A, dl[i]);
        const bool resp = p >= a.start;
        a.advantages[base + p] = resp ? A : 0.f;
        a.returns[base + p] = resp ? A + vl[i] : 0.f;
        if (a.rewards) a.rewards[base + p] = rl[i];
      }
    }
  } else {
    for (int p = t1 - 1; p >= t0; --p) {
      A = fmaf(c, A, delta_at(p));
      const bool resp = p >= a.start;
      a.advantages[base + p] = resp ? A : 0.f;
      a.returns[base + p] = resp ? A + a.values[base + p] : 0.f;
      if (a.rewards) a.rewards[base + p] = reward_at(p, a.kl[base + p]);
    }
  }
}

constexpr int PL_THREADS = 1024;
constexpr int PL_BATCH = 4;  // groups of four tokens per thread requested before use

// Workgroup 0 adds up the policy loss and the clip count, workgroup 1 the value
// loss, the others write the gradients of 4096 tokens each.  One compute unit
// takes in about 65 GB/s, so what a sum reads (12 and 8 bytes a token) bounds
// it: 42900 tokens take 9.9 us; one workgroup that did all of it (28 bytes a
// token) took 20.5, reading 4 bytes at a time 18.6.  Value head (K = 512), GAE
// and loss over 64 x 2048 tokens 138 -> 89 us a step.
// VEC: every array is 16-byte aligned.  A thread's group of four tokens is then
// 4 t .. 4 t + 3 of a block of 4096 in one load per array, and the M % 4 tokens
// left over are taken one by one; else tokens t, t + 1024, ... of the block, so
// that the lanes of a 4-byte load stay side by side (46 x 1659 tokens, four
// neighbouring tokens a thread in 4-byte loads 53.8 us, so 18.5, VEC 13.9).
// REST: there are such tokens (a kernel of its own: the code for them costs a
// small call 0.2 us).
template <bool VEC, bool REST>
__global__ __launch_bounds__(PL_THREADS) void ppo_loss_kernel(PpoLossArgs a) {
  __shared__ float red[2][PL_THREADS / 64];
  constexpr int BLOCK = PL_THREADS * 4;
  const int t = threadIdx.x;
  const int T = a.seq_len;
  const int M = a.n_seq * T;
  const int Mv = REST ? M & ~3 : M;  // tokens taken in groups
  const float inv_n = 1.f / ((float)a.n_seq * (float)(T - a.start));
  const float lo_b = 1.f - a.eps, hi_b = 1.f + a.eps;
  // token i of this thread's group in the block from b on
  auto token = [&](int b, int i) __attribute__((always_inline)) { return VEC ? b + 4 * t + i : b + t + i * PL_THREADS; };
  auto load4 = [&](const float* p, int b) __attribute__((always_inline)) {
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (VEC) {
      if (token(b, 0) < Mv) v = *reinterpret_cast<const f32x4_t*>(p + token(b, 0));
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = token(b, i) < Mv ? p[token(b, i)] : 0.f;
    }
    return v;
  };
  auto store4 = [&](float* p, int b, const f32x4_t& v) __attribute__((always_inline)) {
    if constexpr (VEC) {
      if (token(b, 0) < Mv) *reinterpret_cast<f32x4_t*>(p + token(b, 0)) = v;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (token(b, i) < Mv) p[token(b, i)] = v[i];
    }
  };
  const int stride_pos = PL_THREADS % T;
  // f(i) for the response tokens of this thread's group
  auto each = [&](int b, auto f) __attribute__((always_inline)) {
    int pos = token(b, 0) % T;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (token(b, i) < Mv && pos >= a.start) f(i);
      if constexpr (VEC) {
        pos = pos + 1 == T ? 0 : pos + 1;
      } else {
        pos += stride_pos;
        pos = pos >= T ? pos - T : pos;
      }
    }
  };
  // both terms of the clipped surrogate
  auto terms = [&](float ln, float lo, float A, float& un, float& cl) __attribute__((always_inline)) {
    const float rho = exp_e(ln - lo);
    un = rho * A;
    cl = fminf(fmaxf(rho, lo_b), hi_b) * A;
  };
  auto d_policy = [&](float ln, float lo, float A) __attribute__((always_inline)) {
    float un, cl;
    terms(ln, lo, A, un, cl);
    return un <= cl ? -un * inv_n : 0.f;
  };

  const bool left = REST && t < M - Mv;  // this thread takes the left-over token Mv + t
  auto is_response = [&](int m) __attribute__((always_inline)) { return m % T >= a.start; };

  if (blockIdx.x >= 2) {
    const int b = (blockIdx.x - 2) * BLOCK;
    if (left && blockIdx.x == gridDim.x - 1) {
      const int m = Mv + t;
      const bool on = is_response(m);
      if (a.d_lp) a.d_lp[m] = on ? d_policy(a.lp_new[m], a.lp_old[m], a.adv[m]) : 0.f;
      if (a.d_v) a.d_v[m] = on ? (a.values[m] - a.returns[m]) * inv_n : 0.f;
    }
    if (token(b, 0) >= Mv) return;
    if (a.d_lp) {
      f32x4_t dl = {0.f, 0.f, 0.f, 0.f};
      const f32x4_t ln = load4(a.lp_new, b), lo = load4(a.lp_old, b), ad = load4(a.adv, b);
      each(b, [&](int i) __attribute__((always_inline)) { dl[i] = d_policy(ln[i], lo[i], ad[i]); });
      store4(a.d_lp, b, dl);
    }
    if (a.d_v) {
      f32x4_t dv = {0.f, 0.f, 0.f, 0.f};
      const f32x4_t va = load4(a.values, b), re = load4(a.returns, b);
      each(b, [&](int i) __attribute__((always_inline)) { dv[i] = (va[i] - re[i]) * inv_n; });
      store4(a.d_v, b, dv);
    }
    return;
  }

  float s0 = 0.f, s1 = 0.f;  // the surrogate and the clipped tokens; or the squared error
  const bool policy = blockIdx.x == 0;
  auto add = [&](float x, float y, float z) __attribute__((always_inline)) {
    if (policy) {
      float un, cl;
      terms(x, y, z, un, cl);
      s0 += un <= cl ? un : cl;
      s1 += un <= cl ? 0.f : 1.f;
    } else {
      const float d = x - y;
      s0 = fmaf(0.5f * d, d, s0);
    }
  };
  const float* const p0 = policy ? a.lp_new : a.values;
  const float* const p1 = policy ? a.lp_old : a.returns;
  for (int b0 = 0; token(b0, 0) < Mv; b0 += BLOCK * PL_BATCH) {
    f32x4_t v[3][PL_BATCH];
#pragma unroll
    for (int q = 0; q < PL_BATCH; ++q) {
      const int b = b0 + q * BLOCK;
      v[0][q] = load4(p0, b);
      v[1][q] = load4(p1, b);
      if (policy) v[2][q] = load4(a.adv, b);
    }
#pragma unroll
    for (int q = 0; q < PL_BATCH; ++q) {
      const int b = b0 + q * BLOCK;
      if (token(b, 0) >= Mv) break;
      each(b, [&](int i) __attribute__((always_inline)) { add(v[0][q][i], v[1][q][i], policy ? v[2][q][i] : 0.f); });
    }
  }
  if (left && is_response(Mv + t)) add(p0[Mv + t], p1[Mv + t], policy ? a.adv[Mv + t] : 0.f);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    s0 += __shfl_xor(s0, o);
    s1 += __shfl_xor(s1, o);
  }
  if ((t & 63) == 0) {
    red[0][t >> 6] = s0;
    red[1][t >> 6] = s1;
  }
  __syncthreads();
  if (t == 0) {
    s0 = s1 = 0.f;
    for (int i = 0; i < PL_THREADS / 64; ++i) {
      s0 += red[0][i];
      s1 += red[1][i];
    }
    if (policy) {
      a.losses[0] = -s0 * inv_n;
      a.losses[2] = s1 * inv_n;
    } else {
      a.losses[1] = s0 * inv_n;
    }
  }
}

}  // namespace

hipError_t launch_value_head(const ValueHeadArgs& a, hipStream_t stream) {
  const int rows_per_wg = VH_WAVES * VH_ROWS;
  hipLaunchKernelGGL(value_head_kernel, dim3((a.M + rows_per_wg - 1) / rows_per_wg), dim3(VH_WAVES * 64), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_ppo_loss(const PpoLossArgs& a, hipStream_t stream) {
  const void* ps[7] = {a.lp_new, a.lp_old, a.adv, a.values, a.returns, a.d_lp, a.d_v};
  bool vec = true;
  for (const void* p : ps) vec = vec && (reinterpret_cast<uintptr_t>(p) & 15) == 0;
  const int M = a.n_seq * a.seq_len;
  const int grads = a.d_lp || a.d_v ? (M + PL_THREADS * 4 - 1) / (PL_THREADS * 4) : 0;
  if (!vec)
    hipLaunchKernelGGL((ppo_loss_kernel<false, false>), dim3(2 + grads), dim3(PL_THREADS), 0, stream, a);
  else if (M % 4 != 0)
    hipLaunchKernelGGL((ppo_loss_kernel<true, true>), dim3(2 + grads), dim3(PL_THREADS), 0, stream, a);
  else
    hipLaunchKernelGGL((ppo_loss_kernel<true, false>), dim3(2 + grads), dim3(PL_THREADS), 0, stream, a);
  return hipGetLastError();
}

// Threads per sequence by its length: a thread holds at most 16 positions in
// registers (longer chunks reload them one by one: 8 x 1500 positions took 24.6
// us with one wave a sequence).
hipError_t launch_gae(const GaeArgs& a, hipStream_t stream) {
  if (a.seq_len <= 256)
    hipLaunchKernelGGL(gae_kernel<64>, dim3(a.n_seq), dim3(64), 0, stream, a);
  else if (a.seq_len <= 2048)
    hipLaunchKernelGGL(gae_kernel<256>, dim3(a.n_seq), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(gae_kernel<1024>, dim3(a.n_seq), dim3(1024), 0, stream, a);
  return hipGetLastError();
}

}  // namespace hydra
