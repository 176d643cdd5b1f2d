// survival.hpp -- the prefix-survival model of acceptance length, on the GPU.
//
// App. A.1: with q_j(x, b) the probability that drafted position j is accepted once positions
// 1..j-1 were, the expected accepted length is tau(b; x) = sum_{i<=b} prod_{j<=i} q_j(x, b).
// App. A.2: q_j(x, b) = gamma_j(x) r(b; B), r(b; B) = exp(-alpha (b - B)^2), B the drafter's
// training block size; the best block size of sample x is B*(x) = argmax over the candidates.
// App. A.3: the regret of a predicted size is R(x) = tau(B*(x)) - tau(B_hat(x)), bounded by
// L_tau |B* - B_hat| for the discrete Lipschitz constant L_tau of tau over the candidates.
//
//   survival_tau_kernel     one thread per sample: tau for every candidate, B*, the regret of
//                           B_hat and L_tau.  A workgroup stages its samples' gamma rows
//                           through LDS so the HBM reads are contiguous 16-byte vectors.
//   survival_sample_kernel  Monte Carlo of L_b(x): a wavefront (or a workgroup, where pairs are few)
//                           per (sample, candidate), one trial per lane, the next one as soon as
//                           it ends.  Uniforms come from Philox4x64-10 (Salmon
//                           et al., SC'11) keyed by (seed, 0) at counter ((i-1)/4, t, c, n), word
//                           (i-1) mod 4 for drafted position i, as the top 53 bits over 2^53, so
//                           every trial's draws are fixed by its indices alone.
//
// fp64 throughout: gamma (fp32) widens exactly, the products and sums are fp64.
#pragma once

#include "common.hpp"

namespace sdb {

constexpr int kSurvMaxCands = 64;
constexpr int kSurvMaxPos = 128;
constexpr int kSurvLdsBytes = 65536;  // staging budget of survival_tau_kernel

struct SurvivalArgs {
  const float *gamma;   // [N, P]
  const int *b_hat;     // [N] or null
  double *tau;          // [N, C]
  int *b_star;          // [N]
  double *regret;       // [N] or null
  double *lipschitz;    // [N] or null
  double *mean_len;     // [N, C]   (sampler)
  int *len_hist;        // [N, C, P + 1] or null (sampler)
  unsigned long long seed;
  int N, P, C, train_block, trials;
  double alpha;
  int cands[kSurvMaxCands];
};

__device__ __forceinline__ double retention(int b, int B, double alpha) {
  const double d = (double)(b - B);
  return exp(-alpha * d * d);
}

// One thread per sample, blockDim.x samples per workgroup (64, 128 or 256, so that the
// staged rows fit 64 KB of LDS).  Dynamic LDS: C retention factors (doubles), then the gamma
// rows, row stride P + 1 floats (odd, so a wavefront's per-thread row reads fall in distinct
// banks).
__global__ __launch_bounds__(256) void survival_tau_kernel(SurvivalArgs a) {
  extern __shared__ __attribute__((aligned(16))) double r_lds[];
  const int P = a.P, C = a.C, stride = P + 1;
  float *lds = reinterpret_cast<float *>(r_lds + kSurvMaxCands);
  const int tid = threadIdx.x, spw = blockDim.x;
  const long long n0 = (long long)blockIdx.x * spw;
  const int rows = (int)min((long long)spw, (long long)a.N - n0);
  // the workgroup's rows are one contiguous run of rows * P floats; 16-byte loads when P % 4 == 0
  const float *src = a.gamma + n0 * P;
  const int total = rows * P;
  if ((P & 3) == 0) {
    // batches of 8 vectors per thread, every load of a batch issued before any LDS store
    const float4 *s4 = reinterpret_cast<const float4 *>(src);
    const int nvec = total / 4;
    for (int v0 = tid; v0 < nvec; v0 += 8 * spw) {
      float4 x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = s4[min(v0 + k * spw, nvec - 1)];  // clamped: no per-load branch
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int v = v0 + k * spw;
        if (v < nvec) {
          const int e = 4 * v, row = e / P, col = e % P;  // P % 4 == 0: the 4 floats share a row
          float *d = lds + row * stride + col;
          d[0] = x[k].x;
          d[1] = x[k].y;
          d[2] = x[k].z;
          d[3] = x[k].w;
        }
      }
    }
  } else {
    for (int e = tid; e < total; e += spw) lds[(e / P) * stride + e % P] = src[e];
  }
  if (tid < C) r_lds[tid] = retention(a.cands[tid], a.train_block, a.alpha);
  __syncthreads();
  if (tid >= rows) return;
  const long long n = n0 + tid;
  const float *g = lds + tid * stride;
  double best_tau = -1.0, prev_tau = 0.0, lip = 0.0, hat_tau = 0.0;
  int best_b = a.cands[0], prev_b = 0;
  const int bh = a.b_hat ? a.b_hat[n] : -1;
  bool hat_found = false;
  for (int c = 0; c < C; ++c) {
    const int b = a.cands[c];
    const double r = r_lds[c];
    double prod = 1.0, t = 0.0;
    for (int i = 0; i < b; ++i) {
      prod *= (double)g[i] * r;  // prod_{j<=i+1} q_j
      t += prod;
    }
    a.tau[n * C + c] = t;
    if (t > best_tau) {  // strict: ties keep the smaller block size
      best_tau = t;
      best_b = b;
    }
    // A chord's slope over non-adjacent candidates is a weighted mean of the adjacent slopes
    // it spans, so the largest slope over all pairs is the largest over adjacent pairs.
    if (c > 0) lip = fmax(lip, fabs(t - prev_tau) / (double)(b - prev_b));
    if (b == bh) {
      hat_tau = t;
      hat_found = true;
    }
    prev_tau = t;
    prev_b = b;
  }
  a.b_star[n] = best_b;
  if (a.lipschitz) a.lipschitz[n] = lip;
  if (a.regret) a.regret[n] = hat_found ? best_tau - hat_tau : __builtin_nan("");
}

// ---- Philox4x64-10 ----
constexpr unsigned long long kPhiloxM0 = 0xD2E7470EE14C6C93ull, kPhiloxM1 = 0xCA5A826395121157ull;
constexpr unsigned long long kPhiloxW0 = 0x9E3779B97F4A7C15ull, kPhiloxW1 = 0xBB67AE8584CAA73Bull;

struct U128 {
  unsigned long long hi, lo;
};

// m * x, 64 x 64 -> 128 bits, in seven instructions: every instruction of gfx950 used here costs
// about the same issue slot, v_mad_u64_u32 (32 x 32 + 64 -> 64) included, so what counts is how
// many there are.  The middle products are summed into 65 bits, the carry left by the multiply-add
// in a scalar pair, rather than split into 32-bit halves that the next product would need
// zero-extended (seven moves and additions per product more).
__device__ __forceinline__ U128 mul_join(unsigned long long p0, unsigned long long mid, unsigned long long carry,
                                         unsigned mh, unsigned xh) {
  unsigned c;
  // s_nop: the scalar pair was just written by a VALU instruction
  asm("s_nop 1\n\tv_cndmask_b32 %0, 0, 1, %1" : "=v"(c) : "s"(carry));
  const unsigned long long m2 = ((unsigned long long)c << 32) | (mid >> 32);
  return U128{(unsigned long long)mh * xh + m2, (mid << 32) | (unsigned)p0};
}
__device__ __forceinline__ unsigned long long high_word(unsigned long long v) {
  unsigned long long r;
  asm("v_lshrrev_b64 %0, 32, %1" : "=v"(r) : "v"(v));
  return r;
}
__device__ __forceinline__ U128 mul_full(unsigned long long m, unsigned long long x) {
  const unsigned ml = (unsigned)m, mh = (unsigned)(m >> 32), xl = (unsigned)x, xh = (unsigned)(x >> 32);
  const unsigned long long p0 = (unsigned long long)ml * xl;
  const unsigned long long p1 = (unsigned long long)mh * xl + high_word(p0);  // no carry out
  unsigned long long mid, carry;
  asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(mid), "=s"(carry) : "s"(ml), "v"(xh), "v"(p1));
  return mul_join(p0, mid, carry, mh, xh);
}

__device__ __forceinline__ unsigned long long xor3(unsigned long long a, unsigned long long b, unsigned long long c) {
  const unsigned lo = __builtin_amdgcn_bitop3_b32((unsigned)a, (unsigned)b, (unsigned)c, 0x96);
  const unsigned hi = __builtin_amdgcn_bitop3_b32((unsigned)(a >> 32), (unsigned)(b >> 32), (unsigned)(c >> 32), 0x96);
  return ((unsigned long long)hi << 32) | lo;
}

// q as the threshold of a draw: with u the top 53 bits of word w over 2^53, u < q iff
// w <= draw_limit(q), for every q > 0 (u < q iff w >> 11 < ceil(q 2^53); scaling by 2^53 is exact).
__device__ __forceinline__ unsigned long long draw_limit(double q) {
  return q >= 1.0 ? ~0ull : ((unsigned long long)ceil(q * 9007199254740992.0) << 11) - 1ull;
}

// What one Philox block of four draws needs besides the trial index, per block of a (sample,
// candidate) pair.  The counter is (blk, t, c, n): the first round's products and the second
// round's second one do not depend on the trial.
struct alignas(16) DrawBlock {
  unsigned long long limit[4];  // draw_limit(q) of the block's positions
  unsigned long long c0, c1;    // words 0 and 1 after two rounds
  unsigned long long x2;        // word 2 after two rounds, xor-ed with the high half of M0 * word 0
  unsigned long long pad;
};

constexpr int kSurvWavesPerWg = 4;

// Bytes of dynamic LDS per pair: its DrawBlocks, then the histogram of L (P + 1 ints).
__host__ __device__ inline int surv_pair_lds(int P) { return ((P + 3) / 4) * (int)sizeof(DrawBlock) + ((P + 4) / 4) * 16; }

// WPP wavefronts per (sample, candidate) pair, kSurvWavesPerWg / WPP pairs per workgroup.
// Bound by the instructions of the draws' 64-bit products (about 180 per block of four draws).
// Trials end after one to b / 4 blocks of draws (1.8 on average where gamma ~ U(0.6, 0.97)), so a
// lane that is done takes the pair's next trial at once instead of waiting for the wavefront's
// longest one; the products no trial changes are tabled per block; and a draw is compared as an
// integer.  65536 samples x 5 candidates x 1024 trials: one lane per trial in turn, two full rounds
// more and fp64 compares 8617 us; with these 3462 us; with the products in seven instructions
// (mul_full) and three-input xors 3046 us.
template <int WPP>
__global__ __launch_bounds__(256) void survival_sample_kernel(SurvivalArgs a) {
  extern __shared__ __attribute__((aligned(16))) char slds[];
  __shared__ unsigned long long sh_sum[kSurvWavesPerWg];
  constexpr int NT = 64 * WPP;  // threads per pair
  const int P = a.P, C = a.C;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wp = wave % WPP, tp = wp * 64 + lane;
  DrawBlock *tab = reinterpret_cast<DrawBlock *>(slds + (wave / WPP) * surv_pair_lds(P));
  int *hist = reinterpret_cast<int *>(tab + (P + 3) / 4);
  const long long pair = (long long)blockIdx.x * (kSurvWavesPerWg / WPP) + wave / WPP;
  const bool live = pair < (long long)a.N * C;
  const long long n = live ? pair / C : 0;
  const int c = live ? (int)(pair % C) : 0;
  const int b = a.cands[c];
  const double r = retention(b, a.train_block, a.alpha);
  // key schedule of the first two rounds; the counter words of round 1 that no trial changes
  const unsigned long long k0 = a.seed, k0b = a.seed + kPhiloxW0, k1b = kPhiloxW1;
  const U128 m1 = mul_full(kPhiloxM1, (unsigned long long)c);
  // Positions from the first q <= 0 (or NaN) on accept nothing: they end the block early.
  int be = b;
  for (int i0 = 0; i0 < b && live; i0 += 64) {
    const int i = i0 + lane;
    const double q = i < b ? (double)a.gamma[n * P + i] * r : 1.0;
    const unsigned long long dead = __ballot(!(q > 0.0));
    if (dead) be = min(be, i0 + __ffsll((long long)dead) - 1);
    if (wp == 0 && i < b) tab[i >> 2].limit[i & 3] = draw_limit(q > 0.0 ? q : 1.0);
  }
  const int nblk = (be + 3) / 4;
  for (int k = tp; k < nblk && live; k += NT) {
    const U128 m0 = mul_full(kPhiloxM0, (unsigned long long)k);
    const U128 m1b = mul_full(kPhiloxM1, m0.hi ^ (unsigned long long)n);  // k1 = 0 in round 1
    tab[k].c0 = m1b.hi ^ m1.lo ^ k0b;
    tab[k].c1 = m1b.lo;
    tab[k].x2 = m0.lo ^ k1b;
  }
  for (int i = tp; i <= P; i += NT) hist[i] = 0;
  __syncthreads();
  unsigned long long sum = 0;
  if (live) {
    const unsigned long long w0 = m1.hi ^ k0;  // word 0 after round 1 is w0 ^ t
    const int t_end = (int)((long long)a.trials * (wp + 1) / WPP);
    int next = (int)((long long)a.trials * wp / WPP);  // wavefront-uniform: the next trial to hand out
    int t = next + lane, blk = 0;
    next += 64;
    bool act = t < t_end && be > 0;
    while (__any(act)) {
      const DrawBlock d = tab[blk];
      const U128 p = mul_full(kPhiloxM0, w0 ^ (unsigned long long)(unsigned)t);
      unsigned long long c0 = d.c0, c1 = d.c1, c2 = p.hi ^ d.x2, c3 = p.lo;
      unsigned long long ka = k0b, kb = k1b;
#pragma unroll
      for (int rd = 2; rd < 10; ++rd) {
        ka += kPhiloxW0;
        kb += kPhiloxW1;
        const U128 x = mul_full(kPhiloxM0, c0), y = mul_full(kPhiloxM1, c2);
        c0 = xor3(y.hi, c1, ka);
        c1 = y.lo;
        c2 = xor3(x.hi, c3, kb);
        c3 = x.lo;
      }
      const unsigned acc = (c0 <= d.limit[0] ? 1u : 0u) | (c1 <= d.limit[1] ? 2u : 0u) | (c2 <= d.limit[2] ? 4u : 0u) |
                           (c3 <= d.limit[3] ? 8u : 0u);
      const int lead = __ffs((int)~acc) - 1;  // leading acceptances of the block, 0..4
      const bool end = act && (lead < 4 || 4 * blk + 4 >= be);
      const unsigned long long em = __ballot(end);
      if (end) {
        const int L = min(4 * blk + lead, be);
        sum += (unsigned)L;
        if (a.len_hist) atomicAdd(&hist[L], 1);
        t = next + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(em >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)em, 0u));
        blk = 0;
        act = t < t_end;
      } else {
        blk = act ? blk + 1 : 0;
      }
      next += __popcll(em);
    }
    if (be == 0 && tp == 0 && a.len_hist) hist[0] = a.trials;
  }
  // sum of the lengths (exact integers)
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if (WPP > 1 && lane == 0) sh_sum[wave] = sum;
  __syncthreads();
  if (!live) return;
  if constexpr (WPP > 1) {
    sum = 0;
#pragma unroll
    for (int w = 0; w < WPP; ++w) sum += sh_sum[(wave / WPP) * WPP + w];
  }
  if (tp == 0) a.mean_len[pair] = (double)sum / (double)a.trials;
  if (a.len_hist) {
    int *out = a.len_hist + pair * (P + 1);
    for (int i = tp; i <= P; i += NT) out[i] = hist[i];
  }
}

}  // namespace sdb
