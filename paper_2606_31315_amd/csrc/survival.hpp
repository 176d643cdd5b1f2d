// survival.hpp -- the prefix-survival model of acceptance length, on the GPU.
//
// App. A.1: with q_j(x, b) the probability that drafted position j is accepted once positions
// 1..j-1 were, the expected accepted length is tau(b; x) = sum_{i<=b} prod_{j<=i} q_j(x, b).
// App. A.2: q_j(x, b) = gamma_j(x) r(b; B), r(b; B) = exp(-alpha (b - B)^2), B the drafter's
// training block size; the best block size of sample x is B*(x) = argmax over the candidates.
// App. A.3: the regret of a predicted size is R(x) = tau(B*(x)) - tau(B_hat(x)), bounded by
// L_tau |B* - B_hat| for the discrete Lipschitz constant L_tau of tau over the candidates.
//
//   survival_tau_kernel     one lane per sample: tau for every candidate, B*, the regret of
//                           B_hat and L_tau.  A wavefront stages its samples' gamma rows and
//                           their tau through LDS so the HBM accesses are contiguous.
//   survival_sample_kernel  Monte Carlo of L_b(x): a wavefront (or a workgroup, where pairs are few)
//                           per (sample, candidate), one trial per lane, the next one as soon as
//                           it ends.  Uniforms come from Philox4x64-10 (Salmon
//                           et al., SC'11) keyed by (seed, 0) at counter ((i-1)/4, t, c, n), word
//                           (i-1) mod 4 for drafted position i, as the top 53 bits over 2^53, so
//                           every trial's draws are fixed by its indices alone.
//
// fp64 throughout: gamma (fp32) widens exactly, the products and sums are fp64.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace sdb {

constexpr int kSurvMaxCands = 64;
constexpr int kSurvMaxPos = 128;

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
  int load_nt;          // tau: gamma is read past the caches
  double alpha;
  int cands[kSurvMaxCands];
};

__device__ __forceinline__ double retention(int b, int B, double alpha) {
  const double d = (double)(b - B);
  return exp(-alpha * d * d);
}

// One wavefront per workgroup, one sample per lane: no barrier joins one wavefront's loads to
// another's arithmetic, and the registers hold 16 of them on a CU.  The samples' gamma rows
// are one contiguous run, read as 16-byte vectors (every load of 8 KB in flight at once) into LDS rows of
// odd stride, so that the lanes' row reads fall in distinct banks.  Up to kTauCands candidates
// are carried through one pass over the row, as many independent chains of products as there are;
// their tau go out through LDS, so that the stores are contiguous.
// 2^20 samples x 32 positions x 5 candidates (201 MB): 256 threads with a barrier, one candidate's
// chain at a time and strided stores 47.1 us; this 39.6 us, 5.1 TB/s, the rate of a copy.  On the way
// 46.1 us with every position tested against each candidate's size past the first, 42.5 with a
// division only where candidates are not neighbours and non-temporal accesses, 39.6 with the positions
// between two sizes run for the remaining candidates alone.
// Up to kTauStaged candidates are staged and stored together: a pass's part of a row is stored past the
// caches in pieces of lines otherwise (2^19 samples x 32 positions, 9 / 11 candidates: pass by pass 41.4 /
// 52.0 us, together 32.5 / 36.2; the 256-thread kernel 42.4 / 51.3).  Beyond, the passes are stored
// through the caches unless their parts are whole 64-byte runs (17 candidates 85.4 / 57.2 us; 24 candidates
// x 2^18 x 64 positions 52.9 past the caches, 54.4 through them).
constexpr int kTauCands = 8;
constexpr int kTauStaged = 16;

// Whether gamma is read past the caches: not where a user's next call may find it in the 256 MB Infinity
// Cache and there are so few candidates that the read is most of the time.  us from memory / from the
// cache, past the caches and through them: 2^20 x 20 positions x 3 candidates 29.3 / 28.8 and 30.5 / 25.5 (the
// 256-thread kernel 31.6 / 26.9), 2^20 x 32 x 3 35.3 / 35.3 and 37.5 / 35.9 (40.9 / 39.5), 2^19 x 32 x 5
// 22.5 / 21.8 and 24.0 / 20.5 (28.6 / 25.0).
__host__ inline bool tau_load_nt(int N, int P, int C) { return C > 3 || 4LL * N * P >= (1LL << 27); }

// Candidates whose tau are staged together: all of them up to kTauStaged, else those of a pass.
__host__ __device__ inline int tau_staged(int C) { return C <= kTauStaged ? C : kTauCands; }

// Dynamic LDS: the gamma rows, and the staged tau (where one pass takes every candidate, in
// their place).
__host__ __device__ inline int tau_rows_bytes(int P) { return 64 * ((P + 1) | 1) * (int)sizeof(float); }
__host__ __device__ inline int tau_lds(int P, int C) {
  const int rows = (tau_rows_bytes(P) + 15) & ~15, out = 64 * tau_staged(C) * (int)sizeof(double);
  return C <= kTauCands ? (rows > out ? rows : out) : rows + out;
}

struct TauState {
  double best, prev, lip, hat;
  int best_b, prev_b;
  bool found;
};

// Candidates c0 .. c0 + NC - 1 of the lane's sample (row g): tau into t, r their retention factors.
template <int NC>
__device__ __forceinline__ void tau_pass(const SurvivalArgs &a, const float *g, int c0, double r_lane, int bh,
                                         TauState &st, double (&t)[kTauCands]) {
  double r[NC], prod[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    r[c] = readlane_d(r_lane, c0 + c);
    prod[c] = 1.0;
    t[c] = 0.0;
  }
  // prod_{j<=i+1} q_j of every candidate; sizes ascend, so candidate c - 1 is done where c goes on
  int i = 0;
  auto steps = [&](auto from_c, auto count_c) {  // positions i .. of candidates from_c and up
    constexpr int F = decltype(from_c)::value, K = decltype(count_c)::value;
    float x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = g[i + k];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double gd = (double)x[k];
#pragma unroll
      for (int c = F; c < NC; ++c) {
        prod[c] *= gd * r[c];
        t[c] += prod[c];
      }
    }
    i += K;
  };
  auto runs = [&](auto from_c) {
    const int n = a.cands[c0 + decltype(from_c)::value];
    while (i + 4 <= n) steps(from_c, std::integral_constant<int, 4>{});
    while (i < n) steps(from_c, std::integral_constant<int, 1>{});
  };
  runs(std::integral_constant<int, 0>{});
  if constexpr (NC > 1) runs(std::integral_constant<int, (NC > 1 ? 1 : 0)>{});
  if constexpr (NC > 2) runs(std::integral_constant<int, (NC > 2 ? 2 : 0)>{});
  if constexpr (NC > 3) runs(std::integral_constant<int, (NC > 3 ? 3 : 0)>{});
  if constexpr (NC > 4) runs(std::integral_constant<int, (NC > 4 ? 4 : 0)>{});
  if constexpr (NC > 5) runs(std::integral_constant<int, (NC > 5 ? 5 : 0)>{});
  if constexpr (NC > 6) runs(std::integral_constant<int, (NC > 6 ? 6 : 0)>{});
  if constexpr (NC > 7) runs(std::integral_constant<int, (NC > 7 ? 7 : 0)>{});
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int b = a.cands[c0 + c];
    if (t[c] > st.best) {  // strict: ties keep the smaller block size
      st.best = t[c];
      st.best_b = b;
    }
    // A chord's slope over non-adjacent candidates is a weighted mean of the adjacent slopes
    // it spans, so the largest slope over all pairs is the largest over adjacent pairs.
    if (c0 + c > 0) {
      const double d = fabs(t[c] - st.prev);
      const int gap = b - st.prev_b;  // uniform; a division only where there is one to make
      st.lip = fmax(st.lip, gap == 1 ? d : d / (double)gap);
    }
    if (b == bh) {
      st.hat = t[c];
      st.found = true;
    }
    st.prev = t[c];
    st.prev_b = b;
  }
}

__global__ __launch_bounds__(64) void survival_tau_kernel(SurvivalArgs a) {
  extern __shared__ __attribute__((aligned(16))) char tau_smem[];
  const int P = a.P, C = a.C, stride = (P + 1) | 1;
  float *lds = reinterpret_cast<float *>(tau_smem);
  double *out = reinterpret_cast<double *>(tau_smem + (C <= kTauCands ? 0 : (tau_rows_bytes(P) + 15) & ~15));
  const int lane = threadIdx.x;
  const long long n0 = (long long)blockIdx.x * 64;
  const int rows = (int)min(64LL, (long long)a.N - n0);
  const int bh = (a.b_hat && lane < rows) ? a.b_hat[n0 + lane] : -1;
  // the rows are one contiguous run of rows * P floats from a multiple of 64 P on, so 16-byte aligned
  // whatever P is; element 4 v of the run is (row, col), and 64 vectors on dr rows and dc columns further
  const float *src = a.gamma + n0 * P;
  const int total = rows * P, nvec = total / 4;
  const int dr = 256 / P, dc = 256 - dr * P;
  int row = (4 * lane) / P, col = 4 * lane - row * P;
  auto stage = [&](auto whole_c, auto nt_c) {  // whole_c: P % 4 == 0, a vector's floats share a row
    constexpr bool WHOLE = decltype(whole_c)::value, NT = decltype(nt_c)::value;
    const f32x4 *s4 = reinterpret_cast<const f32x4 *>(src);
    for (int v0 = lane; v0 < nvec; v0 += 8 * 64) {
      f32x4 x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {  // clamped: no per-load branch
        const f32x4 *p = s4 + min(v0 + k * 64, nvec - 1);
        x[k] = NT ? __builtin_nontemporal_load(p) : *p;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (v0 + k * 64 < nvec) {
          int r = row, c = col;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            lds[r * stride + c] = x[k][e];
            ++c;
            if (!WHOLE && c == P) {
              c = 0;
              ++r;
            }
          }
        }
        row += dr;
        col += dc;
        if (col >= P) {
          col -= P;
          ++row;
        }
      }
    }
  };
  using std::false_type;
  using std::true_type;
  if ((P & 3) == 0) {
    if (a.load_nt) stage(true_type{}, true_type{});
    else stage(true_type{}, false_type{});
  } else {
    if (a.load_nt) stage(false_type{}, true_type{});
    else stage(false_type{}, false_type{});
    const int e = 4 * nvec + lane;
    if (e < total) lds[(e / P) * stride + e % P] = src[e];
  }
  const double r_lane = retention(a.cands[min(lane, C - 1)], a.train_block, a.alpha);
  __syncthreads();
  const float *g = lds + min(lane, rows - 1) * stride;
  TauState st{-1.0, 0.0, 0.0, 0.0, a.cands[0], 0, false};
  for (int c0 = 0; c0 < C; c0 += kTauCands) {
    const int nc = min(C - c0, kTauCands);
    double t[kTauCands];
    switch (nc) {  // uniform
      case 1: tau_pass<1>(a, g, c0, r_lane, bh, st, t); break;
      case 2: tau_pass<2>(a, g, c0, r_lane, bh, st, t); break;
      case 3: tau_pass<3>(a, g, c0, r_lane, bh, st, t); break;
      case 4: tau_pass<4>(a, g, c0, r_lane, bh, st, t); break;
      case 5: tau_pass<5>(a, g, c0, r_lane, bh, st, t); break;
      case 6: tau_pass<6>(a, g, c0, r_lane, bh, st, t); break;
      case 7: tau_pass<7>(a, g, c0, r_lane, bh, st, t); break;
      default: tau_pass<8>(a, g, c0, r_lane, bh, st, t); break;
    }
    __syncthreads();  // the rows are read (their place is reused where this is the only pass)
    const bool all = C <= kTauStaged;
    const int ow = all ? C : nc, oc = all ? c0 : 0;  // the staged row's width, this pass's place in it
#pragma unroll
    for (int c = 0; c < kTauCands; ++c)
      if (c < nc) out[lane * ow + oc + c] = t[c];
    if (all && c0 + nc < C) continue;
    __syncthreads();
    if (all) {
      for (int f = lane; f < rows * C; f += 64) __builtin_nontemporal_store(out[f], a.tau + n0 * C + f);
    } else if ((C & 7) == 0) {  // whole 64-byte runs
      for (int f = lane; f < rows * kTauCands; f += 64)
        __builtin_nontemporal_store(out[f], a.tau + (n0 + f / kTauCands) * C + c0 + f % kTauCands);
    } else {
      for (int f = lane; f < rows * nc; f += 64) a.tau[(n0 + f / nc) * C + c0 + f % nc] = out[f];
    }
    __syncthreads();  // before the next pass writes out
  }
  if (lane >= rows) return;
  const long long n = n0 + lane;
  a.b_star[n] = st.best_b;
  if (a.lipschitz) a.lipschitz[n] = st.lip;
  if (a.regret) a.regret[n] = st.found ? st.best - st.hat : __builtin_nan("");
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
