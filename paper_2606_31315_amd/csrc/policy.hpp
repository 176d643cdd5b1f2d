// policy.hpp -- the block-size policy on the GPU, run once per prompt after prefill.
//
// Sec. 2.3-2.4: the predictive distribution of the prompt's last token, p = softmax(z) over the
// vocabulary, is the input of a small MLP (two hidden layers of width 2048 by default, Sec. 3.1)
// whose outputs score the 2k+1 candidate block sizes {B-k, ..., B+k}; the block size is the
// argmax of the scores (Eq. 9).  Here:
//   h1 = relu(W1 p + b1),  h2 = relu(W2 h1 + b2),  o = W3 h2 + b3,  B_hat = B - k + argmax o.
//
// Kernels (gfx950).  The W1 product dominates: W1 is [hidden, V] bf16 (622 MB for Qwen3's
// vocabulary), read once, so the policy is HBM-bound.
//   policy_first_kernel   W1 p on matrix cores, up to 16 prompts per pass, split over vocabulary
//                         chunks; makes p's terms on the fly.  policy_merge_kernel combines the
//                         chunks and applies softmax's normaliser, the bias and the activation.
//   policy_second_kernel  relu(W2 h1 + b2) on matrix cores.
//   policy_head_kernel    one workgroup per prompt, one wavefront per candidate: the 2k+1 scores
//                         and their argmax.
// Where those are slower or do not apply (few prompts over short rows of W1, or rows that are not whole
// cache lines: policy_plan; a workspace without room for the chunk partials):
//   policy_stats_kernel   grid (prompt, chunk): (max, sum exp(z - max)) of one vocabulary chunk,
//                         one online pass per thread.
//   policy_dense_kernel   y = act(W x + b) for every prompt: a workgroup owns R rows of W and
//                         streams them once with 16-byte loads, all prompts' FMAs per element.
//                         For the first layer x is p = softmax(z), made on the fly from the
//                         logits and the merged chunk records (p is never written out; the
//                         logits stay L2-resident: 2 or 4 bytes per element per prompt).
#pragma once

#include "common.hpp"

namespace sdb {

constexpr int kPolicyChunks = 64;   // vocabulary chunks of the softmax passes
constexpr int kPolicyMaxPrompts = 8;  // prompts per dense pass (accumulators per thread)
constexpr int kDenseRows = 2;       // rows of W per dense workgroup

struct PolicyArgs {
  const void *logits;   // [P, V] bf16 or fp32
  float2 *stats;        // [P, kPolicyChunks] (max, sum exp(z - max))
  int P, V, logits_bf16;
};

constexpr float kLog2e = 1.4426950408889634f;

template <bool BF16>
__device__ __forceinline__ float ld_logit(const void *base, long long i) {
  if constexpr (BF16) return __uint_as_float(((uint32_t)reinterpret_cast<const uint16_t *>(base)[i]) << 16);
  else return reinterpret_cast<const float *>(base)[i];
}

__device__ __forceinline__ void chunk_range(int V, int c, int &e0, int &e1) {
  e0 = (int)((long long)V * c / kPolicyChunks);
  e1 = (int)((long long)V * (c + 1) / kPolicyChunks);
}

template <bool BF16>
__global__ __launch_bounds__(256) void policy_stats_kernel(PolicyArgs a) {
  __shared__ float sh_m[4], sh_s[4];
  const int pr = blockIdx.x / kPolicyChunks, c = blockIdx.x % kPolicyChunks;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int e0, e1;
  chunk_range(a.V, c, e0, e1);
  const long long row = (long long)pr * a.V;
  // online (max, sum) per thread: one rescale when the maximum moves
  float m = -INFINITY, s = 0.f;
  for (int e = e0 + tid; e < e1; e += 256) {
    const float z = ld_logit<BF16>(a.logits, row + e);
    if (z > m) {
      s = (m == -INFINITY) ? 0.f : s * fast_exp2((m - z) * kLog2e);
      m = z;
    }
    if (m != -INFINITY) s += fast_exp2((z - m) * kLog2e);  // a -inf logit adds 0
  }
  const float wm = wave_max_f(m);
  float ws = (m == -INFINITY) ? 0.f : s * fast_exp2((m - wm) * kLog2e);
  ws = wave_sum_f(ws);
  if (lane == 0) {
    sh_m[wave] = wm;
    sh_s[wave] = ws;
  }
  __syncthreads();
  if (tid == 0) {
    const float M = fmaxf(fmaxf(sh_m[0], sh_m[1]), fmaxf(sh_m[2], sh_m[3]));
    float S = 0.f;
    for (int w = 0; w < 4; ++w)
      if (sh_m[w] != -INFINITY) S += sh_s[w] * fast_exp2((sh_m[w] - M) * kLog2e);
    a.stats[blockIdx.x] = float2{M, S};
  }
}

// y[p, n] = act(sum_i W[n, i] x[p, i] + b[n]) for rows n of this workgroup and every prompt p.
// W [rows, cols] bf16 row-major (cols % 8 == 0), y [P, rows] fp32.  x [P, cols] is
//   XM = 0: fp32 activations;
//   XM = 1, 2: bf16 (1) or fp32 (2) logits z, and the layer's input is p = softmax(z), made here
//   from z and the prompt's kPolicyChunks chunk records: p_i = 2^((z_i - M) log2 e) / Z.
struct DenseArgs {
  const uint16_t *w;
  const void *x;
  const float *b;
  float *y;
  int rows, cols, P;
  const float2 *stats;  // XM != 0: [P, kPolicyChunks]
};

// U vectors per row are loaded before any is used (clamped indices, no per-load branch), so a
// thread keeps U * (R + NP * (1 or 2)) 16-byte loads in flight.
template <int NP, bool RELU, int XM>
__global__ __launch_bounds__(256) void policy_dense_kernel(DenseArgs a) {
  constexpr int R = kDenseRows;
  constexpr int U = NP <= 2 ? 4 : (NP <= 4 ? 2 : 1);
  constexpr int XV = (XM == 1) ? 1 : 2;  // 16-byte x loads per 8 elements
  static_assert(kPolicyChunks == kWave, "one chunk record per lane");
  __shared__ float sh[4][R][NP];
  __shared__ float sh_norm[2][NP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = blockIdx.x * R;
  const int nv = a.cols / 8;  // 16-byte vectors of bf16 per row
  float mx[NP], inv[NP];
  if constexpr (XM != 0) {
    // merge the prompt's chunk records: M = max of the chunk maxima, Z = sum of the rescaled sums
    if (wave == 0) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const float2 r = a.stats[(size_t)min(p, a.P - 1) * kPolicyChunks + lane];
        const float M = wave_max_f(r.x);
        const double z = wave_sum_d(r.x != -INFINITY ? (double)r.y * (double)fast_exp2((r.x - M) * kLog2e) : 0.0);
        if (lane == 0) {
          sh_norm[0][p] = M;
          sh_norm[1][p] = (float)(1.0 / z);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      mx[p] = sh_norm[0][p];
      inv[p] = sh_norm[1][p];
    }
  }
  float acc[R][NP];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int p = 0; p < NP; ++p) acc[r][p] = 0.f;
  const u32x4 *wr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) wr[r] = reinterpret_cast<const u32x4 *>(a.w + (size_t)min(n0 + r, a.rows - 1) * a.cols);
  const u32x4 *xr[NP];
  const size_t xrow = (size_t)a.cols * (XM == 1 ? 2 : 4) / 16;  // 16-byte vectors per x row
#pragma unroll
  for (int p = 0; p < NP; ++p) xr[p] = reinterpret_cast<const u32x4 *>(a.x) + (size_t)min(p, a.P - 1) * xrow;
  for (int v0 = tid; v0 < nv; v0 += 256 * U) {
    u32x4 wv[U][R];
    u32x4 xv[U][NP][XV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = min(v0 + 256 * u, nv - 1);
#pragma unroll
      for (int r = 0; r < R; ++r) wv[u][r] = wr[r][v];
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int k = 0; k < XV; ++k) xv[u][p][k] = xr[p][XV * v + k];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (v0 + 256 * u >= nv) break;
      float x[NP][8];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if constexpr (XM == 1) {
          const u32x4 z = xv[u][p][0];
          const float zz[8] = {bf16_lo(z.x), bf16_hi(z.x), bf16_lo(z.y), bf16_hi(z.y),
                               bf16_lo(z.z), bf16_hi(z.z), bf16_lo(z.w), bf16_hi(z.w)};
#pragma unroll
          for (int e = 0; e < 8; ++e) x[p][e] = fast_exp2((zz[e] - mx[p]) * kLog2e) * inv[p];
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const u32x4 h = xv[u][p][e >> 2];
            const uint32_t bits = (e & 3) == 0 ? h.x : (e & 3) == 1 ? h.y : (e & 3) == 2 ? h.z : h.w;
            const float f = __uint_as_float(bits);
            x[p][e] = (XM == 2) ? fast_exp2((f - mx[p]) * kLog2e) * inv[p] : f;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float w[8] = {bf16_lo(wv[u][r].x), bf16_hi(wv[u][r].x), bf16_lo(wv[u][r].y), bf16_hi(wv[u][r].y),
                            bf16_lo(wv[u][r].z), bf16_hi(wv[u][r].z), bf16_lo(wv[u][r].w), bf16_hi(wv[u][r].w)};
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[r][p] = fmaf(w[e], x[p][e], acc[r][p]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const float s = wave_sum_f(acc[r][p]);
      if (lane == 0) sh[wave][r][p] = s;
    }
  __syncthreads();
  if (tid < R * NP) {
    const int r = tid / NP, p = tid % NP;
    const int n = n0 + r;
    if (n < a.rows && p < a.P) {
      float y = (sh[0][r][p] + sh[1][r][p]) + (sh[2][r][p] + sh[3][r][p]) + a.b[n];
      if (RELU) y = fmaxf(y, 0.f);
      a.y[(size_t)p * a.rows + n] = y;
    }
  }
}

// ---- the layers on matrix cores: up to 16 prompts per pass over W1 ----
//
// The dense pass above makes every prompt's p again in each workgroup and multiplies on the vector
// units, which falls behind the memory from two prompts on.  Here the first layer runs on
// v_mfma_f32_16x16x32_bf16 with one column per prompt: W1 is bf16, and an fp32 term is the exact sum
// of three bf16 numbers, so three products per weight give the fp32 product and the sums stay fp32.
//   Grid (chunk of the vocabulary, 512 rows of W1), chunk fastest: where the chunks are a multiple of 8
//   a chunk's workgroups share an XCD, whose L2 holds the chunk's logits; elsewhere several XCDs read them.  A workgroup's 8 wavefronts own 64 rows each
//   and make the terms 2^((z - m) log2 e) of a 64-element tile together, against the chunk's
//   maximum m (one pass over the chunk's logits while the first tiles are on their way).  No softmax
//   pass comes first: the workgroup files its partial sums with (m, sum of the terms), and
//   policy_merge_kernel combines the chunks.
//   W1 and the logits come by load-to-LDS transfers into a ring of two stages, each wavefront's part
//   its own; a tile is read into registers at once, which frees its stage for the tile after next.
//   One barrier per tile, for the terms.
// Bound by HBM: W1 of 2048 x 151936 (622 MB) in 94 us, 6.6 TB/s, for 1 to 16 prompts (the dense
// kernel 105 us for one prompt, 299 us for eight).  Measured on the way (eight prompts): the terms
// made by each wavefront for its own rows and fp32 products (v_mfma_f32_16x16x4_f32) 127 us with 64
// rows per wavefront and 147 us with 32: the terms' arithmetic, not the memory, set the pace.
constexpr int kFirstWaves = 8;
constexpr int kFirstRows = 64 * kFirstWaves;  // rows of W1 per workgroup
constexpr int kFirstKT = 64;                  // vocabulary elements per tile
constexpr int kFirstPrompts = 16;             // prompts per pass
constexpr int kFirstMaxChunks = 256;

struct FirstArgs {
  const uint16_t *w;   // [H, V]
  const void *logits;  // [P, V] of this pass
  float *part;         // [nch, P, H] sums of 2^((z - m) log2 e) W1 over a chunk
  float2 *stats;       // [nch, P] (m, sum of the terms)
  int H, V, P, nch;
};

__device__ __forceinline__ float bf16_at(const v4u32 &v, int e) {
  const uint32_t w = v[e >> 1];
  return (e & 1) ? bf16_hi(w) : bf16_lo(w);
}

// Two terms as three bf16 pairs whose sums they are, exactly: each piece takes the next 8 bits.
__device__ __forceinline__ void split3(float x, float y, uint32_t (&pc)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    pc[i] = cvt_pk_bf16(x, y);
    x -= bf16_lo(pc[i]);
    y -= bf16_hi(pc[i]);
  }
}

template <bool BF16>
__global__ __launch_bounds__(64 * kFirstWaves) void policy_first_kernel(FirstArgs a) {
  constexpr int WT = 64 * kFirstKT * 2;              // bytes of W1 per wavefront and tile
  constexpr int ZT = BF16 ? 256 : 1024;              // logits: 8 elements of 16 prompts (fp32: twice over)
  constexpr int STAGE = kFirstWaves * (WT + ZT);
  constexpr int BT = 3 * 2048;                       // the tile's terms: [piece][step][kgrp][prompt] 16 bytes
  constexpr int ZE = BF16 ? 8 : 4, ZB = BF16 ? 2 : 4;  // logits per 16-byte vector, bytes per logit
  __shared__ __attribute__((aligned(1024))) char lds[2 * STAGE + 2 * BT];
  __shared__ float sh_m[16];
  __shared__ double sh_s[kFirstWaves][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kgrp = lane >> 4;
  const int chunk = blockIdx.x % a.nch, n0 = (blockIdx.x / a.nch) * kFirstRows + wave * 64;
  char SDB_LDS *ring = (char SDB_LDS *)(SDB_LDS void *)lds;
  char SDB_LDS *wring = ring + wave * WT;
  char SDB_LDS *zring = ring + kFirstWaves * WT + wave * ZT;
  const int nt = (a.V + kFirstKT - 1) / kFirstKT;
  const int t0 = (int)((long long)nt * chunk / a.nch), t1 = (int)((long long)nt * (chunk + 1) / a.nch);

  // ---- load-to-LDS sources.  A transfer writes LDS in lane order: rows of 8 vectors, each lane
  // fetching the vector that the XOR swizzle (vector ^ row mod 8) puts at its place.
  const char *wsrc[8];
  const int wk = ((lane & 7) ^ (lane >> 3)) * 8;  // element of the lane's vector within the tile
#pragma unroll
  for (int q = 0; q < 8; ++q)
    wsrc[q] = reinterpret_cast<const char *>(a.w) + (size_t)min(n0 + q * 8 + (lane >> 3), a.H - 1) * a.V * 2;
  // this wavefront's 8 logits of every prompt: bf16 [prompt][4 words], fp32 [prompt][2 vectors]
  const int zrow = BF16 ? lane >> 2 : (lane & 31) >> 1;
  const int zk = wave * 8 + (BF16 ? (lane & 3) * 2 : (lane & 1) * 4);
  const char *zsrc = reinterpret_cast<const char *>(a.logits) + (size_t)min(zrow, a.P - 1) * a.V * ZB;
  const bool lines = a.V % 64 == 0;
  auto issue = [&](int t) {
    const int so = ((t - t0) & 1) * STAGE, k0 = t * kFirstKT;
    // vectors past the row's end re-read its last one; their terms are 0
    // rows of whole 128-byte lines are read once, non-temporally; otherwise a tile's 128 bytes of a
    // row straddle two lines, and the next tile finds the second in L2
    const size_t ko = (size_t)min(k0 + wk, a.V - 8) * 2;
    if (lines) {
#pragma unroll
      for (int q = 0; q < 8; ++q)
        __builtin_amdgcn_global_load_lds((const void *)(wsrc[q] + ko), (SDB_LDS void *)(wring + so + q * 1024), 16, 0, kLoadNT);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q)
        __builtin_amdgcn_global_load_lds((const void *)(wsrc[q] + ko), (SDB_LDS void *)(wring + so + q * 1024), 16, 0, 0);
    }
    if constexpr (BF16)
      __builtin_amdgcn_global_load_lds((const void *)(zsrc + (size_t)min(k0 + zk, a.V - 2) * ZB), (SDB_LDS void *)(zring + so), 4, 0, 0);
    else
      __builtin_amdgcn_global_load_lds((const void *)(zsrc + (size_t)min(k0 + zk, a.V - 4) * ZB), (SDB_LDS void *)(zring + so), 16, 0, 0);
  };
  if (t0 < t1) issue(t0);
  if (t0 + 1 < t1) issue(t0 + 1);

  // ---- the chunk's maximum per prompt, wavefront w for prompts w and w + 8 ----
  {
    const int vb = t0 * kFirstKT / ZE, ve = min(t1 * kFirstKT, a.V) / ZE;  // vectors of the chunk (V % 8 == 0)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int pr = wave + 8 * h;
      float m = -INFINITY;
      if (pr < a.P) {  // uniform
        const v4u32 *row = reinterpret_cast<const v4u32 *>(reinterpret_cast<const char *>(a.logits) + (size_t)pr * a.V * ZB);
        for (int v0 = vb + lane; v0 < ve; v0 += 64 * 5) {
          v4u32 x[5];
#pragma unroll
          for (int u = 0; u < 5; ++u) x[u] = row[min(v0 + 64 * u, ve - 1)];  // clamped: no per-load branch
#pragma unroll
          for (int u = 0; u < 5; ++u)
#pragma unroll
            for (int e = 0; e < ZE; ++e) m = fmaxf(m, BF16 ? bf16_at(x[u], e) : __uint_as_float(x[u][e & 3]));
        }
      }
      m = wave_max_f(m);
      if (lane == 0) sh_m[pr] = m;
    }
  }
  __syncthreads();
  const int pr = min(l16, a.P - 1);  // columns past P repeat the last prompt
  const float m = sh_m[pr];
  const float mu = (m == -INFINITY) ? 0.f : m;

  // ---- LDS addresses within a stage: W1 vector (step st, 16-row tile j) = row j*16 + l16 ----
  const unsigned lbase = (unsigned)(uintptr_t)ring;
  const unsigned wa0 = lbase + wave * WT + l16 * 128 + ((kgrp ^ (l16 & 7)) << 4);
  const unsigned wa1 = lbase + wave * WT + l16 * 128 + (((4 + kgrp) ^ (l16 & 7)) << 4);
  const unsigned za = lbase + kFirstWaves * WT + wave * ZT + l16 * (BF16 ? 16 : 32) + kgrp * (BF16 ? 4 : 8);
  // terms: this lane makes elements wave*8 + kgrp*2, +1 of the tile for prompt l16
  const unsigned bw = lbase + 2 * STAGE + (wave >> 2) * 1024 + ((wave & 3) * 16 + l16) * 16 + kgrp * 4;
  const unsigned br = lbase + 2 * STAGE + (kgrp * 16 + l16) * 16;

  // sums of the leading pieces' products by step, and of the other two pieces' (2^-8 of them)
  f32x4 acc[3][4];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  double sum = 0.0;
  for (int t = t0; t < t1; ++t) {
    const unsigned so = ((t - t0) & 1) * STAGE, bo = ((t - t0) & 1) * BT;
    if (t + 1 < t1) wait_vmcnt<9>();
    else wait_vmcnt<0>();
    // the tile's terms
    uint32_t za0;
    float x, y;
    if constexpr (BF16) {
      asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(za0) : "v"(za + so) : "memory");
      x = bf16_lo(za0);
      y = bf16_hi(za0);
    } else {
      unsigned long long zz;
      asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(zz) : "v"(za + so) : "memory");
      x = __uint_as_float((uint32_t)zz);
      y = __uint_as_float((uint32_t)(zz >> 32));
    }
    const bool in = t * kFirstKT + wave * 8 < a.V;  // uniform: whole vectors of 8
    // the difference first: folded into one fma, the rounding of m log2 e would differ from chunk to chunk
    x = in ? fast_exp2((x - mu) * kLog2e) : 0.f;
    y = in ? fast_exp2((y - mu) * kLog2e) : 0.f;
    sum += (double)(x + y);
    uint32_t pc[3];
    split3(x, y, pc);
    asm volatile("ds_write_b32 %0, %1\n\tds_write_b32 %0, %2 offset:2048\n\tds_write_b32 %0, %3 offset:4096\n\t"
                 "s_waitcnt lgkmcnt(0)\n\ts_barrier" ::"v"(bw + bo), "v"(pc[0]), "v"(pc[1]), "v"(pc[2]) : "memory");
    // the operands: the tile's W1 rows and every wavefront's terms, waited for in the same block
    bf16x8 w[2][4], b[3][2];
    asm volatile("ds_read_b128 %0, %14\n\tds_read_b128 %1, %14 offset:2048\n\t"
                 "ds_read_b128 %2, %14 offset:4096\n\tds_read_b128 %3, %14 offset:6144\n\t"
                 "ds_read_b128 %4, %15\n\tds_read_b128 %5, %15 offset:2048\n\t"
                 "ds_read_b128 %6, %15 offset:4096\n\tds_read_b128 %7, %15 offset:6144\n\t"
                 "ds_read_b128 %8, %16\n\tds_read_b128 %9, %16 offset:1024\n\t"
                 "ds_read_b128 %10, %16 offset:2048\n\tds_read_b128 %11, %16 offset:3072\n\t"
                 "ds_read_b128 %12, %16 offset:4096\n\tds_read_b128 %13, %16 offset:5120\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[0][2]), "=&v"(w[0][3]), "=&v"(w[1][0]), "=&v"(w[1][1]),
                   "=&v"(w[1][2]), "=&v"(w[1][3]), "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[1][0]), "=&v"(b[1][1]),
                   "=&v"(b[2][0]), "=&v"(b[2][1])
                 : "v"(wa0 + so), "v"(wa1 + so), "v"(br + bo)
                 : "memory");
    if (t + 2 < t1) issue(t + 2);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4 &c = acc[i == 0 ? st : 2][j];
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[st][j], b[i][st], c, 0, 0, 0);
        }
  }

  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  if (lane < 16) sh_s[wave][l16] = sum;
  __syncthreads();
  if (l16 < a.P) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + j * 16 + kgrp * 4;  // H % 8 == 0: four rows at once
      if (n < a.H)
        *reinterpret_cast<f32x4 *>(a.part + ((size_t)chunk * a.P + l16) * a.H + n) = (acc[0][j] + acc[1][j]) + acc[2][j];
    }
    if (n0 == 0 && lane < 16) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kFirstWaves; ++w) s += sh_s[w][l16];
      a.stats[(size_t)chunk * a.P + l16] = float2{m, (float)s};
    }
  }
}

// h1 = relu(W1 p + b1) from the chunk partials.  Grid (prompt, 64 rows): the four wavefronts take the
// chunks in turn, a row per lane.  An infinite weight times a piece that is 0 is NaN above though its
// product with p is not, and sums of large weights may overflow before the normaliser: a row that is not
// finite, of a prompt whose softmax is sound, is summed again here, p times the weight, element by element.
struct MergeArgs {
  const float *part;    // [nch, P, H]
  const float2 *stats;  // [nch, P]
  const float *b;       // [H]
  float *y;             // [P, H]
  const uint16_t *w;    // [H, V]
  const void *logits;   // [P, V]
  int H, V, P, nch;
};

template <bool BF16>
__global__ __launch_bounds__(256) void policy_merge_kernel(MergeArgs a) {
  __shared__ float sh_f[kFirstMaxChunks], sh_y[4][64], sh_m[4];
  __shared__ double sh_z[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nb = (a.H + 63) / 64;
  const int pr = blockIdx.x / nb, n = (blockIdx.x % nb) * 64 + lane;
  const float *src = a.part + (size_t)pr * a.H + min(n, a.H - 1);
  const size_t cs = (size_t)a.P * a.H;
  static_assert(kFirstMaxChunks == 256, "a chunk per thread");
  const float2 st = a.stats[(size_t)min(tid, a.nch - 1) * a.P + pr];
  const float bias = a.b[min(n, a.H - 1)];
  constexpr int U = 16;
  float v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = src[(size_t)min(wave + 4 * u, a.nch - 1) * cs];  // clamped: no per-load branch
  // chunk c's factor 2^((m_c - M) log2 e) / Z
  const float wm = wave_max_f(st.x);
  if (lane == 0) sh_m[wave] = wm;
  __syncthreads();
  const float M = fmaxf(fmaxf(sh_m[0], sh_m[1]), fmaxf(sh_m[2], sh_m[3]));
  const float f = fast_exp2((st.x - M) * kLog2e);
  const double wz = wave_sum_d(tid < a.nch && st.x != -INFINITY ? (double)st.y * (double)f : 0.0);
  if (lane == 0) sh_z[wave] = wz;
  sh_f[tid] = f;
  __syncthreads();
  const float inv = (float)(1.0 / ((sh_z[0] + sh_z[1]) + (sh_z[2] + sh_z[3])));
  float y = 0.f;
  for (int c0 = wave; c0 < a.nch; c0 += 4 * U) {
    if (c0 != wave) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = src[(size_t)min(c0 + 4 * u, a.nch - 1) * cs];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c0 + 4 * u < a.nch) y = fmaf(v[u], sh_f[c0 + 4 * u], y);
  }
  sh_y[wave][lane] = y;
  __syncthreads();
  if (wave) return;
  y = ((sh_y[0][lane] + sh_y[1][lane]) + (sh_y[2][lane] + sh_y[3][lane])) * inv;
  unsigned long long bad = __ballot(!(fabsf(y) < INFINITY) && inv > 0.f && inv < INFINITY && fabsf(M) < INFINITY && n < a.H);
  while (bad) {
    const int l = __ffsll((long long)bad) - 1;
    bad &= bad - 1;
    const uint16_t *wr = a.w + (size_t)(n - lane + l) * a.V;
    float s = 0.f;
    for (int i = lane; i < a.V; i += 64)
      s = fmaf(__uint_as_float((uint32_t)wr[i] << 16),
               fast_exp2((ld_logit<BF16>(a.logits, (long long)pr * a.V + i) - M) * kLog2e) * inv, s);
    s = wave_sum_f(s);
    y = (lane == l) ? s : y;
  }
  if (n < a.H) a.y[(size_t)pr * a.H + n] = fmaxf(y + bias, 0.f);
}

// Second layer: 16 rows of W2 per workgroup, its wavefronts striding over 32-element steps of the
// contraction.
struct SecondArgs {
  const uint16_t *w;  // [H, H]
  const float *x;     // [P, H]
  const float *b;     // [H]
  float *y;           // [P, H]
  int H, P;
};
constexpr int kSecondWaves = 16;

__global__ __launch_bounds__(64 * kSecondWaves) void policy_second_kernel(SecondArgs a) {
  __shared__ float sh_o[kSecondWaves][4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kgrp = lane >> 4;
  const int n0 = blockIdx.x * 16;
  const float *xrow = a.x + (size_t)min(l16, a.P - 1) * a.H;  // columns past P repeat the last prompt
  const uint16_t *wrow = a.w + (size_t)min(n0 + l16, a.H - 1) * a.H;
  f32x4 acc[4] = {};
  constexpr int U = 4;  // steps in flight
  for (int k0 = wave * 32; k0 < a.H; k0 += U * kSecondWaves * 32) {
    v4u32 wv[U];
    f32x4 xa[U], xb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // clamped: no per-load branch (H % 8 == 0: whole vectors)
      const int k = min(k0 + u * kSecondWaves * 32 + kgrp * 8, a.H - 8);
      wv[u] = *reinterpret_cast<const v4u32 *>(wrow + k);
      xa[u] = *reinterpret_cast<const f32x4 *>(xrow + k);
      xb[u] = *reinterpret_cast<const f32x4 *>(xrow + k + 4);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = k0 + u * kSecondWaves * 32 + kgrp * 8 < a.H;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        acc[e & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? bf16_at(wv[u], e) : 0.f,
                                                          in ? (e < 4 ? xa[u][e & 3] : xb[u][e & 3]) : 0.f, acc[e & 3], 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) sh_o[wave][r][lane] = (acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r]);
  __syncthreads();
  if (tid < 256) {  // row n0 + (lane / 16) * 4 + r of prompt l16, r = wave
    float y = 0.f;
#pragma unroll
    for (int w = 0; w < kSecondWaves; ++w) y += sh_o[w][wave][lane];
    const int n = n0 + kgrp * 4 + wave;
    if (n < a.H && l16 < a.P) a.y[(size_t)l16 * a.H + n] = fmaxf(y + a.b[n], 0.f);
  }
}

// Scores of the C candidates for prompt p and their argmax (lowest index on ties):
// o = W3 h2 + b3, W3 [C, H] bf16, h2 [P, H] fp32.
struct HeadArgs {
  const uint16_t *w;
  const float *x;
  const float *b;
  float *scores;      // [P, C]
  int *block_size;    // [P]
  int C, H, base, radius;
};

// One workgroup per prompt, a wavefront per candidate up to 16 (then in turn): each lane takes
// 8-element slices of the candidate's W3 row (one 16-byte load) and of h2 (two 16-byte
// loads), four slices in flight, then a wavefront sum.  W3 rows are 16-byte aligned (H % 8 == 0).
__global__ __launch_bounds__(1024) void policy_head_kernel(HeadArgs a) {
  __shared__ float sc[64];
  const int pr = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const f32x4 *x4 = reinterpret_cast<const f32x4 *>(a.x + (size_t)pr * a.H);
  const int nv = a.H / 8;  // 8-element slices per row
  for (int c = wave; c < a.C; c += nw) {
    const u32x4 *w4 = reinterpret_cast<const u32x4 *>(a.w + (size_t)c * a.H);
    const float bias = a.b[c];
    float s = 0.f;
    for (int v0 = lane; v0 < nv; v0 += 64 * 4) {
      u32x4 wv[4];
      f32x4 xv[4][2];
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // clamped: no per-load branch
        const int v = min(v0 + 64 * u, nv - 1);
        wv[u] = w4[v];
        xv[u][0] = x4[2 * v];
        xv[u][1] = x4[2 * v + 1];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (v0 + 64 * u >= nv) break;
        const float w[8] = {bf16_lo(wv[u].x), bf16_hi(wv[u].x), bf16_lo(wv[u].y), bf16_hi(wv[u].y),
                            bf16_lo(wv[u].z), bf16_hi(wv[u].z), bf16_lo(wv[u].w), bf16_hi(wv[u].w)};
#pragma unroll
        for (int e = 0; e < 8; ++e) s = fmaf(w[e], xv[u][e >> 2][e & 3], s);
      }
    }
    s = wave_sum_f(s);
    if (lane == 0) sc[c] = s + bias;
  }
  __syncthreads();
  if (tid < 64) {  // lane c holds candidate c: the first one that no other beats
    const float v = sc[min(tid, a.C - 1)];
    if (tid < a.C) a.scores[(size_t)pr * a.C + tid] = v;
    int best = 0;
    float bv = sc[0];
    for (int c = 1; c < a.C; ++c) {
      const float o = lane_f(v, c);
      if (o > bv) {
        bv = o;
        best = c;
      }
    }
    if (tid == 0) a.block_size[pr] = a.base - a.radius + best;
  }
}

}  // namespace sdb
