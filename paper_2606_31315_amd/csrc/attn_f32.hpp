// attn_f32.hpp -- fp32 block attention on v_mfma_f32_16x16x4_f32.
//
// Same operation and partials as the bf16 kernel (attn_bf16.hpp), with the work dealt for the fp32
// matrix rate (157 TFLOP/s: 16 keys of a 16-row m-tile take a SIMD 64 products of 32 cycles), which
// bounds it from three or four m-tiles on; below that HBM does.
//   * A work item is a group of up to four m-tiles of a (sequence, kv head) pair over a run of keys, its
//     workgroup 16 wavefronts.  Wavefront w takes keys 16 (w mod 4) .. +15 of every 64 for m-tile w / 4 of
//     the group, with an online softmax of its own; wavefront w runs on SIMD w mod 4, so every SIMD
//     has the same work whatever the block.  The four states of a row are merged through LDS at the end.
//     (One wavefront per SIMD holding all the group's m-tiles, with a ring of its own, read each byte
//     once from LDS but ran slower: its unrolled code, up to 50 KB, came through the instruction cache
//     once per launch, about 27 us of every call.)
//   * S^T = K Q^T: a K operand is four dims of one key (16-byte LDS reads, rows XOR-swizzled by 16-byte
//     vectors), each lane then owns four keys of one query row, the B operand of O^T += V^T P^T.
//   * V^T operands come from the row-major tile by 16-byte reads too: lane l16 reads dims 4 l16 .. +3
//     of a key, one for each of four products whose output rows are the dims 4 i + j, i = 0..15; so V is
//     neither transposed nor swizzled.
//   * Every (sequence, kv head, group) is cut into splits of about the same work, as many as fill the
//     chip once (f32_item).  Shares that run on from one pair into the next, as the bf16 plan has them,
//     were slower here: the second piece's start cost 10 us of the 38 (4 sequences x 8 kv heads).
// Measured (us per call, before: register-staged 32-key tiles, V transposed on its way into LDS, one to
// four m-tiles per wavefront): 4 sequences x 8 kv heads, contexts 850-2686, blocks of 7-17 116 -> 36.2;
// contexts 2048, blocks of 4 / 8 / 16 / 32 / 64 60 / 61 / 63 / 79 / 154 -> 25 / 30 / 42 / 61 / 103; contexts 16384,
// blocks of 12 233 -> 140; 32 sequences, contexts 2048, blocks of 16 241 -> 171.  Of the 28.8 us of the
// first one's split kernel the plan takes 1.9, the query rows 3.5, the first tile 2.4, four or five tiles 3.2
// each, the merge of the states 2.
//   * Where whole pairs are the better cut (few keys, or more groups than CUs and contexts that are not
//     long; AttnPlan::whole) the same kernel runs with two key slots: 8 wavefronts and 67 KB of LDS, so that
//     a CU holds two of them, and no merge launch.  us per call, register-staged kernel / splits / whole
//     pairs, G = 4 and head_dim 128 unless named: 99 sequences x 8 kv heads, contexts 0-5, blocks of 11
//     21.6 / 38.6 / 20.3; 91 x 4, G = 1, contexts 0-1, blocks of 12-26 10.5 / 15.8 / 7.7; 100 x 8, contexts
//     120-184, blocks of 8 87.9 / 73.5 / 43.1; 224 x 8, G = 2, head_dim 64, the same contexts 84.4 / 85.5 / 38.3.
//     Geometric means over random shapes, splits and whole pairs, of the time over the register-staged
//     kernel's: up to 32 keys 1.14-1.6 and 0.77-0.95; up to 256 groups, 100-192 keys 0.49-0.63 and 0.50-0.58, 384
//     keys 0.53 and 0.58-0.69; more groups, 64-192 keys 0.62-1.24 and 0.49-0.66, 384-1024 keys 0.49-0.69 and 0.40-0.57
//     (these before a workgroup found its pair without a look at the others: f32_whole_item).
#pragma once

#include "attn.hpp"

namespace sdb {

// NK key slots of 16 keys: a wavefront for each slot and m-tile.
template <int D, int NK>
struct F32Tile {
  static constexpr int NW = NK * kF32GroupMT;     // wavefronts
  static constexpr int ROWB = D * 4;              // bytes per key row
  static constexpr int CPR = ROWB / 16;           // 16-byte vectors per row
  static constexpr int TILEB = 16 * NK * ROWB;    // bytes of a K (or V) tile
  static constexpr int RPI = 1024 / ROWB;         // rows written by one 1 KB transfer
  static constexpr int LPI = TILEB / 1024;        // transfers per K (or V) tile
  static constexpr int LPW = 2 * LPI / NW;        // transfers per wavefront and tile
  static constexpr int STAGEB = 2 * TILEB;        // K tile then V tile; two stages
  static constexpr int QB = 16 * kF32GroupMT * ROWB;  // bytes of the query rows
};

// K operands of a 16-key tile: k[t] dims 16 t + 4 kgrp .. +3 of key l16.  V operands: v[r][h] dims
// 64 h + 4 l16 .. +3 of key 4 kgrp + r.
// (the swizzled vector (4 t + kgrp) ^ l16 of a row lies at the address of t = 0 with bits 6.. xor t).
__device__ __forceinline__ void f32_read_k(f32x4 (&k)[8], unsigned ka) {
  asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
               "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3]), "=&v"(k[4]), "=&v"(k[5]), "=&v"(k[6]), "=&v"(k[7])
               : "v"(ka), "v"(ka ^ 64u), "v"(ka ^ 128u), "v"(ka ^ 192u), "v"(ka ^ 256u), "v"(ka ^ 320u), "v"(ka ^ 384u),
                 "v"(ka ^ 448u)
               : "memory");
}
__device__ __forceinline__ void f32_read_k(f32x4 (&k)[4], unsigned ka) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3])
               : "v"(ka), "v"(ka ^ 64u), "v"(ka ^ 128u), "v"(ka ^ 192u)
               : "memory");
}
__device__ __forceinline__ void f32_read_v(f32x4 (&v)[4][2], unsigned va) {
  asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:256\n\t"
               "ds_read_b128 %2, %8 offset:512\n\tds_read_b128 %3, %8 offset:768\n\t"
               "ds_read_b128 %4, %8 offset:1024\n\tds_read_b128 %5, %8 offset:1280\n\t"
               "ds_read_b128 %6, %8 offset:1536\n\tds_read_b128 %7, %8 offset:1792\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v[0][0]), "=&v"(v[0][1]), "=&v"(v[1][0]), "=&v"(v[1][1]), "=&v"(v[2][0]), "=&v"(v[2][1]),
                 "=&v"(v[3][0]), "=&v"(v[3][1])
               : "v"(va)
               : "memory");
}
__device__ __forceinline__ void f32_read_v(f32x4 (&v)[4][1], unsigned va) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:256\n\t"
               "ds_read_b128 %2, %4 offset:512\n\tds_read_b128 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v[0][0]), "=&v"(v[1][0]), "=&v"(v[2][0]), "=&v"(v[3][0])
               : "v"(va)
               : "memory");
}

struct F32Item {
  int s, g, grp, gmt, split, nsplit, slot, tiles, ctx, B, qoff;
};

// Work item of workgroup b: pairs are cut into splits of at most `per` units, numbered densely.  per is
// the least of W / grid x (1 + k / 16), k = 0 .. 15 (one per wavefront), at which the splits number at most
// a.bal_grid, else the largest; whole pairs without the workspace for partials (a.bal = 0).
__device__ __forceinline__ bool f32_item(const AttnArgs &a, int b, F32Item &it) {
  __shared__ int sh_n[kF32Waves];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const F32Seq first = f32_seq(a, lane);
  int per = 1 << 30;
  if (a.bal) {
    int W = 0;
    for (int c0 = 0; c0 < a.S; c0 += 64) {
      const F32Seq q = c0 == 0 ? first : f32_seq(a, c0 + lane);
      W += __builtin_amdgcn_readlane(wave_scan_i(q.tiles * q.weight * q.pairs), 63);
    }
    const int per0 = f32_per0(W, a.bal_grid, a.bal_min_tiles);
    int n = 0;
    const int pk = f32_per(per0, wave);
    for (int c0 = 0; c0 < a.S; c0 += 64) {
      const F32Seq q = c0 == 0 ? first : f32_seq(a, c0 + lane);
      n += __builtin_amdgcn_readlane(wave_scan_i(f32_splits(q.tiles, q.weight, pk) * q.pairs), 63);
    }
    if (lane == 0) sh_n[wave] = n;
    __syncthreads();
    const unsigned long long fit = __ballot(lane < kF32Waves && sh_n[lane & (kF32Waves - 1)] <= a.bal_grid);
    const int k = fit ? __ffsll((long long)fit) - 1 : kF32Waves - 1;
    per = f32_per(per0, k);
    if (b == 0 && threadIdx.x == 0) *a.plan = per;
  }
  int before = 0;
  for (int c0 = 0; c0 < a.S; c0 += 64) {
    const F32Seq q = c0 == 0 ? first : f32_seq(a, c0 + lane);
    const int n = f32_splits(q.tiles, q.weight, per), items = n * q.pairs, incl = before + wave_scan_i(items);
    const unsigned long long hit = __ballot(incl > b && incl - items <= b);
    if (hit) {
      const int l = __ffsll((long long)hit) - 1;  // wave-uniform
      it.s = c0 + l;
      it.ctx = __builtin_amdgcn_readlane(q.ctx, l);
      it.B = __builtin_amdgcn_readlane(q.B, l);
      it.qoff = __builtin_amdgcn_readlane(q.off, l);
      it.tiles = __builtin_amdgcn_readlane(q.tiles, l);
      it.nsplit = __builtin_amdgcn_readlane(n, l);
      const F32Groups gr = f32_groups(plan_mtiles(a.G, it.B), a.group_mt);
      const int r = b - __builtin_amdgcn_readlane(incl - items, l);
      const int p = r / it.nsplit;
      it.split = r - p * it.nsplit;
      it.g = p / gr.n;
      it.grp = p - it.g * gr.n;
      it.gmt = gr.mt;
      it.slot = b;
      return true;
    }
    before = __builtin_amdgcn_readlane(incl, 63);
  }
  return false;  // past the last item
}

// Whole pairs: workgroup b of S x Hkv x a.groups, without a look at the other sequences.
__device__ __forceinline__ bool f32_whole_item(const AttnArgs &a, int b, F32Item &it) {
  const int pair = b / a.groups;
  it.grp = b - pair * a.groups;
  it.s = pair / a.Hkv;
  it.g = pair - it.s * a.Hkv;
  it.ctx = ld_uniform(a.ctx_lens, it.s);
  it.B = ld_uniform(a.block_lens, it.s);
  it.qoff = ld_uniform(a.q_offsets, it.s);
  const F32Groups gr = f32_groups(plan_mtiles(a.G, it.B), a.group_mt);
  it.gmt = gr.mt;
  it.split = it.slot = 0;
  it.nsplit = 1;
  return it.B > 0 && it.grp < gr.n;
}

// NK = 4: f32_item's splits; NK = 2: whole pairs (a.bal = 0).
template <int D, int NK>
__global__ __launch_bounds__(64 * NK * kF32GroupMT, 4) void block_attn_f32_kernel(AttnArgs a) {
  using T = F32Tile<D, NK>;
  constexpr int NT4 = D / 16, NH = D / 64, NO = NH * 16;  // NO: output floats per lane
  constexpr int KT = 16 * NK;
  constexpr bool PLAN = NK == 4;
  static_assert(T::NW * NO * 256 <= 2 * T::STAGEB, "the states are exchanged through the ring");
  static_assert(!PLAN || (KT == kF32KT && T::NW == kF32Waves), "the plan's tiles and wavefronts");
  static_assert(T::QB <= T::STAGEB, "the query rows take the second stage's place");
  __shared__ __attribute__((aligned(1024))) char ring_raw[2 * T::STAGEB];
  __shared__ float sh_m[T::NW][16], sh_l[T::NW][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kgrp = lane >> 4;
  const int ks = wave % NK, mt = wave / NK;  // key slot, m-tile of the group
  char SDB_LDS *ring = (char SDB_LDS *)(SDB_LDS void *)ring_raw;

  // load-to-LDS: this wavefront's rows of a tile, all of K (the first half of them) or all of V; K swizzled
  const bool isv = wave >= T::NW / 2;
  const int row0 = (wave * T::LPW - (isv ? T::LPI : 0)) * T::RPI + lane / T::CPR;
  // operand addresses within a stage
  const unsigned lbase = (unsigned)(uintptr_t)ring + ks * 16 * T::ROWB;
  const unsigned ka = lbase + l16 * T::ROWB + ((kgrp ^ l16) << 4);
  const unsigned va = lbase + T::TILEB + kgrp * 4 * T::ROWB + l16 * 16;

  F32Item it;
  if (PLAN ? !f32_item(a, blockIdx.x, it) : !f32_whole_item(a, blockIdx.x, it)) return;
  const int s = it.s, g = it.g, ctx = it.ctx, qoff = it.qoff;
  const int k0 = PLAN ? (int)((long long)it.tiles * it.split / it.nsplit) * KT : 0;
  const int k1 = PLAN ? min((int)((long long)it.tiles * (it.split + 1) / it.nsplit) * KT, ctx + it.B) : ctx + it.B;
  const int M = a.G * it.B;
  const int m0 = it.grp * it.gmt * 16;          // the group's first query row
  const int m = m0 + mt * 16 + l16;             // this lane's
  const bool act = mt < it.gmt && m0 + mt * 16 < M;  // uniform per wavefront
  const bool valid = act && m < M;
  const char *src = reinterpret_cast<const char *>(isv ? a.v : a.k) + ((size_t)(s * a.Hkv + g) * a.Lmax) * T::ROWB;
  // byte offset of query row r of the pair in q and out
  auto qrow_off = [&](int r) { return ((size_t)(qoff + r / a.G) * a.Hq + g * a.G + r % a.G) * T::ROWB; };
  auto issue = [&](int t) {
    char SDB_LDS *st = ring + (t & 1) * T::STAGEB + wave * T::LPW * 1024;
#pragma unroll
    for (int q = 0; q < T::LPW; ++q) {  // rows past the item's last key re-read it
      const int row = row0 + q * T::RPI;
      const int col = ((lane % T::CPR) ^ (isv ? 0 : row % 16)) * 16;
      __builtin_amdgcn_global_load_lds((const void *)(src + (size_t)min(k0 + t * KT + row, k1 - 1) * T::ROWB + col),
                                       (SDB_LDS void *)(st + q * 1024), 16, 0, kLoadNT);
    }
  };
  const int ntiles = (k1 - k0 + KT - 1) / KT;
  // The query rows come the same way, into the second stage and laid out as K rows, before the first
  // tile (plain loads would be waited for together with every transfer in flight).
  {
    constexpr int QPW = (kF32GroupMT * 16 / T::RPI) / T::NW;  // transfers per wavefront
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
      const int row = (wave * QPW + q) * T::RPI + lane / T::CPR;  // rows past the block re-read its last
      const int col = ((lane % T::CPR) ^ (row % 16)) * 16;
      __builtin_amdgcn_global_load_lds((const void *)(reinterpret_cast<const char *>(a.q) + qrow_off(min(m0 + row, M - 1)) + col),
                                       (SDB_LDS void *)(ring + T::STAGEB + (wave * QPW + q) * 1024), 16, 0, 0);
    }
  }
  issue(0);
  f32x4 qop[NT4], oacc[NH][4];
  const int row_i = valid ? m / a.G : 0;
  wait_vmcnt<T::LPW>();
  __syncthreads();
  f32_read_k(qop, (unsigned)(uintptr_t)ring + T::STAGEB + (mt * 16 + l16) * T::ROWB + ((kgrp ^ l16) << 4));
  __syncthreads();
  if (ntiles > 1) issue(1);
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) oacc[h][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float sl2 = a.scale_log2;

  for (int t = 0; t < ntiles; ++t) {
    if (t + 1 < ntiles) wait_vmcnt<T::LPW>();
    else wait_vmcnt<0>();
    __syncthreads();  // tile t landed for every wavefront
    const unsigned so = (t & 1) * T::STAGEB;
    const int kb = k0 + t * KT + ks * 16;
    const bool on = act && kb < k1;  // uniform: the last tile may have no key for this slot
    // p[r]: key kb + 4 kgrp + r of row l16; two chains of products
    f32x4 p{0.f, 0.f, 0.f, 0.f}, p1 = p, v[4][NH];
    if (on) {
      f32x4 k[NT4];
      f32_read_k(k, ka + so);
#pragma unroll
      for (int i = 0; i < NT4; ++i)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          p = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i][e], qop[i][e], p, 0, 0, 0);
          p1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i][e + 1], qop[i][e + 1], p1, 0, 0, 0);
        }
      f32_read_v(v, va + so);
    }
    __syncthreads();  // the stage is free again
    if (t + 2 < ntiles) issue(t + 2);
    if (!on) continue;
    p += p1;
    if (kb + 16 > (a.causal ? min(k1, ctx + 1) : k1)) {  // some key is masked for some row
      const int lim = a.causal ? min(k1, ctx + row_i + 1) : k1;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (kb + kgrp * 4 + r >= lim) p[r] = -INFINITY;
    }
    const float tmax = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
    const float2 p16 = pair_x16(tmax);
    const float2 p32 = pair_x32(fmaxf(p16.x, p16.y));
    const float mnew = fmaxf(m_run, fmaxf(p32.x, p32.y) * sl2);
    const float muse = (mnew == -INFINITY) ? 0.f : mnew;
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = fast_exp2(fmaf(p[r], sl2, -muse));
    if (__any(mnew != m_run)) {
      const float alpha = fast_exp2(m_run - muse);
      l_run *= alpha;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) oacc[h][i] *= alpha;
    }
    m_run = mnew;
    l_run += (p[0] + p[1]) + (p[2] + p[3]);
    // oacc[h][i] row 4 kgrp + r is dim 64 h + 4 (4 kgrp + r) + i
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          oacc[h][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r][h][i], p[r], oacc[h][i], 0, 0, 0);
  }

  // ---- the slots' states to one: common maximum, then the scaled sums through LDS ----
  {
    const float2 p16 = pair_x16(l_run);
    const float2 p32 = pair_x32(p16.x + p16.y);
    l_run = p32.x + p32.y;
  }
  if (lane < 16) {
    sh_m[wave][l16] = m_run;
    sh_l[wave][l16] = l_run;
  }
  __syncthreads();  // and every wavefront is done with the ring
  float *xch = reinterpret_cast<float *>(ring_raw);  // [wave][h][r][i][lane]
  float mx = -INFINITY, ls = 0.f;
#pragma unroll
  for (int w = 0; w < NK; ++w) mx = fmaxf(mx, sh_m[mt * NK + w][l16]);
  const float mu = (mx == -INFINITY) ? 0.f : mx;
#pragma unroll
  for (int w = 0; w < NK; ++w) ls = fmaf(sh_l[mt * NK + w][l16], fast_exp2(sh_m[mt * NK + w][l16] - mu), ls);
  if (act) {
    const float f = fast_exp2(m_run - mu);
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) xch[(wave * NO + (h * 4 + r) * 4 + i) * 64 + lane] = oacc[h][i][r] * f;
  }
  __syncthreads();
  if (valid) {  // slot ks finishes the dims 64 h + 16 kgrp + 4 r .. +3 of the m-tile's rows, r = ks, ks + NK ..
    const bool direct = it.nsplit == 1;
    const size_t prow = (size_t)it.slot * a.part_rows + mt * 16 + l16;
    float *dst = direct ? reinterpret_cast<float *>(reinterpret_cast<char *>(a.out) + qrow_off(m)) : a.part_o + prow * D;
    const float inv = direct ? 1.f / ls : 1.f;
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int r0 = 0; r0 < 4; r0 += NK) {
        const int r = r0 + ks;
        f32x4 o{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NK; ++w)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] += xch[((mt * NK + w) * NO + (h * 4 + r) * 4 + i) * 64 + lane];
        *reinterpret_cast<f32x4 *>(dst + h * 64 + (kgrp * 4 + r) * 4) = o * inv;
      }
    if (!direct && ks == 0 && kgrp == 0) a.part_ml[prow] = float2{mx, ls};
  }
}

}  // namespace sdb
