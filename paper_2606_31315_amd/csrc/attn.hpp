// attn.hpp -- block attention over a GQA KV cache with ragged per-sequence blocks.
//
// Operation (Sec. 2.1): the B_s block rows of sequence s attend to their committed
// context and to the block itself, causally for target verification or
// bidirectionally for the block-diffusion drafter.  Query head h reads kv head
// h / G with G = Hq / Hkv.
//
// This file holds what the split kernels (attn_bf16.hpp, attn_f32.hpp) share: the kernel arguments,
// the plans that cut the keys of every (sequence, kv head) pair into work items on the device, and the
// merge.  All G*B_s query rows of a sequence's kv-head group are packed into 16-row MFMA tiles
// (m-tiles), so each K/V byte is read from HBM once for the whole group.  A pair whose keys fit one
// split writes its output directly.  Otherwise each split writes fp32 partials (unnormalised O, row
// max in log2 units, row sum) and a second launch, block_attn_merge_kernel, combines them.  The kernel
// boundary is the only cross-workgroup synchronisation: a release fence per workgroup writes back the
// XCD's L2, and merging in the split kernel without fences (tagged partials, the last arrivals polling)
// was slower too, 38.65 against 33.35 us per call on the ragged batch.
//
// The plans' arithmetic comes first: plain integers, for the device, for the launchers and, in a build
// without HIP, for a check of the plans on the CPU.
#pragma once

#if defined(__HIPCC__)
#include "common.hpp"
#define SDB_HD __host__ __device__ __forceinline__
#else
#define SDB_HD inline
#endif

namespace sdb {

SDB_HD int plan_min(int a, int b) { return a < b ? a : b; }
SDB_HD int plan_max(int a, int b) { return a > b ? a : b; }
SDB_HD int plan_mtiles(int G, int B) { return (G * plan_max(B, 0) + 15) >> 4; }  // 16-row query tiles of a block

// ---- balanced plan (bf16) ----------------------------------------------------------
// Relative time of one key tile by the block's m-tiles (16-row query tiles): up to 3 m-tiles
// the split kernel streams a tile at the memory's pace; beyond that the wavefronts' LDS reads
// and arithmetic add to it (8 sequences x 8 kv heads, contexts 4096, one wave, MI355X: 33.1 us
// per call at 2 m-tiles, 33.7 at 3, 34.5 at 4, 35.5 at 5, 37.9 at 6, 40.0 at 7, 41.6 at 8).
// Chosen by A/B on the multi-wave batches: against the steeper table measured before the
// kernel's lane swaps (20, 23, 25, 28, 32, 33 for 1-3 ... 8 m-tiles), 16 sequences with contexts
// 1k-8k 82.75 -> 81.14 us per call, 32 sequences with contexts 8k-32k 472.9 -> 452.1 us.
constexpr int kBalWeightMax8 = 31;  // the weight at 8 m-tiles; 4 more per m-tile past 8
SDB_HD int bal_weight(int nmt) {
  constexpr int kw[9] = {20, 20, 20, 20, 22, 24, 26, 29, kBalWeightMax8};
  return nmt <= 8 ? kw[nmt] : kBalWeightMax8 + 4 * (nmt - 8);
}

constexpr int kBalGrid = 256;     // workgroups of the balanced plan: one per CU of the MI355X
constexpr int kMaxMTiles = 16;    // (Hq / Hkv) * max_block <= 256

// Units a pair takes on the line ahead of its first tile: what starting it costs the workgroup
// whose share runs on into it (the pair before filed, query rows and first tiles fetched), about five
// tiles.  Less than the shortest share, so every workgroup between a pair's first and last holds
// a tile of it.  us per call at 0 / 60 / 90 / 110 / 130 / 160 units: 16 sequences, contexts 1k-8k 64.8 / 62.0 / 61.1 /
// 60.4 / 60.7 / 62.0; 32 sequences, contexts 8k-32k 451 / 450 / 443 / 445 / 443 / 444; 20 sequences, head_dim
// 64, contexts 1k-12k 86.8 without, 79.5 / 79.6 / 79.4 at 90 / 110 / 130; 24 sequences, contexts 3k-16k
// 144.1 without, 141.1 / 142.5 / 143.6.
constexpr int kBalPairCost = 100;
// Units per share of W in all.
SDB_HD int bal_per(int W, int min_tiles) { return plan_max((W + kBalGrid - 1) / kBalGrid, min_tiles * bal_weight(1)); }

// Units of one pair of n tiles of weight w (0: no tiles, no pair).
SDB_HD int bal_pair_units(int n, int w) { return n > 0 ? n * w + kBalPairCost : 0; }

// First tile of a pair (first tile's unit p0, weight w) whose first unit is at or after unit u.
SDB_HD int bal_tile_at(int u, int p0, int w) { return u <= p0 ? 0 : (u - p0 + w - 1) / w; }

// What the share [u0, u1) takes of the pair that holds unit u0 (its units from `start` on, ts tiles of
// weight w): tiles [j0, j1), and the cursor after them; none where the next tile is the next pair's (next:
// that pair's first unit) or the next share's (next: u1).
struct BalPiece {
  int j0, j1, next;
  bool any;
};
SDB_HD BalPiece bal_piece(int u0, int u1, int start, int ts, int w) {
  const int p0 = start + kBalPairCost;
  BalPiece b;
  b.j0 = b.j1 = bal_tile_at(u0, p0, w);
  b.any = false;
  if (b.j0 >= ts) {  // past the first unit of the pair's last tile
    b.next = p0 + ts * w;
  } else if (p0 + b.j0 * w >= u1) {
    b.next = u1;
  } else {
    b.any = true;
    b.j1 = plan_min(bal_tile_at(u1, p0, w), ts);  // > j0
    b.next = p0 + b.j1 * w;
  }
  return b;
}

// First and last share that hold a tile of the pair.
struct BalShares {
  int first, last;
};
SDB_HD BalShares bal_shares(int start, int ts, int w, int per) {
  const int p0 = start + kBalPairCost;
  return BalShares{p0 / per, (p0 + (ts - 1) * w) / per};
}

// ---- fp32 plan ---------------------------------------------------------------------
constexpr int kF32KT = 64;       // keys per tile
constexpr int kF32Waves = 16;    // wavefronts of the split kernel, and candidates of f32_per
constexpr int kF32GroupMT = 4;   // m-tiles per work item at most
constexpr int kF32MinTiles = 2;  // shortest share, in tiles

// A block's m-tiles go to groups of at most group_mt (<= 4), evenly: (groups, m-tiles per group).  The
// host keeps the groups of the largest block to four.
struct F32Groups {
  int n, mt;
};
SDB_HD F32Groups f32_groups(int nmt, int group_mt) {
  const int ng = 1 + (nmt > group_mt) + (nmt > 2 * group_mt) + (nmt > 3 * group_mt);
  const int per = ng == 1 ? nmt : ng == 2 ? (nmt + 1) >> 1 : ng == 3 ? ((nmt + 2) * 43) >> 7 : (nmt + 3) >> 2;
  return F32Groups{ng, per};
}
// Relative time of a tile: the matrix products of a group's m-tiles, 2048 cycles of a SIMD each, or the
// memory's pace, 64 KB in about three of them.
SDB_HD int f32_weight(int mt) { return plan_max(mt, 3); }
// Units per split: candidate k = 0 .. kF32Waves - 1 of the total W, ascending.
SDB_HD int f32_per0(int W, int grid, int min_tiles) { return plan_max((W + grid - 1) / grid, min_tiles * 3); }
SDB_HD int f32_per(int per0, int k) { return per0 + ((per0 * k + 15) >> 4); }
// Splits of a pair's group at `per` units of work each.
SDB_HD int f32_splits(int tiles, int weight, int per) {
  const unsigned n = ((unsigned)(tiles * weight) + (unsigned)per - 1u) / (unsigned)per;
  return plan_min((int)n, tiles);
}
// Workgroups that hold every split: the candidates end at per0 x 31 / 16, where the splits number at most
// 16 / 31 grid + pairs; else none is sure to fit the grid and there are at most as many more as pairs.
SDB_HD int f32_launch(int pairs, int grid) { return 31 * pairs <= 15 * grid ? grid : grid + pairs; }

#if defined(__HIPCC__)

struct AttnArgs {
  const void *q;
  const void *k;
  const void *v;
  void *out;
  const int *ctx_lens;
  const int *block_lens;
  const int *q_offsets;
  float *part_o;      // [n_work, Mpad, D] unnormalised partial outputs
  float2 *part_ml;    // [n_work, Mpad]    (row max in log2 units, row sum)
  int S, Hq, Hkv, G, Lmax;
  int split_len;      // longest split (keys), a multiple of gran
  int gran;           // split lengths are multiples of gran keys
  int max_splits;     // splits per (sequence, kv head) at the host-known maximum length
  int Mpad;           // rows reserved per work item in the partial buffers
  int n_work;         // S * Hkv * max_splits
  int per_xcd;        // ceil(n_work / 8): the XCD-grouped deal of a one-wave grid
  int dense;          // more than one wave: work items numbered densely on the device
  float scale_log2;   // softmax scale * log2(e)
  int causal;
  // paged caches only: k, v are page pools [num_pages, Hkv, page_size, D]; logical page j of
  // sequence s is pool page block_table[s * max_pages + j]
  const int *block_table;
  int page_log2, max_pages, num_pages;
  // fused append only: the block's new keys and values [total_q, Hkv, D]
  const void *k_new;
  const void *v_new;
  // balanced plan (bf16; bal_share): shares of at least
  // bal_min_tiles key tiles of bal_kt keys
  int bal, bal_grid, bal_min_tiles, bal_kt;  // bal_grid: fp32, splits at most
  // fp32: m-tiles per workgroup at most (a block's m-tiles go to ceil(m-tiles / group_mt) workgroups,
  // evenly), the groups of the largest block, and the rows of a partial slot
  int group_mt, groups, part_rows;
  int *plan;  // workspace word: the units per split the split kernel took
};

// ---- work items ----------------------------------------------------------------
// Each (sequence, kv head) pair of L keys is cut into nsplit = ceil(L / split_len) splits of
// even length (ceil(L / nsplit) rounded up to gran keys, never more than split_len, so every
// split is non-empty).  One work item per split.
//   One-wave grid (n_work <= one workgroup per CU): workgroup w owns slot w = pair *
//     max_splits + split, dealt so that a pair's splits share an XCD; slots past a pair's
//     nsplit have no work.
//   Larger grids: the items that exist are numbered densely on the device, sequence by
//     sequence, pair by pair, split by split (a prefix sum of Hkv * nsplit over the
//     sequences, 64 per round), and workgroup i takes item i; round-robin dispatch over the
//     XCDs then spreads every long sequence over all of them, and no workgroup is spent on an
//     empty slot.
//   Dense grids whose splits are at the length cap (kLongSplit) instead cut each pair into
//     full splits of split_len keys plus one partial last split, and number all full splits
//     first and then the partial ones, longest first, so the shortest items fill the tail
//     (32 sequences, contexts 8k-32k: 537 -> 513 us).  Shorter capped-below plans keep even
//     splits: there the partial items would be tiny workgroups (16 sequences, contexts 1k-8k:
//     96.0 us even, 100.3 us full + partial).
// Partial slots are the workgroup's slot (one wave) or the pair's slot base + split (dense).
struct AttnItem {
  int s, g, split, nsplit, k0, k1, slot, ctx, B, qoff;
};

// Longest split the planner makes (keys); dense plans at this length order their items
// longest first.
constexpr int kLongSplit = 4096;

__device__ __forceinline__ bool attn_item(const AttnArgs &a, int b, AttnItem &it) {
  if (!a.dense) {
    const int w = xcd_logical_id(b, a.per_xcd);
    if (w >= a.n_work) return false;
    it.split = w % a.max_splits;
    const int sg = w / a.max_splits;
    it.g = sg % a.Hkv;
    it.s = sg / a.Hkv;
    it.ctx = a.ctx_lens[it.s];
    it.B = a.block_lens[it.s];
    it.qoff = a.q_offsets[it.s];
    if (it.B <= 0) return false;
    it.nsplit = (it.ctx + it.B + a.split_len - 1) / a.split_len;
    if (it.split >= it.nsplit) return false;
    it.slot = w;
  } else if (a.split_len >= kLongSplit) {
    // Splits at the length cap (long contexts, several waves): full splits of split_len keys
    // first, sequence by sequence; then each sequence's partial last split, longest first
    // (in sequence order beyond 64 sequences), so the shortest items run last and fill the
    // tail.  Slots stay in the per-pair order the merge reads.
    const int lane = threadIdx.x & 63;
    const int sl = a.split_len;
    int before = 0, sbefore = 0;
    bool found = false;
    for (int c0 = 0; c0 < a.S && !found; c0 += 64) {
      const int k = min(c0 + lane, a.S - 1);  // clamped: no per-load branch
      const int ctx = a.ctx_lens[k], B = a.block_lens[k], off = a.q_offsets[k];
      const bool live = c0 + lane < a.S && B > 0;
      const int n = live ? (ctx + B + sl - 1) / sl : 0;
      const int nf = live ? (ctx + B) / sl : 0;
      const int items = nf * a.Hkv;
      const int incl = before + wave_scan_i(items);
      const int sincl = sbefore + wave_scan_i(n * a.Hkv);
      const unsigned long long hit = __ballot(incl > b && incl - items <= b);
      if (hit) {
        const int l = __ffsll((long long)hit) - 1;  // wave-uniform
        it.s = c0 + l;
        it.ctx = __builtin_amdgcn_readlane(ctx, l);
        it.B = __builtin_amdgcn_readlane(B, l);
        it.qoff = __builtin_amdgcn_readlane(off, l);
        it.nsplit = __builtin_amdgcn_readlane(n, l);
        const int nfl = __builtin_amdgcn_readlane(nf, l);
        const int r = b - __builtin_amdgcn_readlane(incl - items, l);
        it.g = r / nfl;
        it.split = r - it.g * nfl;
        it.slot = __builtin_amdgcn_readlane(sincl - n * a.Hkv, l) + it.g * it.nsplit + it.split;
        found = true;
      }
      before = __builtin_amdgcn_readlane(incl, 63);
      sbefore = __builtin_amdgcn_readlane(sincl, 63);
    }
    if (!found) {
      const int p = b - before;  // index among the partial items
      const int rank = p / a.Hkv;
      const int g = p - rank * a.Hkv;
      int pb = 0;
      sbefore = 0;
      for (int c0 = 0; c0 < a.S && !found; c0 += 64) {
        const int k = min(c0 + lane, a.S - 1);  // clamped: no per-load branch
        const int ctx = a.ctx_lens[k], B = a.block_lens[k], off = a.q_offsets[k];
        const bool live = c0 + lane < a.S && B > 0;
        const int n = live ? (ctx + B + sl - 1) / sl : 0;
        const int part = live ? (ctx + B) % sl : 0;
        const int sincl = sbefore + wave_scan_i(n * a.Hkv);
        int key;  // this lane's position among the partial items (valid where part > 0)
        if (a.S <= 64) {
          key = 0;
          for (int t = 0; t < a.S; ++t) {
            const int pt = __builtin_amdgcn_readlane(part, t);
            key += (pt > part) || (pt == part && t < lane);
          }
        } else {
          const int has = part > 0 ? 1 : 0;
          key = pb + wave_scan_i(has) - has;
          pb = __builtin_amdgcn_readlane(pb + wave_scan_i(has), 63);
        }
        const unsigned long long hit = __ballot(part > 0 && key == rank);
        if (hit) {
          const int l = __ffsll((long long)hit) - 1;  // wave-uniform
          it.s = c0 + l;
          it.ctx = __builtin_amdgcn_readlane(ctx, l);
          it.B = __builtin_amdgcn_readlane(B, l);
          it.qoff = __builtin_amdgcn_readlane(off, l);
          it.nsplit = __builtin_amdgcn_readlane(n, l);
          it.g = g;
          it.split = it.nsplit - 1;
          it.slot = __builtin_amdgcn_readlane(sincl - n * a.Hkv, l) + g * it.nsplit + it.split;
          found = true;
        }
        sbefore = __builtin_amdgcn_readlane(sincl, 63);
      }
      if (!found) return false;  // past the last item
    }
    it.k0 = it.split * sl;
    it.k1 = min(it.k0 + sl, it.ctx + it.B);
    return true;
  } else {
    const int lane = threadIdx.x & 63;
    int before = 0;
    bool found = false;
    for (int c0 = 0; c0 < a.S && !found; c0 += 64) {
      const int k = min(c0 + lane, a.S - 1);  // clamped: no per-load branch
      const int ctx = a.ctx_lens[k], B = a.block_lens[k], off = a.q_offsets[k];
      const int n = (c0 + lane < a.S && B > 0) ? (ctx + B + a.split_len - 1) / a.split_len : 0;
      const int items = n * a.Hkv;
      const int incl = before + wave_scan_i(items);
      const unsigned long long hit = __ballot(incl > b && incl - items <= b);
      if (hit) {
        const int l = __ffsll((long long)hit) - 1;  // wave-uniform
        it.s = c0 + l;
        it.ctx = __builtin_amdgcn_readlane(ctx, l);
        it.B = __builtin_amdgcn_readlane(B, l);
        it.qoff = __builtin_amdgcn_readlane(off, l);
        it.nsplit = __builtin_amdgcn_readlane(n, l);
        const int r = b - __builtin_amdgcn_readlane(incl - items, l);
        it.g = r / it.nsplit;
        it.split = r - it.g * it.nsplit;
        it.slot = b;
        found = true;
      }
      before = __builtin_amdgcn_readlane(incl, 63);
    }
    if (!found) return false;  // past the last item
  }
  const int L = it.ctx + it.B;
  const int slen = (((L + it.nsplit - 1) / it.nsplit + a.gran - 1) / a.gran) * a.gran;
  it.k0 = it.split * slen;
  it.k1 = min(it.k0 + slen, L);
  return true;
}

// ---- balanced plan ---------------------------------------------------------------
// Pair (s, g) holds n = ceil((ctx_s + B_s) / kt) key tiles (none when B_s = 0), each weighing
// w = bal_weight(m-tiles of its block) units, after kBalPairCost units for its start; the pairs line
// up in (sequence, kv head) order, W units in all.  Workgroup w takes the tiles whose first unit lies in [w * per, (w + 1) * per),
// per = max(ceil(W / kBalGrid), bal_min_tiles * the lightest weight), so every workgroup gets
// about the same work whatever the lengths are; its share is cut where it crosses from one pair
// to the next, one work item per piece.  The piece of workgroup w in pair q = s * Hkv + g files
// its partial at slot w + q, so a pair's pieces hold consecutive slots from (first workgroup) + q.
// (Even splits per pair leave ragged batches with fractional waves: 16 sequences, contexts
// 1k-8k, about 350 splits of up to 2064 keys on 256 CUs.)
struct BalShare {
  int per, u0, u1;  // units per share; this workgroup's unit range [u0, u1)
};

// Lanes hold sequence values; per-pair tiles and weight of that sequence (0 past a.S / empty).
__device__ __forceinline__ int bal_seq_tiles(bool live, int ctx, int B, int kt) {
  return (live && B > 0) ? (ctx + B + kt - 1) / kt : 0;
}
__device__ __forceinline__ int bal_seq_weight(const AttnArgs &a, int B) {
  return bal_weight(plan_mtiles(a.G, B));
}

// This workgroup's share: the total W, one round of loads per 64 sequences.
__device__ __forceinline__ BalShare bal_share(const AttnArgs &a, int w, int kt) {
  const int lane = threadIdx.x & 63;
  int W = 0;
  for (int c0 = 0; c0 < a.S; c0 += 64) {
    const int k = min(c0 + lane, a.S - 1);  // clamped: no per-load branch
    const int B = a.block_lens[k];
    const int u = bal_pair_units(bal_seq_tiles(c0 + lane < a.S, a.ctx_lens[k], B, kt), bal_seq_weight(a, B)) * a.Hkv;
    W += __builtin_amdgcn_readlane(wave_scan_i(u), 63);
  }
  BalShare sh;
  sh.per = bal_per(W, a.bal_min_tiles);
  sh.u0 = min(w * sh.per, W);
  sh.u1 = min(sh.u0 + sh.per, W);
  return sh;
}

// The next piece of the share: u0 is a cursor, the first unit not yet handed out.  The first
// tile whose first unit is at or after u0 starts the piece, if that unit lies before u1; the
// piece runs to the last tile of the same pair whose first unit lies before u1, and the cursor
// moves to the first unit of the tile after it.  Every piece moves the cursor forward, so the
// loop over pieces ends.  False when the share is done.
__device__ __forceinline__ bool bal_item(const AttnArgs &a, BalShare &sh, int kt, AttnItem &it) {
  const int lane = threadIdx.x & 63;
  // Two rounds at most: when u0 lies inside a pair's last tile past its first unit, the next
  // tile is the first of the next pair with tiles, whose first unit is that pair's start.
  for (int round = 0; round < 2; ++round) {
    if (sh.u0 >= sh.u1) return false;
    int before = 0;
    bool next_pair = false;
    for (int c0 = 0; c0 < a.S; c0 += 64) {
      const int k = min(c0 + lane, a.S - 1);  // clamped: no per-load branch
      const int ctx = a.ctx_lens[k], B = a.block_lens[k], off = a.q_offsets[k];
      const int t = bal_seq_tiles(c0 + lane < a.S, ctx, B, kt);
      const int wt = bal_seq_weight(a, B);
      const int sequ = bal_pair_units(t, wt) * a.Hkv;
      const int incl = before + wave_scan_i(sequ);
      const unsigned long long hit = __ballot(incl > sh.u0 && incl - sequ <= sh.u0);  // holds unit u0
      if (hit) {
        const int l = __ffsll((long long)hit) - 1;  // wave-uniform
        const int ts = __builtin_amdgcn_readlane(t, l), w = __builtin_amdgcn_readlane(wt, l);
        const int pu = bal_pair_units(ts, w);  // units of each of the sequence's pairs
        const int pre = __builtin_amdgcn_readlane(incl - sequ, l);
        const int g = (sh.u0 - pre) / pu;
        const int start = pre + g * pu;  // first unit of pair (s, g)
        const BalPiece b = bal_piece(sh.u0, sh.u1, start, ts, w);
        sh.u0 = b.next;
        if (!b.any) {
          if (b.next >= sh.u1) return false;
          next_pair = true;
          break;
        }
        it.s = c0 + l;
        it.g = g;
        it.ctx = __builtin_amdgcn_readlane(ctx, l);
        it.B = __builtin_amdgcn_readlane(B, l);
        it.qoff = __builtin_amdgcn_readlane(off, l);
        it.k0 = b.j0 * kt;
        it.k1 = min(b.j1 * kt, it.ctx + it.B);
        const BalShares bs = bal_shares(start, ts, w, sh.per);
        const int wme = blockIdx.x;  // the piece's first unit lies in this workgroup's share
        it.nsplit = bs.last - bs.first + 1;
        it.split = wme - bs.first;
        it.slot = wme + it.s * a.Hkv + g;
        return true;
      }
      before = __builtin_amdgcn_readlane(incl, 63);
    }
    if (!next_pair) return false;  // no sequence holds u0: past the last tile
  }
  return false;
}

// Partial slot of split 0 of pair (s, g) and the pair's split count (0: no block).
__device__ __forceinline__ int2 attn_pair_slots(const AttnArgs &a, int s, int g, int &B) {
  if (a.bal) {
    const int lane = threadIdx.x & 63;
    int W = 0, pre = 0, ts = 0, Bs = 0;
    for (int c0 = 0; c0 < a.S; c0 += 64) {
      const int k = min(c0 + lane, a.S - 1);  // clamped: no per-load branch
      const int Bk = a.block_lens[k];
      const int t = bal_seq_tiles(c0 + lane < a.S, a.ctx_lens[k], Bk, a.bal_kt);
      const int sequ = bal_pair_units(t, bal_seq_weight(a, Bk)) * a.Hkv;
      const int incl = wave_scan_i(sequ);
      if (s >= c0 && s < c0 + 64) {  // wave-uniform
        const int l = s - c0;
        pre = W + __builtin_amdgcn_readlane(incl - sequ, l);
        ts = __builtin_amdgcn_readlane(t, l);
        Bs = __builtin_amdgcn_readlane(Bk, l);
      }
      W += __builtin_amdgcn_readlane(incl, 63);
    }
    B = Bs;
    if (Bs <= 0) return int2{0, 0};
    const int w = bal_seq_weight(a, Bs);
    const BalShares bs = bal_shares(pre + g * bal_pair_units(ts, w), ts, w, bal_per(W, a.bal_min_tiles));
    return int2{bs.first + s * a.Hkv + g, bs.last - bs.first + 1};
  }
  if (!a.dense) {
    // both lengths in one round of scalar loads: one use of both before the branch on B, so the
    // context length's load is not sunk behind it
    B = ld_uniform(a.block_lens, s);
    int ctx = ld_uniform(a.ctx_lens, s);
    asm volatile("" : "+s"(B), "+s"(ctx));
    if (B <= 0) return int2{0, 0};
    return int2{(s * a.Hkv + g) * a.max_splits, (ctx + B + a.split_len - 1) / a.split_len};
  }
  const int lane = threadIdx.x & 63;
  int before = 0;
  for (int c0 = 0; c0 <= s; c0 += 64) {
    const int k = min(c0 + lane, a.S - 1);  // clamped: no per-load branch
    const int ctx = a.ctx_lens[k], Bk = a.block_lens[k];
    const int n = (c0 + lane < a.S && Bk > 0) ? (ctx + Bk + a.split_len - 1) / a.split_len : 0;
    const int incl = before + wave_scan_i(n * a.Hkv);
    if (s < c0 + 64) {
      const int l = s - c0;
      B = __builtin_amdgcn_readlane(Bk, l);
      const int ns = __builtin_amdgcn_readlane(n, l);
      if (B <= 0) return int2{0, 0};
      return int2{__builtin_amdgcn_readlane(incl, l) - ns * a.Hkv + g * ns, ns};
    }
    before = __builtin_amdgcn_readlane(incl, 63);
  }
  B = 0;
  return int2{0, 0};
}

// ---- fp32 plan ---------------------------------------------------------------------
// A sequence on lane k: key tiles of each of its pairs, the relative time of one, and its pairs (kv heads x
// groups; none without a block).
struct F32Seq {
  int ctx, B, off, tiles, weight, pairs;
};
__device__ __forceinline__ F32Seq f32_seq(const AttnArgs &a, int k) {
  const int kc = min(k, a.S - 1);  // clamped: no per-load branch
  F32Seq q;
  q.ctx = a.ctx_lens[kc];
  q.B = a.block_lens[kc];
  q.off = a.q_offsets[kc];
  const bool live = k < a.S && q.B > 0;
  const F32Groups gr = f32_groups(plan_mtiles(a.G, q.B), a.group_mt);
  q.tiles = live ? (q.ctx + q.B + kF32KT - 1) / kF32KT : 0;
  q.weight = f32_weight(gr.mt);
  q.pairs = live ? a.Hkv * gr.n : 0;
  return q;
}
// Merge of the split partials: workgroup (s, g, row block) combines
//   O = sum_sp 2^(m_sp - M) O_sp / sum_sp 2^(m_sp - M) l_sp,  M = max_sp m_sp
// for RB rows of the (sequence, kv head) group, D/4 threads per row, one float4 each.
// SB: splits whose loads are issued together (the host sizes it to the plan's split count).
template <bool BF16, int D, int SB>
__global__ __launch_bounds__(256) void block_attn_merge_kernel(AttnArgs a) {
  constexpr int EB = BF16 ? 2 : 4;
  constexpr int TPR = D / 4;       // threads per row
  constexpr int RB = 256 / TPR;    // rows per workgroup
  const int nrb = a.Mpad / RB + ((a.Mpad % RB) ? 1 : 0);
  const int rb = blockIdx.x % nrb;
  const int sg = blockIdx.x / nrb;
  const int s = sg / a.Hkv, g = sg % a.Hkv;
  const int qoff = ld_uniform(a.q_offsets, s);  // issued with the lengths, not after the merge
  int B;
  [[maybe_unused]] int mw = rb * RB;  // fp32: the workgroup's first row within the partial slots
  int2 ps;
  if constexpr (BF16) {
    ps = attn_pair_slots(a, s, g, B);
  } else {  // the split kernel's numbering: splits of each pair's groups, sequence by sequence
    static_assert(RB <= 16, "a workgroup's rows lie in one m-tile");
    const int lane = threadIdx.x & 63, per = ld_uniform(a.plan, 0);
    int before = 0;
    B = 0;
    ps = int2{0, 0};
    for (int c0 = 0; c0 <= s; c0 += 64) {
      const F32Seq q = f32_seq(a, c0 + lane);
      const int n = f32_splits(q.tiles, q.weight, per), incl = before + wave_scan_i(n * q.pairs);
      if (s < c0 + 64) {
        const int l = s - c0;
        B = __builtin_amdgcn_readlane(q.B, l);
        const int ns = __builtin_amdgcn_readlane(n, l), base = __builtin_amdgcn_readlane(incl - n * q.pairs, l);
        const F32Groups gr = f32_groups(plan_mtiles(a.G, B), a.group_mt);
        const int grp = min(mw / (16 * max(gr.mt, 1)), gr.n - 1);
        mw -= grp * 16 * gr.mt;
        ps = int2{base + (g * gr.n + grp) * ns, B > 0 ? ns : 0};
      }
      before = __builtin_amdgcn_readlane(incl, 63);
    }
  }
  const int nsplit = ps.y;
  if (nsplit <= 1) return;  // no block, or written directly by the split kernel
  const int M = a.G * B;
  const int m = rb * RB + threadIdx.x / TPR;
  if (m >= M) return;
  const int d = (threadIdx.x % TPR) * 4;
  const int rows = BF16 ? a.Mpad : a.part_rows;  // of a partial slot
  const size_t wbase = (size_t)ps.x * rows + (BF16 ? m : mw + (int)threadIdx.x / TPR);  // row m of split 0
  // online merge over batches of SB splits whose loads are issued together (clamped, no
  // per-load branch): one memory round trip per batch instead of one per split
  float mx = -INFINITY, lsum = 0.f;
  f32x4 acc{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < nsplit; s0 += SB) {
    float2 ml[SB];
    f32x4 po[SB];
#pragma unroll
    for (int k = 0; k < SB; ++k) {
      const size_t r = wbase + (size_t)min(s0 + k, nsplit - 1) * rows;
      ml[k] = a.part_ml[r];
      po[k] = *reinterpret_cast<const f32x4 *>(a.part_o + r * D + d);
    }
#pragma unroll
    for (int k = 0; k < SB; ++k) {
      if (s0 + k >= nsplit || ml[k].x == -INFINITY) continue;  // a split with no visible key
      const float mn = fmaxf(mx, ml[k].x);
      const float wo = (mx == -INFINITY) ? 0.f : fast_exp2(mx - mn);
      const float wn = fast_exp2(ml[k].x - mn);
      lsum = lsum * wo + ml[k].y * wn;
      acc = acc * wo + po[k] * wn;
      mx = mn;
    }
  }
  const f32x4 o = acc * (1.f / lsum);
  char *orow = reinterpret_cast<char *>(a.out) + ((size_t)(qoff + m / a.G) * a.Hq + g * a.G + m % a.G) * D * EB;
  if constexpr (BF16)
    *reinterpret_cast<uint2 *>(orow + d * EB) = uint2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
  else
    *reinterpret_cast<f32x4 *>(orow + d * EB) = o;
}

#endif  // __HIPCC__

}  // namespace sdb
