// The plans' arithmetic (the first part of csrc/attn.hpp) on the CPU: the split kernels' and the merge's walks over a
// batch, sequence by sequence where the device scans lanes.  Each check returns 0, or the line that failed.
#include "attn.hpp"

#include <set>
#include <utility>
#include <vector>

using namespace sdb;

#define NEED(x) \
  if (!(x)) return __LINE__

extern "C" int check_bal(int S, int Hkv, int G, const int *ctx, const int *B, int kt, int min_tiles) {
  std::vector<int> tiles(S), w(S), start(S * Hkv);
  int W = 0;
  for (int s = 0; s < S; ++s) {
    tiles[s] = B[s] > 0 ? (ctx[s] + B[s] + kt - 1) / kt : 0;
    w[s] = bal_weight(plan_mtiles(G, B[s]));
    for (int g = 0; g < Hkv; ++g) {
      start[s * Hkv + g] = W;
      W += bal_pair_units(tiles[s], w[s]);
    }
  }
  const int per = bal_per(W, min_tiles);
  std::vector<std::vector<int>> owner(S * Hkv);
  std::vector<int> pieces(S * Hkv, 0);
  std::set<int> slots;
  for (int p = 0; p < S * Hkv; ++p) owner[p].assign(tiles[p / Hkv], -1);
  for (int wg = 0; wg < kBalGrid; ++wg) {
    int u0 = plan_min(wg * per, W);
    const int u1 = plan_min(u0 + per, W);
    int guard = 0;
    while (u0 < u1) {
      NEED(++guard <= 2 * S * Hkv + 2);
      int p = -1;  // the pair that holds u0
      for (int q = 0; q < S * Hkv; ++q)
        if (tiles[q / Hkv] > 0 && start[q] <= u0 && u0 < start[q] + bal_pair_units(tiles[q / Hkv], w[q / Hkv])) p = q;
      if (p < 0) break;
      const int s = p / Hkv;
      const BalPiece b = bal_piece(u0, u1, start[p], tiles[s], w[s]);
      NEED(b.next > u0);
      u0 = b.next;
      if (!b.any) continue;
      NEED(0 <= b.j0 && b.j0 < b.j1 && b.j1 <= tiles[s]);
      for (int j = b.j0; j < b.j1; ++j) {
        NEED(owner[p][j] == -1);
        owner[p][j] = wg;
      }
      const BalShares sh = bal_shares(start[p], tiles[s], w[s], per);
      NEED(sh.first <= wg && wg <= sh.last);
      NEED(slots.insert(wg + p).second && wg + p < kBalGrid + S * Hkv);
      ++pieces[p];
    }
  }
  for (int p = 0; p < S * Hkv; ++p) {
    for (int o : owner[p]) NEED(o >= 0);
    if (tiles[p / Hkv] > 0) {
      const BalShares sh = bal_shares(start[p], tiles[p / Hkv], w[p / Hkv], per);
      NEED(pieces[p] == sh.last - sh.first + 1);  // consecutive slots, no hole
    }
  }
  return 0;
}

// grid: the splits the workspace has room for.  splits[0]: their number.
extern "C" int check_f32(int S, int Hkv, int G, int max_block, const int *ctx, const int *B, int grid, int *splits) {
  const int nmt_max = plan_mtiles(G, max_block);
  const int groups = (nmt_max + kF32GroupMT - 1) / kF32GroupMT, group_mt = (nmt_max + groups - 1) / groups;
  const int pairs_max = S * Hkv * groups;
  NEED(groups <= 4);
  auto seq = [&](int s, int &tiles, int &weight, int &pairs) {
    const F32Groups gr = f32_groups(plan_mtiles(G, B[s]), group_mt);
    tiles = B[s] > 0 ? (ctx[s] + B[s] + kF32KT - 1) / kF32KT : 0;
    weight = f32_weight(gr.mt);
    pairs = B[s] > 0 ? Hkv * gr.n : 0;
    return gr;
  };
  auto count = [&](int per) {
    int n = 0, t, w, p;
    for (int s = 0; s < S; ++s) {
      seq(s, t, w, p);
      n += f32_splits(t, w, per) * p;
    }
    return n;
  };
  int W = 0, t, w, p;
  for (int s = 0; s < S; ++s) {
    const F32Groups gr = seq(s, t, w, p);
    const int nmt = plan_mtiles(G, B[s]);
    NEED(gr.n >= 1 && gr.n <= groups && gr.mt <= group_mt && gr.n * gr.mt >= nmt);  // every m-tile has a group
    NEED(B[s] == 0 || (gr.n - 1) * gr.mt < nmt);                                    // and no group is empty
    W += t * w * p;
  }
  const int per0 = f32_per0(W, grid, kF32MinTiles);
  int k = 0;
  while (k < kF32Waves - 1 && count(f32_per(per0, k)) > grid) ++k;
  const int per = f32_per(per0, k), launched = f32_launch(pairs_max, grid);
  splits[0] = count(per);
  NEED(splits[0] <= launched);
  NEED(launched <= grid + pairs_max);  // the slots of the workspace
  // items densely numbered; splits of a group cover its tiles; the merge's renumbering agrees
  int item = 0;
  for (int s = 0; s < S; ++s) {
    const F32Groups gr = seq(s, t, w, p);
    if (p == 0) continue;
    const int n = f32_splits(t, w, per), base = item;
    NEED(n >= 1 && n <= t);
    for (int q = 0; q < p; ++q)
      for (int i = 0; i < n; ++i, ++item) {
        const int r = item - base, pair = r / n, g = pair / gr.n, grp = pair - g * gr.n;
        NEED(pair == q && r - pair * n == i && g < Hkv && grp < gr.n);
        NEED(base + (g * gr.n + grp) * n + i == item);
        const int k0 = (int)((long long)t * i / n), k1 = (int)((long long)t * (i + 1) / n);
        NEED(k0 < k1 && (i > 0 || k0 == 0) && (i < n - 1 || k1 == t));
      }
  }
  NEED(item == splits[0]);
  return 0;
}
