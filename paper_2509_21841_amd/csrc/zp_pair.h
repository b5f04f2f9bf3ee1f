// Launches that leave much of the chip idle: which of two kernels they take, and the tile table of the one that puts two
// waves on every 16 query rows (host side).
#pragma once
#include <algorithm>
#include <cstring>

#include "zp_common.h"

// Whether a launch's sequences go into its arguments (zp_put_seq) where they fit and the table of its tiles does not, or would be
// written to device memory for the sake of the work counters only. That saves the launch in front that writes the table (3.5 us where
// it is uploaded, 4 to 13 where it is worked out on the device), and gives up claimed items, which launches of 200 us and more
// lose more by. `sum`: key tiles of 64 that the query blocks of 128 see; the limits are on key tiles x heads x head dimension. Of 60
// random batches (3000 to 96000 tokens, 4/2 to 64/8 heads) the 23 forwards under the limit and over 112 tiles or 1024 items are 2 to 7 % faster,
// the 26 without allocation up to 10 % (one 0.3 % slower), the 11 backwards up to 5 %; the next ones
// above the limits lose up to 4 %. us, table / arguments:
//    d   heads   tokens            in arguments                                           not
//    64   8/2    26191             forward 97.6 / 94.0, without allocation 98.9 / 94.0
//    64   4/4    90755             forward 137.0 / 133.3, without allocation 147.0 / 133.3
//   128   4/2     8895             backward 147.4 / 143.6
//    64  32/32   12599             forward 116.9 / 113.0                                  backward 353.6 / 367.4
//    64  32/8    39879                                                                    forward 427.1 / 437.2
constexpr float ZP_SEQS_FWD = 5.3e6f, ZP_SEQS_NOALLOC = 1e7f, ZP_SEQS_BWD = 1.5e6f;
inline bool zp_seqs_pay(int64_t sum, int Hq, int d, float most) { return (float)sum * (float)Hq * (float)d <= most; }

// key tiles of 64 that a tile's last row sees
inline int zp_key_tiles(const zp_tile &t) {
  int64_t n = (int64_t)t.q_pos0 + t.q_rows - t.k_pos0;
  n = n < 0 ? 0 : n > t.k_len ? t.k_len : n;
  return (int)((n + 63) / 64);
}

// The later (half = 1) or earlier 64 rows of a tile.
inline zp_tile zp_half_tile(zp_tile t, int half) {
  t.q_tok0 += 64 * half; t.q_pos0 += 64 * half; t.out_row0 += 64 * half;
  t.q_rows = std::min(64, t.q_rows - 64 * half);
  return t;
}

// Order of n tiles by cost, heaviest first, equal ones as they come.
inline void zp_by_cost(const int *cost, int n, int *order) {
  constexpr int MOST = 255;
  int at[MOST + 2] = {}, most = 0;
  for (int i = 0; i < n; i++) most = std::max(most, cost[i]);
  if (most > MOST) {
    for (int i = 0; i < n; i++) order[i] = i;
    std::sort(order, order + n, [&](int a, int b) { return cost[a] != cost[b] ? cost[a] > cost[b] : a < b; });
    return;
  }
  for (int i = 0; i < n; i++) at[most - cost[i] + 1]++;
  for (int c = 0; c < most; c++) at[c + 1] += at[c];
  for (int i = 0; i < n; i++) order[at[most - cost[i]]++] = i;
}

// Estimated time of a launch in microseconds, from its tiles' costs (descending, each `heads` times): one workgroup per CU up to
// 256 items; beyond, the lightest of the first 256 are followed by the heaviest of the rest.
struct zp_pair_cost {
  float wg, tile, launch, item;  // per workgroup, per key tile, per launch, per item of the launch
  float share;                   // whole items: what a second workgroup on the CU adds of its own time (pairs: 1)
};
inline float zp_pair_estimate(const zp_pair_cost &c, const int *cost, int n, int heads, bool pairs) {
  const int items = n * heads;
  const float head = c.launch + c.item * (float)items;
  auto dur = [&](int i) { return c.wg + c.tile * (float)cost[i / heads]; };
  float most = dur(0);
  if (items <= 256) return head + most;
  if (items <= 512) {
    // tiles of item k or 255 - k, and of item 256 + k, and what is left of their heads
    const int step = pairs ? -1 : 1;
    int a = pairs ? 255 / heads : 0, a_left = pairs ? 255 % heads + 1 : heads, b = 256 / heads, b_left = heads - 256 % heads;
    for (int k = 256; k < items;) {
      const float da = c.wg + c.tile * (float)cost[a], db = c.wg + c.tile * (float)cost[b];
      most = std::max(most, pairs ? da + db : da + c.share * db);
      const int run = std::min(a_left, b_left);
      k += run;
      if ((a_left -= run) == 0) { a += step; a_left = heads; }
      if ((b_left -= run) == 0) { b++; b_left = heads; }
    }
    return head + most;
  }
  float sum = 0.f;
  for (int i = 0; i < n; i++) sum += c.wg + c.tile * (float)cost[i];
  sum *= (float)heads / 256.f;
  return head + (pairs ? std::max(most, 1.03f * sum + 0.5f * dur(items - 1)) : std::max(most + c.share * dur(256), sum * 0.5f * (1.f + c.share)));
}

// Whether a launch (n tiles of 128 rows in the launch arguments, `behind` tiles of another launch behind them) takes the kernel
// with two waves per 16 rows, and how its table is laid out then. With a CU for every workgroup that is always the faster
// one, the launch being its longest chain; beyond, its estimate has to be below `margin` of the other kernel's, or below
// `halves` where the table does not fit and so is not in order of cost.
inline zp_pair_mode zp_take_pairs(zp_inline_tiles &inl, int &n, int behind, int Hkv, int grp, const zp_pair_cost &whole, const zp_pair_cost &pair,
                                  float margin, float halves) {
  const int heads = Hkv * grp;
  zp_tile *tiles = inl.t;
  if (n < 1 || n > ZP_INLINE_TILES || (int64_t)n * heads > 1024) return ZP_PAIR_NONE;
  int m = 0;
  for (int i = 0; i < n; i++) m += tiles[i].q_rows > 64 ? 2 : 1;
  if (m * heads > 1024) return ZP_PAIR_NONE;
  const bool fits = m + behind <= ZP_INLINE_TILES;
  // the 64-row tiles, the later rows of a block first: 2 * tile + half
  int half[2 * ZP_INLINE_TILES], order[2 * ZP_INLINE_TILES];
  for (int i = 0, k = 0; i < n; i++) {
    if (tiles[i].q_rows > 64) half[k++] = 2 * i + 1;
    half[k++] = 2 * i;
  }
  if (((fits ? m : 2 * n) * Hkv + 7) / 8 * grp > 32) {
    // decided by the costs alone: the table is written where the pairs are taken (28 sequences of 256 tokens, 4/2 heads, which
    // are not: 3.9 us with a table sorted beforehand, 1.0 now)
    int cost[2 * ZP_INLINE_TILES], sorted[2 * ZP_INLINE_TILES], order128[ZP_INLINE_TILES];
    for (int i = 0; i < n; i++) cost[i] = zp_key_tiles(tiles[i]);
    zp_by_cost(cost, n, order128);
    for (int i = 0; i < n; i++) sorted[i] = cost[order128[i]];
    const float other = zp_pair_estimate(whole, sorted, n, heads, false);
    for (int k = 0; k < m; k++) cost[k] = zp_key_tiles(zp_half_tile(tiles[half[k] / 2], half[k] & 1));
    zp_by_cost(cost, m, order);
    for (int k = 0; k < m; k++) sorted[k] = cost[order[k]];
    if (!(zp_pair_estimate(pair, sorted, m, heads, true) < (fits ? margin : halves) * other)) return ZP_PAIR_NONE;
  } else {
    for (int k = 0; k < m; k++) order[k] = k;
  }
  if (!fits) return ZP_PAIR_HALVES;
  zp_tile table[ZP_INLINE_TILES];
  for (int k = 0; k < m; k++) table[k] = zp_half_tile(tiles[half[order[k]] / 2], half[order[k]] & 1);
  std::memmove(tiles + m, tiles + n, (size_t)behind * sizeof(zp_tile));
  std::memcpy(tiles, table, (size_t)m * sizeof(zp_tile));
  n = m;
  return ZP_PAIR_TILES;
}

// The forward's two kernels. Constants fitted to 850 launches whose tables fit; the estimates are 4 and 5 % off in the mean of 3996 others
// (2/1 to 64/8 heads; equal, ragged and lognormal lengths, 16 to 13600 tokens). Of the 3361 launches of these that take the pairs 12 are 2
// to 8 % slower with them; all 3996 take 0.78 of the time (geometric mean), and the 121 of the 3361 whose tables do not
// fit 0.77. A limit of 0.91 leaves 8 such losses but gives up 2 to 9 % in 11 launches at d = 128 alone. n sequences of L tokens, us,
// whole / pairs:
//    d   heads    L    taken: pairs                      not taken
//    64   4/4    300   n =  1:   8.0 /  6.1
//    64   4/4   4000   n =  1:  51.9 / 33.5              64/8, L =  762, n = 2:  17.7 / 24.2
//   128   4/4   1000   n =  4:  23.2 / 15.4              64/8, L =  894, n = 2:  27.8 / 35.1
//   128   8/2   2085   n =  1:  41.4 / 27.1              16/4, L =  200, n = 20: 21.9 / 26.2
//   128   4/4   1623   n =  5:  34.8 / 37.7 (as halves, the worst)
inline void zp_plan_fwd_pair(zp_attn_params &p, int d) {
  static const zp_pair_cost whole[2] = {{2.95f, 0.769f, 1.74f, 0.0023f, 0.345f}, {2.20f, 1.074f, 3.19f, 0.0032f, 0.536f}};
  static const zp_pair_cost pair[2] = {{2.03f, 0.471f, 1.95f, 0.0022f, 1.f}, {2.63f, 0.660f, 1.64f, 0.0027f, 1.f}};
  if (p.tiles == nullptr && p.n_seq == 0) p.pair = zp_take_pairs(p.inl, p.n_tiles, 0, p.Hkv, p.grp, whole[d == 128], pair[d == 128], 0.93f, 0.83f);
}

// The dQ kernels, whose tiles have the dK/dV tiles behind them. Constants fitted to 3446 launches (2/1 to 64/8 heads; equal,
// ragged and lognormal lengths, 16 to 7000 tokens); the estimates are 4 to 5 % off in the mean. Of the 2642 launches that take the
// pairs 3 are 2 to 3 % slower with them and none is more; all 3446 take 0.86 of the time (geometric mean). n sequences, us, whole / pairs:
//    d   heads   tokens                              taken: pairs      not taken
//    64   4/4     954,               n =  1:   17.7 / 14.3
//    64   4/4    3780,               n =  1:   55.6 / 44.5
//   128   4/4     983,               n =  1:   26.3 / 20.5
//   128   4/4    3907,               n =  1:   84.8 / 67.5
//   128  16/16    830, longest   88, n = 17:                      9.8 / 11.5
//   128   4/4    5677, equal,        n =  7:                     23.7 / 29.0   (as halves)
inline void zp_plan_dq_pair(zp_bwd_params &p, int d) {
  static const zp_pair_cost whole[2] = {{-0.273f, 0.864f, 4.78f, 0.00305f, 0.584f}, {1.36f, 1.29f, 4.29f, 0.00569f, 0.592f}};
  static const zp_pair_cost pair[2] = {{2.18f, 0.691f, 1.42f, 0.0015f, 1.f}, {3.62f, 1.02f, 1.34f, 0.00266f, 1.f}};
  if (p.dq_tiles == nullptr && p.n_seq == 0)
    p.dq_pair = zp_take_pairs(p.inl, p.n_dq_tiles, p.n_kv_tiles, p.Hkv, p.grp, whole[d == 128], pair[d == 128], 0.91f, 0.76f);
}

// Whether dQ and dK/dV, which take the kernels for launches that leave part of the chip idle (their tiles in the launch arguments), go
// in one launch behind a small one for the row terms: the two leave different parts of the chip idle, and each waits for its longest
// chain. Workgroups take a CU each there. With a CU for all of them it is faster (one key tile at d = 64 and more than 160 workgroups:
// 9.7 / 10.5 us); beyond, where the longest chain is a third longer than a CU's share of all. At d = 128 also with shares of 9 us and more; at 64, where two workgroups of the dK/dV
// kernel by itself share a CU, not. Constants: dQ as above, dK/dV as in dkdv_kernel_for. Of 270 random launches (2/1 to 64/8 heads, 100 to
// 14000 tokens) 240 take it, for 0.77 of the time in the mean, one of them 1.5 % slower. n sequences, us, two launches / one and the small one:
//    d   heads   tokens                              taken              not taken
//    64   4/2    1511,               n =  1:   42.4 / 26.3
//    64   2/1    4919, longest 3033, n =  3:   77.1 / 46.3
//    64  32/32    322, longest  126, n =  4:                      13.1 / 15.7
//    64   8/8    4002, longest 2876, n =  2:                      77.7 / 88.1
//   128   4/2    1218, longest  329, n =  8:   23.8 / 16.6
//   128   2/1    4001, longest 3681, n =  4:  135.7 / 79.4
//   128  16/4     272, longest   17, n = 16:                      12.3 / 13.4
inline bool zp_take_both(const zp_bwd_params &p, int d) {
  if (!p.dq_pair || !p.kv_split || p.dq_tiles != nullptr) return false;
  static const float dq_wg[2] = {2.18f, 3.62f}, dq_tile[2] = {0.691f, 1.02f}, kv_wg[2] = {1.55f, 2.82f}, kv_it[2] = {0.831f, 1.255f};
  const int c = d == 128;
  float longest = 0.f, sum = 0.f;
  int64_t n = 0;
  for (int i = 0; i < p.n_dq_tiles; i++)
    for (int half = 0; half < (p.dq_pair == ZP_PAIR_HALVES && p.inl.t[i].q_rows > 64 ? 2 : 1); half++) {
      const float t = dq_wg[c] + dq_tile[c] * (float)zp_key_tiles(p.dq_pair == ZP_PAIR_HALVES ? zp_half_tile(p.inl.t[i], half) : p.inl.t[i]);
      longest = std::max(longest, t);
      sum += t * (float)p.Hq;
      n += p.Hq;
    }
  for (int i = 0; i < p.n_kv_tiles; i++) {
    const zp_tile &k = p.inl.t[p.n_dq_tiles + i];
    const int parts = (k.k_len + 31) / 32, its = ((k.q_rows + 31) / 32 * p.grp + 3) / 4;
    const float t = kv_wg[c] + kv_it[c] * (float)its;
    longest = std::max(longest, t);
    sum += t * (float)(parts * p.Hkv);
    n += parts * p.Hkv;
  }
  const float share = sum / 256.f;
  return n <= (longest < 3.f ? 160 : 256) || (n > 256 && share <= 0.75f * longest) || (d == 128 && share >= 9.f);
}

// Whether a forward launch at head dimension 128 (n query blocks that see `sum` key tiles of 64 in all, one of them `longest`, each
// `heads` times) takes the kernel of three workgroups per CU. A CU does more with three, and each of them is slower: it pays where a
// CU's share of the launch is several times the longest item, so that nothing waits for that one. Of 278 random launches (2/1 to 64/8
// heads, 600 to 131072 tokens) with a share of 4 and more of the longest 155 take it, 1.06 times faster in the mean; 4 are 1 to 2 %
// slower. From 2 to 4 it is 0.6 % faster in the mean and up to 12 % slower, below 6 % slower in the mean. An item's fixed costs count
// as three key tiles.
inline bool zp_fwd_turns(int d, int64_t sum, int64_t n, int64_t longest, int heads) {
  return d == 128 && (sum + 3 * n) * heads >= 4 * 256 * (longest + 3);
}
