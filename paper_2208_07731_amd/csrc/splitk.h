// Tiles and split-K factors of the adjoint's products over grid rows: host
// arithmetic only, so that it can be checked without a GPU.
#pragma once

#include <stdint.h>

namespace isdf {

constexpr int MAX_SPLITS = 32;

// Tile edge and split-K factor of a product.
struct TilePlan {
  int tile, splits;
};

// Output tiles of edge `tile` of an M x N product (M == N, the tiles on or
// below the diagonal only, when `lower`).
static inline int64_t out_tiles(int64_t M, int64_t N, int64_t tile, int lower) {
  const int64_t tm = (M + tile - 1) / tile, tn = (N + tile - 1) / tile;
  return lower ? tm * (tm + 1) / 2 : tm * tn;
}

// Slices that an M x N product of K-deep sums (its lower tiles only when `lower`)
// takes at least: a slice is one chain of additions, and fewer, longer chains are
// less accurate.  As many as 128-wide tiles at two workgroups per CU are fastest
// with; by time alone splits_for takes a quarter of them in places, which put FP32
// gradients of 40^3 points, 256 orbitals off by 6.5e-7 instead of 4.8e-7 and FP64
// ones of 24^3, 200 points by 1.6e-15 instead of 1.1e-15.
static inline int least_splits(int64_t M, int64_t N, int lower, int64_t K, int slots, int cap) {
  const int64_t tiles = out_tiles(M, N, 128, lower);
  const double t_row = 2.0 * 128 * 128 / (60e12 / slots), bw = 4e12;
  int best = 1;
  double best_t = 0.0;
  for (int s = 1; s <= cap; s = s < 8 ? 8 : s + 8) {
    if (s > 1 && (K + s - 1) / s < 512) break;
    const double waves = (double)((tiles * s + slots - 1) / slots);
    const double t = waves * ((double)K / s) * t_row + (s > 1 ? s * (double)M * (double)N * 16.0 / bw : 0.0);
    if (s == 1 || t < best_t * (1.0 - 1e-9)) {
      best = s;
      best_t = t;
    }
  }
  return best;
}

// Tile and split-K factor of such a product: 1 or a multiple of 8 (one K slice per
// XCD at a time) from least_splits up to `cap`, slices of at least 4 tile edges of
// rows, chosen to minimise the modelled time ceil(tiles s / CUs) (K / s) t_row +
// s M N 16 B / bw, i.e. whole rounds of workgroups against the partial sums' write
// and read.  A round of one workgroup per CU runs at about the rate of two (the
// matrix cores bound both), hence CUs and not resident workgroups.  Small outputs
// get 64-tiles: 256 x 256 lower tiles over 13824 rows 96 us on 128-tiles, 39 on
// these; 512 x 64 over 13824 rows 98 and 29.
static inline TilePlan splits_for(int64_t M, int64_t N, int lower, int64_t K, int slots, int cap) {
  const int64_t cus = slots / 2 > 0 ? slots / 2 : 1;
  const double bw = 4e12;  // B/s for the partials
  const int least = least_splits(M, N, lower, K, slots, cap);
  TilePlan best{128, least};
  double best_t = -1.0;
  for (int tile = 128; tile >= 64; tile /= 2) {
    const int64_t tiles = out_tiles(M, N, tile, lower);
    const double t_row = 2.0 * tile * tile / (60e12 / (double)cus);  // s per k-row and tile
    for (int s = least; s <= cap; s = s < 8 ? 8 : s + 8) {
      if (s > 1 && (K + s - 1) / s < 4 * tile) break;
      const double rounds = (double)((tiles * s + cus - 1) / cus);
      double t = rounds * ((double)K / s) * t_row + (s > 1 ? s * (double)M * (double)N * 16.0 / bw : 0.0);
      if (tile == 64) t *= 1.05;  // twice the operand traffic
      if (best_t < 0.0 || t < best_t * (1.0 - 1e-9)) {
        best = TilePlan{tile, s};
        best_t = t;
      }
    }
  }
  return best;
}

// Split factor of a split-engine product with `tiles` 128 x 128 output tiles
// of mn elements in total, contracted over K grid rows.  The engine holds one
// workgroup per CU (slots / 2 of them, slots counting two FP64 tiles per CU),
// so a launch takes ceil(tiles s / CUs) waves of workgroups: the factor is the
// power of two up to `cap`, with K slices of at least 4096 rows, that minimises
// the modelled time waves (K / s) t_row + s mn 16 B / bw (the partial sums'
// write and read), a larger one taken only for a modelled gain above 2 %.
// t_row is the measured time of one tile per K row (FP16x3 34 ns, BF16x6
// 51 ns); e.g. the 136 lower tiles of a 2048 x 2048 H over 262144 rows run in
// 9 waves of 16 slices instead of 3 waves of 4.
static inline int split_k_for(int64_t tiles, int64_t K, int64_t mn, int slots, bool bf16x6, int64_t cap) {
  const int64_t cus = slots / 2 > 0 ? slots / 2 : 1;
  const double t_row = bf16x6 ? 51e-9 : 34e-9;
  const double bw = 4e12;
  int best = 1;
  double best_t = (double)((tiles + cus - 1) / cus) * (double)K * t_row;
  for (int s = 2; s <= MAX_SPLITS && s <= cap && (K + s - 1) / s >= 4096; s *= 2) {
    const double t = (double)((tiles * s + cus - 1) / cus) * ((double)K / s) * t_row + s * (double)mn * 16.0 / bw;
    if (t < 0.98 * best_t) {
      best = s;
      best_t = t;
    }
  }
  return best;
}

// Plans the adjoint uses for blocks of `rows` rows.
struct BwdSplits {
  TilePlan h;  // Theta^T S (general) or H = G^T g G (fused, lower tiles)
  TilePlan q;  // Abar^T X per orbital set
};

// Factors the adjoint's partial buffers hold: the most that the lengths they are
// sized for take.  Nothing makes a shorter block take fewer (by time alone it may
// take 64-tiles and more, shorter slices), so each block's plan is capped by them.
struct SplitCaps {
  int h, q;
};

static inline BwdSplits bwd_splits(int64_t rows, int64_t n1, int n_mu, int n, bool fused, int slots, SplitCaps cap) {
  BwdSplits b;
  b.h = splits_for(n1, n1, fused ? 1 : 0, rows, slots, cap.h);
  b.q = splits_for(2 * (int64_t)n_mu, 2 * (int64_t)n, 0, rows, slots, cap.q);
  return b;
}

// Sizes the partial buffers by the lengths of a sweep in equal blocks, rblock
// and the grid's remainder, for both losses and both orbital sets.
static inline SplitCaps bwd_split_caps(int64_t nr, int64_t rblock, bool aliased, int n_mu, int n_phi, int n_psi,
                                       int slots) {
  const SplitCaps any{MAX_SPLITS, MAX_SPLITS};
  const int64_t n1 = aliased ? n_mu : 2 * (int64_t)n_mu;
  SplitCaps c{1, 1};
  for (int64_t rows : {rblock, nr - ((nr + rblock - 1) / rblock - 1) * rblock})
    for (int n : {n_phi, n_psi})
      for (bool fused : {false, true}) {
        const BwdSplits b = bwd_splits(rows, n1, n_mu, n, fused, slots, any);
        c.h = b.h.splits > c.h ? b.h.splits : c.h;
        c.q = b.q.splits > c.q ? b.q.splits : c.q;
      }
  return c;
}

}  // namespace isdf
