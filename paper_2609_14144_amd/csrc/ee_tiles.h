// Tiles of the batched pass's products (ee_mm.h) and the choice among them.
// Host code without HIP: the choice is also compiled and examined on its own.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace ee {

// The tile and K split of a product. Every candidate's time is estimated
// (microseconds; constants fitted to a sweep of tiles and splits over the
// products of three decoder widths, 16 to 1024 positions, where the choice
// costs 1.7% over the best on average):
//   * a unit runs the tile's workgroups in rounds of `occ` (what registers
//     and LDS allow); a step of a round takes the matrix-core time of its
//     workgroups or, if longer, the latency of one workgroup's step;
//   * no less than the weights' read from HBM, nor than the tiles' reads of
//     weights and activations from the caches;
//   * the stores of the outputs, and for the residual products the next
//     kernel's reads of the K slices.
struct MmTile {
  int rb, cp, nw, pf, kg, occ;
};
template <typename WT>
double mm_time(const MmTile& t, int P, int N, int K, int splits, bool resid, int n_cu) {
  constexpr double kStep = 0.02127 * (sizeof(WT) == 2 ? 1.0 : 512.0 / 96.0);  // cycles of a step's instructions
  constexpr double wb = sizeof(WT), xb = sizeof(WT) == 2 ? 6.0 : 4.0;
  const double mfma = kStep * t.rb * t.cp * t.nw * t.kg;
  const double lat = (t.pf == 1 ? 0.733 : 0.262) + 0.377 * mfma / t.kg;
  const int tiles = ((N + 16 * t.rb * t.nw - 1) / (16 * t.rb * t.nw)) * ((P + 16 * t.cp - 1) / (16 * t.cp)) * splits;
  const int per_cu = (tiles + n_cu - 1) / n_cu, full = per_cu / t.occ, rest = per_cu % t.occ;
  const int steps = ((K + 63) / 64 + splits * t.kg - 1) / (splits * t.kg);
  const double round = full * std::max(t.occ * mfma, lat) + (rest ? std::max(rest * mfma, lat) : 0.0);
  const double bytes = wb * N * K * ((P + 16 * t.cp - 1) / (16 * t.cp)) +
                       xb * P * K * ((N + 16 * t.rb * t.nw - 1) / (16 * t.rb * t.nw));
  const double out = 4.0 * splits * P * N;
  return 3.2 + std::max({round * steps, wb * N * K / 5.8e6, bytes / 14.8e6}) + out / 8.5e6 + (resid ? out / 5e6 : 0.0);
}

// 16 positions: the weight stream counts, four steps of it in flight. More
// positions: 32 to 64 per workgroup. Eight waves of three row blocks share the
// activations of 64 positions among 384 rows, the fewest cache reads. The QKV
// product of few positions has few tiles and whole sums to finish: four groups
// of waves share a tile's K. fp32 weights come with narrow models (at most 512
// wide), whose few steps want many small tiles.
template <typename WT>
struct MmTiles;
template <>
struct MmTiles<uint16_t> {
  static constexpr MmTile t[] = {{1, 1, 8, 4, 1, 3}, {1, 2, 4, 4, 1, 3}, {2, 2, 4, 2, 1, 4}, {3, 2, 4, 2, 1, 3},
                                 {4, 2, 4, 2, 1, 2}, {3, 3, 4, 2, 1, 2}, {3, 4, 4, 1, 1, 2}, {3, 4, 8, 1, 1, 1},
                                 {2, 4, 8, 1, 1, 1}, {1, 1, 2, 2, 4, 2}, {1, 2, 2, 2, 4, 1}};
};
template <>
struct MmTiles<float> {
  static constexpr MmTile t[] = {{1, 1, 4, 2, 1, 4}, {1, 1, 2, 2, 4, 2}, {1, 2, 4, 2, 1, 3}, {2, 2, 4, 2, 1, 2}};
};
struct MmChoice {
  size_t tile;
  int splits;  // 0: the partial sums do not fit the workspace
};
// resid: the product stores K slices (ws_floats of room), which the next kernel adds; qkv: the QKV product
template <typename WT>
MmChoice mm_choose(bool resid, bool qkv, int P, int N, int K, size_t ws_floats, int n_cu) {
  constexpr size_t kTiles = sizeof(MmTiles<WT>::t) / sizeof(MmTile);
  const int steps = (K + 63) / 64;
  int most = 1;
  if (resid) {
    const size_t per = static_cast<size_t>(P) * N;
    most = static_cast<int>(std::min<size_t>(16, ws_floats / per));
    if (most < 1) return MmChoice{0, 0};
  }
  MmChoice best{kTiles, 0};
  double best_t = 0.0;
  for (size_t i = 0; i < kTiles; ++i) {
    const MmTile& t = MmTiles<WT>::t[i];
    if ((t.cp == 1) != (P <= 16) || (t.kg > 1 && !qkv)) continue;
    // Three position blocks: measured at 350 to 1024 positions this tile took 1.06 to 1.8 times the best one's time
    // in 35 of 36 products, and the estimate does not always see it; it pays below (9728 x 896, 200 positions: 16.0
    // against 16.8 us).
    if (t.cp == 3 && P > 256) continue;
    for (int sp : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16}) {
      if (sp > most || (sp > 1 && steps / sp < 4) || (t.kg > 1 && steps < 2 * t.kg)) break;
      const double us = mm_time<WT>(t, P, N, K, sp, resid, n_cu);
      // of equals the tile of more waves, which reads less from the caches (1024 positions: gate/up 139 against
      // 150 us, down 64 against 75)
      if (best.tile == kTiles || us < best_t || (us == best_t && t.nw > MmTiles<WT>::t[best.tile].nw)) {
        best = MmChoice{i, sp};
        best_t = us;
      }
    }
  }
  return best;
}

}  // namespace ee
