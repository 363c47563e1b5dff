// How the two gradient products of an update are cut and launched: host code that needs no device.
#pragma once
#include <cstddef>
#include <cstdint>

namespace umas {

// How the dH product of a chunk is cut along the vocabulary.  dH has tiles_r x tiles_d tiles of the whole vocabulary's K
// each; with few row tiles that is fewer long tiles than compute units, and the launch lasts as long as one of them (3.6 ms
// at V = 151 936 whether there are 64 rows or 2000).  Below kDhSliceTiles, one tile per compute unit, they are cut into about
// 256 / tiles slices, a piece per compute unit (the dW tiles behind them fill the last round); partial sums cost 256 KB a
// piece.  Gradients and the sum of the slices together with 256 / 384 / 512 / 768 pieces: 64 rows of 2048 467 / 460 / 480 / 488 us, 203 rows
// of 3584 859 / 875 / 869 / 892, 725 rows of 2048 947 / 956 / 959 / 984, 6000 rows 5.91 / 5.90 / 5.98 / 5.90 ms; whole
// tiles took 3.6 to 4 ms for the first three.  A selection that a small workspace cuts into chunks keeps whole tiles, and so the
// same bits of dH, down to chunks of half as many tiles (39 224 rows of 2048, whole and sliced: chunks of 256 tiles 57.8 and
// 58.2 ms, 192 58.8 and 59.3, 160 59.6 and 59.5, 128 61.0 and 59.7, 96 71.9 and 61.6, 8 571 and 141).
constexpr int kDhSliceTiles = 256;
inline int64_t dh_tiles(int64_t rows, int d) { return (rows + 255) / 256 * ((d + 255) / 256); }
// decided by the rows of the call and its chunks, not by those of the last chunk, which may have fewer
inline bool slices_dh(int64_t n_sel, int64_t chunk_rows, int d) { return dh_tiles(chunk_rows, d) < (chunk_rows < n_sel ? kDhSliceTiles / 2 : kDhSliceTiles); }
// dW of one block of rows gets a launch of its own (k_dw_short) where it is large: its stores, which everything else then waits for, are longer than the launch
// and the dH tiles' uneven end that it pays for.  Update in two launches over one, geometric mean over 129 to 256 rows, dW of 0.5, 0.7, 0.9, 1.1, 1.3
// and 1.6 GiB: 2048 columns 1.019, 1.012, 1.008, 0.994 (151 936 entries are 1.16), 2560 1.025, 1.039, 1.017, 0.976, 0.975, 0.957, 3584
// 0.931, 0.920, 0.916, 0.940, 0.952, 0.966, 8192 0.981, 0.983, 0.988, 0.938, 0.949, 0.965.  65 to 128 rows, whose dH tiles are half as long: 2048 columns
// 1.044, 1.031, 0.998, 1.009, 2560 1.052, 1.032, 1.018, 0.975, 1.000, 0.973, 3584 0.983, 0.970, 0.970, 0.954, 0.954, 0.977, 4096 above 1.25 GiB
// 0.978, 4608 1.009, 8192 1.009 to 1.017, 16 384 1.02; 30 rows of 2048 508 and 517 us, 3072 722 and 731.  More than a block: 300 rows of 2048 876 and
// 922, 725 of 3584 2262 and 2258, 2500 6594 and 8070.
constexpr int64_t kDwApartBytes = int64_t{1} << 30;
inline bool dw_apart(int64_t n_sel, int d, int V) {
  const int64_t bytes = static_cast<int64_t>(V) * d * 4;
  if (n_sel <= 128) return n_sel > 64 && d <= 4096 && bytes >= kDwApartBytes / 4 * 5;
  return n_sel <= 256 && bytes >= kDwApartBytes;
}
struct DhPlan {
  int slices, voc_blks;
};
inline size_t dh_part_bytes(const DhPlan& p, int tiles_r, int tiles_d) {
  return p.slices > 1 ? static_cast<size_t>(p.slices) * tiles_r * tiles_d * (256 * 256 * sizeof(float)) : 0;
}
// `alone`: nothing fills a last round, there must be none
inline DhPlan plan_dh(int64_t tiles_r, int64_t tiles_d, int tiles_v, size_t room, bool alone = false) {
  int want = static_cast<int>((kDhSliceTiles + (alone ? 0 : tiles_r * tiles_d - 1)) / (tiles_r * tiles_d));
  const size_t one = static_cast<size_t>(tiles_r * tiles_d) * (256 * 256 * sizeof(float));
  if (static_cast<size_t>(want) > room / one) want = static_cast<int>(room / one);
  if (want > tiles_v) want = tiles_v;
  if (want < 2) return DhPlan{1, tiles_v};
  const int blks = (tiles_v + want - 1) / want;
  return DhPlan{(tiles_v + blks - 1) / blks, blks};
}
// What a chunk of `rows` of the call's n_sel rows gets in `room` bytes for partial sums.  dW gets its launch only where the whole rounds of dH slices that this
// asks for leave few compute units idle; else the plan is that of both products in one launch, whose last round dW fills.
struct GradPlan {
  DhPlan dh;
  bool dw_apart;
};
inline GradPlan plan_gradients(int64_t n_sel, int64_t rows, int d, int V, size_t room) {
  const int64_t tiles_r = (rows + 255) / 256, tiles_d = (d + 255) / 256;
  const int tiles_v = (V + 255) / 256;
  if (dw_apart(n_sel, d, V)) {
    const DhPlan p = plan_dh(tiles_r, tiles_d, tiles_v, room, true);
    if (p.slices * tiles_r * tiles_d >= kDhSliceTiles * 3 / 4) return GradPlan{p, true};
  }
  return GradPlan{plan_dh(tiles_r, tiles_d, tiles_v, room), false};
}

}  // namespace umas
