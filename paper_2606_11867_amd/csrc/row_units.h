// How a launch of the row GEMMs is cut into units of work, and the layout of
// its workspace. Plain arithmetic: the kernels evaluate it on the device, the
// launchers on the host.
#pragma once

#include <stddef.h>

namespace foremoe {

#ifndef FM_ROWS_BK
#define FM_ROWS_BK 64
#endif
#ifndef FM_SPLIT_MAX
#define FM_SPLIT_MAX 4
#endif
constexpr int kSplitMax = FM_SPLIT_MAX;  // pieces per tile at most (2..4)

#define FM_INLINE __attribute__((always_inline)) constexpr

// Row tiles of a slot: 256 rows each; what is left over is a tile of its own,
// of 256 rows if more than 128 are left, of 128 ("short") if more than 64,
// else of 64 ("thin").
struct SlotTiles {
  int full, is_short, is_thin;
};
FM_INLINE SlotTiles slot_tiles(int rows) {
  const int left = rows % 256;
  return {rows / 256 + (left > 128), left > 64 && left <= 128, left > 0 && left <= 64};
}

// Work of one GEMM of a launch: tiles (row tile x 256 columns) in a fixed
// order, the 256-row ones first. The last `r` tiles may be cut: those of 256
// rows into `h` halves of 128 columns, and then every (half) tile into `s`
// pieces along K, each a unit of its own.
struct PhaseUnits {
  int nt;        // column tiles
  int kt;        // k-steps
  int small;     // tiles of 128 or 64 rows
  int plain;     // tiles that are not cut
  int full_cut;  // 256-row tiles among the cut ones
  int h, s;
  int total;     // units
};

// Units of a GEMM that come from tiles cut along K, at most: a cut that fills
// the chip measured slower than the round uncut and spread out.
FM_INLINE int cut_units(int G) { return 7 * G / 8; }

// nfull, nsmall: row tiles of 256 rows and of fewer. r: the tiles of a last,
// partial round (all tiles, if they make less than one round of the G
// workgroups).
FM_INLINE PhaseUnits phase_units(int nfull, int nsmall, int N, int K, int G, int r, bool ws) {
  PhaseUnits u{};
  u.nt = (N + 255) / 256;
  u.kt = K / FM_ROWS_BK;
  u.small = nsmall * u.nt;
  const int tiles = nfull * u.nt + u.small;
  r = r < tiles ? r : tiles;
  u.full_cut = r > u.small ? r - u.small : 0;
  const int rs = r - u.full_cut;
  // A partial last round that leaves the chip less than half busy is cut
  // along N first: two half-width tiles on two workgroups, with no partial
  // sums (measured faster than cutting the same round along K).
  u.h = (u.full_cut > 0 && 8 * (2 * u.full_cut + rs) <= 7 * G) ? 2 : 1;
  // Then, with the workspace, along K: as many pieces as keep at most
  // cut_units busy, none shorter than 16 k-steps (8 for the small tiles,
  // whose partial sums are a quarter). Beside halves a small tile counts as
  // two unless K is long: the halves bound such a round, and pieces of 16
  // k-steps gain little on it (layer of 512 tokens, 12 tiles of 256 rows and 48
  // small ones, K = 2048, in 2 pieces 59.8 us, uncut 61.4) for sums in another
  // fp32 order than the tiles alone give. Long ones gain more (Mixtral-8x7B
  // share, 8192 rows, K = 14336 880 -> 935 us without, K = 28672 1682 -> 1792).
  u.s = 1;
  const int n = u.full_cut * u.h + rs;
  if (ws && n > 0 && (u.full_cut == 0 || (u.h == 2 && u.kt >= 32))) {
    int s = cut_units(G) / (u.kt >= 64 ? n : u.h * r);
    s = s < kSplitMax ? s : kSplitMax;
    const int most = u.kt / (u.full_cut ? 16 : 8);
    s = s < most ? s : most;
    u.s = s < 1 ? 1 : s;
  }
  u.plain = tiles - r;
  u.total = u.plain + n * u.s;
  return u;
}

// A launch of one GEMM (phases 1 or 2) or both (3) on G workgroups.
struct LaunchUnits {
  PhaseUnits u0, u1;
};
FM_INLINE LaunchUnits launch_units(int nfull, int nsmall, int N0, int K0, int N1, int K1, int phases, int G,
                                   bool ws) {
  const bool pair = phases == 3;
  const int rows = nfull + nsmall;
  const int t0 = rows * ((N0 + 255) / 256), t1 = rows * ((N1 + 255) / 256);
  // the first of two GEMMs is cut only if it makes less than a round (its
  // partial round is filled by the second); the last round of the second
  // follows from the work of both
  const int r0 = t0 < G ? t0 : (pair ? 0 : t0 % G);
  int r1 = t1 < G ? t1 : t1 % G;
  if (pair && t0 >= G && t1 >= G) {
    // both in tiles of the second GEMM, by their k-steps
    const float rounds = ((float)t0 * (float)K0 / (float)K1 + (float)t1) / (float)G;
    r1 = (int)((rounds - (float)(int)rounds) * (float)G);
    if (16 * r1 > 7 * G) r1 = 0;
  }
  LaunchUnits l{phase_units(nfull, nsmall, N0, K0, G, r0, ws), phase_units(nfull, nsmall, N1, K1, G, r1, ws)};
  if (!(phases & 1)) l.u0.total = 0;
  if (!(phases & 2)) l.u1.total = 0;
  return l;
}

// Workspace: counters (zero between calls), then the fp32 partial tiles of
// the pieces (at most 128 KiB each), cut_units for each GEMM of a launch.
constexpr size_t kRowsArrivedOff = 0;  // arrival counters of both GEMMs
constexpr size_t kRowsQueueOff = 4096;  // queue counters
constexpr size_t kRowsDoneOff = 12288;  // per row tile
constexpr size_t kRowsPartOff = 65536;
constexpr int kMaxRowTiles = (int)((kRowsPartOff - kRowsDoneOff) / 4);
constexpr int kPieceBytes = 128 * 1024;

// What a caller has to provide on a GPU of G compute units, and what is used
// of it.
FM_INLINE size_t rows_workspace_bytes(int G) { return 4096 + (size_t)G * 256 * 256 * 4; }
FM_INLINE size_t rows_workspace_used(int G) { return kRowsPartOff + (size_t)2 * cut_units(G) * kPieceBytes; }
// Whether the layout fits: it does on 1 to 585 compute units.
FM_INLINE bool rows_workspace_fits(int G) {
  return (size_t)2 * cut_units(G) * 4 <= kRowsQueueOff - kRowsArrivedOff &&
         rows_workspace_used(G) <= rows_workspace_bytes(G);
}

#undef FM_INLINE

}  // namespace foremoe
