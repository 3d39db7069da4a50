// Numbering of the tiles that the persistent GEMM kernels walk, and the plans
// of their launches.  Plain C++ (constexpr functions run on both sides), so
// that a host test can replay a launch.
#pragma once

#include <stdint.h>

namespace sharq {

// Unit of id in [0, units): one to one onto [0, units), the ids of each XCD
// (workgroups are dealt round-robin, id mod 8) taking a contiguous range.  A
// workgroup b of G walks the ids b, b + G, ...: no id is without a unit, so
// none gets more than ceil(units / G).  (With equal ranges of ceil(units / 8)
// ids past the last workgroup held units where units < G was not a multiple of
// 8, and a launch of one round ran two: MXFP4 M 2560, N 4096, K 4096, 220 tiles,
// 72.1 us against 45.7 with these.)
constexpr int xcd_unit(int id, int units) {
  const int x = id & 7, q = units >> 3, rem = units & 7;
  return x * q + (x < rem ? x : rem) + (id >> 3);
}

// Tile u of a grid of gx by gy: groups of 4 row tiles, column by column, so
// that 32 consecutive tiles (the workgroups of one XCD) are 4 by 8.
constexpr void tile_in_groups(int u, int gx, int gy, int& mt, int& nt) {
  const int g = u / (4 * gx), first = 4 * g;
  const int gs = gy - first < 4 ? gy - first : 4;
  const int in = u - g * 4 * gx;
  mt = first + in % gs;
  nt = in / gs;
}

// ---------------------------------------------------------------------------
// MXFP4 on the dense backbone copy, 256 rows x 64 NF columns (k_linear_mx8)
// ---------------------------------------------------------------------------

constexpr int kRows8 = 256;   // rows of a tile

// Launch plan: NF 4 or 3, and whole 256-column tiles (of a last round at most
// half full, tiles run as halves).  us: the estimate per K step, rounds of
// tiles over the CUs times the tile's measured step (1.85, 1.50, and 1.05 for a
// half tile); 128-column tiles alone were never the best.
struct Plan8 {
  int nf, gx, gy, full, grid;
  double us;
};

constexpr Plan8 plan8(int64_t M, int N, int cus) {
  const int gy = (int)((M + kRows8 - 1) / kRows8);
  Plan8 best{};
  for (int nf = 4; nf >= 3; --nf) {
    const int gx = (N + 64 * nf - 1) / (64 * nf);
    const int64_t tiles = (int64_t)gx * gy, r = tiles % cus;
    Plan8 p{nf, gx, gy, (int)tiles, (int)(tiles < cus ? tiles : cus), 0.0};
    p.us = (double)((tiles + cus - 1) / cus) * (nf == 4 ? 1.85 : 1.50);
    if (nf == 4 && tiles > cus && r > 0 && 2 * r <= cus) {
      p.full = (int)(tiles - r);
      p.us = (double)(tiles / cus) * 1.85 + 1.05;
    }
    if (best.nf == 0 || p.us < best.us) best = p;
  }
  return best;
}

// Whether that kernel's estimate is below that of the 4-wavefront one (rounds
// of 128 x 256 tiles at 0.97 us a step, half tiles at 0.85).
constexpr bool use_mx8(int64_t M, int N, int cus) {
  const int64_t tiles = ((M + 127) / 128) * (int64_t)((N + 255) / 256), r = tiles % cus;
  if (tiles <= cus) return false;   // one round there: a tile of half the size ends sooner
  const double old_us = (double)(tiles / cus) * 0.97 + (r == 0 ? 0.0 : 2 * r <= cus ? 0.85 : 0.97);
  return plan8(M, N, cus).us < 0.98 * old_us;
}

// ---------------------------------------------------------------------------
// NVFP4 and HiF4 at prefill sizes, 256 rows x 64 NF columns (k_linear16)
// ---------------------------------------------------------------------------

constexpr int kRows16 = 256;   // rows of a tile

// Tile width and whole tiles of a launch.  A tile of 64 NF columns takes about
// (NF + 1) / 5 of a 256-column one (its activation work does not shrink with
// it; NVFP4 0.63, 0.93 and 1.10 us a step for NF 2, 3 and 4), and the launch as long as its rounds of tiles over the CUs: the
// cheapest width wins, the wider of equals.  A last round of 256-column tiles
// that is at most half full runs as half tiles.
struct Plan16 {
  int nf, gx, gy, full, grid;
  int64_t cost;   // in fifths of a whole 256-column tile
};

constexpr Plan16 plan16(int64_t M, int N, int cus) {
  const int gy = (int)((M + kRows16 - 1) / kRows16);
  Plan16 best{};
  int64_t least = 0;
  for (int nf = 4; nf >= 2; --nf) {
    const int gx = (N + 64 * nf - 1) / (64 * nf);
    const int64_t tiles = (int64_t)gx * gy, r = tiles % cus;
    int64_t cost = (tiles + cus - 1) / cus * (nf + 1);
    Plan16 p{nf, gx, gy, (int)tiles, (int)(tiles < cus ? tiles : cus), 0};
    if (nf == 4 && tiles > cus && r > 0 && 2 * r <= cus) {
      p.full = (int)(tiles - r);
      cost = tiles / cus * 5 + 3;
    }
    if (least == 0 || cost < least) {
      best = p;
      best.cost = least = cost;
    }
  }
  return best;
}

}  // namespace sharq
