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

// A launch may have 2^32 threads at most.  The small-M kernels give few rows
// many threads (up to 8 a column), so the widest layers stay with the tiled ones.
constexpr int64_t kMaxThreads = (int64_t)1 << 31;
constexpr bool small_m_columns(int N) { return 8 * (int64_t)N <= kMaxThreads; }

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
    const int gx = (int)(((int64_t)N + 64 * nf - 1) / (64 * nf));
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
// MXFP4 with few rows (k_linear_mx_skinny)
// ---------------------------------------------------------------------------

// What a kernel reads as backbone: the dense copy, 2:4 or 4:8 compressed.
constexpr int backbone_form(int pat) { return pat == 0 ? 0 : pat == 24 ? 1 : 2; }

// Above 32 rows the workgroups tile M as well: 16 mf rows and 16 nb columns, K
// over ks wavefronts.  A launch takes us[0] + us[1] (R - 1) + us[2] R K / 4096,
// R the rounds of workgroups over the CUs, by the backbone's form.  Fitted to
// about 300 shapes per form with the weight streamed from HBM (N 512 to 28672, K
// 768 to 18944, M 33 to 4096; nine in ten within 6 to 20%).  The forms differ, and
// so does what a round costs beside its share of K: with neither in the
// estimate, 160 x 7168 x 2048 4:8 took 22.2 us here and 18.0 on the main kernel.
struct SkinnyCfg {
  int mf, nb, ks;
  double us[3][3];
};
constexpr SkinnyCfg kSkinnyCfg[6] = {
    {1, 1, 8, {{2.57, 0.16, 2.04}, {2.83, 0.31, 2.31}, {2.96, 0.38, 3.52}}},
    {2, 1, 8, {{2.46, 0.93, 3.64}, {2.89, 0.65, 4.50}, {3.02, 1.33, 7.51}}},
    {2, 2, 8, {{2.68, 1.35, 4.45}, {3.15, 1.53, 5.30}, {3.34, 1.65, 8.20}}},
    {2, 4, 8, {{3.19, 1.93, 5.93}, {3.80, 2.11, 6.33}, {4.23, 2.46, 8.53}}},
    {4, 4, 4, {{5.80, 4.99, 8.41}, {6.67, 5.13, 9.20}, {7.27, 5.44, 15.6}}},
    {2, 4, 4, {{4.17, 0.66, 5.59}, {4.76, 0.82, 6.63}, {4.72, 2.97, 9.73}}},
};

struct SkinnyWide {
  int mf, nb, ks;
  double us;
};

constexpr SkinnyWide skinny_wide(int64_t M, int N, int K, int form, int cus) {
  SkinnyWide best{};
  for (const SkinnyCfg& c : kSkinnyCfg) {
    // its ragged form needs the registers of two wavefronts: 22 us, 12 in the estimate, at 256 x 5000 x 2080
    if (K % 128 != 0 && c.mf == 2 && c.nb == 4 && c.ks == 4) continue;
    const int64_t wgs = ((int64_t)N + 16 * c.nb - 1) / (16 * c.nb) * ((M + 16 * c.mf - 1) / (16 * c.mf));
    if (wgs * 64 * c.ks > kMaxThreads) continue;
    const double r = (double)((wgs + cus - 1) / cus);
    const double us = c.us[form][0] + c.us[form][1] * (r - 1.0) + c.us[form][2] * r * K / 4096.0;
    if (best.mf == 0 || us < best.us) best = {c.mf, c.nb, c.ks, us};
  }
  return best;
}

// The small-M kernel serves M <= 32, and larger M where its estimate is 5%
// below the main kernel's: a start, and per panel and round of 128 x 256 tiles
// over the CUs a share that grows with the CUs at work (same shapes; nine in ten
// within 3 to 6%).  form, main_form: what each of the two would read.
constexpr bool use_skinny(int64_t M, int N, int K, int form, int main_form, int cus) {
  constexpr double kMain[3][3] = {{5.19, 0.553, 0.183}, {5.73, 0.686, 0.163}, {6.51, 0.709, 0.176}};
  if (K < 128 || !small_m_columns(N)) return false;
  if (M <= 32) return true;
  if (M > 4096) return false;
  const SkinnyWide w = skinny_wide(M, N, K, form, cus);
  const int64_t tiles = ((M + 127) / 128) * (((int64_t)N + 255) / 256);
  const double rounds = (double)((tiles + cus - 1) / cus), fill = tiles < cus ? (double)tiles / (double)cus : 1.0;
  const double main_us = kMain[main_form][0] + K / 128.0 * rounds * (kMain[main_form][1] + kMain[main_form][2] * fill);
  return w.mf != 0 && 1.05 * w.us < main_us;
}

// ---------------------------------------------------------------------------
// MXFP4, grouped, with few rows (k_linear_mx_grouped_skinny)
// ---------------------------------------------------------------------------

// 16 rows and 16 nb columns of an expert to a workgroup, K over ks wavefronts.
// 32 columns where a few experts leave the chip idle with 64; K in two parts
// where it has less than 12 panels.  E 128 N 2048 K 768, 512 rows: 24.8 us with 2
// parts, 30.6 with 4; N 1536 K 2048, 256 rows: 35.8, 35.0; E 8 N 2048 K 4096, 64 rows:
// 10.0 with 32 columns, 11.3 with 64.
struct GroupedCfg {
  int nb, ks;
};
constexpr GroupedCfg grouped_cfg(int64_t total, int E, int N, int K, int cus) {
  const int64_t groups = (int64_t)E * (((int64_t)N + 63) / 64);
  if ((groups <= 2 * cus && total <= E) || (groups <= cus && total <= 8 * (int64_t)E)) return {2, 4};
  return {4, (K + 127) / 128 >= 12 ? 4 : 2};
}

// Whether the few-row kernel takes a grouped call of `total` rows, rather than
// the persistent one with its 128-row tiles.  The host does not know the routing.
// With up to 2048 outputs a CU (two workgroups' chunks) it is the faster one
// however the rows are spread, but for 12% at one size.  Above, where even routing
// leaves an expert at most 4 rows, or 8, the line lies at twice and one and a
// half times that: us here / there, E 128 N 2048 K 768, 512 rows 24.8 / 39.6 (on 8
// experts 10.2 / 10.0); N 1536 K 2048, 512 rows 42.6 / 57.6 (16.1 / 14.1); E 64 N 1408
// K 2048, 384 rows 25 / 34 (13.0 / 13.0).
constexpr bool use_grouped_skinny(int64_t total, int E, int N, int cus) {
  const int64_t outputs = total * (int64_t)N, limit = 2048 * (int64_t)cus;
  if (((int64_t)E + total / 16) * (((int64_t)N + 31) / 32) * 256 > kMaxThreads) return false;
  return outputs <= limit || (total <= 4 * (int64_t)E && outputs <= 2 * limit) ||
         (total <= 8 * (int64_t)E && 2 * outputs <= 3 * limit);
}

// ---------------------------------------------------------------------------
// NVFP4 and HiF4 at prefill sizes (k_linear16)
// ---------------------------------------------------------------------------

// By format and backbone: NVFP4 dense copy, NVFP4 2:4 and 4:8 compressed, HiF4 2:4.
constexpr int form16(bool nv, int pat) { return nv ? backbone_form(pat) : 3; }

// Tile and whole tiles of a launch.  The launch takes as long as its rounds of
// tiles over the CUs; the cheapest tile wins, the larger of equals (128 rows: by 7%).  A last round
// of 256 x 256 tiles that is at most half full runs as half tiles of 128 columns.
// us: the estimate per 32 positions, from the measured step of tiles of 256 rows
// x 256, 192 and 128 columns and of 128 rows x 256 columns, by form.  128 rows
// suit M just past a multiple of 256 and HiF4, whose wavefronts then dequantize
// less for each MFMA: NVFP4 dense M 384 N 37888 K 3584 208 us -> 172, HiF4 M 2048 N
// 3584 K 3584 140 -> 116.
struct Plan16 {
  int rows, nf, gx, gy, full, grid;
  double us;
};

constexpr Plan16 plan16(int64_t M, int N, int form, int cus) {
  constexpr double kStep[4][4] = {
      {1.16, 0.93, 0.69, 0.73}, {1.43, 1.08, 0.78, 0.79}, {1.62, 1.25, 1.04, 1.06}, {1.81, 1.48, 1.17, 0.96}};
  constexpr int kTile[4][2] = {{256, 4}, {256, 3}, {256, 2}, {128, 4}};   // rows, columns / 64
  Plan16 best{};
  for (int i = 0; i < 4; ++i) {
    const int rows = kTile[i][0], nf = kTile[i][1];
    const int gx = (int)(((int64_t)N + 64 * nf - 1) / (64 * nf)), gy = (int)((M + rows - 1) / rows);
    const int64_t tiles = (int64_t)gx * gy, r = tiles % cus;
    Plan16 p{rows, nf, gx, gy, (int)tiles, (int)(tiles < cus ? tiles : cus), 0.0};
    p.us = (double)((tiles + cus - 1) / cus) * kStep[form][i];
    if (i == 0 && tiles > cus && r > 0 && 2 * r <= cus) {
      p.full = (int)(tiles - r);
      p.us = (double)(tiles / cus) * kStep[form][0] + kStep[form][2];
    }
    // a last round that is not full runs faster than the others, which favours the larger tile
    if (best.nf == 0 || p.us < (rows == 128 ? 0.93 : 1.0) * best.us) best = p;
  }
  return best;
}

// ---------------------------------------------------------------------------
// NVFP4 and HiF4 with few rows (k_linear_skinny16)
// ---------------------------------------------------------------------------

// Above 32 rows: 16 mf rows and 16 nb columns to a workgroup, K over ks
// wavefronts.  A launch takes us[0] + us[1] (R - 1) + (us[2] R + us[3] R2) panels
// / 32, R and R2 the rounds of workgroups and of pairs of them over the CUs (two
// of some fit a CU), by form; the last three rows: 2:4, 4:8 and HiF4 with K not a
// multiple of 128.  Fitted to 379 and 120 shapes per form with the weight
// streamed from HBM (N 512 to 37888, K 768 to 18944, M 33 to 4096; nine in ten
// within 4 to 10%).  With one figure for every NVFP4 form in their place, 2:4 and
// 4:8 calls ran up to 1.8 times as long here as on the prefill kernel (M 640 N
// 6144 K 4096 4:8: 198 us, there 117).
struct Cfg16 {
  int mf, nb, ks;
  double us[7][4];
};
constexpr double kNotBuilt = 1e9;   // never the least for these forms
constexpr Cfg16 kCfg16[4] = {
    {2, 1, 8, {{3.11, 0.35, 4.42}, {3.26, 0.18, 6.34}, {3.34, 0.16, 9.94}, {3.06, 1.02, 14.2},
               {3.70, 0.24, 5.86, 1.97}, {3.95, 0.10, 9.47, 2.48}, {3.46, 1.20, 17.5}}},
    {2, 2, 8, {{3.27, 1.43, 6.17}, {3.34, 1.33, 8.07}, {3.44, 1.32, 11.8}, {3.38, 1.38, 16.7},
               {3.69, 1.46, 9.90}, {3.80, 1.50, 14.4}, {4.06, 1.78, 20.2}}},
    {2, 4, 4, {{4.69, 1.07, 5.69, 5.88}, {4.95, 1.05, 7.43, 4.95}, {4.79, 2.76, 15.5}, {5.18, 2.96, 23.0},
               {6.11, 1.17, 9.06, 2.85}, {6.54, 1.27, 12.5, 2.37}, {6.60, 4.28, 24.4}}},
    {4, 4, 4, {{kNotBuilt}, {kNotBuilt}, {6.96, 4.68, 27.1}, {7.37, 4.88, 37.1},
               {kNotBuilt}, {9.07, 6.50, 27.3}, {9.86, 7.15, 37.1}}},
};

struct Wide16 {
  int mf, nb, ks;
  double us;
};

constexpr Wide16 wide16(int64_t M, int N, int K, int form, int cus) {
  const double panels = (double)((K + 127) / 128) / 32.0;
  Wide16 best{};
  for (const Cfg16& c : kCfg16) {
    const double(&t)[4] = c.us[K % 128 == 0 ? form : form + 3];   // the dense copy needs K a multiple of 128
    const int64_t wgs = ((int64_t)N + 16 * c.nb - 1) / (16 * c.nb) * ((M + 16 * c.mf - 1) / (16 * c.mf));
    if (wgs * 64 * c.ks > kMaxThreads) continue;
    const double r = (double)((wgs + cus - 1) / cus), r2 = (double)((wgs + 2 * cus - 1) / (2 * cus));
    const double us = t[0] + t[1] * (r - 1.0) + (t[2] * r + t[3] * r2) * panels;
    if (best.mf == 0 || us < best.us) best = {c.mf, c.nb, c.ks, us};
  }
  return best;
}

// Up to 32 rows always (the layer streams its weight); above, where the
// estimate is below the prefill kernel's: a start and its plan's time per 32
// positions, or, K not a multiple of 128, the simpler kernels' rounds of 128 x
// 256 tiles (same shapes; nine in ten within 3 to 9%).
constexpr bool use_skinny16(int64_t M, int N, int K, int form, int cus) {
  constexpr double kStart[4] = {6.0, 6.6, 7.2, 6.2}, kRagged[4] = {1.41, 1.23, 1.41, 1.90};
  if (!small_m_columns(N)) return false;
  if (M <= 32) return true;
  if (M > 4096) return false;
  const Wide16 w = wide16(M, N, K, form, cus);
  double main_us = 0.0;
  if (K % 128 == 0) {
    main_us = kStart[form] + plan16(M, N, form, cus).us * K / 32.0;
  } else {
    const int64_t tiles = ((M + 127) / 128) * (((int64_t)N + 255) / 256);
    main_us = 9.6 + (double)((tiles + cus - 1) / cus) * kRagged[form] * K / 32.0;
  }
  return w.mf != 0 && w.us < main_us;
}

}  // namespace sharq
