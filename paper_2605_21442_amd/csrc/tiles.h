// Which tile of which launch a workgroup takes, and which chunks of a ragged K slice exist: the index
// arithmetic that the kernels of lce.hip and their host code share, in plain integers, so that the host tests
// run the very functions that the kernels run. LCE_HD is the includer's function qualifier.
#pragma once

#ifndef LCE_HD
#error "define LCE_HD, the qualifier of these functions, before including tiles.h"
#endif

#include <stdint.h>

namespace lce_tiles {

constexpr int kTile = 256;        // tokens (or hidden columns) of a tile
constexpr int kTileRows = 384;    // vocabulary ids (or dH tokens) of a 12-wave tile

// ---- chunks of a row-major slice ----------------------------------------------------------------
// The 16-byte chunk of its row that a lane loads for its even-numbered groups of 8 rows (odd groups: ^ 1).
LCE_HD int lane_chunk(int lane) { return (lane & 7) ^ ((lane >> 3) & 7); }

// Whether that chunk of group q lies before K in the slice that starts at k0 (a ragged last slice ends early).
LCE_HD bool chunk_exists(int lane, int q, int k0, int K) { return k0 + (lane_chunk(lane) ^ (q & 1)) * 8 < K; }

// ---- forward and G launches ---------------------------------------------------------------------
// XCD-aware order of the tiles of a forward or G launch: `tiles` vocabulary tiles by nt token tiles,
// workgroups dealt round-robin to the 8 XCDs (block b runs on XCD b mod 8). The first a = tiles & ~7
// vocabulary tiles go in groups of gw tiles (a and gw multiples of 8; a last group may be narrower)
// by all token tiles, vocabulary tiles fastest: XCD x then takes the tiles = x (mod 8) of each
// group, and a round of its ~32 workgroups shares a few W tiles and a few H tiles, while the group's
// W rows stay in the MALL as the token tiles pass. The last tiles - a (< 8) vocabulary tiles are
// dealt by token tile instead: XCD x takes the token tiles = x (mod 8), each with all of them.
// (Dealt the first way, a group whose width is not a multiple of 8 would give every XCD most of the
// group's W tiles.) False for blocks past the last tile.
LCE_HD bool xcd_tile(int b, int tiles, int gw, int nt, int& tm, int& tn) {
  const int a = tiles & ~7, ba = a * nt;
  if (b < ba) {
    const int full = a / gw, g = b / (gw * nt);
    const int wl = g < full ? gw : a - full * gw, r = b - g * gw * nt;
    tm = g * gw + r % wl;
    tn = r / wl;
    return true;
  }
  const int rem = tiles - a, r = b - ba, k = r >> 3;
  if (rem == 0) return false;
  tm = a + k % rem;
  tn = (r & 7) + 8 * (k / rem);
  return tn < nt;
}

// The tiles a forward or G launch leaves for its last, partial round of the 256 CUs (all of them in a small
// launch) are cut into parts of 192 ids x 256 tokens (2 per tile, up to 128 tiles) or 192 x 128 (4 per tile,
// up to 64), so that the round has two or four times the workgroups. A half tile takes about 0.73 and a
// quarter 0.57 of a tile's time (less work per byte loaded), so that more tiles than that are left whole,
// as is everything in launches of more than kSplitTiles tiles, where the last round is a small share.
// Forward, before and after: 3276 x 8192 x 16032 (546 tiles) 784 -> 673 us; 900 x 2048 x 32000 (336) 140 ->
// 122; 2549 x 1000 x 32003 (840) 174 -> 162; 230 x 512 x 4096 (11) 22 -> 12, its G 28 -> 14. `t` is the index
// space of xcd_tile (a multiple of 8, so that all parts of a tile run on one XCD).
constexpr int kSplitTiles = 2048;
LCE_HD int tile_space(int tiles, int nt) {
  const int a = tiles & ~7;
  return a * nt + (tiles - a) * ((nt + 7) / 8 * 8);
}
LCE_HD int tail_parts(int t, bool split) {   // parts of the tail tiles (1: no tail is cut)
  const int rem = t & 255;
  return !split || t > kSplitTiles || rem == 0 || rem > 128 ? 1 : rem > 64 ? 2 : 4;
}
struct TilePart {
  int tm, tn;        // vocabulary tile, token tile
  int parts, part;   // parts of the tile, this block's (bit 0: its ids, bit 1: its tokens)
};
LCE_HD bool tile_part(int b, int tiles, int gw, int nt, bool split, TilePart& p) {
  const int t = tile_space(tiles, nt), parts = tail_parts(t, split), whole = parts > 1 ? t & ~255 : t;
  int l = b;
  p.parts = 1;
  p.part = 0;
  if (b >= whole) {
    if (parts == 1) return false;
    const int j = b - whole;
    l = whole + j / (8 * parts) * 8 + (j & 7);
    p.parts = parts;
    p.part = (j >> 3) % parts;
  }
  return l < t && xcd_tile(l, tiles, gw, nt, p.tm, p.tn);
}

// Grid and group width of a launch in the order of xcd_tile: `tiles` vocabulary tiles by nt token
// tiles, in groups at most `width` tiles wide (rounded down to a multiple of 8). A split launch's parts
// take at most a round of 256 blocks beside the whole tiles.
struct TileOrder {
  unsigned grid;
  int gw;
};
LCE_HD TileOrder tile_order(int64_t tiles, int64_t nt, int64_t width, bool split = false) {
  const int64_t a = tiles & ~(int64_t)7, rem = tiles - a, w = (width < a ? width : a) & ~(int64_t)7;
  return TileOrder{(unsigned)(a * nt + (rem ? 8 * rem * ((nt + 7) / 8) : 0) + (split ? 256 : 0)), (int)(w < 8 ? 8 : w)};
}

// ---- dH launches --------------------------------------------------------------------------------
// dH launches with fewer output tiles than CUs: K is split so that every CU has a block. The host
// reserves kz_max accumulators (2 to 8); the parts taken follow from the live tile count t = ceil(Nv
// / 384) x ceil(D / 256): the number whose rounds of 256 units take the least K together (64 tiles: 4
// parts, one round; 144 tiles: 3 parts, two rounds of a third of K each). The t * parts units
// (part-major) are cut into 8 equal shares, one per XCD, so that all XCDs work whatever the number of
// row tiles, and an XCD's blocks walk one or two K ranges of G and W in step, which its L2 then reads
// once. (With whole row tiles dealt to the XCDs instead, 4 row tiles kept 4 of the 8 XCDs busy: dH of
// 2048 x 4096 x 128256 with 1536 valid tokens 2500 us, now 1154; of 1948 x 3584 x 152064 2220 -> 1257;
// of 4096 x 2048 x 128256, whose 64 tiles took 3 parts by N and take 4 by Nv, 1365 -> 1133.)
LCE_HD int dh_split_parts(int t, int kz_max) {
  int best = 1, rounds = (t + 255) / 256;
  for (int kz = 2; kz <= kz_max; ++kz) {
    const int r = (t * kz + 255) / 256;
    if (r * best < rounds * kz) {
      best = kz;
      rounds = r;
    }
  }
  return best;
}

// dH launches whose K the host did not split. With T = tm_live x dt live output tiles (tm_live =
// ceil(Nv / 384) row tiles of 384 tokens, dt column tiles of 256), XCD x takes the tiles [c0(x),
// c0(x + 1)) of a balanced cut, c0(x) = floor(x T / 8), in an order that keeps consecutive tiles on
// few operand tiles: bands of 4 row tiles, each walked column by column. An XCD runs its ~32
// resident workgroups in rounds; the n_tail tiles of its last, partial round are split along K
// into dh_tail_parts(n_tail) parts, so that they fill that round instead of leaving most of its
// CUs idle. Part 0 of a tile accumulates into the tile's rows of the accumulator (row stride D);
// part z >= 1 of tail tile t into slot dh_slot0(x) + (z - 1) * n_tail + t, a 384 x 256 fp32 block
// (row stride 256) in the accumulator's rows at or past tm_live * 384, which hold no valid token.
// When those rows cannot hold every slot, no tile is split. The finalise adds the parts in order.
constexpr int kDhBand = 4;                       // row tiles per band
constexpr int64_t kDhSlot = 384 * 256;           // floats per slot
LCE_HD int dh_c0(int x, int t) { return (int)(((int64_t)x * t) >> 3); }
LCE_HD int dh_tail_parts(int n_tail) {
  return n_tail > 0 && n_tail <= 16 ? (32 / n_tail < 8 ? 32 / n_tail : 8) : 1;
}
// slots taken by the XCDs before x (the slots are numbered XCD by XCD, each XCD's in part-major
// order); dh_slot0(8, t) is the total
LCE_HD int dh_slot0(int x, int t) {
  int n = 0;
  for (int y = 0; y < x; ++y) {
    const int nt = (dh_c0(y + 1, t) - dh_c0(y, t)) & 31;
    n += (dh_tail_parts(nt) - 1) * nt;
  }
  return n;
}
LCE_HD bool dh_tail_fits(int t, int tm_live, int d, int acc_rows) {
  return (int64_t)dh_slot0(8, t) * kDhSlot <= (int64_t)(acc_rows - tm_live * 384) * d;
}
LCE_HD void dh_band_tile(int l, int tm_live, int dt, int& tm, int& tn) {
  const int band = l / (kDhBand * dt), r0 = band * kDhBand;
  const int rows = tm_live - r0 < kDhBand ? tm_live - r0 : kDhBand;
  const int k = l - band * kDhBand * dt;
  tm = r0 + k % rows;
  tn = k / rows;
}
LCE_HD int dh_band_index(int tm, int tn, int tm_live, int dt) {
  const int band = tm / kDhBand, r0 = band * kDhBand;
  const int rows = tm_live - r0 < kDhBand ? tm_live - r0 : kDhBand;
  return band * kDhBand * dt + tn * rows + (tm - r0);
}

// The unit of block blk of a dH launch over the nv valid tokens: tile (tm, tn), K part z of kz and, of a tail
// tile's parts z >= 1, the slot they accumulate into (else -1). kz_max > 1: the parts that the host reserved.
// False for blocks without one.
struct DhUnit {
  int tm, tn, z, kz, slot;
};
LCE_HD bool dh_unit(int blk, int nv, int d, int kz_max, int acc_rows, DhUnit& u) {
  const int dt = (d + kTile - 1) / kTile, tm_live = (nv + kTileRows - 1) / kTileRows;
  const int t = tm_live * dt, x = blk & 7, k = blk >> 3;
  u.slot = -1;
  if (kz_max > 1) {
    // every tile's K in kz parts (launches with fewer tiles than CUs)
    if (t == 0) return false;
    u.kz = dh_split_parts(t, kz_max);
    const int n = t * u.kz, l = dh_c0(x, n) + k;
    if (l >= dh_c0(x + 1, n)) return false;
    u.z = l / t;
    dh_band_tile(l - u.z * t, tm_live, dt, u.tm, u.tn);
    return true;
  }
  const int c0 = dh_c0(x, t), n = dh_c0(x + 1, t) - c0, nmain = n & ~31, nt = n - nmain;
  u.z = 0;
  u.kz = 1;
  int l = c0 + k;
  if (k >= nmain) {
    const int j = k - nmain;
    u.kz = dh_tail_fits(t, tm_live, d, acc_rows) ? dh_tail_parts(nt) : 1;
    if (j >= u.kz * nt) return false;
    u.z = j / nt;
    l = c0 + nmain + j % nt;
    if (u.z > 0) u.slot = dh_slot0(x, t) + (u.z - 1) * nt + j % nt;
  }
  dh_band_tile(l, tm_live, dt, u.tm, u.tn);
  return true;
}

// Blocks of a dH launch for npad tokens' rows, a multiple of 8: one for each part that the tiles may take or, of a
// launch that the host did not split, 8 XCDs x 32 CUs x (whole rounds of the largest per-XCD share + one round
// for the split tail).
LCE_HD int dh_grid(int64_t npad, int d, int kz_max) {
  const int64_t t = (npad + kTileRows - 1) / kTileRows * ((d + kTile - 1) / kTile);
  return (int)(kz_max > 1 ? (kz_max * t + 7) / 8 * 8 : 256 * ((t + 7) / 8 / 32 + 1));
}

// The K range [k0, k0 + n) of part z of kz over a slab's vs ids (n <= 0: an empty part): all parts but the last
// are whole 64-wide slices.
LCE_HD int dh_k_range(int vs, int kz, int z, int& k0) {
  const int kt = (vs + 63) / 64 * 64, kh = ((kt + kz - 1) / kz + 63) / 64 * 64;
  k0 = z * kh;
  return vs - k0 < kh ? vs - k0 : kh;
}

// ---- dW launches --------------------------------------------------------------------------------
// The tile of block blk: the slab's tm_count x ceil(D / 256) tiles in the balanced cut of the dH launches, XCD x
// taking [c0(x), c0(x + 1)), walked in bands of 4 row tiles, column by column.
LCE_HD bool dw_unit(int blk, int tm_count, int d, int& tm, int& tn) {
  const int dt = (d + kTile - 1) / kTile, t = tm_count * dt, x = blk & 7, k = blk >> 3;
  const int c0 = dh_c0(x, t);
  if (k >= dh_c0(x + 1, t) - c0) return false;
  dh_band_tile(c0 + k, tm_count, dt, tm, tn);
  return true;
}

LCE_HD int dw_grid(int tm_count, int d) {
  return (int)(((int64_t)tm_count * ((d + kTile - 1) / kTile) + 7) / 8 * 8);
}

// One launch for both: block b of the grid's dh_blocks + dw_blocks (both multiples of 8, so that either part's
// blocks keep their XCDs) is block dhdw_block(...) of the dH launch, or dh_blocks more than that of the dW launch.
// The units with the longer K, dH's ids of a part or dW's valid tokens, take the first blocks. (The most parts
// stand for those taken: every block asks, and counting them took each of the 4176 blocks of 187 x 3520 x 114458
// 0.7 us, 438 -> 454 us the launch.)
LCE_HD bool dw_first(int nv, int kz_max, int vs) { return (int64_t)nv * kz_max > vs; }
LCE_HD int dhdw_block(int b, int dh_blocks, int dw_blocks, bool dw_goes_first) {
  if (!dw_goes_first) return b;
  return b < dw_blocks ? b + dh_blocks : b - dw_blocks;
}

}  // namespace lce_tiles
