"""The index functions of paper_2605_21442_amd/csrc/tiles.h, built for the host from the very header that the
kernels include, as Python functions."""
from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_21442_amd", "csrc")

SOURCE = """
#define LCE_HD inline
#include "tiles.h"
using namespace lce_tiles;
extern "C" {
int t_xcd_tile(int b, int tiles, int gw, int nt, int* o) { return xcd_tile(b, tiles, gw, nt, o[0], o[1]); }
int t_tile_space(int tiles, int nt) { return tile_space(tiles, nt); }
int t_tail_parts(int t, int split) { return tail_parts(t, split); }
int t_tile_part(int b, int tiles, int gw, int nt, int split, int* o) {
  TilePart p;
  if (!tile_part(b, tiles, gw, nt, split, p)) return 0;
  o[0] = p.tm; o[1] = p.tn; o[2] = p.parts; o[3] = p.part;
  return 1;
}
void t_tile_order(int tiles, int nt, int width, int split, int* o) {
  const TileOrder r = tile_order(tiles, nt, width, split);
  o[0] = (int)r.grid; o[1] = r.gw;
}
int t_dh_split_parts(int t, int kz_max) { return dh_split_parts(t, kz_max); }
int t_dh_unit(int blk, int nv, int d, int kz_max, int acc_rows, int* o) {
  DhUnit u;
  if (!dh_unit(blk, nv, d, kz_max, acc_rows, u)) return 0;
  o[0] = u.tm; o[1] = u.tn; o[2] = u.z; o[3] = u.kz; o[4] = u.slot;
  return 1;
}
int t_dh_grid(int64_t npad, int d, int kz_max) { return dh_grid(npad, d, kz_max); }
int t_dw_grid(int tm_count, int d) { return dw_grid(tm_count, d); }
int t_dh_k_range(int vs, int kz, int z, int* o) { o[1] = dh_k_range(vs, kz, z, o[0]); return 1; }
int t_dw_unit(int blk, int tm_count, int d, int* o) { return dw_unit(blk, tm_count, d, o[0], o[1]); }
int t_dw_first(int nv, int kz_max, int vs) { return dw_first(nv, kz_max, vs); }
int t_dhdw_block(int b, int dh_blocks, int dw_blocks, int first) { return dhdw_block(b, dh_blocks, dw_blocks, first); }
int t_lane_chunk(int lane) { return lane_chunk(lane); }
int t_chunk_exists(int lane, int q, int k0, int K) { return chunk_exists(lane, q, k0, K); }
}
"""


@functools.lru_cache(maxsize=1)
def _lib():
    with tempfile.TemporaryDirectory() as tmp:
        src, out = os.path.join(tmp, "tiles.cpp"), os.path.join(tmp, "tiles.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-shared", "-fPIC", "-I", CSRC, src, "-o", out],
                       check=True)
        return ctypes.CDLL(out)


def _call(name, count, *args):
    o = (ctypes.c_int * count)()
    return tuple(o) if getattr(_lib(), name)(*args, o) else None


def xcd_tile(b, tiles, gw, nt):
    return _call("t_xcd_tile", 2, b, tiles, gw, nt)


def tile_space(tiles, nt):
    return _lib().t_tile_space(tiles, nt)


def tail_parts(t, split=True):
    return _lib().t_tail_parts(t, int(split))


def tile_part(b, tiles, gw, nt, split=True):
    """(vocabulary tile, token tile, parts, part) of block b, or None."""
    return _call("t_tile_part", 4, b, tiles, gw, nt, int(split))


def tile_order(tiles, nt, width, split=False):
    """(grid, group width)."""
    o = (ctypes.c_int * 2)()
    _lib().t_tile_order(tiles, nt, width, int(split), o)
    return tuple(o)


def dh_split_parts(t, kz_max):
    return _lib().t_dh_split_parts(t, kz_max)


def dh_unit(blk, nv, d, kz_max, acc_rows):
    """(row tile, column tile, K part, parts, slot or -1) of block blk, or None."""
    return _call("t_dh_unit", 5, blk, nv, d, kz_max, acc_rows)


def dh_k_range(vs, kz, z):
    """(first id, ids) of a K part."""
    return _call("t_dh_k_range", 2, vs, kz, z)


def dw_unit(blk, tm_count, d):
    return _call("t_dw_unit", 2, blk, tm_count, d)


def dw_first(nv, kz_max, vs):
    return bool(_lib().t_dw_first(nv, kz_max, vs))


def dhdw_block(b, dh_blocks, dw_blocks, first):
    return _lib().t_dhdw_block(b, dh_blocks, dw_blocks, int(first))


def lane_chunk(lane):
    return _lib().t_lane_chunk(lane)


def chunk_exists(lane, q, k0, K):
    return bool(_lib().t_chunk_exists(lane, q, k0, K))


def dh_grid(n, d, kz_max):
    """Blocks of a dH launch for n tokens."""
    return _lib().t_dh_grid(ctypes.c_int64(-(-max(n, 1) // 256) * 256), d, kz_max)


def dw_grid(tm_count, d):
    return _lib().t_dw_grid(tm_count, d)


def dh_units(n, nv, d, kz_max, acc_rows):
    """(block, row tile, column tile, K part, parts, slot) of every unit of a dH launch."""
    for blk in range(dh_grid(n, d, kz_max)):
        u = dh_unit(blk, nv, d, kz_max, acc_rows)
        if u is not None:
            yield (blk, *u)
