"""Every address the kernels form stays inside its buffer, whatever the hardware's range checks do.

For each launch of the plan (the five heads and small edge shapes, at several valid-token counts
Nv), this test recomputes, from the layout lce_plan_info reports, the largest byte offset that
each kernel's loads, stores and read-modify-writes can form and checks it against the size of
the region (workspace) or of the caller's tensor it addresses. The arithmetic follows the
kernels' index expressions:

* forward and G tiles are 384 x 256 over the gathered rows Hv at every width, and the last round's
  may be cut into 192 x 256 or 192 x 128 parts; the rows of the last vocabulary tile past V, and the
  chunks of a row past D, are loaded through the out-of-range offset (zeros, no address), so the W
  rows addressed are those below V;
* K-major operands send the lanes whose columns lie past D (the hidden width) to the same offset;
* dH runs K over the slab's vs ids (a ragged last slice masks the rest), split into 1 to 8 parts;
* G and the dH accumulators hold rows_g rows, the 384-row tiles of the last token rows included;
* the dW / AdamW epilogues touch only the rows of the slab that exist.

Accesses sent to the out-of-range offset form no address and are not counted. Which workgroup takes
which tile, part, K range or slot is asked of the functions that the kernels run (host_tiles). No GPU
is needed.
"""
import pytest

from paper_2605_21442_amd import binding as B
from tests import host_tiles as T

HEADS = [(256, 512, 4096), (8192, 2048, 128256), (16384, 4096, 128256), (32768, 3584, 152064),
         (16384, 8192, 128256)]
# launches that may be cut, and a ragged width among them
CUT = [(2048, 2048, 128256), (2999, 1000, 32003), (4096, 8192, 16032), (513, 64, 40520), (100, 136, 57607), (709, 2048, 128256)]
EDGES = CUT + [(1, 8, 5), (300, 264, 1000), (257, 64, 9000), (513, 520, 300), (300, 64, 12300), (200, 128, 12289),
         (768, 128, 1536), (520, 64, 40000), (33, 72, 1), (16385, 64, 383), (1000, 136, 385)]


def cdiv(a, b):
    return -(-a // b)


def rup(a, b):
    return cdiv(a, b) * b


class Extents:
    """Largest byte (exclusive end) formed in each buffer, against the buffer's size."""

    def __init__(self):
        self.ends = {}

    def touch(self, buf, end):
        self.ends[buf] = max(self.ends.get(buf, 0), end)

    def check(self, sizes, where):
        for buf, end in self.ends.items():
            assert end <= sizes[buf], f"{where}: {buf} reaches byte {end} of {sizes[buf]}"


def dh_tail_parts(nv, d, acc_rows):
    """The K parts z >= 1 of the tail tiles of a dH launch the host did not split: (xcd, first row of
    the tile, z, parts of the tile, slot)."""
    return [(blk & 7, tm * 384, z, kz, slot) for blk, tm, _, z, kz, slot in T.dh_units(nv, nv, d, 1, acc_rows) if z]


def walk(n, d, v, nv, ld_h=None, ld_w=None):
    """Extents of one lce_forward + lce_backward of an [n, d] x [v, d] problem with nv valid rows."""
    ld_h = ld_h or d
    ld_w = ld_w or d
    info = B.lce_plan_info(B.problem(n, d, v, ld_h=ld_h, ld_w=ld_w))
    npad, rows_g, vc, nslab = info["npad"], info["rows_g"], info["vc"], info["nslab"]
    e = Extents()
    # caller tensors: the last row holds only d elements of its stride
    sizes = {"H": 2 * ((n - 1) * ld_h + d) if n else 0, "W": 2 * ((v - 1) * ld_w + d),
             "dH": 2 * n * d, "dW": 2 * v * d, "lse": 4 * n, "targets": 4 * n,
             "idx": 4 * npad, "pos": 4 * npad, "hv": 2 * npad * d,
             "pm": 4 * info["part_rows"] * npad, "ps": 4 * info["part_rows"] * npad, "terms": 4 * npad,
             "G": 2 * rows_g * vc, "dh32": 4 * rows_g * d * info["dh_kz"]}
    nt, vt3 = cdiv(nv, 256), cdiv(v, 384)

    # compaction: idx[0..nv), pos[0..n), the targets
    if nv:
        e.touch("idx", 4 * nv)
    e.touch("pos", 4 * n)
    e.touch("targets", 4 * n)

    def w_rows(v0, rows):
        # rows [v0, v0 + rows) of W, full K (the rows past V of a last tile are masked)
        last = min(v0 + rows, v) - 1
        e.touch("W", 2 * (last * ld_w + d))

    def part_box(p):
        """First id and token of a tile's part, relative to the launch, and its ids and tokens."""
        tm, tn, parts, part = p
        ih, th = (part & 1, part >> 1) if parts > 1 else (0, 0)
        ids = 192 if parts > 1 else 384
        n0 = tn * 256 + th * 128
        wide = nv - tn * 256 > 128 and parts < 4
        return tm * 384 + ih * 192, n0, ids, 256 if wide else 128

    def hv_tile(n0, rows):
        # a tile's dense rows, those past Nv included
        e.touch("hv", 2 * (n0 + rows) * d)

    # forward statistics
    if nv:
        e.touch("H", 2 * ((n - 1) * ld_h + d))                      # rows gathered through idx (< n)
        e.touch("hv", 2 * rup(nv, 64) * d)                          # gather, zero rows to a multiple of 64
        if info["fwd_one_launch"]:
            cut = vt3 * (npad // 256) <= 4096                       # the launch may be cut (of up to 2048 live tiles)
            grid, gw = T.tile_order(vt3, npad // 256, vt3, cut)
            second = T.tail_parts(T.tile_space(vt3, nt), cut) > 1   # a second row per tile
            for b in range(grid) if vt3 * nt <= 4096 else ():
                p = T.tile_part(b, vt3, gw, nt, cut)
                if p is None:
                    continue
                v0, n0, ids, toks = part_box(p)
                if n0 >= nv:
                    continue
                row = p[0] + (vt3 if p[2] > 1 and p[3] & 1 else 0)
                if v0 < v:
                    w_rows(v0, ids)
                hv_tile(n0, toks)
                e.touch("pm", 4 * (row * npad + min(n0 + toks, nv)))
                if second and p[2] == 1:                            # an empty pair beside a whole tile's
                    e.touch("pm", 4 * ((row + vt3) * npad + min(n0 + 256, nv)))
            e.touch("pm", 4 * (((2 if second else 1) * vt3 - 1) * npad + nv))       # the merge reads these rows
        else:
            gw = (info["part_rows"] - 1) // 2
            e.touch("pm", 4 * (2 * gw * npad + nv))                 # running pair after the two row sets
        w_rows(0, vt3 * 384)
        hv_tile(0, nt * 256)
        e.touch("ps", e.ends["pm"])
        e.touch("terms", 4 * nv)
        e.touch("lse", 4 * n)

    # backward
    if nv:
        e.touch("hv", 2 * rup(nv, 64) * d)
    dh_kz = info["dh_kz"]
    for s in range(nslab):
        v0 = s * vc
        vs = min(vc, v - v0)
        if not nv:
            continue
        # G: W rows v0 + [vt0, vt0 + ids) (masked past V), Hv rows; a tile or part is written whole
        tmg = cdiv(vs, 384)
        grid, gw = T.tile_order(tmg, npad // 256, tmg, True)
        for b in range(grid) if tmg * nt <= 4096 else ():
            p = T.tile_part(b, tmg, gw, nt)
            if p is None:
                continue
            vt0, n0, ids, toks = part_box(p)
            if n0 >= nv or vt0 >= vs:
                continue
            w_rows(v0 + vt0, ids)
            hv_tile(n0, toks)
            e.touch("G", 2 * ((n0 + toks - 1) * vc + vt0 + ids))
        w_rows(v0, tmg * 384)
        e.touch("G", 2 * ((nt * 256 - 1) * vc + tmg * 384))
        # dH: 384-row tiles of G rows, K over [k0, k0 + kzn), W slab rows v0 + k (< v0 + vs), columns < d
        seen = set()
        for _, tm, _, z, kz, slot in T.dh_units(n, nv, d, dh_kz, rows_g):
            if (tm, z, kz, slot) in seen:
                continue
            seen.add((tm, z, kz, slot))
            k0, kzn = T.dh_k_range(vs, kz, z)
            # read-modify-write of the block: rows of the tile in accumulator z (the parts follow each other), or
            # a 384 x 256 slot past the live tiles' rows
            e.touch("dh32", 4 * ((z * rows_g if slot < 0 else 0) + tm * 384 + 384) * d if slot < 0
                    else 4 * (cdiv(nv, 384) * 384 * d + (slot + 1) * 384 * 256))
            if kzn > 0:
                e.touch("G", 2 * ((tm * 384 + 383) * vc + k0 + kzn))
                w_rows(v0 + k0, kzn)
        # dW: G and Hv read K-major over round_up(Nv, 64) token rows; dW rows of the slab only
        kpad = rup(nv, 64)
        for m0 in range(0, vs, 384):
            e.touch("G", 2 * ((kpad - 1) * vc + m0 + 384))
            e.touch("dW", 2 * (v0 + min(vs, m0 + 384)) * d)
        e.touch("hv", 2 * ((kpad - 1) * d + d))
    e.touch("dH", 2 * n * d)
    return e, sizes, info


CASES = [(n, d, v, nv) for (n, d, v) in HEADS + EDGES
         for nv in sorted({0, 1, max(n // 2, 1), max(n - 1, 0), n}) if nv <= n]


@pytest.mark.parametrize("n,d,v,nv", CASES)
def test_no_access_leaves_its_buffer(n, d, v, nv):
    e, sizes, _ = walk(n, d, v, nv)
    e.check(sizes, f"n={n} d={d} v={v} nv={nv}")


@pytest.mark.parametrize("n,d,v", [(300, 64, 1000), (1000, 136, 385), (16384, 4096, 128256)])
def test_no_access_leaves_its_buffer_with_row_strides(n, d, v):
    for nv in (1, n):
        e, sizes, _ = walk(n, d, v, nv, ld_h=d + 64, ld_w=d + 8)
        e.check(sizes, f"strided n={n} d={d} v={v} nv={nv}")


@pytest.mark.parametrize("n,d,v", HEADS + EDGES)
def test_workspace_regions_are_disjoint_and_inside_the_workspace(n, d, v):
    info = B.lce_plan_info(B.problem(n, d, v))
    npad, rows_g, vc = info["npad"], info["rows_g"], info["vc"]
    prefix = [("idx", info["o_idx"], 4 * npad), ("pos", info["o_pos"], 4 * npad), ("nv", info["o_nv"], 4),
              ("hv", info["o_hv"], 2 * npad * d)]
    fwd = prefix + [("pm", info["o_pm"], 4 * info["part_rows"] * npad), ("ps", info["o_ps"], 4 * info["part_rows"] * npad),
                    ("terms", info["o_terms"], 4 * npad)]
    bwd = prefix + [("G", info["o_g"], 2 * rows_g * vc), ("dh32", info["o_dh32"], 4 * rows_g * d * info["dh_kz"])]
    assert 1 <= info["dh_kz"] <= 8
    assert info["o_dh32b"] == (info["o_dh32"] + 4 * rows_g * d if info["dh_kz"] > 1 else 0)
    assert rows_g % 384 == 0 and rows_g >= npad and npad % 256 == 0 and npad >= n
    assert vc % 768 == 0
    for regions, total in ((fwd, info["fwd_bytes"]), (bwd, info["bwd_bytes"])):
        regions = sorted(regions, key=lambda r: r[1])
        for (a, oa, sa), (b, ob, sb) in zip(regions, regions[1:]):
            assert oa + sa <= ob, f"{a} overlaps {b}"
        for name, o, size in regions:
            assert o % 256 == 0, name
        assert regions[-1][1] + regions[-1][2] <= total


@pytest.mark.parametrize("n,d,v", HEADS + EDGES)
def test_in_tile_offsets_fit_a_buffer_resource(n, d, v):
    # buffer resources hold at most 2^31 - 1 bytes; every tile's offsets from its resource base
    # (a W tile, a G tile row block, a dH accumulator tile, a 64-row K slice) stay below that
    info = B.lce_plan_info(B.problem(n, d, v))
    vc = info["vc"]
    lim = 2 ** 31 - 1
    assert 384 * d * 2 <= lim                      # W / Hv tile
    assert 256 * vc * 2 <= lim                     # G rows of one token tile
    assert 384 * d * 4 <= lim                      # dH accumulator tile
    assert 64 * max(d, vc) * 2 <= lim              # one K-major slice


def test_the_walk_flags_regions_sized_to_npad_rows():
    # with G and the dH accumulators sized to Npad rows (not the 384-row tile grid), the dH tiles of
    # the last token rows of the 8B head with every token valid reach past them
    e, sizes, info = walk(16384, 4096, 128256, 16384)
    assert info["rows_g"] > info["npad"]
    for buf, row_bytes in (("G", 2 * info["vc"]), ("dh32", 4 * 4096 * info["dh_kz"])):
        short = dict(sizes)
        short[buf] = info["npad"] * row_bytes
        with pytest.raises(AssertionError, match=buf):
            e.check(short, "npad rows")


@pytest.mark.parametrize("n,d,v,nv", [(1000, 1000, 32003, 900), (4096, 8192, 16032, 3276), (256, 512, 4096, 230),
                                      (900, 2048, 32000, 900)])
def test_the_walk_flags_partial_rows_without_the_second_set(n, d, v, nv):
    # launches whose last tiles are cut write two partial rows per tile
    e, sizes, info = walk(n, d, v, nv)
    vt3 = cdiv(v, 384)
    assert T.tail_parts(T.tile_space(vt3, cdiv(nv, 256))) > 1
    for buf in ("pm", "ps"):
        with pytest.raises(AssertionError, match=buf):
            e.check(dict(sizes, **{buf: 4 * vt3 * info["npad"]}), "one row per tile")


@pytest.mark.parametrize("n,d,v,nv", [(12288, 2048, 1000, 300), (12288, 2048, 1000, 1400), (12288, 2048, 1000, 3686),
                                      (12288, 2048, 1000, 4423), (8192, 4096, 1000, 6209),
                                      (32768, 3584, 152064, 22936), (16384, 8192, 128256, 13107)])
def test_split_dh_tails_stay_inside_the_accumulator(n, d, v, nv):
    # the shapes whose dH tails the kernel splits on the device (and one whose tails do not fit)
    e, sizes, info = walk(n, d, v, nv)
    e.check(sizes, f"n={n} d={d} v={v} nv={nv}")
    parts = dh_tail_parts(nv, d, info["rows_g"])
    slots = sorted(p[4] for p in parts)
    assert slots == list(range(len(slots)))            # numbered densely, each once
    tm_live = cdiv(nv, 384)
    assert len(slots) * 384 * 256 <= (info["rows_g"] - tm_live * 384) * d


@pytest.mark.parametrize("nv,d", [(300, 2048), (3686, 2048), (22936, 3584), (13107, 8192), (12288, 4096), (1, 64)])
def test_split_dh_blocks_cover_every_tile_and_k_part_once(nv, d):
    # the blocks of a launch the host did not split, with room for every slot: every live tile once, with parts
    # 0 .. kz - 1 of one kz, whose K ranges are disjoint and cover the slab
    tm_live, dtc = cdiv(nv, 384), cdiv(d, 256)
    rows_g = rup(rup(max(nv, 1), 256), 384) + 384 * 64
    seen, slots = {}, []
    for _, tm, tn, z, kz, slot in T.dh_units(nv, nv, d, 1, rows_g):
        seen.setdefault((tm, tn, kz), []).append(z)
        assert (slot >= 0) == (z > 0)
        slots += [slot] if z else []
    assert sorted(k[:2] for k in seen) == sorted((tm, tn) for tm in range(tm_live) for tn in range(dtc))
    assert all(sorted(z) == list(range(k[2])) and k[2] <= 8 for k, z in seen.items())
    assert sorted(slots) == list(range(len(slots)))
    for kz in {k[2] for k in seen} | {1, 3, 8}:
        for vs in (1, 63, 64, 1000, 16032, 18432):
            ids = [i for z in range(kz) for k0, k in [T.dh_k_range(vs, kz, z)] for i in range(k0, k0 + max(k, 0))]
            assert ids == list(range(vs))


@pytest.mark.parametrize("tm_count,d", [(48, 4096), (54, 3584), (18, 3584), (64, 2048), (14, 2048), (96, 8192),
                                        (12, 512), (1, 8), (3, 264), (5, 72)])
def test_dw_blocks_cover_every_tile_once_in_balanced_xcd_shares(tm_count, d):
    dtc = cdiv(d, 256)
    t = tm_count * dtc
    grid = T.dw_grid(tm_count, d)
    tiles = [T.dw_unit(b, tm_count, d) for b in range(grid)]
    live = [tt for tt in tiles if tt is not None]
    assert sorted(live) == sorted((tm, tn) for tm in range(tm_count) for tn in range(dtc))
    per_xcd = [sum(tiles[b] is not None for b in range(x, grid, 8)) for x in range(8)]
    assert max(per_xcd) - min(per_xcd) <= 1


def dw_rounds(v, d, r):
    # workgroup rounds of the dW launches with slabs of r row tiles (8 XCDs x 32 CUs)
    dtc, vt = cdiv(d, 256), cdiv(v, 384)
    return sum(cdiv(cdiv(min(r, vt - t0) * dtc, 8), 32) for t0 in range(0, vt, r))


@pytest.mark.parametrize("d,v", [(512, 4096), (2048, 128256), (4096, 128256), (3584, 152064), (8192, 128256),
                                 (2560, 151936), (1536, 151936), (5120, 152064), (3584, 1000)])
def test_the_slab_width_gives_the_dw_launches_the_fewest_rounds_in_its_range(d, v):
    # (more tokens than the few-token rule takes, so that the rule on rounds is the one that acts)
    info = B.lce_plan_info(B.problem(32768, d, v))
    vc = info["vc"]
    assert vc % 768 == 0 and info["nslab"] == cdiv(v, vc)
    assert (info["nslab"] > 1) == (v > 8192)
    lo = max(8192, 4 * d)
    hi = min(rup(v, 768), max(vc, min(24576, (160 << 20) // (2 * d))))
    if vc >= rup(v, 768):
        return                                  # one slab holds the whole vocabulary
    best = min(dw_rounds(v, d, r) for r in range(cdiv(lo, 768) * 2, hi // 384 + 1, 2))
    assert dw_rounds(v, d, vc // 384) <= best
    assert lo <= vc <= hi
    if (d, v) == (3584, 152064):                # the 3584-wide head: whole rounds, as few as the tiles allow
        assert dw_rounds(v, d, vc // 384) == cdiv(cdiv(v, 384) * cdiv(d, 256), 256) == 22


@pytest.mark.parametrize("tiles,nt,width", [(334, 48, 48), (54, 90, 54), (46, 48, 46), (96, 52, 24), (64, 24, 64),
                                            (12, 1, 12), (11, 2, 11), (3, 5, 3), (72, 64, 72), (17, 9, 17), (1, 1, 1),
                                            (8, 7, 8), (40, 33, 16)])
def test_forward_and_g_blocks_cover_every_tile_once_and_keep_w_tiles_on_one_xcd(tiles, nt, width):
    grid, gw = T.tile_order(tiles, nt, width)
    assert gw % 8 == 0
    got = [T.xcd_tile(b, tiles, gw, nt) for b in range(grid)]
    live = [t for t in got if t is not None]
    assert sorted(live) == [(tm, tn) for tm in range(tiles) for tn in range(nt)]
    a = tiles & ~7
    for b, t in enumerate(got):
        if t is None:
            continue
        tm, tn = t
        if tm < a:
            assert tm % 8 == b % 8          # each XCD keeps its own W tiles of the aligned part
        else:
            assert tn % 8 == b % 8          # and its own token tiles of the last few vocabulary tiles


@pytest.mark.parametrize("n,d,v,nslab", [(2048, 4096, 128256, 2), (1948, 3584, 152064, 2), (4096, 8192, 128256, 4),
                                         (4096, 1024, 152064, 3), (1024, 1024, 170000, 1), (4000, 256, 1000001, 16),
                                         (1, 64, 6000000, 9), (8192, 2048, 128256, 6), (16384, 4096, 128256, 7)])
def test_few_token_calls_take_the_fewest_equal_slabs_within_the_budget(n, d, v, nslab):
    info = B.lce_plan_info(B.problem(n, d, v))
    vc = info["vc"]
    assert info["nslab"] == nslab == cdiv(v, vc) and vc % 768 == 0
    rule = rup(max(8192, 4 * d, min(24576, (160 << 20) // (2 * d) // 6144 * 6144)), 6144)
    if rule // 384 * (info["npad"] // 256) > 1024:      # many tokens: the width of the rule (or near it: whole rounds)
        assert vc <= max(rule, 24576)
        return
    assert 2 * info["rows_g"] * vc <= 512 << 20
    assert vc - cdiv(v, nslab) < 768                    # equal slabs
    if nslab > 1:                                       # and one slab fewer would not fit G or a token tile's offsets
        w = rup(cdiv(v, nslab - 1), 768)
        assert 2 * info["rows_g"] * w > 512 << 20 or 512 * w > 2 ** 31 - 1
    for nv in (1, n):
        e, sizes, _ = walk(n, d, v, nv)
        e.check(sizes, f"n={n} d={d} v={v} nv={nv}")


def dh_split_blocks(n, nv, d, kz_max):
    """(xcd, row tile, column tile, K part, parts) of every block of a split dH launch."""
    for blk, tm, tn, z, kz, _ in T.dh_units(n, nv, d, kz_max, rup(rup(n, 256), 384)):
        yield blk & 7, tm, tn, z, kz


@pytest.mark.parametrize("n,d", [(256, 512), (1, 64), (700, 264), (2048, 4096), (1948, 3584), (4096, 2048), (4096, 4096),
                                 (4352, 5120), (1536, 8192), (11008, 2048)])
def test_split_dh_launches_cover_every_tile_and_part_once_on_all_xcds(n, d):
    kz_max = B.lce_plan_info(B.problem(n, d, 9000))["dh_kz"]
    assert kz_max > 1
    for nv in sorted({1, max(n // 3, 1), max(3 * n // 4, 1), n}):
        blocks = list(dh_split_blocks(n, nv, d, kz_max))
        kz = blocks[0][4]
        assert 1 <= kz <= kz_max
        want = sorted((tm, tn, z) for tm in range(cdiv(nv, 384)) for tn in range(cdiv(d, 256)) for z in range(kz))
        assert sorted(b[1:4] for b in blocks) == want
        per_xcd = [sum(b[0] == x for b in blocks) for x in range(8)]
        assert max(per_xcd) - min(per_xcd) <= 1


@pytest.mark.parametrize("d", [8, 56, 64, 72, 264, 1000, 1016])
def test_the_tail_mask_keeps_row_major_loads_inside_their_rows(d):
    # the last K slice of a width that is not a multiple of 64: lane j of a wave loads row j // 8 of each of 4
    # groups of 8 rows, chunk lane_chunk(j) for even groups and that ^ 1 for odd ones (a dense operand takes the odd
    # one's offset, mask included, from lane j ^ 1); every chunk below d is loaded once per row and none past d
    k0 = (cdiv(d, 64) - 1) * 64
    for dense in (True, False):
        for q in range(4):
            got = {}
            for j in range(64):
                src, sq = (j ^ (q & 1), 0) if dense else (j, q)     # whose offset register is used, and its group
                assert src // 8 == j // 8
                chunk = T.lane_chunk(src) ^ (sq & 1)
                assert chunk == T.lane_chunk(j) ^ (q & 1)
                assert T.chunk_exists(src, sq, k0, d) == (k0 + 8 * chunk < d)
                if T.chunk_exists(src, sq, k0, d):
                    got.setdefault(j // 8, []).append(chunk)
            for row in range(8):
                assert sorted(got.get(row, [])) == list(range(cdiv(d - k0, 8)))


@pytest.mark.parametrize("n,d,v", [(60000, 1400, 128256), (3000000, 8, 256), (70000, 1000, 128256), (9000, 72, 9216),
                                   (9000, 72, 9217), (5, 8, 1), (100000, 200, 1000000)])
def test_a_workspace_of_the_former_ragged_width_size_still_serves_the_forward(n, d, v):
    # widths that are not a multiple of 64 once took two partial rows per 256 ids, at most 64: callers may hold
    # workspaces of that size. The forward then takes groups of 24 tiles: 2 x 24 + 1 rows, or the tiles
    # themselves where they are at most 24; where the fixed array of lce_forward_noalloc holds only that form, it
    # is the one reported
    info = B.lce_plan_info(B.problem(n, d, v))
    npad = info["npad"]
    former = info["o_pm"] + 2 * rup(4 * 2 * min(cdiv(v, 256), 32) * npad, 256) + 4 * npad
    vt3 = cdiv(v, 384)
    rows = vt3 if vt3 <= 24 else 49
    least = info["o_pm"] + 2 * rup(4 * rows * npad, 256) + 4 * npad
    assert least <= former
    assert least == info["fwd_bytes"] if info["part_rows"] == rows else least < info["fwd_bytes"]
    ok = dict(H=0x100000, W=0x200000, targets=0x300000, loss=0x400000, lse=0x500000, n_valid=0x600000, dev_status=0,
              workspace=0x700000, stream=0)
    with pytest.raises(B.LceError) as e:                      # (one byte less than the least: refused, nothing launched)
        B.lce_forward(B.problem(n, d, v), **ok, workspace_bytes=least - 1)
    assert e.value.code == B.LCE_ERR_WORKSPACE


@pytest.mark.parametrize("tiles,nt", [(1, 1), (3, 1), (7, 9), (8, 1), (11, 1), (42, 13), (64, 1), (65, 2), (84, 10), (128, 2),
                                      (129, 2), (167, 1), (334, 2), (334, 6), (17, 16), (256, 8), (333, 7)])
def test_split_launches_cover_every_part_once_and_keep_a_tile_on_one_xcd(tiles, nt):
    grid, gw = T.tile_order(tiles, nt, tiles, True)
    seen, xcd = {}, {}
    for b in range(grid):
        p = T.tile_part(b, tiles, gw, nt)
        if p is None:
            continue
        tm, tn, parts, part = p
        assert 0 <= part < parts
        seen.setdefault((tm, tn, parts), []).append(part)
        xcd.setdefault((tm, tn), set()).add(b % 8)
    assert sorted(k[:2] for k in seen) == sorted((tm, tn) for tm in range(tiles) for tn in range(nt))
    for (tm, tn, parts), got in seen.items():
        assert sorted(got) == list(range(parts))
        assert len(xcd[(tm, tn)]) == 1


@pytest.mark.parametrize("v", [1, 385, 4096, 32003, 152064, 196609, 600000, 6000000])
def test_forward_partials_take_at_most_the_stated_bytes_per_token(v):
    # max(2 D, 4096) bytes per token (with a floor of 64 rows) whatever V, and up to 8 MiB more for the second
    # rows of cut tiles
    for d in (8, 64, 72, 1000, 1024, 2048, 4096, 8192):
        for n in (1, 64, 256, 1024, 2048, 4096, 5000, 16384):
            info = B.lce_plan_info(B.problem(n, d, v))
            assert 8 * info["part_rows"] * info["npad"] <= max(2 * d, 4096) * info["npad"] + (8 << 20), (n, d, v)


@pytest.mark.parametrize("n,d,v", [(70000, 1000, 128256), (15616, 8192, 24960), (140000, 72, 100000), (65536, 1024, 152064),
                                   (16384, 4096, 128256), (32768, 3584, 152064), (100000, 1400, 128256), (2048, 2048, 128256),
                                   (300, 264, 1000)])
def test_the_fixed_array_serves_exactly_the_problems_whose_reported_forward_bytes_it_holds(n, d, v):
    # one launch form per problem: what lce_forward_noalloc accepts is what lce_forward's reported size fits, and
    # nothing is launched either way here (no stream, no GPU)
    if __import__("torch").cuda.is_available():
        pytest.skip("host checks on made-up addresses")
    p = B.problem(n, d, v)
    with pytest.raises(B.LceError) as e:
        B.lce_forward_noalloc(p, 0, 0, 0, 0, 0, 0, 0, 0)
    assert (e.value.code == B.LCE_ERR_WORKSPACE) == (B.lce_workspace_size(p)[0] > B.LCE_NOALLOC_SCRATCH_BYTES)


@pytest.mark.parametrize("n,d,v", [(70000, 1000, 128256), (15616, 8192, 24960), (140000, 72, 100000), (65536, 1024, 152064)])
def test_a_forward_that_fits_the_fixed_array_in_the_least_form_reports_that_form(n, d, v):
    info = B.lce_plan_info(B.problem(n, d, v))
    vt3 = cdiv(v, 384)
    assert info["part_rows"] == (49 if d % 64 or vt3 > d // 4 else vt3)
    assert info["fwd_bytes"] <= B.LCE_NOALLOC_SCRATCH_BYTES
    assert info["o_pm"] + 2 * 4 * 2 * vt3 * info["npad"] > B.LCE_NOALLOC_SCRATCH_BYTES or not info["fwd_one_launch"]


@pytest.mark.parametrize("d", [8, 72, 1024, 2048, 4096, 8192])
def test_the_gradient_block_and_the_teacher_block_have_a_bound_that_v_does_not_move(d):
    # the rule's slab (max(8192, 4 D), or up to 24576 ids) of every token, or 512 MiB where that is more: never
    # a share of N V that grows with V. The distillation's block is 4 bytes per id and token
    for n in (1, 700, 2048, 4096, 5000, 16384):
        info = B.lce_plan_info(B.problem(n, d, 152064))
        for v in (152064, 400000, 6000000):
            g = 2 * info["rows_g"] * B.lce_plan_info(B.problem(n, d, v))["vc"]
            assert g <= max(2 * info["rows_g"] * max(30720, rup(4 * d, 6144)), 512 << 20), (n, d, v)
            kd = B.lce_kd_workspace_size(B.kd_problem(n, d, 64, v))[1]
            rest = info["o_hv"] + 2 * info["npad"] * (d + 64) + 4 * info["rows_g"] * d * 8 + 4096
            block = max(6 * info["rows_g"] * rup(max(8192, 4 * d), 6144), 768 << 20)
            assert kd <= rest + block, (n, d, v)
            # the forward: the teacher's block and 20 bytes per 256 of its ids and token, plus a running row
            kf = B.lce_kd_workspace_size(B.kd_problem(n, d, 64, v))[0]
            assert kf <= info["o_hv"] + info["npad"] * (128 + 44) + 4096 + block * 2 // 3 * 65 // 64, (n, d, v)
            assert B.lce_kd_workspace_size_fused(B.kd_problem(n, d, 64, v)) <= rest + block, (n, d, v)


def former_sizes(n, d, v, wide=True):
    """Forward and backward bytes that the library asked for before few-token slabs, cut tiles and one-launch
    forwards of narrow heads (``wide``: the plain calls' slabs, else the distillation's), and its slab width."""
    npad = rup(max(n, 1), 256)
    vt2, vt3, vround = cdiv(v, 256), cdiv(v, 384), rup(v, 768)
    vc = max(4 * d, 8192, min(24576, (160 << 20) // (2 * d) // 6144 * 6144) if wide else 0)
    vc = min(rup(vc, 6144), vround)
    if wide and vc < vround:                    # the multiple of 768 whose dW launches take the fewest rounds
        lo, hi = max(8192, 4 * d), min(vround, max(vc, min(24576, (160 << 20) // (2 * d))))
        cost = c0 = dw_rounds(v, d, vc // 384)
        best = vc // 384
        for r in range(cdiv(lo, 768) * 2, hi // 384 + 1, 2):
            c = dw_rounds(v, d, r)
            if c < cost or (c == cost and c < c0):
                best, cost = r, c
        vc = best * 384
    rows = max(2 * min(vt2, 32), vt3 if vt3 <= d // 4 else 2 * (vc // 384) + 1)
    prefix = 2 * rup(4 * npad, 256) + 256 + rup(2 * d * npad, 256)
    fwd = prefix + 2 * rup(4 * rows * npad, 256) + rup(4 * npad, 256)
    rows_g, dh_tiles = rup(npad, 384), cdiv(npad, 384) * cdiv(d, 256)
    bwd = prefix + rup(2 * rows_g * vc, 256) + 4 * rows_g * d * min(8, cdiv(256, dh_tiles))
    return fwd, bwd, vc


FORMER = [(n, d, v) for n in (1, 256, 700, 2048, 4096, 5000, 16384, 32768) for d in (8, 72, 512, 1000, 2048, 3584, 4096, 8192)
          for v in (5, 4096, 32003, 128256, 600000) if n * d < 1 << 30]


def test_workspaces_of_the_former_sizes_still_hold_every_call():
    # the least form needs no more than what callers were told before; one byte less is refused on the host
    ok = dict(H=0x100000, W=0x200000, targets=0x300000, lse=0x400000, n_valid=0x500000, grad_loss=0x600000, dH=0x700000,
              dW=0x800000, workspace=0x900000, stream=0)
    for n, d, v in FORMER:
        p = B.problem(n, d, v)
        fwd, bwd, _ = former_sizes(n, d, v)
        f, b = B.lce_workspace_size_least(p)
        f1, b1 = B.lce_workspace_size(p)
        assert f <= fwd and b <= bwd and f <= f1 and b <= b1, (n, d, v)
        with pytest.raises(B.LceError) as e:
            B.lce_backward(p, **ok, workspace_bytes=b - 1)
        assert e.value.code == B.LCE_ERR_WORKSPACE


@pytest.mark.parametrize("dt", [1000, 4096])
def test_distillation_workspaces_of_the_former_sizes_still_hold_every_call(dt):
    # (students at least 32 wide: narrower ones have no rows of H to spare for the tiles' values of one slab)
    for n, d, v in FORMER:
        if d < 32:
            continue
        npad, vt2 = rup(max(n, 1), 256), cdiv(v, 256)
        fwd, bwd, vc = former_sizes(n, d, v, wide=False)
        p_bytes, hvt = 4 * vc * npad, rup(2 * dt * npad, 256) if dt % 64 == 0 else 0
        q = rup(8 * vt2 * npad, 256)
        f, b = B.lce_kd_workspace_size_least(B.kd_problem(n, d, dt, v))
        assert f <= fwd + rup(4 * npad, 256) + q + rup(p_bytes, 256) + hvt, (n, d, v)
        assert b <= bwd + p_bytes + hvt, (n, d, v)
        full = B.lce_kd_workspace_size(B.kd_problem(n, d, dt, v))
        assert f <= full[0] and b <= full[1] == B.lce_kd_workspace_size_fused(B.kd_problem(n, d, dt, v))


@pytest.mark.parametrize("n,d,v,nv", [(16384, 256, 8192, 12288), (9000, 512, 3001, 420), (9000, 512, 20000, 420),
                                      (2048, 4096, 64512, 1536), (16384, 4096, 18432, 12288), (300, 264, 1000, 300), (700, 64, 500, 0)])
def test_the_merged_launch_runs_every_block_of_both_and_starts_the_longer_units(n, d, v, nv):
    info = B.lce_plan_info(B.problem(n, d, v))
    dh, dw = T.dh_grid(n, d, info["dh_kz"]), T.dw_grid(cdiv(v, 384), d)
    first = T.dw_first(nv, info["dh_kz"], v)
    got = [T.dhdw_block(b, dh, dw, first) for b in range(dh + dw)]
    assert sorted(got) == list(range(dh + dw))
    for b, g in enumerate(got):
        assert (g if g < dh else g - dh) % 8 == b % 8              # each block of either launch keeps its XCD
    assert first == (nv * info["dh_kz"] > v)                        # dW's K against that of a dH unit's most parts
    assert (got[0] >= dh) == first
