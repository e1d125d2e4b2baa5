"""Host-side tests of plans that the C ABI does not show (no GPU): the tile and
the threads that the items of a batch take, read from the work table before
anything is uploaded, and those of copies between differing records.  A helper
compiled here against the library's own headers calls the planner."""
import ctypes
import os
import subprocess

import pytest

from paper_2106_04284_amd import build as B
from paper_2106_04284_amd import llama as L
from paper_2106_04284_amd import workloads as W

HELPER = r"""
#include "batch.hpp"
using namespace llama;
static uint32_t tile_of(uint32_t kind, const TileHeader& h) { return kind == kItemTile ? 1u << h.log2_tile : 0u; }
extern "C" int batch_table(size_t n, const llama_copy_item* items, const llama_copy_options* o, uint32_t* threads,
                           uint32_t* tiles)
{
    try {
        const BatchTable t = build_batch_table(n, items, o, *threads);
        for (size_t k = 0; k < n && k < t.items.size(); k++)
            tiles[k] = tile_of(t.items[k].kind, t.items[k].h);
        return 0;
    } catch (const Error& e) {
        return e.status;
    }
}
extern "C" int batch_tile(const llama_copy_item* it, uint32_t threads, uint32_t budget, uint32_t* tile)
{
    try {
        const Plan p = batch_plan(make_request(it->src, it->src_blobs, it->dst, it->dst_blobs, true), threads, 0, 0, budget);
        *tile = p.path == LLAMA_PATH_TILE ? 1u << p.tile.h.log2_tile : 0u;
        return 0;
    } catch (const Error& e) {
        return e.status;
    }
}
"""

HELPER += r"""
extern "C" int leaves_tile(const llama_mapping_desc* src, const llama_mapping_desc* dst, const uint32_t* leaf,
                           uint32_t* out)
{
    try {
        const std::vector<Plan> p = leaves_plans(src, nullptr, dst, nullptr, leaf, nullptr, false);
        out[0] = p.size() == 1 && p[0].path == LLAMA_PATH_TILE && (p[0].tile.h.flags & kTileDirectStore);
        out[1] = 1u << p[0].tile.h.log2_tile;
        out[2] = p[0].threads;
        return 0;
    } catch (const Error& e) {
        return e.status;
    }
}
"""

HELPER += r"""
extern "C" int gathered(const llama_mapping_desc* src, const llama_mapping_desc* dst, uint32_t* out)
{
    try {
        const Request rq = make_request(src, nullptr, dst, nullptr, false, true);
        const std::vector<SubCopy> c = split_copies(src, dst, rq, true, nullptr);
        if (c.empty() || !c[0].plan)
            return -1;
        const Plan& p = *c[0].plan;
        out[0] = (p.tile.h.flags & kTileVirtualSrc) != 0;
        out[1] = p.tile.h.slots;
        out[2] = p.lds_bytes;
        out[3] = p.lds_launch;
        return 0;
    } catch (const Error& e) {
        return e.status;
    }
}
"""

HELPER += r"""
extern "C" int aside(const llama_mapping_desc* src, const llama_mapping_desc* dst, uint32_t* out)
{
    try {
        const Plan p = make_plan(make_request(src, nullptr, dst, nullptr, false, false), nullptr);
        out[0] = p.path == LLAMA_PATH_TILE && (p.tile.h.flags & kTileDirectStore);
        out[1] = p.lds_bytes;
        out[2] = p.lds_launch;
        return 0;
    } catch (const Error& e) {
        return e.status;
    }
}
"""

RECORDS = dict(W.RECORDS, small=["u8", "u16"], pair=["f32", "f32"], vec3=[("f32", 3)], twelve=[("f32", 12)], vec4=[("f32", 4)])


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    L.lib()
    d = tmp_path_factory.mktemp("batch_plan")
    src, so = d / "helper.cpp", d / "helper.so"
    src.write_text(HELPER)
    subprocess.run(["g++"] + B.CXX_FLAGS + ["-O1", "-shared", str(src), "-o", str(so), B.LIB,
                                            "-Wl,-rpath," + os.path.dirname(B.LIB)], check=True)
    return ctypes.CDLL(str(so))


def _items(rec, src, dst, counts, at=1 << 40):
    r, out = L.Record(RECORDS[rec]), []
    for n in counts:
        sides = []
        for kind, lanes in (src, dst):
            m = L.Mapping(r, kind, [n], lanes)
            blobs = []
            for size in m.blob_sizes():
                blobs.append((at, size))
                at += (size + 511) // 256 * 256
            sides += [m, blobs]
        out.append(tuple(sides))
    return L._Items(out)


def _tile(planner, rec, src, dst, n, threads=256, budget=0):
    items, tile = _items(rec, src, dst, [n]), ctypes.c_uint32()
    assert planner.batch_tile(items.arr, threads, budget, ctypes.byref(tile)) == 0
    return tile.value


A, S, Q32 = ("aos_packed", 0), ("soa_multi", 0), ("aosoa", 32)


@pytest.mark.parametrize("src,dst", [(A, S), (S, A), (Q32, S), (S, Q32)])
def test_batch_tiles_by_bytes(planner, src, dst):
    """The default tile holds at most 12,800 source bytes, or 256 records, and
    16 records per thread, and no more than the item."""
    for rec, tile in [("small", 4096), ("pair", 1024), ("vec3", 1024), ("vec4", 512), ("particle", 256)]:
        assert _tile(planner, rec, src, dst, 10 ** 6) == tile, rec
    assert _tile(planner, "small", src, dst, 10 ** 6, threads=128) == 2048
    assert _tile(planner, "small", src, dst, 10 ** 6, threads=64) == 1024
    assert _tile(planner, "particle", src, dst, 10 ** 6, threads=64) == 256
    for n, tile in [(100, 128), (300, 512), (1000, 1024), (1025, 2048)]:
        assert _tile(planner, "small", src, dst, n) == tile, n


def test_batch_tiles_of_direct_loads(planner):
    """A tile loaded into registers may hold 100 bytes per thread (512 mixed
    records are 98 per thread of 256); other modes keep 12,800."""
    for threads, tile in [(256, 1024), (128, 512)]:
        assert _tile(planner, "listing1", S, A, 10 ** 6, threads) == tile
    assert _tile(planner, "listing1", A, S, 10 ** 6) == 512
    for threads, tile in [(256, 512), (128, 256)]:
        assert _tile(planner, "mixed", S, A, 10 ** 6, threads) == tile
    assert _tile(planner, "mixed", A, S, 10 ** 6) == 256


def test_batch_tiles_of_a_given_budget(planner):
    """A given LDS budget alone bounds the tile (the autotuner's candidates):
    particles in one region of 28 bytes per record, one 16-byte granule of
    room and the leaf table."""
    assert [_tile(planner, "particle", A, S, 10 ** 6, budget=k * 1024) for k in (8, 16, 31, 48)] == [256, 512, 1024, 1024]
    assert [_tile(planner, "mixed", A, S, 10 ** 6, budget=k * 1024) for k in (16, 31, 64)] == [256, 512, 1024]


@pytest.mark.parametrize("rec,size", [("small", 3), ("pair", 8), ("vec4", 16), ("particle", 28), ("mixed", 49)])
def test_batch_threads_by_item(planner, rec, size):
    """128 threads where every item is small (at most 128 KiB of records),
    whatever its tiles; one larger item, or a count that is given, decides."""
    def threads(counts, given=None):
        items, th = _items(rec, A, S, counts), ctypes.c_uint32()
        tiles = (ctypes.c_uint32 * len(counts))()
        o = L.CopyOptions(0, 0, given, 0, 0) if given else None
        assert planner.batch_table(ctypes.c_size_t(len(counts)), items.arr, ctypes.byref(o) if o else None,
                                   ctypes.byref(th), tiles) == 0
        assert all(0 < t <= max(256, 16 * th.value) for t in tiles)
        return th.value
    edge = 128 * 1024 // size
    many = [100] * 2100  # units enough for the size of the items to decide
    assert threads(many + [edge]) == 128
    assert threads(many + [edge + 1]) == 256
    assert threads([10 ** 6] * 3) == 256
    assert threads([100], given=256) == 256 and threads([10 ** 6], given=64) == 64


def test_small_batches_keep_small_tiles(planner):
    """A batch that would have fewer than 1,024 units (direct stores: 512) keeps
    256 records per tile, and 256 threads unless the first 512 records of its
    items are at most 8 KiB; the same items in a larger batch take the larger
    tile, whichever batch was planned first."""
    def table(rec, counts, src=S, dst=A):
        items, th = _items(rec, src, dst, counts), ctypes.c_uint32()
        tiles = (ctypes.c_uint32 * len(counts))()
        assert planner.batch_table(ctypes.c_size_t(len(counts)), items.arr, None, ctypes.byref(th), tiles) == 0
        return set(tiles), th.value
    for _ in range(2):
        assert table("vec3", [1024] * 800) == ({512}, 128)     # 3,200 units of 256, 1,600 of 512, 800 of 1,024
        assert table("vec3", [1024] * 1024) == ({1024}, 128)
        assert table("vec3", [1024] * 500) == ({256}, 128) and table("vec3", [1024] * 512) == ({512}, 128)
        assert table("vec3", [1024] * 500, A, S) == ({512}, 128)   # a direct store: 1,000 units of 512, 500 of 1,024
        assert table("vec3", [1024] * 512, A, S) == ({1024}, 128)
        assert table("listing1", [10 ** 4] * 50) == ({256}, 256)   # 1,000 units of 512
        assert table("listing1", [10 ** 4] * 60) == ({512}, 256)
        assert table("listing1", [10 ** 4] * 25, A, S) == ({256}, 256)
        assert table("listing1", [10 ** 4] * 26, A, S) == ({512}, 256)
        assert table("mixed", [10 ** 6] * 3) == ({256}, 256)       # tiles of 25 KB: 5,860 units of 512
        assert table("mixed", [10 ** 6] * 4) == ({512}, 256)       # 7,816
        assert table("listing1", [10 ** 6] * 6) == ({512}, 256)    # tiles of 21.5 KB: 5,862 units of 1,024; 10.7 KB fit
        assert table("listing1", [10 ** 6] * 7) == ({1024}, 256)
        assert table("particle", [1000] * 150) == ({256}, 256)     # 600 units, 28,000 bytes each
        assert table("particle", [256] * 150) == ({256}, 128)      # 7,168 bytes each


@pytest.mark.parametrize("src,dst,threads", [
    (("particle",) + A, ("fields",) + S, 256), (("particle",) + Q32, ("fields",) + S, 256),
    (("fields", "soa_multi", 0), ("particle",) + Q32, 256), (("fields", "aos_aligned", 0), ("fields",) + S, 192)])
def test_differing_records_keep_their_threads(planner, src, dst, threads):
    """A particle's fields without the mass, from and into particles: a packed
    side that holds the mass too is sized as before, 256 threads; without one,
    24 bytes of 256 records feed 192."""
    records = {"particle": W.PARTICLE, "fields": [("f32", 6)]}
    a, b = (L.Mapping(L.Record(records[r]), kind, [10 ** 6], lanes) for r, kind, lanes in (src, dst))
    leaf = (ctypes.c_uint32 * 7)(*range(6), L.NO_LEAF)
    out = (ctypes.c_uint32 * 3)()
    assert planner.leaves_tile(ctypes.byref(a.desc), ctypes.byref(b.desc), leaf, out) == 0
    assert list(out) == [1, 256, threads]


@pytest.mark.parametrize("rec,first,count,a,b,dst,least", [
    ("particle", 0, 3, ("aosoa", 32), ("aosoa", 32), A, 6),       # 2 chunks
    ("particle", 0, 5, ("aosoa", 32), ("soa_multi", 0), A, 6),    # 3
    ("particle", 0, 4, ("aosoa", 32), ("soa_multi", 0), A, 8),    # 4
    ("particle", 0, 3, ("aosoa", 32), ("soa_multi", 0), ("aosoa", 8), 8),
    ("lbm", 0, 10, ("soa_multi", 0), ("aosoa", 32), ("aos_aligned", 0), 8)])
def test_gathered_sources_keep_workgroups(planner, rec, first, count, a, b, dst, least):
    """The LDS that a large copy sets aside beyond its tile's own leaves a
    gathered source 6 workgroups per compute unit, 8 from 4 chunks on."""
    n = (5 << 28) // L.Record(RECORDS[rec]).info()[1]  # 1.25 GiB
    src = L.Mapping(L.Record(RECORDS[rec]), "split", [n], split=(first, count, a, b))
    to = L.Mapping(L.Record(RECORDS[rec]), dst[0], [n], dst[1])
    out = (ctypes.c_uint32 * 4)()
    assert planner.gathered(ctypes.byref(src.desc), ctypes.byref(to.desc), out) == 0
    gathered, chunks, own, aside = out
    assert gathered and (chunks <= 3) == (least == 6)
    assert 0 < own <= 160 * 1024 // least and aside <= 160 * 1024 // least


@pytest.mark.parametrize("rec,first,count,a,b", [
    ("listing1", 1, 6, ("aosoa", 32), ("soa_single", 0)), ("mixed", 4, 3, ("aosoa", 64), ("soa_multi", 0))])
def test_gathered_direct_stores_keep_workgroups(planner, rec, first, count, a, b):
    """... and a gathered source that is stored directly 12."""
    n = (5 << 28) // L.Record(RECORDS[rec]).info()[1] // 64 * 64
    src = L.Mapping(L.Record(RECORDS[rec]), "split", [n], split=(first, count, a, b))
    to = L.Mapping(L.Record(RECORDS[rec]), "soa_multi", [n])
    out = (ctypes.c_uint32 * 4)()
    assert planner.gathered(ctypes.byref(src.desc), ctypes.byref(to.desc), out) == 0
    gathered, chunks, own, aside = out
    assert gathered and chunks >= 2
    assert 0 < own <= 160 * 1024 // 10 and 0 < aside <= 160 * 1024 // 12


def _part_of(planner, rec, kind, lanes, leaves):
    """Mode, tile and threads of the copy of some leaves of `rec` into SoA."""
    a = L.Mapping(L.Record(rec), kind, [10 ** 6], lanes)
    b = L.Mapping(L.Record([rec[k] for k in leaves]), "soa_multi", [10 ** 6])
    out = (ctypes.c_uint32 * 3)()
    assert planner.leaves_tile(ctypes.byref(a.desc), ctypes.byref(b.desc), (ctypes.c_uint32 * len(leaves))(*leaves), out) == 0
    return list(out)


@pytest.mark.parametrize("rec,leaves,threads", [
    (["f32"] * 3, [0, 1], 64), (["f32"] * 6, [1, 2, 3, 4], 128), (["f32"] * 6, [0, 1, 2, 3, 4], 192),
    (["f32"] * 7, range(3), 128), (["f32"] * 7, range(6), 256)])
def test_narrow_parts_take_few_threads(planner, rec, leaves, threads):
    """Some leaves of a packed record into SoA: 256 records, and 28 bytes of the
    leaves per thread in whole waves, rounded up from 20 bytes on and where most
    of the record is other leaves."""
    assert _part_of(planner, rec, "aos_packed", 0, list(leaves)) == [1, 256, threads]


@pytest.mark.parametrize("rec,leaves", [
    (["f64"] * 3 + ["f32"] * 4 + ["i32"] * 2 + ["u8"], [7]), (["f64"] * 3 + ["f32"] * 6 + ["u8"], [3, 4]),
    (["u16", "f32", "f32", "f64"] + ["bool"] * 3, [4, 5, 6]), (["u16", "f32", "f32", "f64"] + ["bool"] * 3, [0, 1])])
def test_parts_of_aligned_records_keep_256(planner, rec, leaves):
    """Some leaves of an aligned record: the tile is 8 KiB of whole records."""
    mode, tile, _ = _part_of(planner, rec, "aos_aligned", 0, leaves)
    assert (mode, tile) == (1, 256)


@pytest.mark.parametrize("rec,kind,groups", [
    ("listing1", "aos_aligned", 8), ("mixed", "aos_aligned", 8), ("lbm", "aos_aligned", 5), ("twelve", "aos_packed", 7)])
def test_direct_stores_of_narrow_leaves_keep_workgroups(planner, rec, kind, groups):
    """Large direct stores of leaves under 4 bytes leave 8 workgroups a compute
    unit, others 64 KiB of tiles and 14 waves from records, at least 4."""
    n = (5 << 28) // L.Record(RECORDS[rec]).info()[1] // 64 * 64
    a, b = (L.Mapping(L.Record(RECORDS[rec]), k, [n]) for k in (kind, "soa_multi"))
    out = (ctypes.c_uint32 * 3)()
    assert planner.aside(ctypes.byref(a.desc), ctypes.byref(b.desc), out) == 0
    assert out[0] and out[1] <= 160 * 1024 // groups and out[2] == 160 * 1024 // groups // 512 * 512


def test_wide_tiles_where_they_are_most_of_the_batch(planner):
    """Tiles of more than 12.5 KB raise the LDS of their mode's whole launch:
    they are taken only where their class is three of four units."""
    def tile(rec, src, big, others):
        one, two = _items(rec, src, A, [10 ** 6] * big), _items("particle", A, S, [10 ** 6] * others, 1 << 44)
        n = big + others
        arr = (type(one.arr[0]) * n)(*([one.arr[k] for k in range(big)] + [two.arr[k] for k in range(others)]))
        th, tiles = ctypes.c_uint32(), (ctypes.c_uint32 * n)()
        assert planner.batch_table(ctypes.c_size_t(n), arr, None, ctypes.byref(th), tiles) == 0
        return set(tiles)
    for _ in range(2):
        assert tile("mixed", S, 9, 3) == {256, 512}  # the particles keep 256
        assert tile("mixed", S, 9, 4) == {256}
