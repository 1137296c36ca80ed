"""How a batched launch shares its workgroups out (csrc/launch_shape.h, host code, built here with g++)."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_05699_amd", "csrc")
SOURCE = """
#include "launch_shape.h"
extern "C" int share_out(const long long* tiles, int count, long long budget, srft_share* out, int most, int* grid) {
    return srft_share_out(tiles, count, budget, out, most, grid);
}
extern "C" int even_blocks(long long tiles, long long count, long long budget) { return srft_even_blocks(tiles, count, budget); }
extern "C" int even_segment(unsigned block, int blocks) { return srft_even_segment(block, srft_even_magic(blocks)); }
extern "C" int spread(long long tiles, long long count, long long budget, int* segment, int* place, int* blocks, int most) {
    const int each = srft_even_blocks(tiles, count, budget);
    if (!each) return 0;
    const srft_even_shape e = srft_even_spread(tiles, count, budget, each);
    const int grid = srft_even_grid(e, count);
    for (int b = 0; b < grid && b < most; ++b) {
        const int i = srft_even_segment(b, e), start = srft_even_start(i, e);
        segment[b] = i, place[b] = b - start, blocks[b] = srft_even_start(i + 1, e) - start;
    }
    return grid;
}
extern "C" int even_step(const void* const* p, int count, long long* step) { return srft_even_step(p, count, step); }
extern "C" int flush_fits(long long n_vec, long long page_rows, long long n_seq, long long t, long long units) {
    return srft_flush_fits(n_vec, page_rows, n_seq, t, units);
}
extern "C" int write_staged(int d, int g, int bits, int lines, long long tiles, long long workgroups, long long units) {
    return srft_write_staged(d, g, bits, lines, tiles, workgroups, units);
}
extern "C" int read_through(int d, int lines, long long bytes) { return srft_read_through(d, lines, bytes); }
extern "C" int flush_staged(int d, long long tiles) { return srft_flush_staged(d, tiles); }
extern "C" int fold_through(int d, int bits, int lines, long long bytes) { return srft_fold_through(d, bits, lines, bytes); }
extern "C" int copy_launches(int t) { return srft_copy_launches(t); }
extern "C" long long copy_first(int i) { return srft_copy_first(i); }
extern "C" unsigned copy_tokens(int i, int t) { return srft_copy_tokens(i, t); }
"""


class Share(C.Structure):
    _fields_ = [("segment", C.c_int), ("first_block", C.c_int), ("blocks", C.c_int), ("tile", C.c_longlong), ("tiles", C.c_longlong)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    at = tmp_path_factory.mktemp("launch_shape")
    (at / "s.cpp").write_text(SOURCE)
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(at / "s.cpp"), "-o", str(at / "s.so")], check=True)
    return C.CDLL(str(at / "s.so"))


@pytest.fixture(scope="module")
def share_out(lib):
    def call(tiles, budget, most=64):
        out, grid = (Share * (most + 1))(), C.c_int()
        out[most].segment = -77
        n = lib.share_out((C.c_longlong * len(tiles))(*tiles), len(tiles), C.c_longlong(budget), out, most, C.byref(grid))
        assert out[most].segment == -77 and n <= most
        return list(out[:n]), grid.value
    return call


def _check(shares, grid, tiles):
    """Every tile of every segment once, every workgroup with a tile, places in order."""
    place, done = 0, [0] * len(tiles)
    for s in shares:
        assert s.first_block == place and 1 <= s.blocks <= s.tiles and s.tile == done[s.segment]
        place += s.blocks
        done[s.segment] += s.tiles
    assert place == grid and done == list(tiles)
    assert [s.segment for s in shares] == sorted(s.segment for s in shares)


def _tiles_per_die(shares, grid):
    load, q, r = [], grid // 8, grid % 8
    walked = [s.tiles // s.blocks + (k < s.tiles % s.blocks) for s in shares for k in range(s.blocks)]
    for die in range(8):
        first = die * q + min(die, r)
        load.append(sum(walked[first:first + q + (die < r)]))
    return load


@pytest.mark.parametrize("plans", [1, 2, 4])
@pytest.mark.parametrize("budget", [512, 1024, 1280])
@pytest.mark.parametrize("ratio", [1.02, 1.36, 1.5, 1.99, 2.3, 3.7])
def test_few_plans_load_the_dies_alike(share_out, plans, budget, ratio):
    tiles = [int(budget * ratio / plans)] * plans
    shares, grid = share_out(tiles, budget)
    _check(shares, grid, tiles)
    load = _tiles_per_die(shares, grid)
    assert max(load) - min(load) <= 2, load              # (uncut: 256 against 128 at 2 plans x 698 tiles on 1024 workgroups)


def test_shares_of_random_launches(share_out):
    rng = random.Random(5)
    for _ in range(3000):
        count = rng.choice([1, 2, 3, 4, 5, 9, 33, 57, 58, 63, 64])
        tiles = [rng.choice([1, 2, rng.randint(1, 40), rng.randint(1, 3000)]) for _ in range(count)]
        budget = rng.choice([1, 3, 7, 8, 9, 20, 512, 1023, 1024, 10 ** 9])
        shares, grid = share_out(tiles, budget)
        _check(shares, grid, tiles)
        assert len(shares) <= count + 7
        assert grid <= max(budget, count) + count


def test_the_largest_launch_and_a_full_table(share_out):
    tiles = [2 ** 28] * 64                               # 2^33 vectors each
    shares, grid = share_out(tiles, 1024)
    _check(shares, grid, tiles)
    assert len(shares) == 64
    tiles = [1] * 62 + [700] * 2                         # the cuts would not fit the table: none is made
    shares, grid = share_out(tiles, 1024)
    _check(shares, grid, tiles)
    assert len(shares) == 64


@pytest.mark.parametrize("t", [1, 2 ** 24 - 1, 2 ** 24, 2 ** 24 + 1, 3 * 2 ** 24, 127 * 2 ** 24, 127 * 2 ** 24 + 1, 2 ** 31 - 1])
def test_the_copy_of_new_tokens_takes_every_one_of_them_once(lib, t):
    lib.copy_first.restype, lib.copy_tokens.restype = C.c_longlong, C.c_uint
    done = 0
    for i in range(lib.copy_launches(t)):
        assert lib.copy_first(i) == done and 0 < lib.copy_tokens(i, t) <= 2 ** 24
        done += lib.copy_tokens(i, t)
    assert done == t                                     # (a 32-bit count of tokens never got past 127 x 2^24)


def test_segments_of_one_length_share_like_the_table(lib, share_out):
    """Where a batch of equal segments goes out without a table, every segment gets the workgroups the table would give it."""
    rng, even = random.Random(6), 0
    for _ in range(4000):
        count = rng.choice([1, 2, 3, 4, 5, 8, 9, 33, 56, 64])
        tiles = rng.choice([1, 2, rng.randint(1, 40), rng.randint(1, 40000), 2 ** 28])
        budget = rng.choice([1, 3, 7, 8, 20, 256, 512, 768, 1024, 1280, 10 ** 6])
        blocks = lib.even_blocks(C.c_longlong(tiles), C.c_longlong(count), C.c_longlong(budget))
        shares, grid = share_out([tiles] * count, budget)
        if not blocks:
            assert count > budget or len(shares) > count or blocks_too_many(grid, shares) or count <= 4
            continue
        even += 1
        assert grid == blocks * count                    # (grids of a few workgroups are cut as well: parts of a segment add up)
        assert all(sum(s.blocks for s in shares if s.segment == i) == blocks for i in range(count))
        assert len(shares) == count or blocks < 8
    assert even > 2000


def blocks_too_many(grid, shares):
    return grid * max(s.blocks for s in shares) >= 2 ** 31


@pytest.mark.parametrize("blocks", [1, 2, 3, 7, 18, 19, 85, 256, 511, 512, 1023, 1280, 46340])
def test_workgroup_to_segment_without_a_table(lib, blocks):
    for count in (1, 2, 3, 64, 101, 1280, 8192):
        grid = blocks * count
        if grid * blocks >= 2 ** 31:
            continue
        for block in {0, grid - 1} | {k * blocks + e for k in range(0, count, max(1, count // 50)) for e in (0, blocks - 1)}:
            assert lib.even_segment(block, blocks) == block // blocks, (blocks, count, block)


@pytest.mark.parametrize("n_seq,R", [(1, 1), (1, 16), (2, 16), (3, 7), (8, 16), (70, 5), (512, 16), (46340, 1)])
def test_rows_of_a_flush_divide_exactly(lib, n_seq, R):
    """Row v of a flush is in page v / (n_seq R), there of sequence rest / R, for every size that is let through."""
    page_rows, ll = n_seq * R, C.c_longlong
    most = (2 ** 31 // page_rows - 1) // page_rows * page_rows
    assert most >= page_rows
    rng = random.Random(page_rows)
    for v in {0, most - 1} | {rng.randrange(most) for _ in range(300)} | {k * page_rows + e for k in range(1, most // page_rows, max(1, most // page_rows // 50)) for e in (-1, 0)}:
        page = lib.even_segment(v, page_rows)
        assert page == v // page_rows and lib.even_segment(v - page * page_rows, R) == v % page_rows // R
    # what no longer divides or counts exactly is refused: the rows, the view's units, the new tokens' units
    assert lib.flush_fits(ll(page_rows), ll(page_rows), ll(n_seq), ll(R), ll(4)) == 1
    assert lib.flush_fits(ll(2 ** 31 // page_rows), ll(page_rows), ll(n_seq), ll(R), ll(4)) == 0
    assert lib.flush_fits(ll(page_rows), ll(page_rows), ll(n_seq), ll(2 ** 31 // 4 // n_seq + 1), ll(4)) == 0


def test_a_flush_as_large_as_its_units_are_counted(lib):
    ll = C.c_longlong
    assert lib.flush_fits(ll(2 ** 26 - 33), ll(16), ll(1), ll(2 ** 26 - 1), ll(32)) == 1
    assert lib.flush_fits(ll(2 ** 26 - 16), ll(16), ll(1), ll(2 ** 26 - 1), ll(32)) == 0
    assert lib.flush_fits(ll(2 ** 26 - 33), ll(16), ll(1), ll(2 ** 26), ll(32)) == 0


def test_addresses_a_constant_step_apart(lib):
    def step(*p):
        out = C.c_longlong()
        return (out.value if lib.even_step((C.c_void_p * len(p))(*p), len(p), C.byref(out)) else None)
    assert step(4096) == 0 and step(4096, 4096, 4096) == 0
    assert step(4096, 8192, 12288) == 4096 and step(2 ** 40, 2 ** 40 - 16, 2 ** 40 - 32) == -16
    assert step(4096, 8192, 12304) is None and step(16, 32, 48, 16) is None
    assert step(0x7F0000000000, 0x10) == 0x10 - 0x7F0000000000


# `each`: workgroups that every segment gets, 0 where the batch goes out with a table (one segment cut where the dies meet; more
# segments than workgroups)
@pytest.mark.parametrize("count,tiles,budget,each", [
    (1, 5, 3, 0), (10, 4, 9, 0), (52, 128, 512, 9), (56, 256, 1024, 18), (80, 300, 1024, 12), (100, 22, 768, 7), (7, 9, 8, 1), (5, 3, 14, 2),
    (9, 1, 9, 1), (3, 1000, 7, 2), (1000, 3, 2048, 2), (64, 16, 512, 8), (33, 4096, 1024, 31), (2048, 100, 2048, 1)])
def test_leftover_workgroups_are_spread(lib, count, tiles, budget, each):
    most = 1 << 16
    segment, place, blocks = ((C.c_int * most)() for _ in range(3))
    grid = lib.spread(C.c_longlong(tiles), C.c_longlong(count), C.c_longlong(budget), segment, place, blocks, most)
    assert lib.even_blocks(C.c_longlong(tiles), C.c_longlong(count), C.c_longlong(budget)) == each
    if each == 0:
        assert grid == 0
        return
    assert grid <= most and each * count <= grid <= max(budget, each * count) and grid <= tiles * count
    assert grid == min(budget, tiles * count) or grid * grid * count >= 2 ** 31 or min(budget, tiles * count) ** 2 * count >= 2 ** 31
    seen = {}
    for b in range(grid):                                # every segment once, in order, its workgroups 0 .. blocks - 1
        assert segment[b] == (segment[b - 1] if b and place[b] else (segment[b - 1] + 1 if b else 0))
        assert place[b] == (place[b - 1] + 1 if b and segment[b] == segment[b - 1] else 0)
        seen[segment[b]] = seen.get(segment[b], 0) + 1
    assert sorted(seen) == list(range(count))
    assert all(blocks[b] == seen[segment[b]] and seen[segment[b]] in (each, each + 1) and blocks[b] <= tiles for b in range(grid))


@pytest.mark.parametrize("d,last", [(128, 60_000_000), (256, 200_000_000)])
def test_a_folded_record_is_written_through_where_that_is_faster(lib, d, last):
    """Short launches; of 8-bit records at d = 128 only those that start at a multiple of 64 bytes."""
    ll = C.c_longlong
    for n in (80, 30_000_000, last):
        assert [lib.fold_through(d, bits, lines, ll(n)) for bits, lines in ((4, 1), (4, 0), (8, 1), (8, 0))] == [1, 1, 1, d == 256]
    for n in (last + 1, 56 * 8192 * 336, 1_409_286_144) if d == 128 else (last + 1, 1_409_286_144):
        assert not any(lib.fold_through(d, bits, lines, ll(n)) for bits, lines in ((4, 1), (4, 0), (8, 1), (8, 0)))


# d, g, bits, workgroups that fit, most tiles through LDS, fewest of the sizes beyond that go through LDS again; the last size below
@pytest.mark.parametrize("d,g,bits,wgs,last,again,low", [
    (64, 32, 4, 2048, 9 * 2048, None, 768), (64, 64, 8, 2048, 9 * 2048, None, 768), (96, 32, 4, 1280, 11 * 1280, 22 * 1280, 768), (96, 96, 8, 1024, 11 * 1024, 22 * 1024, 768),
    (128, 16, 4, 768, None, None, 768), (128, 32, 8, 768, None, None, 768), (128, 128, 4, 768, None, None, 768), (128, 32, 4, 768, 14 * 768, None, 768),
    (160, 32, 4, 512, 16 * 512, None, 768), (192, 32, 4, 256, 16 * 256, None, 1152), (224, 16, 8, 256, 16 * 256, None, 896), (256, 32, 4, 256, 16 * 256, None, 768)])
def test_a_plain_record_goes_through_lds_where_that_is_faster(lib, d, g, bits, wgs, last, again, low):
    def staged(tiles, lines=1, units=256):
        return lib.write_staged(d, g, bits, lines, C.c_longlong(tiles), C.c_longlong(wgs), C.c_longlong(units))

    assert not staged(1) and not staged(low) and staged(low + 1)
    assert not staged(low // 4, units=64) and staged(low // 4 + 1, units=64)          # (the least goes with the compute units)
    far = 2 ** 27
    if last is None:
        assert staged(far)
    else:
        assert staged(last) and not staged(last + 1) and staged(far) == (again is not None)
        if again:
            assert not staged(again - 1) and staged(again)
    # 16 bytes into a line: from the lanes up to some tiles a compute unit, at d = 128 always
    at = max(low, {64: 2048, 96: 1280, 160: 0}.get(d, 1536))
    assert not staged(at, lines=0) and staged(at + 1, lines=0) == (d != 128) and staged(far, lines=0) == (again is not None)


def test_a_record_of_d_32_is_always_stored_from_the_lanes(lib):
    assert not any(lib.write_staged(32, 32, 4, 1, C.c_longlong(t), C.c_longlong(2048), C.c_longlong(256)) for t in (1, 769, 5000, 20000, 10 ** 6))


@pytest.mark.parametrize("d", [32, 64, 96, 128, 160, 192, 224, 256])
def test_rows_are_written_through_where_that_is_faster(lib, d):
    def through(n, lines=1):
        return bool(lib.read_through(d, lines, C.c_longlong(n)))

    most = 140_000_000
    assert all(through(n) == (d != 32 or n <= most) for n in (1, 10 ** 6, 8 * 10 ** 7, most, most + 1, 10 ** 10))
    # 16 bytes into a line: only what the matrix cores bound, and not the shortest
    assert all(through(n, lines=0) == (d in (160, 224) and n > 10 ** 6) for n in (1, 10 ** 6, 10 ** 6 + 1, 10 ** 8, 10 ** 10))


@pytest.mark.parametrize("d,last", [(32, None), (64, None), (96, 0), (128, None), (160, 256), (192, None), (224, 1024), (256, 1024)])
def test_a_flush_sends_its_record_through_lds_where_that_is_faster(lib, d, last):
    staged = [bool(lib.flush_staged(d, C.c_longlong(t))) for t in (1, 56, 256, 257, 1024, 1025, 10 ** 6)]
    assert staged == [last is not None and t > last for t in (1, 56, 256, 257, 1024, 1025, 10 ** 6)]
