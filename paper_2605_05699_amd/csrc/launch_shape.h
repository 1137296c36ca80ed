// launch_shape.h -- how launches are laid out; plain C++ for the host, no HIP.
#ifndef SRFT_LAUNCH_SHAPE_H
#define SRFT_LAUNCH_SHAPE_H
#include <algorithm>
#include <cstdint>

#ifdef __HIPCC__
#define SRFT_HOST_DEVICE __host__ __device__
#else
#define SRFT_HOST_DEVICE
#endif

constexpr int kDies = 8;                     // accelerator dies; a launch's workgroups run die by die (srft_work_of_block)

// Workgroups first_block .. first_block + blocks - 1 walk the tiles tile .. tile + tiles - 1 of a segment, each with stride
// `blocks`.
struct srft_share {
    int segment, first_block, blocks;
    long long tile, tiles;
};

// Shares of a launch over segments of tiles[i] >= 1 tiles; returns how many were written to `out` (room for `most` >= count)
// and sets *grid.  Every segment gets at least one workgroup and at most one per tile; when the tiles of all segments exceed
// `budget`, workgroups are shared out in proportion to the tiles.
// Where a share's tiles do not divide evenly, its first workgroups walk one tile more than the others.  A segment that lies on
// several dies would give all of these tiles to the first of them (2 plans x 698 tiles on 1024 workgroups: 256 tiles on one
// die, 128 on another), so it is cut where the dies meet, and each part gets its part of the tiles.  Whole segments against
// cut ones, us: d = 128, 2 plans x 18,836 vectors, write 7.0 -> 5.8, read 6.5 -> 5.9; d = 256, 2 x 9415, write 7.2 -> 6.0; 2 x
// 18,017 10.4 -> 9.0.  Only where it pays: segments of two dies and more (5 to 7 plans even out by themselves, and lose 2 % when
// cut), up to 4 tiles per workgroup (from there on within 1 %).
inline int srft_share_out(const long long* tiles, int count, long long budget, srft_share* out, int most, int* grid) {
    long long total = 0;
    for (int i = 0; i < count; ++i) total += tiles[i];
    int next = 0;
    for (int i = 0; i < count; ++i) {
        const long long blocks = total <= budget ? tiles[i] : std::min(std::max(tiles[i] * budget / total, 1LL), tiles[i]);
        out[i] = {i, next, (int)blocks, 0, tiles[i]};
        next += (int)blocks;
    }
    *grid = next;
    if (total <= budget) return count;
    const int q = next / kDies, r = next % kDies;
    int last[kDies], cuts = 0;               // places up to the end of each die
    for (int die = 0, end = 0; die < kDies; ++die) last[die] = end += q + (die < r);
    const auto cut_at = [&](const srft_share& s, int place) {
        return place > s.first_block && place < s.first_block + s.blocks && s.blocks >= 2 * q && s.tiles > s.blocks && s.tiles < 4LL * s.blocks;
    };
    for (int i = 0, die = 0; i < count; ++i)
        for (; die < kDies && last[die] < out[i].first_block + out[i].blocks; ++die) cuts += cut_at(out[i], last[die]);
    if (cuts == 0 || count + cuts > most) return count;
    // from the last segment to the first: the parts are written behind the segments that are still to be read
    for (int i = count - 1, at = count + cuts, die = kDies - 1; i >= 0; --i) {
        const srft_share s = out[i];
        int end = s.first_block + s.blocks;
        const auto part = [&](int from) {
            const long long t0 = s.tiles * (from - s.first_block) / s.blocks, t1 = s.tiles * (end - s.first_block) / s.blocks;
            out[--at] = {i, from, end - from, t0, t1 - t0};
            end = from;
        };
        for (; die >= 0 && last[die] > s.first_block; --die)
            if (cut_at(s, last[die])) part(last[die]);
        part(s.first_block);
    }
    return count + cuts;
}

// A launch over segments of one length with `blocks` workgroups each: workgroup -> segment as one multiplication.  Exact while
// grid * blocks < 2^31: with magic = 2^31 / blocks + e, 0 <= e < 1, the product exceeds the true quotient by block * e / 2^31 <
// 1 / blocks.
constexpr uint32_t srft_even_magic(int blocks) { return (uint32_t)(((1ULL << 31) + blocks - 1) / blocks); }
SRFT_HOST_DEVICE constexpr int srft_even_segment(uint32_t block, uint32_t magic) { return (int)(((uint64_t)(2 * block) * magic) >> 32); }

// Workgroups per segment for `count` segments of `tiles` tiles each, as srft_share_out would share them out; 0: the segments
// go out cut where the dies meet (see there), or there are more than `budget` of them.
constexpr int srft_even_blocks(long long tiles, long long count, long long budget) {
    if (count > budget) return 0;
    const long long blocks = tiles * count <= budget ? tiles : std::min(std::max(budget / count, 1LL), tiles);
    if (blocks * count * blocks >= (1LL << 31)) return 0;
    return count <= kDies / 2 && tiles > blocks && tiles < 4 * blocks ? 0 : (int)blocks;
}

// Workgroups that `blocks` for every one of `count` segments leaves over are spread evenly over the segments, so that all of the
// budget is at work: workgroup b serves segment (b S + S - 1) / W, whose workgroups start at i W / S, with W workgroups on S
// = count segments (where nothing is left over, or the products get too large to divide exactly, W = blocks on S = 1).  52 x
// 4096 vectors at d = 256, read (512 workgroups for 52 plans: 9 each and 44 over) 36.3 -> 35.5 us, 8-bit 37.6 -> 36.9, 52 x
// 40,000 306 -> 301; d = 128, 80 x 3000 20.3 -> 20.0; 56 x 10,000 at d = 96 33.3 -> 33.1.  Writes are bound by memory
// whichever way: d = 128, 80 x 3000 16.6 -> 16.75; they keep `blocks` each.
struct srft_even_shape {
    int w, s;
    uint32_t w_magic, s_magic;
};
constexpr srft_even_shape srft_even_spread(long long tiles, long long count, long long budget, int blocks) {
    const long long w = tiles * count < budget ? tiles * count : budget;
    if (w == blocks * count || w * w * count >= (1LL << 31)) return {blocks, 1, srft_even_magic(blocks), srft_even_magic(1)};
    return {(int)w, (int)count, srft_even_magic((int)w), srft_even_magic((int)count)};
}
constexpr int srft_even_grid(const srft_even_shape& e, long long count) { return (int)(e.s == 1 ? e.w * count : e.w); }
SRFT_HOST_DEVICE constexpr int srft_even_segment(int block, const srft_even_shape& e) {
    return srft_even_segment((uint32_t)(block * e.s + e.s - 1), e.w_magic);
}
SRFT_HOST_DEVICE constexpr int srft_even_start(int segment, const srft_even_shape& e) {
    return srft_even_segment((uint32_t)(segment * e.w), e.s_magic);
}

// A flush of n_vec rows in pages of page_rows = n_seq * R rows, out of new tokens [n_seq][t][units]: its kernel counts rows and
// 16-byte units with 32 bits, and divides by page_rows and R as above.
constexpr bool srft_flush_fits(long long n_vec, long long page_rows, long long n_seq, long long t, long long units) {
    constexpr long long most = 1LL << 31;
    return n_vec < most / page_rows && (n_vec + page_rows) * units < most && n_seq * t < most / units;
}

// Up to this many tiles per workgroup that fits the chip, a flush is one launch with both paths in it (cache_flush.h has the
// figures): d = 256 and 32 lose from 4 on, d = 128 with g = 16 from 1 on, the others between 8 and 12 or (d = 96) not at all.
// (d = 256, g = 16, 52 plans: two launches -> one, a page of 8 sequences and a step 12.3 -> 11.1 us.)
constexpr int srft_flush_whole_tiles(int d, int g) { return d == 128 && g == 16 ? 1 : d == 256 || d == 32 ? 4 : 8; }

// Whether a record of the write path's plain form goes through LDS and is written through to memory (device_util.h), or is stored from
// the lanes, in pieces of 8 bytes that the L2 puts together; by the tiles of a launch, its workgroups and the compute units.  Time
// through LDS over time from the lanes, over one / three / six sets of buffers in turn (the memory-side cache holds 256 MB).  From some
// 60 MB on where the buffers lie moves the ratio by up to 10 %, from one card and run to the next: two figures for a set are two cards.
//   Up to three tiles a compute unit the way through LDS is only longer: d = 96, 240 vectors 2.33 -> 2.40 us, 17,027 3.15 -> 3.26;
//     64 x 512 (1024 tiles) 4.56 -> 4.48.  d = 192 up to four and a half (15 MB 1.03 / 1.02 / 1.02, 8 plans 1.05 / 1.04 / 1.03; 20 MB
//     0.97 / 0.98 / 0.97), d = 224 three and a half (15 MB 1.02 / 1.03 / 1.02; 20 MB 0.97 / 0.98 / 0.97).
//   Up to some tiles a workgroup nothing is left to write back; from there on the memory-side cache takes the record better from the
//     L2, where the rows are short.
//   d = 64   10 MB 0.96 / 0.94 / 0.94   30 MB 0.91 / 0.93 / 0.92   50 MB 0.95 / 0.92 / 0.77   85 MB 1.00 1.00 / 0.99 0.95 / 1.02 0.98
//     105 MB 0.99 1.00 / 0.85 0.96 / 1.07 0.99   118 MB 0.99 1.01 / 1.16 0.92 / 1.13 1.00   8 bits: 55 MB 0.75 / 0.99 / 0.83,
//     110 MB 1.00 / 0.85 / 1.05   56 plans: 15 MB 0.94 / 0.94 / 0.95, 90 MB 0.99 / 0.91 / 0.99
//   d = 96   10 MB 0.90 / 0.90 / 0.93   40 MB 0.91 / 0.96 / 0.98   60 MB 0.96 0.93 / 1.00 0.92 / 0.93 0.94   90 MB 1.05 0.97 /
//     0.98 0.91 / 1.05 1.04   130 MB 1.05 / 1.08 / 1.12   180 MB 1.02 / 1.06 / 1.00   260 MB 0.97 / 0.95 / 0.96   8 bits: 90 MB
//     1.11 0.93 / 1.03 0.83 / 1.05 1.05, 150 MB 1.04 / 1.05 / 1.08, 300 MB 0.86 / 0.97 / 0.93   56 plans: 90 MB 1.04 0.91 / 0.93 0.80 /
//     0.93 0.91
//   d = 128 (plain at g = 16 and with Walsh-Hadamard)   g = 16: 10 MB 0.88 / 0.90 / 0.91, 60 MB 0.95 / 1.01 / 0.91, 200 MB 1.03 / 0.99 /
//     1.00, 400 MB 0.97 / 0.97 / 0.98; 8 bits 40 MB 0.82 / 0.90 / 0.90, 160 MB 1.12 / 1.02 / 0.99, 300 MB 0.77 / 0.85 / 0.88: always.
//     4 bits, g = 32: 90 MB 0.99 / 0.93 / 0.99, 115 MB 1.04 / 0.90 / 0.98, 160 MB 1.03 / 1.07 / 1.04, 200 MB 1.04 / 1.04 / 1.09, 400 MB
//     1.06 / 1.05 / 1.06
//   d >= 160 is at the matrix cores' rate beyond 16 tiles a workgroup, and no way is the faster one there; before, 30 MB d = 160 0.88 /
//     0.87 / 0.87, d = 192 0.96, d = 224 0.96 / 0.98 / 0.98, d = 256 0.96
//   d = 32, with a vector in an eighth of a line, gains on single plans and loses on several: 400,000 vectors 7.0 -> 6.65 us, 7 plans x
//     51,556 6.8 -> 7.9, 36 x 1494 2.75 -> 3.1, 1,000,000 13.9 -> 14.4: never
// lines: all records of the launch start at multiples of 64 bytes.  16 bytes into a line: d = 64 11 MB 1.11 / 1.04 / 1.02, 33 MB 0.93 /
// 0.94 / 0.94; d = 96 11 MB 1.03 / 1.03 / 1.02, 33 MB 0.94 / 0.95 / 0.95, 300 MB 0.93 / 1.01 / 1.01; d = 128, g = 16 11 MB 1.01 / 1.02 /
// 1.07, 300 MB 0.90 / 1.01 / 1.03; d = 160 11 MB 0.88; d = 192 15 MB 1.03 / 1.02 / 1.02, 33 MB 0.97 / 0.97 / 0.98.  14 ragged plans, whose
// records start anywhere, over three sets: d = 64 5 MB 1.07, 8 MB 1.04, 14 MB 0.98; d = 96 7 MB 1.12, g = 16 9 MB 1.08, 11 MB 0.89, 14 MB
// 0.87; d = 192 22 MB 1.04.
constexpr bool srft_write_staged(int d, int g, int bits, bool lines, long long tiles, long long workgroups, long long compute_units) {
    if (d == 32 || 2 * tiles <= (d == 192 ? 9 : d == 224 ? 7 : 6) * compute_units) return false;
    if (!lines && (d == 128 || tiles <= (d == 64 ? 8 : d == 96 ? 5 : d == 160 ? 0 : 6) * compute_units)) return false;
    if (d == 128 && (g != 32 || bits == 8)) return true;
    if (d == 96 && tiles >= 22 * workgroups) return true;
    return tiles <= (d == 64 ? 9 : d == 96 ? 11 : d == 128 ? 14 : 16) * workgroups;
}

// Whether the read path writes its rows through to memory or leaves them to the L2 (device_util.h), by the bytes of a launch, in and
// out.  Left to the L2 -> written through, over one / three / six sets of buffers in turn (the memory-side cache holds 256 MB):
//   d = 32   20 MB 0.99 / 0.95 / 0.94   40 MB 0.97 / 0.84 / 1.03   60 MB 0.90 / 0.98 / 1.04   90 MB 0.83 / 1.04 / 1.00   130 MB
//     0.83 / 1.02 / 1.01   160 MB 1.01 / 1.02 / 1.02   300 MB 1.04 / 1.04 / 1.04 (there it is the form of the store that costs:
//     1.05 without sc1)
//   d = 64   45 MB 0.91 / 0.89 / 0.90   90 MB 0.89 / 1.02 / 0.99   130 MB 0.90 / 0.99 / 0.99   300 MB 0.98; 56 plans 40 MB 0.88 /
//     0.85 / 0.84, 80 MB 0.76 / 0.95 / 0.93
//   d = 96    60 MB 0.87 / 0.93 / 0.98   88 MB 0.87 / 0.99 / 0.97   160 MB 0.95 / 0.98 / 0.97
//   d = 128   40 MB 0.90 / 0.89 / 0.96   80 MB 0.80 / 1.04 / 0.99   90 MB 0.82 / 1.05 / 1.00   110 MB 0.73 / 1.01 / 1.00   300 MB
//     0.99; 56 plans 40 MB 0.84 / 0.83 / 0.83, 80 MB 0.80 / 0.95 / 0.95; 14 ragged ones 84 MB 0.82 / 0.97 / 0.98; 8 bits 85 MB 0.91
//     / 0.98 / 0.97
//   d = 256   60 MB 0.91 / 0.93 / 0.96   90 MB 0.88 / 1.02 / 1.00   160 MB 0.98 / 0.99 / 0.98; d = 160, 192 and 224 0.93 - 0.99 at
//     all sizes
// (One plan of 64 to 128 channels, its sets just filling the memory-side cache, is 2 to 5 % slower at 75 to 100 MB; with fewer sets the
// same launches are 20 % faster, with more the same, several plans 5 % faster, so they have no way of their own.  sc1 without
// nt is faster there and slower cold: d = 64 1.10 - 1.16, d = 96 1.06 - 1.09, d = 128 1.02.)
// lines: all rows of the launch start at multiples of 64 bytes (half a line does: 64 bytes into a line 0.88 as at its start).  16
// bytes into a line every piece that a wavefront stores ends in a partial line: d = 32 11 MB 1.04, 33 MB 1.14, 300 MB 1.18; d = 64
// and 96 the same; d = 128 11 MB 1.01, 33 MB 1.11, 300 MB 1.20; d = 192 33 MB 1.04, 300 MB 1.02; d = 256 33 MB 1.01, 88 MB 1.04,
// 300 MB 1.05.  d = 160 and 224, which the matrix cores bound, gain still (3000 vectors 0.97, 11 MB 0.92, 33 MB 0.96, 88 MB 0.98)
// but for the shortest launches (300 vectors 1.06 and 1.12).
constexpr bool srft_read_through(int d, bool lines, long long bytes) {
    if (!lines) return (d == 160 || d == 224) && bytes > 1000000;
    return d != 32 || bytes <= 140000000;
}

// Whether the once-folded write path (d = 128; d = 256 with g = 64 and 128) writes its record through to memory or leaves it to the
// L2 (device_util.h), by the bytes of a launch, in and out.  Written through, nothing is left to write back at the end, which is what a
// short launch takes longest over; a long one loses a little by it.  Left to the L2 -> written through, in turn over one / three / six
// sets of buffers (the memory-side cache holds 256 MB):
//   d = 128   11 MB 0.91 / 0.94 / 0.96   30 MB 0.95 / 0.96 / 0.96   50 MB 0.95 / 0.98 / 0.97   60 MB 0.98 / 1.00 / 0.98   80 MB 0.98 /
//     1.02 / 1.01   154 MB 1.00 / 1.01 / 1.02   300 MB 0.99 / 1.03 / 1.02   1 GB 1.01; 56 x 8192 (154 MB) 39.7 -> 40.5 us
//   d = 256   20 MB 0.98 / 0.98 / 0.98   100 MB 0.99 / 0.99 / 1.00   160 MB 0.97 / 0.98 / 0.98   250 MB 1.02 / 1.00 / 1.02   350 MB
//     1.02 / 1.01 / 1.02
// lines: the record starts at a multiple of 64 bytes.  Where it does not, 8-bit rows at d = 128 reach memory as partial lines (16 bytes
// into a line, 33 MB 1.04, 88 MB 1.05, 300 MB 1.05); 4-bit rows and d = 256 do not mind (d = 128, 33 MB 0.96; d = 256, 8 bits, 20
// MB 0.97).
constexpr bool srft_fold_through(int d, int bits, bool lines, long long bytes) {
    return (lines || bits == 4 || d == 256) && bytes <= (d == 128 ? 60000000 : 200000000);
}

// Whether the record of a flush's write half, where that is a launch of its own, goes through LDS (plain form; srft_write_staged), by
// head dimension and the tiles of all plans.  The rows are gathered here, and what follows is the read path's launch, so the line lies
// elsewhere than for a write alone.  us of one append, record from the lanes -> through LDS:
//   d = 64    56 plans 8 x 1000 tokens 30.4 -> 33.0
//   d = 96    56 plans 8 x 1000 55.7 -> 50.4 (shorter ones are one launch)
//   d = 128   (g = 16) 80 plans 2 x 320 16.3 -> 18.4, 56 plans 2 x 1000 25.3 -> 28.1, 8 x 1000 75.9 -> 80.4
//   d = 160   2 plans 1 x 16 7.5 -> 8.1, 56 plans 2 x 16 8.05 -> 8.8, 8 x 16 8.7 -> 9.1, 2 x 100 12.3 -> 11.1, 80 plans 2 x 320 24.2 -> 22.4
//   d = 192   2 plans 1 x 16 7.7 -> 8.4, 56 plans 2 x 16 8.9 -> 9.2, 2 x 100 11.75 -> 12.4, 2 x 1000 38.9 -> 40.2, 8 x 1000 129.8 -> 130.2
//   d = 224   2 plans 1 x 16 9.2 -> 9.9, 56 plans 2 x 100 14.5 -> 14.9, 80 plans 2 x 320 30.5 -> 29.7, 56 plans 2 x 1000 55.5 -> 55.0
//   d = 256   (Walsh-Hadamard) 2 plans 1 x 16 10.4 -> 10.7, 56 plans 2 x 100 16.7 -> 17.1, 80 plans 2 x 320 35.5 -> 34.9
constexpr bool srft_flush_staged(int d, long long tiles) {
    return d == 96 || (d == 160 && tiles > 256) || ((d == 224 || d == 256) && tiles > 1024);
}

// True when count addresses lie a constant step apart; *step is that step in bytes (0 for one).
inline bool srft_even_step(const void* const* p, int count, long long* step) {
    *step = count > 1 ? (long long)((uintptr_t)p[1] - (uintptr_t)p[0]) : 0;
    for (int i = 2; i < count; ++i)
        if ((uintptr_t)p[i] - (uintptr_t)p[i - 1] != (uintptr_t)*step) return false;
    return true;
}

// The cache's copy of t new tokens: launch i of srft_copy_launches(t) copies srft_copy_tokens(i, t) tokens from
// srft_copy_first(i) on.  A launch counts its 16-byte units with 32 bits; t may be anything an int holds.
constexpr long long kCopyTokens = 1 << 24;
constexpr int srft_copy_launches(int t) { return (int)((t + kCopyTokens - 1) / kCopyTokens); }
constexpr long long srft_copy_first(int i) { return i * kCopyTokens; }
constexpr unsigned srft_copy_tokens(int i, int t) { return (unsigned)std::min(kCopyTokens, t - srft_copy_first(i)); }

#endif  // SRFT_LAUNCH_SHAPE_H
