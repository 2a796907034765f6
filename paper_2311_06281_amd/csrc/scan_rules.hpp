// Rules of a launch that follow from sizes and types alone (plain C++, which the tests compile by itself).
#pragma once
#include <stdint.h>

namespace hs {

// A launch of rows of several tiles starts its first tiles one after the other: each waits its ticket times this many
// nanoseconds after it has drawn the ticket.  (The draws queue as well: in one row of 2^26 steps the 512th tile starts 8.5 us
// after the first without the wait and 13.2 us with 12 ns, that is 26 ns a tile, at which their loads are 5.1 TB/s.
// The spacing is the one measured best.)  Started all at once they shared the memory evenly, had their inputs at about
// the same time, waited for one another at the same time and wrote at the same time, and so did the tiles behind them:
// at some times 39 of 512 tiles were loading, at others 488.  One after the other, a tile is waiting or writing while the
// next ones load, from the first to the last.  Measured (none, 6, 9, 12, 15 ns): one row of 2^26 float32 154.1, 152.4,
// 150.3, 149.0, 149.3 us; 700 rows of 40000 69.4, 68.1, 66.7, 66.4, 67.3; bf16, whose tiles are half the bytes, one row of
// 4 * 10^7 81.4, 79.9, 79.5, 79.8, 81.3, 4 rows of 4 * 10^6 37.5, 36.6, 36.8, 39.0, 41.6.
// That pays from the third round of tiles on.  A launch that fits the chip has nothing behind its first tiles (one row of
// 2^23 steps, 512 tiles, 26.5 and with 12 ns 30.0 us), and with less than a second round behind them it comes out even or loses
// (119 rows of 123464, 960 tiles, 42.5 and 43.6, bf16 33.5 and 36.7; 40 x 322896 without logarithms, bf16, 27.3 and 30.0),
// but for float32 in rows so long that nearly all tiles in flight wait for one another, from a few tiles more than a round up to
// 1.6 rounds (one row of 9 * 10^6 35.6 and 33.4, of 1.25 * 10^7 41.5 and 38.8, 9 rows of 1.31 * 10^6 0.96 of the time; without
// logarithms one row 0.95 to 0.99 of the time, several 0.97 to 1.03; one row of 8.40 * 10^6, 513 tiles, 1.03 to 1.08, one of
// 1.5 * 10^7, 1.8 rounds, 0.97 to 1.04).  Of rows of two tiles only every other tile waits, and for one (3000 rows of
// 17000 137.2, 12 ns 138.0).
//
// That is for the tiles of which the chip holds kPacedTiles at a time, two workgroups per compute unit: real output moved
// as vectors (104 to 125 registers).  Element by element (149 to 161 registers) and with complex output (176 to 209) a
// workgroup has its compute unit to itself; tickets 256 and up are then drawn in the middle of the launch, where a wait only
// leaves the unit empty.  Without and with it: 200 rows of 40000 whose pointers are not alike 35.2 and 41.3 us, bf16 104.5
// and 108.9, one row of 1.25 * 10^7 such steps 43.3 and 47.9; complex output, 200 x 40000, 46.2 and 50.5.
constexpr uint32_t kPaceNs = 12, kPaceNsBf16 = 8;
constexpr uint32_t kPacedTiles = 512;
constexpr uint32_t kPacedTilesPerRow = 3, kPacedTilesPerLongRow = 64;

// Whether the tiles kernel for such data may be paced, and the spacing for a launch (0: none).
constexpr bool paced_kernel(bool vectors, bool complex_out) { return vectors && !complex_out; }
constexpr uint32_t pace_ns(bool vectors, bool complex_out, bool bf16, uint32_t tiles_per_row, uint32_t tiles)
{
    const bool many = tiles_per_row >= kPacedTilesPerRow && tiles > 2 * kPacedTiles;
    const bool long_rows = !bf16 && tiles_per_row >= kPacedTilesPerLongRow && tiles >= kPacedTiles + 8 && tiles <= kPacedTiles * 8 / 5;
    if (!paced_kernel(vectors, complex_out) || !(many || long_rows)) return 0;
    return bf16 ? kPaceNsBf16 : kPaceNs;
}

// [B, n, D].  Ticket queues: as many (up to one per compute die) as leave every queue this many columns.  The tiles
// of a column start that many tickets apart, so a tile usually finds the tiles before it done; eight queues
// also keep neighbouring columns on one die, which then reads the lines they share once (6 x 3001 x 770, 73
// columns: 50.5 us with 16 per queue, 48 with 8).  The wide tiles, whose rows are requested by two waves at a time, want
// the queues longer still.  (A queue per die where items lie a power of two apart gains and loses: 128 x 1024 x 512 168 and
// 140 us, 16 x 4096 x 2048 283 and 268, but 64 x 4096 x 512 276 and 311, 64 x 4096 x 1024 627 and 705, 511 x 1024 x 128 147
// and 172.)
constexpr int kMinColsPerQueue = 8, kMinColsPerQueueWide = 128;
constexpr int ticket_queues(int most, int64_t columns, bool wide)
{
    int queues = most;
    while (queues > 1 && columns < queues * (wide ? kMinColsPerQueueWide : kMinColsPerQueue)) queues /= 2;
    return queues;
}

// [B, n, D], few columns: tiles of sixteen waves (512 steps, one workgroup per compute unit) in two carry levels of
// sixteen, instead of eight waves and levels of eight or four.  Half as many tiles lie behind one another in a column and
// 256 of them have their states handed on without a chain, which is what the smaller ones wait for; but a compute unit has
// nothing to load while its one workgroup waits.  So from half a round of the chip (below, a tile's own latency counts: 1 x
// 16384 x 64 12.6 us with eight waves, 16.5 with sixteen) to three (eight and sixteen: one column of 131072 steps 35.8 and
// 24.7, of 262144 57.7 and 47.2, 4 x 65536 51.9 and 45.6, 8 x 32768 51.4 and 44.7, 3 x 131072 70.9 and 67.6; four rounds, 4
// x 131072, 90.0 and 91.2).  Runs in six to eight columns of few tiles, which are short enough not to wait for a chain of states,
// want more of a round (eight columns of 17 18.2 and 19.6, float32 19.6 and 20.4, of 20 20.1 and 21.1, six of 23 18.6 and 19.4; six of 28 20.8
// and 19.8, eight of 26 21.9 and 20.7; bf16 logarithms but for the one).  From 16 columns on a round counts the tiles as the queues deal them: 19 columns of 26 are 494,
// but one of the two queues has 260 for the 256 places of two turns (302 x 12838 x 3 41.9 and 52.0; 50 columns of five, 13
// in a queue, 23.0 and 28.1). One round: up to 32 columns always (16 x 8192 x 64 28.1 and 20.4, 32 x 4096 22.1 and 20.9),
// more as soon as a column is long enough for its carries to cost something (36 columns of seven 20.3 and 18.5, 42 of four
// 16.7 and 15.9, 48 of three 13.7 and 17.5; where lines are cut 34 of seven 23.5 and 21.0, 37 of four 18.1 and 19.4, bf16
// 37 of five 16.2 and 16.9; runs 39 of five 20.9 and 19.7, 41 of four 15.7 and 17.5, bf16 37 of five 18.0 and 18.9).  Two
// rounds: up to 24 columns (24 x 8192 x 64 36.4 and 36.1), and more only where the memory is not what they wait for.
// Columns that cut lines, from one and a half rounds on: 6 x 3001 x 770 47.8 and 43.5, 4 x 7691 x 508 50.8 and 43.8, bf16 2
// x 3840 x 1945 40.1 and 34.7 (78 of four 27.2 and 29.5, bf16 72 of six 30.5 and 31.7).  Runs of up to 32 columns, bf16 16,
// if they nearly fill both: 512 x 8192 x 4 47.6 and 42.9, 128 x 8192 x 16 46.0 and 41.9, bf16 256 x 15835 x 3 44.4 and 38.5
// (24 of 20, 384 x 10203 x 3, 44.9 and 46.6, bf16 192 x 10203 x 5 35.0 and 37.3; more columns gain less and lose: 432 x
// 4608 x 8 45.3 and 42.5, 45 of nine 36.2 and 36.4, 60 of seven 37.5 and 39.4, bf16 949 x 3888 x 4 30.0 and 31.9; 64 of
// eight, 256 x 4096 x 16, 45.3 and 41.0, keep the tile that is promised for them).  Whole lines lose: 32 x 8192 x 64 43.1
// and 45.8, 6 x 3072 x 768 35.9 and 38.8.  Tiles of eight waves that have a compute unit each do not wait (28 columns of
// 2189 steps, 252 of them, 16.9 and 22.7).  Items of two channels, whose runs are the shortest pieces, gain in one round
// that is mostly full (510 x 7936 x 2 28.9 and 21.9; 544 x 4706 22.3 and 23.0, in two rounds 512 x 13158 49.0 and 51.7).
constexpr bool tall_tiles(int64_t columns, int64_t chunks_of_256, int64_t channels, bool runs, bool bf16, int most_queues)
{
    const int64_t chunks = (chunks_of_256 + 1) / 2, tiles = columns * chunks, places = 256;
    if (columns < 16) return tiles > places / 2 && tiles <= 3 * places && !(runs && columns <= 8 && chunks < 24);
    if (columns * chunks_of_256 <= places) return false;
    const int64_t queues = ticket_queues(most_queues, columns, false), dealt = (columns + queues - 1) / queues * queues * chunks;
    const bool cut_lines = !runs && channels % 32 != 0;
    if (channels == 2) return dealt <= places && 10 * tiles > 7 * places;
    if (dealt <= places) return columns <= 32 || (runs || cut_lines ? !bf16 && chunks >= 5 : chunks >= 4);
    if (dealt > 2 * places) return false;
    if (runs) return columns <= (bf16 ? 16 : 32) && 8 * tiles > 15 * places;
    return columns <= 24 || (cut_lines && chunks >= (bf16 ? 7 : 6) && 2 * tiles > 3 * places);
}

// [B, n, D], output in whole lines.  It goes through the L2 at once unless the tiles wait for states that would queue with
// it: tiles of eight waves with one carry level, between one and three per compute unit, where most of the output is
// written while nothing is left to load.  Ordinary stores and through the L2 there: 15 x 1993 x 256 (480 tiles) 20.2 and
// 22.6 us, 32 x 879 x 256 (512) 19.8 and 21.7, 43 x 1013 x 256 (688) 30.1 and 31.2 (long chains differ: 2 x 5593 x 512, 352
// tiles, 22.5 and 21.2); below and above, 2 x 4075 x 512 (256) 15.6 and 14.2, 50 x 3972 x 64 (800) 35.5 and 34.8.
// Sequences of one tile wait for nothing: in this range of tiles 37 x 109 x 512 10.3 and 8.9, 31 x 57 x 1024 7.1 and 5.7,
// 150 x 32 x 256 5.25 and 4.76, 360 x 160 x 64 11.2 and 11.1, 18 x 227 x 1024 14.2 and 14.6.  (Over 700 sizes of up to 256
// steps through the L2 takes 0.90 to 0.98 of the time in the mean, and 1.00, between 0.90 and 1.07, for 17 to 30 MB of
// float32 output.)  Complex output, of whose tiles a compute unit holds one, is faster so as well: 8 x 1956 x 512 33.2 and
// 30.5, 130 x 1013 x 64 39.7 and 36.3.  Narrow items as runs: see runs_in_lines.
// With two carry levels states come from farther back and seldom queue: 1 x 10625 x 384 (252 tiles) 17.0 and 15.8, 1 x 8677 x
// 704 (374) 22.2 and 21.3, bf16 1 x 8160 x 832 (416) 20.0 and 18.4, without logarithms up to seven columns 1 x 25584 x 192 (300)
// 19.6 and 18.5.  From eight columns on tiles without logarithms, which take the least time over their steps, do lose up
// to one round of the chip (2 x 9437 x 256, 296 tiles, 19.3 and 20.6, 2 x 12276 x 320, 480, 23.8 and 25.1; 1 x 11391 x 768, 540
// tiles, 31.9 and 31.5).
constexpr bool waits_behind_stores(int waves, int64_t columns, int64_t chunks, bool two_levels, bool linear, bool runs)
{
    const int64_t tiles = columns * chunks;
    if (waves != 8 || chunks == 1 || runs || tiles <= 256) return false;
    return two_levels ? linear && columns >= 8 && tiles <= 512 : tiles <= 768;
}

// Narrow items as runs: 32 steps are whole lines where items begin on lines, and then go through the L2 at once (0.90 to 0.97
// of the time with ordinary stores).  Where not, the lines at their ends are parts; that pays as long as inputs and output are
// small: over 190 such sizes 0.92 to 0.98 of the time in the mean up to 96 MB, 1.01 up to 128, 1.04 up to 200 (ordinary stores and
// through the L2: 250 x 994 x 17, 49 MB, 15.8 and 14.9 us; 300 x 3000 x 7, 76 MB, 23.0 and 21.3; 1525 x 253 x 25, 116 MB, 30.0 and
// 31.4; 544 x 1294 x 19, 161 MB, 36.9 and 38.4; the other way 1360 x 1012 x 5, 83 MB, 20.9 and 25.1).
constexpr bool runs_in_lines(bool out_on_line, int64_t items, int64_t item_elements, int64_t bytes)
{
    return (out_on_line && (items == 1 || item_elements % 32 == 0)) || bytes <= ((int64_t)96 << 20);
}

} // namespace hs
