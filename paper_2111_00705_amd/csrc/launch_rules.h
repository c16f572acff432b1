// Rules that choose a launch shape from sizes alone: host code without HIP, so that a test can compile them by themselves.
#pragma once
#include <stdint.h>

namespace cams {

// Whether the update of kept values takes a quarter of a tile per workgroup (tk_final_short) instead of a tile (tk_final).
// The quarter form fills the chip and loads the state first.  Up to 320 tiles its 1280 workgroups run at once; it pays up to 448 tiles
// with no more than eight workers, four under naive compression.  Step plus get_theta, the same handles in turn, us, a tile / a
// quarter: error feedback, k = 1 %, n = 8, 367 tiles 73.5 / 69.3, 440 tiles 78.4 / 74.9 (k = 5 % 85.7 / 80.9, Rand-k f16
// 75.5 / 71.4), n = 4, k = 0.1 % 62.5 / 59.0; naive bf16, 440 tiles, n = 1 47.9 / 47.1, n = 2 47.3 / 46.6, n = 4 50.3 / 49.9, but n = 6
// 53.0 / 53.5, n = 8 55.0 / 55.6, 367 tiles 52.7 / 52.9, fp32 57.0 / 57.3; error feedback, 318 tiles, n = 12 80.7 / 75.9, n = 16
// 91.6 / 87.9, n = 24 110.2 / 108.7, n = 32 131.6 / 130.6, n = 48 177.3 / 177.2, naive bf16 n = 32 73.0 / 71.9, n = 48 87.7 / 87.0;
// 196 tiles, n = 24 85.6 / 82.3, n = 32 99.9 / 96.5, n = 48 130.9 / 127.0; 98 tiles, n = 32 73.0 / 69.4, n = 48 92.7 / 88.3.  Beyond, by
// earlier figures: n = 8, 2.1 M, k = 0.1 % 82.4 / 83.5, 2.5 M 96.1 / 96.9; n = 12, 1.8 M 89.2 / 89.7; n = 16, 2.5 M 130.8 / 134.7; Rand-k
// n = 256, 5 tiles 133.4 / 150.2, n = 1000, 5 tiles 446.6 / 514.0.
constexpr int kShortFinalTiles = 320, kShortFinalWorkers = 48;
constexpr int kQuarterTiles = 448, kQuarterWorkers = 8, kQuarterWorkersNaive = 4;
inline bool quarter_final(int64_t n, int64_t n_tiles, bool naive)
{
    if (n <= (naive ? kQuarterWorkersNaive : kQuarterWorkers)) return n_tiles <= kQuarterTiles;
    return n <= kShortFinalWorkers && n_tiles <= kShortFinalTiles;
}

// Workers whose kept values a workgroup of tk_final_short holds at a time.  Eight take 36 KB of LDS, which leaves four
// workgroups on a compute unit, enough for 256 tiles; five take 23 KB.  Step plus get_theta, us, five / eight: n = 48,
// d = 250 000 81.8 / 79.6, n = 32, d = 350 000 bf16 80.7 / 79.2; 293 tiles, n = 16 88.7 / 93.5, 318 tiles, n = 2 46.5 / 48.8.
inline int short_final_batch(int64_t n_tiles) { return n_tiles <= 256 ? 8 : 5; }

// Whether a step with short blocks of at most 256 coordinates is one launch (bs_step_short), with rows = those of a quarter of a tile
// that hold coordinates.  A workgroup goes through all workers of its quarter: beyond 80 (worker, row) pairs the two launches, which
// spread the workers over the chip, are as fast or faster, and beyond 64 tiles the chip is full without that.  Step plus
// get_theta, us, two launches / one: CD-Adam n = 20, d = 300 25.3 / 21.2; n = 48, d = 300 27.4 / 21.1, n = 96 33.7 / 24.8; n = 4,
// d = 4000 21.9 / 20.1, n = 32 (CD-Adam) 26.6 / 26.8, n = 64 30.0 / 34.6; d = 65 536, n = 1 22.6 / 20.1, n = 8 23.9 / 22.2, n = 16
// 25.0 / 24.6, n = 32 29.5 / 29.5; d = 250 000, n = 16 32.3 / 29.3, CD-Adam 33.1 / 31.2; d = 500 000, n = 4 27.8 / 26.3, CD-Adam
// 30.1 / 31.3; d = 1 M, n = 2 31.3 / 32.0, CD-Adam 33.0 / 39.8.
constexpr int kOneLaunchPairs = 80, kOneLaunchTiles = 64;
inline bool one_launch_sign(int64_t n, int64_t d, int64_t n_tiles)
{
    const int64_t rows = d > 3072 ? 4 : (d + 1023) / 1024;
    return n_tiles <= kOneLaunchTiles && n * rows <= kOneLaunchPairs;
}

// Entries that a vector lists in steady state where one workgroup selects from them: 1.2 k for magnitudes; for scores those above the
// guess, kOneSelectSlack fine bins (of 2^17) or min_slack below the k-th largest.
constexpr uint32_t kOneSelectSlack = 16;
inline int64_t one_select_entries(int64_t d, int64_t k, uint32_t min_slack, bool scores)
{
    const int64_t slack = min_slack > kOneSelectSlack ? min_slack : kOneSelectSlack;
    return scores ? k + ((slack * d) >> 17) : k * 5 / 4;
}

// Whether one workgroup per vector selects from lists that lie in several regions (tk_small_select) instead of the three selection
// launches; entries: what is expected to be listed.  It holds kHeldEntries, and a quarter is left for uneven regions.  After a miss
// that workgroup lists the vector again by itself (d = 500 000: 340 us where many workgroups take tens), so magnitudes, whose
// threshold may fall, stop at 64 tiles, and at 128 under CD-Adam, which selects twice and gains twice as much by it (see guess_holds
// for runs that miss often).  Scores do not fall, and stop where a fine bin, which holds d / 2^17 of them, gets near the few that are
// ranked as they are.  Fewer than 16 entries were not measured with magnitudes and stay.  Step plus get_theta, us, three launches /
// one: error feedback n = 8, d = 100 000
// 38.6 / 34.7, d = 300 000, k = 0.1 % 42.8 / 38.9, k = 1 % 44.2 / 39.9, Rand-k 44.8 / 41.9; naive n = 8, d = 3 M bf16, k = 0.3 %
// (Rand-k) 69.5 / 66.3; CD-Adam n = 8, d = 300 000 67.5 / 56.0, d = 500 000 bf16 69.8 / 59.5, n = 2, d = 200 000 62.6 / 50.2, Rand-k
// d = 400 000 71.3 / 63.7.  Rand-k by length: n = 16, d = 1.2 M f16 78.3 / 74.2, n = 8, d = 4 M 117.8 / 114.5, d = 11 M bf16
// 245.3 / 243.0, naive bf16 11 M 155.8 / 154.0, 16 M 204.5 / 203.6, 24 M 284.2 / 283.8, 32 M 380.5 / 386.5, 60 M 668.9 / 676.7, n = 1,
// 40 M fp32 298.2 / 310.3, CD-Adam 11 M 269.5 / 268.3, n = 4, 20 M 330.6 / 331.4.
constexpr int kHeldEntries = 24 * 1024, kOneSelectTiles = 64, kOneSelectScoreTiles = 4096, kOneSelectMin = 16;
inline bool one_launch_select(int64_t entries, int64_t n_tiles, int slices, bool cd, bool scores)
{
    return (slices == 32 || slices == 64) && entries >= kOneSelectMin && entries <= kHeldEntries * 3 / 4 &&
           n_tiles <= (scores ? kOneSelectScoreTiles : (cd ? 2 : 1) * kOneSelectTiles);
}

// Steps after the selection records were reset, or the rows under a guess replaced, whose guesses are not relied on (magnitudes).  The
// first has none.  CD-Adam's second guess misses where gradients are correlated from step to step, its third where they are not, when
// the Markov sequences hold what was kept (n = 8, d = 300 000 101 us with three launches, 278 with one), and here and there its
// fourth.  Error feedback and naive compression missed in 2 of 150 second to fourth steps of a worker.
inline uint64_t settled_steps(bool cd) { return cd ? 4 : 1; }

// Steps that take three selection launches after one workgroup had to list a vector again; last: how many it was the time before,
// since: steps from the end of those until the miss was seen.  One launch saves 4 to 17 us a step and a miss in it costs some 50 to 340,
// so a miss in hundreds of steps is followed by a few, and where every guess misses there is one such step in 256.
constexpr uint64_t kThreeFirst = 16, kThreeMost = 256;
inline uint64_t three_launch_steps(uint64_t last, uint64_t since)
{
    if (since >= kThreeMost || last == 0) return kThreeFirst;
    return 2 * last < kThreeMost ? 2 * last : kThreeMost;
}

// Whether tk_merge loads the server's vectors before the kept values: on few tiles nothing else hides that latency, on many the
// registers (102 against 68) cost more wavefronts.  CD-Adam, step plus get_theta, us, late / early: Top-k n = 2, d = 600 000
// 64.2 / 62.0, n = 8, d = 300 000 65.2 / 63.7, d = 2 M 107.7 / 104.3, Rand-k d = 5 M 188.3 / 188.1, Top-k d = 11.2 M bf16 334 / 337, n = 16
// 502 / 510, n = 8, d = 40 M 861 / 889.
inline bool merge_loads_early(int64_t n_tiles) { return n_tiles < 1024; }

// Entries of one of a vector's candidate regions.  A vector's regions together hold twice max(4 k, d / 64) candidates: 1.2 k are
// listed in steady state (error feedback piles mass up just below the threshold), a first step or a step after a miss lists the
// coarse bin of the k-th largest and above (an eighth of an octave of magnitudes: about a hundredth of the coordinates of a gradient
// spread over several decades), and the factor two covers uneven regions.  What does not fit is found without lists (exact_select),
// which needs k entries in all: 8 k are there.  Never more than every coordinate of the region's tiles.
inline int64_t region_entries(int64_t d, int64_t k, int64_t full, int slices)
{
    const int64_t cands = 4 * k > d / 64 ? 4 * k : d / 64;
    const int64_t per_region = ((2 * cands + slices - 1) / slices + 1023) / 1024 * 1024;
    const int64_t most = per_region > 2048 ? per_region : 2048;
    return full < most ? full : most;
}

// Where the listing pass stores a candidate: the first entry of the tile's region, in 64 bits (a vector's regions hold up to 2^31
// entries), and bytes from there on for the place inside the region, of at most a 32nd of 2^31 entries.
constexpr int64_t region_first(int64_t vector, int slices, int slice, uint32_t region_cap) { return (vector * slices + slice) * region_cap; }
constexpr uint32_t offset_bytes(uint32_t at, uint32_t size) { return at * size; }

// Grid of a kernel with one workgroup per tile (in x) under tile_of_block's mapping.
inline unsigned grid_blocks(int64_t n_tiles, int chunk)
{
    if (chunk <= 0) return (unsigned)n_tiles;
    const int64_t span = 8 * (int64_t)chunk;
    return (unsigned)((n_tiles + span - 1) / span * span);
}

// Chunk, in quarter tiles, of the update without compression; choice: comp_ams_set_tile_order's, in tiles (-1: by size).
// Each XCD working through 16 consecutive tiles (64 quarters) of a row at a time is as fast as the plain order or faster at
// every size measured (d = 3 M to 110 M, n = 1 to 64: 0-6 %), as long as there are tiles enough to reach all XCDs: a vector of
// 65 536 coordinates, one chunk, would run on one of them.  A chunk longer than the vector maps its tiles like one of the
// vector's length, but pads the grid to eight chunks of workgroups that leave at once: chunks of 65 536 tiles, n = 4, d = 65 536,
// step plus get_theta 460 us, cut to the length 20.
inline int plain_chunk(int choice, int n_quarters)
{
    const int chunk = choice >= 0 ? 4 * choice : n_quarters >= 8 * 64 ? 64 : 0;
    return chunk < n_quarters ? chunk : n_quarters;
}

// Workers' rows of which the update without compression has a load in flight at a time.  16-bit gradients: two where one leaves
// few bytes in flight, on vectors below 8 Mi coordinates, and up to 16 Mi where the rows of more than eight workers are most of
// what is read; beyond, where the chip streams from memory all the time, two lose.  Step plus get_theta, us, one / two: n = 2,
// d = 1 M 23.9 / 23.6, 4 M 43.9 / 43.0, 14 M 110.9 / 111.5, 60 M 446 / 450; n = 4, 1 M 24.9 / 24.1, 8 M 76.5 / 76.5, 11.2 M 99.9 / 100.8,
// 14 M 118.6 / 119.9, 60 M 484 / 484; n = 8, 1 M 27.0 / 25.5, 8 M 87.6 / 86.5, 14 M 137.1 / 137.7, 30 M 281.6 / 288.1, 60 M 559 / 574;
// n = 16, 1 M 31.2 / 29.8, 8 M 109.1 / 107.0, 11.2 M 150.0 / 147.9, 15.9 M 198.5 / 197.2, 18 M 220.9 / 219.2, 30 M 361 / 372; n = 32, 1 M
// 39.8 / 38.4, 11.2 M 216.9 / 210.5.  (Four at a time, n = 16: 1.2 M 38.0 against 38.3, 11.2 M 155.2 against 149.6.)
inline int plain_rows_ahead(int64_t n, int64_t d, int bytes_per_gradient)
{
    return bytes_per_gradient == 2 && d < ((int64_t)(n > 8 ? 16 : 8) << 20) ? 2 : 1;
}

}  // namespace cams
