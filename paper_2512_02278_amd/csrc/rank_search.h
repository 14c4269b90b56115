// Search of a query over the ranks of its cluster's rows.
//
// With the keys of all rows of a cluster at hand (key_table.h), the rows are first ranked by (key, id).  The search then needs no
// keys and no sorting any more.  What it has scored is a set of ranks, a bit each: the candidate list is the first itopk bits that
// are set, and bringing a neighbour into it is one LDS "or", whether it has been scored before, enters the list or not.  What
// falls off the list's end needs no care either, as bits are only ever added before it.  A lane holds the bits of 64 consecutive
// ranks; the end of the list and the first unexpanded entries are found with one prefix sum over the lanes and ballots.
//
// Ranking: keys fall into 4 096 buckets, a counting sort puts the rows in the order of their buckets, and rows of one bucket, which
// then stand next to each other, count those that they have to change places with.  The buckets are shared out over 128 cells of the
// keys' range by how many rows each cell holds, and divide a cell evenly; every step rounds once, which keeps them monotonous.  (Evenly
// over 3.25 standard deviations on either side of the mean, rows near the query, of which clusters that consist of groups have
// many, met in one bucket.)  Everything after the keys is exact.  Only the first places are settled that way: rows further away are
// hardly ever expanded, and for those that are scored any rank of their own will do.
//
// What it cannot do is left to beam_search_kernel, in a launch of its own that finds a list of such queries: an edge that leaves the cluster,
// keys that are not finite or all the same, more than 255 keys in a lane's 64 buckets (rows far closer to each other than a cell is wide), a far row
// that has to be expanded or returned.
//
// One wavefront per query.
//
// Measured (before: beam_search_kernel with the table), the whole call: 20 000 queries, clusters of 2 439 rows, list of 256, 256 neighbours a round:
// 880 us (1 175; 871 with buckets of one width); where a cluster consists of 50 groups, own noise 0.8, 0.7, 0.3 of the whole, 150 of 0.7, 8 of 0.3, 3 of 0.2:
// 907, 933, 1 002, 885, 948, 905 (1 178, 1 174, 1 121, 1 161, 1 076, 1 112; with buckets of one width, which left most queries to the other search, 1 264, 2 185,
// 2 071, 1 577, 1 818, 2 065); 5 000 queries of 768 fp16 elements, 512 neighbours, in the same order: 552 (645) and 566, 569, 591, 555, 577, 567 (649, 645, 641, 642, 621, 629).
// Copies of rows make crowded buckets: two of each row 910 us (1 185), eight 1 171 (1 145), twenty 1 667 (1 262), fifty 1 949 (1 335);
// where more than half of the rows have a dozen copies nothing is ranked.
// Of a query's time a third is the ranking; a round is a chain of five LDS round trips and a graph row from L2 or the memory-side
// cache.  With all places settled and the rows of all ranks in LDS thirteen wavefronts of a compute unit found
// room instead of eighteen (0.69 ms instead of 0.52 for the search alone); as a first part of beam_search_kernel its registers were those of both (0.60 ms).
#pragma once

#include "search_params.h"

namespace ann {

constexpr int kRankBuckets = 4096;    // 64 for each lane
constexpr int kRankCells = 128;       // 2 for each lane
constexpr int kMaxRankRows = 3072;    // that is what a lane's registers hold; beyond it buckets get crowded
constexpr int kRankBitWords = 64 * 2 + 4;  // a bit per rank, and one that nobody looks at

constexpr int kRankHalo = 12;              // most places a row of a crowded bucket moves
constexpr int kRankTile = 64 - 2 * kRankHalo;  // places settled by a wavefront's registers
constexpr int kRankTiles = 4;              // that are worked on side by side

// LDS words: rows of the first `places` ranks and a halo; ranks of up to `rows` rows and of one more, before that the buckets; bits and parents.
constexpr int rank_row_words(int places) { return (places + kRankHalo + 7) / 8 * 4; }
constexpr int rank_code_words(int rows) { return rows / 2 + 1 > kRankBuckets / 4 ? (rows / 2 + 4) / 4 * 4 : kRankBuckets / 4; }
constexpr int rank_lds_bytes(int rows, int places) { return 4 * (rank_row_words(places) + rank_code_words(rows) + kRankBitWords + 64); }

// `cpl` registers of 64 neighbours a round: 2, 4 or 8 (with one the list is short too, and nothing would be gained).
hipError_t launch_rank_search(const SearchParams& p, int cpl, unsigned grid, size_t lds_bytes, hipStream_t stream);

}  // namespace ann
