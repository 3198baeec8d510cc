// pic_sort.h -- enqueue functions of the cell sort (pic_sort.hip).
#pragma once
#include <algorithm>

#include "pic_internal.h"

namespace pic {

// Digits of the radix sort: passes of at most kDigitBits bits, as equal as the key's bits allow.  A pass is
// three launches (15 to 20 us on small sorts, of which the work is a third), so the fewest passes win; with
// the launches saved around them, the sort of 240 thousand particles by 20-bit keys takes 65 us for 87
// with three passes of 8 bits, one of 16 thousand by 10-bit keys 25 for 43.  kDigitBits is what the scatter's
// 16-bit counts of a block's wavefronts fit into 32 KB of LDS.
constexpr int kDigitBits = 10;
constexpr int kSortPart = 8 << kDigitBits;   // words of sort_part
constexpr int kCompactPart = 2048;           // words of compact_part

// Keys per radix-sort block: 4096, doubled until at most 2048 blocks cover n keys (the digit
// histogram holds a count per digit and block), and for small sorts halved down to 1024 (one key per
// thread) while fewer than 512 blocks would cover them, so that the blocks fill the 256 CUs.
__host__ __device__ inline int sort_blocks(int n, int shift) { return n > 0 ? ((n - 1) >> shift) + 1 : 0; }
__host__ __device__ inline int sort_shift(int n)  // log2 of the keys per block
{
    int sh = 12;
    while (sort_blocks(n, sh) > 2048) ++sh;
    while (sh > 10 && sort_blocks(n, sh) < 512) --sh;
    return sh;
}

// Sorts of up to kFuseBlocks blocks form the digit totals in the histogram pass, with one atomic per block
// and digit met (sort_part is zero on entry: each scatter pass clears it); larger ones in k_radix_rowsum.
// Up to kDirectBlocks blocks each scatter block scans the histogram itself: its rows are then at most
// 128 KB in L2, and the launch it saves costs as much as the whole pass (4 to 5 us).  Beyond kScanBlocks the
// scan splits the histogram's columns finer (k_radix_rowscan).
constexpr int kFuseBlocks = 1024;
constexpr int kScanBlocks = 512;
constexpr int kDirectBlocks = 32;

// What a sort's launches are sized for: the most particles, histogram blocks, passes, digit bits and tiles of
// the simulations it covers (each kernel takes its own from the table); elem = 4 (FP32 form) or 8.
struct SortShape {
    int n = 0, blocks = 0, passes = 0, bits = 0, ntiles = 0, elem = 4;
    void cover(const SimDev& h, int np)
    {
        n = std::max(n, np);
        blocks = std::max(blocks, sort_blocks(np, sort_shift(np)));
        passes = std::max(passes, h.sort_passes);
        bits = std::max(bits, h.sort_bits);
        ntiles = std::max(ntiles, h.ntiles);
    }
    // do the launches of a table sized for this serve a simulation of shape q as well?
    bool covers(const SortShape& q) const
    {
        return passes >= q.passes && (n > 0 || q.n == 0) && (blocks > kDirectBlocks || q.blocks <= kDirectBlocks) &&
               (blocks > kScanBlocks || q.blocks <= kScanBlocks) && (blocks > kFuseBlocks || q.blocks <= kFuseBlocks);
    }
};

// Stable radix sort by cell key of species s of one simulation (slots = 1), or of the s-th moving species
// that holds particles of every slot of a table (moving), its arrays permuted into the alternates, and
// its tile ranges.  enqueue_compact must follow: it swaps the arrays with their alternates.
hipError_t enqueue_sort(SimDev* sims, int slots, int s, bool moving, const SortShape& q, hipStream_t st);
// Keys of species s into its key buffer (diagnostics).
hipError_t enqueue_keys_only(SimDev* dS, int s, int n, hipStream_t st);

// What the unit lists' launches are sized for: lists of one round, longer ones (their blocks, and those that
// count the active tiles where the units' size is open), field masks.
struct CompactShape {
    bool one = false;
    int blocks = 0, active = 0, masks = 0;
    void cover(const SimDev& h);
    bool covers(const CompactShape& q) const
    {
        return (one || !q.one) && (blocks > 0 || q.blocks == 0) && (active > 0 || q.active == 0);
    }
};

// Unit lists and field masks of the slots; swap: the species whose arrays are swapped with their alternates,
// a bit each, or -1 for every moving one that holds particles.
hipError_t enqueue_compact(SimDev* sims, int slots, const CompactShape& q, int swap, hipStream_t st);

}  // namespace pic
