// pic_sort.hip -- cell sort of libpic: stable LSD radix sort of the int32 tile-major cell keys,
// permutation of the particle arrays, per-tile particle ranges and the work units of the tiles that hold particles.
//
// Keys and permutation are bit-exact with a stable sort: each pass ranks equal digits in
// input order (wavefront multisplit with ballots, then waves in order, then blocks in order).
// All kernels read their arrays through the device SimDev table, so a captured graph stays
// valid when the array pointers are swapped after each sort.
#include <algorithm>

#include "pic_dpp.h"
#include "pic_internal.h"
#include "pic_sort.h"
#include "pic.h"
#include "pic_measure.h"

namespace pic {

constexpr int kRadixMax = 1 << kDigitBits;
constexpr int kSortBlock = 1024;
// the fused digit totals are spread over kPartCopies copies (block b adds into copy b % copies) so
// that fewer blocks queue on each address; the row scan sums the copies
constexpr int kPartCopies = 8;
static_assert(kPartCopies * kRadixMax == kSortPart, "scratch of the digit totals");
static_assert(kRadixMax <= kSortBlock, "a thread of the scatter per digit");
// Which species a launch sorts: species s, or of each of the table's slots (grid.y) its s-th moving one.
struct SortSel {
    int s, moving;
};

// the species that sel names in the slot's entry, or -1
__device__ __forceinline__ int sel_species(const SimDev& S, const SortSel& sel)
{
    if (!sel.moving) return sel.s;
    int j = sel.s;
    for (int s = 0; s < S.nspecies; ++s)
        if (S.sp[s].kind != BOUND && S.sp[s].n > 0 && j-- == 0) return s;
    return -1;
}

// keys[i] = tile-major key of particle i's cell (anchor cell for bound particles)
__device__ __forceinline__ int particle_key(const SimDev& S, const SpeciesDev& sp, int i)
{
    int c[3];
    unpack_cell(S, sp.cell[i], c);
    return cell_key(S, c);
}

__global__ void k_keys(SimDev* __restrict__ S, int s)
{
    const SpeciesDev& sp = S->sp[s];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < sp.n; i += gridDim.x * blockDim.x) sp.keys[i] = particle_key(*S, sp, i);
}

// digit histogram per block: hist[b * nd + d], each block's row written and read whole.  The first pass forms the keys from the cells (the values that
// the passes carry start as the identity, which its scatter forms from the index).
template <bool FIRST>
__global__ void __launch_bounds__(kSortBlock) k_radix_hist(const SimDev* __restrict__ sims, SortSel sel, int pass)
{
    __shared__ int h[kRadixMax];
    const SimDev& S = sims[blockIdx.y];
    const int s = sel_species(S, sel);
    if (s < 0 || pass >= S.sort_passes) return;
    const SpeciesDev& sp = S.sp[s];
    int* keys = (pass & 1) ? sp.keys_alt : sp.keys;
    const int n = sp.n, sh = sort_shift(n), ipb = 1 << sh, nb = sort_blocks(n, sh);
    const int nd = 1 << S.sort_bits, shift = pass * S.sort_bits;
    const bool fuse = nb <= kFuseBlocks && nb > kDirectBlocks;
    for (int b = blockIdx.x; b < nb; b += gridDim.x) {
        for (int d = threadIdx.x; d < nd; d += kSortBlock) h[d] = 0;
        __syncthreads();
        const int lo = b * ipb, hi = min(n, lo + ipb);
        for (int i = lo + threadIdx.x; i < hi; i += kSortBlock) {
            int key;
            if constexpr (FIRST) sp.keys[i] = key = particle_key(S, sp, i);
            else key = keys[i];
            atomicAdd(&h[(key >> shift) & (nd - 1)], 1);
        }
        __syncthreads();
        for (int d = threadIdx.x; d < nd; d += kSortBlock) {
            const int c = h[d];
            S.sort_hist[b * nd + d] = c;
            if (fuse && c) atomicAdd(&S.sort_part[(b % kPartCopies) * kRadixMax + d], c);
        }
        __syncthreads();
    }
}

constexpr int kScanThreads = 1024;
constexpr int kUnitBlock = 4;  // tiles per active axis of a block of the unit list

// inclusive scan of v over a block of NT threads: DPP wavefront scans, then the wave totals in order;
// *total receives the block total
template <int NT = kScanThreads>
__device__ __forceinline__ int block_scan(int v, int* wsum, int* total)
{
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int inc = seg_scan<int>(v, scan_masks(lane));
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int carry = 0, all = 0;
    for (int w = 0; w < NW; ++w) {
        const int x = wsum[w];
        if (w < wave) carry += x;
        all += x;
    }
    __syncthreads();
    *total = all;
    return carry + inc;
}

// Digits of a block of the row scan (64 bytes of each row of hist), and the groups of rows it takes them in.
constexpr int kScanDigits = 16;
constexpr int kScanGroups = kScanThreads / kScanDigits;
// Sums over the blocks b of hist[b * nd + d] (sorts of many blocks: the histogram pass's per-digit atomics would
// queue on the digits' addresses).  The rows are split over kPartCopies blocks, each of which writes a
// copy of the totals: 16 blocks for all rows of a 256-digit pass took 12.6 us on the 256^3 sphere, now 4.5.
__global__ void __launch_bounds__(kScanThreads) k_radix_rowsum(const SimDev* __restrict__ sims, SortSel sel, int pass)
{
    __shared__ int part[kScanGroups][kScanDigits];
    const SimDev& S = sims[blockIdx.y];
    const int s = sel_species(S, sel);
    if (s < 0 || pass >= S.sort_passes) return;
    const int n = S.sp[s].n, nb = sort_blocks(n, sort_shift(n)), nd = 1 << S.sort_bits;
    if (nb <= kFuseBlocks) return;
    const int l = threadIdx.x % kScanDigits, g = threadIdx.x / kScanDigits;
    const int copy = blockIdx.x % kPartCopies;
    for (int d0 = blockIdx.x / kPartCopies * kScanDigits; d0 < nd; d0 += gridDim.x / kPartCopies * kScanDigits) {
        int acc = 0;
        if (d0 + l < nd)
            for (int b = copy * kScanGroups + g; b < nb; b += kPartCopies * kScanGroups) acc += S.sort_hist[(long long)b * nd + d0 + l];
        part[g][l] = acc;
        __syncthreads();
        if (g == 0 && d0 + l < nd) {
            int total = 0;
            for (int k = 0; k < kScanGroups; ++k) total += part[k][l];
            S.sort_part[copy * kRadixMax + d0 + l] = total;
        }
        __syncthreads();
    }
}

// Column d of hist replaced by its exclusive prefix over the blocks, from the sum of the totals of the lower
// digits on: D columns per block, whose rows are split into 1024 / D consecutive groups of at most kScanRows
// rows each, held in registers between the two passes over them.  D = 16 up to kScanBlocks blocks (64 bytes of a
// row a block), 4 for up to the 2048 that a sort has: with 16 blocks of 16 columns, the rows read twice, a
// pass of the 256^3 sphere took 12.8 us, now 8.7 (12.2 where the blocks of a line lie on eight XCDs).
constexpr int kScanRows = 8;
static_assert(kScanRows * (kScanThreads / 16) == kScanBlocks && kScanRows * (kScanThreads / 4) == 2048, "rows of a sort's blocks");
template <int D>
__global__ void __launch_bounds__(kScanThreads) k_radix_rowscan(const SimDev* __restrict__ sims, SortSel sel, int pass)
{
    constexpr int G = kScanThreads / D;
    __shared__ int wsum[kScanThreads / 64];
    __shared__ int part[G][D];
    __shared__ int part8[G / 8][D];
    __shared__ int digit[D];
    const SimDev& S = sims[blockIdx.y];
    const int s = sel_species(S, sel);
    if (s < 0 || pass >= S.sort_passes) return;
    const int n = S.sp[s].n, nb = sort_blocks(n, sort_shift(n)), nd = 1 << S.sort_bits;
    if (nb <= kDirectBlocks || (nb > kScanBlocks) != (D < 16)) return;
    const int l = threadIdx.x % D, g = threadIdx.x / D;
    const int k = (nb + G - 1) / G;
    const int b0 = min(nb, g * k), rows = min(nb - b0, k);
    // neighbouring columns on one XCD: the blocks that write parts of a line meet in one L2
    const int at = gridDim.x % kXcds ? (int)blockIdx.x : (int)(blockIdx.x % kXcds * (gridDim.x / kXcds) + blockIdx.x / kXcds);
    for (int d0 = at * D; d0 < nd; d0 += gridDim.x * D) {
        // the rows first: no condition holds these loads back, so all are in flight while the totals are read
        const bool in = d0 + l < nd && rows > 0;
        int* col = S.sort_hist + (in ? b0 * nd + d0 + l : 0);
        int keep[kScanRows];
#pragma unroll
        for (int t = 0; t < kScanRows; ++t) keep[t] = col[in ? min(t, rows - 1) * nd : 0];
        int lower;  // sum of the totals of digits 0 .. d0 - 1
        int mine = 0;
        for (int t = threadIdx.x; t < d0 + D && t < nd; t += kScanThreads) {
            int x = 0;
#pragma unroll
            for (int c = 0; c < kPartCopies; ++c) x += S.sort_part[c * kRadixMax + t];
            if (t < d0) mine += x;
            else digit[t - d0] = x;
        }
        int run = 0;
#pragma unroll
        for (int t = 0; t < kScanRows; ++t) run += in && t < rows ? keep[t] : 0;
        part[g][l] = run;
        block_scan(mine, wsum, &lower);
        // the groups before: whole eights, then the rest
        if (g % 8 == 0) {
            int x = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t) x += part[g + t][l];
            part8[g / 8][l] = x;
        }
        __syncthreads();
        int acc = lower;
#pragma unroll
        for (int t = 0; t < D; ++t) acc += t < l && d0 + t < nd ? digit[t] : 0;
        for (int t = 0; t < g / 8; ++t) acc += part8[t][l];
        for (int t = g / 8 * 8; t < g; ++t) acc += part[t][l];
#pragma unroll
        for (int t = 0; t < kScanRows; ++t)
            if (in && t < rows) {
                col[t * nd] = acc;
                acc += keep[t];
            }
        __syncthreads();
    }
}

// Stable scatter of one pass, in rounds of K keys per thread (key j of thread t in a round is the
// round's key j * kSortBlock + t, so the keys of a round are taken in input order item by item).
// Each wavefront ranks its lanes' equal digits with ballots and its first lane of each digit
// stores the count; a thread per item and digit then turns the wavefronts' counts, in input order, into the
// position of each group's first key in the round, and every key goes to the digit's next slot (base) plus
// that and its rank.
constexpr int kScatterCounts = (kSortBlock / 64) * kRadixMax;  // 16-bit counts of a round: 32 KB
template <int K>
__device__ __forceinline__ void scatter_block(const SimDev& S, const SpeciesDev& sp, int pass, int n, int ipb, int nb, int b,
                                              int* base, unsigned short* wcnt, int* jtot, int* wsum)
{
    constexpr int NW = kSortBlock / 64;
    constexpr int kBits = kDigitBits - (K == 4 ? 2 : K == 2 ? 1 : 0);  // the most a digit has with this K
    const int* kin = (pass & 1) ? sp.keys_alt : sp.keys;
    const int* vin = (pass & 1) ? sp.vals_alt : sp.vals;
    int* kout = (pass & 1) ? sp.keys : sp.keys_alt;
    int* vout = (pass & 1) ? sp.vals : sp.vals_alt;
    const int bits = S.sort_bits, nd = 1 << bits, shift = pass * bits;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // thread d: the next slot of digit d's keys of this block
    int run = 0;
    if (nb > kDirectBlocks) {
        if (tid < nd) run = S.sort_hist[b * nd + tid];
    } else {
        int total = 0, before = 0, all;
        if (tid < nd)
            for (int k = 0; k < nb; ++k) {
                const int x = S.sort_hist[k * nd + tid];
                total += x;
                before += k < b ? x : 0;
            }
        run = block_scan<kSortBlock>(total, wsum, &all) - total + before;
    }
    if (tid < nd) base[tid] = run;
    const int item = tid >> bits, digit = tid & (nd - 1);  // of the counts
    const int lo = b * ipb, hi = min(n, lo + ipb);
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int first = lo; first < hi; first += K * kSortBlock) {
        unsigned* wz = reinterpret_cast<unsigned*>(wcnt);
        for (int i = tid; i < K * NW * nd / 2; i += kSortBlock) wz[i] = 0u;
        int key[K], val[K], d[K], rank[K];
        bool act[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = first + j * kSortBlock + tid;
            act[j] = i < hi;
            key[j] = act[j] ? kin[i] : 0;
            val[j] = act[j] ? (pass == 0 ? i : vin[i]) : 0;  // the first pass carries each key's own index
            d[j] = (key[j] >> shift) & (nd - 1);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < K; ++j) {
            // lanes of this wave holding the same digit
            unsigned long long peers = __ballot(act[j]);
#pragma unroll
            for (int bit = 0; bit < kBits; ++bit) {
                const unsigned long long m = __ballot(act[j] && ((d[j] >> bit) & 1));
                peers &= ((d[j] >> bit) & 1) ? m : ~m;
            }
            rank[j] = __popcll(peers & lt);
            if (act[j] && rank[j] == 0) wcnt[(j * NW + wave) * nd + d[j]] = (unsigned short)__popcll(peers);
        }
        __syncthreads();
        int acc = 0;
        unsigned short* mine = wcnt + (item * NW) * nd + digit;
        if constexpr (K > 1) {
            if (item < K) {
                int total = 0;
#pragma unroll 4
                for (int w = 0; w < NW; ++w) total += mine[w * nd];
                jtot[tid] = total;
            }
            __syncthreads();
            if (item < K)
                for (int j = 0; j < item; ++j) acc += jtot[(j << bits) + digit];
        }
        if (item < K)
            for (int w = 0; w < NW; w += 4) {
                int c[4];  // (read before the first is replaced: one wait for four)
#pragma unroll
                for (int j = 0; j < 4; ++j) c[j] = mine[(w + j) * nd];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    mine[(w + j) * nd] = (unsigned short)acc;
                    acc += c[j];
                }
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (act[j]) {
                const int off = base[d[j]] + wcnt[(j * NW + wave) * nd + d[j]] + rank[j];
                kout[off] = key[j];
                vout[off] = val[j];
            }
        __syncthreads();
        if (item == K - 1) base[digit] += acc;  // (read again after the next round's barriers)
    }
}

// K items a thread and round: 4 where the digits' counts of four items fit and the blocks hold as many keys;
// 1 for a table, whose members' digits differ (with 4 there where they allow it, two 128^3 spheres of 6.3 million
// electrons each took 431 us a step for 433).
// At most 64 registers, so that two blocks share a CU.
template <int K>
__global__ void __launch_bounds__(kSortBlock, 8) k_radix_scatter(const SimDev* __restrict__ sims, SortSel sel, int pass)
{
    __shared__ int base[kRadixMax];
    __shared__ __align__(4) unsigned short wcnt[kScatterCounts];
    __shared__ int jtot[K > 1 ? kSortBlock : 1];
    __shared__ int wsum[kSortBlock / 64];
    const SimDev& S = sims[blockIdx.y];
    const int s = sel_species(S, sel);
    if (s < 0 || pass >= S.sort_passes) return;
    const SpeciesDev& sp = S.sp[s];
    const int n = sp.n, sh = sort_shift(n), ipb = 1 << sh, nb = sort_blocks(n, sh);
    // the digit totals of this pass were consumed by the row scan: clear them for the next pass
    if (blockIdx.x == 0 && nb > kDirectBlocks)
        for (int d = threadIdx.x; d < kSortPart; d += kSortBlock) S.sort_part[d] = 0;
    for (int b = blockIdx.x; b < nb; b += gridDim.x) {
        scatter_block<K>(S, sp, pass, n, ipb, nb, b, base, wcnt, jtot, wsum);
        __syncthreads();
    }
}

// After the last pass the sorted keys and the source index of each slot sit in keys/vals
// (even number of passes) or keys_alt/vals_alt (odd).  The first nr blocks find tile_start[t] = first sorted index
// whose key >= t * tile volume (lower bound), t = 0..ntiles, the others gather every particle array into
// its alternate buffer: both need only the sorted keys, and the search's chain of loads (7 us as a launch
// of its own) hides behind the gather.
__global__ void k_permute(const SimDev* __restrict__ sims, SortSel sel, int elem, int nr)
{
    const SimDev& S = sims[blockIdx.y];
    const int s = sel_species(S, sel);
    if (s < 0) return;
    const SpeciesDev& sp = S.sp[s];
    const int n = sp.n;
    const bool odd = (S.sort_passes & 1) != 0;
    if ((int)blockIdx.x < nr) {
        const int* keys = odd ? sp.keys_alt : sp.keys;
        const int tvol = S.T[0] * S.T[1] * S.T[2];
        for (int t = blockIdx.x * blockDim.x + threadIdx.x; t <= S.ntiles; t += nr * blockDim.x) {
            const long long target = (long long)t * tvol;
            int lo = 0, hi = n;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if ((long long)keys[mid] < target) lo = mid + 1; else hi = mid;
            }
            sp.tile_start[t] = lo;
        }
        return;
    }
    const int* perm = odd ? sp.vals_alt : sp.vals;
    const int dims = S.dims;
    const bool bound = sp.kind == BOUND;
    for (int i = (blockIdx.x - nr) * blockDim.x + threadIdx.x; i < n; i += (gridDim.x - nr) * blockDim.x) {
        const int j = perm[i];
        sp.cell_alt[i] = sp.cell[j];
        if (elem == 4) {
            for (int a = 0; a < dims; ++a)
                reinterpret_cast<float*>(sp.off_alt[a])[i] = reinterpret_cast<const float*>(sp.off[a])[j];
            for (int a = 0; a < 3; ++a)
                reinterpret_cast<float*>(sp.v_alt[a])[i] = reinterpret_cast<const float*>(sp.v[a])[j];
            if (bound)
                for (int a = 0; a < 3; ++a)
                    reinterpret_cast<float*>(sp.xi_alt[a])[i] = reinterpret_cast<const float*>(sp.xi[a])[j];
            else if (sp.mpp)
                reinterpret_cast<float*>(sp.xi_alt[0])[i] = reinterpret_cast<const float*>(sp.xi[0])[j];
        } else {
            for (int a = 0; a < dims; ++a)
                reinterpret_cast<double*>(sp.off_alt[a])[i] = reinterpret_cast<const double*>(sp.off[a])[j];
            for (int a = 0; a < 3; ++a)
                reinterpret_cast<double*>(sp.v_alt[a])[i] = reinterpret_cast<const double*>(sp.v[a])[j];
            if (bound)
                for (int a = 0; a < 3; ++a)
                    reinterpret_cast<double*>(sp.xi_alt[a])[i] = reinterpret_cast<const double*>(sp.xi[a])[j];
            else if (sp.mpp)
                reinterpret_cast<double*>(sp.xi_alt[0])[i] = reinterpret_cast<const double*>(sp.xi[0])[j];
        }
    }
}

// The particle arrays of the sorted species swapped with their alternates, into which the permutation was
// gathered: mask, a bit per species, or -1 for every moving one that holds particles.
__device__ __forceinline__ void swap_sorted(SimDev* S, int mask)
{
    for (int s = 0; s < S->nspecies; ++s) {
        SpeciesDev& w = S->sp[s];
        if (!(mask < 0 ? w.kind != BOUND && w.n > 0 : (mask >> s) & 1)) continue;
        int* c = w.cell; w.cell = w.cell_alt; w.cell_alt = c;
        for (int a = 0; a < 3; ++a) {
            void* t = w.off[a]; w.off[a] = w.off_alt[a]; w.off_alt[a] = t;
            t = w.v[a]; w.v[a] = w.v_alt[a]; w.v_alt[a] = t;
            t = w.xi[a]; w.xi[a] = w.xi_alt[a]; w.xi_alt[a] = t;
        }
    }
}

// Active tiles (any species has particles) and their work units: a tile holding c particles (all
// species) gets ceil(c / U) units of at most U particles, in its species-concatenated order, U the
// caller's cap or one chosen here (auto_unit_cap); the units of a tile take consecutive slots.
//
// Tiles are listed in blocks of kUnitBlock tiles along each active axis (x fastest inside a block,
// blocks in x-fastest order), so that tiles near each other along every axis are near each other
// in the list, and the particle kernel, which takes units in list order on each XCD, processes them
// close together in time (their shared window halos meet in L2).  Ranks run over the grid of tiles
// padded to whole blocks; a rank whose tile lies beyond the grid is skipped.
//
// A list of one round is built by one block in one launch (k_compact_one).  Longer lists take
// three launches over rounds of kCompactK * 1024 ranks (each thread kCompactK consecutive ranks),
// each block of the first and last taking a contiguous run of rounds: k_compact_count forms each
// block's totals of active tiles and units, k_compact_scan their exclusive prefix in block order
// (and whether the lists fit), k_compact_place places the tiles and units of each round with a
// block scan from its block's prefix.  The block totals and prefixes live in compact_part.
//
// The launches take a slot of the table per grid.y (an empty slot has no tiles), and the first one also
// finds the field masks, in the blocks after those of the list.
constexpr int kCompactK = 4;
constexpr int kCompactBlocks = kCompactPart / 2 - 1;  // block totals in compact_part (its last word: the fit flag)

struct CompactGeom {
    int sh[3], nb[3], vsh, nt, rounds, rpb;
    __device__ __forceinline__ CompactGeom(const SimDev* S, int blocks)
    {
        static_assert((kUnitBlock & (kUnitBlock - 1)) == 0 && kUnitBlock % kCompactK == 0, "blocks of whole thread runs");
        constexpr int kBS = kUnitBlock == 4 ? 2 : (kUnitBlock == 8 ? 3 : 1);  // log2 of kUnitBlock
        for (int a = 0; a < 3; ++a) {
            sh[a] = a < S->dims ? kBS : 0;
            nb[a] = (S->ntile[a] + (1 << sh[a]) - 1) >> sh[a];
        }
        vsh = sh[0] + sh[1] + sh[2];                 // log2 of the ranks per block
        nt = (nb[0] * nb[1] * nb[2]) << vsh;         // padded ranks
        rounds = (nt + kCompactK * kScanThreads - 1) / (kCompactK * kScanThreads);
        rpb = (rounds + blocks - 1) / blocks;        // rounds per block
    }
    // the tiles of ranks r .. r + kCompactK - 1 (-1 beyond the grid); they lie in one block of the
    // list (a block holds a multiple of kCompactK ranks), so its position is divided out once
    __device__ __forceinline__ void tiles_of(const SimDev* S, int r, int (&t)[kCompactK]) const
    {
        const int blk = r >> vsh;
        const int b1 = blk / nb[0];
        const int o0 = (blk - b1 * nb[0]) << sh[0];
        const int b2 = b1 / nb[1];
        const int o1 = (b1 - b2 * nb[1]) << sh[1], o2 = b2 << sh[2];
#pragma unroll
        for (int j = 0; j < kCompactK; ++j) {
            const int w = (r + j) & ((1 << vsh) - 1);
            const int c0 = o0 + (w & ((1 << sh[0]) - 1));
            const int c1 = o1 + ((w >> sh[0]) & ((1 << sh[1]) - 1));
            const int c2 = o2 + (w >> (sh[0] + sh[1]));
            t[j] = r + j < nt && c0 < S->ntile[0] && c1 < S->ntile[1] && c2 < S->ntile[2]
                       ? (c2 * S->ntile[1] + c1) * S->ntile[0] + c0
                       : -1;
        }
    }
};

__device__ __forceinline__ int compact_count(const SimDev* S, int t)
{
    int c = 0;
    for (int s = 0; s < S->nspecies; ++s) c += S->sp[s].tile_start[t + 1] - S->sp[s].tile_start[t];
    return c;
}
__device__ __forceinline__ long long compact_total(const SimDev* S)
{
    long long n = 0;
    for (int s = 0; s < S->nspecies; ++s) n += S->sp[s].n;
    return n;
}
// the cap of the list's units: the caller's, or chosen for its active tiles
__device__ __forceinline__ int compact_cap(const SimDev* S, long long n, int active)
{
    return S->unit_cap > 0 ? S->unit_cap : auto_unit_cap(n, active, S->unit_goal);
}
// ceil(c / cap); below 2^22 particles the quotient of the rounded reciprocal is off by at most one
__device__ __forceinline__ int compact_units(int c, int cap)
{
    if (c >= 1 << 22) return (int)(((unsigned)c - 1u) / (unsigned)cap) + 1;
    int q = (int)((float)c * __builtin_amdgcn_rcpf((float)cap));
    int r = c - q * cap;
    if (r < 0) { --q; r += cap; }
    if (r >= cap) { ++q; r -= cap; }
    return q + (r > 0 ? 1 : 0);
}

// unit q of the k of tile t (c particles), a part of its species-concatenated order: the caller's cap at a time,
// or equal parts, in whole chunks of 64, where the cap is chosen here.  The equal parts are cut between groups
// of kScanGroup of a species' particles, the groups in which the particle kernel adds up deposits
// before it rounds them to quanta: the current is then that of the whole tile as one unit, bit for bit,
// whatever size was chosen (a unit holds at most kScanGroup - 1 particles more than its cap).
__device__ __forceinline__ void put_unit(const SimDev* S, UnitDev& u, int q, int k, int t, int cap)
{
    const int ns = S->nspecies;
    int t0[MAXSP], n[MAXSP], c = 0;
#pragma unroll
    for (int s = 0; s < MAXSP; ++s) {
        t0[s] = s < ns ? S->sp[s].tile_start[t] : 0;
        n[s] = s < ns ? S->sp[s].tile_start[t + 1] - t0[s] : 0;
        c += n[s];
    }
    const bool chosen = S->unit_cap == 0;
    int per = cap;
    if (chosen) {
        per = (c + k - 1) / k;
        per = min((per + 63) / 64 * 64, cap);  // k = ceil(c / cap), so no part is empty
    }
    u.tile = t;
    const int ub = q * per, ue = min(c, (q + 1) * per);
    int base = 0;  // first index of species s in the concatenated order
    auto cut = [&](int at, int s) {
        const int d = min(max(at - base, 0), n[s]);
        return t0[s] + (chosen && d < n[s] ? d & ~(kScanGroup - 1) : d);
    };
#pragma unroll
    for (int s = 0; s < MAXSP; ++s) {
        u.range[s][0] = cut(ub, s);
        u.range[s][1] = cut(ue, s);
        base += n[s];
    }
}

// fmask of every field task: the columns (x index) of active particle tiles whose deposits reach it, as bits
// from the first reaching column on; one bit for all of them where there are more than 32 (tiles
// narrower than 3 cells), and in 1D.  A task reaches one cell past its own along each axis (the last
// one along an open axis also owns node n).  The active tiles change only with the sort, so the field
// kernel reads the mask and does not search the tiles itself: its search of up to 150 of them was 2 of
// the 13 us of the 16^3 cube's field kernel.  One wavefront per task, one candidate tile per lane; block b
// of nb.
template <int DIM>
__device__ __forceinline__ void field_masks(const SimDev& S, int b, int nb)
{
    const int lane = threadIdx.x & 63;
    for (int ft = __builtin_amdgcn_readfirstlane(b * (kScanThreads / 64) + (threadIdx.x >> 6)); ft < S.nftiles;
         ft += nb * (kScanThreads / 64)) {
        const int tf[3] = {ft % S.nft[0], (ft / S.nft[0]) % S.nft[1], ft / (S.nft[0] * S.nft[1])};
        int tlo[3] = {0, 0, 0}, cnt[3] = {1, 1, 1};
        for (int a = 0; a < DIM; ++a) {
            int x0 = tf[a] * S.FT[a], x1 = x0 + S.FT[a];
            if (DIM == 3 && a == 1) {
                // the plane march's row groups end at the last row
                x0 = max(0, min(x0, S.L[1] - S.FT[1]));
                x1 = x0 + S.FT[1];
            }
            if (DIM == 3 && a == 2 && tf[2] == S.nft[2] - 1) x1 = S.L[2];
            reaching_tiles(S, a, x0, S.periodic[a] ? min(x1, S.n[a]) : x1, tlo[a], cnt[a]);
        }
        unsigned xm = 0u;
        for (int t = lane; t < cnt[0] * cnt[1] * cnt[2]; t += 64) {
            int t3[3] = {tlo[0] + t % cnt[0], tlo[1] + (t / cnt[0]) % cnt[1], tlo[2] + t / (cnt[0] * cnt[1])};
            bool in = true;
            for (int a = 0; a < DIM; ++a) {
                if (S.periodic[a]) {
                    t3[a] %= S.ntile[a];
                    if (t3[a] < 0) t3[a] += S.ntile[a];
                } else if (t3[a] < 0 || t3[a] >= S.ntile[a]) {
                    in = false;
                }
            }
            if (in && compact_count(&S, (t3[2] * S.ntile[1] + t3[1]) * S.ntile[0] + t3[0]) > 0)
                xm |= DIM > 1 && cnt[0] <= 32 ? 1u << (t % cnt[0]) : ~0u;
        }
        for (int off = 32; off > 0; off >>= 1) xm |= (unsigned)__shfl_xor((int)xm, off, 64);
        if (lane == 0) S.fmask[ft] = xm;
    }
}

__device__ __forceinline__ void field_masks(const SimDev& S, int b, int nb)
{
    if (S.dims == 1) field_masks<1>(S, b, nb);
    else if (S.dims == 2) field_masks<2>(S, b, nb);
    else field_masks<3>(S, b, nb);
}

// Active tiles per block (sort_hist, free once the species are sorted), where the cap is chosen from
// their number.
__global__ void __launch_bounds__(kScanThreads) k_compact_active(const SimDev* sims)
{
    __shared__ int wsum[kScanThreads / 64];
    const SimDev* S = sims + blockIdx.y;
    if (S->unit_cap > 0 || CompactGeom(S, 1).rounds <= 1) return;
    int ca = 0;
    for (int t = blockIdx.x * kScanThreads + threadIdx.x; t < S->ntiles; t += gridDim.x * kScanThreads)
        ca += compact_count(S, t) > 0 ? 1 : 0;
    int ta;
    block_scan(ca, wsum, &ta);
    if (threadIdx.x == 0) S->sort_hist[blockIdx.x] = ta;
}

__global__ void __launch_bounds__(kScanThreads) k_compact_count(SimDev* sims, int nactive, int nblocks)
{
    __shared__ int wsum[kScanThreads / 64];
    SimDev* S = sims + blockIdx.y;
    const CompactGeom G(S, nblocks);
    if (G.rounds <= 1) return;
    if ((int)blockIdx.x >= nblocks) {
        field_masks(*S, blockIdx.x - nblocks, gridDim.x - nblocks);
        return;
    }
    int ca = 0, cu = 0;
    int active = 0;
    if (S->unit_cap == 0) block_scan((int)threadIdx.x < nactive ? S->sort_hist[threadIdx.x] : 0, wsum, &active);
    const int cap = compact_cap(S, compact_total(S), active);
    const int r0 = blockIdx.x * G.rpb, r1 = min(G.rounds, r0 + G.rpb);
    for (int round = r0; round < r1; ++round) {
        int t[kCompactK];
        G.tiles_of(S, round * kCompactK * kScanThreads + threadIdx.x * kCompactK, t);
#pragma unroll
        for (int j = 0; j < kCompactK; ++j) {
            const int c = t[j] >= 0 ? compact_count(S, t[j]) : 0;
            ca += c > 0 ? 1 : 0;
            cu += compact_units(c, cap);
        }
    }
    int ta, tu;
    block_scan(ca, wsum, &ta);
    block_scan(cu, wsum, &tu);
    if (threadIdx.x == 0) {
        S->compact_part[2 * blockIdx.x] = ta;
        S->compact_part[2 * blockIdx.x + 1] = tu;
        if (blockIdx.x == 0) S->unit_now = cap;
    }
}

// one block: the blocks' exclusive prefixes in place of their totals, the list lengths, and whether
// the lists fit (a list that does not fit, with particles in tiles the capacity did not count, is
// dropped whole and flagged: no particle moves this period)
__global__ void __launch_bounds__(kScanThreads) k_compact_scan(SimDev* sims, int nblocks)
{
    __shared__ int wsum[kScanThreads / 64];
    __shared__ int carry[2];
    SimDev* S = sims + blockIdx.y;
    if (CompactGeom(S, 1).rounds <= 1) return;
    if (threadIdx.x < 2) carry[threadIdx.x] = 0;
    __syncthreads();
    for (int base = 0; base < nblocks; base += kScanThreads) {
        const int b = base + threadIdx.x;
        const int a = b < nblocks ? S->compact_part[2 * b] : 0, u = b < nblocks ? S->compact_part[2 * b + 1] : 0;
        int sa, su;
        const int pa = block_scan(a, wsum, &sa) - a + carry[0];
        const int pu = block_scan(u, wsum, &su) - u + carry[1];
        if (b < nblocks) {
            S->compact_part[2 * b] = pa;
            S->compact_part[2 * b + 1] = pu;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            carry[0] += sa;
            carry[1] += su;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int ta = carry[0], tu = carry[1];
        const bool fits = ta <= S->max_slots && tu <= S->max_units;
        S->compact_part[kCompactPart - 1] = fits ? 1 : 0;
        *S->n_active = fits ? ta : 0;
        *S->n_units = fits ? tu : 0;
        if (!fits) atomicAdd(S->over_count, 1ull << 40);
    }
}

// A list of one round (small grids): the three steps in block 0, the field masks in the others, in one launch.
// The tiles' first units sit in LDS once the cap is chosen, so the unit records are written by as many
// threads as there are units, each finding its tile by bisection (a thread per tile wrote them one after
// another: 21 us on the 1024^2 disk, now 14, the launch and a chain of loads and scans).
__global__ void __launch_bounds__(kScanThreads) k_compact_one(SimDev* sims, int swap)
{
    __shared__ int wsum[2 * (kScanThreads / 64)];
    __shared__ int s_tile[kCompactK * kScanThreads], s_first[kCompactK * kScanThreads];
    SimDev* S = sims + blockIdx.y;
    const CompactGeom G(S, 1);
    if (G.nt == 0 || G.rounds > 1) return;
    if (blockIdx.x > 0) {
        field_masks(*S, blockIdx.x - 1, gridDim.x - 1);
        return;
    }
    const int tid = threadIdx.x;
    int c[kCompactK], tt[kCompactK];
    int ra = 0, ru = 0;
    G.tiles_of(S, tid * kCompactK, tt);
#pragma unroll
    for (int j = 0; j < kCompactK; ++j) {
        c[j] = tt[j] >= 0 ? compact_count(S, tt[j]) : 0;
        ra += c[j] > 0 ? 1 : 0;
    }
    int ta, tu;
    int pa = block_scan(ra, wsum, &ta) - ra;
    const long long npart = compact_total(S);
    int cap = compact_cap(S, npart, ta);
    if (S->unit_cap == 0 && ta > 0 && ta < S->unit_goal) {
        // the bound behind the chosen cap counts a part unit for every tile; the tiles are at hand here, so
        // the smallest cap (in chunks) that keeps to the goal is searched for between N / goal and it
        // (a barrier per try: the wavefronts' counts alternate between two rows)
        int lo = max(unit_floor(npart), (int)min((npart / S->unit_goal + 64) / 64 * 64, (long long)cap));
        int row = 0;
        while (lo < cap) {
            const int mid = (lo + (cap - lo) / 2) / 64 * 64;
            int u = 0;
            if (__any(ra > 0)) {
#pragma unroll
                for (int j = 0; j < kCompactK; ++j) u += compact_units(c[j], mid);
                u = seg_scan<int>(u, scan_masks(tid & 63));
            }
            if ((tid & 63) == 63) wsum[row * (kScanThreads / 64) + (tid >> 6)] = u;
            __syncthreads();
            int tot = 0;
#pragma unroll
            for (int w = 0; w < kScanThreads / 64; ++w) tot += wsum[row * (kScanThreads / 64) + w];
            if (tot <= S->unit_goal) cap = mid;
            else lo = mid + 64;
            row ^= 1;
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < kCompactK; ++j) ru += compact_units(c[j], cap);
    int pu = block_scan(ru, wsum, &tu) - ru;
    const bool fits = ta <= S->max_slots && tu <= S->max_units;
    if (tid == 0) {
        *S->n_active = fits ? ta : 0;
        *S->n_units = fits ? tu : 0;
        S->unit_now = cap;
        if (!fits) atomicAdd(S->over_count, 1ull << 40);
        swap_sorted(S, swap);
    }
    if (!fits) return;
#pragma unroll
    for (int j = 0; j < kCompactK; ++j)
        if (c[j] > 0) {
            s_tile[pa] = tt[j];
            s_first[pa] = pu;
            ++pa;
            pu += compact_units(c[j], cap);
        }
    __syncthreads();
    for (int u = tid; u < tu; u += kScanThreads) {
        int lo = 0, hi = ta;  // the last tile whose first unit is at or before u
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_first[mid] <= u) lo = mid; else hi = mid;
        }
        const int f = s_first[lo], k = (lo + 1 < ta ? s_first[lo + 1] : tu) - f;
        put_unit(S, S->units[u], u - f, k, s_tile[lo], cap);
    }
}

__global__ void __launch_bounds__(kScanThreads) k_compact_place(SimDev* sims, int swap)
{
    __shared__ int wsum[kScanThreads / 64];
    SimDev* S = sims + blockIdx.y;
    const CompactGeom G(S, gridDim.x);
    if (G.rounds <= 1) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) swap_sorted(S, swap);
    const int cap = S->unit_now;
    if (S->compact_part[kCompactPart - 1] == 0) return;  // the list does not fit
    int ou = S->compact_part[2 * blockIdx.x + 1];        // the blocks before
    const int r0 = blockIdx.x * G.rpb, r1 = min(G.rounds, r0 + G.rpb);
    for (int round = r0; round < r1; ++round) {
        int k[kCompactK], tt[kCompactK];
        int ru = 0;
        G.tiles_of(S, round * kCompactK * kScanThreads + threadIdx.x * kCompactK, tt);
#pragma unroll
        for (int j = 0; j < kCompactK; ++j) ru += k[j] = tt[j] >= 0 ? compact_units(compact_count(S, tt[j]), cap) : 0;
        int su;
        int pu = block_scan(ru, wsum, &su) - ru + ou;
#pragma unroll
        for (int j = 0; j < kCompactK; ++j)
            for (int q = 0; q < k[j]; ++q) put_unit(S, S->units[pu++], q, k[j], tt[j], cap);
        ou += su;
    }
}

// --------------------------------------------------------------------------------------------
hipError_t enqueue_sort(SimDev* sims, int slots, int s, bool moving, const SortShape& q, hipStream_t st)
{
    const SortSel sel{s, moving ? 1 : 0};
    const auto grid = [&](long long blocks) { return dim3((unsigned)std::max(1LL, blocks), slots); };
    // a table's launches take the blocks of its slots in turns: 512 keep every CU busy
    const int nb = slots > 1 ? std::min(q.blocks, 512) : q.blocks;
    const int rows = ((1 << q.bits) + kScanDigits - 1) / kScanDigits;
    if (q.n > 0)
        for (int p = 0; p < q.passes; ++p) {
            if (p == 0) hipLaunchKernelGGL(k_radix_hist<true>, grid(nb), dim3(kSortBlock), 0, st, sims, sel, p);
            else hipLaunchKernelGGL(k_radix_hist<false>, grid(nb), dim3(kSortBlock), 0, st, sims, sel, p);
            if (q.blocks > kFuseBlocks)
                hipLaunchKernelGGL(k_radix_rowsum, grid(rows * kPartCopies), dim3(kScanThreads), 0, st, sims, sel, p);
            // (a table takes both, each for its members: in fours for all of them cost 16 requests 94 us a sort)
            if (q.blocks > kDirectBlocks && (moving || q.blocks <= kScanBlocks))
                hipLaunchKernelGGL(k_radix_rowscan<16>, grid(rows), dim3(kScanThreads), 0, st, sims, sel, p);
            if (q.blocks > kScanBlocks)
                hipLaunchKernelGGL(k_radix_rowscan<4>, grid(moving ? rows : 4 * rows), dim3(kScanThreads), 0, st, sims, sel, p);
            if (!moving && q.n > 4 * kSortBlock * 512 && q.bits <= kDigitBits - 2)
                hipLaunchKernelGGL(k_radix_scatter<4>, grid(nb), dim3(kSortBlock), 0, st, sims, sel, p);
            else if (!moving && q.n > 2 * kSortBlock * 512 && q.bits <= kDigitBits - 1)
                hipLaunchKernelGGL(k_radix_scatter<2>, grid(nb), dim3(kSortBlock), 0, st, sims, sel, p);
            else
                hipLaunchKernelGGL(k_radix_scatter<1>, grid(nb), dim3(kSortBlock), 0, st, sims, sel, p);
        }
    const int np = (int)std::min<long long>(((long long)q.n + 255) / 256, slots > 1 ? 1024 : 4096);
    const int nr = std::min((q.ntiles + 1 + 255) / 256, slots > 1 ? 256 : 4096);
    hipLaunchKernelGGL(k_permute, grid(np + nr), dim3(256), 0, st, sims, sel, q.elem, nr);
    return hipGetLastError();
}

hipError_t enqueue_keys_only(SimDev* dS, int s, int n, hipStream_t st)
{
    const int g = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
    hipLaunchKernelGGL(k_keys, dim3(g > 0 ? g : 1), dim3(256), 0, st, dS, s);
    return hipGetLastError();
}

// the rounds of a grid's list (its padded ranks, as CompactGeom counts them)
static long long compact_rounds(const SimDev& h)
{
    long long nt = 1;
    for (int a = 0; a < 3; ++a) {
        const int b = a < h.dims ? kUnitBlock : 1;
        nt *= (long long)((h.ntile[a] + b - 1) / b) * b;
    }
    return (nt + kCompactK * kScanThreads - 1) / (kCompactK * kScanThreads);
}

void CompactShape::cover(const SimDev& h)
{
    const long long r = compact_rounds(h);
    if (r <= 1) one = true;
    else {
        blocks = std::max(blocks, (int)std::min<long long>(r, kCompactBlocks));
        // (a round per block within the scratch of the smallest sort, 256 counts; four blocks took 20 us over
        // the 65536 tiles of the 256^3 sphere, 64 take 5)
        if (h.unit_cap == 0) active = std::max(active, std::min(256, (h.ntiles + kScanThreads - 1) / kScanThreads));
    }
    masks = std::max(masks, (h.nftiles + kScanThreads / 64 - 1) / (kScanThreads / 64));
}

hipError_t enqueue_compact(SimDev* sims, int slots, const CompactShape& q, int swap, hipStream_t st)
{
    const int nm = slots > 1 ? std::min(q.masks, 256) : q.masks;
    if (q.one) hipLaunchKernelGGL(k_compact_one, dim3(1 + nm, slots), dim3(kScanThreads), 0, st, sims, swap);
    if (q.blocks > 0) {
        if (q.active > 0) hipLaunchKernelGGL(k_compact_active, dim3(q.active, slots), dim3(kScanThreads), 0, st, sims);
        hipLaunchKernelGGL(k_compact_count, dim3(q.blocks + nm, slots), dim3(kScanThreads), 0, st, sims, q.active, q.blocks);
        hipLaunchKernelGGL(k_compact_scan, dim3(1, slots), dim3(kScanThreads), 0, st, sims, q.blocks);
        hipLaunchKernelGGL(k_compact_place, dim3(q.blocks, slots), dim3(kScanThreads), 0, st, sims, swap);
    }
    return hipGetLastError();
}

}  // namespace pic

namespace pic {

// ---- untyped helpers ---------------------------------------------------------------------------
// even words get lo, odd words hi (a 64-bit pattern; lo == hi for a 32-bit one)
__global__ void k_fill(unsigned* __restrict__ p, long long nwords, unsigned lo, unsigned hi)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < nwords; i += (long long)gridDim.x * blockDim.x)
        p[i] = (i & 1) ? hi : lo;
}

hipError_t enqueue_fill_pattern(void* p, size_t bytes, unsigned lo, unsigned hi, hipStream_t st)
{
    const long long nw = (long long)(bytes / 4);
    if (nw <= 0) return hipSuccess;
    long long g = (nw + 255) / 256;
    if (g > 16384) g = 16384;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)g), dim3(256), 0, st, reinterpret_cast<unsigned*>(p), nw, lo, hi);
    return hipGetLastError();
}

hipError_t enqueue_fill(void* p, size_t bytes, hipStream_t st) { return enqueue_fill_pattern(p, bytes, 0u, 0u, st); }

__global__ void __launch_bounds__(256) k_sum(const double* __restrict__ x, long long n, double* part)
{
    __shared__ double sh[256];
    double acc = 0.0;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) acc += x[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

hipError_t enqueue_sum(const double* x, long long n, double* part, int nb, hipStream_t st)
{
    hipLaunchKernelGGL(k_sum, dim3(nb), dim3(256), 0, st, x, n, part);
    return hipGetLastError();
}

// out[v] = reduction over b of part[b * nv + v] (op 0 sum, 1 max), in a fixed order: each thread its
// strided entries, then a tree (one thread in turn took 88 us for 1024 partials, most of a reading of
// an energy)
__global__ void __launch_bounds__(256) k_final(const double* __restrict__ part, int nb, int nv, int op, double* out)
{
    __shared__ double sh[256];
    for (int v = 0; v < nv; ++v) {
        double acc = 0.0;
        for (int b = threadIdx.x; b < nb; b += 256) {
            const double x = part[b * nv + v];
            acc = op ? fmax(acc, x) : acc + x;
        }
        sh[threadIdx.x] = acc;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) {
                const double x = sh[threadIdx.x + w];
                sh[threadIdx.x] = op ? fmax(sh[threadIdx.x], x) : sh[threadIdx.x] + x;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) out[v] = sh[0];
        __syncthreads();
    }
}

hipError_t enqueue_final(const double* part, int nb, int nv, int op, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_final, dim3(1), dim3(256), 0, st, part, nb, nv, op, out);
    return hipGetLastError();
}

// fixed ion background: -rho node by node, or minus the mean of rho (total / number of nodes)
__global__ void k_ion(SimDev* __restrict__ S, const double* __restrict__ rho, int uniform, const double* total)
{
    const double mean = uniform ? *total / (double)S->Lvol : 0.0;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < S->Lvol; q += (long long)gridDim.x * blockDim.x)
        S->rho_ion[q] = uniform ? -mean : -rho[q];
}

hipError_t enqueue_ion(SimDev* dS, const double* rho, int uniform, const double* total, hipStream_t st)
{
    hipLaunchKernelGGL(k_ion, dim3(1024), dim3(256), 0, st, dS, rho, uniform, total);
    return hipGetLastError();
}

// ---- measurement helper: a structure-of-arrays streaming copy of known size ----
struct SoaPtrs {
    const float* src[PIC_MEASURE_MAX_ARRAYS];
    float* dst[PIC_MEASURE_MAX_ARRAYS];
};

__global__ void __launch_bounds__(256) k_measure_soa_copy(SoaPtrs p, int narrays, long long n)
{
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        float v[PIC_MEASURE_MAX_ARRAYS];
#pragma unroll
        for (int k = 0; k < PIC_MEASURE_MAX_ARRAYS; ++k)
            if (k < narrays) v[k] = p.src[k][i];
#pragma unroll
        for (int k = 0; k < PIC_MEASURE_MAX_ARRAYS; ++k)
            if (k < narrays) p.dst[k][i] = v[k];
    }
}

}  // namespace pic

extern "C" int pic_measure_soa_copy(const float* const* src, float* const* dst, int narrays, long long n,
                                    void* hip_stream)
{
    if (!src || !dst || narrays < 1 || narrays > PIC_MEASURE_MAX_ARRAYS || n < 0) return PIC_EINVAL;
    pic::SoaPtrs p{};
    for (int k = 0; k < narrays; ++k) {
        if (!src[k] || !dst[k]) return PIC_EINVAL;
        p.src[k] = src[k];
        p.dst[k] = dst[k];
    }
    if (n == 0) return PIC_OK;
    const long long blocks = (n + 255) / 256;
    const int grid = (int)(blocks < 8192 ? blocks : 8192);
    hipLaunchKernelGGL(pic::k_measure_soa_copy, dim3(grid), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream),
                       p, narrays, n);
    return hipGetLastError() == hipSuccess ? PIC_OK : PIC_EDEVICE;
}
