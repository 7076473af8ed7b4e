// The passes of an array-valued reduce.  Host logic without HIP.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "sparkcl_dev.h"

namespace sparkcl {

constexpr uint32_t kTreeMaxChunk = 4096; // leaves per chunk the kernel's counter holds
constexpr uint32_t kTreeMaxChunks = 65535;

// One pass: `count` leaves folded in chunks of `chunk` (a power of two unless
// it is the only chunk) into `rows` rows; the other fields as in TreeArgs.
struct TreePass {
    uint32_t count = 0, chunk = 0, rows = 0;
    uint32_t cpt = 1, threads = kBlock, groups = 0, cols = 0;
};

inline uint32_t pow2_floor(uint64_t v)
{
    uint32_t p = 1;
    while ((uint64_t)p * 2 <= v && p < (1u << 31))
        p *= 2;
    return p;
}

// Whole columns of `count` leaves: one pass when the columns alone fill the
// GPU (then long per-thread chains are hidden by other waves) or the chain is
// short; else chunks so that the grid of columns x chunks fills it.
// Everything has float4 columns from 4 floats on (the last one may overlap
// the one before): leaves and out need only their 4-byte alignment (a 16-byte
// access at a 4-byte-aligned address is one dwordx4 instruction).  48 arrays
// of 1000003 floats took 39.7 us in single columns.  `least`: as few rows as
// the kernel can leave, whatever time that takes.
inline TreePass tree_columns(uint32_t count, uint64_t len, uint32_t cus, bool least)
{
    TreePass a;
    a.count = count;
    const uint64_t ncol = (len + 3) / 4;
    const uint64_t colblocks = (ncol + kBlock - 1) / kBlock;
    const uint64_t target = 4ull * cus; // blocks that fill the GPU
    // the wide kernel (leaf pairs, 2 or 4 columns per thread, chunks of up to
    // 64 leaves) when its grid still fills half the GPU's block slots and at
    // most one more pass follows (many short columns fold better in the deeper
    // chunks of the 8-leaf kernel: 65536 rows of 4096 floats took 189 us
    // through 64-leaf chunks and four passes, 181 us in three); the most
    // columns per thread first, in blocks of kTreeWideBig threads when those
    // alone give every CU two blocks (64 arrays of 2^22 floats: 163 us against
    // 170 us in 256-thread blocks)
    const uint32_t ch = std::min<uint32_t>(count, kTreeWideChunk);
    const uint64_t nch = (count + (uint64_t)ch - 1) / ch;
    if (!least && nch <= kTreeWideChunk) {
        const uint64_t cb_big = (ncol + kTreeWideBig * 4ull - 1) / (kTreeWideBig * 4ull);
        if (cb_big * nch >= 2ull * cus) {
            a.cpt = 4;
            a.threads = kTreeWideBig;
        }
        for (uint32_t c : {4u, 2u}) {
            if (a.cpt > 1)
                break;
            const uint64_t cb = (ncol + (uint64_t)kBlock * c - 1) / ((uint64_t)kBlock * c);
            if (cb * nch >= target / 2)
                a.cpt = c;
        }
    }
    if (a.cpt > 1) {
        a.chunk = ch;
    } else if (count <= kTreeMaxChunk && (least || colblocks >= target || count <= 64)) {
        a.chunk = count; // final pass
    } else {
        a.chunk = least ? kTreeMaxChunk
                        : pow2_floor(std::max<uint64_t>(1, (uint64_t)count * colblocks / target));
        a.chunk = std::min(std::max(a.chunk, 8u), kTreeMaxChunk);
        while ((count + (uint64_t)a.chunk - 1) / a.chunk > kTreeMaxChunks)
            a.chunk *= 2;
        if (a.chunk >= count)
            a.chunk = count;
    }
    a.rows = (uint32_t)((count + (uint64_t)a.chunk - 1) / a.chunk);
    return a;
}

// Short arrays: as many groups of threads as a block holds, each folding
// leaves of its own.  Rows past 1 KiB (64 quads) are cut into column tiles of
// about that while the input fits the memory-side cache, which spreads a pass
// over more blocks (8000 rows of 1024 floats: 12 us, whole rows 17; 65536 rows
// of 1000: 50 and 56).  A pass that one block per tile can read as 128 KiB at
// most is the last; one before it takes 8 to 64 leaves per thread, as many as
// still leave two blocks per CU (2^20 rows of 64: 49 us, with four blocks 57).
inline TreePass tree_groups(uint32_t count, uint64_t len, uint32_t cus)
{
    TreePass a;
    a.count = count;
    const uint64_t ncol = len < 4 ? len : (len + 3) / 4;
    const uint64_t most = (uint64_t)count * len * 4 <= kTreeCached ? 64 : kTreeFlatThreads;
    const uint64_t tiles = (ncol + most - 1) / most;
    a.cols = (uint32_t)((ncol + tiles - 1) / tiles);
    a.groups = pow2_floor(kTreeFlatThreads / a.cols);
    a.threads = (a.cols * a.groups + 63) / 64 * 64;
    uint32_t per;
    if ((uint64_t)count * a.cols * 16 <= (128u << 10)) {
        per = pow2_floor(2ull * ((count + a.groups - 1) / a.groups) - 1);
    } else {
        const uint64_t fill = 2ull * cus * a.groups;
        per = pow2_floor(std::max<uint64_t>(1, count * tiles / fill));
        per = std::min(std::max(per, 8u), kTreeFlatPer);
    }
    a.chunk = per * a.groups;
    a.rows = (uint32_t)(((uint64_t)count + a.chunk - 1) / a.chunk);
    return a;
}

inline TreePass tree_pass(uint32_t count, uint64_t len, uint32_t cus, bool least)
{
    const uint64_t ncol = len < 4 ? len : (len + 3) / 4;
    if (len < 4)
        return tree_groups(count, len, cus); // the only kernel of such arrays
    const TreePass columns = tree_columns(count, len, cus, least);
    if (least || ncol > kTreeFlatThreads)
        return columns;
    // A group folds 64 leaves at most, a column 4096: where a block holds one
    // or two groups the rows grow with the input, and with them the scratch
    // (2^20 rows of 4096 floats: 256 MiB, in columns 4) and the next passes
    // (65536 rows of 4096: 200 us, in columns 189).
    const TreePass groups = tree_groups(count, len, cus);
    const uint64_t row = len * sizeof(float);
    return groups.rows * row <= std::max<uint64_t>(columns.rows * row, kTreeScratch) ? groups
                                                                                     : columns;
}

// The passes over k leaves of len floats: each folds the rows that the one
// before left, the last leaves one.
inline std::vector<TreePass> tree_passes(uint32_t k, uint64_t len, uint32_t cus, bool least)
{
    std::vector<TreePass> p;
    for (uint32_t count = k;; count = p.back().rows) {
        p.push_back(tree_pass(count, len, cus, least));
        if (p.back().rows == 1)
            return p;
    }
}

} // namespace sparkcl
