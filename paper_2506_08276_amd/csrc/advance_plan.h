// LDS of a block of advance_kernel (search.hip), in bytes.  Host code without HIP types.
#pragma once
#include <algorithm>

constexpr int CU_LDS = 160 * 1024;
constexpr int ADV_FIXED = 6 * 1024;  // room for the kernel's fixed arrays; search_init_device compares
constexpr int ADV_DYNAMIC_MAX = CU_LDS - ADV_FIXED;
constexpr int LDS_GRAIN = 1280;   // LDS is handed out in pieces of
constexpr int AQ_NEAR_MAX = 64;   // rows of AQ's 64 columns in LDS

constexpr int ADV_BLOCKS = 3;     // blocks that the kernel's registers (130 to 167) let share a CU
constexpr int ADV_MORE_BLOCKS = 4;  // as compiled for 128 registers, which rows of up to 6 pieces of 4 bytes per lane get by with

struct AdvancePlan {
    int blocks;  // that share a CU; ADV_MORE_BLOCKS: the kernel compiled for it is meant
    int near;    // rows of AQ's columns that a running block keeps in LDS
    int bytes;   // dynamic LDS: lookup table, EQ (keys, CSR rows, marks in steps of 256), near rows at an odd pitch
};

// A block per query: a CU shall hold as many at once as there are queries for it, as far as registers, table and EQ let it.  What a
// block's share of the LDS has left is the head of AQ.  A query waits for latencies nearly all the time, so another one on the
// CU gains more than it costs to keep rows of AQ in memory (without any in LDS a query takes 5 % longer) or, with ADV_MORE_BLOCKS, to
// get by with fewer registers (8 %).  4000 queries, all embeddings stored, ef 200, d = 384, N = 12288: 11.4 -> 6.6 ms with 64 subspaces
// (one block a CU -> two), 5.7 -> 4.2 with 32 (two -> three), 5.6 -> 3.4 with 16 (two -> four); 500 queries with 64 subspaces 2.0 -> 1.3.
// Where hardly more queries are there than one block fewer would hold, the longest query counts instead (770 at ef 200, d = 384, 16
// subspaces: three blocks 1.11 ms, four 1.20; 832 1.29, 1.19; 1100 1.65, 1.40; at ef 64 832 0.63, 0.64 and 960 0.69, 0.64; at ef 500
// 960 2.57, 2.86 and 1100 3.10, 2.92), so a sixteenth of a query per CU has to be over, a quarter with ADV_MORE_BLOCKS.
// Not looked at: what the queue will need.  535 to 850 queries at ef 500 with 32 subspaces take 6 % longer with three blocks than with two.
// pieces: of 4 bytes per lane of an embedding row.  bytes > ADV_DYNAMIC_MAX: does not fit.
inline AdvancePlan plan_advance(int m_sub, int ef, int queries, int cus, int pieces)
{
    const int fixed = m_sub * 256 * 4 + ef * 16 + (ef + 255) / 256 * 256;
    auto bytes = [&](int near) { return fixed + 64 * 8 * (near | 1); };
    auto share = [](int blocks) { return CU_LDS / blocks / LDS_GRAIN * LDS_GRAIN - ADV_FIXED; };
    const int most = pieces <= 6 ? ADV_MORE_BLOCKS : ADV_BLOCKS;
    int blocks = 1;
    while (blocks < most && bytes(0) <= share(blocks + 1) && queries > blocks * cus + cus / (blocks + 1 == ADV_MORE_BLOCKS ? 4 : 16)) ++blocks;
    const int near = std::min(AQ_NEAR_MAX, std::max(0, (share(blocks) - fixed) / (64 * 8) - 1));  // - 1: the pitch is odd
    return {blocks, near, bytes(near)};
}
