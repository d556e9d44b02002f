// LDS of a block of advance_kernel (search.hip), in bytes.  Host code without HIP types.
#pragma once
#include <algorithm>

constexpr int CU_LDS = 160 * 1024;
constexpr int ADV_FIXED = 6 * 1024;  // room for the kernel's fixed arrays; search_init_device compares
constexpr int ADV_DYNAMIC_MAX = CU_LDS - ADV_FIXED;
constexpr int ADV_DYNAMIC_SHARED = 74 * 1024;      // with two blocks on a CU
constexpr int AQ_NEAR_MIN = 32, AQ_NEAR_MAX = 64;  // rows of AQ's 64 columns in LDS

struct AdvancePlan {
    int near;   // rows of AQ's columns that a running block keeps in LDS
    int bytes;  // dynamic LDS: lookup table, EQ (keys, CSR rows, marks in steps of 256), near rows at an odd pitch
};

// What table and queue leave holds the head of AQ: as much as lets two blocks share a CU, but no less than AQ_NEAR_MIN rows if there
// is room.  bytes > ADV_DYNAMIC_MAX: does not fit.
inline AdvancePlan plan_advance(int m_sub, int ef)
{
    const int fixed = m_sub * 256 * 4 + ef * 16 + (ef + 255) / 256 * 256;
    auto rows_in = [&](int limit) { return std::max(0, (limit - fixed) / (64 * 8) - 1); };  // - 1: the pitch is odd
    const int near = std::min(std::max(std::min(AQ_NEAR_MIN, rows_in(ADV_DYNAMIC_MAX)), rows_in(ADV_DYNAMIC_SHARED)), AQ_NEAR_MAX);
    return {near, fixed + 64 * (near | 1) * 8};
}
