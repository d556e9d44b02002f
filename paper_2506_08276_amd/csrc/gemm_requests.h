// Where gemm_large_kernel's wavefronts request W.  Plain code without HIP types, for the host as for the device.
#pragma once
#include <stdint.h>

// A slab (32 elements of K) of 32 columns of W as a buffer.  W lies in rows of K or in operand order (packed), where the 64 bytes of K elements of 32 columns
// are together and so is a slab of them.  Columns beyond N, which the last column tile may reach, are a buffer of no bytes: a buffer's
// bounds are checked against the lane's offset (a scalar offset beyond the end need not be found), so a request has no other.
struct WeightSlab {
    int64_t first;  // element
    int bytes;
};

constexpr WeightSlab weight_slab(int first_col, int slab, int N, int K, int packed)
{
    return {(int64_t)first_col * K + slab * (packed ? 1024 : 32), first_col >= N ? 0 : packed ? 2048 : 62 * K + 64};
}

// A lane's offset in it: `part` 0 or 1, 16 elements of K in operand order, else 16 columns, whose 16-byte chunks are permuted so that chunk c of row r lands at
// c ^ ((r >> 2) & 3).
constexpr int weight_offset(int lane, int part, int K, int packed)
{
    return packed ? part * 1024 + lane * 16 : part * 32 * K + (lane >> 2) * 2 * K + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
}
