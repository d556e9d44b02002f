// bf16 MFMA products of large passes: 256 rows per tile, two groups of wavefronts that take turns (gfx950).
#pragma once
#include "common.h"
#include "gemm.h"
#include "gemm_requests.h"

namespace {

typedef __attribute__((address_space(3))) void lds_t;

// A tile of the kernel below: WM x (8 / WM) wavefronts of TM x TN 32x32 MFMA tiles.
template <int WM, int TM, int TN>
struct LargeCfg {
    static constexpr int WN = 8 / WM, BM = WM * TM * 32, BN = WN * TN * 32;
    static constexpr int A_BYTES = BM * GEMM_BK * 2, STAGE = (BM + BN) * GEMM_BK * 2;
    static constexpr int SMEM = 4 * STAGE + 8 * 2048;  // four stages; per wavefront the bias of its columns, then 32 x 32 outputs on their way
    static constexpr int LOADS = 2 + (BN == 256 ? 2 : 1);  // requests of 1 KB per wavefront and slab, at least
    static constexpr int STORES = 2 * TN;                  // per 32 rows of outputs
    // Memory requests of a wavefront that may still be on their way when slab s + 1 has to be there: those of slabs s + 2 and s + 3, and
    // the stores that were issued since.  Requests complete in order.
    static constexpr int in_flight(int s)
    {
        int batches = 0;
        for (int t = s - 2; t <= s; ++t) batches += t >= 0 && t < TM;
        return 2 * LOADS + batches * STORES;
    }
};

template <int VM>
__device__ inline void wait_memory_and_lds()  // VM requests may be on their way, no LDS access
{
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x70);
}

// Nothing is moved across, neither by the compiler's passes nor by its scheduler.
__device__ inline void fence()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ inline void barrier()
{
    fence();
    __builtin_amdgcn_s_barrier();
    fence();
}

// The product of gemm_kernel (same MFMAs, same order over K, sums that start at the bias: the same bits).
// What bounds it at K = 3072 is the matrix cores at the clock that they leave (busy 80 % of the cycles at 1.72 GHz); at K = 768 (46 to 54 % at 2.0) what a tile
// costs besides its slabs: by the two, a slab takes some 1060 cycles, 1024 of them MFMA, and a tile 19 000 more.  Next to that, how a slab's operands
// get from L2 to LDS: 32 KB per 1024 MFMA clocks of a CU.
//  - Operands go from memory to LDS without registers, 1 KB per request and every request whole lines: A lies in planes of the slab's 32
//    columns (see gemm.h), W in the MFMA's operand order (or, where a context has no memory for that copy, in rows, whose pieces are fetched to
//    where operand order has them).  In rows of K, a request's 64-byte pieces kept L2 busy for twice the time: without its requests
//    the loop was a third faster, with requests that wait half as long for their slab it was no slower.
//  - Four stages: a slab is requested three slabs ahead.
//  - Wavefronts 0..3 and 4..7, one of each on a SIMD, take turns: while one group multiplies a slab, the other reads the next one's
//    operands from LDS and requests a slab; barriers hand over.  In the memory phase of slab s, stage (s + 3) % 4 is requested, which
//    held slab s - 1: both groups have read it, each before the barrier that ended its memory phase of s - 1.  A group waits at the end of
//    its memory phase of slab s until what it has requested of slab s + 1 is there; the other group's next barrier then makes
//    slab s + 1 whole for either's memory phase.
//  - A finished tile is rounded into registers (64 at 256 x 256) and written out in the next tile's first memory phases, 32 rows in each,
//    so that no group waits for stores.  Of the epilogue only GELU and the rounding are left on the chain.  Every wavefront issues every
//    store (beyond N, or before the first tile, with an offset behind the buffer's end), as waits count them.
// Per launch, a 256 x 256 tile of gemm_kernel's way (operands through registers, rows of K elements) and this one, microseconds, TFLOP/s now:
//     N x K          T = 131072             T = 327680
//   2304 x  768       431    381   1216      1132    991   1170
//    768 x  768       144    122   1265       402    360   1073
//   3072 x  768 GELU  629    592   1045      1626   1531   1010
//    768 x 3072       548    466   1326      1417   1206   1282
// Two independent blocks of 128 x 256 per CU, so that one's GELU runs beside the other's MFMAs, need 1.5 times the operands: 426, 143, 627, 540
// at T = 131072.  Output planes of 64 columns, written in half lines, cost 2304 x 768 a quarter at T = 327680.
// 256 x 192 (WM 4, TM 2, TN 3) is for what 256 columns leave of the chip or of N: see gemm_plan.h.
template <int WM, int TM, int TN, int EPI>
__global__ __launch_bounds__(512, 1) void gemm_large_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W,
                                                            const float *__restrict__ bias, bf16_t *__restrict__ out,
                                                            const int32_t *__restrict__ T_dev, int N, int K, int tiles_n, int gcols, int plane,
                                                            int w_packed)
{
    typedef LargeCfg<WM, TM, TN> Cfg;
    constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = GEMM_BK;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [4][A, W], [8][2 KB]
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    const bool second = wave >= 4;  // the group that multiplies in the other's memory phases

    // Persistent blocks, as in gemm_kernel.
    const int T = *T_dev;
    const int n_tiles = ((T + BM - 1) / BM) * tiles_n, tiles_m = n_tiles / tiles_n;
    const int per_xcd = (n_tiles + 7) >> 3, blocks_per_xcd = gridDim.x >> 3;
    auto tile_at = [&](int step, int &tm, int &tn) -> bool {
        const int in_xcd = step * blocks_per_xcd + (int)(blockIdx.x >> 3);
        const int logical = (int)(blockIdx.x & 7) * per_xcd + in_xcd;
        if (in_xcd >= per_xcd || logical >= n_tiles) return false;
        const int g = logical / (tiles_m * gcols), r = logical - g * tiles_m * gcols, cg = min(gcols, tiles_n - g * gcols);
        tm = r / cg;
        tn = g * gcols + r % cg;
        return true;
    };
    int tile_m = 0, tile_n = 0;
    if (!tile_at(0, tile_m, tile_n)) return;
    const int KT = K / BK;  // a multiple of 4, at least 8: the host checks

    // Requests.  A: two of 16 rows per wavefront, the lanes' 16-byte chunks permuted so that chunk c of row r lands at c ^ ((r >> 2) & 3): 16 rows'
    // reads of one chunk reach all banks.  W: two for every 32 columns, 16 elements of K each, operand order in LDS too; from rows, 16
    // columns each, as A's.  The last column tile may reach past N: zeros.
    const int a_off = weight_offset(lane, 0, BK, 0);  // a plane's rows are 32 elements long
    const int w_ct = BN == 256 || !second ? wave : 4 + ((wave - 4) >> 1), w_i = BN == 256 || !second ? 0 : wave & 1;  // 192 columns: the second group has one request
    const int w_off[2] = {weight_offset(lane, w_i, K, w_packed), weight_offset(lane, 1, K, w_packed)};
    auto a_tile = [&](int tm) { return A + (size_t)tm * BM * PLANE; };
    auto request = [&](const bf16_t *a, int tn, int slab, int stage) {
        const auto ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a + (size_t)slab * plane), 0, BM * BK * 2, 0x00020000);
        const WeightSlab ws = weight_slab(tn * BN + w_ct * 32, slab, N, K, w_packed);
        const auto wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(W + ws.first), 0, ws.bytes, 0x00020000);
        unsigned char *to = smem + stage * Cfg::STAGE;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ar, (lds_t *)(to + wave * 2048 + i * 1024), 16, a_off, wave * 2048 + i * 1024, 0, 0);
            if (i == 0 || BN == 256 || !second)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_t *)(to + Cfg::A_BYTES + w_ct * 2048 + (w_i + i) * 1024), 16, w_off[i], 0, 0, 0);
        }
    };
    unsigned char *own = smem + 4 * Cfg::STAGE + wave * 2048;
    const auto bias_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(bias), 0, N * 4, 0x00020000);
    auto request_bias = [&](int tn) {
#pragma unroll
        for (int i = 0; i < TN * 32; i += 64)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(bias_rsrc, (lds_t *)(own + i * 4), 4, (tn * BN + wn * TN * 32 + i + lane) * 4, 0, 0, 0);
    };

    int foff[2], wfoff[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        foff[ks] = l32 * 64 + (((ks * 2 + half) ^ ((lane >> 2) & 3)) << 4);
        wfoff[ks] = w_packed ? ks * 1024 + lane * 16 : foff[ks];
    }
    bf16x8 af[2][TM], bf[2][TN];
    f32x16 acc[TM][TN];
    auto read = [&](int stage) {
        const unsigned char *at = smem + stage * Cfg::STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
                bf[ks][ni] = *reinterpret_cast<const bf16x8 *>(at + Cfg::A_BYTES + (wn * TN + ni) * 2048 + wfoff[ks]);
#pragma unroll
            for (int mi = 0; mi < TM; ++mi) af[ks][mi] = *reinterpret_cast<const bf16x8 *>(at + (wm * TM + mi) * 2048 + foff[ks]);
        }
    };
    auto multiply = [&](int ks) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[ks][ni], af[ks][mi], acc[mi][ni], 0, 0, 0);
    };
    auto compute_phase = [&] {
        barrier();
        __builtin_amdgcn_s_setprio(1);
        multiply(0);
        multiply(1);
        __builtin_amdgcn_s_setprio(0);
        barrier();
    };

    // The tile before, rounded: a lane owns row l32 of 32 and, per g, the columns 8g + 4 half + 0..3 of 32.  32 x 32 outputs at a time go through the
    // wavefront's own 2 KB (16-byte chunk c of a row at c ^ ((row >> 2) & 3)) to stores of 16 bytes per lane, a plane's rows in a run.
    bf16x4 done[TM][TN][4];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int g = 0; g < 4; ++g) done[mi][ni][g] = bf16x4{};
    constexpr int NOWHERE = 0x7ff00000;
    int done_m = 0, done_col = N;  // rows and columns that it has; none before the first one
    auto write_out = [&](int mi) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            const int col = min(done_col + ni * 32, N - 32), o = done_col + ni * 32 < N ? lane * 16 : NOWHERE;
            const auto to = __builtin_amdgcn_make_buffer_rsrc(out + plane_at(col, done_m + mi * 32, plane), 0, 2048, 0x00020000);
#pragma unroll
            for (int g = 0; g < 4; ++g) *reinterpret_cast<bf16x4 *>(own + l32 * 64 + ((g ^ ((l32 >> 2) & 3)) << 4) + half * 8) = done[mi][ni][g];
            __builtin_amdgcn_wave_barrier();  // LDS serves a wavefront's accesses in order
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(own + j * 1024 + (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4));
                __builtin_amdgcn_raw_buffer_store_b128(v, to, o, j * 1024, 2);  // streaming: a later kernel reads it
            }
            __builtin_amdgcn_wave_barrier();
        }
    };

    const bf16_t *a = a_tile(tile_m);
    request_bias(tile_n);
    request(a, tile_n, 0, 0);
    request(a, tile_n, 1, 1);
    request(a, tile_n, 2, 2);
    wait_memory_and_lds<2 * Cfg::LOADS>();
    barrier();
    if (second) barrier();  // a phase behind
    for (int step = 0;; ++step) {
        // without a tile after this one its first slabs are requested again (in bounds, unused)
        int next_m = tile_m, next_n = tile_n;
        const bool have_next = tile_at(step + 1, next_m, next_n);
        const bf16_t *a_next = a_tile(next_m);
        {  // slab 0: the sums start at the bias
            f32x16 start[TN];
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 b = *reinterpret_cast<const f32x4 *>(own + (ni * 32 + 8 * g + 4 * half) * 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) start[ni][4 * g + i] = b[i];
                }
            read(0);
            request(a, tile_n, 3, 3);
            write_out(0);
            wait_memory_and_lds<Cfg::in_flight(0)>();
            barrier();
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
#pragma unroll
                for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[0][ni], af[0][mi], start[ni], 0, 0, 0);
            multiply(1);
            __builtin_amdgcn_s_setprio(0);
            barrier();
        }
        read(1);
        request(a, tile_n, 4, 0);
        write_out(1);
        wait_memory_and_lds<Cfg::in_flight(1)>();
        compute_phase();
        read(2);
        request(a, tile_n, 5, 1);
        if constexpr (TM > 2) write_out(2);
        wait_memory_and_lds<Cfg::in_flight(2)>();
        compute_phase();
        read(3);
        request(a, tile_n, 6, 2);
        if constexpr (TM > 2) write_out(3);
        wait_memory_and_lds<Cfg::in_flight(3)>();
        compute_phase();
        for (int s = 4; s < KT - 4; s += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                read(u);
                request(a, tile_n, s + u + 3, (u + 3) & 3);
                wait_memory_and_lds<2 * Cfg::LOADS>();
                compute_phase();
            }
        }
        request_bias(next_n);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            read(u);
            if (u == 0) request(a, tile_n, KT - 1, 3);
            else request(a_next, next_n, u - 1, u - 1);
            wait_memory_and_lds<2 * Cfg::LOADS>();
            compute_phase();
        }
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float v = acc[mi][ni][4 * g + i];
                        done[mi][ni][g][i] = (bf16_t)(EPI == EPI_BIAS_GELU ? gelu_erf(v) : v);
                    }
        done_m = tile_m * BM + wm * TM * 32;
        done_col = tile_n * BN + wn * TN * 32;
        if (!have_next) break;
        tile_m = next_m;
        tile_n = next_n;
        a = a_next;
    }
    if (!second) barrier();
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) write_out(mi);
    wait_memory_and_lds<0>();  // nothing is on its way to LDS when the block's space becomes another's
}

}  // namespace
