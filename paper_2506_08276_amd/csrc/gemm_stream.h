// bf16 MFMA products of passes that fill the chip once: W from memory to registers, A through LDS (gfx950).
#pragma once
#include "common.h"
#include "gemm.h"

namespace {

// W[N][K] in the order in which the MFMA reads it: 32 rows by 16 elements are 1 KB, lane l's 16 bytes (row l % 32, elements
// 8 (l / 32) ..) at l; then the next 16 elements along K, then the next 32 rows.  One thread per 16 bytes, once per context.
__global__ __launch_bounds__(256) void pack_weights_kernel(const bf16_t *__restrict__ W, int N, int K, bf16_t *__restrict__ packed)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)N * K / 8) return;
    const int lane = (int)(i & 63);
    const int64_t frag = i >> 6;
    const int ks = (int)(frag % (K / 16)), ct = (int)(frag / (K / 16));
    reinterpret_cast<u32x4 *>(packed)[i] =
        *reinterpret_cast<const u32x4 *>(W + (size_t)(ct * 32 + (lane & 31)) * K + ks * 16 + (lane >> 5) * 8);
}

// The product of gemm_kernel (same MFMAs, same order over K, sums that start at the bias: the same bits) for passes in which
// every CU gets one tile at most.  Latency bounds it: a launch is some 2.3 us, the first operands come from beyond L2, and no other
// tile's work hides a wait.  What counts then is how many bytes a CU has on their way and that nothing on the chain over K waits for LDS:
//  - W is kept a second time in operand order, so a multiplying wavefront reads its own 32 columns straight into registers, DW
//    steps of 16 elements ahead, 1 KB per request.  W takes no LDS space, stores or reads, and no barrier.
//  - A goes through LDS: four wavefronts fetch K-slabs of 128 (whole lines: rows are adjacent in their planes), three slabs ahead in registers, into
//    a ring of three stages (with six ahead, the first one waits longer: 0.1 to 0.4 us per launch up to 64 x 128).  A multiplying
//    wavefront has 32 R rows by 32 columns of the tile and reads A up to AHEAD steps ahead, across slabs: the slab after the current
//    one is always there already.  One barrier per slab, at which only the fetching wavefronts wait for their LDS stores.  A slab
//    row is 16 chunks of 16 bytes; chunk c of row r sits at c ^ (r & 15): the stores (16 lanes, one row) and the reads (16 lanes, 16
//    rows) both reach all banks.
//  - The first requests go out before the token count is there.
// Three slabs per turn of the loop, with one exit at its end: with more of them, or with a test between the first requests and the
// loop, the compiled code moves requests behind it and waits for all that are in flight (the first build did: 1.3 us more at 80
// rows, 4 us more at K = 3072).  Where K is no multiple of 384, the slabs behind its end are zeros.
// Before, operands of both matrices went through LDS (48 KB of LDS traffic per slab at a 64 x 64 tile, which bounded it) and through
// gemm_kernel<64,64> / <128,128> above 64 x 64; microseconds per launch in a row of dependent launches, W not in L2:
//     rows x N x K     before   now           rows x N x K     before   now
//   450 x 2304 x  768    9.8    5.5         2000 x  768 x 3072   26.2   14.2
//  1040 x 2304 x  768   10.7    7.4         8000 x  768 x 3072   51.2   37.0
//  2000 x 3072 x  768   19.0   13.4
constexpr int STREAM_BK = 128;

// A launch's N, K (multiples of 128) and grid in one word: 14 words of arguments come in registers with the dispatch, and one more, read
// from memory, would be the first link of the chain.  A's offsets have 31 bits.
inline bool stream_covers(int N, int K, int plane) { return N < 128 << 15 && K < 128 << 15 && (int64_t)K / PLANE * plane < (int64_t)1 << 29; }
inline uint32_t stream_shape(int N, int K, int xr) { return (uint32_t)(N / 128) | (uint32_t)(K / 128) << 15 | (uint32_t)__builtin_ctz(xr) << 30; }
__device__ inline int stream_n(uint32_t shape) { return (shape & 0x7fff) * 128; }
__device__ inline int stream_k(uint32_t shape)
{
    int K = (shape >> 15 & 0x7fff) * 128;
    asm("" : "+s"(K));  // any number: of one that it knows the bounds of, the compiler splits the loop over K, whose waits then count fewer requests (5.9 us instead of 5.0 at K = 3072)
    return K;
}

// The four wavefronts that fetch A (thread ft of them) for a tile of 16 RB rows from row m0 on, see gemm_stream_kernel.  A slab is four planes'
// 64 bytes of every row; a request is of four rows in each.
template <int RB, int TURN>
__device__ inline void fetch_a(const bf16_t *A, const int32_t *T_dev, unsigned char *smem, int ft, int m0, int K, int plane, int slabs, int turns_end)
{
    constexpr int ROWS = 16 * RB, STAGE = ROWS * STREAM_BK * (int)sizeof(bf16_t);
    constexpr int LPT = RB;  // 16-byte loads per thread and slab
    const int lrow = ft >> 4, lch = ft & 15;
    const int plane_bytes = plane * (int)sizeof(bf16_t), toff = (lch >> 2) * plane_bytes + lrow * 64 + (lch & 3) * 16;
    const int slab_bytes = 4 * plane_bytes;
    const auto ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(A + (size_t)m0 * PLANE), 0,
                                                      (K / PLANE - 1) * plane_bytes + ROWS * 64, 0x00020000);
    const int soff = lrow * 256 + ((lch ^ lrow) << 4);  // rows 16 apart share the swizzle term
    u32x4 rg[TURN][LPT];
    // Every step issues its loads: a slab past the end gets an offset beyond the buffer (nothing is fetched, zeros
    // come back).  Loads return in order and a wait counts the loads behind the one it is for; where a load may or may
    // not have been issued, the compiler would have to wait for all of them.
#define STREAM_ALOAD(p, slab)                                                                            \
    {                                                                                                    \
        const int o_ = (slab) < slabs ? toff + (slab) * slab_bytes : 0x7ff00000;                         \
        _Pragma("unroll") for (int i = 0; i < LPT; ++i)                                                  \
            rg[p][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ar, o_, i * 16 * 64, 0)); \
    }
#pragma unroll
    for (int p = 0; p < TURN; ++p) {
        STREAM_ALOAD(p, p)
        __builtin_amdgcn_sched_barrier(0);  // slab after slab: in the compiler's own order the first wait was for all of them
    }
    const int end = m0 < *T_dev ? turns_end : TURN;
    int s0 = 0;
    do {
#pragma unroll
        for (int p = 0; p < TURN; ++p) {
            unsigned char *to = smem + p * STAGE + soff;
#pragma unroll
            for (int i = 0; i < LPT; ++i) *reinterpret_cast<u32x4 *>(to + i * 16 * 256) = rg[p][i];
            STREAM_ALOAD(p, s0 + p + TURN)
            __syncthreads();  // slab s0 + p is there; slab s0 + p - 2 has been read
        }
        s0 += TURN;
    } while (s0 < end);
#undef STREAM_ALOAD
}

// R: 32-row blocks of the tile, all of them in every multiplying wavefront; NM: multiplying wavefronts, 32 columns each.
template <int R, int NM>
struct StreamCfg {
    static constexpr int ROWS = 32 * R, COLS = 32 * NM;
    static constexpr int THREADS = 64 * (NM + 4);
    static constexpr int TURN = 3;                             // slabs per turn of the loop = stages
    static constexpr int STAGE = ROWS * STREAM_BK * (int)sizeof(bf16_t);
    static constexpr int SMEM = TURN * STAGE + NM * 2048;      // stages, output staging
    static constexpr int DW = NM >= 6 ? 12 : 24;               // steps of W in flight, a divisor of a turn's 24; ten wavefronts have 168 registers each
    static constexpr int AHEAD = R == 1 ? 7 : R == 2 ? 3 : 1;  // steps of A read ahead
};

template <int R, int NM, int EPI>
__global__ __launch_bounds__(64 * (NM + 4)) void gemm_stream_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ Wp,
                                                                    const float *__restrict__ bias, bf16_t *__restrict__ out,
                                                                    const int32_t *__restrict__ T_dev, int max_rows, int likely_rows,
                                                                    uint32_t shape)
{
    typedef StreamCfg<R, NM> Cfg;
    constexpr int DW = Cfg::DW, TURN = Cfg::TURN, AHEAD = Cfg::AHEAD;
    const int N = stream_n(shape), K = stream_k(shape), xr_bits = shape >> 30, plane = pass_pitch(max_rows) * PLANE;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [TURN][ROWS][128] bf16, staging
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // blocks go round-robin to the 8 XCDs (gridDim.x is a multiple of 8), which stand in a grid of xr x 8 / xr: an XCD takes every
    // xr-th row tile and every (8 / xr)-th column tile, the row tiles that may turn out to be empty last
    const int xcd = blockIdx.x & 7;
    const int tm = (blockIdx.y << xr_bits) + (xcd & ((1 << xr_bits) - 1)), tn = ((blockIdx.x >> 3) << (3 - xr_bits)) + (xcd >> xr_bits);
    const int m0 = tm * Cfg::ROWS, n0 = tn * Cfg::COLS;
    if (m0 >= max_rows || n0 >= N) return;
    // Tiles that likely hold rows request their slabs before the token count is there: it is the same chain of latencies as a slab's.
    if (m0 >= likely_rows && m0 >= *T_dev) return;
    const int slabs = K / STREAM_BK;  // the host checks K % 128 == 0
    const int turns_end = (slabs + TURN - 1) / TURN * TURN;
    // A tile that turns out to hold no row goes through one turn and stores nothing.

    if (wave >= NM) {
        fetch_a<2 * R, TURN>(A, T_dev, smem, tid - 64 * NM, m0, K, plane, slabs, turns_end);
        return;
    }

    const int ct = (n0 >> 5) + wave;  // the wavefront's 32 columns; the last tile may reach past N: zeros, not stored
    const bool on = ct * 32 < N;
    const int steps = K >> 4;
    const auto wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(Wp + (size_t)ct * 32 * K), 0, on ? K * 64 : 0, 0x00020000);
    u32x4 wr[DW];
#define STREAM_WLOAD(p, step)                                                                            \
    wr[p] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (step) < steps ? lane * 16 + (step) * 1024 : 0x7ff00000, 0, 0));
    f32x16 acc[R];  // the sums start at the bias: register 4g + i of a lane is column 8g + 4 half + i
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + min(ct, (N >> 5) - 1) * 32 + 8 * g + 4 * half);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[r][4 * g + i] = b[i];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < DW; ++p) {
        STREAM_WLOAD(p, p)
        __builtin_amdgcn_sched_barrier(0);
    }
    int aoff[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) aoff[j] = l32 * 256 + (((2 * j + half) ^ (l32 & 15)) << 4);
    bf16x8 af[AHEAD + 1][R];
#define STREAM_AREAD(step, stage)                                                                        \
    _Pragma("unroll") for (int r = 0; r < R; ++r)                                                        \
        af[(step) % (AHEAD + 1)][r] = *reinterpret_cast<const bf16x8 *>(smem + (stage) * Cfg::STAGE + aoff[(step) & 7] + r * 32 * 256);
    // the turn's slab u, the pass's slab s
#define STREAM_SLAB(s, u)                                                                                \
    _Pragma("unroll") for (int j = 0; j < 8; ++j) {                                                      \
        STREAM_AREAD(j + AHEAD, (j + AHEAD < 8 ? (u) : (u) + 1) % TURN)                                  \
        _Pragma("unroll") for (int r = 0; r < R; ++r)                                                    \
            acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wr[((u) * 8 + j) % DW]), af[j % (AHEAD + 1)][r], acc[r], 0, 0, 0); \
        STREAM_WLOAD(((u) * 8 + j) % DW, (s) * 8 + j + DW)                                               \
        __builtin_amdgcn_sched_barrier(0);                                                               \
    }
    // The barrier without the wait for this wavefront's LDS reads that __syncthreads() adds: what it has read of the slab before has
    // been used by an MFMA, and the slabs it is reading are not stored to until the next barrier.
#define STREAM_BARRIER                                                                                   \
    asm volatile("" ::: "memory");                                                                       \
    __builtin_amdgcn_s_barrier();                                                                        \
    asm volatile("" ::: "memory");
    const int T = *T_dev;
    const int end = m0 < T ? turns_end : TURN;
    STREAM_BARRIER  // the fetching wavefronts' first one: slab 0
    STREAM_BARRIER  // slab 1; before slab s there have been s + 2 of them, end in all
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) { STREAM_AREAD(j, 0) }
    int s = 0;
    do {
        STREAM_SLAB(s, 0)
        STREAM_BARRIER
        STREAM_SLAB(s + 1, 1)
        if (s + TURN < end) { STREAM_BARRIER }
        STREAM_SLAB(s + 2, 2)  // its reads ahead at the very end are of a stage that is there and go unused
        s += TURN;
        if (s < end) { STREAM_BARRIER }
    } while (s < end);
#undef STREAM_BARRIER
#undef STREAM_SLAB
#undef STREAM_AREAD
#undef STREAM_WLOAD
    if (!on || m0 >= T) return;
    // 32 x 32 outputs at a time through the wavefront's own 2 KB: 16-byte chunk c of a row at c ^ ((row >> 1) & 3), then 16-byte stores
    unsigned char *stg = smem + TURN * Cfg::STAGE + wave * 2048;
    bf16_t *to = out + plane_at(ct * 32, m0, plane);
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 o4;
#pragma unroll
            for (int i = 0; i < 4; ++i) o4[i] = (bf16_t)(EPI == EPI_BIAS_GELU ? gelu_erf(acc[r][4 * g + i]) : acc[r][4 * g + i]);
            *reinterpret_cast<bf16x4 *>(stg + l32 * 64 + ((g ^ ((l32 >> 1) & 3)) << 4) + half * 8) = o4;
        }
        __builtin_amdgcn_wave_barrier();  // LDS serves a wave's accesses in order
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int rr = j * 16 + (lane >> 2), ch = lane & 3;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(stg + rr * 64 + ((ch ^ ((rr >> 1) & 3)) << 4));
            *reinterpret_cast<u32x4 *>(to + (r * 32 + rr) * PLANE + ch * 8) = v;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// The same product for the smallest tiles, where one wavefront's MFMAs over K are the chain (32 x 32 outputs keep a SIMD's matrix core
// busy for 32 clocks per 16 elements of K, with three SIMDs idle): a multiplying wavefront has 16 columns instead of 32, and 16 RB rows,
// by MFMA 16x16x32, whose result for 32 elements of K has the bits of two 32x32x16 on this part (sums over groups of eight elements,
// one after the other).  A chunk's embedding would otherwise depend on the pass it is in: fp32 results were compared for eleven kinds of
// inputs (exponents over 2^40, opposite pairs, biases up to 2^40, denormals, infinities, ties; none of 8.6 million differs), and the
// tests compare the tiles bit for bit, with sums that cancel too.  So a tile's columns spread over twice as many SIMDs.  W is read
// from the same copy: of its 2 KB per 32 columns and 32 elements of K a lane takes the row and the eight elements that its operand slot
// has.  Per launch, before (32x32 of gemm_stream_kernel) and now: 80 x 768 x 768 3.2 and 2.7 us, 80 x 768 x 3072 6.7 and 5.2,
// 244 x 768 x 3072 7.0 and 5.8, 1040 x 768 x 3072 11.4 and 10.1 (64x64).  24 steps of W ahead instead of 12, in turns of six slabs, were 0.2 us
// slower at K = 768 and no faster at 3072; slabs of 256 elements, with half the barriers, 0.1 to 0.5 us slower.
template <int RB, int NM>
struct Stream16Cfg {
    static constexpr int ROWS = 16 * RB, COLS = 16 * NM;
    static constexpr int THREADS = 64 * (NM + 4);
    static constexpr int TURN = 3, DW = 4 * TURN;              // slabs per turn of the loop = stages; steps of W in flight, a turn's
    static constexpr int STAGE = ROWS * STREAM_BK * (int)sizeof(bf16_t);
    static constexpr int SMEM = TURN * STAGE + NM * RB * 512;  // stages, output staging
    static constexpr int AHEAD = 2, SLOTS = AHEAD + 1;         // steps of A read ahead; its registers, a divisor of a turn's 12 steps
};

template <int RB, int NM, int EPI>
__global__ __launch_bounds__(64 * (NM + 4)) void gemm_stream16_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ Wp,
                                                                      const float *__restrict__ bias, bf16_t *__restrict__ out,
                                                                      const int32_t *__restrict__ T_dev, int max_rows, int likely_rows,
                                                                      uint32_t shape)
{
    typedef Stream16Cfg<RB, NM> Cfg;
    constexpr int DW = Cfg::DW, TURN = Cfg::TURN, AHEAD = Cfg::AHEAD, SLOTS = Cfg::SLOTS;
    const int N = stream_n(shape), K = stream_k(shape), xr_bits = shape >> 30, plane = pass_pitch(max_rows) * PLANE;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [TURN][ROWS][128] bf16, staging
    const int tid = threadIdx.x, lane = tid & 63, quarter = lane >> 4, l16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = blockIdx.x & 7;  // as in gemm_stream_kernel
    const int tm = (blockIdx.y << xr_bits) + (xcd & ((1 << xr_bits) - 1)), tn = ((blockIdx.x >> 3) << (3 - xr_bits)) + (xcd >> xr_bits);
    const int m0 = tm * Cfg::ROWS, n0 = tn * Cfg::COLS;
    if (m0 >= max_rows || n0 >= N) return;
    if (m0 >= likely_rows && m0 >= *T_dev) return;
    const int slabs = K / STREAM_BK;  // the host checks K % 128 == 0
    const int turns_end = (slabs + TURN - 1) / TURN * TURN;

    if (wave >= NM) {
        fetch_a<RB, TURN>(A, T_dev, smem, tid - 64 * NM, m0, K, plane, slabs, turns_end);
        return;
    }

    const int ct = (n0 >> 4) + wave;  // the wavefront's 16 columns; the last tile may reach past N: zeros, not stored
    const bool on = ct * 16 < N;
    const int steps = K >> 5;
    const auto wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(Wp + (size_t)(ct >> 1) * 32 * K), 0, on ? K * 64 : 0, 0x00020000);
    const int woff = (quarter >> 1) * 1024 + ((quarter & 1) * 32 + (ct & 1) * 16 + l16) * 16;
    u32x4 wr[DW];
#define STREAM_WLOAD(p, step)                                                                            \
    wr[p] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (step) < steps ? woff + (step) * 2048 : 0x7ff00000, 0, 0));
    f32x4 acc[RB];  // the sums start at the bias: register i of a lane is column 4 quarter + i
    {
        const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + min(ct, (N >> 4) - 1) * 16 + 4 * quarter);
#pragma unroll
        for (int r = 0; r < RB; ++r) acc[r] = b;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < DW; ++p) {
        STREAM_WLOAD(p, p)
        __builtin_amdgcn_sched_barrier(0);
    }
    int aoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) aoff[j] = l16 * 256 + (((4 * j + quarter) ^ l16) << 4);
    bf16x8 af[SLOTS][RB];
#define STREAM_AREAD(step, stage)                                                                        \
    _Pragma("unroll") for (int r = 0; r < RB; ++r)                                                       \
        af[(step) % SLOTS][r] = *reinterpret_cast<const bf16x8 *>(smem + (stage) * Cfg::STAGE + aoff[(step) & 3] + r * 16 * 256);
#define STREAM_BARRIER                                                                                   \
    asm volatile("" ::: "memory");                                                                       \
    __builtin_amdgcn_s_barrier();                                                                        \
    asm volatile("" ::: "memory");
    const int T = *T_dev;
    const int end = m0 < T ? turns_end : TURN;
    STREAM_BARRIER  // the fetching wavefronts' first one: slab 0
    STREAM_BARRIER  // slab 1; before slab s there have been s + 2 of them, end in all
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) { STREAM_AREAD(j, 0) }
    int s = 0;
    do {
#pragma unroll
        for (int u = 0; u < TURN; ++u) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                STREAM_AREAD(u * 4 + j + AHEAD, (j + AHEAD < 4 ? u : u + 1) % TURN)  // at the very end of a stage that is there, unused
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[u * 4 + j]), af[(u * 4 + j) % SLOTS][r], acc[r], 0, 0, 0);
                STREAM_WLOAD(u * 4 + j, (s + u) * 4 + j + DW)
                __builtin_amdgcn_sched_barrier(0);
            }
            if (u < TURN - 2 || s + TURN < end) { STREAM_BARRIER }
        }
        s += TURN;
    } while (s < end);
#undef STREAM_BARRIER
#undef STREAM_AREAD
#undef STREAM_WLOAD
    if (!on || m0 >= T) return;
    // 16 RB x 16 outputs through the wavefront's own LDS, a row's 32 bytes together, 8-byte unit u at u ^ 2 in every other eight rows; then 16-byte stores
    unsigned char *stg = smem + TURN * Cfg::STAGE + wave * (RB * 512);
    bf16_t *to = out + plane_at(ct * 16, m0, plane);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        bf16x4 o4;
#pragma unroll
        for (int i = 0; i < 4; ++i) o4[i] = (bf16_t)(EPI == EPI_BIAS_GELU ? gelu_erf(acc[r][i]) : acc[r][i]);
        *reinterpret_cast<bf16x4 *>(stg + (r * 16 + l16) * 32 + ((quarter ^ ((l16 >> 2) & 2)) << 3)) = o4;
    }
    __builtin_amdgcn_wave_barrier();  // LDS serves a wave's accesses in order
#pragma unroll
    for (int i = 0; i < RB / 2; ++i) {
        const int row = i * 32 + (lane >> 1), ch = lane & 1;
        const u32x4 v = *reinterpret_cast<const u32x4 *>(stg + row * 32 + ((ch ^ ((row >> 3) & 1)) << 4));
        *reinterpret_cast<u32x4 *>(to + row * PLANE + ch * 8) = v;
    }
}

}  // namespace
