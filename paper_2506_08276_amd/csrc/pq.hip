// Product quantisation: training, encoding, per-query lookup tables and the stand-alone ADC scorer
// (LEANN Sec. 3 offline stage: the PQ table kept in place of the embeddings; Alg. 2: the approximate distance that
// ranks new neighbours).  256 centroids per subspace.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "common.h"
#include "wave.h"

namespace {

constexpr int KSUB = 256;
constexpr int MAX_TRAIN = 65536;
constexpr int MAX_DSUB = 32;

__host__ __device__ inline uint64_t splitmix64(uint64_t &st)
{
    uint64_t z = (st += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// The seeded Fisher-Yates permutation's first nt entries on the device.  Step i = n - 1 .. 1 swaps the entries i and j(i) <= i.  After it, entry i is
// final: what was at j(i).  Who put that there is known without running the steps: the last step before it (the smallest t > i) with
// j(t) = j(i), which brought there what was at its own position t; so
//   at(p) = what is at position p just before step p = at(t) for the smallest t > p with j(t) = p, or p if there is none,
//   final entry i = at(t) for the smallest t > i with j(t) = j(i), or j(i) if there is none; entry 0: at(0).
// The draws do not depend on each other, nor do the chains (a logarithm of n long): n = 100000 took the host 450 us and a copy of the
// rows behind it, the three kernels take 23 us (a whole call of 6 iterations at d = 768: 2290 and 2050 us).
constexpr uint32_t NO_STEP = 0xffffffffu;

struct Steps {
    uint32_t *j;     // [n] a step's draw
    uint32_t *first; // [n] of position p: the smallest step t > p with j(t) = p
    uint32_t *head, *link;  // [n] the steps with j(t) = p, in any order: head[p], then link[]
};

__global__ __launch_bounds__(256) void clear_steps_kernel(Steps s, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) s.first[i] = s.head[i] = NO_STEP;
}

__global__ __launch_bounds__(256) void draw_steps_kernel(Steps s, int64_t n, uint64_t seed)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < 1 || i >= n) return;
    uint64_t state = seed + (uint64_t)(n - 1 - i) * 0x9e3779b97f4a7c15ull;  // of the generator before draw n - 1 - i
    const uint32_t j = (uint32_t)(splitmix64(state) % (uint64_t)(i + 1));
    s.j[i] = j;
    s.link[i] = atomicExch(&s.head[j], (uint32_t)i);
    if (j < i) atomicMin(&s.first[j], (uint32_t)i);
}

__global__ __launch_bounds__(256) void training_rows_kernel(Steps s, int64_t nt, int64_t *__restrict__ rows)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nt) return;
    uint32_t p = 0, t = s.first[0];
    if (i > 0) {
        p = s.j[i];
        t = NO_STEP;
        for (uint32_t u = s.head[p]; u != NO_STEP; u = s.link[u])
            if (u > (uint32_t)i && u < t) t = u;
    }
    while (t != NO_STEP) {
        p = t;
        t = s.first[p];
    }
    rows[i] = p;
}

// The training rows: rows[i] of x (fp32 [n][d]) -> xt[m][i][d / m_sub], a plane per subspace, so that kernels that work on one
// subspace read nothing else: pieces of 96 bytes straddle 128-byte lines, and in rows the line's rest belongs to other subspaces.  A block
// takes GATHER_ROWS rows: that many pieces of a plane lie together.  65536 x 768 from 100000: 73 us, copied row by row 98; a call's
// assignments of such rows (and the last one, of rows as they are) took 148 us on average, 151 with training rows as they are (135 now).
constexpr int GATHER_ROWS = 16;

template <class Piece>  // f32x4 where every sub-vector consists of such and begins at one
__global__ __launch_bounds__(256) void gather_rows_kernel(const float *__restrict__ x, const int64_t *__restrict__ rows, int64_t nt, int d,
                                                          int dsub, float *__restrict__ xt)
{
    constexpr int W = sizeof(Piece) / sizeof(float);
    const int64_t t0 = (int64_t)blockIdx.x * GATHER_ROWS;
    const uint32_t per_row = dsub / W, per_plane = GATHER_ROWS * per_row, all = GATHER_ROWS * (d / W);
    for (uint32_t e = threadIdx.x; e < all; e += 256) {
        const uint32_t m = e / per_plane, in_plane = e - m * per_plane, i = in_plane / per_row, j = in_plane - i * per_row;
        if (t0 + i >= nt) continue;
        *reinterpret_cast<Piece *>(xt + ((int64_t)m * nt + t0 + i) * dsub + j * W) =
            *reinterpret_cast<const Piece *>(x + rows[t0 + i] * d + m * dsub + j * W);
    }
}

// The first 256 training rows (wrapping when there are fewer) as the centroids training starts from.
__global__ void first_centroids_kernel(const float *__restrict__ xt, int64_t nt, int dsub, float *__restrict__ codebook)
{
    const int m = blockIdx.y;
    for (int i = threadIdx.x; i < dsub; i += blockDim.x)
        codebook[((size_t)m * KSUB + blockIdx.x) * dsub + i] = xt[((size_t)m * nt + blockIdx.x % nt) * dsub + i];
}

// Nearest centroid (squared L2, ties to the lowest index) of every row in one subspace; row r's sub-vector m begins at
// x[r * x_row + m * x_sub], its code is out[r * row_pitch + m * m_pitch].
//
// What decides is the fp32 sum s(c) = sum_j (x_j - c_j)^2, j ascending.  Computing all 256 of them on the vector ALU bounds
// the kernel there (two instructions per element: 1814 us at 65536 rows, d = 768, 32 subspaces), so the matrix cores
// find the nearest centroid first and s(c) is only computed where they cannot tell:
//  - x and c are centred on a common point u (differences to u instead of to the origin: what is left to round scales
//    with the spread of the data), split into two bf16 each, and |c'|^2 - 2 x'.c' is accumulated in fp32 by three MFMAs
//    per 16 elements (hi.hi, hi.lo, lo.hi), 32 centroids by 32 rows at a time; a lane owns a row and half the centroids.
//  - the running minimum and second minimum are kept as floats with 7 bits of index in the low mantissa bits.  Of the minimum and two
//    values the smallest is the new minimum and the median the one that may be the new second: nine instructions for four values, a bit operation for
//    each, two medians and three minima of three (132 us; one value after the other, twelve instructions, 138: 65536 rows, d = 768, 32 subspaces).
//  - With X = |x'|, C = max |c'|, U = (X + C)^2 and bf16's rounding of 2^-8, a centroid's value is off by, in units of
//    2^-16 U: the split 1 (each low part rounded by 2^-17 of its operand and low.low left out: 4 * 2^-17 of |2x'||c'| <= U / 2),
//    the additions of the six MFMAs at most 0.75 (each of the 96 counted with 2^-23 U, a whole unit), |c'|^2 0.13, s(c) itself
//    0.13, the centring 0.01: 4.04 for two centroids.  The index bits (2^7 units in the last place) move a value by 2^-16 of
//    itself; p - 2^-16 |p| grows with p, so the second minimum's share covers all other centroids.  A gap of more than
//    2^-16 (5.5 U + |minimum| + |second|) therefore leaves no doubt.  The other rows (few on embeddings; all of them where anything
//    could overflow or is not a number, or where the nearest centroids are equal) get s(c) for all centroids by one wavefront.
//    Such a row is read once, an element per lane, and eight elements' centroids are read together (an element after the other, each waited for: 132 us
//    where it takes 124).
// So the result is s(c)'s for every input.  65536 rows, d = 768, 32 subspaces: 124 us, of them 15 before the first row, 32 for the rows' way in and
// their splitting, 10 for each of the eight tiles (5 of matrix instructions, 4 of the nine above) and some 8 for the rows in doubt.  No faster: the next
// rows' lines asked for while the tiles run (131), a wavefront's priority raised for its matrix instructions or lowered (124).
constexpr int ASSIGN_THREADS = 512;

__host__ __device__ constexpr int assign_smem(int ks, int dsub)
{
    return 2 * ks * KSUB * 16 * 2 + KSUB * (dsub | 1) * 4 + KSUB * 4 + MAX_DSUB * 4 + 4 * 4;
}

template <int KS>  // 16-element steps of the (zero-padded) sub-vector
__global__ __launch_bounds__(ASSIGN_THREADS, 4) void assign_kernel(const float *__restrict__ x, int64_t x_row, int64_t x_sub, int64_t n, int dsub, int m_sub,
                                                                const float *__restrict__ codebook, int64_t rows_per_block, int xcd_bits,
                                                                uint8_t *__restrict__ out, int64_t row_pitch, int64_t m_pitch)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int P = dsub | 1;  // odd row pitch: 64 centroids' elements lie in different banks
    bf16_t *frag = reinterpret_cast<bf16_t *>(smem);  // [hi, lo][KS][256][16]
    float *c2 = reinterpret_cast<float *>(frag + 2 * KS * KSUB * 16);  // |c'|^2, read four at a time
    float *mu = c2 + KSUB;
    uint32_t *cmax = reinterpret_cast<uint32_t *>(mu + MAX_DSUB);
    float *cbf = reinterpret_cast<float *>(cmax + 4);  // [256][P]
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // blocks go round-robin to the 8 XCDs: with xcd_bits = 3 all subspaces of a run of rows are on one XCD, whose L2 then holds
    // the 128-byte lines that neighbouring subspaces share where x holds whole rows (training rows lie in a plane per subspace)
    const int m = (blockIdx.x >> xcd_bits) % m_sub;
    const int64_t chunk = ((int64_t)((blockIdx.x >> xcd_bits) / m_sub) << xcd_bits) + (blockIdx.x & ((1 << xcd_bits) - 1));
    const int64_t beg = chunk * rows_per_block, end = beg + rows_per_block < n ? beg + rows_per_block : n;
    if (beg >= end) return;

    for (int i = tid; i < KSUB * dsub; i += ASSIGN_THREADS) cbf[(i / dsub) * P + i % dsub] = codebook[(size_t)m * KSUB * dsub + i];
    __syncthreads();
    if (tid < dsub) {
        float s = 0.f;
        for (int c = 0; c < KSUB; c += 8) s += cbf[c * P + tid];
        mu[tid] = s * (8.0f / KSUB);
    }
    __syncthreads();
    if (tid < KSUB) {
        float s = 0.f;
#pragma unroll
        for (int p = 0; p < 2 * KS; ++p) {
            bf16x8 hi, lo;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = p * 8 + i;
                const float v = j < dsub ? cbf[tid * P + j] - mu[j] : 0.f;
                s += v * v;
                hi[i] = (bf16_t)v;
                lo[i] = (bf16_t)(v - (float)hi[i]);
            }
            *reinterpret_cast<bf16x8 *>(frag + ((p >> 1) * KSUB + tid) * 16 + (p & 1) * 8) = hi;
            *reinterpret_cast<bf16x8 *>(frag + ((KS + (p >> 1)) * KSUB + tid) * 16 + (p & 1) * 8) = lo;
        }
        c2[tid] = s;
        const uint32_t top = wave_max(__float_as_uint(s));  // not negative: the bits are in order, NaN above all
        if (lane == 0) cmax[wave] = top;
    }
    __syncthreads();
    const uint32_t top = max(max(cmax[0], cmax[1]), max(cmax[2], cmax[3]));
    const float C = sqrtf(__uint_as_float(top));
    const bool vec = (dsub & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;  // then every sub-vector starts at 16 bytes

    for (int64_t r0 = beg + wave * 64; r0 < end; r0 += ASSIGN_THREADS) {
        bf16x8 bh[2][KS], bl[2][KS];
        float m1[2], m2[2], X[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int64_t row = min(r0 + g * 32 + l32, end - 1);
            const float *xr = x + row * x_row + m * x_sub;
            float sq = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int k0 = ks * 16 + half * 8;
                float v[8];
                if (vec) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        f32x4 w = {0.f, 0.f, 0.f, 0.f};
                        if (k0 + 4 * q < dsub) w = *reinterpret_cast<const f32x4 *>(xr + k0 + 4 * q) - *reinterpret_cast<const f32x4 *>(mu + k0 + 4 * q);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[4 * q + i] = w[i];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = k0 + i < dsub ? xr[k0 + i] - mu[k0 + i] : 0.f;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    sq += v[i] * v[i];
                    const float w = -2.f * v[i];
                    bh[g][ks][i] = (bf16_t)w;
                    bl[g][ks][i] = (bf16_t)(w - (float)bh[g][ks][i]);
                }
            }
            const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(sq), __float_as_uint(sq), false, false);
            X[g] = sqrtf(__uint_as_float(p[0]) + __uint_as_float(p[1]));
            m1[g] = m2[g] = INFINITY;
        }
        // A tile's fragments are read while the vector ALU goes through the tile before.
        bf16x8 ch[KS], cl[KS];
        auto fetch = [&](int t) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                ch[ks] = *reinterpret_cast<const bf16x8 *>(frag + (ks * KSUB + t * 32 + l32) * 16 + half * 8);
                cl[ks] = *reinterpret_cast<const bf16x8 *>(frag + ((KS + ks) * KSUB + t * 32 + l32) * 16 + half * 8);
            }
        };
        fetch(0);
        uint32_t keep = ~0x7fu;
        asm("" : "+v"(keep));  // a literal and a scalar register do not fit into one instruction
#pragma unroll 1  // unrolled, the fragments of several tiles are held at once and spill
        for (int t = 0; t < KSUB / 32; ++t) {
            f32x16 acc[2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 cc = *reinterpret_cast<const f32x4 *>(c2 + t * 32 + 8 * q + 4 * half);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[0][4 * q + i] = acc[1][4 * q + i] = cc[i];
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int g = 0; g < 2; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch[ks], bh[g][ks], acc[g], 0, 0, 0);
#pragma unroll
                for (int g = 0; g < 2; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch[ks], bl[g][ks], acc[g], 0, 0, 0);
#pragma unroll
                for (int g = 0; g < 2; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cl[ks], bh[g][ks], acc[g], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            fetch(min(t + 1, KSUB / 32 - 1));
            asm volatile("" ::: "memory");  // here, not where they are used
#pragma unroll
            for (int r = 0; r < 16; r += 4) {  // register r: centroid 32t + 8(r/4) + 4 half + r%4
                // The index in a scalar register, and the minima by their instructions: otherwise the compiler adds the index in two and
                // quiets the operands.
                uint32_t index[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    index[i] = t * 16 + r + i;
                    asm("" : "+s"(index[i]));
                }
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    float v[4], second[2];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = __uint_as_float((__float_as_uint(acc[g][r + i]) & keep) | index[i]);
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        second[i] = __builtin_amdgcn_fmed3f(m1[g], v[2 * i], v[2 * i + 1]);
                        asm("v_min3_f32 %0, %1, %2, %3" : "=v"(m1[g]) : "v"(m1[g]), "v"(v[2 * i]), "v"(v[2 * i + 1]));
                    }
                    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(m2[g]) : "v"(m2[g]), "v"(second[0]), "v"(second[1]));
                }
            }
        }
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const auto p1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m1[g]), __float_as_uint(m1[g]), false, false);
            const auto p2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m2[g]), __float_as_uint(m2[g]), false, false);
            const float a1 = __uint_as_float(p1[0]), b1 = __uint_as_float(p1[1]);  // lower half's centroids, upper half's
            const bool upper = b1 < a1;
            const float first = upper ? b1 : a1, other = upper ? a1 : b1;
            const float second = fminf(other, fminf(__uint_as_float(p2[0]), __uint_as_float(p2[1])));
            const uint32_t i7 = __float_as_uint(first) & 0x7fu;
            int code = (int)((i7 >> 4) * 32 + ((i7 & 15) >> 2) * 8 + (i7 & 3)) + (upper ? 4 : 0);
            const float S = X[g] + C;
            // the constant covers flushed denormals; from S = 1e19 on an intermediate sum can overflow, and an infinity with index
            // bits in it is a NaN to the medians
            const bool sure = S < 1e19f && second - first > fmaf(5.5f / 65536.f * S, S, fmaf(fabsf(first) + fabsf(second), 1.f / 65536.f, 1e-33f));
            const int64_t row = r0 + g * 32 + l32;
            unsigned long long doubt = __ballot(!sure && half == 0 && row < end);
            while (doubt) {
                const int who = __ffsll((long long)doubt) - 1;
                doubt &= doubt - 1;
                const float *xr = x + (r0 + g * 32 + who) * x_row + m * x_sub;
                float s[4] = {0.f, 0.f, 0.f, 0.f};
                const int own = __float_as_int(xr[min(lane, dsub - 1)]);
#pragma unroll 8
                for (int j = 0; j < dsub; ++j) {
                    const float xv = __int_as_float(__builtin_amdgcn_readlane(own, j));
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float t = xv - cbf[(k * 64 + lane) * P + j];
                        s[k] = fmaf(t, t, s[k]);
                    }
                }
                // the smallest finite sum, the lowest index among equals; index 0 if there is none
                uint32_t b = 0x7f800000u, c = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (s[k] < __uint_as_float(b)) {
                        b = __float_as_uint(s[k]);
                        c = k * 64 + lane;
                    }
                const uint32_t least = ~wave_max(~b);
                const uint32_t idx = ~wave_max(b == least && b < 0x7f800000u ? ~c : 0u);
                if (lane == who) code = least < 0x7f800000u ? (int)idx : 0;
            }
            if (half == 0 && row < end) out[row * row_pitch + m * m_pitch] = (uint8_t)code;
        }
    }
}

// Training rows of every centroid: order[m][..] holds the row numbers sorted by centroid, ascending within one;
// first[m][c] .. first[m][c + 1] are centroid c's.  Counting sort in two launches, GROUP_BLOCKS blocks of 16 wavefronts per
// subspace, each wavefront a run of consecutive rows: count_rows_kernel leaves every run's rows per centroid in
// counts[m][run][c], group_rows_kernel puts the rows behind those of the smaller centroids and the earlier runs (one block
// per subspace left most of the chip idle: 65 us at 65536 rows and 32 subspaces).
constexpr int GROUP_BLOCKS = 4, GROUP_RUNS = 16 * GROUP_BLOCKS;

__device__ inline int run_rows(int nt) { return ((nt + GROUP_RUNS - 1) / GROUP_RUNS + 63) & ~63; }

__global__ __launch_bounds__(1024) void count_rows_kernel(const uint8_t *__restrict__ assign, int nt, int32_t *__restrict__ counts)
{
    __shared__ int cnt[16][KSUB];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint8_t *as = assign + (size_t)m * nt;
    const int per = run_rows(nt), run = blockIdx.y * 16 + wave;
    const int beg = min(nt, run * per), end = min(nt, beg + per);
    for (int i = tid; i < 16 * KSUB; i += 1024) (&cnt[0][0])[i] = 0;
    __syncthreads();
    for (int r = beg + lane; r < end; r += 64) atomicAdd(&cnt[wave][as[r]], 1);
    __syncthreads();
    int32_t *out = counts + ((size_t)m * GROUP_RUNS + blockIdx.y * 16) * KSUB;
    for (int i = tid; i < 16 * KSUB; i += 1024) out[i] = (&cnt[0][0])[i];
}

__global__ __launch_bounds__(1024) void group_rows_kernel(const uint8_t *__restrict__ assign, int nt,
                                                          const int32_t *__restrict__ counts, int32_t *__restrict__ order,
                                                          int32_t *__restrict__ first)
{
    __shared__ int cnt[16][KSUB];  // where the wavefront's next row of a centroid goes
    __shared__ int total[KSUB];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint8_t *as = assign + (size_t)m * nt;
    const int per = run_rows(nt), run0 = blockIdx.y * 16, run = run0 + wave;
    const int beg = min(nt, run * per), end = min(nt, beg + per);
    const int32_t *cm = counts + (size_t)m * GROUP_RUNS * KSUB;
    int before = 0;  // rows of centroid tid in the runs of earlier blocks
    if (tid < KSUB) {
        int s = 0;
#pragma unroll 16
        for (int w = 0; w < GROUP_RUNS; ++w) {
            const int c = cm[w * KSUB + tid];
            s += c;
            if (w < run0) before += c;
            if (w >= run0 && w < run0 + 16) cnt[w - run0][tid] = c;
        }
        total[tid] = s;
    }
    __syncthreads();
    if (wave == 0) {  // exclusive scan over the 256 centroids, four per lane
        int t[4], s = 0;
        for (int i = 0; i < 4; ++i) {
            t[i] = s;
            s += total[lane * 4 + i];
        }
        int incl = s;
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        for (int i = 0; i < 4; ++i) total[lane * 4 + i] = incl - s + t[i];
    }
    __syncthreads();
    if (tid < KSUB) {
        int at = total[tid];
        if (blockIdx.y == 0) {
            first[(size_t)m * (KSUB + 1) + tid] = at;
            if (tid == 0) first[(size_t)m * (KSUB + 1) + KSUB] = nt;
        }
        at += before;
        for (int w = 0; w < 16; ++w) {
            const int c = cnt[w][tid];
            cnt[w][tid] = at;
            at += c;
        }
    }
    __syncthreads();
    for (int r0 = beg; r0 < end; r0 += 64) {
        const int r = r0 + lane;
        const bool on = r < end;
        const uint32_t c = on ? as[r] : 0;
        unsigned long long same = __ballot(on);  // lanes with this lane's centroid
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const unsigned long long set = __ballot(c >> b & 1u);
            same &= (c >> b & 1u) ? set : ~set;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        const int at = cnt[wave][c];
        __builtin_amdgcn_wave_barrier();
        if (on) {
            order[(size_t)m * nt + at + rank] = r;
            if (rank == 0) cnt[wave][c] = at + __popcll(same);
        }
        __builtin_amdgcn_wave_barrier();  // LDS serves a wave's accesses in order
    }
}

// Centroid (c = blockIdx.x, m = blockIdx.y) <- mean of its training rows.  The sum's order is fixed: partial sum p adds the
// rows with r % 256 == p in ascending order, then the 256 partial sums are added pairwise (p, p + 128), (p, p + 64), ...
// The partial sums are in LDS; a group of 32 lanes (one per element) adds the rows with r % 8 equal to the group's number.
// Latency bounds it (row numbers, then the rows' pieces from beyond L2): 256 row numbers are looked through at a time and each
// group's rows listed first, so that a group has UPDATE_AHEAD of them in flight however they are spread.  Reads every training
// row once per round: 85 us at 65536 rows, d = 768, 32 subspaces (89 with the subspaces' pieces in the rows and a subspace's centroids on
// all XCDs; some 130 with 32 row numbers at a time, four rows in flight and a step of the pairwise sum per barrier).
constexpr int UPDATE_AHEAD = 16;

__global__ __launch_bounds__(256) void update_kernel(const float *__restrict__ xt, int64_t nt, int dsub, int xcd_bits,
                                                     const int32_t *__restrict__ order, const int32_t *__restrict__ first,
                                                     float *__restrict__ codebook)
{
    extern __shared__ __attribute__((aligned(16))) float part[];  // [256][dsub]
    __shared__ int32_t mine[8][256 + UPDATE_AHEAD];  // a group's rows among the 256, any valid row behind them
    // with xcd_bits = 3 all centroids of a subspace are on one XCD: its blocks go through the same plane at about the same pace, and
    // lines that pieces of different centroids share come into its L2 once
    const int c = (blockIdx.x >> xcd_bits) % KSUB, tid = threadIdx.x;
    const int m = ((int)(blockIdx.x >> xcd_bits) / KSUB << xcd_bits) + (blockIdx.x & ((1 << xcd_bits) - 1));
    const int lane32 = tid & 31, group = tid >> 5, shift = tid & 32;
    const int beg = first[(size_t)m * (KSUB + 1) + c], cnt = first[(size_t)m * (KSUB + 1) + c + 1] - beg;
    if (cnt == 0) return;  // an empty cluster keeps its centroid
    const int32_t *rows = order + (size_t)m * nt + beg;
    const float *xm = xt + (size_t)m * nt * dsub + min(lane32, dsub - 1);
    int32_t r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) r[k] = rows[min(k * 32 + lane32, cnt - 1)];
    for (int i = tid; i < 256 * dsub; i += 256) part[i] = 0.f;
    for (int i = tid; i < 8 * (256 + UPDATE_AHEAD); i += 256) (&mine[0][0])[i] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < cnt; i0 += 256) {
        int n_mine = 0;  // the same for the group's 32 lanes
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool on = i0 + k * 32 + lane32 < cnt && (r[k] & 7) == group;
            const uint32_t mask = (uint32_t)(__ballot(on) >> shift);
            if (on) mine[group][n_mine + __popc(mask & ((1u << lane32) - 1u))] = r[k];
            n_mine += __popc(mask);
        }
        if (i0 + 256 < cnt)
#pragma unroll
            for (int k = 0; k < 8; ++k) r[k] = rows[min(i0 + 256 + k * 32 + lane32, cnt - 1)];
        __builtin_amdgcn_wave_barrier();  // LDS serves a wavefront's accesses in order
        for (int j0 = 0; __any(j0 < n_mine); j0 += UPDATE_AHEAD) {
            int rr[UPDATE_AHEAD];
            float v[UPDATE_AHEAD];
#pragma unroll
            for (int k = 0; k < UPDATE_AHEAD; ++k) rr[k] = mine[group][min(j0, 256) + k];
#pragma unroll
            for (int k = 0; k < UPDATE_AHEAD; ++k) v[k] = xm[(size_t)rr[k] * dsub];
#pragma unroll
            for (int k = 0; k < UPDATE_AHEAD; ++k)
                if (j0 + k < n_mine && lane32 < dsub) part[(rr[k] & 255) * dsub + lane32] += v[k];
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // two steps of the pairwise sum at a time
    auto halve_twice = [&](auto *sum, int width) {
        for (int o = 64; o > 0; o >>= 2) {
            for (int i = tid; i < o * width; i += 256)
                sum[i] = (sum[i] + sum[i + 2 * o * width]) + (sum[i + o * width] + sum[i + 3 * o * width]);
            __syncthreads();
        }
    };
    if ((dsub & 3) == 0) halve_twice(reinterpret_cast<f32x4 *>(part), dsub >> 2);
    else halve_twice(part, dsub);
    if (tid < dsub) codebook[((size_t)m * KSUB + c) * dsub + tid] = part[tid] / (float)cnt;
}

// -|q_m - c|^2 (PQ's asymmetric distance, negated so that larger is closer), elements in index order.
__device__ inline float neg_dist(const float *__restrict__ q, const float *__restrict__ c, int dsub, bool vec)
{
    float s = 0.f;
    if (vec) {
        for (int j = 0; j < dsub; j += 4) {
            const f32x4 cv = *reinterpret_cast<const f32x4 *>(c + j);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float t = q[j + i] - cv[i];
                s = fmaf(t, t, s);
            }
        }
    } else {
        for (int j = 0; j < dsub; ++j) {
            const float t = q[j] - c[j];
            s = fmaf(t, t, s);
        }
    }
    return -s;
}

// lut[q][m][c] = -|q_m - codebook[m][c]|^2.  grid (ceil(nq / LUT_QUERIES), m_sub), 256 threads; a thread keeps its
// centroid in registers for all of the block's queries (21 us for 1024 queries of 768 elements; a block per query read the
// codebook out of L2 once for each of them: 53 us).
constexpr int LUT_QUERIES = 8;

__global__ __launch_bounds__(256) void lut_kernel(const float *__restrict__ queries, int64_t nq, int d, int m_sub,
                                                  const float *__restrict__ codebook, float *__restrict__ lut)
{
    __shared__ __attribute__((aligned(16))) float qs[LUT_QUERIES][MAX_DSUB];
    const int m = blockIdx.y, dsub = d / m_sub, c = threadIdx.x;
    const int64_t q0 = (int64_t)blockIdx.x * LUT_QUERIES;
    const int nb = (int)min((int64_t)LUT_QUERIES, nq - q0);
    const int ql = threadIdx.x >> 5, j0 = threadIdx.x & 31;
    static_assert(LUT_QUERIES * MAX_DSUB == 256, "one element per thread");
    qs[ql][j0] = ql < nb && j0 < dsub ? queries[(size_t)(q0 + ql) * d + m * dsub + j0] : 0.f;
    float cv[MAX_DSUB];  // zeros past the sub-vector, there as in qs: they add nothing, and the sums below go without a test per element
    const float *cb = codebook + ((size_t)m * KSUB + c) * dsub;
    if ((dsub & 3) == 0) {  // the codebook is an allocation of its own: its rows start at 16 bytes then
#pragma unroll
        for (int j = 0; j < MAX_DSUB; j += 4) {
            const f32x4 v = j < dsub ? *reinterpret_cast<const f32x4 *>(cb + j) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i) cv[j + i] = v[i];
        }
    } else {
#pragma unroll
        for (int j = 0; j < MAX_DSUB; ++j) cv[j] = j < dsub ? cb[j] : 0.f;
    }
    __syncthreads();
    for (int i = 0; i < nb; ++i) {
        float s = 0.f;
#pragma unroll
        for (int j0 = 0; j0 < MAX_DSUB; j0 += 8)
            if (j0 < dsub) {
#pragma unroll
                for (int j = j0; j < j0 + 8; ++j) {
                    const float t = qs[i][j] - cv[j];
                    s = fmaf(t, t, s);
                }
            }
        lut[((size_t)(q0 + i) * m_sub + m) * KSUB + c] = -s;
    }
}

void launch_lut(hipStream_t st, const float *queries, int64_t nq, const leann_pq *pq, float *lut)
{
    hipLaunchKernelGGL(lut_kernel, dim3((unsigned)((nq + LUT_QUERIES - 1) / LUT_QUERIES), pq->m_sub), dim3(256), 0, st, queries, nq,
                       pq->d, pq->m_sub, pq->codebook, lut);
}

// The scores without a table, for calls with few candidates: the table entries that they name are computed one by one (the
// same operations: the same bits) and added in subspace order.  grid (nq, ceil(nc / DIRECT_CAND)), 256 threads.
constexpr int DIRECT_CAND = 16;

// A struct, so that the arguments are read from memory: brought into registers with the dispatch they let a chain of launches run
// closer together, but this kernel runs alone and starts later for it (one query, 64 candidates, whole call 18.1 us; 17.8 read).
struct DirectArgs {
    const float *queries;
    const float *codebook;
    const uint8_t *codes;
    const uint32_t *cand;
    float *out;
    int *err;
    int64_t n;
    int d, m_sub, nc;
};

__global__ __launch_bounds__(256) void adc_direct_kernel(DirectArgs a)
{
    const float *__restrict__ queries = a.queries, *__restrict__ codebook = a.codebook;
    const uint8_t *__restrict__ codes = a.codes;
    const uint32_t *__restrict__ cand = a.cand;
    float *__restrict__ out = a.out;
    const int d = a.d, m_sub = a.m_sub, nc = a.nc;
    const int64_t n = a.n;
    extern __shared__ float part[];  // [DIRECT_CAND][m_sub | 1]
    const int q = blockIdx.x, j0 = blockIdx.y * DIRECT_CAND, here = min(DIRECT_CAND, nc - j0);
    const int dsub = d / m_sub, pitch = m_sub | 1;
    const float *qv = queries + (size_t)q * d;
    const uint32_t *cq = cand + (size_t)q * nc + j0;
    for (int i = threadIdx.x; i < here * m_sub; i += 256) {
        const int c = i / m_sub, m = i - c * m_sub;
        const uint32_t id = cq[c];
        float v = -INFINITY;
        if (id < n) v = neg_dist(qv + m * dsub, codebook + ((size_t)m * KSUB + codes[(size_t)id * m_sub + m]) * dsub, dsub, (dsub & 3) == 0);
        part[c * pitch + m] = v;
    }
    __syncthreads();
    if (threadIdx.x < here) {
        float s = 0.f;
        for (int m = 0; m < m_sub; ++m) s += part[threadIdx.x * pitch + m];
        if (cq[threadIdx.x] >= n) {
            s = -INFINITY;
            *a.err = 1;
        }
        out[(size_t)q * nc + j0 + threadIdx.x] = s;
    }
}

// out[q][j] = sum_m lut[q][m][codes[cand[q][j]][m]], m ascending.  grid (nq, parts), 256 threads; the query's table
// sits in LDS and serves the block's whole share of the candidates (`per_block`, a multiple of 2048): the 32 KB table
// load is paid once per block, not once per 2048 candidates.  A thread owns 8 candidates per round: all their ids,
// then all their code rows are requested before the first lookup, so that the random row gathers overlap instead of
// queueing up; the ids of the next round are fetched while the current round's lookups run.
constexpr int64_t ADC_DIRECT_MAX = 16384;  // candidates of a call that are scored without a table at most
constexpr int ADC_PER_ROUND = 2048, ADC_PER_THREAD = ADC_PER_ROUND / 256;

__global__ __launch_bounds__(256) void adc_kernel(const float *__restrict__ lut, const uint8_t *__restrict__ codes,
                                                  int64_t n, int m_sub, const uint32_t *__restrict__ cand, int nc,
                                                  int per_block, float *__restrict__ out, int *__restrict__ err)
{
    extern __shared__ float tab[];  // [m_sub][256]
    const int q = blockIdx.x;
    const int beg = blockIdx.y * per_block, end = min(nc, beg + per_block);
    if (beg >= end) return;
    const uint32_t *cq = cand + (size_t)q * nc;
    float *oq = out + (size_t)q * nc;
    uint32_t v[ADC_PER_THREAD];
#pragma unroll
    for (int i = 0; i < ADC_PER_THREAD; ++i) {
        const int j = beg + threadIdx.x + i * 256;
        v[i] = j < end ? cq[j] : 0xffffffffu;
    }
    const float4 *src = reinterpret_cast<const float4 *>(lut + (size_t)q * m_sub * KSUB);
    for (int i = threadIdx.x; i < m_sub * KSUB / 4; i += 256) reinterpret_cast<float4 *>(tab)[i] = src[i];
    bool bad = false;
    if (m_sub == 32) {  // 32-byte rows: both halves of every row in flight before any lookup
        for (int j0 = beg + threadIdx.x; j0 < end + threadIdx.x; j0 += ADC_PER_ROUND) {
            u32x4 c0[ADC_PER_THREAD], c1[ADC_PER_THREAD];
            bool ok[ADC_PER_THREAD];
#pragma unroll
            for (int i = 0; i < ADC_PER_THREAD; ++i) {
                ok[i] = v[i] < n;
                const uint8_t *code = codes + (size_t)(ok[i] ? v[i] : 0) * 32;
                c0[i] = *reinterpret_cast<const u32x4 *>(code);  // plain loads: streaming ("nontemporal") ones are 15-35 % slower here
                c1[i] = *reinterpret_cast<const u32x4 *>(code + 16);
            }
#pragma unroll
            for (int i = 0; i < ADC_PER_THREAD; ++i) {  // ids of the next round
                const int j = j0 + ADC_PER_ROUND + i * 256;
                v[i] = j < end ? cq[j] : 0xffffffffu;
            }
            if (j0 < beg + ADC_PER_ROUND) __syncthreads();  // first round: the table is complete (uniform condition)
#pragma unroll
            for (int i = 0; i < ADC_PER_THREAD; ++i) {
                const int j = j0 + i * 256;
                if (j >= end) continue;
                float s = 0.f;  // subspace order; the compiler issues the lookups in runs ahead of the additions
#pragma unroll
                for (int m = 0; m < 16; ++m) s += tab[m * KSUB + ((c0[i][m >> 2] >> (8 * (m & 3))) & 255u)];
#pragma unroll
                for (int m = 0; m < 16; ++m) s += tab[(16 + m) * KSUB + ((c1[i][m >> 2] >> (8 * (m & 3))) & 255u)];
                if (!ok[i]) {
                    bad = true;
                    s = -INFINITY;
                }
                oq[j] = s;
            }
        }
        if (bad) *err = 1;
        return;
    }
    __syncthreads();
    for (int j0 = beg + threadIdx.x; j0 < end + threadIdx.x; j0 += ADC_PER_ROUND) {
#pragma unroll
        for (int i = 0; i < ADC_PER_THREAD; ++i) {
            const int j = j0 + i * 256;
            if (j >= end) continue;
            const uint32_t id = cq[j];
            float s = -INFINITY;
            if (id < n) {
                const uint8_t *code = codes + (size_t)id * m_sub;
                s = 0.f;
                if ((m_sub & 15) == 0) {
                    for (int m0 = 0; m0 < m_sub; m0 += 16) {
                        const u32x4 w = *reinterpret_cast<const u32x4 *>(code + m0);
#pragma unroll
                        for (int m = 0; m < 16; ++m) s += tab[(m0 + m) * KSUB + ((w[m >> 2] >> (8 * (m & 3))) & 255u)];
                    }
                } else {
                    for (int m = 0; m < m_sub; ++m) s += tab[m * KSUB + code[m]];
                }
            } else {
                bad = true;
            }
            oq[j] = s;
        }
    }
    if (bad) *err = 1;
}

// Two blocks per CU, as many as stay there at once (four, one round after the other, pay the set-up twice: 173 us, not 162), each with a
// multiple of what its wavefronts take at once.  A multiple of 8 runs of rows is aimed at
// where there are rows enough, so that the XCDs get even shares (rounded down: up, 24 subspaces were 6 % slower); with fewer than
// 8 runs the subspaces are spread over the XCDs instead.  65536 rows of 384 subspaces of 2 elements take 1004 us per launch,
// 1000 rows of 192 subspaces of one 43; with a kernel of five instructions per value 1431 and 49, and 5358 and 129 where all
// subspaces of a run were on one XCD however few the runs (two in both cases).
void launch_assign(leann_ctx *ctx, const float *x, int64_t x_row, int64_t x_sub, int64_t n, int dsub, int m_sub, const float *codebook, uint8_t *out,
                   int64_t row_pitch, int64_t m_pitch)
{
    const int64_t want = std::max<int64_t>(8, 2 * ctx->num_cus / m_sub / 8 * 8);
    const int64_t rows = ((n + want - 1) / want + ASSIGN_THREADS - 1) / ASSIGN_THREADS * ASSIGN_THREADS;
    const int64_t runs = (n + rows - 1) / rows;
    const int xcd_bits = runs >= 8 ? 3 : 0;
    const int64_t blocks = ((((runs - 1) >> xcd_bits) + 1) << xcd_bits) * m_sub;
    auto *kernel = dsub <= 16 ? assign_kernel<1> : assign_kernel<2>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(ASSIGN_THREADS), assign_smem(dsub <= 16 ? 1 : 2, dsub),
                       ctx->stream, x, x_row, x_sub, n, dsub, m_sub, codebook, rows, xcd_bits, out, row_pitch, m_pitch);
}

// Launch shape of adc_kernel: enough blocks to fill the chip several times over, each with as large a share of its
// query's candidates as that allows.
void adc_launch_shape(int64_t nq, int nc, int *parts, int *per_block)
{
    const int rounds = (nc + ADC_PER_ROUND - 1) / ADC_PER_ROUND;
    const int64_t want_blocks = 256 * 64;  // blocks in the grid at least (when there is that much work): many short tails even out
    int64_t p = (want_blocks + nq - 1) / nq;
    if (p < 1) p = 1;
    if (p > rounds) p = rounds;
    const int rounds_per_block = (int)((rounds + p - 1) / p);
    *per_block = rounds_per_block * ADC_PER_ROUND;
    *parts = (rounds + rounds_per_block - 1) / rounds_per_block;
}

// The same permutation on the host.  Index: as narrow as n allows (the swaps are random reads
// and writes of the whole permutation).
template <class Index>
std::vector<int64_t> training_rows(int64_t n, int64_t nt, uint64_t seed)
{
    std::vector<Index> perm((size_t)n);
    for (int64_t i = 0; i < n; ++i) perm[i] = (Index)i;
    for (int64_t i = n - 1; i >= 1; --i) {
        const uint64_t j = splitmix64(seed) % (uint64_t)(i + 1);
        std::swap(perm[i], perm[j]);
    }
    return std::vector<int64_t>(perm.begin(), perm.begin() + nt);
}

int check_pq_shape(int64_t n, int32_t d, int32_t m_sub)
{
    if (n < 1 || d < 1 || m_sub < 1 || d % m_sub) {
        leann_set_error("PQ shape: n=%lld d=%d m_sub=%d (need d %% m_sub == 0)", (long long)n, d, m_sub);
        return LEANN_EINVAL;
    }
    if (d / m_sub > MAX_DSUB) {
        leann_set_error("PQ sub-vector length %d exceeds %d", d / m_sub, MAX_DSUB);
        return LEANN_ESHAPE;
    }
    return LEANN_OK;
}

int alloc_pq(leann_ctx *ctx, int64_t n, int32_t d, int32_t m_sub, bool own_codes, leann_pq **out)
{
    leann_pq *pq = new leann_pq();
    pq->n = n;
    pq->d = d;
    pq->m_sub = m_sub;
    pq->device = ctx->device;
    pq->owns_codes = own_codes;
    DevBuf codebook, codes;
    int rc = ctx->reserve(codebook, (size_t)m_sub * KSUB * (d / m_sub) * sizeof(float));
    if (rc == LEANN_OK && own_codes) rc = ctx->reserve(codes, (size_t)n * m_sub);
    pq->codebook = (float *)codebook.p;
    pq->codes = (uint8_t *)codes.p;
    if (rc != LEANN_OK) {
        leann_pq_free(pq);
        return rc;
    }
    *out = pq;
    return LEANN_OK;
}

// ---- workspace of leann_adc_noalloc: a fixed device array instead of a grown allocation.
// Layout: lookup tables fp32 [NOALLOC_MAX_QUERIES][m_sub][256] with m_sub * 256 * 4 <= NOALLOC_LUT_BYTES per query,
// then one 256-byte slot whose first int is the kernel's bad-id flag.  Every GPU the library runs on holds its own
// copy of the array until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; what kernels and copies get is the per-device address looked up below.
constexpr int NOALLOC_MAX_QUERIES = 128;
constexpr int NOALLOC_LUT_BYTES = 32 * KSUB * (int)sizeof(float);  // per query: up to 32 subspaces
constexpr size_t NOALLOC_FLAG_OFFSET = (size_t)NOALLOC_MAX_QUERIES * NOALLOC_LUT_BYTES;
static __device__ __align__(256) unsigned char scratch[NOALLOC_FLAG_OFFSET + 256];

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};  // device address of `scratch` on each device, 0 = not looked up yet

__global__ void clear_flag_kernel(int *flag) { *flag = 0; }

}  // namespace

int pq_init_device()
{
    LEANN_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(adc_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
    LEANN_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(assign_kernel<2>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, assign_smem(2, MAX_DSUB)));
    // once per device, with that device current (leann_create made it so): where this device keeps `scratch`
    int dev = -1;
    LEANN_HIP(hipGetDevice(&dev));
    if (dev >= 0 && dev < NOALLOC_MAX_DEVICES) {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void *ptr = nullptr;
            LEANN_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
            g_scratch_ptr[dev] = ptr;
        }
    }
    return LEANN_OK;
}

int pq_build_lut(leann_ctx *ctx, const float *queries_dev, int64_t nq, const leann_pq *pq, float *lut_dev)
{
    if (nq <= 0) return LEANN_OK;
    ProfScope prof(ctx, LEANN_PROF_LUT);
    launch_lut(ctx->stream, queries_dev, nq, pq, lut_dev);
    LEANN_HIP(hipGetLastError());
    return LEANN_OK;
}

extern "C" {

int leann_build_pq(leann_ctx *ctx, const float *emb_dev, int64_t n, int32_t d, int32_t m_sub, int32_t iters,
                   uint64_t seed, leann_pq **out)
{
    if (!ctx || !emb_dev || !out || iters < 0) {
        leann_set_error("leann_build_pq: null argument or negative iteration count");
        return LEANN_EINVAL;
    }
    LEANN_TRY(check_pq_shape(n, d, m_sub));
    LEANN_HIP(hipSetDevice(ctx->device));
    const int dsub = d / m_sub;
    const int64_t nt = n < MAX_TRAIN ? n : MAX_TRAIN;
    leann_pq *pq = nullptr;
    LEANN_TRY(alloc_pq(ctx, n, d, m_sub, true, &pq));
    // scratch: training rows | their copies | assignments | rows grouped by centroid | where each group starts | counts; before that, from the
    // copies on, the permutation's steps where they fit
    size_t off = 0;
    auto carve = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    const size_t o_rows = carve((size_t)nt * sizeof(int64_t)), o_xt = carve((size_t)nt * d * sizeof(float));
    const size_t o_assign = carve((size_t)nt * m_sub), o_order = carve((size_t)nt * m_sub * sizeof(int32_t));
    const size_t o_first = carve((size_t)m_sub * (KSUB + 1) * sizeof(int32_t));
    const size_t o_counts = carve((size_t)m_sub * GROUP_RUNS * KSUB * sizeof(int32_t));
    const size_t step_bytes = ((size_t)n * sizeof(uint32_t) + 255) & ~(size_t)255;
    auto fail = [&](int code) {
        leann_pq_free(pq);
        return code;
    };
    std::lock_guard<std::mutex> turn(ctx->pq_work_mutex);
    struct GiveBack {
        DevBuf &work;
        DevBuf steps;  // those that the scratch has no room for: nothing that grows with the table is kept
        ~GiveBack()
        {
            steps.release();
            if (work.bytes > PQ_WORK_KEEP) work.release();
        }
    } mem{ctx->pq_work, {}};
    if (ctx->pq_work.reserve(off) != LEANN_OK) return fail(LEANN_ENOMEM);
    // The steps take 16 bytes per row, beside rows of at least 4: on the host where that is more than a context ever keeps, or where the
    // device has no room; also where its loop is over before three more launches would be (whole calls of 384 dimensions,
    // 32 subspaces and 2 iterations, host and device: 1000 rows 168 and 176 us, 4000 rows 197 and 196, 6000 rows 223 and 215, 40 000 rows 560 and 463).
    const bool in_scratch = o_xt + 4 * step_bytes <= off;
    const bool on_device = n > 4096 && 4 * step_bytes <= PQ_WORK_KEEP && (in_scratch || mem.steps.reserve(4 * step_bytes) == LEANN_OK);
    unsigned char *scr = (unsigned char *)ctx->pq_work.p;
    int64_t *rows_dev = (int64_t *)(scr + o_rows);
    float *xt = (float *)(scr + o_xt);
    uint8_t *assign = scr + o_assign;
    int32_t *order = (int32_t *)(scr + o_order), *first = (int32_t *)(scr + o_first), *counts = (int32_t *)(scr + o_counts);
    std::vector<int64_t> train;  // read by the copy until the stream has been waited for
    if (on_device) {
        unsigned char *at = in_scratch ? scr + o_xt : (unsigned char *)mem.steps.p;
        auto steps = [&](int k) { return (uint32_t *)(at + k * step_bytes); };
        const Steps st = {steps(0), steps(1), steps(2), steps(3)};
        const dim3 all((unsigned)((n + 255) / 256)), some((unsigned)((nt + 255) / 256));
        hipLaunchKernelGGL(clear_steps_kernel, all, dim3(256), 0, ctx->stream, st, n);
        hipLaunchKernelGGL(draw_steps_kernel, all, dim3(256), 0, ctx->stream, st, n, seed);
        hipLaunchKernelGGL(training_rows_kernel, some, dim3(256), 0, ctx->stream, st, nt, rows_dev);
    } else {
        train = n <= 0xffffffffll ? training_rows<uint32_t>(n, nt, seed) : training_rows<int64_t>(n, nt, seed);
        if (hipMemcpyAsync(rows_dev, train.data(), (size_t)nt * sizeof(int64_t), hipMemcpyHostToDevice, ctx->stream) != hipSuccess)
            return fail(LEANN_EDEVICE);
    }
    const bool by_four = (dsub & 3) == 0 && (reinterpret_cast<uintptr_t>(emb_dev) & 15) == 0;
    hipLaunchKernelGGL(by_four ? gather_rows_kernel<f32x4> : gather_rows_kernel<float>, dim3((unsigned)((nt + GATHER_ROWS - 1) / GATHER_ROWS)),
                       dim3(256), 0, ctx->stream, emb_dev, rows_dev, nt, d, dsub, xt);
    hipLaunchKernelGGL(first_centroids_kernel, dim3(KSUB, m_sub), dim3(64), 0, ctx->stream, xt, nt, dsub, pq->codebook);
    const int xcd_bits = m_sub % 8 == 0 ? 3 : 0;  // other numbers of subspaces would not spread evenly over the XCDs
    for (int it = 0; it < iters; ++it) {
        launch_assign(ctx, xt, dsub, nt * dsub, nt, dsub, m_sub, pq->codebook, assign, 1, nt);
        hipLaunchKernelGGL(count_rows_kernel, dim3(m_sub, GROUP_BLOCKS), dim3(1024), 0, ctx->stream, assign, (int)nt, counts);
        hipLaunchKernelGGL(group_rows_kernel, dim3(m_sub, GROUP_BLOCKS), dim3(1024), 0, ctx->stream, assign, (int)nt, counts, order,
                           first);
        hipLaunchKernelGGL(update_kernel, dim3(KSUB * m_sub), dim3(256), (size_t)256 * dsub * sizeof(float), ctx->stream, xt, nt, dsub, xcd_bits,
                           order, first, pq->codebook);
    }
    launch_assign(ctx, emb_dev, d, dsub, n, dsub, m_sub, pq->codebook, pq->codes, m_sub, 1);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(ctx->stream) != hipSuccess) {
        leann_set_error("PQ training kernels failed");
        return fail(LEANN_EDEVICE);
    }
    *out = pq;
    return LEANN_OK;
}

int leann_pq_export(leann_ctx *ctx, const leann_pq *pq, float *codebook_host, uint8_t *codes_host)
{
    if (!ctx || !pq) {
        leann_set_error("leann_pq_export: null handle");
        return LEANN_EINVAL;
    }
    LEANN_HIP(hipSetDevice(ctx->device));
    LEANN_HIP(hipStreamSynchronize(ctx->stream));
    if (codebook_host)
        LEANN_HIP(hipMemcpy(codebook_host, pq->codebook, (size_t)pq->m_sub * KSUB * (pq->d / pq->m_sub) * sizeof(float),
                            hipMemcpyDeviceToHost));
    if (codes_host) LEANN_HIP(hipMemcpy(codes_host, pq->codes, (size_t)pq->n * pq->m_sub, hipMemcpyDeviceToHost));
    return LEANN_OK;
}

int leann_pq_import(leann_ctx *ctx, const float *codebook_host, const uint8_t *codes_host, int64_t n, int32_t d,
                    int32_t m_sub, leann_pq **out)
{
    if (!ctx || !codebook_host || !codes_host || !out) {
        leann_set_error("leann_pq_import: null argument");
        return LEANN_EINVAL;
    }
    LEANN_TRY(check_pq_shape(n, d, m_sub));
    LEANN_HIP(hipSetDevice(ctx->device));
    leann_pq *pq = nullptr;
    LEANN_TRY(alloc_pq(ctx, n, d, m_sub, true, &pq));
    if (hipMemcpy(pq->codebook, codebook_host, (size_t)m_sub * KSUB * (d / m_sub) * sizeof(float),
                  hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(pq->codes, codes_host, (size_t)n * m_sub, hipMemcpyHostToDevice) != hipSuccess) {
        leann_set_error("copying the PQ table to the device failed");
        leann_pq_free(pq);
        return LEANN_EDEVICE;
    }
    *out = pq;
    return LEANN_OK;
}

int leann_pq_wrap(leann_ctx *ctx, const float *codebook_host, const uint8_t *codes_dev, int64_t n, int32_t d,
                  int32_t m_sub, leann_pq **out)
{
    if (!ctx || !codebook_host || !codes_dev || !out) {
        leann_set_error("leann_pq_wrap: null argument");
        return LEANN_EINVAL;
    }
    LEANN_TRY(check_pq_shape(n, d, m_sub));
    LEANN_HIP(hipSetDevice(ctx->device));
    leann_pq *pq = nullptr;
    LEANN_TRY(alloc_pq(ctx, n, d, m_sub, false, &pq));
    pq->codes = const_cast<uint8_t *>(codes_dev);
    if (hipMemcpy(pq->codebook, codebook_host, (size_t)m_sub * KSUB * (d / m_sub) * sizeof(float),
                  hipMemcpyHostToDevice) != hipSuccess) {
        leann_set_error("copying the codebook to the device failed");
        leann_pq_free(pq);
        return LEANN_EDEVICE;
    }
    *out = pq;
    return LEANN_OK;
}

int leann_pq_info(const leann_pq *pq, int64_t *n, int32_t *d, int32_t *m_sub)
{
    if (!pq) {
        leann_set_error("leann_pq_info: null handle");
        return LEANN_EINVAL;
    }
    if (n) *n = pq->n;
    if (d) *d = pq->d;
    if (m_sub) *m_sub = pq->m_sub;
    return LEANN_OK;
}

void leann_pq_free(leann_pq *pq)
{
    if (!pq) return;
    (void)hipFree(pq->codebook);
    if (pq->owns_codes) (void)hipFree(pq->codes);
    delete pq;
}

int leann_adc(leann_ctx *ctx, const float *queries_dev, int64_t nq, const leann_pq *pq, const uint32_t *cand_ids_dev,
              int32_t nc, float *out_dev)
{
    if (!ctx || !queries_dev || !pq || !cand_ids_dev || !out_dev || nq < 0 || nc < 0) {
        leann_set_error("leann_adc: null argument or negative count");
        return LEANN_EINVAL;
    }
    if (nq == 0 || nc == 0) return LEANN_OK;
    LEANN_HIP(hipSetDevice(ctx->device));
    const int smem = pq->m_sub * KSUB * (int)sizeof(float);
    if (smem > 96 * 1024) {
        leann_set_error("lookup table of %d bytes does not fit the ADC kernel's LDS budget", smem);
        return LEANN_ESHAPE;
    }
    LEANN_TRY(clear_host_flags(ctx));
    int *flag = ctx->host_flags + FLAG_CANDIDATE;
    // A lookup table holds 256 entries per subspace: for fewer candidates than that, and few enough of them in all that
    // launches and not work are what counts, computing the entries that are used is less of both (d = 768, 32 subspaces,
    // whole call: one query, 64 candidates 18 us, with a table 23; 64 x 64 20 and 31 us; 128 x 128 29 us, 256 x 128
    // with a table 34).
    if (nc <= KSUB && nq * nc <= ADC_DIRECT_MAX) {
        ProfScope prof(ctx, LEANN_PROF_ADC);
        hipLaunchKernelGGL(adc_direct_kernel, dim3((unsigned)nq, (nc + DIRECT_CAND - 1) / DIRECT_CAND), dim3(256),
                           DIRECT_CAND * (pq->m_sub | 1) * sizeof(float), ctx->stream,
                           DirectArgs{queries_dev, pq->codebook, pq->codes, cand_ids_dev, out_dev, flag, pq->n, pq->d, pq->m_sub, nc});
    } else {
        LEANN_TRY(ctx->reserve(ctx->s_lut, (size_t)nq * pq->m_sub * KSUB * sizeof(float)));
        LEANN_TRY(pq_build_lut(ctx, queries_dev, nq, pq, (float *)ctx->s_lut.p));
        ProfScope prof(ctx, LEANN_PROF_ADC);
        int parts = 1, per_block = ADC_PER_ROUND;
        adc_launch_shape(nq, nc, &parts, &per_block);
        hipLaunchKernelGGL(adc_kernel, dim3((unsigned)nq, parts), dim3(256), smem, ctx->stream,
                           (const float *)ctx->s_lut.p, pq->codes, pq->n, pq->m_sub, cand_ids_dev, nc, per_block, out_dev,
                           flag);
    }
    LEANN_HIP(hipGetLastError());
    LEANN_HIP(hipStreamSynchronize(ctx->stream));
    if (*(volatile int *)flag) {
        leann_set_error("leann_adc: candidate id outside [0, n)");
        return LEANN_EINVAL;
    }
    return LEANN_OK;
}

int leann_adc_noalloc(leann_ctx *ctx, const float *queries_dev, int64_t nq, const leann_pq *pq,
                      const uint32_t *cand_ids_dev, int32_t nc, float *out_dev)
{
    if (!ctx || !queries_dev || !pq || !cand_ids_dev || !out_dev || nq < 0 || nc < 0) {
        leann_set_error("leann_adc_noalloc: null argument or negative count");
        return LEANN_EINVAL;
    }
    const int smem = pq->m_sub * KSUB * (int)sizeof(float);
    if (nq > NOALLOC_MAX_QUERIES || smem > NOALLOC_LUT_BYTES) {
        leann_set_error("leann_adc_noalloc: %lld queries x %d subspaces exceed the fixed workspace (at most %d queries, "
                        "%d subspaces); use leann_adc", (long long)nq, pq->m_sub, NOALLOC_MAX_QUERIES,
                        NOALLOC_LUT_BYTES / (KSUB * (int)sizeof(float)));
        return LEANN_ECAPACITY;
    }
    if (ctx->device < 0 || ctx->device >= NOALLOC_MAX_DEVICES || !g_scratch_ptr[ctx->device]) {
        leann_set_error("leann_adc_noalloc: no fixed workspace was set up for device %d", ctx->device);
        return LEANN_EDEVICE;
    }
    if (nq == 0 || nc == 0) return LEANN_OK;
    LEANN_HIP(hipSetDevice(ctx->device));
    unsigned char *base = static_cast<unsigned char *>(g_scratch_ptr[ctx->device]);
    float *lut = reinterpret_cast<float *>(base);
    int *flag = reinterpret_cast<int *>(base + NOALLOC_FLAG_OFFSET);
    // the array keeps the last call's contents: the flag starts at zero (a kernel, not a memset, so that the call
    // can be recorded into a graph); the tables are overwritten for exactly the queries that are read
    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, ctx->stream, flag);
    launch_lut(ctx->stream, queries_dev, nq, pq, lut);
    int parts = 1, per_block = ADC_PER_ROUND;
    adc_launch_shape(nq, nc, &parts, &per_block);
    hipLaunchKernelGGL(adc_kernel, dim3((unsigned)nq, parts), dim3(256), smem, ctx->stream, (const float *)lut, pq->codes,
                       pq->n, pq->m_sub, cand_ids_dev, nc, per_block, out_dev, flag);
    LEANN_HIP(hipGetLastError());
    return LEANN_OK;
}

}  // extern "C"
