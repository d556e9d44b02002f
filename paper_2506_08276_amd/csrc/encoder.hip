// Encoder forward pass for embedding recomputation (LEANN Alg. 2, the recomputation step; Sec. 3 online
// stage), written for gfx950: bf16 MFMA GEMMs with LDS-staged, swizzled tiles, an MFMA attention kernel
// working on ragged (token-packed) batches, and fp32 LayerNorm / pooling.
//
// Tokens of all chunks of a pass are packed back to back (no padding rows): chunk i owns rows
// cu[i] .. cu[i+1] of every activation matrix (in planes of 32 columns, see gemm.h).  The number of valid rows T is only known on the device,
// so grids are sized for the worst case and blocks beyond T leave at once.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm.h"
#include "gemm_large.h"
#include "gemm_plan.h"
#include "gemm_stream.h"
#include "wave.h"

namespace {

// ------------------------------------------------------------------ pass set-up
// lengths of the requested chunks -> exclusive prefix sum cu[0..n], cu[n] = T.  One block of 1024 threads, or of PREP_FEW for up to
// as many chunks: a wavefront's scan without barriers, in the passes where a microsecond counts.
constexpr int PREP_FEW = 64;

__global__ __launch_bounds__(1024) void prep_kernel(const int32_t *__restrict__ lengths, const int64_t *__restrict__ ids,
                                                    int64_t first_id, int n, int64_t n_store, int seq,
                                                    int32_t *__restrict__ cu, int64_t *__restrict__ chunk_of,
                                                    int *__restrict__ err, int64_t *__restrict__ tok_count,
                                                    int64_t *__restrict__ tok_count2, bool report)
{
    __shared__ int part[1024];
    const int tid = threadIdx.x;
    auto chunk_length = [&](int i) -> int {
        int64_t id = ids ? ids[i] : first_id + i;
        int len = 0;
        if (id < 0 || id >= n_store) {
            err[FLAG_CHUNK_ID] = 1;
            id = 0;
        } else {
            len = lengths[id];
            if (len < 1 || len > seq) {
                err[FLAG_LENGTH] = 1;
                len = 0;
            }
        }
        chunk_of[i] = id;
        return len;
    };
    if (n <= PREP_FEW) {
        const int len = tid < n ? chunk_length(tid) : 0;
        int up_to = len;
#pragma unroll
        for (int o = 1; o < PREP_FEW; o <<= 1) {
            const int before = __shfl_up(up_to, o, 64);
            if (tid >= o) up_to += before;
        }
        if (tid < n) cu[tid] = up_to - len;
        if (tid == n - 1) {
            cu[n] = up_to;
            if (report) err[PASS_TOKENS] = up_to;
            if (tok_count) *tok_count += up_to;
            if (tok_count2) *tok_count2 += up_to;
        }
        return;
    }
    const int per = (n + 1023) / 1024;
    const int beg = tid * per, end = min(n, beg + per);
    int s = 0;
    for (int i = beg; i < end; ++i) {
        const int len = chunk_length(i);
        cu[i] = len;  // temporarily the length
        s += len;
    }
    part[tid] = s;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        int v = tid >= o ? part[tid - o] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int run = tid ? part[tid - 1] : 0;
    for (int i = beg; i < end; ++i) {
        int len = cu[i];
        cu[i] = run;
        run += len;
    }
    if (tid == 1023) {
        cu[n] = part[1023];
        if (report) err[PASS_TOKENS] = part[1023];
        if (tok_count) *tok_count += part[1023];
        if (tok_count2) *tok_count2 += part[1023];
    }
}

// ------------------------------------------------------------------ embedding + LayerNorm
// one wave per (chunk, position); x[cu[i]+t] = LN(tok_emb[id] + pos_emb[t] + seg_emb) in bf16
__global__ __launch_bounds__(256) void embed_ln_kernel(const int32_t *__restrict__ tokens, const int64_t *__restrict__ chunk_of,
                                                       const int32_t *__restrict__ cu, int n, int seq, int d, int vocab,
                                                       const bf16_t *__restrict__ tok_emb, const bf16_t *__restrict__ pos_emb,
                                                       const bf16_t *__restrict__ seg_emb, const float *__restrict__ g,
                                                       const float *__restrict__ b, float eps, bf16_t *__restrict__ x,
                                                       int plane, int *__restrict__ err)
{
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int i = (int)(w / seq), t = (int)(w % seq);
    if (i >= n) return;
    const int row0 = cu[i], len = cu[i + 1] - row0;
    if (t >= len) return;
    int tok = tokens[chunk_of[i] * seq + t];
    if (tok < 0 || tok >= vocab) {
        if (lane == 0) err[FLAG_TOKEN] = 1;
        tok = 0;
    }
    // a lane owns 16-byte pieces (8 elements) j*64 + lane of the row
    const int pieces = d >> 3;
    const bf16_t *te = tok_emb + (size_t)tok * d, *pe = pos_emb + (size_t)t * d;
    float v[2][8];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (j * 64 + lane < pieces) {
            const int c0 = (j * 64 + lane) * 8;
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(te + c0);
            const bf16x8 p = *reinterpret_cast<const bf16x8 *>(pe + c0);
            const bf16x8 sg = *reinterpret_cast<const bf16x8 *>(seg_emb + c0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[j][i] = (float)a[i] + (float)p[i] + (float)sg[i];
                s += v[j][i];
            }
        }
    const float mean = wave_sum(s) / (float)d;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (j * 64 + lane < pieces) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float c = v[j][i] - mean;
                q += c * c;
            }
        }
    const float inv = 1.0f / sqrtf(wave_sum(q) / (float)d + eps);
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (j * 64 + lane < pieces) {
            const int c0 = (j * 64 + lane) * 8;
            const f32x4 g0 = *reinterpret_cast<const f32x4 *>(g + c0), g1 = *reinterpret_cast<const f32x4 *>(g + c0 + 4);
            const f32x4 b0 = *reinterpret_cast<const f32x4 *>(b + c0), b1 = *reinterpret_cast<const f32x4 *>(b + c0 + 4);
            bf16x8 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                o[i] = (bf16_t)((v[j][i] - mean) * inv * g0[i] + b0[i]);
                o[i + 4] = (bf16_t)((v[j][i + 4] - mean) * inv * g1[i] + b1[i]);
            }
            *reinterpret_cast<bf16x8 *>(x + plane_at(c0, row0 + t, plane)) = o;
        }
}

// ------------------------------------------------------------------ residual add + LayerNorm, in place
// x[row] = LN(x[row] + delta[row]): delta is a sublayer's output (bf16, written by the O / FFN2 GEMM), the sum, the
// statistics and the normalisation are fp32.  The rows of a wave are in its registers before anything is written.  Two-pass statistics on
// the registers: mean, then the biased variance of the centred values.
// A row's sum is defined on its 16-byte pieces p (8 elements, at most 128): 64 sums of the elements of the pieces l and l + 64 in order, then pairwise over
// l ^ 32, 16, 8, 4, 2, 1.
//  - Small passes (EARLY, see ln_few_rows), which are nothing but this chain of latencies: a wave takes one row, lane l the pieces l and l + 64.  The
//    first row is requested before the token count is there (the buffers reach past the last block's rows); with many rows per wavefront that
//    order costs 3 % of the bandwidth.
//  - Large ones: a wave takes a pair of rows, 2p and 2p + 1, whose pieces of a plane are one 128-byte line, eight lanes of 16 bytes; lane bit 2
//    tells the row, and the lane's other bits, q, that it has the pieces q, q + 32, q + 64 and q + 96: the sums l = q and q + 32.  An odd
//    last row's neighbour is normalised too and means nothing (the buffers reach past it).
// PIECES: of a lane, as many as rows of up to 512 (EARLY) or 256 elements per piece need.
template <bool EARLY>
__device__ inline float row_sum(float s0, float s1)  // large passes: s0 of the sums l = q, s1 of q + 32; in all lanes of the row
{
    if constexpr (EARLY) {
        return wave_sum(s0);
    } else {
        float v = s0 + s1;
        {
            const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
        }
        {
            const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
        }
        v += __uint_as_float(dpp_mov<DPP_ROW_ROR8>(__float_as_uint(v)));
        v += __uint_as_float(dpp_mov<DPP_QUAD_XOR2>(__float_as_uint(v)));
        v += __uint_as_float(dpp_mov<DPP_QUAD_XOR1>(__float_as_uint(v)));
        return v;
    }
}

template <int PIECES, bool EARLY>
__global__ __launch_bounds__(256) void ln_kernel(const bf16_t *__restrict__ delta, const float *__restrict__ g,
                                                 const float *__restrict__ b, bf16_t *__restrict__ x,
                                                 const int32_t *__restrict__ T_dev, int d, int plane, float eps, int nwaves)
{
    constexpr int ROWS = EARLY ? 1 : 2, SUMS = EARLY ? 1 : 2;  // rows of a wave, sums of a lane
    const int lane = threadIdx.x & 63;
    const int planes = d / PLANE, plane0 = EARLY ? lane >> 2 : lane >> 3, apart = EARLY ? 16 : 8;  // planes of a lane: plane0, plane0 + apart, ..
    int at = blockIdx.x * 4 + (threadIdx.x >> 6);  // row or pair
    int T = 0;
    if constexpr (!EARLY) {
        T = *T_dev;
        if (ROWS * at >= T) return;
    }
    // a wave goes through rows or pairs at, at + nwaves, ...: the scale and shift of its pieces stay in registers, and the
    // next one's loads are issued before the current one's arithmetic (nwaves, of the grid, is an argument: as the grid's it is read from memory)
    f32x4 gg[PIECES][2], bb[PIECES][2];
    bf16x8 dn[PIECES], xn[PIECES];
    const size_t step = (size_t)apart * plane;  // between a lane's pieces
    const size_t lane_at = (size_t)plane0 * plane + (EARLY ? lane & 3 : lane & 7) * 8;
    auto on = [&](int j) { return j * apart + plane0 < planes; };
#pragma unroll
    for (int j = 0; j < PIECES; ++j)
        if (on(j)) {
            const int c0 = (j * apart + plane0) * PLANE + (lane & 3) * 8;
            gg[j][0] = *reinterpret_cast<const f32x4 *>(g + c0);
            gg[j][1] = *reinterpret_cast<const f32x4 *>(g + c0 + 4);
            bb[j][0] = *reinterpret_cast<const f32x4 *>(b + c0);
            bb[j][1] = *reinterpret_cast<const f32x4 *>(b + c0 + 4);
            const size_t o = lane_at + j * step + (size_t)at * (ROWS * PLANE);
            dn[j] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(delta + o));
            xn[j] = *reinterpret_cast<const bf16x8 *>(x + o);
        }
    if constexpr (EARLY) T = *T_dev;
    for (; ROWS * at < T; at += nwaves) {
        float v[PIECES][8], s[2] = {0.f, 0.f};
#pragma unroll
        for (int j = 0; j < PIECES; ++j)
            if (on(j)) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    v[j][i] = (float)xn[j][i] + (float)dn[j][i];
                    s[j % SUMS] += v[j][i];
                }
            }
        const int next = at + nwaves;
        if (ROWS * next < T) {
#pragma unroll
            for (int j = 0; j < PIECES; ++j)
                if (on(j)) {
                    const size_t o = lane_at + j * step + (size_t)next * (ROWS * PLANE);
                    dn[j] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(delta + o));
                    xn[j] = *reinterpret_cast<const bf16x8 *>(x + o);
                }
        }
        const float mean = row_sum<EARLY>(s[0], s[1]) / (float)d;
        float q[2] = {0.f, 0.f};  // fused where it says so: every variant of the kernel has to round alike
#pragma unroll
        for (int j = 0; j < PIECES; ++j)
            if (on(j)) {
                float &sq = q[j % SUMS];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[j][i] -= mean;
                if (j < SUMS) sq = fmaf(v[j][0], v[j][0], v[j][1] * v[j][1]);
                else sq = fmaf(v[j][1], v[j][1], fmaf(v[j][0], v[j][0], sq));
#pragma unroll
                for (int i = 2; i < 8; ++i) sq = fmaf(v[j][i], v[j][i], sq);
            }
        const float inv = 1.0f / sqrtf(row_sum<EARLY>(q[0], q[1]) / (float)d + eps);
#pragma unroll
        for (int j = 0; j < PIECES; ++j)
            if (on(j)) {
                bf16x8 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    o[i] = (bf16_t)fmaf(v[j][i] * inv, gg[j][0][i], bb[j][0][i]);
                    o[i + 4] = (bf16_t)fmaf(v[j][i + 4] * inv, gg[j][1][i], bb[j][1][i]);
                }
                *reinterpret_cast<bf16x8 *>(x + lane_at + j * step + (size_t)at * (ROWS * PLANE)) = o;
            }
    }
}

// Whether a pass has its rows one per wave.  Twice as many waves with half as long a chain, until the chip has more rows than it hides; rows of up to 256
// elements leave half of a wave idle that has one alone.  Whole passes of twelve layers, one row and a pair per wave, microseconds
// (tokens: 2000, 3600, 5000, 6600, 8200):
//     128 columns   +2    +5    +7    +6   +15  of 400 to 600         512 columns   -7    -9    -8    -2   +15  of 600 to 1500
//     256           +4    +5   +10   +12   +12                        768          -10   -10   -11    -1    +5  of 800 to 2200
//     384           -6   -11    -9    -7    -2  of 490 to 930        1024          -28   -13   -23    -7    +9
bool ln_few_rows(int d, int rows) { return rows <= (d <= 256 ? 2048 : d <= 384 ? 7168 : 5120); }

auto ln_kernel_for(int d, bool early)  // leann_create takes rows of up to 1024 elements
{
    if (early) return d <= 512 ? ln_kernel<1, true> : ln_kernel<2, true>;
    switch ((d + 255) / 256) {
    case 1: return ln_kernel<1, false>;
    case 2: return ln_kernel<2, false>;
    case 3: return ln_kernel<3, false>;
    default: return ln_kernel<4, false>;
    }
}

// ------------------------------------------------------------------ attention
// One block per (chunk, head), head size 64, up to 256 keys.  K (row-major, swizzled) and V^T live in LDS.
// Each wave takes 32 query rows and computes S^T = K Q^T with MFMA, so that a lane owns one
// query column: the softmax reductions run over the lane's own registers plus one exchange with lane^32.
// P^T (bf16) then feeds O^T = V^T P^T directly from registers: accumulator registers 8u..8u+7 of key tile t
// are exactly the eight k-slots of one MFMA step when V^T is read with the matching key order.
// NW = wavefronts, one per 32 query rows and 32 keys the block can hold: 4 for sequences up to 128, 8 for up to 256.
// The scores are computed twice, once for the maxima and once tile by tile for the rest: the matrix cores have the time, and a
// wavefront that does not hold the scores of 256 keys (128 registers) leaves room for three more on its SIMD, so that every 32
// queries have their own.  It also makes the key tiles loops (4.9 KB of code; unrolled 12.8), which counts in passes of few chunks,
// whose every launch fetches its code anew.  Per launch, before and now: one chunk of 80 tokens 5.8 and 5.0 us, 13 chunks 5.9 and
// 5.3, 300 x 160 tokens of 384 elements 49.5 and 43, 2048 x 160 tokens of 768 605 and 542 (3.7 TB/s of the 4.8 that a copy reaches;
// two blocks' loads and arithmetic take turns on a CU).
template <int NW>
struct AttCfg {
    static constexpr int LP = NW * 32;            // padded key capacity = V^T row pitch (bf16)
    static constexpr int KV_BYTES = (LP * 64 + 64 * LP) * (int)sizeof(bf16_t);
    static constexpr int SMEM = KV_BYTES + NW * 16 * 128;  // plus, per wave, 16 output rows of 64 bf16
};

// V^T in LDS: row = output dimension (64 of them), LP keys per row in 16-byte groups of eight.  Inside a group of 16
// keys the order follows the MFMA operand slots of P^T (a lane of half h holds, in slots 0..7, keys 4h + 0..3 and
// 8 + 4h + 0..3): stored position 16j + 8h + slot, so that a lane's operand is one 16-byte read.  The group index is
// XORed with a function of the row: the 16 rows that one pass of a 16-byte read serves, and the (chunk, half) pairs
// that one pass of the staging stores serves, then fall into 16 different bank groups (no bank conflicts either way).
__device__ inline int vt_swizzle(int row) { return (row & 15) ^ (((row >> 4) & 3) << 1); }

// K in LDS: 16 rows' reads of one chunk reach all banks, and so do stores of four chunks of four rows.
__device__ inline int k_swizzle(int row) { return ((row >> 1) & 1) << 2 | ((row >> 2) & 3); }

template <int NW>
__global__ __launch_bounds__(64 * NW, 4) void attention_kernel(const bf16_t *__restrict__ qkv, const int32_t *__restrict__ cu,
                                                               bf16_t *__restrict__ out, int d, int plane, float scale_log2e)
{
    constexpr int LP = AttCfg<NW>::LP;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    bf16_t *Ks = reinterpret_cast<bf16_t *>(smem);  // [LP][64], 16-byte chunks XOR-swizzled by row
    bf16_t *Vt = Ks + LP * 64;                      // [64][LP], see vt_swizzle
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive blocks are the heads of one chunk; a head's queries, keys and values of a chunk are two runs of memory each
    const int H = d >> 6;
    const int c = blockIdx.x / H, h = blockIdx.x % H;
    const int t0 = cu[c], L = cu[c + 1] - t0;
    if (L <= 0) return;
    const int nkt = (L + 31) >> 5;
    const int Lp = nkt << 5;
    const int half = lane >> 5, l32 = lane & 31;
    const int qb = wave, qrow = qb * 32 + l32;

    // Staging.  Half of the wavefronts bring V, half K, each 128 keys of one plane; all global loads of a thread are issued before its first
    // LDS store.  Of K and V the chunk's rows and no more: reads of keys >= L bring zeros.  With a test per read the compiled code waited twice
    // for all earlier ones in between, half a microsecond each.
    // V: thread (j16, hf, ch) takes the eight keys 16 j16 + 4 hf + {0..3, 8..11} of the 16-byte chunk ch (eight
    // output dimensions) and writes, per dimension, the eight keys as one 16-byte group.  j16 and hf are spread over the lanes so that 16 of them
    // store to all banks.
    // K: rows as they are, 16-byte chunk ch of row key at position ch ^ k_swizzle(key).
    constexpr int row_bytes = PLANE * (int)sizeof(bf16_t);
    const bool brings_v = wave < NW / 2;
    const int part = wave & (NW / 2 - 1), which = part & 1, ch = which * 4 + (lane & 3), keys0 = (part >> 1) * 128;
    const int hf = (lane >> 2) & 1, j16 = (keys0 >> 4) + ((lane >> 5) & 1) * 4 + ((lane >> 3) & 1) * 2 + ((lane >> 4) & 1);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(qkv + plane_at((brings_v ? 2 : 1) * d + h * 64 + which * PLANE, t0, plane)), 0,
                                                        L * row_bytes, 0x00020000);
    u32x4 in[8];
    {
        // V: rows key0 + {0..3, 8..11}; K: rows key0 + 16 r
        const int key0 = brings_v ? j16 * 16 + 4 * hf : keys0 + (lane >> 2), step = brings_v ? 1 : 16, step4 = brings_v ? 8 : 64;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            in[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (key0 + (r & 3) * step + (r >> 2) * step4) * row_bytes + (lane & 3) * 16, 0, 0));
    }
    // the wave's query rows go to registers while K and V are on their way to LDS
    bf16x8 qf[4];
    {
        const bf16_t *qp = qkv + plane_at(h * 64, t0, plane) + min(qrow, L - 1) * PLANE + half * 8;
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[s] = *reinterpret_cast<const bf16x8 *>(qp + (s >> 1) * (size_t)plane + (s & 1) * 16);
    }
    if (!brings_v) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int key = keys0 + (lane >> 2) + 16 * r;
            if (key < Lp) *reinterpret_cast<u32x4 *>(Ks + key * 64 + ((ch ^ k_swizzle(key)) << 3)) = in[r];
        }
    } else if (j16 * 16 < Lp) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {  // output dimension ch * 8 + i: element i of each of the eight key rows
            u32x4 o;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t a = in[2 * w][i >> 1], b = in[2 * w + 1][i >> 1];
                o[w] = (i & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
            }
            const int row = ch * 8 + i;
            *reinterpret_cast<u32x4 *>(Vt + row * LP + (((2 * j16 + hf) ^ vt_swizzle(row)) << 3)) = o;
        }
    }
    __syncthreads();
    if (qb >= nkt) return;

    const int kswz = k_swizzle(l32);  // rows 32 apart share it
    bf16x8 kf[4];
    auto read_k = [&](int t) {
#pragma unroll
        for (int s = 0; s < 4; ++s) kf[s] = *reinterpret_cast<const bf16x8 *>(Ks + (t * 32 + l32) * 64 + (((s * 2 + half) ^ kswz) << 3));
    };
    // Scores of key tile t, whose rows are in kf; then kf holds tile `next`.  The lane owns query column l32 and keys
    // 32t + 8(r/4) + 4*half + r%4; only the last tile can hold keys >= L.
    auto scores = [&](int t, int next) -> f32x16 {
        f32x16 sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], sc, 0, 0, 0);
        read_k(next);
        if (t == nkt - 1) {
            const int keys = L - t * 32 - 4 * half;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) >= keys) sc[r] = -INFINITY;
        }
        return sc;
    };
    read_k(0);
    float mx = -INFINITY;
#pragma unroll 1
    for (int t = 0; t < nkt; ++t) {
        const f32x16 sc = scores(t, t + 1 < nkt ? t + 1 : 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float moff = mx * scale_log2e;
    float den = 0.f;
    f32x16 oacc[2];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
#pragma unroll 1
    for (int t = 0; t < nkt; ++t) {
        f32x16 sc = scores(t, t + 1 < nkt ? t + 1 : 0);
        bf16x8 vf[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                const int pg = 4 * t + 2 * u + half;  // the lane's group: slots 0..3 = keys 32t + 16u + 4 half + 0..3, slots 4..7 = those + 8
                const int row = dt * 32 + l32;
                vf[u][dt] = *reinterpret_cast<const bf16x8 *>(Vt + row * LP + ((pg ^ vt_swizzle(row)) << 3));
            }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = __builtin_amdgcn_exp2f(sc[r] * scale_log2e - moff);  // argument <= 0: no overflow, underflow to 0 is exact enough
            sc[r] = p;
            den += p;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            bf16x8 pf;
#pragma unroll
            for (int i = 0; i < 8; ++i) pf[i] = (bf16_t)sc[8 * u + i];
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u][dt], pf, oacc[dt], 0, 0, 0);
        }
    }
    den += __shfl_xor(den, 32, 64);

    // The lane owns query l32 and, per (dt, g), the four adjacent outputs dt*32 + 8g + 4*half + 0..3.  Sixteen
    // queries at a time go through the wave's own 2 KB of LDS (8-byte unit u of a row at position u ^ swz(row):
    // the 16 lanes served together hit all banks once), so that the global stores are 16 bytes per lane and
    // eight adjacent rows in two planes (stores of 8 bytes per lane to 32 rows cost a quarter of the kernel's time).
    const float inv = 1.0f / den;
    unsigned char *ostg = smem + AttCfg<NW>::KV_BYTES + wave * (16 * 128);
    const int r16 = l32 & 15;
    const int wswz = ((r16 & 7) << 1) | (r16 >> 3);
    const int orow = lane >> 3, och = lane & 7;
    bf16_t *to = out + plane_at(h * 64, t0, plane) + (size_t)(och >> 2) * plane + (och & 3) * 8;
#pragma unroll
    for (int hp = 0; hp < 2; ++hp) {
        if ((l32 >> 4) == hp) {
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    bf16x4 o4;
#pragma unroll
                    for (int i = 0; i < 4; ++i) o4[i] = (bf16_t)(oacc[dt][4 * g + i] * inv);
                    const int u = dt * 8 + 2 * g + half;
                    *reinterpret_cast<bf16x4 *>(ostg + r16 * 128 + ((u ^ wswz) << 3)) = o4;
                }
        }
        __builtin_amdgcn_wave_barrier();  // LDS serves a wave's accesses in order
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lr = j * 8 + orow, q = qb * 32 + hp * 16 + lr;
            u32x4 v = *reinterpret_cast<const u32x4 *>(ostg + lr * 128 + ((och ^ orow) << 4));
            if (j & 1) v = u32x4{v[2], v[3], v[0], v[1]};  // rows 8..15 hold the halves of a chunk swapped
            if (q < L) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(to + q * PLANE));
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ------------------------------------------------------------------ masked mean pool + L2 normalise
// One block per chunk.  Partial sum p of a column is of the rows p, p + 4, ... in order, then the four are added in order: the result does
// not depend on anything but the chunk.  A wavefront reads pairs of adjacent rows, 16 bytes per lane (lane bit 2 tells which: whole lines where a chunk
// begins at an even row): wavefronts 0 and 2 the rows of partial sums 0 and 1, the others those of 2 and 3; 0 and 1 the first half of the planes, 8
// of them per access, 2 and 3 the others.
constexpr int POOL_AHEAD = 8;

template <int J>  // accesses per pair of rows and half: rows of up to 512 J elements
__global__ __launch_bounds__(256) void pool_kernel(const bf16_t *__restrict__ x, const int32_t *__restrict__ cu, int d, int plane,
                                                   float *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) float part[4][1024];
    __shared__ float red[256];
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = cu[c], L = cu[c + 1] - t0;
    const int planes = d / PLANE / 2, mine = (wave & 1) * 2 + ((lane >> 2) & 1), plane0 = (wave >> 1) * planes;
    float acc[J][8];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[j][i] = 0.f;
    // POOL_AHEAD rows of a lane are in flight, then added in order.  Rows past the end and planes past the last one are read from the last
    // and not used: a test per read would have every read wait for the one before.
    const bf16_t *xj[J];
#pragma unroll
    for (int j = 0; j < J; ++j)
        xj[j] = x + (size_t)(plane0 + min(j * 8 + (lane >> 3), planes - 1)) * plane + (size_t)t0 * PLANE + (lane & 3) * 8;
    for (int t = 0; t < L; t += 4 * POOL_AHEAD) {
        bf16x8 r[POOL_AHEAD][J];
#pragma unroll
        for (int k = 0; k < POOL_AHEAD; ++k) {
            const int at = min(t + 4 * k + mine, L - 1) * PLANE;
#pragma unroll
            for (int j = 0; j < J; ++j) r[k][j] = *reinterpret_cast<const bf16x8 *>(xj[j] + at);
        }
#pragma unroll
        for (int k = 0; k < POOL_AHEAD; ++k)
            if (t + 4 * k + mine < L) {
#pragma unroll
                for (int j = 0; j < J; ++j)
#pragma unroll
                    for (int i = 0; i < 8; ++i) acc[j][i] += (float)r[k][j][i];
            }
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
        if (j * 8 + (lane >> 3) < planes) {
#pragma unroll
            for (int i = 0; i < 8; i += 4)
                *reinterpret_cast<f32x4 *>(&part[mine][(plane0 + j * 8 + (lane >> 3)) * PLANE + (lane & 3) * 8 + i]) =
                    f32x4{acc[j][i], acc[j][i + 1], acc[j][i + 2], acc[j][i + 3]};
        }
    __syncthreads();
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    float sq = 0.f;
    if (L > 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = tid + 256 * j;
            if (col < d) {
                v[j] = (((part[0][col] + part[1][col]) + part[2][col]) + part[3][col]) / (float)L;
                sq += v[j] * v[j];
            }
        }
    }
    red[tid] = sq;
    __syncthreads();
    // pairwise over the threads: (t, t + 128), (t, t + 64), then inside the wavefront
    const float nrm = fmaxf(sqrtf(wave_sum((red[lane] + red[lane + 128]) + (red[lane + 64] + red[lane + 192]))), 1e-12f);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int col = tid + 256 * j;
        if (col < d) out[(size_t)c * d + col] = v[j] / nrm;
    }
}

// A product's two copies of the weights, see pack_weights_kernel; no packed one where the context found no memory for it.
struct Weights {
    const bf16_t *rows, *packed;
};

// W beyond the 4 MB of L2 an XCD has is evicted between its uses; if the output is wide (so that A is small next
// to it) the column tiles go in groups that fit (measured on FFN1: +4-5 %; on QKV, whose W fits, a loss).
int column_group(int tiles_n, int N, int K)
{
    if ((size_t)N * K * sizeof(bf16_t) <= ((size_t)4 << 20) || N < 4 * K) return tiles_n;
    const int groups = (int)(((size_t)N * K * sizeof(bf16_t) + ((size_t)5 << 19) - 1) / ((size_t)5 << 19));  // 2.5 MB each
    return (tiles_n + groups - 1) / groups;
}

// Persistent blocks: one per CU slot (a multiple of 8), fewer when there are fewer tiles.
int persistent_grid(int slots, int tiles) { return std::max(8, std::min(slots, (tiles + 7) & ~7) & ~7); }

template <int EPI>
int launch_gemm(leann_ctx *ctx, int prof_kind, const bf16_t *A, const bf16_t *W, const float *bias, bf16_t *out,
                const int32_t *T_dev, int max_rows, int N, int K, int plane)
{
    if (N % 128 || K % (4 * GEMM_BK)) {
        leann_set_error("GEMM shape N=%d K=%d not covered by the 128x128 tile", N, K);
        return LEANN_ESHAPE;
    }
    const int tiles_n = N / 128, tiles = ((max_rows + 127) / 128) * tiles_n;
    ProfScope prof(ctx, prof_kind);
    hipLaunchKernelGGL((gemm_kernel<EPI>), dim3(persistent_grid(2 * ctx->num_cus, tiles)), dim3(256), GEMM_SMEM, ctx->stream, A, W, bias, out, T_dev,
                       N, K, tiles_n, column_group(tiles_n, N, K), plane);
    LEANN_HIP(hipGetLastError());
    return LEANN_OK;
}

template <int WM, int TM, int TN, int EPI>
int launch_gemm_large(leann_ctx *ctx, int prof_kind, const bf16_t *A, const Weights &W, const float *bias, bf16_t *out,
                      const int32_t *T_dev, int max_rows, int N, int K, int plane)
{
    typedef LargeCfg<WM, TM, TN> Cfg;
    if (N % 64 || K % (4 * GEMM_BK) || K < 8 * GEMM_BK) {
        leann_set_error("GEMM shape N=%d K=%d not covered by the %dx%d tile", N, K, Cfg::BM, Cfg::BN);
        return LEANN_ESHAPE;
    }
    const int tiles_n = (N + Cfg::BN - 1) / Cfg::BN, tiles = ((max_rows + Cfg::BM - 1) / Cfg::BM) * tiles_n;
    ProfScope prof(ctx, prof_kind);
    hipLaunchKernelGGL((gemm_large_kernel<WM, TM, TN, EPI>), dim3(persistent_grid(ctx->num_cus, tiles)), dim3(512), Cfg::SMEM, ctx->stream, A,
                       W.packed ? W.packed : W.rows, bias, out, T_dev, N, K, tiles_n, column_group(tiles_n, N, K), plane,
                       W.packed != nullptr);
    LEANN_HIP(hipGetLastError());
    return LEANN_OK;
}

// A tile of the stream kernels: R blocks of W rows by NM wavefronts of W columns.
template <int W, int R, int NM, int EPI>
struct StreamTile {
    static_assert(W == 16 || W == 32, "the MFMA's width");
    typedef std::conditional_t<W == 16, Stream16Cfg<R, NM>, StreamCfg<R, NM>> Cfg;
    static auto kernel()
    {
        if constexpr (W == 16) return gemm_stream16_kernel<R, NM, EPI>;
        else return gemm_stream_kernel<R, NM, EPI>;
    }
};

template <int W, int R, int NM, int EPI>
int launch_gemm_stream(leann_ctx *ctx, int prof_kind, const bf16_t *A, const bf16_t *Wp, const float *bias, bf16_t *out,
                       const int32_t *T_dev, int max_rows, int likely_rows, int N, int K, int xr)
{
    typedef StreamTile<W, R, NM, EPI> Tile;
    typedef typename Tile::Cfg Cfg;
    const int rt = (max_rows + Cfg::ROWS - 1) / Cfg::ROWS, ct = (N + Cfg::COLS - 1) / Cfg::COLS, xc = 8 / xr;
    ProfScope prof(ctx, prof_kind);
    hipLaunchKernelGGL(Tile::kernel(), dim3(8 * ((ct + xc - 1) / xc), (rt + xr - 1) / xr), dim3(Cfg::THREADS),
                       Cfg::SMEM, ctx->stream, A, Wp, bias, out, T_dev, max_rows, likely_rows, stream_shape(N, K, xr));
    LEANN_HIP(hipGetLastError());
    return LEANN_OK;
}

// One product, through the tile that choose_gemm (gemm_plan.h) takes.
template <int EPI>
int gemm(leann_ctx *ctx, int prof_kind, const bf16_t *A, const Weights &W, const float *bias, bf16_t *out,
         const int32_t *T_dev, int max_rows, int rows, int N, int K, int plane)
{
    const GemmChoice c = choose_gemm(ctx->num_cus, ctx->gemm_large_tile, W.packed && stream_covers(N, K, plane) ? ctx->gemm_small_rows : 0, rows, N, K);
    int tile = 0;
#define LEANN_TILE(WIDTH, R, NM, US, US_K)                                                                            \
    if (c.stream == tile++)                                                                                           \
        return launch_gemm_stream<WIDTH, R, NM, EPI>(ctx, prof_kind, A, W.packed, bias, out, T_dev, max_rows, rows, N, K, c.xr);
    LEANN_STREAM_TILES(LEANN_TILE)
#undef LEANN_TILE
    if (c.large == 256 && c.cols == 192) return launch_gemm_large<4, 2, 3, EPI>(ctx, prof_kind, A, W, bias, out, T_dev, max_rows, N, K, plane);
    if (c.large == 256) return launch_gemm_large<2, 4, 2, EPI>(ctx, prof_kind, A, W, bias, out, T_dev, max_rows, N, K, plane);
    return launch_gemm<EPI>(ctx, prof_kind, A, W.rows, bias, out, T_dev, max_rows, N, K, plane);
}

template <int W, int R, int NM, int EPI>
int gemm_stream_allow_lds()
{
    typedef StreamTile<W, R, NM, EPI> Tile;
    LEANN_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(Tile::kernel()), hipFuncAttributeMaxDynamicSharedMemorySize, Tile::Cfg::SMEM));
    return LEANN_OK;
}

template <int WM, int TM, int TN, int EPI>
int gemm_large_allow_lds()
{
    LEANN_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_large_kernel<WM, TM, TN, EPI>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, LargeCfg<WM, TM, TN>::SMEM));
    return LEANN_OK;
}

}  // namespace

// Kernels that use more dynamic LDS than the default limit are allowed their size on the current device.
int enc_ln_blocks_per_cu(int d, int *out)
{
    int n = 0;
    LEANN_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(ln_kernel_for(d, false)), 256, 0));
    *out = n > 0 ? n : 1;
    return LEANN_OK;
}

int enc_init_device()
{
    LEANN_TRY((gemm_large_allow_lds<2, 4, 2, EPI_BIAS>()));
    LEANN_TRY((gemm_large_allow_lds<2, 4, 2, EPI_BIAS_GELU>()));
    LEANN_TRY((gemm_large_allow_lds<4, 2, 3, EPI_BIAS>()));
    LEANN_TRY((gemm_large_allow_lds<4, 2, 3, EPI_BIAS_GELU>()));
#define LEANN_TILE(W, R, NM, US, US_K)                            \
    LEANN_TRY((gemm_stream_allow_lds<W, R, NM, EPI_BIAS>()));      \
    LEANN_TRY((gemm_stream_allow_lds<W, R, NM, EPI_BIAS_GELU>()));
    LEANN_STREAM_TILES(LEANN_TILE)
#undef LEANN_TILE
    LEANN_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(attention_kernel<8>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, AttCfg<8>::SMEM));
    return LEANN_OK;
}

int enc_pack_weights(leann_ctx *ctx, const bf16_t *W, int N, int K, bf16_t *packed)
{
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)(((int64_t)N * K / 8 + 255) / 256)), dim3(256), 0, ctx->stream, W, N, K, packed);
    LEANN_HIP(hipGetLastError());
    return LEANN_OK;
}

int enc_forward(leann_ctx *ctx, const leann_chunks *chunks, const int64_t *ids_dev, int64_t first_id, int64_t n,
                float *out_dev, int64_t *tok_count_dev, int64_t tokens)
{
    const leann_encoder_desc &e = ctx->desc;
    const int d = e.hidden, F = e.ffn, H = e.heads, seq = chunks->seq;
    if (n <= 0) return LEANN_OK;
    if (seq < 1 || seq > 256 || seq > e.max_pos) {
        leann_set_error("sequence length %d not covered (1..min(256, max_pos))", seq);
        return LEANN_ESHAPE;
    }
    int64_t per_pass = ctx->max_tokens / seq;
    if (per_pass < 1) per_pass = 1;
    if (per_pass > n) per_pass = n;
    const size_t rows = pass_pitch((int)(per_pass * seq));
    LEANN_TRY(ctx->reserve_for_pass(ctx->x, rows * d * sizeof(bf16_t)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->qkv, rows * 3 * d * sizeof(bf16_t)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->att, rows * d * sizeof(bf16_t)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->delta, rows * d * sizeof(bf16_t)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->hid, rows * F * sizeof(bf16_t)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->cu, (size_t)(per_pass + 1) * sizeof(int32_t)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->enc_ids, (size_t)per_pass * sizeof(int64_t)));
    bf16_t *x = (bf16_t *)ctx->x.p, *qkv = (bf16_t *)ctx->qkv.p, *att = (bf16_t *)ctx->att.p, *hid = (bf16_t *)ctx->hid.p;
    bf16_t *delta = (bf16_t *)ctx->delta.p;  // sublayer output waiting for its residual add + LayerNorm
    int32_t *cu = (int32_t *)ctx->cu.p;
    int64_t *chunk_of = (int64_t *)ctx->enc_ids.p;
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)(d / H));
    for (int64_t s = 0; s < n; s += per_pass) {
        const int m = (int)((n - s < per_pass) ? n - s : per_pass);
        const int max_rows = m * seq;
        // How many of the rows hold tokens decides the tiles.  Where the caller does not know, the host waits for the count while
        // the embedding kernel runs, or, in small passes, takes chunks to be five eighths full.
        const bool ask = tokens <= 0 && max_rows > ASK_ROWS;
        int rows = (int)std::min<int64_t>(max_rows, tokens > 0 ? (tokens * m + n - 1) / n : guessed_rows(max_rows));
        const int32_t *T_dev = cu + m;
        const int plane = pass_pitch(max_rows) * PLANE;
        {
            ProfScope prof(ctx, LEANN_PROF_ENC_OTHER);
            hipLaunchKernelGGL(prep_kernel, dim3(1), dim3(m <= PREP_FEW ? PREP_FEW : 1024), 0, ctx->stream, chunks->lengths,
                               ids_dev ? ids_dev + s : nullptr, first_id + s, m, chunks->n, seq, cu, chunk_of, ctx->host_flags,
                               tok_count_dev, ctx->prof_on ? (int64_t *)ctx->prof_tokens.p : nullptr, ask);
        }
        if (ask) LEANN_HIP(hipEventRecord(ctx->pass_event, ctx->stream));
        {
            ProfScope prof(ctx, LEANN_PROF_ENC_OTHER);
            hipLaunchKernelGGL(embed_ln_kernel, dim3((unsigned)(((int64_t)m * seq + 3) / 4)), dim3(256), 0, ctx->stream,
                               chunks->tokens, chunk_of, cu, m, seq, d, e.vocab, ctx->tok_emb, ctx->pos_emb, ctx->seg_emb,
                               ctx->emb_g, ctx->emb_b, e.ln_eps, x, plane, ctx->host_flags);
        }
        if (ask) {
            LEANN_HIP(hipEventSynchronize(ctx->pass_event));
            const volatile int *report = ctx->host_flags;
            rows = std::max(1, +report[PASS_TOKENS]);
        }
        // as many blocks as are resident at once (measured: 10 % faster than a row per wave, and than twice as
        // many blocks); their waves go through several rows each
        const bool few_rows = ln_few_rows(d, rows);
        const int ln_grid = std::min((max_rows + (few_rows ? 3 : 7)) / (few_rows ? 4 : 8), ctx->num_cus * ctx->ln_blocks_per_cu);
        const auto ln = ln_kernel_for(d, few_rows);
        auto layer_norm = [&](const float *g, const float *b) {
            ProfScope prof(ctx, LEANN_PROF_LAYERNORM);
            hipLaunchKernelGGL(ln, dim3(ln_grid), dim3(256), 0, ctx->stream, delta, g, b, x, T_dev, d, plane, e.ln_eps, 4 * ln_grid);
        };
        for (int l = 0; l < e.layers; ++l) {
            const LayerWeights &w = ctx->layers[l];
            LEANN_TRY(gemm<EPI_BIAS>(ctx, LEANN_PROF_GEMM_QKV, x, {w.wqkv, w.wqkv_p}, w.bqkv, qkv, T_dev, max_rows, rows, 3 * d, d, plane));
            {
                ProfScope prof(ctx, LEANN_PROF_ATTENTION);
                if (seq <= 128)
                    hipLaunchKernelGGL(attention_kernel<4>, dim3((unsigned)m * H), dim3(64 * 4), AttCfg<4>::SMEM, ctx->stream, qkv, cu,
                                       att, d, plane, scale_log2e);
                else
                    hipLaunchKernelGGL(attention_kernel<8>, dim3((unsigned)m * H), dim3(64 * 8), AttCfg<8>::SMEM, ctx->stream, qkv, cu,
                                       att, d, plane, scale_log2e);
            }
            LEANN_TRY(gemm<EPI_BIAS>(ctx, LEANN_PROF_GEMM_O, att, {w.wo, w.wo_p}, w.bo, delta, T_dev, max_rows, rows, d, d, plane));
            layer_norm(w.g1, w.be1);
            LEANN_TRY(gemm<EPI_BIAS_GELU>(ctx, LEANN_PROF_GEMM_FFN1, x, {w.w1, w.w1_p}, w.b1, hid, T_dev, max_rows, rows, F, d, plane));
            LEANN_TRY(gemm<EPI_BIAS>(ctx, LEANN_PROF_GEMM_FFN2, hid, {w.w2, w.w2_p}, w.b2, delta, T_dev, max_rows, rows, d, F, plane));
            layer_norm(w.g2, w.be2);
        }
        {
            ProfScope prof(ctx, LEANN_PROF_ENC_OTHER);
            hipLaunchKernelGGL(d <= 512 ? pool_kernel<1> : pool_kernel<2>, dim3(m), dim3(256), 0, ctx->stream, x, cu, d, plane, out_dev + (size_t)s * d);
        }
        LEANN_HIP(hipGetLastError());
    }
    return LEANN_OK;
}
