// Two-level search with dynamic batching (LEANN Algorithm 2, Sec. 4.1-4.2), every stage on the device.
//
// All queries of a call advance in rounds.  In a round each active query runs hops on its own block (advance_kernel:
// take the best unvisited node of the exact queue EQ, gather its CSR neighbours, ADC-score the new ones out of an
// LDS-resident lookup table, push them into the approximate queue AQ, move the top re-rank fraction to the pending
// list P) until |P| >= batch or EQ has no unvisited node.  The pending lists of all queries are then packed into one
// list (collect_kernel) and re-embedded by the encoder in large cross-query batches; the next advance_kernel scores them
// against their own query and try-inserts them into EQ.  Per query this is exactly the sequential algorithm; batching
// across queries changes no value because the encoder's output for a chunk does not depend on the rest of the batch.
#include <algorithm>
#include <type_traits>

#include "advance_plan.h"
#include "common.h"
#include "wave.h"

namespace {

constexpr int KSUB = 256;
constexpr int EF_MAX = 1024;  // leann_search refuses longer queues

struct SearchState {
    uint64_t *eq_key;     // [G][ef] exact queue, best first (queue_key)
    uint64_t *eq_row;     // [G][ef] CSR row of the entry, see pack_row
    uint8_t *eq_vis;      // [G][ef]
    int32_t *eq_n;        // [G]
    uint64_t *aq_key;     // [G][64][aq_rows] approximate queue in 64 columns, 0 where an entry has been taken out
    uint64_t *aq_max;     // [G][64] best entry of each column
    int32_t *aq_tail;     // [G] end of the used part
    int32_t *aq_live;     // [G] entries in it
    uint32_t *seen;       // [G][words]
    uint32_t *pend;       // [G][pcap]
    int32_t *n_pend;      // [G]
    int32_t *src;         // [G][pcap] row of the encoder output, for entries that own their chunk
    int32_t *own;         // [G][pcap] the entry that owns this entry's chunk
    unsigned long long *owner;  // [N] (~round << 32 | entry) of the chunk's smallest entry in the newest round that asked for it
    int32_t *memo_slot;   // [N] row of the call's embedding memo that holds the chunk, -1: none; NULL: memo off
    const float *memo_emb;  // [memo rows][d]
    int32_t *done;        // [G]
    int32_t *n_flush;     // [G] flushes so far
    int64_t *enc_ids;     // [G * pcap]
    long long *counters;  // see CTR_*
    long long *host_counters;  // the same in host memory and, behind them, the number of the last publish()
    const float *lut;     // [G][m_sub][256]
    const int32_t *slot_of;     // stored-embedding table, NULL: none
    const float *cache_emb;
    int64_t cache_rows;
    int64_t words;
    int32_t ef, aqcap, pcap;
    int32_t aq_rows;   // entries per column of AQ
    int32_t aq_near;   // of these, the first ones that a running block keeps in LDS
};

// CTR_ROUNDS: most flushes of a query, belongs to one group of queries; CTR_PENDING .. CTR_TICKET belong to one round
enum { CTR_HOPS = 0, CTR_ADC, CTR_RECOMP, CTR_FLUSH, CTR_ERR, CTR_TOKENS, CTR_MAXDEG, CTR_HITS, CTR_MEMO_HITS, CTR_ROUNDS, CTR_PENDING, CTR_NENC, CTR_ROUND_TOKENS, CTR_TICKET,
       // wall_clock64() at the start of the first init_kernel, of the round's advance_kernel; from there to collect_kernel's end, all
       // rounds added up; at the call's end
       CTR_T_START, CTR_T_ROUND, CTR_T_TRAVERSE, CTR_T_END,
       CTR_COUNT };
enum { ERR_BAD_NEIGHBOUR = 1, ERR_AQ_OVERFLOW = 2, ERR_P_OVERFLOW = 4, ERR_BAD_SLOT = 8 };

__device__ inline bool better(float sa, uint32_t ia, float sb, uint32_t ib) { return sa > sb || (sa == sb && ia < ib); }

// wave-wide arg-best under (score desc, id asc); pos < 0 marks "nothing".  Result is uniform.
__device__ inline void wave_best(float &s, uint32_t &id, int &pos)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        float s2 = __shfl_xor(s, o, 64);
        uint32_t id2 = __shfl_xor(id, o, 64);
        int p2 = __shfl_xor(pos, o, 64);
        if (p2 >= 0 && (pos < 0 || better(s2, id2, s, id))) {
            s = s2;
            id = id2;
            pos = p2;
        }
    }
}

template <class T>
__device__ inline void store_through(T *p, T v)  // past the L2
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ inline void wait_for_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The counters to the host, and then `seq`, which it waits for: by the last of a grid's blocks to get here, one wavefront of each.  Lane
// 0 has done its block's atomics on them.  A round's end is a chain of latencies from the last hop to the encoder's first kernel:
// hipStreamSynchronize comes back 10.7 us after an empty kernel's launch, a host that looks at a word of pinned memory 6.3 us after it.
// Only the counters have to be there (device-scope atomics and stores past the L2, in order by waits; a fence would also write back
// the L2): the kernels that use a round's other results come behind it in the stream.  ends_round: the time since the round's start is
// added to CTR_T_TRAVERSE, by whose clock it does not matter (the XCDs' differ by half a microsecond at most).
__device__ inline void publish(long long *counters, long long *host_counters, long long seq, bool ends_round)
{
    const int lane = threadIdx.x & 63;
    int last = 0;
    wait_for_stores();  // the atomics: those whose results nobody reads, too
    if (lane == 0) last = gridDim.x == 1 || __hip_atomic_fetch_add(&counters[CTR_TICKET], 1ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    if (lane == CTR_TICKET) __hip_atomic_store(&counters[CTR_TICKET], 0ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    long long value = lane < CTR_COUNT ? __hip_atomic_load(&counters[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const long long round_start = __shfl(value, CTR_T_ROUND, 64);
    if (ends_round && lane == CTR_T_TRAVERSE) {
        value += (long long)wall_clock64() - round_start;
        __hip_atomic_store(&counters[CTR_T_TRAVERSE], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane < CTR_COUNT) store_through(&host_counters[lane], value);
    wait_for_stores();
    if (lane == 0) store_through(&host_counters[CTR_COUNT], seq);
}

__global__ __launch_bounds__(256) void maxdeg_kernel(const uint64_t *__restrict__ row_ptr, int64_t n, long long *__restrict__ counters,
                                                     long long *__restrict__ host_counters, long long seq)
{
    __shared__ long long part[4];
    long long best = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        best = max(best, (long long)(row_ptr[i + 1] - row_ptr[i]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = max(best, (long long)__shfl_xor(best, o, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = best;
    __syncthreads();
    // one atomic per block: a thousand of them on one word, one per wavefront, were most of the kernel's 13.5 us
    if (threadIdx.x == 0) atomicMax(&counters[CTR_MAXDEG], max(max(part[0], part[1]), max(part[2], part[3])));
    if (threadIdx.x < 64) publish(counters, host_counters, seq, false);
}

// The state of a group of queries at its start, grid (any, queries).  n > 0: the call's first group, the owners of its n chunks are
// cleared too.
__global__ __launch_bounds__(256) void init_kernel(SearchState s, uint32_t entry, int64_t n)
{
    const int q = blockIdx.y;
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x, across = (int64_t)gridDim.x * 256;
    if (q == 0 && x == 0 && n > 0) s.counters[CTR_T_START] = wall_clock64();
    for (int64_t i = q * across + x; i < n; i += gridDim.y * across) s.owner[i] = ~0ull;
    for (int64_t w = x; w < s.words; w += across) s.seen[q * s.words + w] = w == entry >> 5 ? 1u << (entry & 31) : 0u;
    if (x > 0) return;
    s.eq_n[q] = 0;
    s.aq_tail[q] = 0;
    s.aq_live[q] = 0;
    s.done[q] = 0;
    s.n_flush[q] = 0;
    if (q == 0) s.counters[CTR_ROUNDS] = 0;
    s.n_pend[q] = 1;  // the entry point's exact score is the first flush
    s.pend[(size_t)q * s.pcap] = entry;
}

// Score, expand, score again: one block per query takes its query as far as it goes without the encoder.
//
// A launch starts with the exact scores of the pending chunks that the encoder (or a stored table) has supplied since the
// last one, then runs hops until a flush is due.  A flush whose chunks all come from the stored-embedding table is scored on
// the spot and the hops go on; otherwise the block claims its chunks (see claim below) and leaves.  So a search over
// stored embeddings is one launch, and with recomputation a round is this kernel, collect_kernel and the encoder.
//
// Latency bounds it: a hop is a chain of dependent reads, so everything that does not depend on the hop before is taken out
// of the chain.
//  - EQ is sorted (keys of score and id, LDS).  It does not change between flushes, so the next hops are known: a group of
//    up to GROUP_HOPS of them is prepared by the whole block.  Their neighbours' ids come in together, three wavefronts
//    take the approximate scores of all of them (seen or not) while the first one sets the visited marks, hop after hop, without
//    waiting in between.  This assumes that the hardware performs a wavefront's atomics on one word in the order of their
//    issue, also those of different lanes, as gfx950 does (one path to one slice of L2); the memory model promises it
//    for a single lane only.  Then they return what each hop would have found; in another order a neighbour of two hops of a
//    group would be counted for the later one.  Marks of hops that turn out not to be run (a flush is due first) are taken back.  What
//    is left of a hop, for one wavefront, is the new neighbours into AQ and the best ones of AQ out of it, in some hundred
//    instructions.
//  - AQ is unsorted.  Entry p is in column p % 64, which belongs to lane p % 64: an entry that comes in is compared with its
//    lane's best, nothing else.  Taking out the best is one maximum over the lanes and one over the column it was in, whose
//    entries (adjacent in memory, one per lane) are read meanwhile.  A taken entry leaves a hole; holes are squeezed out when the
//    end reaches the capacity, so AQ overflows when more than aqcap entries are alive, not earlier.
//  - a flush's exact scores are taken side by side (four wavefronts, each with up to four rows in flight), and merged into EQ
//    by counting.  "Insert if there is room or better than the worst" entry by entry leaves the ef best of both, which is
//    what the merge keeps.
// Measured with every embedding stored (500 queries, ef 200, N = 12288, d = 768; 238 hops and 37 flushes per query on average, 78 in
// the longest): 466 us; 720 us where a hop waited for its own marks and neighbours (2750 of 4300 clocks) and AQ was kept in
// runs.  Now a hop takes 1290 clocks, a flush and its group 10300.  The compiler keeps 118 scalar registers in lanes of vector ones (58
// before), a v_readlane or two where a hop needs one back.  How many queries share a CU: plan_advance.
constexpr int ADV_THREADS = 256;
constexpr int GROUP_HOPS = 16;                 // hops that are prepared together
constexpr int GROUP_CAND = ADV_THREADS - 64;   // their neighbours (of a row, the first 64) at most
constexpr int PEND_LDS = 128;                  // pending entries that a running block keeps in LDS

// LDS pointers that say so: of "LDS or memory" by index the compiler otherwise makes one flat access, which waits for both.
template <class T>
using lds_ptr = __attribute__((address_space(3))) T *;
template <class T>
__device__ inline lds_ptr<T> in_lds(T *p)
{
    return (lds_ptr<T>)p;
}

// A CSR row as one word: where it begins (40 bits) and its length; a length that does not fit is ROW_LONG and read again.
constexpr uint32_t ROW_LONG = (1u << 24) - 1;
__device__ inline uint64_t pack_row(uint64_t beg, uint64_t end) { return beg << 24 | min(end - beg, (uint64_t)ROW_LONG); }

// Sum over lanes 0 .. lane, for the first 16 lanes of a wavefront.
__device__ inline int sum_to_lane16(int v)
{
    v += (int)dpp_mov<0x111>((uint32_t)v);  // row_shr 1, 2, 4, 8: zeros come in at the row's start
    v += (int)dpp_mov<0x112>((uint32_t)v);
    v += (int)dpp_mov<0x114>((uint32_t)v);
    v += (int)dpp_mov<0x118>((uint32_t)v);
    return v;
}

// NV: 4-byte pieces of an embedding row per lane.  BLOCKS: that the registers shall let share a CU; 1: the compiler's choice (130 to
// 167 registers, three blocks), whose schedule takes 8 % less time per query.
template <int NV, int BLOCKS>
__global__ __launch_bounds__(ADV_THREADS, BLOCKS) void advance_kernel(SearchState s, const uint64_t *__restrict__ row_ptr,
                                                              const uint32_t *__restrict__ col_idx, int64_t n,
                                                              const uint8_t *__restrict__ codes, int m_sub, float alpha, int batch,
                                                              const float *__restrict__ queries, int d,
                                                              const float *__restrict__ enc_emb, bool have_results, uint32_t round)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int pitch = s.aq_near | 1;  // odd: the lanes' columns begin in different banks
    float *tab = reinterpret_cast<float *>(smem);                        // [m_sub][256]
    uint64_t *eqk = reinterpret_cast<uint64_t *>(tab + m_sub * KSUB);    // [ef]
    uint64_t *eqr = eqk + s.ef;                                          // [ef]
    uint64_t *aql = eqr + s.ef;                                          // [64][pitch]
    uint8_t *eqv = reinterpret_cast<uint8_t *>(aql + 64 * pitch);        // [ef], read in steps of 256
    __shared__ __attribute__((aligned(16))) uint64_t new_key[64];
    __shared__ const float *new_row[64];
    __shared__ uint32_t new_id[64];
    __shared__ uint64_t new_csr[64];
    __shared__ int better_old[ADV_THREADS / 64][64];  // entries of EQ that are better than a newcomer, per wavefront's share of them
    __shared__ int list[GROUP_HOPS];             // the group's hops: positions in EQ
    __shared__ uint64_t hop_beg[GROUP_HOPS];     // where their CSR rows begin
    __shared__ int hop_off[GROUP_HOPS + 1];      // where their candidates begin
    __shared__ uint64_t hop_fresh[GROUP_HOPS];   // the candidates that are met for the first time
    __shared__ int hop_base[GROUP_HOPS];         // where those begin in fresh_key
    __shared__ uint32_t cand_id[GROUP_CAND];
    __shared__ uint64_t fresh_key[GROUP_CAND];
    __shared__ uint32_t pend_l[PEND_LDS];
    __shared__ int sh_pend, sh_tail, sh_hops, sh_missing, sh_bad;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (q == 0 && tid == 0) {  // the round's counters: collect_kernel, which runs next, adds to them
        for (int i = CTR_PENDING; i < CTR_TICKET; ++i) s.counters[i] = 0;
        s.counters[CTR_T_ROUND] = wall_clock64();
    }
    if (s.done[q]) return;
    uint32_t *pend = s.pend + (size_t)q * s.pcap;
    uint64_t *aqg = s.aq_key + (size_t)q * 64 * s.aq_rows;
    uint32_t *seen = s.seen + (size_t)q * s.words;
    int n_pend = s.n_pend[q], n_eq = s.eq_n[q], tail = s.aq_tail[q], live = s.aq_live[q];
    int hops = 0, adc = 0, err = 0, recomp = 0, flushes = 0, hits = 0;
    for (int i = tid; i < n_eq; i += ADV_THREADS) {
        eqk[i] = s.eq_key[(size_t)q * s.ef + i];
        eqr[i] = s.eq_row[(size_t)q * s.ef + i];
        eqv[i] = s.eq_vis[(size_t)q * s.ef + i];
    }
    const lds_ptr<uint64_t> aq_near = in_lds(aql);
    auto copy_near = [&](int end, bool in) {  // the rows that are in use, between memory and LDS
        const int rows = min((end + 63) >> 6, s.aq_near);
        for (int i = tid; i < 64 * rows; i += ADV_THREADS) {
            const int c = i / rows, r = i - c * rows;
            if (in) aq_near[c * pitch + r] = aqg[(size_t)c * s.aq_rows + r];
            else aqg[(size_t)c * s.aq_rows + r] = aq_near[c * pitch + r];
        }
    };
    copy_near(tail, true);
    {
        const float4 *src = reinterpret_cast<const float4 *>(s.lut + (size_t)q * m_sub * KSUB);
        for (int i = tid; i < m_sub * KSUB / 4; i += ADV_THREADS) reinterpret_cast<float4 *>(tab)[i] = src[i];
    }
    for (int i = tid; i < min(n_pend, PEND_LDS); i += ADV_THREADS) pend_l[i] = pend[i];
    RowDots<NV> dots;
    dots.load(queries + (size_t)q * d, d, lane);
    if (tid == 0) {
        sh_tail = tail;
        sh_missing = sh_bad = 0;
    }
    const lds_ptr<uint32_t> pend_near = in_lds(pend_l);
    auto pending = [&](int j) -> uint32_t {
        if (j < PEND_LDS) return pend_near[j];
        return pend[j];
    };
    auto adc_score = [&](uint32_t v) -> float {  // table entries summed in subspace order
        const uint8_t *row = codes + (size_t)v * m_sub;
        float sc = 0.f;
        if ((m_sub & 15) == 0) {
            u32x4 w = *reinterpret_cast<const u32x4 *>(row);
            for (int m0 = 0; m0 < m_sub; m0 += 16) {
                const u32x4 next = *reinterpret_cast<const u32x4 *>(row + min(m0 + 16, m_sub - 16));
#pragma unroll
                for (int m = 0; m < 16; ++m) sc += tab[(m0 + m) * KSUB + ((w[m >> 2] >> (8 * (m & 3))) & 255u)];
                w = next;
            }
        } else {
            for (int m = 0; m < m_sub; ++m) sc += tab[m * KSUB + row[m]];
        }
        return sc;
    };
    // The cnt newcomers in new_key go into EQ.  An entry moves down by the number of better newcomers; a newcomer (lane j of
    // wavefront 0: newcomer j) goes behind everything better, old or new.
    auto merge = [&](int cnt, auto shares) {
        constexpr int SHARES = decltype(shares)::value;  // of EQ per thread
        uint64_t k[SHARES], csr[SHARES];
        uint8_t vis[SHARES];
        int to[SHARES];
#pragma unroll
        for (int c = 0; c < SHARES; ++c) {
            const int i = c * ADV_THREADS + tid;
            to[c] = s.ef;
            k[c] = 0;
            if (i < n_eq) {
                k[c] = eqk[i];
                csr[c] = eqr[i];
                vis[c] = eqv[i];
                to[c] = i;
            }
        }
        const uint64_t mine = lane < cnt ? new_key[lane] : ~0ull;
        int old = 0, fresh_rank = 0;
        for (int j0 = 0; j0 < cnt; j0 += 4) {
            uint64_t kj[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) kj[i] = new_key[j0 + i];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                fresh_rank += kj[i] > mine;
                int count = 0;
#pragma unroll
                for (int c = 0; c < SHARES; ++c)
                    if (c * ADV_THREADS < n_eq) {
                        to[c] += kj[i] > k[c];
                        count += (int)__popcll(__ballot(k[c] > kj[i]));
                    }
                if (lane == j0 + i) old = count;
            }
        }
        better_old[wave][lane] = old;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < SHARES; ++c)
            if (c * ADV_THREADS + tid < n_eq && to[c] < s.ef) {
                eqk[to[c]] = k[c];
                eqr[to[c]] = csr[c];
                eqv[to[c]] = vis[c];
            }
        if (tid < cnt) {
            int p = fresh_rank;
#pragma unroll
            for (int w = 0; w < ADV_THREADS / 64; ++w) p += better_old[w][lane];
            if (p < s.ef) {
                eqk[p] = mine;
                eqr[p] = new_csr[lane];
                eqv[p] = 0;
            }
        }
    };
    // AQ belongs to wavefront 0.
    auto aq_get = [&](int c, int r) -> uint64_t {
        if (r < s.aq_near) return aq_near[c * pitch + r];
        return aqg[(size_t)c * s.aq_rows + r];
    };
    auto aq_put = [&](int c, int r, uint64_t k) {
        if (r < s.aq_near) aq_near[c * pitch + r] = k;
        else aqg[(size_t)c * s.aq_rows + r] = k;
    };
    uint64_t col_best = wave == 0 && lane < tail ? s.aq_max[(size_t)q * 64 + lane] : 0;
    // What pop() takes out leaves its column by settle(), which the next one calls first: the column's entries come in meanwhile.
    uint64_t taken = 0, taken_k = 0;
    int taken_col = -1;
    auto column = [&](int r0) -> uint64_t {  // entry r0 + lane of that column
        const int r = r0 + lane;
        if (r * 64 + taken_col >= tail) return 0;
        return aq_get(taken_col, r);
    };
    auto settle = [&]() {
        if (taken_col < 0) return;
        uint64_t rest = 0;
        for (int r0 = 0; r0 * 64 < tail; r0 += 64) {
            const uint64_t k = r0 ? column(r0) : taken_k;
            if (k == taken) aq_put(taken_col, r0 + lane, 0);
            else rest = max(rest, k);
        }
        rest = wave_max_key(rest);
        if (lane == taken_col) col_best = max(col_best, rest);
        taken_col = -1;
    };
    // key: of the lane whose column comes next the first one, and so on; cnt of them
    auto push = [&](uint64_t key, int cnt) {
        if (__builtin_expect(tail + cnt > s.aqcap, 0)) {
            if (live + cnt <= s.aqcap) {  // squeeze the holes out, and bring the keys to the lanes of the new end
                settle();
                const uint64_t in_order = shfl_key(key, (tail + lane) & 63);
                int out = 0;
                for (int r = 0; r * 64 < tail; ++r) {
                    __threadfence_block();
                    const uint64_t k = r * 64 + lane < tail ? aq_get(lane, r) : 0;
                    const unsigned long long full = __ballot(k != 0);
                    const int p = out + __popcll(full & ((1ull << lane) - 1ull));
                    if (k) aq_put(p & 63, p >> 6, k);
                    out += __popcll(full);
                }
                __threadfence_block();
                tail = out;
                col_best = 0;
                for (int r = 0; r * 64 + lane < tail; ++r) col_best = max(col_best, aq_get(lane, r));
                key = shfl_key(in_order, (lane - tail) & 63);
            } else {
                err |= ERR_AQ_OVERFLOW;
                cnt = min(cnt, s.aqcap - tail);
            }
        }
        const int i = (lane - tail) & 63;
        if (i < cnt) {
            aq_put(lane, (tail + i) >> 6, key);
            col_best = max(col_best, key);
        }
        tail += cnt;
        live += cnt;
    };
    auto pop = [&]() {  // the best entry of AQ moves to the pending list
        settle();
        taken = wave_max_key(col_best);
        taken_col = __ffsll((long long)__ballot(col_best == taken)) - 1;
        if (tail > s.aq_near * 64) __threadfence_block();  // this wave's AQ stores to memory before the reads
        taken_k = column(0);
        if (lane == taken_col) col_best = 0;
        if (lane == 0) {
            if (n_pend < PEND_LDS) pend_near[n_pend] = key_id(taken);
            else if (n_pend < s.pcap) pend[n_pend] = key_id(taken);
        }
        if (n_pend >= s.pcap) err |= ERR_P_OVERFLOW;
        n_pend = min(n_pend + 1, s.pcap);
        --live;
    };
    auto mark = [&](uint32_t v, bool on) -> uint32_t {  // the word of marks before; v's bit set where it has been met
        return on ? atomicOr(&seen[v >> 5], 1u << (v & 31)) : ~0u;
    };
    __syncthreads();

    bool ready = have_results;  // the pending chunks' embeddings are there
    bool finished = false;
    for (;;) {
        if (tid < 64) new_key[tid] = 0;  // merge reads them four at a time
        if (!ready) {  // all of them in the stored table?
            for (int j = tid; j < n_pend; j += ADV_THREADS) {
                const uint32_t id = pending(j);
                const int slot = s.slot_of ? s.slot_of[id] : -1;
                if (slot < 0) sh_missing = 1;
                else if (slot >= s.cache_rows) sh_bad = 1;
                if (j < 64) {
                    new_id[j] = id;
                    new_csr[j] = pack_row(row_ptr[id], row_ptr[id + 1]);
                    new_row[j] = s.cache_emb + (size_t)max(slot, 0) * d;
                }
            }
            __syncthreads();
            if (sh_bad) err |= ERR_BAD_SLOT;  // reported; the host ends the search before anything reads through the slot
            if (sh_missing | sh_bad) break;
            hits += n_pend;
        }
        // exact scores, 64 entries at a time, and their merge into EQ
        for (int j0 = 0; j0 < n_pend; j0 += 64) {
            const int cnt = min(64, n_pend - j0);
            if (ready || j0 > 0) {
                if (tid < 64) new_key[tid] = 0;
                if (tid < cnt) {
                    const uint32_t id = pending(j0 + tid);
                    const int slot = s.slot_of ? s.slot_of[id] : -1;
                    const int mslot = slot < 0 && s.memo_slot ? s.memo_slot[id] : -1;
                    new_id[tid] = id;
                    new_csr[tid] = pack_row(row_ptr[id], row_ptr[id + 1]);
                    new_row[tid] = slot >= 0    ? s.cache_emb + (size_t)slot * d
                                   : mslot >= 0 ? s.memo_emb + (size_t)mslot * d
                                                : enc_emb + (size_t)s.src[s.own[(size_t)q * s.pcap + j0 + tid]] * d;
                }
                __syncthreads();
            }
            for (int i0 = wave; i0 < cnt; i0 += ADV_THREADS / 16) {
                const int c = min(4, (cnt - i0 + 3) / 4);
                float dv[4];
                dots.four([&](int k) { return new_row[i0 + 4 * k]; }, c, dv);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k < c && lane == 0) new_key[i0 + 4 * k] = queue_key(dv[k], new_id[i0 + 4 * k]);
            }
            __syncthreads();
            if (n_eq <= ADV_THREADS) merge(cnt, std::integral_constant<int, 1>());
            else merge(cnt, std::integral_constant<int, EF_MAX / ADV_THREADS>());
            n_eq = min(s.ef, n_eq + cnt);
            __syncthreads();
        }
        if (n_pend > 0) {
            recomp += n_pend;
            ++flushes;
        }
        n_pend = 0;
        ready = false;

        bool last = false;             // no open entry of EQ is left after this group
        int hop_pos = 0, hop_deg = 0;  // wavefront 0, lane h: hop h's position in EQ, its row's length
        for (;;) {
            if (wave == 0) {  // the next hops: the best entries of EQ that have not been expanded
                int m = 0, found = 0;
                if (n_pend < batch && !last)
                    for (int b = 0; b < n_eq && found <= GROUP_HOPS; b += 256) {  // lane l looks at positions b + 4l .. b + 4l + 3
                        const uint32_t vis = *reinterpret_cast<const uint32_t *>(eqv + b + 4 * lane);
                        bool open[4];
                        int at = found;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            open[i] = b + 4 * lane + i < n_eq && !(vis >> (8 * i) & 255u);
                            const unsigned long long mask = __ballot(open[i]);
                            at += __popcll(mask & ((1ull << lane) - 1ull));
                            found += (int)__popcll(mask);
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (open[i]) {
                                if (at < GROUP_HOPS) list[at] = b + 4 * lane + i;
                                ++at;
                            }
                    }
                m = min(GROUP_HOPS, found);
                __builtin_amdgcn_wave_barrier();
                if (m > 0) {
                    uint64_t beg = 0;
                    hop_deg = 0;
                    if (lane < m) {
                        hop_pos = list[lane];
                        beg = eqr[hop_pos] >> 24;
                        hop_deg = (int)(eqr[hop_pos] & ROW_LONG);
                        if (hop_deg == (int)ROW_LONG) hop_deg = (int)(row_ptr[key_id(eqk[hop_pos]) + 1] - beg);
                    }
                    // a row longer than a wavefront ends the group: the rest of it is taken when its hop is run
                    const unsigned long long longer = __ballot(hop_deg > 64);
                    if (longer) m = min(m, (int)__ffsll((long long)longer));
                    const int end = sum_to_lane16(min(hop_deg, 64));
                    m = min(m, (int)__popcll(__ballot(lane < GROUP_HOPS && end <= GROUP_CAND)));
                    if (lane < m) {
                        hop_beg[lane] = beg;
                        hop_off[lane + 1] = end;
                    }
                    if (lane == 0) hop_off[0] = 0;
                    last = found == m;
                }
                if (lane == 0) {
                    sh_hops = m;
                    sh_pend = n_pend;
                    sh_tail = tail;
                }
            }
            __syncthreads();
            const int m = __builtin_amdgcn_readfirstlane(sh_hops);
            if (m == 0) break;
            const int off = hop_off[min(lane, m)];
            const int t = tid - 64;  // wavefronts 1 to 3: a candidate each
            int hop = 0;
            uint32_t v = 0;
            const bool mine = t >= 0 && t < __builtin_amdgcn_readlane(off, m);
            if (mine) {
                for (int i = 1; i < m; ++i) hop += t >= __builtin_amdgcn_readlane(off, i);
                v = col_idx[hop_beg[hop] + (t - hop_off[hop])];
                cand_id[t] = v;
            }
            __syncthreads();
            uint64_t key = 0, fresh_h = 0;  // lane h of wavefront 0: hop h's mask
            int base_h = 0;
            bool bad_h = false;
            if (wave == 0) {
                uint32_t before[GROUP_HOPS], bit[GROUP_HOPS];
#pragma unroll
                for (int h0 = 0; h0 < GROUP_HOPS; h0 += 4) {
#pragma unroll
                    for (int h = h0; h < h0 + 4; ++h) before[h] = bit[h] = 0;
                    if (h0 < m) {
                        uint32_t w[4];
                        bool on[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int o = __builtin_amdgcn_readlane(off, h0 + i);
                            on[i] = lane < __builtin_amdgcn_readlane(off, h0 + i + 1) - o;
                            w[i] = cand_id[min(o + lane, GROUP_CAND - 1)];
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if (__ballot(on[i] && w[i] >= n) && lane == h0 + i) bad_h = true;
                            bit[h0 + i] = on[i] ? 1u << (w[i] & 31) : 0u;
                            before[h0 + i] = mark(w[i], on[i] && w[i] < n);
                        }
                    }
                }
#pragma unroll
                for (int h = 0; h < GROUP_HOPS; ++h) {
                    const unsigned long long mask = __ballot(bit[h] & ~before[h]);
                    if (lane == h) fresh_h = mask;
                }
                const int cnt = __popcll(fresh_h);
                base_h = sum_to_lane16(cnt) - cnt;
                if (lane < GROUP_HOPS) {
                    hop_fresh[lane] = fresh_h;
                    hop_base[lane] = base_h;
                }
            } else if (mine && v < n) {
                key = queue_key(adc_score(v), v);
            }
            __syncthreads();
            if (mine) {
                const int j = t - hop_off[hop];
                const uint64_t fresh = hop_fresh[hop];
                if (fresh >> j & 1u) fresh_key[hop_base[hop] + __popcll(fresh & ((1ull << j) - 1ull))] = key;
            }
            __syncthreads();
            if (wave != 0) continue;
            const int r_h = (int)ceilf(alpha * (float)__popcll(fresh_h));
            const int fresh_end = base_h + (int)__popcll(fresh_h);
            int h = 0;
            uint64_t next = fresh_key[(lane - tail) & 63];
            if (tail + __builtin_amdgcn_readlane(fresh_end, m - 1) <= min(s.aq_near * 64, s.aqcap) && __builtin_amdgcn_readlane(hop_deg, m - 1) <= 64) {
                // all in LDS, and no row is longer than a wavefront: the usual case
                for (; h < m && n_pend < batch; ++h) {
                    const int end = __builtin_amdgcn_readlane(fresh_end, h), n_new = end - __builtin_amdgcn_readlane(base_h, h);
                    const int i = (lane - tail) & 63;
                    if (i < n_new) {
                        aq_near[lane * pitch + ((tail + i) >> 6)] = next;
                        col_best = max(col_best, next);
                    }
                    tail += n_new;
                    live += n_new;
                    next = fresh_key[min(end + ((lane - tail) & 63), GROUP_CAND - 1)];  // the next hop's, for the lanes they go to
                    for (int r = __builtin_amdgcn_readlane(r_h, h); r > 0 && live > 0; --r) {
                        if (taken_col >= 0) {
                            if (taken_k == taken) {
                                aq_near[taken_col * pitch + lane] = 0;
                                taken_k = 0;
                            }
                            const uint64_t rest = wave_max_key(taken_k);
                            if (lane == taken_col) col_best = max(col_best, rest);
                        }
                        taken_col = wave_max_lane(col_best);
                        taken = key_of_lane(col_best, taken_col);
                        taken_k = 0;
                        if (lane * 64 + taken_col < tail) taken_k = aq_near[taken_col * pitch + lane];
                        if (lane == taken_col) col_best = 0;
                        if (lane == 0) {
                            if (n_pend < PEND_LDS) pend_near[n_pend] = key_id(taken);
                            else if (n_pend < s.pcap) pend[n_pend] = key_id(taken);
                        }
                        if (n_pend >= s.pcap) err |= ERR_P_OVERFLOW;
                        n_pend = min(n_pend + 1, s.pcap);
                        --live;
                    }
                }
                adc += h > 0 ? __builtin_amdgcn_readlane(fresh_end, h - 1) : 0;
            } else {
                for (; h < m && n_pend < batch; ++h) {
                    int n_new = __builtin_amdgcn_readlane(fresh_end, h) - __builtin_amdgcn_readlane(base_h, h), r = __builtin_amdgcn_readlane(r_h, h);
                    push(fresh_key[min(__builtin_amdgcn_readlane(base_h, h) + ((lane - tail) & 63), GROUP_CAND - 1)], n_new);
                    const int deg = __builtin_amdgcn_readlane(hop_deg, h);
                    if (deg > 64) {  // the rest of a row longer than a wavefront
                        for (int b = 64; b < deg; b += 64) {
                            const bool in = b + lane < deg;
                            const uint32_t w = in ? col_idx[hop_beg[h] + b + lane] : 0;
                            if (w >= n) err |= ERR_BAD_NEIGHBOUR;
                            const bool first_time = !(mark(w, in && w < n) >> (w & 31) & 1u);
                            const unsigned long long mask = __ballot(first_time);
                            if (first_time) new_key[__popcll(mask & ((1ull << lane) - 1ull))] = queue_key(adc_score(w), w);
                            __builtin_amdgcn_wave_barrier();
                            push(new_key[(lane - tail) & 63], __popcll(mask));
                            __builtin_amdgcn_wave_barrier();
                            n_new += __popcll(mask);
                        }
                        r = (int)ceilf(alpha * (float)n_new);
                    }
                    adc += n_new;
                    for (int i = 0; i < r && live > 0; ++i) pop();
                }
            }
            settle();
            hops += h;
            if (lane < h) eqv[hop_pos] = 1;
            if (__ballot(lane < h && bad_h)) err |= ERR_BAD_NEIGHBOUR;
            for (; h < m; ++h) {  // not run: the marks are taken back
                const uint32_t w = cand_id[min(__builtin_amdgcn_readlane(off, h) + lane, GROUP_CAND - 1)];
                if (key_of_lane(fresh_h, h) >> lane & 1u) atomicAnd(&seen[w >> 5], ~(1u << (w & 31)));
            }
        }
        n_pend = sh_pend;
        if (n_pend == 0) {  // no unvisited node and nothing pending
            finished = true;
            break;
        }
    }

    for (int i = tid; i < n_eq; i += ADV_THREADS) {
        s.eq_key[(size_t)q * s.ef + i] = eqk[i];
        s.eq_row[(size_t)q * s.ef + i] = eqr[i];
        s.eq_vis[(size_t)q * s.ef + i] = eqv[i];
    }
    int mine = 0, memo_hits = 0;  // of the pending entries: served by the stored table, by the memo
    if (!finished) {
        copy_near(sh_tail, false);
        if (wave == 0) s.aq_max[(size_t)q * 64 + lane] = col_best;
        // Claim.  Chunks that several queries ask for in the same round are encoded once: the pending entry with the
        // smallest number (q * pcap + j) owns the chunk.  The encoder's output for a chunk does not depend on its batch, so
        // every query still sees exactly the scores it would compute alone.  Newer rounds have smaller values: nothing has
        // to be taken back.
        for (int j = tid; j < n_pend; j += ADV_THREADS) {
            const uint32_t c = pending(j);
            if (j < PEND_LDS) pend[j] = c;
            if (s.slot_of && s.slot_of[c] >= 0) ++mine;
            else if (s.memo_slot && s.memo_slot[c] >= 0) ++memo_hits;  // encoded earlier in this call
            else atomicMin(&s.owner[c], (unsigned long long)~round << 32 | (uint32_t)(q * s.pcap + j));
        }
    }
    if (mine) atomicAdd((unsigned long long *)&s.counters[CTR_HITS], (unsigned long long)mine);
    if (memo_hits) atomicAdd((unsigned long long *)&s.counters[CTR_MEMO_HITS], (unsigned long long)memo_hits);
    if (err) atomicOr((unsigned long long *)&s.counters[CTR_ERR], (unsigned long long)err);
    if (tid == 0) {  // wavefront 0 has counted the hops
        s.eq_n[q] = n_eq;
        s.aq_tail[q] = tail;
        s.aq_live[q] = live;
        s.n_pend[q] = n_pend;
        const int all_flushes = s.n_flush[q] + flushes;
        s.n_flush[q] = all_flushes;
        if (finished) {
            s.done[q] = 1;
            atomicMax(&s.counters[CTR_ROUNDS], (long long)all_flushes);
        }
        atomicAdd((unsigned long long *)&s.counters[CTR_HOPS], (unsigned long long)hops);
        atomicAdd((unsigned long long *)&s.counters[CTR_ADC], (unsigned long long)adc);
        atomicAdd((unsigned long long *)&s.counters[CTR_RECOMP], (unsigned long long)recomp);
        atomicAdd((unsigned long long *)&s.counters[CTR_FLUSH], (unsigned long long)flushes);
        atomicAdd((unsigned long long *)&s.counters[CTR_HITS], (unsigned long long)hits);
    }
}

// Pack the round: encoder input list (one entry per owned chunk; the order does not matter), owners' rows, the round's
// totals.  One wavefront per query; the last block hands the counters to the host.
__global__ __launch_bounds__(64) void collect_kernel(SearchState s, const int32_t *__restrict__ lengths, int seq, long long number)
{
    const int q = blockIdx.x, lane = threadIdx.x;
    const int np = s.done[q] ? 0 : s.n_pend[q];
    int tokens = 0;
    for (int j0 = 0; j0 < np; j0 += 64) {
        const int j = j0 + lane, e = q * s.pcap + j;
        bool mine = false;
        uint32_t c = 0;
        if (j < np) {
            c = s.pend[e];
            if (!(s.slot_of && s.slot_of[c] >= 0) && !(s.memo_slot && s.memo_slot[c] >= 0)) {
                const int o = (int)(uint32_t)s.owner[c];
                s.own[e] = o;
                mine = o == e;
            }
        }
        const unsigned long long mask = __ballot(mine);
        if (!mask) continue;
        int at = 0;
        if (lane == 0) at = (int)atomicAdd((unsigned long long *)&s.counters[CTR_NENC], (unsigned long long)__popcll(mask));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(mask & ((1ull << lane) - 1ull));
        if (mine) {
            s.enc_ids[at] = c;
            s.src[e] = at;
            const int len = lengths[c];
            if (len >= 1 && len <= seq) tokens += len;  // others are reported by the encoder
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tokens += __shfl_xor(tokens, o, 64);
    if (lane == 0) {
        if (np) {
            atomicAdd((unsigned long long *)&s.counters[CTR_PENDING], (unsigned long long)np);
            atomicAdd((unsigned long long *)&s.counters[CTR_ROUND_TOKENS], (unsigned long long)tokens);
        }
    }
    publish(s.counters, s.host_counters, number, true);
}

// The call's end: behind the last finalize_kernel, whose results are then where all readers see them.
__global__ __launch_bounds__(64) void end_kernel(SearchState s, long long seq)
{
    if (threadIdx.x == 0) __hip_atomic_store(&s.counters[CTR_T_END], (long long)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    publish(s.counters, s.host_counters, seq, false);
}

// The call's embedding memo: rows the encoder produced in this round are kept (while there is room) so that a later
// round of the same call reads them instead of encoding the chunk again.  The encoder's rows come in no fixed order, so in the
// round that fills the memo, where not all have room, the first ones by query and pending entry are picked: what is
// encoded again later does not depend on scheduling.  One block of 1024 threads, once per call.
__global__ __launch_bounds__(1024) void memo_pick_kernel(SearchState s, int g, int64_t room, int32_t *__restrict__ pick)
{
    __shared__ int part[1024];
    const int tid = threadIdx.x, per = (g + 1023) / 1024;
    const int beg = min(g, tid * per), end = min(g, beg + per);
    auto owned = [&](int q, int j) {  // entry j of query q has had its chunk encoded in this round
        const int e = q * s.pcap + j;
        const uint32_t c = s.pend[e];
        return !(s.slot_of && s.slot_of[c] >= 0) && s.memo_slot[c] < 0 && s.own[e] == e;
    };
    int count = 0;
    for (int q = beg; q < end; ++q)
        for (int j = 0; j < (s.done[q] ? 0 : s.n_pend[q]); ++j) count += owned(q, j);
    part[tid] = count;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int v = tid >= o ? part[tid - o] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int64_t at = tid ? part[tid - 1] : 0;
    for (int q = beg; q < end && at < room; ++q)
        for (int j = 0; j < (s.done[q] ? 0 : s.n_pend[q]) && at < room; ++j)
            if (owned(q, j)) pick[at++] = s.src[q * s.pcap + j];
}

// Row base + i of the memo takes the encoder's row pick[i] (pick NULL: row i).  One wavefront per row.
__global__ __launch_bounds__(256) void memo_store_kernel(const float *__restrict__ enc_emb, const int64_t *__restrict__ enc_ids,
                                                         const int32_t *__restrict__ pick, int rows, int d, int64_t base,
                                                         float *__restrict__ memo_emb, int32_t *__restrict__ memo_slot)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= rows) return;
    const int row = pick ? pick[i] : i;
    const float *srcp = enc_emb + (size_t)row * d;
    float *dst = memo_emb + (size_t)(base + i) * d;
    for (int c = lane; c < d; c += 64) dst[c] = srcp[c];
    if (lane == 0) memo_slot[enc_ids[row]] = (int32_t)(base + i);
}

// Exact scores of the add buffer (App. B "Batched Add Operation": buffered chunks are scanned, not traversed):
// out[q][r] = <queries[q], buf[r]>.  One wavefront per (query, buffer row).
__global__ __launch_bounds__(256) void buffer_score_kernel(const float *__restrict__ queries, const float *__restrict__ buf,
                                                           int nb, int d, float *__restrict__ out)
{
    const int q = blockIdx.y, r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= nb) return;
    const float *qv = queries + (size_t)q * d, *e = buf + (size_t)r * d;
    float acc = 0.f;
    for (int i = lane; i < d; i += 64) acc += qv[i] * e[i];
    for (int o = 32; o; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) out[(size_t)q * nb + r] = acc;
}

// Output stage: the k best of (EQ without soft-deleted nodes) united with the scored add buffer, under
// (score desc, id asc); padded with id -1 / score -inf.  One wavefront per query; position p < n_eq is an EQ
// entry, p >= n_eq a buffer row.  Ids are unique over both, so "strictly after the last one emitted" selects the
// next.
__global__ __launch_bounds__(64) void finalize_kernel(SearchState s, int k, const uint32_t *__restrict__ deleted_bits,
                                                      const float *__restrict__ buf_scores,
                                                      const uint32_t *__restrict__ buf_ids, int nb,
                                                      int64_t *__restrict__ out_ids, float *__restrict__ out_scores)
{
    const int q = blockIdx.x, lane = threadIdx.x;
    const int n_eq = s.eq_n[q];
    const uint64_t *eqk = s.eq_key + (size_t)q * s.ef;
    const float *bsc = buf_scores + (size_t)q * nb;
    float last_s = INFINITY;
    uint32_t last_id = 0;
    bool have_last = false, exhausted = false;
    for (int j = 0; j < k; ++j) {
        float bs = -INFINITY;
        uint32_t bid = 0xffffffffu;
        int bpos = -1;
        if (!exhausted)
            for (int i = lane; i < n_eq + nb; i += 64) {
                float x;
                uint32_t id;
                if (i < n_eq) {
                    x = key_score(eqk[i]);
                    id = key_id(eqk[i]);
                    if (deleted_bits && (deleted_bits[id >> 5] >> (id & 31) & 1u)) continue;
                } else {
                    x = bsc[i - n_eq];
                    id = buf_ids[i - n_eq];
                }
                if (have_last && !better(last_s, last_id, x, id)) continue;  // already emitted
                if (bpos < 0 || better(x, id, bs, bid)) {
                    bs = x;
                    bid = id;
                    bpos = i;
                }
            }
        wave_best(bs, bid, bpos);
        if (lane == 0) {
            out_ids[(size_t)q * k + j] = bpos >= 0 ? (int64_t)bid : -1;
            out_scores[(size_t)q * k + j] = bpos >= 0 ? bs : -INFINITY;
        }
        if (bpos < 0) exhausted = true;
        have_last = true;
        last_s = bs;
        last_id = bid;
    }
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

namespace {

// pieces of advance_kernel for rows of d elements (the encoder's widths end at 1024)
int pieces_for(int d) { return d <= 128 ? 2 : d <= 384 ? 6 : d <= 768 ? 12 : 16; }

auto advance_for(int d, int blocks) -> decltype(&advance_kernel<2, 1>)
{
    const int nv = pieces_for(d);
    if (blocks == ADV_MORE_BLOCKS) return nv == 2 ? advance_kernel<2, ADV_MORE_BLOCKS> : advance_kernel<6, ADV_MORE_BLOCKS>;
    return nv == 2 ? advance_kernel<2, 1> : nv == 6 ? advance_kernel<6, 1> : nv == 12 ? advance_kernel<12, 1> : advance_kernel<16, 1>;
}

}  // namespace

int search_init_device()
{
    for (auto kernel : {advance_for(128, 1), advance_for(384, 1), advance_for(768, 1), advance_for(1024, 1),
                        advance_for(128, ADV_MORE_BLOCKS), advance_for(384, ADV_MORE_BLOCKS)}) {
        hipFuncAttributes attr;
        LEANN_HIP(hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(kernel)));
        if (attr.sharedSizeBytes > (size_t)ADV_FIXED) {  // else only the largest tables with long queues would fail to launch
            leann_set_error("advance_kernel's fixed arrays take %zu bytes of LDS, planned are %d", attr.sharedSizeBytes, ADV_FIXED);
            return LEANN_EDEVICE;
        }
        LEANN_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, ADV_DYNAMIC_MAX));
    }
    return LEANN_OK;
}

int search_run(leann_ctx *ctx, const float *queries_dev, int64_t nq, const leann_graph *graph, const leann_pq *pq,
               const leann_chunks *chunks, const leann_emb_cache *cache, const leann_updates *upd, int32_t ef, int32_t k,
               float alpha, int32_t batch, int64_t *out_ids_dev, float *out_scores_dev, leann_search_stats *stats)
{
    const int d = ctx->desc.hidden, m_sub = pq->m_sub;
    const int64_t n = graph->n;
    hipStream_t st = ctx->stream;
    LEANN_TRY(ctx->reserve_for_pass(ctx->s_misc, CTR_COUNT * sizeof(long long)));
    long long *counters = (long long *)ctx->s_misc.p;
    LEANN_HIP(hipMemsetAsync(counters, 0, CTR_COUNT * sizeof(long long), st));
    LEANN_TRY(clear_host_flags(ctx));
    HostWord &published = ctx->published;
    if (!ctx->host_counters) {
        LEANN_HIP(hipHostMalloc((void **)&ctx->host_counters, (CTR_COUNT + 1) * sizeof(long long), hipHostMallocDefault));
        ctx->host_counters[CTR_COUNT] = 0;
    }
    long long *h_ctr = ctx->host_counters;  // device kernels write it too: read after wait() only
    auto wait = [&]() -> int {  // for the publish() that was launched last
        LEANN_HIP(hipGetLastError());
        if (!published.arrives(reinterpret_cast<const uint32_t *>(&h_ctr[CTR_COUNT]))) LEANN_HIP(hipStreamSynchronize(st));
        return LEANN_OK;
    };
    hipLaunchKernelGGL(maxdeg_kernel, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(256, (n + 2047) / 2048))), dim3(256), 0, st,
                       graph->row_ptr, n, counters, h_ctr, (long long)published.next());
    LEANN_TRY(wait());
    const long long maxdeg = h_ctr[CTR_MAXDEG];

    // capacities
    const int64_t rmax = (int64_t)ceilf(alpha * (float)maxdeg);
    int64_t pcap64 = std::min<int64_t>((int64_t)batch - 1 + rmax, n) + 1;
    const int32_t pcap = (int32_t)std::max<int64_t>(pcap64, 2);
    const int32_t aqcap = (int32_t)std::max<int64_t>(1, std::min<int64_t>(n, ctx->aq_capacity > 0 ? ctx->aq_capacity : 32768));
    const int64_t words = (n + 31) / 32;
    // queries in flight: bounded by a 4 GiB budget for pending embeddings and for the visited bitmaps
    const size_t budget = (size_t)4 << 30;
    int64_t g_max = std::min<int64_t>(nq, 4096);
    g_max = std::min<int64_t>(g_max, std::max<int64_t>(1, (int64_t)(budget / ((size_t)pcap * d * sizeof(float)))));
    g_max = std::min<int64_t>(g_max, std::max<int64_t>(1, (int64_t)(budget / ((size_t)words * 4))));
    const int G = (int)g_max;

    // carve the state out of one allocation
    size_t off = 0;
    auto carve = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    const int32_t aq_rows = (aqcap + 63) / 64;
    const size_t o_eqk = carve((size_t)G * ef * 8), o_eqr = carve((size_t)G * ef * 8), o_eqv = carve((size_t)G * ef), o_eqn = carve((size_t)G * 4);
    const size_t o_aqk = carve((size_t)G * 64 * aq_rows * 8), o_aqm = carve((size_t)G * 64 * 8);
    const size_t o_aqt = carve((size_t)G * 4), o_aql = carve((size_t)G * 4), o_pend = carve((size_t)G * pcap * 4);
    const size_t o_np = carve((size_t)G * 4), o_src = carve((size_t)G * pcap * 4), o_own = carve((size_t)G * pcap * 4);
    const size_t o_done = carve((size_t)G * 4), o_nfl = carve((size_t)G * 4), o_eids = carve((size_t)G * pcap * 8);
    const int64_t memo_cap = std::min<int64_t>(ctx->memo_rows, (1 << 30) - 1);
    const size_t o_pick = carve(memo_cap > 0 ? (size_t)std::min<int64_t>(memo_cap, (int64_t)G * pcap) * 4 : 0);
    LEANN_TRY(ctx->reserve_for_pass(ctx->s_state, off));
    LEANN_TRY(ctx->reserve_for_pass(ctx->s_seen, (size_t)G * words * 4));
    LEANN_TRY(ctx->reserve_for_pass(ctx->s_lut, (size_t)G * m_sub * KSUB * sizeof(float)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->s_emb, (size_t)G * pcap * d * sizeof(float)));
    LEANN_TRY(ctx->reserve_for_pass(ctx->s_owner, (size_t)n * sizeof(unsigned long long)));
    // per-call embedding memo (leann_set_call_memo): empty at the start of every call
    int64_t memo_n = 0;
    if (memo_cap > 0) {
        LEANN_TRY(ctx->reserve_for_pass(ctx->s_memo_slot, (size_t)n * sizeof(int32_t)));
        LEANN_TRY(ctx->reserve_for_pass(ctx->s_memo_emb, (size_t)memo_cap * d * sizeof(float)));
        LEANN_HIP(hipMemsetAsync(ctx->s_memo_slot.p, 0xff, (size_t)n * sizeof(int32_t), st));
    }
    char *base = (char *)ctx->s_state.p;
    SearchState s;
    s.eq_key = (uint64_t *)(base + o_eqk);
    s.eq_row = (uint64_t *)(base + o_eqr);
    s.eq_vis = (uint8_t *)(base + o_eqv);
    s.eq_n = (int32_t *)(base + o_eqn);
    s.aq_key = (uint64_t *)(base + o_aqk);
    s.aq_max = (uint64_t *)(base + o_aqm);
    s.aq_tail = (int32_t *)(base + o_aqt);
    s.aq_live = (int32_t *)(base + o_aql);
    s.seen = (uint32_t *)ctx->s_seen.p;
    s.pend = (uint32_t *)(base + o_pend);
    s.n_pend = (int32_t *)(base + o_np);
    s.src = (int32_t *)(base + o_src);
    s.own = (int32_t *)(base + o_own);
    s.done = (int32_t *)(base + o_done);
    s.n_flush = (int32_t *)(base + o_nfl);
    s.owner = (unsigned long long *)ctx->s_owner.p;
    s.memo_slot = memo_cap > 0 ? (int32_t *)ctx->s_memo_slot.p : nullptr;
    s.memo_emb = memo_cap > 0 ? (const float *)ctx->s_memo_emb.p : nullptr;
    s.enc_ids = (int64_t *)(base + o_eids);
    int32_t *memo_pick = (int32_t *)(base + o_pick);
    s.counters = counters;
    s.lut = (const float *)ctx->s_lut.p;
    s.words = words;
    s.ef = ef;
    s.aqcap = aqcap;
    s.pcap = pcap;
    s.aq_rows = aq_rows;
    s.host_counters = h_ctr;
    s.slot_of = cache ? cache->slot_of : nullptr;
    s.cache_emb = cache ? cache->emb : nullptr;
    s.cache_rows = cache ? cache->rows : 0;

    const int table_smem = m_sub * KSUB * (int)sizeof(float) + ef * 9 + 16;
    if (table_smem > 150 * 1024) {
        leann_set_error("lookup table + queue of %d bytes exceed the LDS budget", table_smem);
        return LEANN_ESHAPE;
    }
    const AdvancePlan plan = plan_advance(m_sub, ef, G, ctx->num_cus, pieces_for(d));
    s.aq_near = plan.near;
    if (plan.bytes > ADV_DYNAMIC_MAX) {  // not with the widths that encoders and PQ tables have: at most 128 subspaces get here
        leann_set_error("lookup table + queue of %d bytes exceed the LDS budget", plan.bytes);
        return LEANN_ESHAPE;
    }
    const auto advance = advance_for(d, plan.blocks);
    uint32_t launches = 0;

    int rc = LEANN_OK;
    int64_t rounds = 0, encoded = 0;
    for (int64_t q0 = 0; q0 < nq && rc == LEANN_OK; q0 += G) {
        const int g = (int)std::min<int64_t>(G, nq - q0);
        const float *qg = queries_dev + (size_t)q0 * d;
        const int64_t per_query = std::min<int64_t>((words + 255) / 256, (8 * ctx->num_cus + g - 1) / g);
        hipLaunchKernelGGL(init_kernel, dim3((unsigned)per_query, g), dim3(256), 0, st, s, graph->entry, q0 == 0 ? n : 0);
        LEANN_TRY(pq_build_lut(ctx, qg, g, pq, (float *)ctx->s_lut.p));
        for (bool have_results = false;; have_results = true) {
            {
                ProfScope prof(ctx, LEANN_PROF_TRAVERSE);
                hipLaunchKernelGGL(advance, dim3(g), dim3(ADV_THREADS), plan.bytes, st, s, graph->row_ptr, graph->col_idx, n,
                                   pq->codes, m_sub, alpha, batch, qg, d, (const float *)ctx->s_emb.p, have_results, ++launches);
            }
            {
                ProfScope prof(ctx, LEANN_PROF_COLLECT);
                hipLaunchKernelGGL(collect_kernel, dim3(g), dim3(64), 0, st, s, chunks->lengths, chunks->seq, (long long)published.next());
            }
            LEANN_TRY(wait());
            if (h_ctr[CTR_ERR]) {
                rc = (h_ctr[CTR_ERR] & (ERR_BAD_NEIGHBOUR | ERR_BAD_SLOT)) ? LEANN_EINVAL : LEANN_ECAPACITY;
                leann_set_error((h_ctr[CTR_ERR] & ERR_BAD_NEIGHBOUR) ? "graph holds a neighbour id >= n"
                                : (h_ctr[CTR_ERR] & ERR_BAD_SLOT) ? "embedding cache: slot_of holds a row >= rows"
                                : "a per-query queue outgrew its capacity (see leann_set_limits)");
                break;
            }
            if (h_ctr[CTR_PENDING] == 0) {  // the launch that found that has scored and traversed all the same: its events count
                rounds += h_ctr[CTR_ROUNDS];
                break;
            }
            const int64_t n_enc = h_ctr[CTR_NENC];
            if (n_enc > 0) {
                rc = enc_forward(ctx, chunks, s.enc_ids, 0, n_enc, (float *)ctx->s_emb.p,
                                 (int64_t *)&counters[CTR_TOKENS], h_ctr[CTR_ROUND_TOKENS]);
                if (rc != LEANN_OK) break;
                encoded += n_enc;
                if (memo_n < memo_cap) {
                    const int64_t room = memo_cap - memo_n, rows = std::min<int64_t>(n_enc, room);
                    if (rows < n_enc) hipLaunchKernelGGL(memo_pick_kernel, dim3(1), dim3(1024), 0, st, s, g, room, memo_pick);
                    hipLaunchKernelGGL(memo_store_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st,
                                       (const float *)ctx->s_emb.p, s.enc_ids, rows < n_enc ? memo_pick : nullptr, (int)rows, d,
                                       memo_n, (float *)ctx->s_memo_emb.p, s.memo_slot);
                    memo_n += rows;
                }
            }
        }
        if (rc != LEANN_OK) break;
        const int nb = upd ? (int)upd->buffer_n : 0;
        const float *buf_scores = nullptr;
        if (nb > 0) {
            if ((size_t)g * nb * sizeof(float) > ((size_t)4 << 30)) {
                leann_set_error("leann_search: %d queries x %d buffered rows exceed the 4 GiB score workspace", g, nb);
                rc = LEANN_ECAPACITY;
                break;
            }
            LEANN_TRY(ctx->reserve_for_pass(ctx->s_buf, (size_t)g * nb * sizeof(float)));
            buf_scores = (const float *)ctx->s_buf.p;
            hipLaunchKernelGGL(buffer_score_kernel, dim3((nb + 3) / 4, g), dim3(256), 0, st, queries_dev + (size_t)q0 * d,
                               upd->buffer_emb, nb, d, (float *)ctx->s_buf.p);
        }
        hipLaunchKernelGGL(finalize_kernel, dim3(g), dim3(64), 0, st, s, k, upd ? upd->deleted_bits : nullptr, buf_scores,
                           upd ? upd->buffer_ids : nullptr, nb, out_ids_dev + (size_t)q0 * k,
                           out_scores_dev + (size_t)q0 * k);
    }
    if (rc == LEANN_OK) hipLaunchKernelGGL(end_kernel, dim3(1), dim3(64), 0, st, s, (long long)published.next());
    // The call's last wait is for the stream: a caller who waits for it next, as most do, would otherwise pay for that.
    const hipError_t sync_rc = hipStreamSynchronize(st);
    if (rc == LEANN_OK && sync_rc != hipSuccess) {
        leann_set_error("search kernels failed: %s", hipGetErrorString(sync_rc));
        rc = LEANN_EDEVICE;
    }
    const volatile int *bad = ctx->host_flags;
    if (rc == LEANN_OK && (bad[FLAG_CHUNK_ID] || bad[FLAG_LENGTH] || bad[FLAG_TOKEN])) {
        leann_set_error("chunk store holds a token id or length outside its range (flags %d)",
                        (bad[FLAG_CHUNK_ID] ? 1 : 0) | (bad[FLAG_LENGTH] ? 2 : 0) | (bad[FLAG_TOKEN] ? 4 : 0));
        rc = LEANN_EINVAL;
    }
    if (rc == LEANN_OK && stats) {
        stats->hops = h_ctr[CTR_HOPS];
        stats->adc_candidates = h_ctr[CTR_ADC];
        stats->recomputed_chunks = h_ctr[CTR_RECOMP];
        stats->cache_hits = h_ctr[CTR_HITS];
        stats->memo_hits = h_ctr[CTR_MEMO_HITS];
        stats->encoded_chunks = encoded;
        stats->encoded_tokens = h_ctr[CTR_TOKENS];
        stats->flushes = h_ctr[CTR_FLUSH];
        stats->rounds = rounds;
        const float total = (float)((h_ctr[CTR_T_END] - h_ctr[CTR_T_START]) / ctx->clock_khz);
        const float trav = (float)(h_ctr[CTR_T_TRAVERSE] / ctx->clock_khz);
        stats->total_ms = total;
        stats->traverse_ms = trav;
        stats->encoder_ms = total - trav;
    }
    return rc;
}
