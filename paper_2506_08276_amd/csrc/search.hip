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
#include <vector>

#include "common.h"
#include "wave.h"

namespace {

constexpr int KSUB = 256;

struct SearchState {
    uint64_t *eq_key;     // [G][ef] exact queue, best first (queue_key)
    uint8_t *eq_vis;      // [G][ef]
    int32_t *eq_n;        // [G]
    uint64_t *aq_key;     // [G][aqcap] approximate queue, 0 where an entry has been taken out
    uint64_t *aq_max;     // [G][aq_groups] best entry of each run of aq_run entries
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
    long long *host_counters;  // the same in host memory, written at the end of every round
    const float *lut;     // [G][m_sub][256]
    const int32_t *slot_of;     // stored-embedding table, NULL: none
    const float *cache_emb;
    int64_t cache_rows;
    int64_t words;
    int32_t ef, aqcap, pcap;
    int32_t aq_run, aq_groups;  // run length (a multiple of 64), number of runs
    int32_t aq_lds;             // entries of AQ that a running block keeps in LDS (a multiple of 64)
};

// CTR_ROUNDS: most flushes of a query, belongs to one group of queries; CTR_PENDING .. CTR_TICKET belong to one round
enum { CTR_HOPS = 0, CTR_ADC, CTR_RECOMP, CTR_FLUSH, CTR_ERR, CTR_TOKENS, CTR_MAXDEG, CTR_HITS, CTR_MEMO_HITS, CTR_ROUNDS, CTR_PENDING, CTR_NENC, CTR_ROUND_TOKENS, CTR_TICKET, CTR_COUNT };
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

__global__ void maxdeg_kernel(const uint64_t *__restrict__ row_ptr, int64_t n, long long *__restrict__ counters)
{
    long long best = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        best = max(best, (long long)(row_ptr[i + 1] - row_ptr[i]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = max(best, (long long)__shfl_xor(best, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(&counters[CTR_MAXDEG], best);
}

__global__ void init_kernel(SearchState s, int g, uint32_t entry)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= g) return;
    s.eq_n[q] = 0;
    s.aq_tail[q] = 0;
    s.aq_live[q] = 0;
    s.done[q] = 0;
    s.n_flush[q] = 0;
    if (q == 0) s.counters[CTR_ROUNDS] = 0;
    s.n_pend[q] = 1;  // the entry point's exact score is the first flush
    s.pend[(size_t)q * s.pcap] = entry;
    s.seen[(size_t)q * s.words + (entry >> 5)] = 1u << (entry & 31);
}

// Score, expand, score again: one block per query takes its query as far as it goes without the encoder.
//
// A launch starts with the exact scores of the pending chunks that the encoder (or a stored table) has supplied since the
// last one, then runs hops until a flush is due.  A flush whose chunks all come from the stored-embedding table is scored on
// the spot and the hops go on; otherwise the block claims its chunks (see claim below) and leaves.  So a search over
// stored embeddings is one launch, and with recomputation a round is this kernel, collect_kernel and the encoder.
//
// Latency bounds it: a hop is a chain of dependent reads, so the chain is kept short.
//  - EQ is sorted (keys of score and id, LDS).  It does not change between flushes, so the next hops are known: their CSR
//    rows are fetched two hops ahead, the PQ codes of all neighbours (seen or not) one hop ahead, and the visited marks one
//    hop ahead where it is certain that the next hop will be run.  So a hop has one wait for all of these instead of
//    a chain of three; it does have that one, as the marks' result is made a flag where they are set.
//  - AQ is unsorted in runs of aq_run entries, the best entry of every run on the side: taking out the best of some
//    thousand entries reads the runs' best and one run.  A taken entry leaves a hole; holes are squeezed out when the
//    end reaches the capacity, so AQ overflows when more than aqcap entries are alive, not earlier.
//  - a flush's exact scores are taken side by side (four wavefronts, each with one or two rows in flight), and merged into EQ
//    by counting.  "Insert if there is room or better than the worst" entry by entry leaves the ef best of both, which is
//    what the merge keeps.
// Measured with every embedding stored (500 queries, ef 200, N = 12288, d = 768): a search of 239 hops, 37 flushes and 248
// exact scores per query takes 0.9 ms; one wavefront per query with scans over both queues and a host round per flush
// took 13.8 ms (78 rounds of 77 us hops, 44 us scores and 24 us packing).
constexpr int ADV_THREADS = 256;
constexpr int AQ_LDS_MAX = 2048, AQ_GROUPS_MAX = 512;

__device__ inline uint64_t readlane64(uint64_t v, int l)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

template <int NV>  // 4-byte pieces of an embedding row per lane
__global__ __launch_bounds__(ADV_THREADS) void advance_kernel(SearchState s, const uint64_t *__restrict__ row_ptr,
                                                              const uint32_t *__restrict__ col_idx, int64_t n,
                                                              const uint8_t *__restrict__ codes, int m_sub, float alpha, int batch,
                                                              const float *__restrict__ queries, int d,
                                                              const float *__restrict__ enc_emb, bool have_results, uint32_t round)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float *tab = reinterpret_cast<float *>(smem);                        // [m_sub][256]
    uint64_t *eqk = reinterpret_cast<uint64_t *>(tab + m_sub * KSUB);    // [ef]
    uint64_t *aqm = eqk + s.ef;                                          // [aq_groups]
    uint64_t *aql = aqm + s.aq_groups;                                   // [aq_lds]
    uint8_t *eqv = reinterpret_cast<uint8_t *>(aql + s.aq_lds);          // [ef]
    __shared__ uint64_t new_key[64];
    __shared__ const float *new_row[64];
    __shared__ uint32_t new_id[64];
    __shared__ int list[64];
    __shared__ int sh_pend, sh_tail;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (q == 0 && tid == 0)  // the round's counters: collect_kernel, which runs next, adds to them
        for (int i = CTR_PENDING; i <= CTR_TICKET; ++i) s.counters[i] = 0;
    if (s.done[q]) return;
    uint32_t *pend = s.pend + (size_t)q * s.pcap;
    uint64_t *aqg = s.aq_key + (size_t)q * s.aqcap;
    uint32_t *seen = s.seen + (size_t)q * s.words;
    int n_pend = s.n_pend[q], n_eq = s.eq_n[q], tail = s.aq_tail[q], live = s.aq_live[q];
    int hops = 0, adc = 0, err = 0, recomp = 0, flushes = 0, hits = 0;
    for (int i = tid; i < n_eq; i += ADV_THREADS) {
        eqk[i] = s.eq_key[(size_t)q * s.ef + i];
        eqv[i] = s.eq_vis[(size_t)q * s.ef + i];
    }
    for (int i = tid; i < s.aq_groups; i += ADV_THREADS) aqm[i] = i * s.aq_run < tail ? s.aq_max[(size_t)q * s.aq_groups + i] : 0;
    for (int i = tid; i < min(tail, s.aq_lds); i += ADV_THREADS) aql[i] = aqg[i];
    {
        const float4 *src = reinterpret_cast<const float4 *>(s.lut + (size_t)q * m_sub * KSUB);
        for (int i = tid; i < m_sub * KSUB / 4; i += ADV_THREADS) reinterpret_cast<float4 *>(tab)[i] = src[i];
    }
    RowDots<NV> dots;
    dots.load(queries + (size_t)q * d, d, lane);
    if (tid == 0) sh_tail = tail;
    __syncthreads();

    bool ready = have_results;  // the pending chunks' embeddings are there
    bool finished = false;
    for (;;) {
        if (!ready) {  // all of them in the stored table?
            int missing = 0, bad = 0;
            for (int j = tid; j < n_pend; j += ADV_THREADS) {
                const int slot = s.slot_of ? s.slot_of[pend[j]] : -1;
                missing |= slot < 0;
                bad |= slot >= 0 && slot >= s.cache_rows;
            }
            if (__syncthreads_or(bad)) {  // reported; the host ends the search before anything reads through the slot
                err |= ERR_BAD_SLOT;
                break;
            }
            if (__syncthreads_or(missing)) break;
            hits += n_pend;
        }
        // exact scores, 64 entries at a time, and their merge into EQ
        for (int j0 = 0; j0 < n_pend; j0 += 64) {
            const int cnt = min(64, n_pend - j0);
            if (tid < cnt) {
                const uint32_t id = pend[j0 + tid];
                const int slot = s.slot_of ? s.slot_of[id] : -1;
                const int mslot = slot < 0 && s.memo_slot ? s.memo_slot[id] : -1;
                new_id[tid] = id;
                new_row[tid] = slot >= 0    ? s.cache_emb + (size_t)slot * d
                               : mslot >= 0 ? s.memo_emb + (size_t)mslot * d
                                            : enc_emb + (size_t)s.src[s.own[(size_t)q * s.pcap + j0 + tid]] * d;
            }
            __syncthreads();
            for (int i0 = wave; i0 < cnt; i0 += ADV_THREADS / 16) {
                const int c = min(4, (cnt - i0 + 3) / 4);
                float dv[4];
                dots.four([&](int k) { return new_row[i0 + 4 * k]; }, c, dv);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k < c && lane == 0) new_key[i0 + 4 * k] = queue_key(dv[k], new_id[i0 + 4 * k]);
            }
            __syncthreads();
            int to = s.ef;  // where newcomer tid goes: behind everything better, old or new
            uint64_t mine = 0;
            if (tid < cnt) {
                mine = new_key[tid];
                int lo = 0, hi = n_eq;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (eqk[mid] > mine) lo = mid + 1;
                    else hi = mid;
                }
                to = lo;
                for (int j = 0; j < cnt; ++j) to += new_key[j] > mine;
            }
            __syncthreads();
            for (int base = (n_eq - 1) / ADV_THREADS * ADV_THREADS; base >= 0; base -= ADV_THREADS) {  // from the back: entries only move down
                const int i = base + tid;
                uint64_t k = 0;
                uint8_t v = 0;
                int p = s.ef;
                if (i < n_eq) {
                    k = eqk[i];
                    v = eqv[i];
                    p = i;
                    for (int j = 0; j < cnt; ++j) p += new_key[j] > k;
                }
                __syncthreads();
                if (p < s.ef) {
                    eqk[p] = k;
                    eqv[p] = v;
                }
                __syncthreads();
            }
            if (to < s.ef) {
                eqk[to] = mine;
                eqv[to] = 0;
            }
            n_eq = min(s.ef, n_eq + cnt);
            __syncthreads();
        }
        if (n_pend > 0) {
            recomp += n_pend;
            ++flushes;
        }
        n_pend = 0;
        ready = false;

        if (wave == 0) {
            const int runs64 = s.aq_run >> 6;
            auto aq_get = [&](int p) -> uint64_t { return p < s.aq_lds ? aql[p] : aqg[p]; };
            auto aq_put = [&](int p, uint64_t k) {
                if (p < s.aq_lds) aql[p] = k;
                else aqg[p] = k;
            };
            const int n16 = (m_sub & 15) == 0 && m_sub <= 64 ? m_sub >> 4 : 0;  // 16-byte pieces of a code row that are fetched ahead
            auto fetch_codes = [&](uint32_t v, bool on, u32x4 (&c)[4]) {
                if (!on) return;
                const uint8_t *row = codes + (size_t)v * m_sub;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (i < n16) c[i] = *reinterpret_cast<const u32x4 *>(row + 16 * i);
            };
            auto mark = [&](uint32_t v, bool on) -> bool {  // first time this query meets v?
                if (!on) return false;
                const uint32_t bit = 1u << (v & 31);
                return !(atomicOr(&seen[v >> 5], bit) & bit);
            };
            // the neighbours that are new go to AQ with their approximate scores; returns how many there are
            auto take = [&](uint32_t v, bool is_new, const u32x4 (&c)[4]) -> int {
                float sc = 0.f;
                if (is_new) {  // table entries summed in subspace order
                    if (n16 > 0) {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (i < n16) {
#pragma unroll
                                for (int m = 0; m < 16; ++m) sc += tab[(16 * i + m) * KSUB + ((c[i][m >> 2] >> (8 * (m & 3))) & 255u)];
                            }
                    } else if ((m_sub & 15) == 0) {
                        const uint8_t *row = codes + (size_t)v * m_sub;
                        for (int m0 = 0; m0 < m_sub; m0 += 16) {
                            const u32x4 w = *reinterpret_cast<const u32x4 *>(row + m0);
#pragma unroll
                            for (int m = 0; m < 16; ++m) sc += tab[(m0 + m) * KSUB + ((w[m >> 2] >> (8 * (m & 3))) & 255u)];
                        }
                    } else {
                        const uint8_t *row = codes + (size_t)v * m_sub;
                        for (int m = 0; m < m_sub; ++m) sc += tab[m * KSUB + row[m]];
                    }
                }
                const unsigned long long mask = __ballot(is_new);
                const int cnt = __popcll(mask);
                if (tail + cnt > s.aqcap && live + cnt <= s.aqcap) {  // squeeze the holes out
                    __threadfence_block();
                    int out = 0;
                    for (int b = 0; b < tail; b += 64) {
                        const uint64_t k = b + lane < tail ? aq_get(b + lane) : 0;
                        const unsigned long long full = __ballot(k != 0);
                        if (k) aq_put(out + __popcll(full & ((1ull << lane) - 1ull)), k);
                        out += __popcll(full);
                    }
                    tail = out;
                    __threadfence_block();
                    for (int g = 0; g < s.aq_groups; ++g) {
                        uint64_t best = 0;
                        for (int b = g * s.aq_run + lane; b < min(tail, (g + 1) * s.aq_run); b += 64) best = max(best, aq_get(b));
                        best = wave_max_key(best);
                        if (lane == 0) aqm[g] = best;
                    }
                }
                const int pos = tail + __popcll(mask & ((1ull << lane) - 1ull));
                if (is_new) {
                    if (pos < s.aqcap) {
                        const uint64_t k = queue_key(sc, v);
                        aq_put(pos, k);
                        atomicMax(reinterpret_cast<unsigned long long *>(&aqm[pos / s.aq_run]), (unsigned long long)k);
                    } else {
                        err |= ERR_AQ_OVERFLOW;
                    }
                }
                const int fit = min(cnt, s.aqcap - tail);
                tail += fit;
                live += fit;
                return cnt;
            };
            bool more = true;
            while (more && n_pend < batch) {
                // the next hops: the best 64 entries of EQ that have not been expanded
                int m = 0;
                for (int b = 0; b < n_eq && m < 64; b += 64) {
                    const bool open = b + lane < n_eq && !eqv[b + lane];
                    const unsigned long long mask = __ballot(open);
                    const int at = m + __popcll(mask & ((1ull << lane) - 1ull));
                    if (open && at < 64) list[at] = b + lane;
                    m = min(64, m + __popcll(mask));
                }
                if (m == 0) break;
                more = m == 64;
                __builtin_amdgcn_wave_barrier();
                const int at = lane < m ? list[lane] : 0;
                const uint32_t u = lane < m ? key_id(eqk[at]) : 0;
                uint64_t beg = 0;
                int deg = 0;
                if (lane < m) {
                    beg = row_ptr[u];
                    deg = (int)(row_ptr[u + 1] - beg);
                }
                auto fetch_row = [&](int h) -> uint32_t {  // the first 64 neighbours of hop h
                    uint32_t v = 0;
                    if (h < m && lane < __builtin_amdgcn_readlane(deg, h)) v = col_idx[readlane64(beg, h) + lane];
                    return v;
                };
                uint32_t v0 = fetch_row(0), v1 = fetch_row(1);
                u32x4 c0[4], c1[4];
                bool on0 = lane < __builtin_amdgcn_readlane(deg, 0) && v0 < n;
                fetch_codes(v0, on0, c0);
                bool marked = false, fresh = false;  // hop h's marks have been set a hop ahead; what that said
                int h = 0;
                for (; h < m && n_pend < batch; ++h) {
                    const int dh = __builtin_amdgcn_readlane(deg, h);
                    const uint64_t bh = readlane64(beg, h);
                    if (lane == 0) eqv[__builtin_amdgcn_readlane(at, h)] = 1;
                    ++hops;
                    if (lane < dh && v0 >= n) err |= ERR_BAD_NEIGHBOUR;
                    if (!marked) fresh = mark(v0, on0);
                    // the next hop's codes, the row of the one after it
                    const int dn = h + 1 < m ? __builtin_amdgcn_readlane(deg, h + 1) : 0;
                    const bool on1 = lane < dn && v1 < n;
                    fetch_codes(v1, on1, c1);
                    const uint32_t v2 = fetch_row(h + 2);
                    bool fresh1 = false;
                    const bool certain = h + 1 < m && dh <= 64 && n_pend + (int)ceilf(alpha * (float)dh) < batch;
                    if (certain) fresh1 = mark(v1, on1);
                    int n_new = take(v0, fresh, c0);
                    for (int b = 64; b < dh; b += 64) {  // rows longer than a wavefront
                        uint32_t v = 0;
                        const bool in = b + lane < dh;
                        if (in) v = col_idx[bh + b + lane];
                        if (in && v >= n) err |= ERR_BAD_NEIGHBOUR;
                        u32x4 c[4];
                        const bool is_new = mark(v, in && v < n);
                        fetch_codes(v, is_new, c);
                        n_new += take(v, is_new, c);
                    }
                    adc += n_new;
                    if (tail > s.aq_lds) __threadfence_block();  // orders this wave's AQ stores before the reads below
                    // move the r best entries of AQ to the pending list
                    const int r = (int)ceilf(alpha * (float)n_new);
                    const int groups = (tail + s.aq_run - 1) / s.aq_run;
                    for (int t = 0; t < r && live > 0; ++t) {
                        uint64_t best = 0;
                        int from = 0;
                        for (int g = lane; g < groups; g += 64)
                            if (aqm[g] > best) {
                                best = aqm[g];
                                from = g;
                            }
                        const uint64_t top = wave_max_key(best);
                        const int g = __builtin_amdgcn_readlane(from, __ffsll((long long)__ballot(best == top)) - 1);
                        uint64_t rest = 0;
                        for (int i = 0; i < runs64; ++i) {
                            const int p = g * s.aq_run + i * 64 + lane;
                            const uint64_t k = p < tail ? aq_get(p) : 0;
                            if (k == top) aq_put(p, 0);
                            else rest = max(rest, k);
                        }
                        rest = wave_max_key(rest);
                        if (lane == 0) {
                            aqm[g] = rest;
                            if (n_pend < s.pcap) pend[n_pend] = key_id(top);
                        }
                        if (tail > s.aq_lds) __threadfence_block();
                        if (n_pend >= s.pcap) err |= ERR_P_OVERFLOW;
                        n_pend = min(n_pend + 1, s.pcap);
                        --live;
                    }
                    v0 = v1;
                    on0 = on1;
                    v1 = v2;
                    marked = certain;
                    fresh = fresh1;
#pragma unroll
                    for (int i = 0; i < 4; ++i) c0[i] = c1[i];
                }
            }
            if (lane == 0) {
                sh_pend = n_pend;
                sh_tail = tail;
            }
        }
        __syncthreads();
        n_pend = sh_pend;
        if (n_pend == 0) {  // no unvisited node and nothing pending
            finished = true;
            break;
        }
    }

    for (int i = tid; i < n_eq; i += ADV_THREADS) {
        s.eq_key[(size_t)q * s.ef + i] = eqk[i];
        s.eq_vis[(size_t)q * s.ef + i] = eqv[i];
    }
    int mine = 0, memo_hits = 0;  // of the pending entries: served by the stored table, by the memo
    if (!finished) {
        const int end = sh_tail;
        for (int i = tid; i < min(end, s.aq_lds); i += ADV_THREADS) aqg[i] = aql[i];
        for (int i = tid; i < s.aq_groups; i += ADV_THREADS) s.aq_max[(size_t)q * s.aq_groups + i] = aqm[i];
        // Claim.  Chunks that several queries ask for in the same round are encoded once: the pending entry with the
        // smallest number (q * pcap + j) owns the chunk.  The encoder's output for a chunk does not depend on its batch, so
        // every query still sees exactly the scores it would compute alone.  Newer rounds have smaller values: nothing has
        // to be taken back.
        for (int j = tid; j < n_pend; j += ADV_THREADS) {
            const uint32_t c = pend[j];
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
__global__ __launch_bounds__(64) void collect_kernel(SearchState s, const int32_t *__restrict__ lengths, int seq)
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
    int last = 0;
    if (lane == 0) {
        if (np) {
            atomicAdd((unsigned long long *)&s.counters[CTR_PENDING], (unsigned long long)np);
            atomicAdd((unsigned long long *)&s.counters[CTR_ROUND_TOKENS], (unsigned long long)tokens);
        }
        __threadfence();
        last = atomicAdd((unsigned long long *)&s.counters[CTR_TICKET], 1ull) == gridDim.x - 1;
    }
    if (__builtin_amdgcn_readfirstlane(last)) {
        __threadfence();
        if (lane < CTR_COUNT)
            __hip_atomic_store(&s.host_counters[lane], __hip_atomic_load(&s.counters[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __threadfence_system();
    }
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

constexpr int LDS_LIMIT = 158 * 1024;  // dynamic LDS of advance_kernel, beside its few fixed arrays

// advance_kernel for rows of d elements (the encoder's widths end at 1024)
auto advance_for(int d) -> decltype(&advance_kernel<2>)
{
    return d <= 128 ? advance_kernel<2> : d <= 384 ? advance_kernel<6> : d <= 768 ? advance_kernel<12> : advance_kernel<16>;
}

}  // namespace

int search_init_device()
{
    for (int d : {128, 384, 768, 1024})
        LEANN_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(advance_for(d)), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      LDS_LIMIT));
    return LEANN_OK;
}

int search_run(leann_ctx *ctx, const float *queries_dev, int64_t nq, const leann_graph *graph, const leann_pq *pq,
               const leann_chunks *chunks, const leann_emb_cache *cache, const leann_updates *upd, int32_t ef, int32_t k,
               float alpha, int32_t batch, int64_t *out_ids_dev, float *out_scores_dev, leann_search_stats *stats)
{
    const int d = ctx->desc.hidden, m_sub = pq->m_sub;
    const int64_t n = graph->n;
    hipStream_t st = ctx->stream;
    LEANN_TRY(ctx->s_misc.reserve(CTR_COUNT * sizeof(long long)));
    long long *counters = (long long *)ctx->s_misc.p;
    LEANN_HIP(hipMemsetAsync(counters, 0, CTR_COUNT * sizeof(long long), st));
    LEANN_TRY(clear_host_flags(ctx));
    hipLaunchKernelGGL(maxdeg_kernel, dim3(256), dim3(256), 0, st, graph->row_ptr, n, counters);
    if (!ctx->host_counters) LEANN_HIP(hipHostMalloc((void **)&ctx->host_counters, CTR_COUNT * sizeof(long long), hipHostMallocDefault));
    long long *h_ctr = ctx->host_counters;  // device kernels write it too: read after a synchronisation only
    const size_t ctr_bytes = CTR_COUNT * sizeof(long long);
    LEANN_HIP(hipMemcpyAsync(h_ctr, counters, ctr_bytes, hipMemcpyDeviceToHost, st));
    LEANN_HIP(hipStreamSynchronize(st));
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
    const int32_t aq_run = (int32_t)(((int64_t)aqcap + AQ_GROUPS_MAX * 64 - 1) / (AQ_GROUPS_MAX * 64) * 64);
    const int32_t aq_groups = (int32_t)(((int64_t)aqcap + aq_run - 1) / aq_run);
    const size_t o_eqk = carve((size_t)G * ef * 8), o_eqv = carve((size_t)G * ef), o_eqn = carve((size_t)G * 4);
    const size_t o_aqk = carve((size_t)G * aqcap * 8), o_aqm = carve((size_t)G * aq_groups * 8);
    const size_t o_aqt = carve((size_t)G * 4), o_aql = carve((size_t)G * 4), o_pend = carve((size_t)G * pcap * 4);
    const size_t o_np = carve((size_t)G * 4), o_src = carve((size_t)G * pcap * 4), o_own = carve((size_t)G * pcap * 4);
    const size_t o_done = carve((size_t)G * 4), o_nfl = carve((size_t)G * 4), o_eids = carve((size_t)G * pcap * 8);
    const int64_t memo_cap = std::min<int64_t>(ctx->memo_rows, (1 << 30) - 1);
    const size_t o_pick = carve(memo_cap > 0 ? (size_t)std::min<int64_t>(memo_cap, (int64_t)G * pcap) * 4 : 0);
    LEANN_TRY(ctx->s_state.reserve(off));
    LEANN_TRY(ctx->s_seen.reserve((size_t)G * words * 4));
    LEANN_TRY(ctx->s_lut.reserve((size_t)G * m_sub * KSUB * sizeof(float)));
    LEANN_TRY(ctx->s_emb.reserve((size_t)G * pcap * d * sizeof(float)));
    LEANN_TRY(ctx->s_owner.reserve((size_t)n * sizeof(unsigned long long)));
    LEANN_HIP(hipMemsetAsync(ctx->s_owner.p, 0xff, (size_t)n * sizeof(unsigned long long), st));
    // per-call embedding memo (leann_set_call_memo): empty at the start of every call
    int64_t memo_n = 0;
    if (memo_cap > 0) {
        LEANN_TRY(ctx->s_memo_slot.reserve((size_t)n * sizeof(int32_t)));
        LEANN_TRY(ctx->s_memo_emb.reserve((size_t)memo_cap * d * sizeof(float)));
        LEANN_HIP(hipMemsetAsync(ctx->s_memo_slot.p, 0xff, (size_t)n * sizeof(int32_t), st));
    }
    char *base = (char *)ctx->s_state.p;
    SearchState s;
    s.eq_key = (uint64_t *)(base + o_eqk);
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
    s.aq_run = aq_run;
    s.aq_groups = aq_groups;
    s.host_counters = h_ctr;
    s.slot_of = cache ? cache->slot_of : nullptr;
    s.cache_emb = cache ? cache->emb : nullptr;
    s.cache_rows = cache ? cache->rows : 0;

    const int table_smem = m_sub * KSUB * (int)sizeof(float) + ef * 9 + 16;
    if (table_smem > 150 * 1024) {
        leann_set_error("lookup table + queue of %d bytes exceed the LDS budget", table_smem);
        return LEANN_ESHAPE;
    }
    // what is left holds the head of AQ
    const int aq_room = (LDS_LIMIT - table_smem - aq_groups * 8) / (64 * 8) * 64;
    s.aq_lds = std::min(AQ_LDS_MAX, aq_room);
    const int adv_smem = table_smem + aq_groups * 8 + s.aq_lds * 8;
    const auto advance = advance_for(d);
    uint32_t launches = 0;

    struct Events : std::vector<hipEvent_t> {  // destroyed on every way out of this function
        ~Events()
        {
            for (hipEvent_t e : *this) (void)hipEventDestroy(e);
        }
    } evs;
    auto mark = [&]() -> int {
        hipEvent_t e;
        LEANN_HIP(hipEventCreate(&e));
        LEANN_HIP(hipEventRecord(e, st));
        evs.push_back(e);
        return LEANN_OK;
    };
    int rc = LEANN_OK;
    int64_t rounds = 0, encoded = 0;
    LEANN_TRY(mark());  // evs[0]: start
    for (int64_t q0 = 0; q0 < nq && rc == LEANN_OK; q0 += G) {
        const int g = (int)std::min<int64_t>(G, nq - q0);
        const float *qg = queries_dev + (size_t)q0 * d;
        LEANN_HIP(hipMemsetAsync(s.seen, 0, (size_t)g * words * 4, st));
        hipLaunchKernelGGL(init_kernel, dim3((g + 255) / 256), dim3(256), 0, st, s, g, graph->entry);
        LEANN_TRY(pq_build_lut(ctx, qg, g, pq, (float *)ctx->s_lut.p));
        for (bool have_results = false;; have_results = true) {
            LEANN_TRY(mark());
            {
                ProfScope prof(ctx, LEANN_PROF_TRAVERSE);
                hipLaunchKernelGGL(advance, dim3(g), dim3(ADV_THREADS), adv_smem, st, s, graph->row_ptr, graph->col_idx, n,
                                   pq->codes, m_sub, alpha, batch, qg, d, (const float *)ctx->s_emb.p, have_results, ++launches);
            }
            {
                ProfScope prof(ctx, LEANN_PROF_COLLECT);
                hipLaunchKernelGGL(collect_kernel, dim3(g), dim3(64), 0, st, s, chunks->lengths, chunks->seq);
            }
            LEANN_TRY(mark());
            LEANN_HIP(hipStreamSynchronize(st));
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
            LEANN_TRY(ctx->s_buf.reserve((size_t)g * nb * sizeof(float)));
            buf_scores = (const float *)ctx->s_buf.p;
            hipLaunchKernelGGL(buffer_score_kernel, dim3((nb + 3) / 4, g), dim3(256), 0, st, queries_dev + (size_t)q0 * d,
                               upd->buffer_emb, nb, d, (float *)ctx->s_buf.p);
        }
        hipLaunchKernelGGL(finalize_kernel, dim3(g), dim3(64), 0, st, s, k, upd ? upd->deleted_bits : nullptr, buf_scores,
                           upd ? upd->buffer_ids : nullptr, nb, out_ids_dev + (size_t)q0 * k,
                           out_scores_dev + (size_t)q0 * k);
    }
    if (rc == LEANN_OK) rc = mark();
    if (rc == LEANN_OK) {
        LEANN_HIP(hipMemcpyAsync(h_ctr, counters, ctr_bytes, hipMemcpyDeviceToHost, st));
    }
    hipError_t sync_rc = hipStreamSynchronize(st);
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
        float total = 0.f, trav = 0.f;
        (void)hipEventElapsedTime(&total, evs.front(), evs.back());
        // events come in (round start, after collect) pairs between the first and the last one
        for (size_t i = 1; i + 1 < evs.size(); i += 2) {
            float t = 0.f;
            (void)hipEventElapsedTime(&t, evs[i], evs[i + 1]);
            trav += t;
        }
        stats->total_ms = total;
        stats->traverse_ms = trav;
        stats->encoder_ms = total - trav;
    }
    return rc;
}
