// Graph construction by insertion (Algorithm 3 and the node-insertion listing of the update appendix) on the device.
//
// Nodes enter in id order, in batches: the nodes of a batch search the graph as it was before the batch (Algorithm 1
// with exact similarities from the stored embeddings), pick their neighbours with the RNG rule, then the forward and
// reverse edges of the batch are committed and every node that received edges is brought back under the degree cap M.
// With batch = 1 this is the sequential listing; larger batches are what fills the device (one block per
// inserted node).  Batch k holds min(batch, max(1, inserted / ramp)) nodes, so the first nodes still go in one by one.
#include "common.h"
#include "wave.h"

#include <algorithm>

namespace {

constexpr int EFC_MAX = 256;    // construction queue length
constexpr int M_MAX = 64;       // degree cap
constexpr int BATCH_MAX = 1024;  // nodes per batch
constexpr int LIST_MAX = M_MAX + BATCH_MAX;
constexpr int64_t BITMAP_NODES = 262144;  // visited marks of a search as a bitmap in LDS up to here (32 KB: four blocks per CU)

struct BuildState {
    const float *emb;   // [n][d]
    int d;
    int32_t *adj;       // [n][stride]
    int32_t *deg;       // [n] current list length
    int32_t *deg0;      // [n] list length when the batch started
    int stride;         // M + batch
    uint16_t *stamp;    // [batch][n] visited marks of the searches where a bitmap in LDS is too large: seen iff == epoch
    int64_t n;
    int32_t *fwd;       // [batch][M] neighbours chosen by the nodes of the batch
    int32_t *fwd_n;     // [batch]
    int32_t *touched;   // nodes that received reverse edges in this batch
    int32_t *n_touched;
    const uint8_t *is_hub;
    int M, m, efC;
};

__device__ inline const float *row_of(const BuildState &s, int id) { return s.emb + (size_t)id * s.d; }

// RNG selection among cnt candidates (keys of similarity to the anchor and id, best first, LDS) into out[] (LDS), at most
// cap: walk them in order; keep x unless a kept y is closer to x than the anchor is.  The whole block works on it: a group
// of as many candidates as there are wavefronts is checked at once, each wavefront its candidate against everything kept
// so far and, if it survives, against the earlier candidates of the group; which of those count is settled afterwards, in
// order.  Returns the number kept (uniform).
constexpr int WAVES_MAX = 16;

template <int NV>
__device__ inline int block_shrink(const BuildState &s, const uint64_t *key, int cnt, int cap, int32_t *out, uint32_t *flags)
{
    constexpr uint32_t DROPPED = 1u << 31;
    const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int kept = 0;
    for (int base = 0; base < cnt && kept < cap; base += nw) {
        uint32_t res = DROPPED;
        if (base + wave < cnt) {
            const uint64_t kx = key[base + wave];
            const int x = __builtin_amdgcn_readfirstlane((int)key_id(kx));
            const float bs = key_score(kx);
            RowDots<NV> dots;
            dots.load(s.emb + (size_t)x * s.d, s.d, lane);
            float dv[4];
            bool ok = true;
            for (int j = 0; j < kept && ok; j += 4) {
                const int c = min(4, kept - j);
                dots.four([&](int k) { return row_of(s, out[j + k]); }, c, dv);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k < c && dv[k] > bs) ok = false;
            }
            if (ok) {
                res = 0;
                for (int j = 0; j < wave; j += 4) {
                    const int c = min(4, wave - j);
                    dots.four([&](int k) { return row_of(s, (int)key_id(key[base + j + k])); }, c, dv);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (k < c && dv[k] > bs) res |= 1u << (j + k);
                }
            }
        }
        if (lane == 0) flags[wave] = res;
        __syncthreads();
        uint32_t group = 0;  // candidates of this group that are kept
        for (int b = 0; b < nw && kept < cap; ++b) {
            const uint32_t f = flags[b];
            if (f == DROPPED || (f & group)) continue;
            if (tid == 0) out[kept] = (int32_t)key_id(key[base + b]);
            group |= 1u << b;
            ++kept;
        }
        __syncthreads();
    }
    return kept;
}

// One block per node of the batch: Search(v, efC) on the graph of the first `inserted` nodes, then Shrink(W, M0).
// Latency bounds it: a hop is a chain of reads (list, vectors) and the next hop depends on its similarities.  So all the
// wavefronts of a block share a hop: the neighbours' similarities are taken side by side, and the queue W is kept sorted
// (two copies, the hop's newcomers are merged from one into the other by counting), which makes "closest not expanded" one
// ballot and dropping the worst a bound.  The next node to expand is the closest open entry of the queue before the hop (the
// runner-up, known while the vectors are on their way; its list is requested then) or the closest newcomer: wavefront 0
// takes it on, reads its list and marks its neighbours while the others merge the queue.
// Measured at n = 8192, d = 768, efC = 128, batches of up to 1024: 171 us per batch on average (a hop of 11 newcomers 3760
// clocks); 220 us (4800) with the merge before the next list and a wavefront's vectors one after the other.
// words > 0: the visited marks are a bitmap of that many words in LDS (the caller has made sure that it fits), else 16-bit
// stamps in memory.
template <int NV>
__global__ __launch_bounds__(64 * WAVES_MAX) void build_search_select_kernel(BuildState s, int64_t inserted, int epoch, int words)
{
    extern __shared__ uint32_t seen[];
    __shared__ __attribute__((aligned(16))) uint64_t w_key[2][EFC_MAX];  // 0 behind the last entry
    __shared__ __attribute__((aligned(4))) uint8_t w_vis[2][EFC_MAX];    // 1: expanded before the node of this hop, or no entry there
    __shared__ uint64_t new_key[64];
    __shared__ int32_t new_id[64], kept_ids[M_MAX];
    __shared__ uint32_t flags[WAVES_MAX];
    __shared__ int n_new_s;
    __shared__ uint64_t node_s;
    const int slot = blockIdx.x, tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t v = inserted + slot;
    if (slot == 0 && tid == 0) *s.n_touched = 0;  // counted by the commit kernel, which runs next
    if (inserted == 0) {  // the first node has nothing to link to
        if (tid == 0) s.fwd_n[slot] = 0;
        return;
    }
    uint16_t *stamp = s.stamp + (size_t)slot * s.n;
    RowDots<NV> dots;
    dots.load(s.emb + (size_t)v * s.d, s.d, lane);
    for (int i = tid; i < words; i += blockDim.x) seen[i] = i == 0;  // node 0 is the entry point: seen from the start
    for (int i = tid; i < 2 * EFC_MAX; i += blockDim.x) {
        (&w_key[0][0])[i] = 0;
        (&w_vis[0][0])[i] = 1;
    }
    __syncthreads();

    struct List {  // of a node: neighbour `lane` (any value from the list's end on) and the list's length, as they come from memory
        int32_t x, deg;
    };
    int zero = 0;
    asm volatile("" : "+v"(zero));  // a scalar load of the length would make the LDS reads behind it wait for memory
    auto list_of = [&](int u) -> List {  // deg <= M: lists are under the cap between batches
        return {s.adj[(size_t)u * s.stride + min(lane, s.stride - 1)], s.deg[u + zero]};
    };
    auto mark = [&](int32_t x) -> bool {  // x has not been met before
        if (words > 0) return !(atomicOr(&seen[x >> 5], 1u << (x & 31)) >> (x & 31) & 1u);
        if (x == 0 || stamp[x] == (uint16_t)epoch) return false;
        stamp[x] = (uint16_t)epoch;
        return true;
    };
    auto start_hop = [&](uint64_t node, const List &l) {  // wavefront 0: the neighbours to be scored
        const bool on = node != 0 && lane < l.deg && mark(l.x);
        const unsigned long long fresh = __ballot(on);
        if (on) new_id[__popcll(fresh & ((1ull << lane) - 1ull))] = l.x;
        if (lane == 0) {
            n_new_s = __popcll(fresh);
            node_s = node;
        }
    };
    float dv[4];
    if (wave == 0) {
        const List l = list_of(0);
        dots.four([&](int) { return s.emb; }, 1, dv);
        const uint64_t k = queue_key(dv[0], 0);
        if (lane == 0) {
            w_key[0][0] = k;
            w_vis[0][0] = 0;
        }
        start_hop(k, l);
    }
    __syncthreads();
    int n_w = 1, cur = 0;
    for (;;) {
        const int n_new = __builtin_amdgcn_readfirstlane(n_new_s);
        const uint64_t node = node_s;  // 0: every entry has been expanded
        if (node == 0) break;
        uint64_t runner = 0;
        List next_list = {0, 0};
        if (wave == 0) {  // the best entry that has not been expanded, besides this hop's: lane l looks at positions 4l .. 4l + 3
            static_assert(EFC_MAX == 256, "four entries per lane");
            const uint32_t open = ~reinterpret_cast<const uint32_t *>(w_vis[cur])[lane];
            uint64_t first = 0;
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                const uint64_t k = w_key[cur][4 * lane + i];
                if ((open >> (8 * i) & 1u) && k != node) first = k;
            }
            const unsigned long long any = __ballot(first != 0);
            if (any) {
                runner = key_of_lane(first, __ffsll((long long)any) - 1);
                next_list = list_of((int)key_id(runner));
            }
            if (lane >= n_new) new_key[lane] = 0;  // the padding of keys_above
        }
        for (int i0 = wave > 0 ? wave - 1 : nw - 1; i0 < n_new; i0 += 4 * nw) {
            const int c = min(4, (n_new - i0 + nw - 1) / nw);
            dots.four([&](int k) { return row_of(s, new_id[i0 + k * nw]); }, c, dv);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < c && lane == 0) new_key[i0 + k * nw] = queue_key(dv[k], (uint32_t)new_id[i0 + k * nw]);
        }
        __syncthreads();
        const uint64_t fresh_key = lane < n_new ? new_key[lane] : 0;
        const int nxt = cur ^ 1;
        if (wave == 0) {
            uint64_t best = wave_max_key(fresh_key);
            if (n_w == s.efC && best < w_key[cur][s.efC - 1]) best = 0;  // does not get into the queue
            // a runner-up that is better than every newcomer stays in the queue
            const uint64_t next = max(best, runner);
            if (next != runner) next_list = list_of((int)key_id(next));
            start_hop(next, next_list);
        } else {
            // Merge.  An entry moves down by the number of better newcomers.  Where there are lanes enough, four share an entry.
            const int share = (nw - 1) * 16 >= n_w ? 2 : 0;
            for (int e = tid - 64; e < n_w << share; e += blockDim.x - 64) {
                const int i = e >> share;
                const uint64_t k = w_key[cur][i];
                const uint8_t vis = w_vis[cur][i];
                int p = i;
                if (share) {
                    int above = 0;
                    for (int j = e & 3; j < n_new; j += 16)
#pragma unroll
                        for (int t = 0; t < 4; ++t) above += new_key[j + 4 * t] > k;
                    above += (int)dpp_mov<DPP_QUAD_XOR1>((uint32_t)above);
                    above += (int)dpp_mov<DPP_QUAD_XOR2>((uint32_t)above);
                    p += above;
                } else {
                    p += keys_above(new_key, n_new, k);
                }
                if ((share == 0 || (e & 3) == 0) && p < s.efC) {
                    w_key[nxt][p] = k;
                    w_vis[nxt][p] = vis | (uint8_t)(k == node);
                }
            }
            // A newcomer lands behind everything better, old or new; the wavefronts that have no entries begin.
            if (nw - 1 - wave < n_new) {
                uint64_t own[EFC_MAX / 64];
#pragma unroll
                for (int j = 0; j < EFC_MAX / 64; ++j) own[j] = w_key[cur][j * 64 + lane];
                for (int i = nw - 1 - wave; i < n_new; i += nw - 1) {
                    const uint64_t k = key_of_lane(fresh_key, i);
                    int p = __popcll(__ballot(fresh_key > k));
#pragma unroll
                    for (int j = 0; j < EFC_MAX / 64; ++j) p += __popcll(__ballot(own[j] > k));
                    if (p < s.efC && lane == 0) {
                        w_key[nxt][p] = k;
                        w_vis[nxt][p] = 0;
                    }
                }
            }
        }
        n_w = min(n_w + n_new, s.efC);
        cur = nxt;
        __syncthreads();
    }
    const int cap = (!s.is_hub || s.is_hub[v]) ? s.M : s.m;
    const int kept = block_shrink<NV>(s, w_key[cur], n_w, cap, kept_ids, flags);
    if (tid < kept) s.fwd[(size_t)slot * s.M + tid] = kept_ids[tid];
    if (tid == 0) s.fwd_n[slot] = kept;
}

// Forward lists of the batch's nodes, reverse edges appended to their targets (order fixed later), targets noted.
__global__ __launch_bounds__(64) void build_commit_kernel(BuildState s, int64_t inserted)
{
    const int slot = blockIdx.x, lane = threadIdx.x;
    const int64_t v = inserted + slot;
    const int cnt = s.fwd_n[slot];
    if (lane < cnt) {
        const int32_t r = s.fwd[(size_t)slot * s.M + lane];
        s.adj[(size_t)v * s.stride + lane] = r;
        const int pos = atomicAdd(&s.deg[r], 1);  // < deg0[r] + batch <= stride
        s.adj[(size_t)r * s.stride + pos] = (int32_t)v;
        if (pos == s.deg0[r]) s.touched[atomicAdd(s.n_touched, 1)] = r;
    }
    if (lane == 0) {
        s.deg[v] = cnt;
        s.deg0[v] = cnt;
    }
}

// One block per node that received reverse edges: put the new edges in id order (the order of insertion), and if the
// list exceeds M shrink it with the RNG rule anchored at the node (up to M * cnt / 2 similarities, shared by the block's
// wavefronts: 20 us per batch at the sizes above, 347 with one wavefront).
template <int NV>
__global__ __launch_bounds__(64 * WAVES_MAX) void build_reverse_kernel(BuildState s)
{
    __shared__ int32_t list[LIST_MAX];
    __shared__ uint64_t key[LIST_MAX], sorted[LIST_MAX];
    __shared__ int32_t kept_ids[M_MAX];
    __shared__ uint32_t flags[WAVES_MAX];
    const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= *s.n_touched) return;
    const int r = __builtin_amdgcn_readfirstlane(s.touched[blockIdx.x]);
    const int cnt = s.deg[r], old = s.deg0[r];
    int32_t *row = s.adj + (size_t)r * s.stride;
    if (cnt <= s.M) {  // at most 64 entries: a lane's appended id goes behind the smaller ones (all are different)
        if (wave > 0) return;
        const int32_t x = lane >= old && lane < cnt ? row[lane] : 0x7fffffff;
        int rank = old;
        for (int j = old; j < cnt; ++j) rank += __builtin_amdgcn_readlane(x, j) < x;
        if (lane >= old && lane < cnt) row[rank] = x;
        if (lane == 0) s.deg0[r] = cnt;
        return;
    }
    for (int i = tid; i < cnt; i += blockDim.x) list[i] = row[i];
    __syncthreads();
    RowDots<NV> dots;
    dots.load(s.emb + (size_t)r * s.d, s.d, lane);
    for (int i0 = wave; i0 < cnt; i0 += 4 * nw) {
        const int c = min(4, (cnt - i0 + nw - 1) / nw);
        float dv[4];
        dots.four([&](int k) { return row_of(s, list[i0 + k * nw]); }, c, dv);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < c && lane == 0) key[i0 + k * nw] = queue_key(dv[k], (uint32_t)list[i0 + k * nw]);
    }
    static_assert(LIST_MAX % 8 == 0, "keys_above's padding");
    if (tid < (-cnt & 7)) key[cnt + tid] = 0;
    __syncthreads();
    for (int i = tid; i < cnt; i += blockDim.x) {
        const uint64_t k = key[i];
        sorted[keys_above(key, cnt, k)] = k;
    }
    __syncthreads();
    const int kept = block_shrink<NV>(s, sorted, cnt, s.M, kept_ids, flags);
    if (tid < kept) row[tid] = kept_ids[tid];
    if (tid == 0) {
        s.deg[r] = kept;
        s.deg0[r] = kept;
    }
}

// CSR out of the fixed-stride lists: row_ptr by a chunked scan in one block, then a wavefront per node copies its list.
__global__ __launch_bounds__(1024) void build_row_ptr_kernel(BuildState s, uint64_t *__restrict__ row_ptr)
{
    __shared__ unsigned long long part[1024];
    const int tid = threadIdx.x;
    const int64_t per = (s.n + 1023) / 1024;
    const int64_t beg = tid * per, end = beg + per < s.n ? beg + per : s.n;
    unsigned long long sum = 0;
    for (int64_t v = beg; v < end; ++v) sum += (unsigned long long)s.deg[v];
    part[tid] = sum;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const unsigned long long t = tid >= o ? part[tid - o] : 0;
        __syncthreads();
        part[tid] += t;
        __syncthreads();
    }
    unsigned long long run = tid ? part[tid - 1] : 0;
    for (int64_t v = beg; v < end; ++v) {
        row_ptr[v] = run;
        run += (unsigned long long)s.deg[v];
    }
    if (tid == 1023) row_ptr[s.n] = part[1023];
}

__global__ __launch_bounds__(256) void build_col_idx_kernel(BuildState s, const uint64_t *__restrict__ row_ptr,
                                                            uint32_t *__restrict__ col_idx)
{
    const int lane = threadIdx.x & 63;
    for (int64_t v = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); v < s.n; v += (int64_t)gridDim.x * 4)
        if (lane < s.deg[v]) col_idx[row_ptr[v] + lane] = (uint32_t)s.adj[(size_t)v * s.stride + lane];  // deg <= M <= 64
}

// Flags of the ceil(beta * n) nodes of largest out-degree, ties to the lower id.  One block: histogram of the degrees,
// the threshold degree, then the lowest ids at the threshold by a chunked count.
__global__ __launch_bounds__(1024) void top_degree_kernel(const uint64_t *__restrict__ row_ptr, int64_t n, int64_t want,
                                                          uint8_t *__restrict__ is_hub, int *__restrict__ err)
{
    constexpr int DMAX = 4096;
    __shared__ unsigned int hist[DMAX + 1];
    __shared__ unsigned long long part[1024];
    __shared__ int thr_s;
    __shared__ long long need_s;
    const int tid = threadIdx.x;
    for (int i = tid; i <= DMAX; i += 1024) hist[i] = 0;
    __syncthreads();
    const int64_t per = (n + 1023) / 1024;
    const int64_t beg = tid * per, end = beg + per < n ? beg + per : n;
    for (int64_t v = beg; v < end; ++v) {
        const unsigned long long dv = row_ptr[v + 1] - row_ptr[v];
        if (dv > DMAX) {
            atomicOr(err, 1);
            continue;
        }
        atomicAdd(&hist[dv], 1u);
    }
    __syncthreads();
    if (tid == 0) {
        long long left = want;
        int t = DMAX;
        while (t > 0 && left > (long long)hist[t]) left -= hist[t--];
        thr_s = t;         // degrees above t are all in; `left` of those at t (lowest ids)
        need_s = left;
    }
    __syncthreads();
    const int thr = thr_s;
    const long long need = need_s;
    unsigned long long at = 0;
    for (int64_t v = beg; v < end; ++v) at += (row_ptr[v + 1] - row_ptr[v]) == (unsigned long long)thr;
    part[tid] = at;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const unsigned long long t = tid >= o ? part[tid - o] : 0;
        __syncthreads();
        part[tid] += t;
        __syncthreads();
    }
    long long before = tid ? (long long)part[tid - 1] : 0;
    for (int64_t v = beg; v < end; ++v) {
        const unsigned long long dv = row_ptr[v + 1] - row_ptr[v];
        uint8_t flag = 0;
        if (dv <= DMAX) {
            if ((int)dv > thr) flag = 1;
            else if ((int)dv == thr) flag = before++ < need;
        }
        is_hub[v] = flag;
    }
}

// The construction kernels for rows of d elements.
struct BuildKernels {
    void (*search_select)(BuildState, int64_t, int, int);
    void (*reverse)(BuildState);
};

BuildKernels build_kernels(int d)
{
    if (d <= 128) return {build_search_select_kernel<2>, build_reverse_kernel<2>};
    if (d <= 256) return {build_search_select_kernel<4>, build_reverse_kernel<4>};
    if (d <= 384) return {build_search_select_kernel<6>, build_reverse_kernel<6>};
    if (d <= 512) return {build_search_select_kernel<8>, build_reverse_kernel<8>};
    if (d <= 768) return {build_search_select_kernel<12>, build_reverse_kernel<12>};
    if (d <= 1024) return {build_search_select_kernel<16>, build_reverse_kernel<16>};
    return {build_search_select_kernel<0>, build_reverse_kernel<0>};
}

}  // namespace

int leann_build_graph(leann_ctx *ctx, const float *emb_dev, int64_t n, int32_t d, const uint8_t *is_hub_dev, int32_t efC,
                      int32_t M, int32_t m, int32_t batch, int32_t ramp, uint64_t *row_ptr_dev, uint32_t *col_idx_dev,
                      int64_t *n_edges_host)
{
    if (!ctx || !emb_dev || !row_ptr_dev || !col_idx_dev || n < 1 || d < 1) {
        leann_set_error("leann_build_graph: null argument or empty input");
        return LEANN_EINVAL;
    }
    if (efC < 1 || efC > EFC_MAX || M < 1 || M > M_MAX || m < 1 || m > M || batch < 1 || batch > BATCH_MAX || ramp < 1 ||
        n > 0x7fffffffll) {
        leann_set_error("leann_build_graph: need 1 <= efC <= %d, 1 <= m <= M <= %d, 1 <= batch <= %d, ramp >= 1, n < 2^31",
                        EFC_MAX, M_MAX, BATCH_MAX);
        return LEANN_EINVAL;
    }
    LEANN_HIP(hipSetDevice(ctx->device));
    hipStream_t st = ctx->stream;
    const int stride = M + batch;
    DevBuf adj, deg, stamp, misc;
    int rc = LEANN_OK;
    auto done = [&](int code) {
        (void)hipStreamSynchronize(st);
        adj.release();
        deg.release();
        stamp.release();
        misc.release();
        return code;
    };
    if ((rc = ctx->reserve(adj, (size_t)n * stride * sizeof(int32_t))) != LEANN_OK) return done(rc);
    if ((rc = ctx->reserve(deg, (size_t)n * 2 * sizeof(int32_t))) != LEANN_OK) return done(rc);
    const int words = n <= BITMAP_NODES ? (int)((n + 31) / 32) : 0;
    if (words == 0 && (rc = ctx->reserve(stamp, (size_t)batch * n * sizeof(uint16_t))) != LEANN_OK) return done(rc);
    const size_t fwd_bytes = (size_t)batch * M * sizeof(int32_t);
    if ((rc = ctx->reserve(misc, fwd_bytes + (size_t)batch * sizeof(int32_t) + (size_t)batch * M * sizeof(int32_t) + 256)) != LEANN_OK)
        return done(rc);
    BuildState s;
    s.emb = emb_dev;
    s.d = d;
    s.adj = (int32_t *)adj.p;
    s.deg = (int32_t *)deg.p;
    s.deg0 = s.deg + n;
    s.stride = stride;
    s.stamp = (uint16_t *)stamp.p;
    s.n = n;
    s.fwd = (int32_t *)misc.p;
    s.fwd_n = s.fwd + (size_t)batch * M;
    s.touched = s.fwd_n + batch;
    s.n_touched = s.touched + (size_t)batch * M;
    s.is_hub = is_hub_dev;
    s.M = M;
    s.m = m;
    s.efC = efC;
    hipError_t e = hipMemsetAsync(deg.p, 0, (size_t)n * 2 * sizeof(int32_t), st);
    if (e == hipSuccess && words == 0) e = hipMemsetAsync(stamp.p, 0, (size_t)batch * n * sizeof(uint16_t), st);
    const BuildKernels kernels = build_kernels(d);
    int epoch = 0;
    for (int64_t ins = 0; ins < n && e == hipSuccess;) {
        int64_t b = std::max<int64_t>(1, ins / ramp);
        b = std::min<int64_t>(std::min<int64_t>(b, batch), n - ins);
        if (words == 0 && ++epoch == 65536) {  // the 16-bit marks wrap: start over with clean ones
            e = hipMemsetAsync(stamp.p, 0, (size_t)batch * n * sizeof(uint16_t), st);
            epoch = 1;
            if (e != hipSuccess) break;
        }
        // Wavefronts per node: 16 per CU in all, so that small batches, which are bound by one node's chain of hops, spread each
        // hop widest.  That is what the registers let stay on a CU at d = 768 and 1024 (98 and 122); they are 58 to 66 up to
        // d = 384.  8192 nodes, efC 128, batches up to 1024: 16.3 ms at d = 768 and 19.2 at d = 1024; with 8 up to 256 nodes 16.4 and
        // 19.3, with 16 up to 512 17.6 and 20.4, with 4 from 257 on 17.2 and 19.9, with 8 from 257 on 16.9 and 19.5.  At d = 128 and
        // 384, 8 from 257 on would take 11.9 and 13.3 instead of 12.2 and 13.8.
        const int threads = 64 * (b <= ctx->num_cus ? 16 : b <= 2 * ctx->num_cus ? 8 : 4);
        hipLaunchKernelGGL(kernels.search_select, dim3((unsigned)b), dim3(threads), words * sizeof(uint32_t), st, s, ins,
                           epoch, words);
        hipLaunchKernelGGL(build_commit_kernel, dim3((unsigned)b), dim3(64), 0, st, s, ins);
        // a node receives edges at most once per batch into the list of touched ones, and only inserted nodes do
        if (ins > 0)
            hipLaunchKernelGGL(kernels.reverse, dim3((unsigned)std::min<int64_t>(b * M, ins)), dim3(512), 0, st, s);
        ins += b;
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(build_row_ptr_kernel, dim3(1), dim3(1024), 0, st, s, row_ptr_dev);
        hipLaunchKernelGGL(build_col_idx_kernel, dim3((unsigned)std::min<int64_t>((n + 3) / 4, 8192)), dim3(256), 0, st, s,
                           row_ptr_dev, col_idx_dev);
        e = hipGetLastError();
    }
    unsigned long long edges = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&edges, row_ptr_dev + n, sizeof(edges), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        leann_set_error("leann_build_graph: %s", hipGetErrorString(e));
        return done(LEANN_EDEVICE);
    }
    if (n_edges_host) *n_edges_host = (int64_t)edges;
    return done(LEANN_OK);
}

int leann_top_degree(leann_ctx *ctx, const uint64_t *row_ptr_dev, int64_t n, double beta, uint8_t *is_hub_dev)
{
    if (!ctx || !row_ptr_dev || !is_hub_dev || n < 1 || !(beta >= 0.0) || beta > 1.0) {
        leann_set_error("leann_top_degree: null argument, empty graph or beta outside [0, 1]");
        return LEANN_EINVAL;
    }
    LEANN_HIP(hipSetDevice(ctx->device));
    LEANN_TRY(ctx->reserve(ctx->meta, 256));
    int *err = (int *)ctx->meta.p;
    LEANN_HIP(hipMemsetAsync(err, 0, sizeof(int), ctx->stream));
    int64_t want = (int64_t)ceil(beta * (double)n);
    if (want > n) want = n;
    hipLaunchKernelGGL(top_degree_kernel, dim3(1), dim3(1024), 0, ctx->stream, row_ptr_dev, n, want, is_hub_dev, err);
    LEANN_HIP(hipGetLastError());
    int h_err = 0;
    LEANN_HIP(hipMemcpyAsync(&h_err, err, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    LEANN_HIP(hipStreamSynchronize(ctx->stream));
    if (h_err) {
        leann_set_error("leann_top_degree: a node has more than 4096 neighbours");
        return LEANN_ECAPACITY;
    }
    return LEANN_OK;
}
