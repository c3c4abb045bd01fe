// Search with the finished index (Alg. 1) for gfx950: the trees give a query its first
// candidates, the kNN graph expands them (NN-expansion).
//
// One wave per query (a few when there are few queries), queries grid-strided over blocks.
//   1. trees   lane t searches tree t for the N_node = P / S / T + 1 closest leaves, best
//              bin first: going down it takes the child on the query's side of the split and
//              puts the other aside with the priority of the branch it follows plus the
//              squared distance from the query's coordinate to the node's mean; after a leaf
//              it continues from the branch with the smallest (priority, link) put aside.
//              Priorities are float64, computed with the same operations as any other
//              implementation of this rule would use (one division, one fused multiply-add).
//   2. pool    the members of those leaves are looked up in the set of checked points, those that
//              are new to it wait until 64 are there, are evaluated together (four lanes per
//              row, the library's fixed-order distance) and merged into the pool, a sorted
//              list in LDS of at most E keys.
//   3. expand  `iters` times: every pool member that has not been expanded yet hands in its
//              graph neighbours; those not checked before are evaluated and merged, the pool
//              keeping the P closest.
// "Checked" is a hash set in LDS; a query that fills it moves it to one in the block's slice of the
// workspace, and from there perhaps to a larger one; their entries carry the number of the query they
// belong to (cleared when a block first needs them, never between queries).  Queries that find nothing near check
// thousands of points, so it has to be cheap: 20 000 queries of 50 000 x 96, half of them uniform (4500 checked on
// average, up to 10 000), rows of 50, pool of 200: 11.6 ms; with look-ups in the full set and in the other 35,
// with the workspace's set alone 14.0.
// Bound: fetching the rows.  100 000 queries against 10^6 x 128, pool of 200: 37.6 GB at the fabric in 6.25 ms
// = 6.0 TB/s, a copy reaches 6.2.  (12.5 ms with the set in memory, batches of 64 neighbours
// evaluated whether four or sixty of them were new, and counting merges.)
#include "common.h"

namespace {

constexpr int kMaxPool = 1024;
constexpr size_t kLdsLimit = 160 * 1024;

struct Branch {
    double prio;
    int link;
    int pad;
};

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// What the waves of a block tell one another, a word of LDS each: a word that stood for two things could be
// written for the one before every wave has read the other.
enum { kWaiting, kToExpand, kPoolMembers, kSharedWords };

// LDS of a block, offsets in words
struct SearchLds {
    int cur, batch, keys, expand, fid, leaves, lofs, found, shared, tab;
};
__host__ __device__ inline SearchLds search_lds(int d, int P, int T, int want, int max_first, int W, bool q_lds)
{
    SearchLds l;
    l.cur = q_lds ? (d + 15) & ~15 : 0;
    l.batch = l.cur + 2 * P;
    l.keys = l.batch + 2 * EF_WAVE;
    l.expand = l.keys + (W > 1 ? 2 * EF_WAVE * W : 0);
    l.fid = l.expand + (P > max_first ? P : max_first);
    l.leaves = l.fid + 5 * EF_WAVE * W;
    l.lofs = l.leaves + T * want;
    l.found = l.lofs + T * want + 1;
    l.shared = l.found + T;
    l.tab = (l.shared + kSharedWords + 3) & ~3;
    return l;
}

struct SearchShape {
    int want;           // leaves per tree
    int heap_cap;       // branches one tree can have put aside
    int max_first;      // most points the trees can hand in
    int table;          // entries of a block's slice for sets of checked points (power of two)
    int waves;          // blocks, a query at a time each (of w waves)
    size_t heap_bytes, table_bytes, roots_bytes, bytes;
    int lds_slots, w;   // entries of the LDS set, waves per query
    bool q_lds;
    size_t lds;
    bool ok;
};

// LDS is handed out in pieces of 1280 bytes, 128 of them per CU.
constexpr size_t kLdsGranule = 1280;
constexpr int kLdsGranules = 128;

// Waves per query.  A query is a chain of dependent steps (down the trees, look up, fetch, merge, look
// up ...): with few queries its length is the call's time, and more waves make every step of it
// wider; with many the chip is full and the waves that wait for wave 0's merges are lost.  100 000 x 128,
// pool of 100, 1 / 4 / 8 waves: 64 queries 152 / 107 / 100 us, 256: 170 / 118 / 113, 512: 180 / 125 / 173,
// 1024: 186 / 187 / 303.  (Either side of the lines at 50 000 x 32 and x 960, pools of 40 and 400: 256 queries on eight waves
// 66, 147, 153, 253 us, 300 on four 68, 166, 161, 320; 768 on four 72, 170, 190, 430, 800 on one 81, 226, 222, 505.)
inline int waves_per_query(int64_t nq) { return nq <= 256 ? 8 : nq <= 768 ? 4 : 1; }

SearchShape search_shape(int64_t nq, int d, int T, int S, int tree_depth, int Kg, int P, int iters)
{
    SearchShape sh;
    sh.want = P / S / T + 1;
    sh.heap_cap = sh.want * (tree_depth + 2) + 2;      // a descent puts aside one branch per level
    sh.max_first = sh.want * T * S;
    long most = (long)sh.max_first + (long)iters * P * Kg;
    sh.table = 64;
    while (sh.table < 2 * most) sh.table <<= 1;
    // blocks: twice what is resident at a time evens out queries of different length
    sh.waves = (int)(nq < 1024 * 6 ? nq : 1024 * 6);
    if (sh.waves < 1) sh.waves = 1;
    sh.heap_bytes = align_up((size_t)sh.waves * T * sh.heap_cap * sizeof(Branch));
    sh.table_bytes = align_up((size_t)sh.waves * sh.table * 8);
    sh.roots_bytes = align_up((size_t)T * 4);
    sh.bytes = sh.heap_bytes + sh.table_bytes + sh.roots_bytes;
    // The documented limit: query, pool, a batch's keys, expansion list, leaf members and leaves in 160 KB.
    sh.ok = (size_t)((d + 15) & ~15) * 4 + (size_t)P * 8 + 64 * 8 + (size_t)P * 4 + (size_t)sh.max_first * 4 +
                (size_t)T * sh.want * 4 + (size_t)T * 4 + 64 <= kLdsLimit;
    if (!sh.ok) return sh;
    sh.w = waves_per_query(nq);
    sh.q_lds = true;
    auto base = [&]() { return (size_t)search_lds(d, P, T, sh.want, sh.max_first, sh.w, sh.q_lds).tab * 4; };
    sh.lds_slots = 0;
    if (sh.w > 1) {      // few queries: LDS is there for the asking
        sh.lds_slots = sh.w == 8 ? 8192 : 4096;
        if (base() + (size_t)sh.lds_slots * 4 > kLdsLimit) {
            sh.w = 1;
            sh.lds_slots = 0;
        }
    }
    if (sh.w == 1) {
        if (base() + 256 > kLdsLimit) sh.q_lds = false;      // (vectors of forty thousand coordinates)
        // As many blocks per CU as leave a set that few queries overflow where they find near neighbours (the
        // number of points checked grows slowly with the pool: 370, 500, 630, 830, 1030 on average for 50 .. 800),
        // a multiple of the four SIMDs: P = 200 with 12 / 11 blocks 6.4 / 8.2 ms per 10^5 queries, P = 400
        // with 9 / 8 blocks 16.0 / 13.9.  Fewer than eight only where they leave next to no set, or while four
        // hold all queries: P = 1000 with 8 / 4 blocks 58 / 71 ms, of the queries described above 32 / 55 per
        // 20 000, but 1000 queries 1.60 / 1.05.
        const long need = 1400 + P / 2;
        for (int blocks : {12, 8, 4, 2, 1}) {
            const size_t room = (size_t)(kLdsGranules / blocks) * kLdsGranule;
            if (room < base() + 256) continue;
            const long slots = (long)((room - base()) / 16 * 4);
            sh.lds_slots = (int)(slots < 8192 ? slots : 8192);
            if (slots >= need || (blocks == 8 && slots >= 1024 && nq > 4 * 256)) break;
        }
    }
    sh.lds = base() + (size_t)sh.lds_slots * 4;
    return sh;
}

struct LeafCounts {      // the trees' leaf counts, handed to the kernels by value
    int of[EFANNA_MAX_TREES];
};

// root of every tree: the node without a parent (0 for a tree that is a single leaf)
__global__ void find_roots_kernel(const efanna_node *__restrict__ nodes, int max_leaves, int T,
                                  LeafCounts n_leaves, int *roots)
{
    const int t = blockIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    if (j == 0 && n_leaves.of[t] <= 1) roots[t] = 0;
    if (j >= 1 && j < n_leaves.of[t] && nodes[(size_t)t * (max_leaves + 1) + j].parent < 0) roots[t] = j;
}

// The sets of checked points in a block's slice of the workspace: kSmallSet entries at its start, then half the
// slice, which holds all that a query can check (a slice of no more than two small ones: a single set, all of
// it).  A block clears a set before its first use, and half a megabyte instead of two is most of what a
// short call pays for sets that overflow (2000 queries of 50 000 x 32, pool of 1000: 1.95 -> 1.41 ms).
constexpr int kSmallSet = 65536;
// id joins such a set; true if it was not in it.  Entries are
// tag << 32 | id, the tag naming the query, so that one query's entries are free slots to the next.
__device__ inline bool checked_insert(u64 *table, int mask, u32 tag, int id)
{
    u32 h = (u32)(ef_mix64((u64)(u32)id) >> 40) & (u32)mask;
    const u64 mine = ((u64)tag << 32) | (u32)id;
    for (int probes = 0; probes <= mask; ++probes) {
        u64 v = table[h];
        while ((u32)(v >> 32) != tag) {      // free, or left over from another query
            const u64 old = atomicCAS(&table[h], v, mine);
            if (old == v) return true;
            v = old;
        }
        if (v == mine) return false;
        h = (h + 1) & (u32)mask;
    }
    return false;      // (every id of the query is in it: a set has a slot for each)
}
// The same set in LDS (ids, -1 = free; never more than fifteen sixteenths full).
// BUCKETS: of four slots, which one read brings; they fill in order and are never freed, so whoever finds the id
// absent and takes the first free slot has it alone, and whoever loses that slot looks again (10^5 x 128, pool of
// 400: 12.9 -> 12.5 ms per 10^5 queries, 200 000 x 32 with rows of 100: 4.1 -> 2.9 per 20 000).  Else slot by slot: one
// trip to LDS where most slots are free, which is so for few queries (a single one: 62.5 us instead of 64).
template <bool BUCKETS>
__device__ inline bool checked_lds(int *tab, int slots, int id)      // true: was not in it
{
    if (!BUCKETS) {
        int h = (int)__umulhi((u32)id * 0x9E3779B1u, (u32)slots);
        for (;;) {
            const int v = atomicCAS(&tab[h], -1, id);
            if (v == -1) return true;
            if (v == id) return false;
            h = h + 1 == slots ? 0 : h + 1;
        }
    }
    int h = 4 * (int)__umulhi((u32)id * 0x9E3779B1u, (u32)slots >> 2);
    for (;;) {
        const int4 four = *reinterpret_cast<const int4 *>(tab + h);
        if (four.x == id || four.y == id || four.z == id || four.w == id) return false;
        const int at = four.x == -1 ? 0 : four.y == -1 ? 1 : four.z == -1 ? 2 : four.w == -1 ? 3 : -1;
        if (at < 0) {
            h = h + 4 >= slots ? 0 : h + 4;
            continue;
        }
        const int v = atomicCAS(&tab[h + at], -1, id);
        if (v == -1) return true;
        if (v == id) return false;
    }
}

// The library's distance between the query (LDS) and the row of every lane's candidate (`id`, lanes
// 0 .. cnt-1 have one), by the whole wave: sixteen candidates at a time, four lanes each.  Lane
// (r, g) = lane r + 16 g loads the 16-byte pieces 16 s + 4 g of row r, so that four lanes fetch 64
// contiguous bytes and every byte fetched is used (a lane reading a whole row alone touches 64 rows
// per load and finds their lines evicted before it comes back for the rest); it accumulates
// partial sums 4g..4g+3 of the fixed order, and the four lanes of a row add up 8 apart, 4
// apart, 2 apart, 1 apart.  The candidate of lane 16 g + r is handled in round g by column r,
// so the lane that owns it is among the four that end up with its distance.  Two rounds' rows
// travel together.
// Requires d % 4 == 0 and a 16-byte aligned X; PADDED: q holds zeros from d up to a multiple of 16.
template <bool PADDED>
__device__ inline float wave_distances(const float *q, const float *__restrict__ X, int d, int id, int cnt)
{
    const int lane = ef_lane(), r16 = lane & 15, g = lane >> 4;
    float mine = 0.0f;
    for (int round = 0; 16 * round < cnt; round += 2) {
        const bool both = 16 * (round + 1) < cnt;
        const float *row[2];
        float p[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {      // (a lane without a candidate reads row 0 along)
            row[h] = X + (size_t)max(__shfl(id, 16 * (round + h) + r16, EF_WAVE), 0) * d;
            p[h][0] = p[h][1] = p[h][2] = p[h][3] = 0.0f;
        }
        for (int c0 = 0; c0 < d; c0 += 128) {
            float4 v[2][8];
            const int n_whole = (d - c0) >> 4;      // sixteens that lie inside (uniform)
            const bool tail_in = 16 * n_whole + 4 * g < d - c0;      // d % 4 == 0: a piece is in or out
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && !both) break;
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    v[h][s] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (s < n_whole || (s == n_whole && tail_in))
                        v[h][s] = *reinterpret_cast<const float4 *>(row[h] + c0 + 4 * g + 16 * s);
                }
            }
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if (c0 + 16 * s >= d) break;
                const int j = c0 + 16 * s + 4 * g;      // (zeros beyond d on both sides)
                const float4 y = PADDED || j + 3 < d ? *reinterpret_cast<const float4 *>(q + j) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (h == 1 && !both) break;
                    const float d0 = y.x - v[h][s].x, d1 = y.y - v[h][s].y, d2 = y.z - v[h][s].z, d3 = y.w - v[h][s].w;
                    p[h][0] = __builtin_fmaf(d0, d0, p[h][0]);
                    p[h][1] = __builtin_fmaf(d1, d1, p[h][1]);
                    p[h][2] = __builtin_fmaf(d2, d2, p[h][2]);
                    p[h][3] = __builtin_fmaf(d3, d3, p[h][3]);
                }
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int k = 0; k < 4; ++k) p[h][k] += __shfl_xor(p[h][k], 32, EF_WAVE);
#pragma unroll
            for (int k = 0; k < 4; ++k) p[h][k] += __shfl_xor(p[h][k], 16, EF_WAVE);
            const float dist = (p[h][0] + p[h][2]) + (p[h][1] + p[h][3]);
            if (g == round + h) mine = dist;
        }
    }
    return mine;
}

// orders the LDS accesses of one wave (its LDS operations complete in program order)
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Merge the wave's batch (one key per lane, ~0 = none) into the sorted pool (count keys, room for
// cap), in place.  Returns the new count.  Keys are distinct.
// The fresh keys are packed to the front of `batch` and ranked among each other (every lane looks at
// all of them, eight at a time), and put in order; a pool member then finds the number of fresh keys
// below it with a binary search, a fresh key the number of pool members below it.  (Counting for
// the pool members as well was two thirds of the search's instructions: P = 200 9.4 -> 8.0 ms
// per 10^5 queries, P = 800 41 -> 31.8.)  Pool members below the smallest fresh key stay where
// they are; the others move up by the number of fresh keys below
// them, 64 at a time from the top (a chunk is read before it is written, and it only writes at
// or above its own places), and the fresh keys take the places left free.
__device__ inline int pool_merge(u64 *pool, int count, int cap, u64 key, u64 *batch)
{
    const int lane = ef_lane();
    const u64 there = __ballot(key != ~0ULL);
    const int fresh = __popcll(there);
    if (lane >= fresh) batch[lane] = ~0ULL;
    if (key != ~0ULL) batch[__popcll(there & ((1ULL << lane) - 1))] = key;
    wave_sync();
    int rank = 0;
    for (int o = 0; o < fresh; o += 8) {
#pragma unroll
        for (int k = 0; k < 8; ++k) rank += batch[o + k] < key ? 1 : 0;
    }
    int lo = count;
    if (key != ~0ULL) {
        int hi = count;
        lo = 0;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (pool[mid] < key) lo = mid + 1;
            else hi = mid;
        }
    }
    wave_sync();
    if (key != ~0ULL) batch[rank] = key;
    wave_sync();
    const int first = __shfl(lo, __ffsll((unsigned long long)__ballot(key != ~0ULL && rank == 0)) - 1, EF_WAVE);
    int step0 = 1;                   // a power of two above half the fresh keys
    while (2 * step0 <= fresh) step0 <<= 1;
    for (int top = count; top > first; top -= EF_WAVE) {
        const int j = top - EF_WAVE + lane;
        u64 e = 0;
        int up = 0;
        if (j >= first) {
            e = pool[j];
            for (int step = step0; step > 0; step >>= 1)
                if (up + step <= EF_WAVE && batch[up + step - 1] < e) up += step;
        }
        wave_sync();                 // the chunk is in registers before any of it is overwritten
        if (j >= first && j + up < cap) pool[j + up] = e;
        wave_sync();
    }
    if (key != ~0ULL && lo + rank < cap) pool[lo + rank] = key;
    wave_sync();
    return min(cap, count + fresh);
}

// W waves per query.  The waves of a block look candidates up together and evaluate 64 each; wave 0
// searches the trees and keeps the pool.
// Q_LDS: the query sits in LDS (else, for vectors that fill it, it is read from memory every time).
template <int W, bool Q_LDS>
__global__ void __launch_bounds__(W * EF_WAVE) __attribute__((amdgpu_waves_per_eu(3)))
search_kernel(const float *__restrict__ X, int d, int n, const int *__restrict__ perm,
              const int *__restrict__ leaf_off, int max_leaves, LeafCounts n_leaves,
              const efanna_node *__restrict__ nodes, const int *__restrict__ roots, int T, int S,
              const int *__restrict__ graph_ids, int Kg, u32 kg_magic, const float *__restrict__ queries, int nq,
              int K, int P, int E, int iters, int want, int heap_cap, int max_first, int table_size, int lds_slots,
              Branch *heaps, u64 *tables, int *out_ids, float *out_dists, int *out_checked)
{
    extern __shared__ __align__(16) float smem[];
    constexpr int kThreads = W * EF_WAVE;
    const SearchLds at = search_lds(d, P, T, want, max_first, W, Q_LDS);
    u64 *cur = (u64 *)(smem + at.cur);                 // [P] the pool, ascending
    u64 *batch = (u64 *)(smem + at.batch);             // [64]
    u64 *keys = (u64 *)(smem + at.keys);               // [64 W] evaluated candidates on their way to wave 0 (W > 1)
    int *expand = (int *)smem + at.expand;             // [P] members whose neighbours are next; before that
    int *first = expand;                               // [max_first] members of the leaves found
    int *fid = (int *)smem + at.fid;                   // [320 W] candidates waiting to be evaluated
    int *leaves = (int *)smem + at.leaves;             // [T][want] leaves, then where they start
    int *lofs = (int *)smem + at.lofs;                 // [T][want] where their members start in `first`, and the end
    int *n_found = (int *)smem + at.found;             // [T]
    int *shared = (int *)smem + at.shared;             // [kSharedWords] candidates waiting, members to expand, pool members at the end
    int *tab = (int *)smem + at.tab;                   // [lds_slots] points checked (the trees' branches before that)
    const int dq = (d + 15) & ~15;
    const int tid = threadIdx.x, lane = ef_lane(), wave = tid / EF_WAVE;
    u64 *table = tables + (size_t)blockIdx.x * table_size;
    const int small_set = table_size > 2 * kSmallSet ? kSmallSet : table_size, large_set = table_size / 2;
    const int lds_limit = lds_slots - lds_slots / 16;
    int cleared = 0;      // entries of the largest set of the block's slice that has been cleared
    const bool lds_heap = (size_t)T * heap_cap * sizeof(Branch) <= (size_t)lds_slots * 4;
    for (int qi = blockIdx.x; qi < nq; qi += gridDim.x) {
        const u32 tag = (u32)qi + 1u;
        __syncthreads();                  // the previous query's LDS reads are done
        const float *q = Q_LDS ? smem : queries + (size_t)qi * d;      // in LDS: [dq], zeros from d on
        if (Q_LDS)
            for (int j = tid; j < dq; j += kThreads) smem[j] = j < d ? queries[(size_t)qi * d + j] : 0.0f;
        __syncthreads();
        // ---- 1. trees: lane t searches tree t -----------------------------------------------
        for (int t = tid; t < T; t += kThreads) {
            const efanna_node *nd_t = nodes + (size_t)t * (max_leaves + 1);
            const int last = n_leaves.of[t] - 1;
            Branch *heap = lds_heap ? (Branch *)tab + t * heap_cap : heaps + ((size_t)blockIdx.x * T + t) * heap_cap;
            int n_heap = 0, found = 0;
            int link = last <= 0 ? ~0 : roots[t];
            double prio = 0.0;
            for (;;) {
                for (int steps = 0; link >= 0 && steps < 4096; ++steps) {      // down to a leaf
                    const efanna_node nd = nd_t[min(link, last)];
                    bool left = true;
                    double other = prio;
                    if (ef_has_test(nd.dim)) {
                        const long long diff = (long long)nd.cnt * ef_node_value([&](int j) { return q[j]; }, d, nd.dim) - nd.sum;
                        left = diff < 0;
                        const double gap = (double)diff / ((double)nd.cnt * 1048576.0);
                        other = __fma_rn(gap, gap, prio);
                    }
                    if (n_heap < heap_cap) {
                        heap[n_heap].prio = other;
                        heap[n_heap].link = nd.child[left ? 1 : 0];
                        ++n_heap;
                    }
                    link = nd.child[left ? 0 : 1];
                }
                leaves[t * want + found++] = link >= 0 ? 0 : min(~link, max(last, 0));
                if (found == want || n_heap == 0) break;
                int best = 0;
                double bp = heap[0].prio;
                int bl = heap[0].link;
                for (int h = 1; h < n_heap; ++h) {
                    const double hp = heap[h].prio;
                    const int hl = heap[h].link;
                    if (hp < bp || (hp == bp && hl < bl)) {
                        best = h;
                        bp = hp;
                        bl = hl;
                    }
                }
                prio = bp;
                link = bl;
                --n_heap;
                heap[best] = heap[n_heap];
            }
            n_found[t] = found;
        }
        __syncthreads();
        // ---- 2. the members of the leaves found; nothing is checked yet -----------------------
        for (int j = tid; j < lds_slots / 4; j += kThreads) reinterpret_cast<int4 *>(tab)[j] = make_int4(-1, -1, -1, -1);
        const int n_lists = T * want;
        if (wave == 0) {
            int end = 0;
            for (int l0 = 0; l0 < n_lists; l0 += EF_WAVE) {
                const int l = l0 + lane;
                int b = 0, s = 0;
                if (l < n_lists) {
                    const int t = l / want;
                    if (l - t * want < n_found[t]) {
                        const int *off = leaf_off + (size_t)t * (max_leaves + 1) + leaves[l];
                        b = off[0];
                        s = max(0, min(off[1] - b, S));
                    }
                }
                const int upto = end + ef_wave_scan_i32(s);
                if (l < n_lists) {
                    leaves[l] = b;
                    lofs[l] = upto - s;
                }
                end = __shfl(upto, EF_WAVE - 1, EF_WAVE);
            }
            if (lane == 0) {
                lofs[n_lists] = end;
                shared[kWaiting] = 0;
            }
        }
        __syncthreads();
        for (int l = tid >> 4; l < n_lists; l += kThreads / 16) {
            const int at0 = lofs[l], s = lofs[l + 1] - at0;
            const int *src = perm + (size_t)(l / want) * n + leaves[l];
            for (int r = tid & 15; r < s; r += 16) first[at0 + r] = src[r];
        }
        __syncthreads();
        int count = 0, checked = 0;      // count: kept by wave 0
        int set_size = 0;                // entries of the workspace set in use (0: the set in LDS)
        u64 *set = table;
        int waiting = 0;
        // ---- 3. the first pool from the leaves' members (it = -1), then NN-expansion -----------------
        for (int it = -1; it < iters; ++it) {
            int total = lofs[n_lists];
            const int cap = it < 0 ? E : P;
            if (it >= 0) {
                // members not expanded yet (mark bit set) lose the mark and go to the list
                int n_exp = 0;
                if (wave == 0) {
                    for (int j0 = 0; j0 < count; j0 += EF_WAVE) {
                        const int j = j0 + lane;
                        const u64 e = j < count ? cur[j] : 0;
                        const bool take = j < count && (e & 1);
                        const u64 bal = __ballot(take);
                        if (take) {
                            cur[j] = e & ~1ULL;
                            expand[n_exp + __popcll(bal & ((1ULL << lane) - 1))] = ef_id(e);
                        }
                        n_exp += __popcll(bal);
                    }
                    if (W > 1 && lane == 0) shared[kToExpand] = n_exp;
                }
                __syncthreads();
                if (W > 1) n_exp = shared[kToExpand];
                if (n_exp == 0) break;
                total = n_exp * Kg;
            }
            // Looks the candidates up, four per thread at a time, and evaluates those that were never
            // checked before in full batches: most neighbours of neighbours were (four in five at a
            // pool of 200), and the rows of a batch cost the same however many of its lanes have one.
            for (int f0 = 0; f0 < total; f0 += 4 * kThreads) {
                const int then = checked + min(total - f0, 4 * kThreads);
                if (set_size == 0 ? then > lds_limit : set_size < large_set && then > set_size - set_size / 4) {
                    // on to the next larger set: all threads, what was checked so far goes along
                    const int size = set_size == 0 ? small_set : large_set;
                    u64 *to = set_size == 0 ? table : table + large_set;
                    if (cleared < size) {
                        for (int j = tid; j < size / 2; j += kThreads) reinterpret_cast<uint4 *>(to)[j] = make_uint4(0, 0, 0, 0);
                        cleared = size;
                        __threadfence();      // (the cleared entries are in place before any wave swaps one)
                        __syncthreads();
                    }
                    if (set_size == 0) {
                        for (int j = tid; j < lds_slots; j += kThreads)
                            if (tab[j] >= 0) checked_insert(to, size - 1, tag, tab[j]);
                    } else {
                        for (int j = tid; j < set_size; j += 4 * kThreads) {
                            u64 v[4];
#pragma unroll
                            for (int k = 0; k < 4; ++k) v[k] = j + k * kThreads < set_size ? ef_load_coherent(set + j + k * kThreads) : 0;
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                if ((u32)(v[k] >> 32) == tag) checked_insert(to, size - 1, tag, (int)(u32)v[k]);
                        }
                    }
                    set = to;
                    set_size = size;
                    __syncthreads();
                }
                int id[4];
                u64 new_mask[4];
                int n_new = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int f = f0 + k * kThreads + tid;
                    id[k] = -1;
                    if (f < total) {
                        if (it < 0) {
                            id[k] = first[f];
                        } else {
                            const int src = kg_magic ? (int)(((u64)(u32)f * kg_magic) >> 32) : f / Kg;
                            id[k] = graph_ids[(size_t)expand[src] * Kg + (f - src * Kg)];
                        }
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    bool fresh = false;
                    if (id[k] >= 0 && id[k] < n) {
                        fresh = set_size == 0 ? checked_lds<W == 1>(tab, lds_slots, id[k])
                                              : checked_insert(set, set_size - 1, tag, id[k]);
                    }
                    new_mask[k] = __ballot(fresh);
                    n_new += __popcll(new_mask[k]);
                }
                int to = waiting;
                if (W > 1) {
                    if (lane == 0 && n_new) to = atomicAdd(&shared[kWaiting], n_new);
                    to = __shfl(to, 0, EF_WAVE);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if ((new_mask[k] >> lane) & 1) fid[to + __popcll(new_mask[k] & ((1ULL << lane) - 1))] = id[k];
                    to += __popcll(new_mask[k]);
                }
                __syncthreads();
                const int now = W > 1 ? shared[kWaiting] : waiting + n_new;
                checked += now - waiting;
                waiting = now;
                const bool last = f0 + 4 * kThreads >= total;
                while (waiting >= kThreads || (last && waiting > 0)) {
                    // up to 64 candidates per wave are evaluated and merged into the pool
                    const int cnt = min(waiting, kThreads), mine = min(cnt - EF_WAVE * wave, EF_WAVE);
                    waiting -= cnt;
                    u64 key = ~0ULL;
                    if (mine > 0) {
                        const int c = lane < mine ? fid[waiting + EF_WAVE * wave + lane] : -1;
                        const float dist = wave_distances<Q_LDS>(q, X, d, c, mine);
                        if (c >= 0) key = ef_pack(dist, c, 1);
                    }
                    if (W > 1) {
                        keys[tid] = key;
                        __syncthreads();
                    }
                    if (wave == 0)
                        for (int c0 = 0; c0 < cnt; c0 += EF_WAVE) {
                            if (W > 1) key = keys[c0 + lane];
                            if (count == cap && key >= cur[cap - 1]) key = ~0ULL;      // a full pool takes nothing beyond its last key
                            if (__ballot(key != ~0ULL) != 0) count = pool_merge(cur, count, cap, key, batch);
                        }
                    __syncthreads();
                }
                if (W > 1) {
                    __syncthreads();      // everyone has read the count
                    if (tid == 0) shared[kWaiting] = waiting;
                    __syncthreads();
                }
            }
        }
        // ---- result: the K closest --------------------------------------------------------------
        if (W > 1) {
            if (tid == 0) shared[kPoolMembers] = count;      // (a late wave may still be reading what there was to expand)
            __syncthreads();
            count = shared[kPoolMembers];
        }
        for (int c = tid; c < K; c += kThreads) {
            const bool live = c < count;
            out_ids[(size_t)qi * K + c] = live ? ef_id(cur[c]) : -1;
            out_dists[(size_t)qi * K + c] = live ? __uint_as_float(ef_dist_bits(cur[c])) : __uint_as_float(EF_INF_BITS);
        }
        if (out_checked && tid == 0) out_checked[qi] = checked;
    }
}

}  // namespace

extern "C" size_t efanna_search_workspace_bytes(int64_t nq, int32_t d, int32_t n_trees,
                                                int32_t leaf_size, int32_t tree_depth,
                                                int32_t graph_k, int32_t pool, int32_t iters)
{
    if (nq < 1 || d < 1 || n_trees < 1 || leaf_size < 1 || graph_k < 1 || pool < 1 || iters < 0 ||
        tree_depth < -1)
        return 0;
    return search_shape(nq, d, n_trees, leaf_size, tree_depth, graph_k, pool, iters).bytes;
}

extern "C" int efanna_search(const float *X, int64_t n, int32_t d, const int32_t *perm,
                             const int32_t *leaf_off, int32_t max_leaves, const int32_t *n_leaves,
                             const efanna_node *nodes, int32_t tree_depth, int32_t n_trees,
                             int32_t leaf_size, const int32_t *graph_ids, int32_t graph_k,
                             const float *queries, int64_t nq, int32_t k, int32_t pool,
                             int32_t expand, int32_t iters, int32_t *ids, float *dists,
                             int32_t *checked, void *ws, size_t ws_bytes, void *stream)
{
    if (!X || !perm || !leaf_off || !n_leaves || !nodes || !graph_ids || !queries || !ids || !dists)
        return EFANNA_EINVAL;
    if (n < 1 || d < 1 || n_trees < 1 || n_trees > EFANNA_MAX_TREES || leaf_size < 1 ||
        leaf_size > EFANNA_MAX_LEAF || max_leaves < 1 || graph_k < 1 || nq < 1 || k < 1 || pool < k ||
        expand < 1 || expand > pool || iters < 0 || tree_depth < -1 || n >= 2147483647LL - 256 ||
        nq >= 2147483647LL - 256)
        return EFANNA_EINVAL;
    for (int t = 0; t < n_trees; ++t)
        if (n_leaves[t] < 1 || n_leaves[t] > max_leaves) return EFANNA_EINVAL;
    if (pool > kMaxPool || (d & 3) || ((uintptr_t)X & 15) || ((uintptr_t)queries & 15) || tree_depth > 4000)
        return EFANNA_EUNSUPPORTED;
    const SearchShape sh = search_shape(nq, d, n_trees, leaf_size, tree_depth, graph_k, pool, iters);
    if (!sh.ok) return EFANNA_EUNSUPPORTED;
    if (!ws || ((uintptr_t)ws & 255) || ws_bytes < sh.bytes) return EFANNA_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)ws;
    Branch *heaps = (Branch *)base;
    u64 *tables = (u64 *)(base + sh.heap_bytes);
    int *roots = (int *)(base + sh.heap_bytes + sh.table_bytes);
    LeafCounts counts = {};
    for (int t = 0; t < n_trees; ++t) counts.of[t] = n_leaves[t];
    find_roots_kernel<<<dim3((unsigned)((max_leaves + 255) / 256), (unsigned)n_trees), 256, 0, st>>>(
        nodes, max_leaves, n_trees, counts, roots);
    // f / graph_k as f * kg_magic >> 32 for the f < pool * graph_k there are: ceil(2^32 / graph_k) is less than
    // graph_k / 2^32 of it too large, so exact while f * graph_k <= 2^32.  Rows too long for that (or of one id): 0, divide.
    const u32 kg_magic = graph_k > 1 && (u64)graph_k * graph_k * pool <= 1ULL << 32
                             ? (u32)(((1ULL << 32) + graph_k - 1) / graph_k) : 0;
#define EF_SEARCH(W, Q_LDS)                                                                              \
    do {                                                                                                 \
        EF_HIP_CHECK(hipFuncSetAttribute((const void *)search_kernel<W, Q_LDS>,                          \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh.lds));      \
        search_kernel<W, Q_LDS><<<sh.waves, (W) * EF_WAVE, sh.lds, st>>>(                                \
            X, d, (int)n, perm, leaf_off, max_leaves, counts, nodes, roots, n_trees, leaf_size,          \
            graph_ids, graph_k, kg_magic, queries, (int)nq, k, pool, expand, iters, sh.want,             \
            sh.heap_cap, sh.max_first, sh.table, sh.lds_slots, heaps, tables, ids, dists, checked);      \
    } while (0)
    if (!sh.q_lds) EF_SEARCH(1, false);
    else if (sh.w == 1) EF_SEARCH(1, true);
    else if (sh.w == 4) EF_SEARCH(4, true);
    else EF_SEARCH(8, true);
#undef EF_SEARCH
    EF_HIP_CHECK(hipGetLastError());
    // (the call is documented to wait)
    EF_HIP_CHECK(hipStreamSynchronize(st));
    return EFANNA_OK;
}
