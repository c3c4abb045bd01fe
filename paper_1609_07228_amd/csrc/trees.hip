// Randomized truncated KD-trees (Alg. 2) for gfx950.
//
// All trees are built together, one level per launch group.  The ids of tree t live in
// positions [t*n, (t+1)*n) of one array of T*n "positions"; a node is a segment of
// positions.  Per level:
//   1. sum      every position adds its quantised coordinate (on the node's dimension)
//               to the node's 64-bit integer sum (wave-reduced when a wave lies inside
//               one node, integer atomics otherwise: exact in any order);
//   2. scan     the "goes left" predicate cnt*q(x) < sum as bits with a device-wide prefix sum of their
//               counts, from which every position derives its rank inside
//               its node, i.e. a stable partition without any per-node launch;
//   3. children one thread per node fixes the split point, appends the children that
//               still hold more than leaf_size points to the next level's node table
//               and marks the first position of children that became leaves;
//   4. scatter  every position moves its id to its place in the child segment.
// The host reads one counter per level (the number of nodes of the next level).
#include "common.h"

namespace {

constexpr int kBlock = 256;
constexpr int kScanItems = 8;                       // per thread
constexpr int kScanTile = kBlock * kScanItems;      // positions per scan block

struct Node {
    int b, e;        // segment of positions [b, e)
    u64 heap;        // heap id: root 1, children 2h, 2h+1
    long long sum;   // sum of quantised coordinates
    int dim;         // split dimension, -1: positional split only (depth cap)
    int depth;
    int mid;         // first position of the right child
    int moved;       // 1: mean split, 0: positional halves (ids stay where they are)
    int child[2];    // index in the next level's table, -1 if that child is a leaf
    int parent;      // position where the parent's right part starts, -1 for a root
    int left_before; // positions before b that go left in their nodes (see LeftCount)
};
static_assert(sizeof(Node) == 56, "the workspace has room for records of that size");

struct Counters {
    int n_nodes[2];     // live nodes of level l in n_nodes[l & 1]; children_kernel fills the other one
    int bad_input;
    int small_nodes;
    int max_depth;      // deepest internal node (only tracked with node export)
    int wide_input;     // some |x| >= kNarrow
};

// A node small enough to be finished inside one workgroup (finish_kernel).
struct SmallNode {
    int b, e;
    u64 heap;
    int depth, parent;      // parent: as in Node
};

// Record of an internal node kept for the conquer step above the leaves (Alg. 3), stored at
// the position where the node's right part starts (unique per node).  child[s] >= 0: the
// position that identifies an internal child, < 0: ~(first position of a leaf child).  Every
// field is written exactly once: sum .. depth by the node itself, child[s] by the node for a
// leaf child and by the child for an internal one.
struct NodeRec {
    long long sum;
    int dim, cnt, parent, depth;
    int child[2];
};
static_assert(sizeof(NodeRec) == sizeof(efanna_node), "record and exported node share a layout");

__device__ inline void record_node(NodeRec *rec, int *leaf_rec, int mid, long long sum, int dim,
                                   int cnt, int parent, int depth)
{
    NodeRec &r = rec[mid];
    r.sum = sum;
    r.dim = dim;
    r.cnt = cnt;
    r.parent = parent;
    r.depth = depth;
    if (parent >= 0) rec[parent].child[mid > parent ? 1 : 0] = mid;
    (void)leaf_rec;
}
__device__ inline void record_leaf(NodeRec *rec, int *leaf_rec, int b, int parent)
{
    leaf_rec[b] = parent;
    if (parent >= 0) rec[parent].child[b >= parent ? 1 : 0] = ~b;
}

// What a finish_kernel block takes: segments of at most fin_max positions, kFinNodes of them per level at most, four
// positions to a thread.  Splits by one coordinate take twice as much as the other rules: a level less of the device-wide
// kernels, which cost six launches (builds of 10^4 x 32 778 -> 752 us, 200 003 x 50 4.77 -> 4.72 ms, 10^6 x 128 15.89 -> 15.77).  Splits by variance
// have no registers for a thousand threads, projections are the faster the fewer rows they read at a time.
constexpr int kFinNodes = 512;     // nodes of one level inside a segment, at most
__host__ __device__ constexpr int fin_max(int rule) { return rule == EFANNA_SPLIT_UNIFORM ? 4096 : 2048; }
constexpr int kFinFew = 512;        // points up to which a position per thread is enough (see finish_kernel)
__host__ __device__ constexpr int fin_threads(int rule) { return fin_max(rule) / 4; }
inline int finish_limit(int S, int rule)
{
    const long f = (long)kFinNodes * (S + 1);     // so that a level never has more than kFinNodes live nodes
    return f < fin_max(rule) ? (int)f : fin_max(rule);
}


// Transposed copy XT[d][n] of the data, with the input check folded in.  The splits read
// one coordinate of many points: in the row-major layout the upper levels (ids still
// nearly consecutive) would touch one 4-byte word out of every row, a stride that keeps
// hitting the same memory channels; in the transposed copy those reads are contiguous.
// Tiles of 64 x 64, 16 bytes per load and store (at any multiple of four bytes); the pitch of 65
// spreads both ways through the tile over all banks.  (32 x 32 tiles with 4-byte accesses: 10^6 x 960
// 2.06 -> 1.51 ms, 10^6 x 128 255 -> 192 us.)
constexpr int kTrTile = 64;
constexpr float kNarrow = 256.0f;      // below it eight quantised coordinates add up in 32 bits, a hundred squares in 64
__global__ void __launch_bounds__(kBlock)
transpose_check_kernel(const float *__restrict__ X, int n, int d, float *__restrict__ XT, Counters *c, double terms)
{
    __shared__ float tile[kTrTile][kTrTile + 1];      // [coordinate][point]
    const int t4 = 4 * (threadIdx.x & 15), t16 = threadIdx.x >> 4;      // 16 threads along, 16 across
    const int r0 = blockIdx.x * kTrTile, c0 = blockIdx.y * kTrTile;
    bool bad = false;
    float largest = 0.0f;
#pragma unroll
    for (int k = 0; k < kTrTile / 16; ++k) {
        const int row = r0 + t16 + 16 * k, col = c0 + t4;
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row < n) {
            const float *src = X + (size_t)row * d + col;
            if (col + 3 < d) {
                const ef_f32x4_u w = *reinterpret_cast<const ef_f32x4_u *>(src);
                v[0] = w.x, v[1] = w.y, v[2] = w.z, v[3] = w.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (col + j < d) v[j] = src[j];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bad |= !(fabsf(v[j]) < 1048576.0f);      // NaN and inf as well
            largest = fmaxf(largest, fabsf(v[j]));
            tile[t4 + j][t16 + 16 * k] = v[j];
        }
    }
    // n |x| < 2^43 keeps cnt * q(x) and the sums below 2^63 (terms: how many coordinates a node's test
    // adds up, 1 or kProjectionTerms)
    bad |= (double)largest * (double)n * terms >= 8796093022208.0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTrTile / 16; ++k) {
        const int col = c0 + t16 + 16 * k, row = r0 + t4;
        if (col >= d) continue;
        const float *src = &tile[t16 + 16 * k][t4];
        float *dst = XT + (size_t)col * n + row;
        if (row + 3 < n) {
            ef_f32x4_u w;
            w.x = src[0], w.y = src[1], w.z = src[2], w.w = src[3];
            *reinterpret_cast<ef_f32x4_u *>(dst) = w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (row + j < n) dst[j] = src[j];
        }
    }
    if (__any(bad) && ef_lane() == 0) atomicOr(&c->bad_input, 1);
    if (__any(!(largest < kNarrow)) && ef_lane() == 0) c->wide_input = 1;      // (whoever writes it writes a 1)
}

// ---------------------------------------------------------------------------------------
// Split dimension by variance (split_rule 1), the rule of the randomized KD-tree that Sec. 3.2
// takes over: over the node's first kVarSample positions, the kVarDims dimensions with the
// largest integer variance m * sum(q^2) - sum(q)^2 of the quantised coordinates (equal ones:
// the smaller dimension first); the node's draw picks one of them.  One whole wave per node:
// lane l takes dimensions l, l + 64, ... and keeps its own best five in registers, then five
// rounds of a wave-wide maximum pop the overall order.  `ids` may point into LDS or global
// memory; every lane of the wave must call with the same arguments.
constexpr int kVarSample = 100, kVarDims = 5;

// The largest of the wave's values, in every lane: exchanges inside the rows of sixteen lanes by lane permutations of the vector
// ALU, then of rows and half waves.
__device__ inline u32 ef_wave_max_u32(u32 v)
{
#define EF_MAX_DPP(CTRL) v = max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false))
    EF_MAX_DPP(0xB1);       // lanes 0 <-> 1, 2 <-> 3
    EF_MAX_DPP(0x4E);       // lanes 0, 1 <-> 2, 3
    EF_MAX_DPP(0x141);      // the halves of a row, mirrored
    EF_MAX_DPP(0x140);      // the row mirrored
#undef EF_MAX_DPP
    const u32 a = max((u32)__builtin_amdgcn_readlane((int)v, 0), (u32)__builtin_amdgcn_readlane((int)v, 16));
    return max(a, max((u32)__builtin_amdgcn_readlane((int)v, 32), (u32)__builtin_amdgcn_readlane((int)v, 48)));
}
constexpr int kDimPending = -2;      // Node::dim of a node whose dimension is still to be chosen

struct VarKey {
    __int128 v;
    int j;
};
__device__ inline bool var_before(const VarKey &a, const VarKey &b)
{
    return a.v > b.v || (a.v == b.v && a.j < b.j);
}

// What bounds this: the rows of the samples, up to 100 whole rows per node and level.  Two dimensions
// per lane and eight rows are fetched together (one row at a time left a node waiting for a hundred
// memory round trips in turn).  A value is taken apart into whole units and steps, q = hi 2^20 + lo with
// |hi|, |lo| <= 2^20: truncation, the fraction and its 2^20-fold are exact in float32, the steps round
// as q does (hi 2^20 is even), the products and sums of a hundred of them fit 64 bits whatever the values,
// and only the result is put together in 128.  10^6 x 128, eight trees of leaves of 16: the in-LDS finish
// 14.9 -> 5.0 ms, the levels above 3.05 -> 0.32.  Where all |x| < 256 (the pass that checks the input says so) q fits 29 bits:
// eight of them add up in 32, a hundred squares in 64, five instructions per value instead of eleven.  With that,
// rows addressed from scalar registers (the compiler had masked the choice of the id per lane), a lane's own best two instead of five
// up to 128 dimensions and the wave's maximum by lane permutations: 5.13 -> 3.61 and 0.32 -> 0.18 (wide values: the tree build of 10^6 x 128 7.75 -> 6.54 ms, others 7.85 -> 6.18).  (Sums of q - q(first row) in 64 bits, with a second pass in 128
// where values lie 256.0 or more apart: 9.0 and 0.55; with that pass 10^4 x 32 took 1.20 ms in all, now 0.79.)
template <bool NARROW, bool ONE>      // all |x| < kNarrow; d <= 128: one pass over the dimensions, two to a lane
__device__ inline int variance_dim_wave(const float *__restrict__ X, int d, const int *ids, int cnt, u64 draw)
{
    const int lane = ef_lane();
    // (uniform, and said to be: the sample's rows are addressed from scalar registers)
    const int m = __builtin_amdgcn_readfirstlane(cnt < kVarSample ? cnt : kVarSample);
    const int id_lo = ids[min(lane, m - 1)], id_hi = m > EF_WAVE ? ids[min(EF_WAVE + lane, m - 1)] : 0;
    constexpr int N = ONE ? 2 : kVarDims;      // (a lane's own best)
    VarKey top[N];
#pragma unroll
    for (int r = 0; r < N; ++r) {
        top[r].v = -1;      // below every variance
        top[r].j = 0x7FFFFFFF;
    }
    for (int j0 = 0; j0 < (ONE ? 1 : d); j0 += 2 * EF_WAVE) {
        const int j[2] = {j0 + lane, j0 + EF_WAVE + lane};
        const int jc[2] = {min(j[0], d - 1), min(j[1], d - 1)};      // (lanes beyond d read along)
        const bool second = j0 + EF_WAVE < d;
        int s_hi[2] = {0, 0}, s_lo[2] = {0, 0};                             // sums of hi and lo
        long long s_hh[2] = {0, 0}, s_hl[2] = {0, 0}, s_ll[2] = {0, 0};     // ... of hi^2, hi lo and lo^2
        long long s_q[2] = {0, 0}, s_qq[2] = {0, 0};                        // narrow values: sums of q and q^2
        for (int p0 = 0; p0 < m; p0 += 8) {
            float x[2][8];
            const float *row[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int p = min(p0 + u, m - 1), lo = __builtin_amdgcn_readlane(id_lo, p & 63), hi = __builtin_amdgcn_readlane(id_hi, p & 63);
                row[u] = X + (size_t)(p < EF_WAVE ? lo : hi) * d;
                x[0][u] = row[u][jc[0]];
            }
            if (second) {
#pragma unroll
                for (int u = 0; u < 8; ++u) x[1][u] = row[u][jc[1]];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && !second) break;
                if (NARROW) {
                    int sum = 0;      // (eight values of less than 2^28)
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int q = p0 + u < m ? (int)__builtin_rintf(x[h][u] * 1048576.0f) : 0;
                        sum += q;
                        s_qq[h] += (long long)q * q;
                    }
                    s_q[h] += sum;
                    continue;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (p0 + u >= m) break;
                    const float whole = __builtin_truncf(x[h][u]);
                    const int hi = (int)whole, lo = (int)__builtin_rintf((x[h][u] - whole) * 1048576.0f);
                    s_hi[h] += hi;
                    s_lo[h] += lo;
                    s_hh[h] += (long long)hi * hi;
                    s_hl[h] += (long long)hi * lo;
                    s_ll[h] += (long long)lo * lo;
                }
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 1 && !second) break;
            VarKey c;
            c.j = j[h];
            const long long s1 = NARROW ? s_q[h] : (long long)s_hi[h] * 1048576 + s_lo[h];
            const __int128 s2 = NARROW ? (__int128)s_qq[h] : (__int128)s_hh[h] * ((__int128)1 << 40) + (__int128)s_hl[h] * ((__int128)1 << 21) + s_ll[h];
            c.v = s2 * m - (__int128)s1 * s1;
            if (j[h] >= d) continue;
            if (j0 == 0 && h == 0) {      // (up to 128 dimensions a lane has two: one comparison puts them in order)
                top[0] = c;
            } else if (j0 == 0) {
                top[1] = c;
                if (var_before(c, top[0])) {
                    top[1] = top[0];
                    top[0] = c;
                }
            } else {
#pragma unroll
                for (int r = 0; r < N; ++r)
                    if (var_before(c, top[r])) {
                        const VarKey t = top[r];
                        top[r] = c;
                        c = t;
                    }
            }
        }
    }
    const int want = d < kVarDims ? (int)(draw % (u64)d) : (int)(draw % (u64)kVarDims);
    int chosen = 0;
    for (int r = 0; r <= want; ++r) {      // (uniform)
        // the largest of the lanes' best: by the leading 64 bits of variances below 2^71 (all bits of
        // them where one is larger), the rare ties among those exactly
        const u64 head = top[0].v < 0 ? 0 : (u64)(top[0].v >> 64) >= 128 ? ~0ULL : (u64)(top[0].v >> 7);
        const u32 high = ef_wave_max_u32((u32)(head >> 32));
        const u64 best = (u64)high << 32 | ef_wave_max_u32((u32)(head >> 32) == high ? (u32)head : 0u);
        u64 tied = __ballot(head == best && top[0].v >= 0);
        int winner = __ffsll((unsigned long long)tied) - 1;
        if (tied & (tied - 1)) {
            VarKey w;
            w.v = -1;
            w.j = 0x7FFFFFFF;
            for (u64 left = tied; left; left &= left - 1) {
                const int l = __ffsll((unsigned long long)left) - 1;
                VarKey k;
                const u64 lo = __shfl((u64)top[0].v, l, EF_WAVE), hi = __shfl((u64)(top[0].v >> 64), l, EF_WAVE);
                k.v = (__int128)(((unsigned __int128)hi << 64) | lo);
                k.j = __shfl(top[0].j, l, EF_WAVE);
                if (var_before(k, w)) {
                    w = k;
                    winner = l;
                }
            }
        }
        chosen = __shfl(top[0].j, winner, EF_WAVE);
        if (lane == winner) {      // the winner's lane moves on to its next one
#pragma unroll
            for (int q = 0; q + 1 < N; ++q) top[q] = top[q + 1];
            top[N - 1].v = -1;
            top[N - 1].j = 0x7FFFFFFF;
        }
    }
    return chosen;
}

// a fresh node's dimension code from its draw: the coordinate, "to be chosen by variance", or a projection
__device__ inline int node_dim(int rule, u64 draw, int d)
{
    return rule == 1 ? kDimPending : rule == 2 ? ef_projection_code(draw) : (int)(draw % (u64)d);
}

// One wave per live node of the level: fixes the dimension of the nodes that wait for one.
template <bool NARROW, bool ONE>
__global__ void __launch_bounds__(kBlock)
choose_dims_kernel(const float *__restrict__ X, int d, int n, const int *__restrict__ perm, Node *nodes,
                   int *dims, const Counters *c, int level, u64 seed)
{
    const int n_cur = c->n_nodes[level & 1];
    const int n_waves = gridDim.x * (kBlock / EF_WAVE);
    for (int s = blockIdx.x * (kBlock / EF_WAVE) + threadIdx.x / EF_WAVE; s < n_cur; s += n_waves) {
        const int b = nodes[s].b, e = nodes[s].e;
        if (nodes[s].dim != kDimPending) continue;      // (uniform)
        const u64 draw = ef_mix64(ef_stream_key(seed, b / n) + nodes[s].heap);
        const int dim = variance_dim_wave<NARROW, ONE>(X, d, perm + b, e - b, draw);
        if (ef_lane() == 0) {
            nodes[s].dim = dim;
            dims[s] = dim;
        }
    }
}

__global__ void roots_kernel(Node *nodes, int *dims, int *node_of, unsigned char *leaf_flag, int n,
                             int T, int S, int fin, SmallNode *small, u64 seed, int d, Counters *c, int rule)
{
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)n * T;
    const bool live = n > fin;       // otherwise the whole tree is finished in one workgroup
    if (p < (size_t)T && !live && n > S) {
        SmallNode sn;
        sn.b = (int)p * n;
        sn.e = sn.b + n;
        sn.heap = 1;
        sn.depth = 0;
        sn.parent = -1;
        small[p] = sn;
        if (p == 0) c->small_nodes = T;
    }
    if (p < total) {
        node_of[p] = live ? (int)(p / (size_t)n) : -1;
        leaf_flag[p] = (n <= S && p % (size_t)n == 0) ? 1 : 0;
    }
    if (p < (size_t)T && live) {
        Node nd;
        nd.b = (int)p * n;
        nd.e = nd.b + n;
        nd.heap = 1;
        nd.sum = 0;
        const u64 draw = ef_mix64(ef_stream_key(seed, (int)p) + 1);
        nd.dim = rule == 1 ? kDimPending : rule == 2 ? ef_projection_code(draw) : (int)(draw % (u64)d);
        nd.depth = 0;
        nd.mid = nd.b;
        nd.moved = 0;
        nd.child[0] = nd.child[1] = -1;
        nd.parent = -1;
        nodes[p] = nd;
        dims[p] = nd.dim;
    }
    if (p == 0) {
        c->n_nodes[0] = live ? T : 0;
        c->n_nodes[1] = 0;
    }
}

// `tiles` consecutive tiles of kBlock positions per block.  Near the root every tile of a block
// lies in the same node: their sums are carried in a register and go out as one atomic (the
// few node records of the top levels would otherwise take one atomic per tile, all to the same
// few addresses, which serialise).
// What the split test will look at is kept for it: the coordinate in val, a projection as 64 bits in
// val and val_hi (8 gathers and 8 numbers drawn per position: adding them up again for the test made
// the test as expensive as the sums, 200 000 x 960 with eight trees 5.9 -> 3.4 ms).
// A projection's coordinates come from the rows, or from the transposed copy where the ids of a
// node lie so close together that a 128-byte line of a column holds several of them: about 32 >> level,
// times eight lines per position, against as many lines as a row has but eight at most.
template <bool PROJECTION>      // (compiled apart: the other rules' kernels carry none of it)
__global__ void __launch_bounds__(kBlock)
sum_kernel(const float *__restrict__ XT, int n, const int *__restrict__ perm,
           const int *__restrict__ node_of, Node *nodes, const int *__restrict__ dims,
           float *__restrict__ val, size_t total, Counters *c, int level, int tiles,
           int *__restrict__ val_hi, const float *__restrict__ X, int d)      // X: the rows
{
    const bool columns = PROJECTION && level < 5 && (1 << level) < 4 * min(kProjectionTerms, (d + 31) / 32);
    if (blockIdx.x == 0 && threadIdx.x == 0) c->n_nodes[(level + 1) & 1] = 0;      // filled by children_kernel
    __shared__ long long wave_tot[kBlock / EF_WAVE];
    __shared__ int wave_node[kBlock / EF_WAVE];
    int carry_node = -1;          // thread 0: node and sum of the uniform tiles seen so far
    long long carry = 0;
    for (int tile = 0; tile < tiles; ++tile) {
        const size_t p = ((size_t)blockIdx.x * tiles + tile) * kBlock + threadIdx.x;
        if (((size_t)blockIdx.x * tiles + tile) * kBlock >= total) break;
        int s = -1;
        long long q = 0;
        if (p < total) {
            s = node_of[p];
            if (s >= 0) {
                // the split dimension comes from its own array: the node records are being hit
                // by the sum atomics of this very kernel, and reads of such a line crawl
                int dim = dims[s];
                if (dim >= 0) {
                    float x = XT[(size_t)dim * n + perm[p]];
                    val[p] = x;
                    q = ef_quantise(x);
                } else if (PROJECTION && dim <= -3) {
                    const int id = perm[p];
                    const float *row = columns ? XT + id : X + (size_t)id * d;
                    const size_t pitch = columns ? (size_t)n : 1;
                    q = ef_node_value([&](int j) { return row[j * pitch]; }, d, dim);
                    val[p] = __int_as_float((int)(u32)(u64)q);
                    val_hi[p] = (int)(q >> 32);
                } else {
                    s = -1;
                }
            }
        }
        // Positions of a node are contiguous, so inside a wave equal node indices form runs.
        // Segmented inclusive scan over the runs; the last lane of a run then holds its sum.
        const int lane = ef_lane(), wave = threadIdx.x / EF_WAVE;
        for (int o = 1; o < EF_WAVE; o <<= 1) {
            const long long q_up = __shfl_up(q, o, EF_WAVE);
            const int s_up = __shfl_up(s, o, EF_WAVE);
            if (lane >= o && s_up == s) q += q_up;
        }
        const int s_next = __shfl_down(s, 1, EF_WAVE);
        const bool tail = lane == EF_WAVE - 1 || s_next != s;
        const int s_first = __shfl(s, 0, EF_WAVE);
        const bool uniform = __all(s == s_first);      // the whole wave lies in one node
        if (lane == EF_WAVE - 1) {
            wave_tot[wave] = q;
            wave_node[wave] = uniform ? s : -2;
        }
        __syncthreads();
        // near the root a whole tile lies in one node: one sum for the tile
        bool tile_uniform = true;
        for (int w = 0; w < kBlock / EF_WAVE; ++w) tile_uniform &= wave_node[w] == wave_node[0] && wave_node[0] != -2;
        if (tile_uniform) {
            if (threadIdx.x == 0 && wave_node[0] >= 0) {
                long long tot = 0;
                for (int w = 0; w < kBlock / EF_WAVE; ++w) tot += wave_tot[w];
                if (wave_node[0] != carry_node) {
                    if (carry_node >= 0) atomicAdd((u64 *)&nodes[carry_node].sum, (u64)carry);
                    carry_node = wave_node[0];
                    carry = 0;
                }
                carry += tot;
            }
        } else if (tail && s >= 0) {
            atomicAdd((u64 *)&nodes[s].sum, (u64)q);
        }
        __syncthreads();      // wave_tot / wave_node are free for the next tile
    }
    if (threadIdx.x == 0 && carry_node >= 0) atomicAdd((u64 *)&nodes[carry_node].sum, (u64)carry);
}

// predicate sources for the scan
template <bool PROJECTION>
struct LeftPred {
    const int *node_of;
    const Node *nodes;
    const float *val;
    const int *val_hi;      // (see sum_kernel)
    __device__ int operator()(size_t p) const
    {
        int s = node_of[p];
        if (s < 0) return 0;
        const Node &nd = nodes[s];
        if (!ef_has_test(nd.dim)) return 0;
        const long long cnt = nd.e - nd.b;
        const long long q = !PROJECTION || nd.dim >= 0
                                ? ef_quantise(val[p])
                                : (long long)(((u64)(u32)val_hi[p] << 32) | (u32)__float_as_int(val[p]));
        return cnt * q < nd.sum ? 1 : 0;
    }
};
struct FlagPred {
    const unsigned char *flag;
    __device__ int operator()(size_t p) const { return flag[p]; }
};
// A scan block covers kScanTile consecutive positions; thread t looks at positions t,
// t + kBlock, ... of the tile, so that a wave reads consecutive words.  The predicates are
// single bits: a wave counts them with a ballot.
// bits (or null): the predicate of positions 64 w .. 64 w + 63 goes to bits[w], for the kernels that need it again, and
// before[w] says how often it holds in the tile before those.
template <class Pred>
__global__ void scan_reduce_kernel(Pred pred, size_t total, int *block_sums, u64 *__restrict__ bits, unsigned short *__restrict__ before)
{
    constexpr int kWords = kScanTile / EF_WAVE;
    static_assert(kWords <= EF_WAVE, "a wave adds up the words of a tile");
    __shared__ int sh[kWords];
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const size_t p = base + (size_t)k * kBlock;      // lane 0: a multiple of 64
        const u64 bal = __ballot(p < total && pred(p));
        if (ef_lane() == 0) {
            sh[k * (kBlock / EF_WAVE) + threadIdx.x / EF_WAVE] = __popcll(bal);
            if (bits && p < total) bits[p >> 6] = bal;
        }
    }
    __syncthreads();
    if (threadIdx.x < EF_WAVE) {
        const int c = threadIdx.x < kWords ? sh[threadIdx.x] : 0, incl = ef_wave_scan_i32(c);
        const size_t w = (size_t)blockIdx.x * kWords + threadIdx.x;
        if (bits && threadIdx.x < kWords && w < (total + 63) / 64) before[w] = (unsigned short)(incl - c);
        if (threadIdx.x == EF_WAVE - 1) block_sums[blockIdx.x] = incl;
    }
}

// How often the predicate holds before position p, p <= total, from what the two scan kernels leave behind.  (A prefix sum
// written out per position cost a pass of 32 MB per level and reading it back; with the scan of the tiles in one round
// instead of sixteen, 10^6 x 128, eight trees, ten levels: 0.25 ms of 3.2.)
struct LeftCount {
    const u64 *bits;
    const unsigned short *before;
    const int *block_sums;
    size_t total;
    int nb;
    __device__ int operator()(size_t p) const
    {
        if (p >= total) return block_sums[nb];
        return block_sums[p / kScanTile] + before[p >> 6] + __popcll(bits[p >> 6] & ((1ULL << (p & 63)) - 1));
    }
};

// exclusive scan of block_sums in place, single block; block_sums[nb] = grand total
constexpr int kSumThreads = 1024, kSumItems = 4;      // (10^6 points, eight trees: 3907 tiles, one round)
__global__ void __launch_bounds__(kSumThreads) scan_blocksums_kernel(int *block_sums, int nb)
{
    __shared__ int sh[2][kSumThreads / EF_WAVE];
    int carry = 0;
    for (int base = 0, r = 0; base < nb; base += kSumThreads * kSumItems, r ^= 1) {
        const int i0 = base + (int)threadIdx.x * kSumItems;
        int v[kSumItems], sum = 0;
#pragma unroll
        for (int k = 0; k < kSumItems; ++k) {
            v[k] = i0 + k < nb ? block_sums[i0 + k] : 0;
            sum += v[k];
        }
        const int inc = ef_wave_scan_i32(sum);
        if (ef_lane() == EF_WAVE - 1) sh[r][threadIdx.x / EF_WAVE] = inc;
        __syncthreads();      // (the other half of sh is free: everybody is past the round before)
        int off = carry + inc - sum;
        for (int w = 0; w < kSumThreads / EF_WAVE; ++w) {
            off += w < (int)(threadIdx.x / EF_WAVE) ? sh[r][w] : 0;
            carry += sh[r][w];
        }
#pragma unroll
        for (int k = 0; k < kSumItems; ++k) {
            if (i0 + k < nb) block_sums[i0 + k] = off;
            off += v[k];
        }
    }
    if (threadIdx.x == 0) block_sums[nb] = carry;
}

// out[p] = number of set predicates before p; out[total] = grand total
template <class Pred>
__global__ void scan_apply_kernel(Pred pred, size_t total, const int *block_sums, int nb, int *out)
{
    __shared__ int sh[kScanItems][kBlock / EF_WAVE];      // set bits per row of kBlock positions and wave
    const int lane = ef_lane(), wave = threadIdx.x / EF_WAVE;
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
    int before[kScanItems];      // set bits before this position inside its wave's 64 positions
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const size_t p = base + (size_t)k * kBlock;
        const u64 bal = __ballot(p < total && pred(p));
        before[k] = __popcll(bal & ((1ULL << lane) - 1));
        if (lane == 0) sh[k][wave] = __popcll(bal);
    }
    __syncthreads();
    int off = block_sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const size_t p = base + (size_t)k * kBlock;
        int mine = off + before[k];
        for (int w = 0; w < kBlock / EF_WAVE; ++w) {
            const int c = sh[k][w];
            mine += w < wave ? c : 0;
            off += c;
        }
        if (p < total) out[p] = mine;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[total] = block_sums[nb];
}

__global__ void children_kernel(Node *cur, int level, Node *next, int *next_dims,
                                LeftCount left,
                                unsigned char *leaf_flag, int S, int fin, SmallNode *small, u64 seed,
                                int n, int d, Counters *c, NodeRec *rec, int *leaf_rec, int rule)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    int kind[2] = {0, 0};      // 0 leaf, 1 finished later inside one workgroup, 2 next level
    Node nd;
    const int n_cur = c->n_nodes[level & 1];      // the launch covers the most nodes a level can have
    if (s < n_cur) {
        nd = cur[s];
        int cnt = nd.e - nd.b;
        nd.left_before = left(nd.b);
        int nl = ef_has_test(nd.dim) ? left(nd.e) - nd.left_before : 0;
        if (nl == 0 || nl == cnt) {
            nd.moved = 0;
            nd.mid = nd.b + cnt / 2;
        } else {
            nd.moved = 1;
            nd.mid = nd.b + nl;
        }
        const int sz[2] = {nd.mid - nd.b, nd.e - nd.mid};
        for (int side = 0; side < 2; ++side) kind[side] = sz[side] <= S ? 0 : (sz[side] <= fin ? 1 : 2);
    }
    // one counter bump per wave and list
    const int want = (kind[0] == 2) + (kind[1] == 2), want_s = (kind[0] == 1) + (kind[1] == 1);
    const int inc = ef_wave_scan_i32(want), inc_s = ef_wave_scan_i32(want_s);
    const int wave_total = __shfl(inc, EF_WAVE - 1, EF_WAVE), wave_total_s = __shfl(inc_s, EF_WAVE - 1, EF_WAVE);
    int base = 0, base_s = 0;
    if (ef_lane() == EF_WAVE - 1) {
        if (wave_total > 0) base = atomicAdd(&c->n_nodes[(level + 1) & 1], wave_total);
        if (wave_total_s > 0) base_s = atomicAdd(&c->small_nodes, wave_total_s);
    }
    base = __shfl(base, EF_WAVE - 1, EF_WAVE);
    base_s = __shfl(base_s, EF_WAVE - 1, EF_WAVE);
    if (s >= n_cur) return;
    int slot = base + inc - want, slot_s = base_s + inc_s - want_s;
    if (rec) {
        record_node(rec, leaf_rec, nd.mid, nd.sum, nd.dim, nd.e - nd.b, nd.parent, nd.depth);
        if (s == 0) atomicMax(&c->max_depth, nd.depth);      // all nodes of a level share their depth
    }
    const int tree = nd.b / n;
    const u64 key = ef_stream_key(seed, tree);
    for (int side = 0; side < 2; ++side) {
        int cb = side ? nd.mid : nd.b, ce = side ? nd.e : nd.mid;
        // below depth 60 heap ids would overflow: such nodes only split positionally
        const u64 ch_heap = nd.depth < 60 ? 2 * nd.heap + side : nd.heap;
        nd.child[side] = -1;
        if (kind[side] == 2) {
            Node ch;
            ch.b = cb;
            ch.e = ce;
            ch.depth = nd.depth + 1;
            ch.heap = ch_heap;
            ch.dim = ch.depth < 60 ? node_dim(rule, ef_mix64(key + ch.heap), d) : -1;
            ch.sum = 0;
            ch.mid = cb;
            ch.moved = 0;
            ch.child[0] = ch.child[1] = -1;
            ch.parent = nd.mid;
            next[slot] = ch;
            next_dims[slot] = ch.dim;
            nd.child[side] = slot++;
        } else if (kind[side] == 1) {
            SmallNode sn;
            sn.b = cb;
            sn.e = ce;
            sn.heap = ch_heap;
            sn.depth = nd.depth + 1;
            sn.parent = nd.mid;
            small[slot_s++] = sn;
        } else {
            leaf_flag[cb] = 1;
            if (rec) record_leaf(rec, leaf_rec, cb, nd.mid);
        }
    }
    cur[s] = nd;
}

__global__ void scatter_kernel(const int *__restrict__ perm_in, int *__restrict__ perm_out,
                               const int *__restrict__ node_in, int *__restrict__ node_out,
                               const Node *__restrict__ nodes, LeftCount left)
{
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= left.total) return;
    int s = node_in[p];
    int id = perm_in[p];
    if (s < 0) {
        perm_out[p] = id;
        node_out[p] = -1;
        return;
    }
    const Node nd = nodes[s];
    size_t dst = p;
    if (nd.moved) {
        const bool goes_left = (left.bits[p >> 6] >> (p & 63)) & 1;      // the split test, as the scan evaluated it
        const int lc = left(p) - nd.left_before;
        dst = goes_left ? (size_t)nd.b + lc : (size_t)nd.mid + ((int)(p - nd.b) - lc);
    }
    perm_out[dst] = id;
    node_out[dst] = nd.child[dst < (size_t)nd.mid ? 0 : 1];
}

// Finishes the subtree of one small node (at most fin_max positions) inside a workgroup:
// the same four steps per level as the device-wide kernels (integer sums, prefix sum of
// the "goes left" predicate, children, stable scatter), but with the ids, the node table
// and the prefix sums in LDS, so the lower half of a tree costs one launch instead of
// half a dozen per level.
struct LNode {
    int b, e, mid, moved;      // local positions
    u64 heap;
    long long sum;
    int dim, depth;
    int child[2];
    int parent, pad;           // parent: global position, as in Node
};

// LDS of a block: ids, node indexes of 16 bits, the split tests as bits, two node tables of `nodes`.  A thread keeps the
// ids, nodes and tested values of its positions (every kFinThreads-th) in registers.  Leaves of 16: 52 KB for the 4096 positions of splits by one
// coordinate, two blocks of 1024 threads per CU; 26 KB for 2048 positions and 512 threads, three blocks in the registers of splits by
// variance (with all of it and prefix sums in LDS 78 KB, two blocks).  What bounds it, 10^6 x 128, eight trees: splits by one coordinate
// the scattered 4-byte gathers (64 M of them in eight levels, 128-byte lines at 6.8 TB/s; 1.22 ms), splits by variance the rows of the
// samples (14.5 GB, at 4.0 TB/s; 5.13 -> 3.61 ms, see variance_dim_wave; two blocks per CU 3.83).
// Random projections ask for one block per CU: the eight lines that a position reads of its row come the faster the fewer
// waves ask for others in between (200 000 x 960: one block 1.65 ms, two 1.74, three 1.81, four 1.86).
constexpr size_t kFinProjLds = 96 * 1024;
inline size_t finish_lds(int rule, int nodes)
{
    return (size_t)fin_max(rule) * 6 + fin_max(rule) / EF_WAVE * 12 + 64 + 2 * (size_t)nodes * sizeof(LNode);
}

// RULE: the split rule; NARROW, ONE: see variance_dim_wave, which wants more registers; kFinMax, PER: positions a block and a thread
// have room for.  Up to kFinFew points a root is its tree's only segment, and a position per thread spares the empty rounds: 512 points, four
// trees 98 -> 93 us, 100 points 84 -> 82.
template <int RULE, bool NARROW, bool ONE, int kFinMax = fin_max(RULE), int PER = 4>
__global__ void __launch_bounds__(kFinMax / PER) __attribute__((amdgpu_waves_per_eu(RULE == 1 ? 6 : RULE == 2 ? 4 : 8)))
finish_kernel(const float *__restrict__ XT, int d, int *perm, const SmallNode *__restrict__ small,
              unsigned char *leaf_flag, int S, u64 seed, int n, NodeRec *rec, int *leaf_rec,
              int *max_depth, const float *__restrict__ X, int nodes)
{
    // One 16-byte aligned LDS block carved by hand (no separate static LDS variables, whose
    // size would shift the 8-byte node records off their alignment).
    extern __shared__ __align__(16) int fsm[];
    constexpr int kFinThreads = kFinMax / PER, kFinWords = kFinMax / EF_WAVE, kDone = 0xFFFF;
    static_assert(kFinWords <= EF_WAVE, "a wave adds up the words");
    LNode *const tabs_base = (LNode *)fsm;                          // [2][nodes]
    u64 *const bits = (u64 *)(tabs_base + 2 * nodes);               // [kFinWords] "goes left", one bit per position
    int *const before = (int *)(bits + kFinWords);                  // [kFinWords + 1] set bits before each word
    int *const n_next_sh = before + kFinWords + 1;                  // [2]
    int &depth_sh = n_next_sh[2];                                   // deepest node of this subtree
    int *const ids = before + kFinWords + 16;                       // [kFinMax]
    unsigned short *const nidx = (unsigned short *)(ids + kFinMax); // [kFinMax], kDone: in a leaf
    const SmallNode seg = small[blockIdx.x];
    const int cnt = seg.e - seg.b, tid = threadIdx.x, lane = ef_lane();
    const u64 key = ef_stream_key(seed, seg.b / n);
    for (int p = tid; p < cnt; p += kFinThreads) {
        ids[p] = perm[seg.b + p];
        nidx[p] = 0;
    }
    if (tid == 0) {
        LNode r;
        r.b = 0;
        r.e = cnt;
        r.mid = 0;
        r.moved = 0;
        r.heap = seg.heap;
        r.sum = 0;
        r.depth = seg.depth;
        r.dim = seg.depth < 60 ? node_dim(RULE, ef_mix64(key + seg.heap), d) : -1;
        r.child[0] = r.child[1] = -1;
        r.parent = seg.parent;
        r.pad = 0;
        tabs_base[0] = r;
        n_next_sh[0] = n_next_sh[1] = 0;
        depth_sh = seg.depth;
    }
    __syncthreads();
    for (int cur = 0, n_cur = 1; n_cur > 0; cur ^= 1) {
        LNode *tc = tabs_base + cur * nodes, *tn = tabs_base + (cur ^ 1) * nodes;
        int id[PER], k[PER];
        long long q[PER];
        // 0. split dimensions by variance, one wave per node
        if (RULE == 1) {
            for (int s = tid / EF_WAVE; s < n_cur; s += kFinThreads / EF_WAVE) {
                if (tc[s].dim != kDimPending) continue;      // (uniform)
                const int dim = variance_dim_wave<NARROW, ONE>(X, d, ids + tc[s].b, tc[s].e - tc[s].b, ef_mix64(key + tc[s].heap));
                if (lane == 0) tc[s].dim = dim;
            }
            __syncthreads();
        }
        // 1. sums
        float x[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int p = tid + u * kFinThreads;
            id[u] = p < cnt ? ids[p] : 0;
            k[u] = p < cnt ? (int)nidx[p] : kDone;
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int dim = k[u] != kDone ? tc[k[u]].dim : -1;
            x[u] = dim >= 0 ? XT[(size_t)dim * n + id[u]] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int dim = k[u] != kDone ? tc[k[u]].dim : -1;
            q[u] = ef_quantise(x[u]);
            if (RULE == 2 && dim <= -3) {
                const float *row = X + (size_t)id[u] * d;
                q[u] = ef_node_value([&](int j) { return row[j]; }, d, dim);
            }
            // (positions of a node are neighbours: near the top a wave lies in one node and adds up among its lanes)
            const int k0 = __builtin_amdgcn_readfirstlane(k[u]);
            if (__all(k[u] == k0)) {
                if (k0 == kDone) continue;
                long long sum = q[u];
                for (int o = EF_WAVE / 2; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, EF_WAVE);
                if (lane == 0) atomicAdd((u64 *)&tc[k0].sum, (u64)sum);
            } else if (ef_has_test(dim))
                atomicAdd((u64 *)&tc[k[u]].sum, (u64)q[u]);
        }
        if (tid == 0) n_next_sh[cur ^ 1] = 0;
        __syncthreads();
        // 2. the "goes left" predicate, and how often it holds before every word of positions
        u32 left = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            bool f = false;
            if (k[u] != kDone) {
                const LNode &nd = tc[k[u]];
                f = ef_has_test(nd.dim) && (long long)(nd.e - nd.b) * q[u] < nd.sum;
            }
            const u64 word = __ballot(f);
            if (lane == 0) bits[(tid + u * kFinThreads) / EF_WAVE] = word;
            left |= (f ? 1u : 0u) << u;
        }
        __syncthreads();
        if (tid < EF_WAVE) {
            const int c = tid < kFinWords ? __popcll(bits[tid]) : 0, incl = ef_wave_scan_i32(c);
            if (tid < kFinWords) before[tid] = incl - c;
            if (tid == EF_WAVE - 1) before[kFinWords] = incl;
        }
        __syncthreads();
        auto left_before = [&](int p) {      // p <= kFinMax
            return before[p / EF_WAVE] + (p % EF_WAVE ? __popcll(bits[p / EF_WAVE] << (EF_WAVE - p % EF_WAVE)) : 0);
        };
        // 3. children
        for (int s = tid; s < n_cur; s += kFinThreads) {
            LNode nd = tc[s];
            const int c = nd.e - nd.b;
            const int nl = ef_has_test(nd.dim) ? left_before(nd.e) - left_before(nd.b) : 0;
            if (nl == 0 || nl == c) {
                nd.moved = 0;
                nd.mid = nd.b + c / 2;
            } else {
                nd.moved = 1;
                nd.mid = nd.b + nl;
            }
            if (rec) {
                record_node(rec, leaf_rec, seg.b + nd.mid, nd.sum, nd.dim, c, nd.parent, nd.depth);
                if (s == 0) depth_sh = nd.depth;      // levels are visited in order of depth
            }
            for (int side = 0; side < 2; ++side) {
                const int cb = side ? nd.mid : nd.b, ce = side ? nd.e : nd.mid;
                nd.child[side] = -1;
                if (ce - cb > S) {
                    LNode ch;
                    ch.b = cb;
                    ch.e = ce;
                    ch.mid = cb;
                    ch.moved = 0;
                    ch.depth = nd.depth + 1;
                    ch.heap = nd.depth < 60 ? 2 * nd.heap + side : nd.heap;
                    ch.dim = ch.depth < 60 ? node_dim(RULE, ef_mix64(key + ch.heap), d) : -1;
                    ch.sum = 0;
                    ch.child[0] = ch.child[1] = -1;
                    ch.parent = seg.b + nd.mid;
                    ch.pad = 0;
                    const int slot = atomicAdd(&n_next_sh[cur], 1);
                    tn[slot] = ch;
                    nd.child[side] = slot;
                } else {
                    leaf_flag[seg.b + cb] = 1;
                    if (rec) record_leaf(rec, leaf_rec, seg.b + cb, seg.b + nd.mid);
                }
            }
            tc[s] = nd;
        }
        __syncthreads();
        // 4. stable scatter (in place: everybody holds its ids)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (k[u] == kDone) continue;      // (stays where it is)
            const int p = tid + u * kFinThreads;
            const LNode &nd = tc[k[u]];
            int dst = p;
            if (nd.moved) {
                const int lc = left_before(p) - left_before(nd.b);
                dst = (left >> u) & 1 ? nd.b + lc : nd.mid + (p - nd.b - lc);
            }
            ids[dst] = id[u];
            nidx[dst] = (unsigned short)nd.child[dst < nd.mid ? 0 : 1];      // (-1: kDone)
        }
        n_cur = n_next_sh[cur];
        __syncthreads();
    }
    for (int p = tid; p < cnt; p += kFinThreads) perm[seg.b + p] = ids[p];
    if (rec && tid == 0) atomicMax(max_depth, depth_sh);
}

__global__ void iota_kernel(int *perm, int n, size_t total)
{
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < total) perm[p] = (int)(p % (size_t)n);
}

__global__ void leaf_offsets_kernel(const unsigned char *__restrict__ leaf_flag,
                                    const int *__restrict__ rank, int n, int T, int max_leaves,
                                    int *__restrict__ leaf_off, int *__restrict__ n_leaves_dev)
{
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)n * T;
    if (p < total && leaf_flag[p]) {
        int t = (int)(p / (size_t)n);
        int idx = rank[p] - rank[(size_t)t * n];
        if (idx < max_leaves) leaf_off[(size_t)t * (max_leaves + 1) + idx] = (int)(p - (size_t)t * n);
    }
    if (p < (size_t)T) {
        int t = (int)p;
        int cnt = rank[(size_t)(t + 1) * n] - rank[(size_t)t * n];
        n_leaves_dev[t] = cnt;
        if (cnt <= max_leaves) leaf_off[(size_t)t * (max_leaves + 1) + cnt] = n;
    }
}

// Internal nodes and leaf parents, renumbered by leaves: the node whose right part starts with
// leaf l becomes node l of its tree (l >= 1), a leaf is named by its index.
__global__ void export_nodes_kernel(const unsigned char *__restrict__ leaf_flag,
                                    const int *__restrict__ rank, const NodeRec *__restrict__ rec,
                                    const int *__restrict__ leaf_rec, int n, int T, int max_leaves,
                                    efanna_node *__restrict__ nodes, int *__restrict__ leaf_up)
{
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)n * T;
    if (p >= total || !leaf_flag[p]) return;
    const int t = (int)(p / (size_t)n);
    const int r0 = rank[(size_t)t * n];
    const int l = rank[p] - r0;
    if (l >= max_leaves) return;
    const size_t base = (size_t)t * (max_leaves + 1);
    // positions read back from the records are clamped into the tree: a slip in the
    // bookkeeping then shows as a wrong table, never as a stray read
    const int lo = t * n, hi = lo + n - 1;
    auto at = [&](int pos) { return rank[min(max(pos, lo), hi)] - r0; };
    const int par = leaf_rec[p];
    leaf_up[base + l] = par < 0 ? -1 : at(par) * 2 + (p >= (size_t)par ? 1 : 0);
    if (p == (size_t)t * n) return;      // the first leaf starts no node's right part
    const NodeRec r = rec[p];
    efanna_node o;
    o.sum = r.sum;
    o.dim = r.dim;
    o.cnt = r.cnt;
    o.parent = r.parent < 0 ? -1 : at(r.parent);
    o.depth = r.depth;
    for (int s = 0; s < 2; ++s) o.child[s] = r.child[s] >= 0 ? at(r.child[s]) : ~at(~r.child[s]);
    nodes[base + l] = o;
}

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

struct TreeWs {
    int *perm_tmp, *node_a, *node_b, *lcount, *block_sums, *n_leaves_dev;
    float *val, *xt;
    unsigned char *leaf_flag;
    u64 *left_bits;      // the split test of every position, one bit each
    Node *nodes_a, *nodes_b;
    int *dims_a, *dims_b;
    SmallNode *small;
    Counters *counters;
    NodeRec *rec;        // only with node export
    int *leaf_rec;
    size_t bytes;
};

TreeWs carve(void *ws, int64_t n, int32_t d, int32_t T, int32_t S, bool with_nodes)
{
    size_t total = (size_t)n * T;
    size_t max_nodes = total / (size_t)(S + 1) + (size_t)T + 1;
    size_t nb = (total + kScanTile - 1) / kScanTile;
    char *p = (char *)ws;
    size_t off = 0;
    TreeWs w;
    auto take = [&](size_t bytes) {
        char *r = p ? p + off : nullptr;
        off += align_up(bytes);
        return r;
    };
    w.perm_tmp = (int *)take(total * 4);
    w.node_a = (int *)take(total * 4);
    w.node_b = (int *)take(total * 4);
    w.lcount = (int *)take((total + 1) * 4);
    w.val = (float *)take(total * 4);
    w.left_bits = (u64 *)take((total / 64 + 1) * 8);
    w.leaf_flag = (unsigned char *)take(total);
    w.block_sums = (int *)take((nb + 1) * 4);
    w.nodes_a = (Node *)take(max_nodes * sizeof(Node));
    w.nodes_b = (Node *)take(max_nodes * sizeof(Node));
    w.small = (SmallNode *)take(max_nodes * sizeof(SmallNode));
    w.dims_a = (int *)take(max_nodes * 4);
    w.dims_b = (int *)take(max_nodes * 4);
    w.n_leaves_dev = (int *)take((size_t)T * 4);
    w.counters = (Counters *)take(sizeof(Counters));
    w.xt = (float *)take((size_t)n * d * 4);
    w.rec = with_nodes ? (NodeRec *)take(total * sizeof(NodeRec)) : nullptr;
    w.leaf_rec = with_nodes ? (int *)take(total * 4) : nullptr;
    w.bytes = off;
    return w;
}

inline int scan_blocks(size_t total) { return (int)((total + kScanTile - 1) / kScanTile); }

}  // namespace

extern "C" size_t efanna_trees_workspace_bytes(int64_t n, int32_t d, int32_t n_trees,
                                               int32_t leaf_size, int32_t with_nodes)
{
    if (n < 1 || d < 1 || n_trees < 1 || leaf_size < 1) return 0;
    return carve(nullptr, n, d, n_trees, leaf_size, with_nodes != 0).bytes;
}

extern "C" int efanna_build_trees_rule(const float *X, int64_t n, int32_t d, int32_t n_trees,
                                       int32_t leaf_size, uint64_t seed, int32_t split_rule, int32_t *perm,
                                       int32_t *leaf_off, int32_t max_leaves, int32_t *n_leaves,
                                       efanna_node *nodes, int32_t *leaf_up, int32_t *tree_depth,
                                       void *ws, size_t ws_bytes, void *stream)
{
    if (!X || !perm || !leaf_off || !n_leaves || (!nodes) != (!leaf_up)) return EFANNA_EINVAL;
    if (split_rule != EFANNA_SPLIT_UNIFORM && split_rule != EFANNA_SPLIT_VARIANCE &&
        split_rule != EFANNA_SPLIT_PROJECTION)
        return EFANNA_EINVAL;
    if (n < 1 || d < 1 || n_trees < 1 || n_trees > EFANNA_MAX_TREES || leaf_size < 1 ||
        leaf_size > EFANNA_MAX_LEAF || max_leaves < 1)
        return EFANNA_EINVAL;
    if ((double)n * n_trees >= 2147483647.0 - 4096.0) return EFANNA_EINVAL;
    if (!ws || ((uintptr_t)ws & 255) ||
        ws_bytes < efanna_trees_workspace_bytes(n, d, n_trees, leaf_size, nodes != nullptr))
        return EFANNA_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const int T = n_trees, S = leaf_size;
    const size_t total = (size_t)n * T;
    const int grid_pos = (int)((total + kBlock - 1) / kBlock);
    TreeWs w = carve(ws, n, d, T, S, nodes != nullptr);

    EF_HIP_CHECK(hipMemsetAsync(w.counters, 0, sizeof(Counters), st));
    if (nodes) EF_HIP_CHECK(hipMemsetAsync(w.leaf_rec, 0xFF, total * 4, st));      // a lone root leaf has no parent
    transpose_check_kernel<<<dim3((unsigned)((n + kTrTile - 1) / kTrTile), (unsigned)((d + kTrTile - 1) / kTrTile)), kBlock, 0, st>>>(
        X, (int)n, d, w.xt, w.counters, split_rule == EFANNA_SPLIT_PROJECTION ? (double)kProjectionTerms : 1.0);
    iota_kernel<<<grid_pos, kBlock, 0, st>>>(perm, (int)n, total);
    const int fin = finish_limit(S, split_rule);
    roots_kernel<<<grid_pos, kBlock, 0, st>>>(w.nodes_a, w.dims_a, w.node_a, w.leaf_flag, (int)n, T, S, fin,
                                              w.small, seed, d, w.counters, split_rule);
    // The level counters are read into pinned host memory (one small buffer per calling thread,
    // kept for the life of the process): a copy to pageable memory is staged and takes some 20 us
    // longer, during which the GPU has nothing to do.  Without pinned memory: a local variable.
    Counters host_local;
    thread_local Counters *host_pinned = nullptr;
    if (!host_pinned && hipHostMalloc((void **)&host_pinned, sizeof(Counters), hipHostMallocDefault) != hipSuccess) {
        host_pinned = nullptr;
        (void)hipGetLastError();
    }
    Counters &host_c = host_pinned ? *host_pinned : host_local;
    // Splits by variance want to know the size of the values before the first level, and trees that are finished inside a
    // workgroup have no other stop; otherwise the first look at the level counters says whether the input is good (until then
    // a bad value only decides which side a position goes to).
    if (n <= fin || split_rule == EFANNA_SPLIT_VARIANCE) {
        EF_HIP_CHECK(hipMemcpyAsync(&host_c, w.counters, sizeof(Counters), hipMemcpyDeviceToHost, st));
        EF_HIP_CHECK(hipStreamSynchronize(st));
        if (host_c.bad_input) return EFANNA_EINPUT;
    } else
        host_c = Counters{};

    int *perm_cur = perm, *perm_nxt = w.perm_tmp;
    int *node_cur = w.node_a, *node_nxt = w.node_b;
    Node *nodes_cur = w.nodes_a, *nodes_nxt = w.nodes_b;
    int *dims_cur = w.dims_a, *dims_nxt = w.dims_b;
    // Nodes of more than `fin` positions are split level by level, device-wide.  While
    // 2^level * fin < n some node of the level is certainly that large, so those levels are
    // enqueued without asking; after them the host looks at the count after every level.
    // A level has at most total / (fin + 1) + T live nodes (they are disjoint).
    int sure = 0;
    if (n > fin)
        for (long long cap = fin; cap < n; cap *= 2) ++sure;
    const int max_live = (int)(total / (size_t)(fin + 1)) + T;
    const int grid_nodes = (max_live + kBlock - 1) / kBlock;
    int n_cur = n > fin ? T : 0;
    for (int level = 0; n_cur > 0; ++level) {
        // sixteen tiles per block while nodes are a million positions and more (levels 0..3 of the headline)
        const int tiles = (total >> level) / (size_t)T >= (size_t)kBlock * 256 ? 16 : 1;
        auto choose = d <= 2 * EF_WAVE ? (host_c.wide_input ? choose_dims_kernel<false, true> : choose_dims_kernel<true, true>)
                                       : (host_c.wide_input ? choose_dims_kernel<false, false> : choose_dims_kernel<true, false>);
        if (split_rule == EFANNA_SPLIT_VARIANCE)
            // (a wave per node: a quarter of the waves and the level waits four nodes long)
            choose<<<min((max_live + kBlock / EF_WAVE - 1) / (kBlock / EF_WAVE), 2048), kBlock, 0, st>>>(
                X, d, (int)n, perm_cur, nodes_cur, dims_cur, w.counters, level, seed);
        const LeftCount left{w.left_bits, (const unsigned short *)w.lcount, w.block_sums, total, scan_blocks(total)};
#define EF_SUM_AND_TEST(PROJECTION)      /* (node_nxt: free until the scatter, lcount: until the leaves are numbered) */ \
    do {                                                                                                 \
        sum_kernel<PROJECTION><<<(grid_pos + tiles - 1) / tiles, kBlock, 0, st>>>(                       \
            w.xt, (int)n, perm_cur, node_cur, nodes_cur, dims_cur, w.val, total, w.counters, level,      \
            tiles, node_nxt, X, d);                                                                      \
        scan_reduce_kernel<<<left.nb, kBlock, 0, st>>>(LeftPred<PROJECTION>{node_cur, nodes_cur, w.val, node_nxt}, total, \
                                                       w.block_sums, w.left_bits, (unsigned short *)w.lcount); \
    } while (0)
        if (split_rule == EFANNA_SPLIT_PROJECTION) EF_SUM_AND_TEST(true);
        else EF_SUM_AND_TEST(false);
#undef EF_SUM_AND_TEST
        scan_blocksums_kernel<<<1, kSumThreads, 0, st>>>(w.block_sums, left.nb);
        children_kernel<<<grid_nodes, kBlock, 0, st>>>(
            nodes_cur, level, nodes_nxt, dims_nxt, left, w.leaf_flag, S, fin, w.small, seed, (int)n, d,
            w.counters, w.rec, w.leaf_rec, split_rule);
        scatter_kernel<<<grid_pos, kBlock, 0, st>>>(perm_cur, perm_nxt, node_cur, node_nxt, nodes_cur, left);
        if (level + 1 >= sure) {
            EF_HIP_CHECK(hipMemcpyAsync(&host_c, w.counters, sizeof(Counters), hipMemcpyDeviceToHost, st));
            EF_HIP_CHECK(hipStreamSynchronize(st));
            if (host_c.bad_input) return EFANNA_EINPUT;
            n_cur = host_c.n_nodes[(level + 1) & 1];
        }
        int *tp = perm_cur; perm_cur = perm_nxt; perm_nxt = tp;
        int *tn = node_cur; node_cur = node_nxt; node_nxt = tn;
        Node *tq = nodes_cur; nodes_cur = nodes_nxt; nodes_nxt = tq;
        int *td = dims_cur; dims_cur = dims_nxt; dims_nxt = td;
    }
    // host_c.small_nodes is current: it was read after the last level (or after the roots)
    if (host_c.small_nodes > 0) {
        const int fin_nodes = max(1, fin / (S + 1));      // live nodes have more than S positions
        const size_t fin_lds = max(finish_lds(split_rule, fin_nodes), (size_t)(split_rule == EFANNA_SPLIT_PROJECTION ? kFinProjLds : 0));
        constexpr int V = EFANNA_SPLIT_VARIANCE;
        const bool few = split_rule == EFANNA_SPLIT_UNIFORM && n <= kFinFew;
        auto finish = split_rule == EFANNA_SPLIT_PROJECTION ? finish_kernel<EFANNA_SPLIT_PROJECTION, false, false>
                      : few                                 ? finish_kernel<EFANNA_SPLIT_UNIFORM, false, false, kFinFew, 1>
                      : split_rule == EFANNA_SPLIT_UNIFORM  ? finish_kernel<EFANNA_SPLIT_UNIFORM, false, false>
                      : d <= 2 * EF_WAVE ? (host_c.wide_input ? finish_kernel<V, false, true> : finish_kernel<V, true, true>)
                                         : (host_c.wide_input ? finish_kernel<V, false, false> : finish_kernel<V, true, false>);
        EF_HIP_CHECK(hipFuncSetAttribute((const void *)finish, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fin_lds));
        finish<<<host_c.small_nodes, few ? kFinFew : fin_threads(split_rule), fin_lds, st>>>(w.xt, d, perm_cur, w.small, w.leaf_flag, S, seed, (int)n, w.rec,
                                                                 w.leaf_rec, &w.counters->max_depth, X, fin_nodes);
    }
    if (perm_cur != perm)
        EF_HIP_CHECK(hipMemcpyAsync(perm, perm_cur, total * 4, hipMemcpyDeviceToDevice, st));

    FlagPred fp{w.leaf_flag};
    const int nb = scan_blocks(total);
    scan_reduce_kernel<<<nb, kBlock, 0, st>>>(fp, total, w.block_sums, (u64 *)nullptr, (unsigned short *)nullptr);
    scan_blocksums_kernel<<<1, kSumThreads, 0, st>>>(w.block_sums, nb);
    scan_apply_kernel<<<nb, kBlock, 0, st>>>(fp, total, w.block_sums, nb, w.lcount);
    leaf_offsets_kernel<<<grid_pos, kBlock, 0, st>>>(w.leaf_flag, w.lcount, (int)n, T, max_leaves,
                                                     leaf_off, w.n_leaves_dev);
    if (nodes)
        export_nodes_kernel<<<grid_pos, kBlock, 0, st>>>(w.leaf_flag, w.lcount, w.rec, w.leaf_rec, (int)n, T,
                                                         max_leaves, nodes, leaf_up);
    EF_HIP_CHECK(hipMemcpyAsync(n_leaves, w.n_leaves_dev, (size_t)T * 4, hipMemcpyDeviceToHost, st));
    if (nodes) EF_HIP_CHECK(hipMemcpyAsync(&host_c, w.counters, sizeof(Counters), hipMemcpyDeviceToHost, st));
    EF_HIP_CHECK(hipStreamSynchronize(st));
    if (tree_depth) {
        *tree_depth = -1;      // no internal node anywhere: every tree is a single leaf
        for (int t = 0; t < T; ++t)
            if (nodes && n_leaves[t] > 1) *tree_depth = host_c.max_depth;
    }
    EF_HIP_CHECK(hipGetLastError());
    for (int t = 0; t < T; ++t)
        if (n_leaves[t] > max_leaves) return EFANNA_ECAPACITY;
    return EFANNA_OK;
}

extern "C" int efanna_build_trees(const float *X, int64_t n, int32_t d, int32_t n_trees,
                                  int32_t leaf_size, uint64_t seed, int32_t *perm,
                                  int32_t *leaf_off, int32_t max_leaves, int32_t *n_leaves,
                                  efanna_node *nodes, int32_t *leaf_up, int32_t *tree_depth,
                                  void *ws, size_t ws_bytes, void *stream)
{
    return efanna_build_trees_rule(X, n, d, n_trees, leaf_size, seed, EFANNA_SPLIT_UNIFORM, perm, leaf_off,
                                   max_leaves, n_leaves, nodes, leaf_up, tree_depth, ws, ws_bytes, stream);
}
