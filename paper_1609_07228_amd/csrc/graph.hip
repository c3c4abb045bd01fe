// Graph kernels for gfx950: leaf brute force (Alg. 3 at the leaves), NN-descent
// (Alg. 4) and packing / unpacking of graph rows.
//
// Distance blocks are computed by groups of 16 lanes.  Lane l of a group owns the
// partial sum of coordinates j = l mod 16, which is exactly the library's fixed
// order of operations; a group works on a 4x4 tile of pairs at a time (4 + 4 row
// values feed 16 fused multiply-adds per lane and step), and a transposed butterfly
// leaves the finished distance of pair l in lane l.  Each lane then offers its pair to
// the two rows concerned through the lock-free bounded insertion.
#include <atomic>
#include <type_traits>
#include <vector>

#include "common.h"

namespace {

constexpr int kBlock = 256;
constexpr int kRegGrid = 256 * 128;    // blocks of the register-operand join kernels (grid-strided over the work list)
constexpr int kLeafGrid = 256 * 256;   // blocks of the register-operand leaf kernels (a leaf or two each: measured 1.55 ms
                                       // per headline graph against 1.74 ms with 256 * 32, where a block walks eleven)
constexpr int kMaxLargeGrid = 256 * 32 * 2;     // most blocks the LDS-row join kernel is launched with
constexpr int kRowPad = 4;   // floats appended to each LDS row
constexpr int kMaxClasses = 8;      // most work lists (size classes of joins)

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }
// LDS regions are laid out in units of floats; round to 16 bytes so that 8- and 16-byte
// accesses stay aligned
__host__ __device__ inline int align4(int x) { return (x + 3) & ~3; }

// ---------------------------------------------------------------------------------------
// fills

// number of overflow queues of the reverse lists, and ints between their counters
constexpr int kOvfQueues = 256, kOvfCounterPitch = 16;

// per-iteration reset of the counter scheme: reverse-list fill counts and bounds, work-list sizes.
// The lists themselves need no reset: the first L arrivals
// overwrite slots 0..L-1 in some order, readers stop at min(count, L), and the bounded
// insertion only ever touches lists that are full.
__global__ void fill_reverse_kernel(int *a_count, int *b_count, u64 *list_max, size_t n, int *work_count, int *ovf_count)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMaxClasses) work_count[i] = 0;     // the work lists
    for (size_t j = i; j < (size_t)kOvfQueues * kOvfCounterPitch; j += (size_t)gridDim.x * blockDim.x) ovf_count[j] = 0;
    if (i < n) {
        a_count[i] = 0;
        b_count[i] = 0;
        list_max[i] = ~0ULL;
        list_max[n + i] = ~0ULL;
    }
}

// ---------------------------------------------------------------------------------------
// one 4x4 tile of squared distances by a 16-lane group.
// rows: LDS, `stride` floats per row.  ra[r], rb[c]: row indices.  Returns in lane gl the
// distance of pair (ra[gl >> 2], rb[gl & 3]).
__device__ inline float tile_distance(const float *rows, int stride, int d, const int (&ra)[4],
                                      const int (&rb)[4], int gl)
{
    float acc[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = 0.0f;
    const float *pa0 = rows + ra[0] * stride, *pa1 = rows + ra[1] * stride,
                *pa2 = rows + ra[2] * stride, *pa3 = rows + ra[3] * stride;
    const float *pb0 = rows + rb[0] * stride, *pb1 = rows + rb[1] * stride,
                *pb2 = rows + rb[2] * stride, *pb3 = rows + rb[3] * stride;
    for (int j = gl; j < d; j += 16) {
        float a[4] = {pa0[j], pa1[j], pa2[j], pa3[j]};
        float b[4] = {pb0[j], pb1[j], pb2[j], pb3[j]};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float diff = a[r] - b[c];
                acc[r * 4 + c] = __builtin_fmaf(diff, diff, acc[r * 4 + c]);
            }
    }
    return ef_group_transpose_reduce16(acc, gl);
}

// Number of set bits of a ballot below the calling lane.
__device__ inline int lanes_below(u64 ballot)
{
    return (int)__builtin_amdgcn_mbcnt_hi((u32)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((u32)ballot, 0u));
}

__device__ inline float4 load_unaligned4(const float *p)
{
    const ef_f32x4_u v = *reinterpret_cast<const ef_f32x4_u *>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

// The register kernels read vectors in 16-byte pieces: the lanes (r, g) of row r take the
// coordinates c0 + 16 s + 4 g .. + 3, s = 0..7, of a 128-coordinate stretch; what lies beyond d
// counts as zero (zeros on both sides add nothing to a distance, in any position).
// ALIGNED (d % 4 == 0 and X 16-byte aligned): a piece is inside the vector or not at all.
// Else (d >= 4, rows at any multiple of four bytes): the pieces of the last, incomplete sixteen
// coordinates are read from d - 4 where they would leave the vector, and moved into place.
// (Such rows took the LDS kernels before.  Builds, before and after: 200 003 x 50, degree 15:
// 10.5 -> 5.6 ms; 100 000 x 187, degree 10: 9.8 -> 3.5; 50 000 x 957: 55 -> 4.6; 50 000 x 77, degree 60:
// 27 -> 15.4.)
// ok: this lane has a row (`row` names a vector of the data either way: no branch around the loads)
template <bool ALIGNED, int N>
__device__ inline void load_pieces(float4 (&v)[N], const float *row, int c0, int g, int d, bool ok)
{
    if (ALIGNED) {
#pragma unroll
        for (int s = 0; s < N; ++s) {
            const int j = c0 + 16 * s + 4 * g;
            v[s] = ok && j + 3 < d ? *reinterpret_cast<const float4 *>(row + j) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        return;
    }
    const int n_whole = (d - c0) >> 4;      // sixteens that lie inside (uniform)
    const float *p = row + c0 + 4 * g;
#pragma unroll
    for (int s = 0; s < N; ++s) v[s] = s < n_whole ? load_unaligned4(p + 16 * s) : make_float4(0.f, 0.f, 0.f, 0.f);
    if (n_whole < N && ((d - c0) & 15)) {
        const int j = c0 + 16 * n_whole + 4 * g, jb = min(j, d - 4), over = j - jb;
        const float4 w = load_unaligned4(row + jb);
        float4 t;
        t.x = over == 0 ? w.x : over == 1 ? w.y : over == 2 ? w.z : over == 3 ? w.w : 0.f;
        t.y = over == 0 ? w.y : over == 1 ? w.z : over == 2 ? w.w : 0.f;
        t.z = over == 0 ? w.z : over == 1 ? w.w : 0.f;
        t.w = over == 0 ? w.w : 0.f;
#pragma unroll
        for (int s = 0; s < N; ++s)
            if (s == n_whole) v[s] = t;
    }
    if (!ok)
#pragma unroll
        for (int s = 0; s < N; ++s) v[s] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// The same for a row of the data of at most 128 coordinates, without a mask per lane for the sixteens that lie inside
// the vector (the tile join, where a sixth of the instructions went into those masks; the kernels that
// hold more in registers spill with it).
template <bool ALIGNED>
__device__ inline void load_row(float4 (&v)[8], const float *row, int g, int d)
{
    if (!ALIGNED) return load_pieces<false>(v, row, 0, g, d, true);
    const int n_whole = d >> 4;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        v[s] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (s < n_whole) v[s] = *reinterpret_cast<const float4 *>(row + 16 * s + 4 * g);
        else if (s == n_whole && 16 * s + 4 * g < d) v[s] = *reinterpret_cast<const float4 *>(row + 16 * s + 4 * g);
    }
}

// The value, by a way the compiler does not see through: what is derived from it inside a loop is not kept in
// registers across the rest of the loop.
__device__ inline int ef_opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// A proposal waiting in the block's LDS queue: entry `key` offered to row `target`.
struct Proposal {
    u64 key;
    int target;
    int pad;
};

// Coalesced gather of m rows of X into LDS.  The block's threads walk the 16-byte pieces,
// ceil(d/4) per row, eight loads in flight per thread (rows that are not 16-byte aligned: four at
// 4-byte alignment, the last piece of a row moved back so that it ends with the row).
// q4_magic = ceil(2^32 / ceil(d/4)) turns the piece index into (row, column) without a
// division (exact while pieces * ceil(d/4) < 2^32).
__device__ inline void gather_rows(const float *__restrict__ X, int d, int stride, u32 q4_magic,
                                   const int *uid, int m, float *rows, int tid, int nthr)
{
    if ((d & 3) == 0 && ((uintptr_t)X & 15) == 0) {
        const int q4 = d >> 2, total = m * q4;
        for (int f0 = tid; f0 < total; f0 += nthr * 8) {
            float4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int f = min(f0 + k * nthr, total - 1);   // clamped: always a valid piece
                const int r = q4 == 1 ? f : (int)(((u64)(u32)f * q4_magic) >> 32), c = f - r * q4;
                v[k] = *reinterpret_cast<const float4 *>(X + (size_t)uid[r] * d + 4 * c);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int f = f0 + k * nthr;
                if (f < total) {
                    const int r = q4 == 1 ? f : (int)(((u64)(u32)f * q4_magic) >> 32), c = f - r * q4;
                    *reinterpret_cast<float4 *>(rows + r * stride + 4 * c) = v[k];
                }
            }
        }
    } else if (d >= 4) {
        const int q4 = (d + 3) >> 2, total = m * q4;
        for (int f0 = tid; f0 < total; f0 += nthr * 4) {
            ef_f32x4_u v[4];
            int to[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int f = min(f0 + k * nthr, total - 1);      // (a piece may be copied twice)
                const int r = q4 == 1 ? f : (int)(((u64)(u32)f * q4_magic) >> 32), c = min(4 * (f - r * q4), d - 4);
                v[k] = *reinterpret_cast<const ef_f32x4_u *>(X + (size_t)uid[r] * d + c);
                to[k] = r * stride + c;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) *reinterpret_cast<ef_f32x4_u *>(rows + to[k]) = v[k];
        }
    } else {
        const int total = m * d;
        for (int f = tid; f < total; f += nthr) {
            const int r = f / d, c = f - r * d;
            rows[r * stride + c] = X[(size_t)uid[r] * d + c];
        }
    }
}

// Drain the proposal queue: every thread applies whole proposals on its own, so all the
// row reads of up to blockDim proposals are in flight together.
__device__ inline int drain_queue(const Proposal *queue, int count, u64 *graph, u32 *worst, int K,
                                  int tid, int nthr)
{
    int updates = 0;
    for (int e = tid; e < count; e += nthr) {
        const Proposal p = queue[e];
        u64 new_max;
        if (ef_bounded_insert(graph + (size_t)p.target * K, K, p.key, 1, &new_max)) {
            atomicMin(worst + p.target, ef_dist_bits(new_max));
            ++updates;
        }
    }
    return updates;
}

// The same for rows of 2 .. 16 entries (see ef_bounded_insert_row).
__device__ inline int drain_queue_row(const Proposal *queue, int count, u64 *graph, u32 *worst, int K, int tid, int nthr)
{
    int updates = 0;
    for (int e = tid; e < count; e += nthr) {
        const Proposal p = queue[e];
        u32 new_max_bits;
        if (ef_bounded_insert_row(graph + (size_t)p.target * K, K, p.key, &new_max_bits)) {
            atomicMin(worst + p.target, new_max_bits);
            ++updates;
        }
    }
    return updates;
}

// The same for long rows in the join with rows in LDS: a group of sixteen threads per
// proposal (nthr a multiple of 16; all threads of the block call this together).
__device__ inline int drain_queue_g16(const Proposal *queue, int count, u64 *graph, u32 *worst, int K, int tid, int nthr)
{
    int updates = 0;
    for (int e = tid >> 4; e < count; e += nthr >> 4) {
        const Proposal p = queue[e];
        u64 new_max;
        if (ef_bounded_insert_g16(graph + (size_t)p.target * K, K, p.key, &new_max, tid & 15) && (tid & 15) == 0) {
            atomicMin(worst + p.target, ef_dist_bits(new_max));
            ++updates;
        }
    }
    return updates;
}

// The same for long rows in the tile join: a group of eight threads per
// proposal (nthr a multiple of 8; all threads of the block call this together).
// gid: the mirror of the rows' ids (graph_ids_kernel), kept up to date with the insertions.
template <bool ODD>      // (see ef_bounded_insert_g8)
__device__ inline int drain_queue_g8(const Proposal *queue, int count, u64 *graph, u32 *worst, int K,
                                     int tid, int nthr, int *gid)
{
    int updates = 0;
    for (int e = tid >> 3; e < count; e += nthr >> 3) {
        const Proposal p = queue[e];
        u32 new_max_bits;
        int slot;
        if (ef_bounded_insert_g8<ODD>(graph + (size_t)p.target * K, K, p.key, &new_max_bits, tid & 7, &slot) && slot >= 0) {
            atomicMin(worst + p.target, new_max_bits);
            // (a plain store: whatever order stores to a slot land in, the slot names an id that was in the row)
            gid[(size_t)p.target * K + slot] = ef_id(p.key);
            ++updates;
        }
    }
    return updates;
}

// ---------------------------------------------------------------------------------------
// Alg. 3 at the leaves, one tree per launch, one block per leaf (256 threads per 16 leaf
// slots).  Within one tree every point lies in exactly one leaf, so a block owns the graph
// rows of its members for the duration of the launch and needs no atomics.  Launches of
// successive trees are ordered by the stream.
//
// Rows and the members' old graph rows (ascending) go to LDS; distances come in 4x4 tiles by
// 16-lane groups; then every (row a, mate o) pair becomes a candidate key and the rows are
// merged by rank: a candidate's rank is the number of old entries below it (binary search,
// which also finds it if an earlier tree put it there already) plus the number of candidates
// of its row below it, an old entry's rank is its index plus the number of candidates below
// it; ranks below K are stored straight to the row.  Every slot of a row is written exactly
// once (K old entries plus the fresh candidates are at least K keys, all distinct).

__global__ void __launch_bounds__(1024)
init_tree_kernel(const float *__restrict__ X, int d, int stride, u32 q4_magic, int S,
                 const int *__restrict__ perm_t, const int *__restrict__ leaf_off_t, int K,
                 u64 *graph, int first_tree)
{
    extern __shared__ __align__(16) float smem[];
    float *rows = smem;                                   // [S][stride]
    float *dmat = smem + align4(S * stride);              // [S][S] distances, then (as int) old entries below
    u64 *pools = (u64 *)(dmat + align4(S * S));           // [S][K] old rows, ascending
    u64 *cand = pools + (size_t)S * K;                    // [S][S + 1] candidate keys of each row
    int *uid = (int *)(cand + (size_t)S * (S + 1));       // [S]
    int *ncand = uid + S;                                 // [S] candidates of each row that may enter it
    int *below = (int *)dmat;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int b = leaf_off_t[blockIdx.x];
    const int s = min(leaf_off_t[blockIdx.x + 1] - b, S);   // never overrun the buffers
    if (tid < s) uid[tid] = perm_t[b + tid];
    __syncthreads();
    gather_rows(X, d, stride, q4_magic, uid, s, rows, tid, nthr);
    for (int e = tid; e < s * K; e += nthr) {
        const int r = e / K, c = e - r * K;
        pools[e] = first_tree ? ef_empty_entry(K - 1 - c) : graph[(size_t)uid[r] * K + c];
    }
    __syncthreads();
    const int nt = (s + 3) >> 2, n_tiles = nt * (nt + 1) / 2;
    const int grp = tid >> 4, gl = tid & 15, n_grp = nthr >> 4;
    for (int q = grp; q < n_tiles; q += n_grp) {
        int ti = 0, rem = q;
        while (rem >= nt - ti) {
            rem -= nt - ti;
            ++ti;
        }
        const int tj = ti + rem;
        int ra[4], rb[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            ra[r] = min(4 * ti + r, s - 1);
            rb[r] = min(4 * tj + r, s - 1);
        }
        const float dist = tile_distance(rows, stride, d, ra, rb, gl);
        const int ia = 4 * ti + (gl >> 2), ib = 4 * tj + (gl & 3);
        if (ia < ib && ib < s) {
            dmat[ia * S + ib] = dist;
            dmat[ib * S + ia] = dist;
        }
    }
    __syncthreads();
    // candidate keys; the distance's slot then holds the number of old entries below the key
    const int pitch = S + 1;
    for (int e = tid; e < s * s; e += nthr) {
        const int a = e / s, o = e - a * s;
        u64 key = ~0ULL;
        int lo = 0;
        if (o != a) {
            key = ef_pack(dmat[a * S + o], uid[o], 1);
            if (!first_tree) {
                const u64 *row = pools + (size_t)a * K;
                int hi = K;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (row[mid] < key) lo = mid + 1;
                    else hi = mid;
                }
                if (lo < K && row[lo] == key) key = ~0ULL;      // already there from an earlier tree
            }
        }
        // A key above all K old entries stays out of the row, and so does every candidate above
        // it: it counts for nobody.  (Rows are full after a tree or two; from then on this is what
        // happens to most candidates.)
        if (lo >= K) key = ~0ULL;
        cand[a * pitch + o] = key;
        below[a * S + o] = lo;
    }
    __syncthreads();
    // the candidates still in the race move to the front of their row (a wave per row: its
    // lanes read the row before any of them writes), their number to ncand
    for (int a = tid / EF_WAVE; a < s; a += nthr / EF_WAVE) {
        const int o = ef_lane();
        const u64 key = o < s ? cand[a * pitch + o] : ~0ULL;
        const int lo = o < s ? below[a * S + o] : 0;
        const u64 alive = __ballot(key != ~0ULL);
        if (key != ~0ULL) {
            const int pos = __popcll(alive & ((1ULL << o) - 1));
            cand[a * pitch + pos] = key;
            below[a * S + pos] = lo;
        }
        if (o == 0) ncand[a] = __popcll(alive);
    }
    __syncthreads();
    for (int e = tid; e < s * s; e += nthr) {      // the candidates' places
        const int a = e / s, o = e - a * s, nc = ncand[a];
        if (o >= nc) continue;
        const u64 key = cand[a * pitch + o];
        int rank = below[a * S + o];
        for (int k = 0; k < nc; ++k) rank += cand[a * pitch + k] < key ? 1 : 0;
        if (rank < K) graph[(size_t)uid[a] * K + rank] = key;
    }
    for (int e = tid; e < s * K; e += nthr) {      // the old entries' places (a row without candidates stays as it is)
        const int a = e / K, j = e - a * K, nc = ncand[a];
        if (nc == 0 && !first_tree) continue;
        const u64 en = pools[e];
        int rank = j;
        for (int k = 0; k < nc; ++k) rank += cand[a * pitch + k] < en ? 1 : 0;
        if (rank < K) graph[(size_t)uid[a] * K + rank] = en;
    }
}

// ---------------------------------------------------------------------------------------
// The same step for leaves of at most 16 points (d >= 4), without a
// row buffer: persistent waves, one leaf at a time.
//
// Lane (r, g) = lane r + 16 g keeps, of member r of the leaf, the coordinates 16 s + 4 g + k
// (s = 0..7, k = 0..3) of the current 128-coordinate piece, i.e. terms of partial sums
// 4g..4g+3 of the library's fixed order.  Rotating the 16 lanes of a row by t (a DPP modifier, no memory traffic) puts
// member r opposite member r +- t, so eight rotations meet all pairs of the leaf; the four
// lanes of a column then add their partial sums in the fixed tree (8 apart, 4 apart, 2
// apart, 1 apart), transposed so that lane (r, g) ends up with the distances of rotations
// 2g+1 and 2g+2, and fetches the two that its mirror lanes computed towards r.
//
// Merge: the leaf owns its members' graph rows during the launch.  The old row (ascending,
// in LDS) and the row's up to 15 candidates are merged by rank: a candidate's rank is the
// number of old entries below it (binary search, which also finds it if it is already in
// the row) plus the number of candidates below it; an old entry's rank is its index plus
// the number of candidates below it.  Ranks below K are stored straight to the row.
#define EF_ROW_BCAST(x, a) __builtin_amdgcn_update_dpp(0, (x), 0x150 | (a), 0xF, 0xF, false)      // lane a of each sixteen to all of them
#define EF_ROW_ROR(x, t) __builtin_amdgcn_update_dpp(0, (x), 0x120 | (t), 0xF, 0xF, false)

template <int T, int N>
__device__ inline void init_round(const float4 (&va)[N], int n_pieces, float (&p)[4])
{
#pragma unroll
    for (int s = 0; s < N; ++s) {
        if (s >= n_pieces) break;
        const float d0 = va[s].x - __int_as_float(EF_ROW_ROR(__float_as_int(va[s].x), T));
        const float d1 = va[s].y - __int_as_float(EF_ROW_ROR(__float_as_int(va[s].y), T));
        const float d2 = va[s].z - __int_as_float(EF_ROW_ROR(__float_as_int(va[s].z), T));
        const float d3 = va[s].w - __int_as_float(EF_ROW_ROR(__float_as_int(va[s].w), T));
        p[0] = __builtin_fmaf(d0, d0, p[0]);
        p[1] = __builtin_fmaf(d1, d1, p[1]);
        p[2] = __builtin_fmaf(d2, d2, p[2]);
        p[3] = __builtin_fmaf(d3, d3, p[3]);
    }
}

// the same for two sets of sixteen rows: row r of the first against row r + T (rotation) of the second
template <int T>
__device__ inline void cross_round(const float4 (&va)[8], const float4 (&vb)[8], int n_pieces, float (&p)[4])
{
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        if (s >= n_pieces) break;
        float4 w = vb[s];
        if (T != 0) {      // (T ? T : 1: the rotation count is an immediate and 0 is not a valid one, used or not)
            w.x = __int_as_float(EF_ROW_ROR(__float_as_int(vb[s].x), T ? T : 1));
            w.y = __int_as_float(EF_ROW_ROR(__float_as_int(vb[s].y), T ? T : 1));
            w.z = __int_as_float(EF_ROW_ROR(__float_as_int(vb[s].z), T ? T : 1));
            w.w = __int_as_float(EF_ROW_ROR(__float_as_int(vb[s].w), T ? T : 1));
        }
        const float d0 = va[s].x - w.x, d1 = va[s].y - w.y, d2 = va[s].z - w.z, d3 = va[s].w - w.w;
        p[0] = __builtin_fmaf(d0, d0, p[0]);
        p[1] = __builtin_fmaf(d1, d1, p[1]);
        p[2] = __builtin_fmaf(d2, d2, p[2]);
        p[3] = __builtin_fmaf(d3, d3, p[3]);
    }
}

// row A of the first set against every row of the second
template <int A, int N>
__device__ inline void broadcast_round(const float4 (&va)[N], const float4 (&vb)[N], int n_pieces, float (&p)[4])
{
#pragma unroll
    for (int s = 0; s < N; ++s) {
        if (s >= n_pieces) break;
        const float d0 = vb[s].x - __int_as_float(EF_ROW_BCAST(__float_as_int(va[s].x), A));
        const float d1 = vb[s].y - __int_as_float(EF_ROW_BCAST(__float_as_int(va[s].y), A));
        const float d2 = vb[s].z - __int_as_float(EF_ROW_BCAST(__float_as_int(va[s].z), A));
        const float d3 = vb[s].w - __int_as_float(EF_ROW_BCAST(__float_as_int(va[s].w), A));
        p[0] = __builtin_fmaf(d0, d0, p[0]);
        p[1] = __builtin_fmaf(d1, d1, p[1]);
        p[2] = __builtin_fmaf(d2, d2, p[2]);
        p[3] = __builtin_fmaf(d3, d3, p[3]);
    }
}

// x summed over lanes l and l + 32 in the lower half of the wave, y in the upper one; then the same with
// neighbouring sixteens: x in the even ones, y in the odd ones.  One exchange of the vector ALU and an add
// (the addends in either order: a float32 sum is the same), where a shuffle through the LDS took two selects, an
// address and a wait besides.  All lanes of the wave must be active.  Builds: 10^6 x 128 16.53 -> 16.45 ms, 200 003 x 50
// 5.31 -> 5.23, 10^5 x 128 4.89 -> 4.86, 10^6 x 96 at degree 100 328 -> 324; conquer three levels up 11.96 -> 11.84.
__device__ inline float ef_add_halves(float x, float y)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ inline float ef_add_rows(float x, float y)
{
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

// The fixed order's tree over the sixteen partial sums of a pair, which lie four in each of the lanes r, r + 16,
// r + 32, r + 48; all four lanes get the distance.
__device__ inline float ef_sum_partials(float p0, float p1, float p2, float p3)
{
    const float s = ef_add_rows(ef_add_halves(p0, p2), ef_add_halves(p1, p3));      // sum of p[g] in lane r + 16 g: 0 1 2 3 -> p0 p1 p2 p3
    const float t = ef_add_halves(s, s);      // p0 + p2 in the even sixteens, p1 + p3 in the odd ones
    return ef_add_rows(t, t);
}

// eight partial-sum sets (one per pair) -> lane g keeps the finished distances of pairs 2g
// and 2g+1 of the eight; same adds, in the same tree, as the fixed order
__device__ inline void reduce_rotations(const float (&P)[8][4], float (&out)[2])
{
    float Q[4][4], R[2][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) Q[t][k] = ef_add_halves(P[t][k], P[t + 4][k]);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) R[t][k] = ef_add_rows(Q[t][k], Q[t + 2][k]);
#pragma unroll
    for (int t = 0; t < 2; ++t) out[t] = (R[t][0] + R[t][2]) + (R[t][1] + R[t][3]);
}

// The same for four rotations (T0 + 1 .. T0 + 4 in P[0..3]): lane (r, g) ends up with the distance
// from row r to the row T0 + 1 + g places on.
__device__ inline float reduce_rotations4(const float (&P)[4][4])
{
    float Q[2][4], R[4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) Q[t][k] = ef_add_halves(P[t][k], P[t + 2][k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) R[k] = ef_add_rows(Q[0][k], Q[1][k]);
    return (R[0] + R[2]) + (R[1] + R[3]);
}

constexpr int kCandPitch = 17;      // u64 per row of the candidate table (odd: rows on different banks)

template <bool ALIGNED>      // (see load_pieces)
__global__ void __launch_bounds__(EF_WAVE) __attribute__((amdgpu_waves_per_eu(4)))
init_reg_kernel(const float *__restrict__ X, int d, const int *__restrict__ perm_t,
                const int *__restrict__ leaf_off_t, int n_leaves, int K, u64 *graph, int first_tree)
{
    extern __shared__ __align__(16) float smem[];
    u64 *pools = (u64 *)smem;                         // [16][K] old rows, ascending
    u64 *cand = pools + 16 * (size_t)K;               // [16][kCandPitch] candidates of each row
    int *uid = (int *)(cand + 16 * kCandPitch);       // [16]
    const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
    // which way the rotation moves data: lane r receives from lane r + dirn (mod 16)
    const int dirn = (EF_ROW_ROR(r16, 1) - r16) & 15;
    // leaf boundaries are fetched two leaves ahead and member ids one leaf ahead
    int leaf = blockIdx.x;
    int b0 = leaf < n_leaves ? leaf_off_t[leaf] : 0;
    int s0 = leaf < n_leaves ? min(leaf_off_t[leaf + 1] - b0, 16) : 0;
    int id_pre = r16 < s0 ? perm_t[b0 + r16] : -1;
    int leaf1 = leaf + (int)gridDim.x;
    int b1 = leaf1 < n_leaves ? leaf_off_t[leaf1] : 0;
    int s1 = leaf1 < n_leaves ? min(leaf_off_t[leaf1 + 1] - b1, 16) : 0;
    for (; leaf < n_leaves; leaf += gridDim.x) {
        const int s = s0, my_id = id_pre;
        __syncthreads();                  // the previous leaf's LDS reads are done
        if (g == 0) uid[r16] = my_id;
        // old rows of this leaf
        for (int c = g; c < K; c += 4)
            pools[r16 * K + c] = first_tree || r16 >= s ? ef_empty_entry(K - 1 - c)
                                                        : graph[(size_t)my_id * K + c];
        // prefetch for the leaves to come
        s0 = s1;
        b0 = b1;
        id_pre = r16 < s0 ? perm_t[b0 + r16] : -1;
        leaf1 += gridDim.x;
        b1 = leaf1 < n_leaves ? leaf_off_t[leaf1] : 0;
        s1 = leaf1 < n_leaves ? min(leaf_off_t[leaf1 + 1] - b1, 16) : 0;
        // ---- distances: rotations 1..8, 128 coordinates at a time ---------------------------
        float P[8][4];
#pragma unroll
        for (int t = 0; t < 8; ++t) P[t][0] = P[t][1] = P[t][2] = P[t][3] = 0.0f;
        const float *pa = X + (size_t)max(my_id, 0) * d;
        for (int c0 = 0; c0 < d; c0 += 128) {
            float4 va[8];
            load_pieces<ALIGNED>(va, pa, c0, g, d, r16 < s);
            const int n_pieces = min(8, (d - c0 + 15) >> 4);
            init_round<1>(va, n_pieces, P[0]);
            init_round<2>(va, n_pieces, P[1]);
            init_round<3>(va, n_pieces, P[2]);
            init_round<4>(va, n_pieces, P[3]);
            init_round<5>(va, n_pieces, P[4]);
            init_round<6>(va, n_pieces, P[5]);
            init_round<7>(va, n_pieces, P[6]);
            init_round<8>(va, n_pieces, P[7]);
        }
        // partial sums l and l+8 live 2 lanes-of-g apart (xor 32), l and l+4 one apart (xor 16)
        float two[2];
        reduce_rotations(P, two);
        __syncthreads();                  // uid, pools visible
        // ---- candidates of row r16: rotations 2g+1, 2g+2, forwards and from the mirror lane ---
        u64 key[4];
        int lt[4];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const float dist = two[t];
            const int rot = 2 * g + 1 + t;
            const int bf = (r16 + dirn * rot) & 15, br = (r16 - dirn * rot) & 15;
            const float dist_r = __shfl(dist, br + 16 * g, EF_WAVE);     // lane br met r16 at this rotation
            key[t] = r16 < s && bf < s ? ef_pack(dist, uid[bf], 1) : ~0ULL;
            key[2 + t] = r16 < s && br < s && rot != 8 ? ef_pack(dist_r, uid[br], 1) : ~0ULL;
        }
        const u64 *row = pools + r16 * K;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            int lo = 0, hi_ = K;
            if (key[c] != ~0ULL && !first_tree) {
                while (lo < hi_) {
                    const int mid = (lo + hi_) >> 1;
                    if (row[mid] < key[c]) lo = mid + 1;
                    else hi_ = mid;
                }
                if (lo < K && row[lo] == key[c]) key[c] = ~0ULL;      // already there from an earlier tree
            }
            lt[c] = lo;
            cand[r16 * kCandPitch + 4 * g + c] = key[c];
        }
        __syncthreads();
        // ---- ranks ----------------------------------------------------------------------------
        u64 cs[16];
#pragma unroll
        for (int o = 0; o < 16; ++o) cs[o] = cand[r16 * kCandPitch + o];
        if (r16 < s) {
            u64 *out = graph + (size_t)my_id * K;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (key[c] == ~0ULL) continue;
                int rank = lt[c];
#pragma unroll
                for (int o = 0; o < 16; ++o) rank += cs[o] < key[c] ? 1 : 0;
                if (rank < K) out[rank] = key[c];
            }
            for (int j = g; j < K; j += 4) {
                const u64 e = row[j];
                int rank = j;
#pragma unroll
                for (int o = 0; o < 16; ++o) rank += cs[o] < e ? 1 : 0;
                if (rank < K) out[rank] = e;
            }
        }
    }
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));

// Eight coordinates of a vector, times a power of two, as half-precision numbers rounded towards
// zero: an operand of the 16x16x32 matrix instruction.  Both operands of a Gram block are packed
// the same way, so the order of the coordinates inside the operand does not matter.
template <bool SCALED>
__device__ inline f16x8 ef_pack_f16(const float4 &lo, const float4 &hi, float s)
{
    union {
        fp16x2 h[4];
        f16x8 v;
    } u;
    if (SCALED) {
        u.h[0] = __builtin_amdgcn_cvt_pkrtz(lo.x * s, lo.y * s);
        u.h[1] = __builtin_amdgcn_cvt_pkrtz(lo.z * s, lo.w * s);
        u.h[2] = __builtin_amdgcn_cvt_pkrtz(hi.x * s, hi.y * s);
        u.h[3] = __builtin_amdgcn_cvt_pkrtz(hi.z * s, hi.w * s);
    } else {
        u.h[0] = __builtin_amdgcn_cvt_pkrtz(lo.x, lo.y);
        u.h[1] = __builtin_amdgcn_cvt_pkrtz(lo.z, lo.w);
        u.h[2] = __builtin_amdgcn_cvt_pkrtz(hi.x, hi.y);
        u.h[3] = __builtin_amdgcn_cvt_pkrtz(hi.z, hi.w);
    }
    return u.v;
}

// The power of two that brings numbers of at most the given magnitude (its float bits) to 2^14 .. 2^15, so
// that half precision never overflows, or of less than 2^-10, whose coordinates would fall among its subnormal
// numbers and pass the filter nearly all (10^5 x 96 below 10^-5, degree 60: build 26.2 ms, scaled up 22.7); 1 for
// those between.  At most 2^40: what the distances themselves lose below the smallest float32,
// some (d + 16) 2^-149 of their square, then stays far below the filter's slack of 2 % of (2 r0)^2.
__device__ inline float ef_f16_scale(u32 max_bits)
{
    const int x_exp = (int)(max_bits >> 23) - 127;
    return x_exp >= 15 || x_exp < -10 ? __uint_as_float((u32)(127 + min(14 - x_exp, 40)) << 23) : 1.0f;
}
// A threshold as the filter compares it: thr (a float's bits) times thr_scale scale^2.  One scale goes to either
// factor: the square of a scale below 2^-74 (coordinates from 2^89 on) is no float, the product may well be one.
__device__ inline float ef_scaled_threshold(u32 thr, float scale, float thr_scale)
{
    return (__uint_as_float(thr) * scale) * (scale * thr_scale);
}
// Square roots for the filter only, never too small: the instruction is good to one unit in the last
// place, and inputs below the normal numbers are taken for the smallest of them.
__device__ inline float ef_sqrt_up(float t) { return fmaxf(__builtin_amdgcn_sqrtf(t), 1.1e-19f) * 1.000001f; }

// What the half-precision filter needs to know about the dimension (see nndescent_run for the bound).
struct F16Filter {
    float margin, thr_scale, u, rho0;
};
inline F16Filter f16_filter(int d)
{
    const int dpad = (d + 15) & ~15;
    F16Filter f;
    f.margin = (float)(4.0 * (dpad + 4.0) * 1.1920928955078125e-07 + 16.0 * 5.9604644775390625e-08);
    f.thr_scale = (float)((1.0 + 4.0 * (d / 16.0 + 8.0) * 5.9604644775390625e-08) * (1.0 + 1e-6));
    f.u = (float)(1.01 / 1023.0);
    f.rho0 = (float)(1.01 * sqrt((double)d) * 5.9604644775390625e-08);
    return f;
}

// ---------------------------------------------------------------------------------------
// Alg. 3 above the leaves: for every ancestor N of a point's leaf with depth >= dep, the point
// is sent down the subtree of N's other child by the split test of each node it meets, and the
// members of the leaf it reaches become candidates.  Runs after the leaf step of the same
// tree, in two kernels: classify_kernel finds the leaf reached for every point and level,
// conquer_kernel (one wave per home leaf, which owns its members' graph rows during the
// launch) evaluates the distances and merges.
//
// The members of a home leaf share their ancestors but land in different leaves of a sibling
// subtree more often than not, so every member is handled against its own leaf: lane (r, g)
// keeps its share of home member r as in init_reg_kernel and loads the same share of the
// members of the leaf that r reached, one after the other (members that reached the same leaf
// find those rows in the cache).  Eight such members give eight sets of partial sums, which
// the four lanes of a row add up in the fixed tree, transposed, as for rotations.  Rows are
// merged by rank in LDS after every level and stored at the end.
// Requires leaves of at most 16 points and d >= 4.

// partial sums of one pair: lane (r, g) adds the terms of its coordinates
__device__ inline void accumulate_pair(const float4 (&va)[8], const float4 (&vb)[8], int n_pieces, float (&p)[4])
{
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        if (s >= n_pieces) break;
        const float d0 = va[s].x - vb[s].x, d1 = va[s].y - vb[s].y, d2 = va[s].z - vb[s].z,
                    d3 = va[s].w - vb[s].w;
        p[0] = __builtin_fmaf(d0, d0, p[0]);
        p[1] = __builtin_fmaf(d1, d1, p[1]);
        p[2] = __builtin_fmaf(d2, d2, p[2]);
        p[3] = __builtin_fmaf(d3, d3, p[3]);
    }
}

// Which leaf of each sibling subtree every point reaches: etab[p * levels + k] for the point at
// position p of the tree's id array and the k-th ancestor of its leaf (k = 0: the leaf's
// parent), -1 where there is no such ancestor or its depth is below dep.  A wave takes one
// leaf at a time: all lanes climb the ancestors together (the links are the same for every
// member), then lane (member r, slot g) sends member r down the sibling subtrees of ancestors
// g, g+4, ...  Light on registers, so that many waves hide the chains of dependent loads.
// Node j is the right child of its parent pj iff j > pj, leaf l iff l >= pj (nodes are
// numbered by the leaf that starts their right part).  Links are clamped to the tables and
// walks are bounded, so tables that are not the tree builder's cannot lead out of them.
__global__ void __launch_bounds__(kBlock)
classify_kernel(const float *__restrict__ X, int d, const int *__restrict__ perm_t,
                const int *__restrict__ leaf_off_t, int n_leaves,
                const efanna_node *__restrict__ nodes_t, const int *__restrict__ leaf_up_t, int dep,
                int levels, int *__restrict__ etab)
{
    __shared__ int sib_sh[kBlock / EF_WAVE][64];      // sibling subtree of the k-th ancestor
    const int lane = ef_lane(), wave = threadIdx.x / EF_WAVE, r16 = lane & 15, g = lane >> 4;
    const int last = n_leaves - 1;
    const int n_waves = gridDim.x * (kBlock / EF_WAVE);
    for (int leaf = blockIdx.x * (kBlock / EF_WAVE) + wave; leaf < n_leaves; leaf += n_waves) {
        const int b0 = leaf_off_t[leaf];
        const int s = min(leaf_off_t[leaf + 1] - b0, 16);
        const int my_id = r16 < s ? perm_t[b0 + r16] : -1;
        int n_lev = 0;
        int up = min(leaf_up_t[leaf], 2 * last + 1);
        while (up >= 0 && n_lev < levels && n_lev < 64) {
            const int j = up >> 1;
            const efanna_node anc = nodes_t[j];
            if (anc.depth < dep) break;
            if (lane == 0) sib_sh[wave][n_lev] = anc.child[1 - (up & 1)];
            ++n_lev;
            const int pj = min(anc.parent, last);
            up = pj < 0 ? -1 : pj * 2 + (j > pj ? 1 : 0);
        }
        // one wave: its LDS operations complete in program order; keep the compiler from moving
        // the reads below above the writes
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (r16 < s) {
            for (int k = g; k < levels; k += 4) {
                int e = -1;
                if (k < n_lev) {
                    int c = sib_sh[wave][k];
                    for (int steps = 0; c >= 0 && steps < 4096; ++steps) {
                        const efanna_node nd = nodes_t[min(c, last)];
                        const float *xi = X + (size_t)my_id * d;
                        const bool left = !ef_has_test(nd.dim) ||
                                          (long long)nd.cnt * ef_node_value([&](int j) { return xi[j]; }, d, nd.dim) < nd.sum;
                        c = nd.child[left ? 0 : 1];
                    }
                    e = c >= 0 ? 0 : min(~c, last);
                }
                etab[(size_t)(b0 + r16) * levels + k] = e;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

template <bool ALIGNED>      // (three waves per SIMD: two lose 20 % on the headline data, whatever the spills of the unaligned form)
__global__ void __launch_bounds__(EF_WAVE) __attribute__((amdgpu_waves_per_eu(3)))
conquer_kernel(const float *__restrict__ X, int d, const int *__restrict__ perm_t,
               const int *__restrict__ leaf_off_t, int n_leaves, const int *__restrict__ etab,
               int levels, int K, u64 *graph)
{
    extern __shared__ __align__(16) float smem[];
    u64 *pools_a = (u64 *)smem;                       // [16][K] rows being merged, ascending
    u64 *pools_b = pools_a + 16 * (size_t)K;          // [16][K] the other copy
    u64 *cand = pools_b + 16 * (size_t)K;             // [16][kCandPitch]
    int *uid_b = (int *)(cand + 16 * kCandPitch);     // [16][16] members of the leaf each row reached
    const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
    for (int leaf = blockIdx.x; leaf < n_leaves; leaf += gridDim.x) {
        const int b0 = leaf_off_t[leaf];
        const int s = min(leaf_off_t[leaf + 1] - b0, 16);
        // the ancestors are those of the leaf: a level exists for all members or for none
        int e = r16 < s ? etab[(size_t)(b0 + r16) * levels] : -1;
        if (__ballot(e >= 0) == 0) continue;      // nothing above this leaf to visit
        const int my_id = r16 < s ? perm_t[b0 + r16] : -1;
        const float *pa = X + (size_t)max(my_id, 0) * d;
        __syncthreads();                  // the previous leaf's LDS reads are done
        u64 *cur = pools_a, *nxt = pools_b;
        for (int c = g; c < K; c += 4)
            cur[r16 * K + c] = r16 < s ? graph[(size_t)my_id * K + c] : ef_empty_entry(K - 1 - c);
        for (int k = 0; k < levels; ++k) {
            if (k > 0) {
                e = r16 < s ? etab[(size_t)(b0 + r16) * levels + k] : -1;
                if (__ballot(e >= 0) == 0) break;
            }
            e = min(e, n_leaves - 1);
            {
                // ---- every member against the members of the leaf it reached ----------------------
                const bool target = e >= 0;
                const int bb = target ? leaf_off_t[e] : 0;
                const int sb = target ? min(leaf_off_t[e + 1] - bb, 16) : 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int j = 4 * g + q;
                    uid_b[r16 * 16 + j] = j < sb ? perm_t[bb + j] : -1;
                }
                __syncthreads();                  // uid_b and the current rows are visible
                float dist[4];      // members 2g, 2g+1, 8+2g, 8+2g+1 of that leaf
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    float P[8][4];
#pragma unroll
                    for (int t = 0; t < 8; ++t) P[t][0] = P[t][1] = P[t][2] = P[t][3] = 0.0f;
                    for (int c0 = 0; c0 < d; c0 += 128) {
                        float4 va[8];
                        load_pieces<ALIGNED>(va, pa, c0, g, d, r16 < s);
                        const int n_pieces = min(8, (d - c0 + 15) >> 4);
#pragma unroll
                        for (int t = 0; t < 8; ++t) {
                            const int id_b = uid_b[r16 * 16 + 8 * half + t];
                            float4 vb[8];
                            load_pieces<ALIGNED>(vb, X + (size_t)max(id_b, 0) * d, c0, g, d, id_b >= 0);
                            accumulate_pair(va, vb, n_pieces, P[t]);
                        }
                    }
                    float two[2];
                    reduce_rotations(P, two);
                    dist[2 * half] = two[0];
                    dist[2 * half + 1] = two[1];
                }
                // ---- candidates of row r16 and their ranks ------------------------------------
                u64 key[4];
                int lt[4];
                const u64 *row = cur + r16 * K;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int bm = 8 * (c >> 1) + 2 * g + (c & 1);      // member of the leaf reached
                    key[c] = bm < sb ? ef_pack(dist[c], uid_b[r16 * 16 + bm], 1) : ~0ULL;
                    int lo = 0, hi_ = K;
                    if (key[c] != ~0ULL) {
                        while (lo < hi_) {
                            const int mid = (lo + hi_) >> 1;
                            if (row[mid] < key[c]) lo = mid + 1;
                            else hi_ = mid;
                        }
                        if (lo < K && row[lo] == key[c]) key[c] = ~0ULL;      // already in the row
                    }
                    lt[c] = lo;
                    cand[r16 * kCandPitch + 4 * g + c] = key[c];
                }
                __syncthreads();
                u64 cs[16];
#pragma unroll
                for (int o = 0; o < 16; ++o) cs[o] = cand[r16 * kCandPitch + o];
                u64 *out = nxt + r16 * K;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (key[c] == ~0ULL) continue;
                    int rank = lt[c];
#pragma unroll
                    for (int o = 0; o < 16; ++o) rank += cs[o] < key[c] ? 1 : 0;
                    if (rank < K) out[rank] = key[c];
                }
                for (int j = g; j < K; j += 4) {
                    const u64 en = row[j];
                    int rank = j;
#pragma unroll
                    for (int o = 0; o < 16; ++o) rank += cs[o] < en ? 1 : 0;
                    if (rank < K) out[rank] = en;
                }
                __syncthreads();                  // merged rows complete before they are read again
                u64 *tmp = cur;
                cur = nxt;
                nxt = tmp;
            }
        }
        if (r16 < s)
            for (int c = g; c < K; c += 4) graph[(size_t)my_id * K + c] = cur[r16 * K + c];
    }
}

// The same for vectors of at most 128 coordinates, by the leaves reached instead of by members: the
// members of a home leaf that reach the same leaf are handled together, so that the rows of that leaf are
// fetched once for all of them (the sibling of a leaf is mostly a leaf: one fetch where conquer_kernel
// has up to sixteen; three levels up there are four leaves to reach), and the home rows once for all
// levels.  A Gram block in half precision with the joins' bound and the rows' own K-th distances
// drops most pairs (scale: from the rows in hand); the others get their fixed-order distance from
// the same registers as in join_tile_kernel and become candidates of their row.
// conquer_kernel fetched 135 GB of rows through the caches for three levels of eight trees of 10^6 x 128:
// 12.3 -> 6.2 ms.  (At one level above the leaves, 10^5 x 96: 1.31 -> 1.12 ms with the trees; at seven, 3 10^5 x 100:
// 10.5 -> 6.2.)
template <bool ALIGNED>
__global__ void __launch_bounds__(EF_WAVE) __attribute__((amdgpu_waves_per_eu(4)))
conquer_tile_kernel(const float *__restrict__ X, int d, const int *__restrict__ perm_t,
                    const int *__restrict__ leaf_off_t, int n_leaves, const int *__restrict__ etab,
                    int levels, int K, F16Filter flt, u64 *graph)
{
    extern __shared__ __align__(16) float smem[];
    u64 *pools_a = (u64 *)smem;                       // [16][K] rows being merged, ascending
    u64 *pools_b = pools_a + 16 * (size_t)K;          // [16][K] the other copy
    u64 *cand = pools_b + 16 * (size_t)K;             // [16][kCandPitch]
    float *fa = (float *)(cand + 16 * kCandPitch);    // [4][16] the filter's terms of the home rows
    float *fb = fa + 64;                              // [2][16] ... of the rows of the leaf reached
    int *uid_b = (int *)(fb + 32);                    // [16] members of the leaf reached
    int *ncand = uid_b + 16;                          // [16] candidates of each home row
    unsigned short *surv = (unsigned short *)(ncand + 16);      // [256] surviving pairs
    const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
    auto wave_max = [](u32 m) {
        for (int o = 32; o >= 1; o >>= 1) m = max(m, (u32)__shfl_xor((int)m, o, EF_WAVE));
        return m;
    };
    auto magnitude = [&](const float4 (&v)[8]) {      // float bits of the largest |coordinate| of a tile
        float m = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) m = fmaxf(fmaxf(fmaxf(m, fabsf(v[s].x)), fmaxf(fabsf(v[s].y), fabsf(v[s].z))), fabsf(v[s].w));
        return wave_max(__float_as_uint(m));
    };
    auto diagonal = [&](const floatx4 &acc) {      // in lane (r16, r16 >> 2): row r16's
        const int kd = r16 & 3;
        return kd == 0 ? acc[0] : kd == 1 ? acc[1] : kd == 2 ? acc[2] : acc[3];
    };
    for (int leaf = blockIdx.x; leaf < n_leaves; leaf += gridDim.x) {
        const int b0 = leaf_off_t[leaf];
        const int s = min(leaf_off_t[leaf + 1] - b0, 16);
        // the ancestors are those of the leaf: a level exists for all members or for none
        int e = r16 < s ? etab[(size_t)(b0 + r16) * levels] : -1;
        if (__ballot(e >= 0) == 0) continue;      // nothing above this leaf to visit
        const int my_id = r16 < s ? perm_t[b0 + r16] : -1;
        float4 va[8];
        load_pieces<ALIGNED>(va, X + (size_t)max(my_id, 0) * d, 0, g, d, r16 < s);
        __syncthreads();                  // the previous leaf's LDS reads are done
        u64 *cur = pools_a, *nxt = pools_b;
        for (int c = g; c < K; c += 4)
            cur[r16 * K + c] = r16 < s ? graph[(size_t)my_id * K + c] : ef_empty_entry(K - 1 - c);
        const u32 mag_a = magnitude(va);
        for (int k = 0; k < levels; ++k) {
            if (k > 0) {
                e = r16 < s ? etab[(size_t)(b0 + r16) * levels + k] : -1;
                if (__ballot(e >= 0) == 0) break;
            }
            e = min(e, n_leaves - 1);
            if (lane < 16) ncand[lane] = 0;
            __syncthreads();
            const u32 thr = ef_dist_bits(cur[r16 * K + K - 1]);      // a row's largest entry
            for (u32 left = (u32)__ballot(e >= 0) & 0xFFFFu; left;) {
                // ---- the members that reach the same leaf as the first of those left --------------
                const int t = __shfl(e, __ffs(left) - 1, EF_WAVE);
                const u32 members = (u32)__ballot(e == t) & 0xFFFFu;
                left &= ~members;
                const int bb = leaf_off_t[t], sb = min(leaf_off_t[t + 1] - bb, 16);
                const int id_b = r16 < sb ? perm_t[bb + r16] : -1;
                float4 vb[8];
                load_pieces<ALIGNED>(vb, X + (size_t)max(id_b, 0) * d, 0, g, d, r16 < sb);
                const float scale = ef_f16_scale(max(mag_a, magnitude(vb)));
                floatx4 ab = {0.f, 0.f, 0.f, 0.f}, aa = ab, bbq = ab;
#pragma unroll
                for (int q = 0; q < 8; q += 2) {
                    if (16 * q >= d) break;
                    const f16x8 oa = ef_pack_f16<true>(va[q], va[q + 1], scale), ob = ef_pack_f16<true>(vb[q], vb[q + 1], scale);
                    ab = __builtin_amdgcn_mfma_f32_16x16x32_f16(oa, ob, ab, 0, 0, 0);
                    aa = __builtin_amdgcn_mfma_f32_16x16x32_f16(oa, oa, aa, 0, 0, 0);
                    bbq = __builtin_amdgcn_mfma_f32_16x16x32_f16(ob, ob, bbq, 0, 0, 0);
                }
                if (g == 0) uid_b[r16] = id_b;
                if ((r16 >> 2) == g) {
                    const float da = diagonal(aa), db = diagonal(bbq), th = ef_scaled_threshold(thr, scale, flt.thr_scale);
                    fa[r16] = da * (1.0f - flt.margin);
                    fa[16 + r16] = __builtin_fmaf(flt.u, ef_sqrt_up(da), flt.rho0);
                    fa[32 + r16] = th;
                    fa[48 + r16] = 2.0f * ef_sqrt_up(th);
                    fb[r16] = db * (1.0f - flt.margin);
                    fb[16 + r16] = __builtin_fmaf(flt.u, ef_sqrt_up(db), flt.rho0);
                }
                __syncthreads();
                // ---- filter: the lane holds G[a = 4 g + k][b = r16] --------------------------------
                const float nfb = fb[r16], rrb = fb[16 + r16];
                int n_surv = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int a = 4 * g + q;
                    const float lhs = __builtin_fmaf(-2.0f, ab[q], fa[a] + nfb), rad = fa[16 + a] + rrb;
                    const bool keep = r16 < sb && ((members >> a) & 1) && !(lhs > __builtin_fmaf(rad, fa[48 + a] + rad, fa[32 + a]));
                    const u64 kept = __ballot(keep);
                    if (keep) surv[n_surv + lanes_below(kept)] = (unsigned short)(a | (r16 << 8));
                    n_surv += __popcll(kept);
                }
                __syncthreads();
                // ---- survivors from registers, sixteen pairs per round (see join_reg_kernel) ---------
                for (int p0 = 0; p0 < n_surv; p0 += 16) {
                    const bool has = p0 + r16 < n_surv;
                    const u32 ent = surv[min(p0 + r16, n_surv - 1)];
                    const int al = ent & 15, bl = (ent >> 8) & 15;
                    const int src_a = al + 16 * g, src_b = bl + 16 * g;
                    float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        if (16 * q >= d) break;
                        const float d0 = __shfl(va[q].x, src_a, EF_WAVE) - __shfl(vb[q].x, src_b, EF_WAVE);
                        const float d1 = __shfl(va[q].y, src_a, EF_WAVE) - __shfl(vb[q].y, src_b, EF_WAVE);
                        const float d2 = __shfl(va[q].z, src_a, EF_WAVE) - __shfl(vb[q].z, src_b, EF_WAVE);
                        const float d3 = __shfl(va[q].w, src_a, EF_WAVE) - __shfl(vb[q].w, src_b, EF_WAVE);
                        p[0] = __builtin_fmaf(d0, d0, p[0]);
                        p[1] = __builtin_fmaf(d1, d1, p[1]);
                        p[2] = __builtin_fmaf(d2, d2, p[2]);
                        p[3] = __builtin_fmaf(d3, d3, p[3]);
                    }
                    const float dist = ef_sum_partials(p[0], p[1], p[2], p[3]);
                    if (has && g == 0) cand[al * kCandPitch + atomicAdd(&ncand[al], 1)] = ef_pack(dist, uid_b[bl], 1);
                }
                __syncthreads();
            }
            // ---- candidates of row r16 and their ranks ------------------------------------------
            const int nc = ncand[r16];
            if (__ballot(nc > 0) == 0) continue;      // no row has one: the rows stay as they are
            u64 key[4];
            int lt[4];
            const u64 *row = cur + r16 * K;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                key[c] = 4 * g + c < nc ? cand[r16 * kCandPitch + 4 * g + c] : ~0ULL;
                int lo = 0, hi_ = K;
                if (key[c] != ~0ULL) {
                    while (lo < hi_) {
                        const int mid = (lo + hi_) >> 1;
                        if (row[mid] < key[c]) lo = mid + 1;
                        else hi_ = mid;
                    }
                    if (lo < K && row[lo] == key[c]) key[c] = ~0ULL;      // already in the row
                }
                lt[c] = lo;
            }
            __syncthreads();                  // every candidate is read before any slot is written again
#pragma unroll
            for (int c = 0; c < 4; ++c) cand[r16 * kCandPitch + 4 * g + c] = key[c];
            __syncthreads();
            u64 cs[16];
#pragma unroll
            for (int o = 0; o < 16; ++o) cs[o] = cand[r16 * kCandPitch + o];
            u64 *out = nxt + r16 * K;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (key[c] == ~0ULL) continue;
                int rank = lt[c];
#pragma unroll
                for (int o = 0; o < 16; ++o) rank += cs[o] < key[c] ? 1 : 0;
                if (rank < K) out[rank] = key[c];
            }
            for (int j = g; j < K; j += 4) {
                const u64 en = row[j];
                int rank = j;
#pragma unroll
                for (int o = 0; o < 16; ++o) rank += cs[o] < en ? 1 : 0;
                if (rank < K) out[rank] = en;
            }
            __syncthreads();                  // merged rows complete before they are read again
            u64 *tmp = cur;
            cur = nxt;
            nxt = tmp;
        }
        if (r16 < s)
            for (int c = g; c < K; c += 4) graph[(size_t)my_id * K + c] = cur[r16 * K + c];
    }
}

// ---------------------------------------------------------------------------------------
// The same step for any leaf size up to 64 and any dimension (the kernels above want leaves of at
// most 16 points and d >= 4).  classify_any_kernel: one wave per leaf, lane r sends member r
// down the sibling subtree of every ancestor in range.  conquer_any_kernel: one wave per member
// (the waves of a block take the members of one home leaf, which owns its members' rows during
// the launch); per level the wave evaluates its member against the members of the leaf reached,
// one pair per group of sixteen lanes in the library's fixed order, and merges by rank in LDS.
__global__ void __launch_bounds__(kBlock)
classify_any_kernel(const float *__restrict__ X, int d, const int *__restrict__ perm_t,
                    const int *__restrict__ leaf_off_t, int n_leaves,
                    const efanna_node *__restrict__ nodes_t, const int *__restrict__ leaf_up_t, int dep,
                    int levels, int *__restrict__ etab)
{
    const int lane = ef_lane(), wave = threadIdx.x / EF_WAVE;
    const int last = n_leaves - 1;
    const int n_waves = gridDim.x * (kBlock / EF_WAVE);
    for (int leaf = blockIdx.x * (kBlock / EF_WAVE) + wave; leaf < n_leaves; leaf += n_waves) {
        const int b0 = leaf_off_t[leaf];
        const int s = min(leaf_off_t[leaf + 1] - b0, EF_WAVE);
        if (lane >= s) continue;
        const int my_id = perm_t[b0 + lane];
        int up = min(leaf_up_t[leaf], 2 * last + 1);
        for (int k = 0; k < levels; ++k) {
            int e = -1;
            if (up >= 0) {
                const int j = up >> 1;
                const efanna_node anc = nodes_t[j];
                if (anc.depth >= dep) {
                    int c = anc.child[1 - (up & 1)];
                    for (int steps = 0; c >= 0 && steps < 4096; ++steps) {      // (bounded: foreign tables cannot hold it)
                        const efanna_node nd = nodes_t[min(c, last)];
                        const float *xi = X + (size_t)my_id * d;
                        const bool left = !ef_has_test(nd.dim) ||
                                          (long long)nd.cnt * ef_node_value([&](int j) { return xi[j]; }, d, nd.dim) < nd.sum;
                        c = nd.child[left ? 0 : 1];
                    }
                    e = c >= 0 ? 0 : min(~c, last);
                    const int pj = min(anc.parent, last);
                    up = pj < 0 ? -1 : pj * 2 + (j > pj ? 1 : 0);
                } else {
                    up = -1;
                }
            }
            etab[(size_t)(b0 + lane) * levels + k] = e;
        }
    }
}

__global__ void __launch_bounds__(kBlock)
conquer_any_kernel(const float *__restrict__ X, int d, const int *__restrict__ perm_t,
                   const int *__restrict__ leaf_off_t, int n_leaves, const int *__restrict__ etab,
                   int levels, int K, u64 *graph)
{
    extern __shared__ __align__(16) float smem[];
    const int lane = ef_lane(), wave = threadIdx.x / EF_WAVE, n_waves = kBlock / EF_WAVE;
    const int grp = lane >> 4, gl = lane & 15;
    u64 *row_a = (u64 *)smem + (size_t)wave * (2 * K + EF_WAVE);      // [K] the row being merged, ascending
    u64 *row_b = row_a + K;                                           // [K] the other copy
    u64 *cand = row_b + K;                                            // [64] candidates of the level in hand
    auto wave_sync = [&]() {      // one wave: its LDS operations complete in program order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int leaf = blockIdx.x; leaf < n_leaves; leaf += gridDim.x) {
        const int b0 = leaf_off_t[leaf];
        const int s = min(leaf_off_t[leaf + 1] - b0, EF_WAVE);
        for (int r = wave; r < s; r += n_waves) {
            if (levels < 1 || etab[(size_t)(b0 + r) * levels] < 0) continue;      // nothing above this leaf to visit
            const int my_id = perm_t[b0 + r];
            const float *xa = X + (size_t)my_id * d;
            u64 *cur = row_a, *nxt = row_b;
            wave_sync();
            for (int c = lane; c < K; c += EF_WAVE) cur[c] = graph[(size_t)my_id * K + c];
            for (int k = 0; k < levels; ++k) {
                const int e = etab[(size_t)(b0 + r) * levels + k];
                if (e < 0) break;      // the ancestors in range are the first ones
                const int bb = leaf_off_t[min(e, n_leaves - 1)];
                const int sb = min(leaf_off_t[min(e, n_leaves - 1) + 1] - bb, EF_WAVE);
                // ---- distances to the members of the leaf reached, four pairs at a time -----------
                for (int j0 = 0; j0 < sb; j0 += 4) {
                    const int j = min(j0 + grp, sb - 1);      // (whole groups stay busy)
                    const int id_b = perm_t[bb + j];
                    const float *xb = X + (size_t)id_b * d;
                    float acc = 0.0f;
                    for (int t = gl; t < d; t += 16) {
                        const float diff = xa[t] - xb[t];
                        acc = __builtin_fmaf(diff, diff, acc);
                    }
                    acc = ef_group_reduce16(acc);
                    if (gl == 0 && j0 + grp < sb) cand[j0 + grp] = id_b != my_id ? ef_pack(acc, id_b, 1) : ~0ULL;
                }
                wave_sync();
                // ---- merge by rank: K old entries and sb candidates, the K smallest stay ------------
                u64 key = ~0ULL;
                int below = 0;      // old entries below the candidate
                if (lane < sb) {
                    key = cand[lane];
                    int lo = 0, hi = K;
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (cur[mid] < key) lo = mid + 1;
                        else hi = mid;
                    }
                    if (lo < K && cur[lo] == key) key = ~0ULL;      // already in the row
                    below = lo;
                }
                wave_sync();
                cand[lane] = key;      // (dropped candidates become the largest key: they count for nobody)
                wave_sync();
                if (key != ~0ULL) {
                    int rank = below;
                    for (int o = 0; o < sb; ++o) rank += cand[o] < key ? 1 : 0;
                    if (rank < K) nxt[rank] = key;
                }
                for (int c = lane; c < K; c += EF_WAVE) {
                    const u64 en = cur[c];
                    int rank = c;
                    for (int o = 0; o < sb; ++o) rank += cand[o] < en ? 1 : 0;
                    if (rank < K) nxt[rank] = en;
                }
                wave_sync();
                u64 *tmp = cur;
                cur = nxt;
                nxt = tmp;
            }
            for (int c = lane; c < K; c += EF_WAVE) graph[(size_t)my_id * K + c] = cur[c];
        }
    }
}

// ---------------------------------------------------------------------------------------
// Alg. 4 step 1+2: sample the new / old sets of every row, clear the sampled marks,
// refresh the row's threshold and enter the row's id into the reverse lists of the
// sampled neighbours.
//
// A row is handled by a group of G lanes holding E entries each (G*E >= K); ranks among
// the marked and the unmarked entries come from broadcasting every entry to the group.
//
// Reverse lists keep the L members with the smallest (hash, source) key.  Most lists
// never overflow, so the first L arrivals of a list just take the next free slot (one
// counter bump); later arrivals are parked in an overflow queue and settled by
// reverse_overflow_kernel, after this kernel has finished, with the bounded insertion.
// Whatever the arrival order, a list ends up with the L smallest keys offered to it.

struct Overflow {
    u64 key;      // hash << 32 | source
    int target;   // list owner
    int which;    // 0: reverse-new, 1: reverse-old
};

// Parked keys go to kOvfQueues dense queues, block b of the sampling kernels to queue
// b % kOvfQueues: a wave bumps its queue's counter once for all the keys it parks (bumps of one
// address serialise, so the counters are many and a cache line apart), and
// reverse_overflow_kernel gets one thread per parked key instead of a sweep over all rows.
// A row parks at most K keys, so a queue holds at most (blocks per queue) x (rows per block) x K.

__host__ __device__ inline int sample_group_for(int K) { return K <= 16 ? 16 : (K <= 32 ? 32 : 64); }

__host__ __device__ inline size_t ovf_region_for(int64_t n, int K)
{
    const int G = sample_group_for(K);
    const size_t blocks = ((size_t)n * G + kBlock - 1) / kBlock;
    return (blocks + kOvfQueues - 1) / kOvfQueues * (size_t)(kBlock / G) * K;
}

// All lanes of the wave call this together; lanes with `parked` set file `o`.
__device__ inline void park_keys(bool parked, const Overflow &o, Overflow *overflow, size_t region,
                                 int *ovf_count)
{
    const u64 mask = __ballot(parked);
    if (mask == 0) return;
    const int q = blockIdx.x % kOvfQueues, leader = __ffsll((unsigned long long)mask) - 1;
    int base = 0;
    if (ef_lane() == leader) base = atomicAdd(ovf_count + q * kOvfCounterPitch, __popcll(mask));
    base = __shfl(base, leader, EF_WAVE);
    if (parked) overflow[(size_t)q * region + base + lanes_below(mask)] = o;
}

// Offer `key` to reverse list v.  Returns true if the list had no free slot: the caller
// parks the key for reverse_overflow_kernel.  Every offer bumps the list's counter, full or
// not: a read beforehand to spare full lists the bump costs more transactions than it saves
// (bumps of one counter serialise at about 11 ns each, so a point that is the neighbour of
// c others costs c * 11 ns at worst).
__device__ inline bool reverse_offer(u64 *lists, int *counts, int L, int v, u64 key)
{
    const int pos = atomicAdd(&counts[v], 1);
    if (pos >= L) return true;
    lists[(size_t)v * L + pos] = key;
    return false;
}

// Entry gl + h * G of row i for lane gl of the row's group (the largest key where there is none).
template <int G, int E>
__device__ inline void sample_load(const u64 *graph, int i, bool row_ok, int K, u64 (&e)[E])
{
    const int gl = threadIdx.x & (G - 1);
#pragma unroll
    for (int h = 0; h < E; ++h) {
        const int slot = gl + h * G;
        e[h] = row_ok && slot < K ? graph[(size_t)i * K + slot] : ~0ULL;
    }
}

// The sampling of row i by its group of G lanes, which hold the row's entries e as sample_load
// delivers them (all lanes of the wave call this together, rows past the end with row_ok false).
// offer(take, id): called by every lane once per entry it holds; lanes with `take` set offer
// row i to the reverse-new list of point id.
template <int G, int E, class Offer>
__device__ inline void sample_row(u64 *graph, const u64 (&e)[E], int i, bool row_ok, int K, int L,
                                  int *__restrict__ nw, int *__restrict__ od, int *__restrict__ nw_c,
                                  int *__restrict__ od_c, u32 *worst, Offer &&offer)
{
    const int gl = threadIdx.x & (G - 1);
    int rn[E], ro[E];
    const bool all_sampled = K <= L;
    u64 sampled_to = ~0ULL;      // key of the L-th new entry, if there is one (a row to a wave)
    if (all_sampled) {
        // Rows no longer than the sample: every marked entry is sampled and every other entry is
        // old, whatever their ranks.  The two lists are sets (their order decides nothing), so
        // the places in them are handed out by compaction: a ballot instead of K broadcasts.
        const int lane = ef_lane();
        const u64 group = (G == 64 ? ~0ULL : ((1ULL << (G & 63)) - 1)) << (lane & ~(G - 1));
        const u64 below = group & ((1ULL << lane) - 1);
        int base_n = 0, base_o = 0;
#pragma unroll
        for (int h = 0; h < E; ++h) {
            const bool valid = gl + h * G < K;
            const u64 bn = __ballot(valid && (e[h] & 1)) & group;
            const u64 bo = __ballot(valid && !(e[h] & 1) && !ef_is_empty(e[h])) & group;
            rn[h] = base_n + __popcll(bn & below);
            ro[h] = base_o + __popcll(bo & below);
            base_n += __popcll(bn);
            base_o += __popcll(bo);
        }
    } else if (G == 64) {
        // A row to a wave (K > 32): the L-th smallest new key bit by bit from ballots - 32 steps over the
        // distances, and as many over the rest only if that distance is not unique - and then places by
        // compaction as above.  (Ranks by broadcasting every entry, as below, took 1400 instructions a
        // row at K = 100: 10^6 rows 2.6 -> 1.2 ms per iteration.)
        bool nw_e[E];
        int n_new = 0;
#pragma unroll
        for (int h = 0; h < E; ++h) {
            nw_e[h] = gl + h * G < K && (e[h] & 1);
            n_new += __popcll(__ballot(nw_e[h]));
        }
        if (n_new >= L) {
            auto kth = [&](auto part, auto in, int k) {      // the k-th smallest part(e) among the entries with in(h)
                u32 t = 0;
                for (u32 bit = 1u << 31; bit; bit >>= 1) {
                    int c = 0;
#pragma unroll
                    for (int h = 0; h < E; ++h) c += __popcll(__ballot(in(h) && part(e[h]) < (t | bit)));
                    if (c < k) t |= bit;
                }
                return t;
            };
            auto hi = [](u64 x) { return (u32)(x >> 32); };
            auto lo = [](u64 x) { return (u32)x; };
            const u32 dist = kth(hi, [&](int h) { return nw_e[h]; }, L);
            int below = 0, ties = 0;
            u64 tied = 0;
#pragma unroll
            for (int h = 0; h < E; ++h) {
                below += __popcll(__ballot(nw_e[h] && hi(e[h]) < dist));
                const u64 at = __ballot(nw_e[h] && hi(e[h]) == dist);
                ties += __popcll(at);
                if (at) tied = __shfl(e[h], __ffsll((unsigned long long)at) - 1, EF_WAVE);
            }
            sampled_to = ties == 1 ? tied
                                   : (u64)dist << 32 | kth(lo, [&](int h) { return nw_e[h] && hi(e[h]) == dist; }, L - below);
        }
        int base_n = 0, base_o = 0;
#pragma unroll
        for (int h = 0; h < E; ++h) {
            const u64 bn = __ballot(nw_e[h] && e[h] <= sampled_to);
            const u64 bo = __ballot(gl + h * G < K && !(e[h] & 1) && !ef_is_empty(e[h]) && e[h] < sampled_to);
            rn[h] = nw_e[h] && e[h] <= sampled_to ? base_n + lanes_below(bn) : L;
            ro[h] = base_o + lanes_below(bo);
            base_n += __popcll(bn);
            base_o += __popcll(bo);
        }
    } else {
        // ranks among new-marked and among old entries (all lanes of the group take part)
#pragma unroll
        for (int h = 0; h < E; ++h) rn[h] = ro[h] = 0;
#pragma unroll
        for (int part = 0; part < E; ++part) {
            const int k_end = min(K - part * G, G);
            for (int k = 0; k < k_end; ++k) {
                const u64 o = __shfl(e[part], k, G);
                const bool o_new = o & 1, o_old = !o_new && !ef_is_empty(o);
#pragma unroll
                for (int h = 0; h < E; ++h) {
                    const bool less = o < e[h];
                    rn[h] += (less && o_new) ? 1 : 0;
                    ro[h] += (less && o_old) ? 1 : 0;
                }
            }
        }
    }
    bool is_new[E], is_old[E], take_new[E];
    int total_new = 0;
    u32 wbits = 0;
    u64 stop = ~0ULL;      // key of the L-th new entry, if there is one
#pragma unroll
    for (int h = 0; h < E; ++h) {
        const bool valid = gl + h * G < K;
        is_new[h] = valid && (e[h] & 1);
        is_old[h] = valid && !(e[h] & 1) && !ef_is_empty(e[h]);
        take_new[h] = is_new[h] && rn[h] < L;
        total_new += is_new[h] ? 1 : 0;
        if (valid) wbits = max(wbits, ef_dist_bits(e[h]));
        if (G != 64 && !all_sampled && take_new[h] && rn[h] == L - 1) stop = e[h];
    }
    for (int m = G / 2; m >= 1; m >>= 1) {
        total_new += __shfl_xor(total_new, m, G);
        wbits = max(wbits, (u32)__shfl_xor((int)wbits, m, G));
        if (G != 64) {
            const u64 other = __shfl_xor(stop, m, G);
            stop = other < stop ? other : stop;
        }
    }
    if (G == 64 && !all_sampled) stop = sampled_to;
    // sampled new entries lose their mark, go to the new list and are offered to the reverse-new
    // list of the neighbour; old entries only go to the old list here (reverse_old_kernel offers
    // them once it is known which points take part in a join at all)
    int n_old = 0;
#pragma unroll
    for (int h = 0; h < E; ++h) {
        const int slot = gl + h * G;
        const int id = ef_id(e[h]);
        if (row_ok && is_old[h] && e[h] < stop) {
            od[(size_t)i * K + ro[h]] = id;
            ++n_old;
        }
        const bool take = row_ok && take_new[h];
        if (take) {
            nw[(size_t)i * L + rn[h]] = id;
            graph[(size_t)i * K + slot] = e[h] & ~1ULL;
        }
        offer(take, id);
    }
    for (int m = G / 2; m >= 1; m >>= 1) n_old += __shfl_xor(n_old, m, G);
    if (!row_ok) return;
    // unused tails of both lists read as -1, so the join needs no counts to parse them
    const int n_new = min(total_new, L);
    for (int s = n_new + gl; s < L; s += G) nw[(size_t)i * L + s] = -1;
    for (int s = n_old + gl; s < K; s += G) od[(size_t)i * K + s] = -1;
    if (gl == 0) {
        nw_c[i] = n_new;
        od_c[i] = n_old;
        worst[i] = wbits;
    }
}

// The key under which `source` competes for a place in a reverse list of `target`.
__device__ inline u64 reverse_key(u64 stream_key, int target, int source)
{
    return (ef_mix64(stream_key + (((u64)(u32)target << 32) | (u32)source)) >> 32 << 32) | (u32)source;
}

template <int G, int E>
__global__ void __launch_bounds__(kBlock)
sample_kernel(u64 *graph, int n, int K, int L, u64 key_new, int *__restrict__ nw,
              int *__restrict__ od, int *__restrict__ nw_c, int *__restrict__ od_c, u64 *rnew,
              int *rnew_c, Overflow *overflow, size_t ovf_region, int *ovf_count, u32 *worst)
{
    const int i = (int)(((size_t)blockIdx.x * kBlock + threadIdx.x) / G);
    u64 e[E];
    sample_load<G, E>(graph, i, i < n, K, e);
    sample_row<G, E>(graph, e, i, i < n, K, L, nw, od, nw_c, od_c, worst, [&](bool take, int id) {
        bool parked = false;
        u64 hk = 0;
        if (take) {
            hk = reverse_key(key_new, id, i);
            parked = reverse_offer(rnew, rnew_c, L, id, hk);
        }
        park_keys(parked, Overflow{hk, id, 0}, overflow, ovf_region, ovf_count);
    });
}

// Bit i of `active` says whether point i has a non-empty U_new (a sampled new neighbour or a
// reverse-new member), i.e. whether it joins anything in this iteration.  One bit per point:
// the map of a million points is 128 KB and stays in L2 for the random look-ups that follow.
__global__ void __launch_bounds__(kBlock)
active_kernel(const int *__restrict__ nw_c, const int *__restrict__ rnew_c, int n, u64 *__restrict__ active)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const u64 mask = __ballot(i < n && (nw_c[i] > 0 || rnew_c[i] > 0));
    if (ef_lane() == 0 && (i & ~(EF_WAVE - 1)) < n) active[i / EF_WAVE] = mask;
}

// Reverse-old lists, after sampling: row i offers itself to the reverse-old list of each of its
// sampled old neighbours -- but only to those that join something; the list of a point whose
// U_new is empty is never read (Alg. 4 pairs U_old only with U_new), so it stays empty.
// One lane per slot of the old list, a group of G lanes per row as in sample_kernel; parked keys
// go behind the ones sample_kernel parked for the row.
template <int G>
__global__ void __launch_bounds__(kBlock)
reverse_old_kernel(const int *__restrict__ od, int n, int K, int L, u64 key_old,
                   const u64 *__restrict__ active, u64 *rold, int *rold_c, Overflow *overflow,
                   size_t ovf_region, int *ovf_count)
{
    const int gl = threadIdx.x & (G - 1);
    const int i = (int)(((size_t)blockIdx.x * kBlock + threadIdx.x) / G);
    const bool row_ok = i < n;
    for (int s0 = 0; s0 < K; s0 += G) {
        const int slot = s0 + gl;
        const int id = row_ok && slot < K ? od[(size_t)i * K + slot] : -1;
        bool parked = false;
        u64 hk = 0;
        if (id >= 0 && ((active[id / EF_WAVE] >> (id % EF_WAVE)) & 1)) {
            hk = reverse_key(key_old, id, i);
            parked = reverse_offer(rold, rold_c, L, id, hk);
        }
        park_keys(parked, Overflow{hk, id, 1}, overflow, ovf_region, ovf_count);
    }
}

// One thread per parked key (queue blockIdx.y, blocks of a queue stride over its keys).
// list_max[which][v] is an upper bound of the largest key of (full) list v, lowered after
// every successful insertion: the many keys offered to a popular point are turned away after
// one read instead of a scan of the list.
constexpr int kOvfBlocksPerQueue = 16;

// WIDE: lists of fifty keys or more are read fifty keys at a time.
template <bool WIDE>
__global__ void __launch_bounds__(kBlock)
reverse_overflow_kernel(const Overflow *__restrict__ overflow, size_t ovf_region,
                        const int *__restrict__ ovf_count, size_t n, u64 *rnew, u64 *rold,
                        u64 *list_max, int L)
{
    const int q = blockIdx.y, parked = ovf_count[q * kOvfCounterPitch];
    for (int e = blockIdx.x * kBlock + threadIdx.x; e < parked; e += kOvfBlocksPerQueue * kBlock) {
        const Overflow ov = overflow[(size_t)q * ovf_region + e];
        u64 *bound = list_max + (size_t)ov.which * n + ov.target;
        if (ov.key >= ef_load_coherent(bound)) continue;
        u64 nm;
        if (ef_bounded_insert_t<WIDE, true>((ov.which ? rold : rnew) + (size_t)ov.target * L, L, ov.key, 0, &nm))
            atomicMin(bound, nm);
    }
}

// ---------------------------------------------------------------------------------------
// Reverse lists without device-wide atomics, for short rows and lists (K, L <= 32) of at most
// 2^21 points (2^20 if L > 16; longer rows and lists: see wide_lists).  A counter bump per offer is bound by the rate of atomics on random addresses;
// here the offers are sorted by target range instead, and the lists of a range are built in LDS:
//   1. an offer block (one thread per row) handles 1024 consecutive source rows (256 of few points,
//      see BucketShape), keeps their
//      offers (one word: target << row bits | source row inside the block) in LDS, counts them per
//      bucket (a range of up to 1024 targets, of 512 if L > 16: the lists of a range have to fit the
//      LDS), and writes them to its own part of the offer array, bucket after bucket;
//      table[block][bucket] = start << 16 | count of that run (written in one piece; by bucket, a word into each
//      of as many lines as there are buckets, it cost the offer kernels 8 us a launch at 10^6 points, reading it across 2);
//   2. a list block (one per bucket) walks the runs of its bucket, sorts the offers by target in LDS and
//      writes every target's list (bucket_lists_kernel).
// Whatever the order of the offers, a list ends up with the L smallest keys offered to it.

constexpr int kBktRows = 1024;        // source rows per offer block, at most
constexpr int kBktThreads = 1024;
constexpr int kBktMany = 800;         // as many buckets are enough
// lists that take the bounded insertion (see bucket_insert_kernel)
__host__ __device__ inline bool insert_lists(int64_t n, int K, int L)
{
    return L <= 6 || (L == 7 && n > (1 << 17)) || (K <= 10 && L <= 10 && n <= 256);
}
constexpr int kBktFew = 4;            // offers per thread up to which it looks for their runs
constexpr int kBktWords = 16;         // offers a thread of a list block holds while they are sorted
                                      // (twice as many of long rows; two iterations with 12 and 24: the same where offers are spread evenly, 3 to 10 % longer
                                      // for data sorted by norm at degrees 32 and 64; 20 and 40: 1 to 2 % longer at degree 10 from 6 10^5 points on,
                                      // where a block less fits a CU, 4 to 8 % shorter by norm at degree 32 up to 3 10^5)
constexpr int kBktMaxRuns = 2 * kBktThreads;    // buckets and offer blocks a block-wide scan of two per thread takes

// log2 of the targets per bucket where the buckets are as large as LDS lets them be
__host__ __device__ inline int bucket_shift(int L) { return L <= 16 ? 10 : 9; }

__host__ __device__ inline size_t bucket_lists_lds(int L, int shift, int n_blocks);

__host__ __device__ inline bool bucketed_lists(int64_t n, int K, int L)
{
    if (K > 32 || L > 32 || n > (1 << 21)) return false;      // (targets fit 21 bits of an offer word)
    const int64_t n_blocks = (n + kBktRows - 1) / kBktRows, n_buckets = ((n - 1) >> bucket_shift(L)) + 1;
    return n_blocks <= kBktMaxRuns && n_buckets <= kBktMaxRuns &&
           bucket_lists_lds(L, bucket_shift(L), (int)n_blocks) <= 160 * 1024 - 256;
}

// How the offers are cut up.  Blocks of 1024 rows and ranges of 1024 targets leave most of the 256 CUs
// idle below some ten thousand points (10 blocks at 10^4), each with ten thousand offers to enter.
// Up to 2^16 points: offer blocks of 256 rows, and the smallest
// ranges that make at most 512 buckets (from 32 targets up).  (The table of runs is then larger, up to
// 8 bytes per point, and lies in the half of the reverse-old lists' room that 32-bit sources leave
// free: L >= 4.)  Builds of 2500 x 24 / 10^4 x 32 / 6 10^4 x 100 with degree 10, and of the last with degree 20: 660 ->
// 575 us, 890 -> 815, 2135 -> 2085, 3745 -> 3645.
// Beyond, ranges of 128 targets up, as large as make kBktMany of them (all list kernels of 10^5 points, degree 10, from a random
// start: 390 -> 328 us; degree 20 235 -> 230), and no larger than lets 1024 threads hold ten offers each.  (More of them
// for a million points, 1954 instead of 977: 998 -> 1039, and the offer kernels, which count and write runs per range, 1076 -> 1190.)
// There at least 512 threads for ranges of 256 targets up, because of popular points side by side, whose offers one block has to look at alone
// (200 000 x 8 from rows that name low ids more often, degree 10: 4.67 ms with 256, 3.54 with 512).  Ranges of 128 have 256: waves without
// offers cost 2 us a launch (100 000 x 8, degree 10, 1112 us, 1125 with 512); where they are offered more than ten each they
// have the LDS of 512 (see roomy).
struct BucketShape {
    int row_bits, blocks;           // log2 of the source rows of an offer block, number of blocks
    int shift, buckets, threads;    // log2 of the targets of a bucket, number of buckets, threads of a list block
    bool table_behind;              // the table of runs lies behind the reverse-old lists' 32-bit sources
};
inline BucketShape bucket_shape(int64_t n, int K, int L)
{
    const int per = K > L ? K : L;      // offers per target on average, if all rows are full
    BucketShape b;
    auto cut = [&](int row_bits, int shift) {
        b.row_bits = row_bits;
        b.shift = shift;
        b.blocks = (int)((n + (1 << row_bits) - 1) >> row_bits);
        b.buckets = (int)((n - 1) >> shift) + 1;
        b.threads = (per <= 10 || insert_lists(n, K, L) ? 1 : per <= 20 ? 2 : 4) << shift;
        const int least = insert_lists(n, K, L) || row_bits == 8 || shift <= 7 ? 256 : 512;
        b.threads = b.threads < least ? least : b.threads > kBktThreads ? kBktThreads : b.threads;
        b.table_behind = (int64_t)b.blocks * b.buckets <= n * L;
    };
    if (n <= (1 << 16) && L >= 4) {
        int shift = 5;
        while (((n - 1) >> shift) + 1 > 512) ++shift;
        cut(8, shift);
        if (b.table_behind) return b;
    }
    const int top = per <= 10 ? 10 : per <= 20 ? 9 : 8;
    for (int shift = 7; !insert_lists(n, K, L) && (shift <= 9 || shift <= top); ++shift) {
        cut(10, shift);
        if (b.table_behind && b.buckets <= (shift < top ? kBktMany : kBktMaxRuns) && b.blocks <= 2 * b.threads) return b;
    }
    cut(10, bucket_shift(L));
    b.table_behind = false;
    return b;
}

// Longer rows or lists (K or L > 32) of at most 2^20 points: the same with a wave per row (sample_wide_kernel), 256 source
// rows per offer block (their offers fill its LDS), 64 of up to 2^16 points, and ranges of 256 targets, of 128 for
// more than a hundred offers each, smaller ones as long as there are fewer than 512.  Offers and table lie where the
// counter scheme has its queues.  2^20 points are the most whose ranges an offer block and whose blocks a range can count
// (4096 of each, four to a thread); what more of them would give has not been measured.
// 10^6 x 96, degree 100, lists of 50, eight iterations: sampling, offers and lists 62.7 -> 19.9 ms (the queues' overflow, a
// thread per parked key and a scan of fifty keys each, was 34 of them), build 327.6 -> 284.7; 65 536 x 64, degree 40 8.46 -> 7.05,
// 10^4 x 64, degree 100 9.71 -> 8.17, 400 000 x 16, degree 128 and lists of 32 121.8 -> 115.6.
// Short samples, and few points, stay with counters and queues: where few entries are offered, a launch of offer and list blocks costs
// more than the counters' bumps.  Whole builds of clustered and even data, four iterations, time with counters over time with ranges:
// degree 40, lists of 4 0.82 to 0.86 at 600 points, 0.95 to 0.99 from 3000 on; of 6 0.89 to 0.92 at 600, 1.01 to 1.04 at 3000 to 12 000, 0.98 to 1.02
// beyond; of 8 0.94 to 0.97 at 600, 1.02 to 1.05 at 1500, up to 1.10 beyond; of 12 0.92 to 0.97 at 150, 1.04 at 600; of 20 1.0 to 1.12 at 150.  Degree 100,
// lists of 6 0.97 to 1.0.  Rows of 20, lists of 33 0.91 to 1.23 at 250, 1.07 at 600, 1.3 to 2.3 from 1500 on; rows of 32, lists of 40 1.06 at 250; rows of 10,
// lists of 64 0.91 to 1.39 at 1500, the same beyond; rows of 4, lists of 40 0.85 to 1.12, the same beyond.
inline bool wide_pays(int64_t n, int K, int L)
{
    if (K <= 32) return n >= 1000 ? 8 * K >= L : 4 * K >= 3 * L;
    return L >= 20 || (L >= 12 && n >= 500) || (L >= 8 && n >= 1000) || (L >= 6 && 10 * L >= K && n >= 3000);
}
inline size_t wide_offer_lds(int per_row, const BucketShape &b) { return ((size_t)per_row << b.row_bits) * 4 + ((size_t)2 * b.buckets + 4) * 4; }
inline bool wide_lists(int64_t n, int K, int L, BucketShape *shape = nullptr)
{
    if (bucketed_lists(n, K, L) || K > 128 || n > (1 << 20) || !wide_pays(n, K, L)) return false;
    const int per = K > L ? K : L;
    BucketShape b;
    b.row_bits = n <= (1 << 16) ? 6 : 8;
    b.blocks = (int)((n + (1 << b.row_bits) - 1) >> b.row_bits);
    b.shift = per <= 100 ? 8 : 7;
    while (b.shift < 8 && (n - 1) >> b.shift >= 4 << 10) ++b.shift;
    while (b.shift > 5 && (n - 1) >> (b.shift - 1) < 512) --b.shift;
    b.buckets = (int)((n - 1) >> b.shift) + 1;
    b.threads = b.shift == 8 ? 1024 : b.shift == 7 ? 512 : 256;
    b.table_behind = false;
    if (shape) *shape = b;
    return b.buckets <= 16 << b.row_bits && b.blocks <= 4 * b.threads && wide_offer_lds(per, b) <= 160 * 1024 - 512 &&
           (((size_t)per << b.row_bits) + b.buckets) * b.blocks * 4 <= ovf_region_for(n, K) * kOvfQueues * sizeof(Overflow);
}

// All lanes of the wave call this together; lanes with `take` set append `offer`.
template <int RB>      // RB: row bits of an offer
__device__ inline void offer_append(bool take, u32 offer, int shift, u32 *offers, int *hist, int *fill)
{
    const u64 mask = __ballot(take);
    if (mask == 0) return;
    const int leader = __ffsll((unsigned long long)mask) - 1;
    int base = 0;
    if (ef_lane() == leader) base = atomicAdd(fill, __popcll(mask));
    base = __shfl(base, leader, EF_WAVE);
    if (take) {
        offers[base + lanes_below(mask)] = offer;
        atomicAdd(&hist[offer >> (RB + shift)], 1);
    }
}

// End of an offer block: runs per bucket in `out` (this block's part of the offer array) and
// the block's row of the table.  hist, cursor: [n_buckets] in LDS; n_buckets is at most PER times the threads.
template <int RB, int PER>
__device__ inline void offers_flush(const u32 *offers, const int *hist, int *cursor, int n_buckets, int shift,
                                    int total, u32 *__restrict__ out, u32 *__restrict__ table)
{
    __shared__ int wave_tot[kBktThreads / EF_WAVE];
    const int t = threadIdx.x, b0 = PER * t;
    int c[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        c[k] = b0 + k < n_buckets ? hist[b0 + k] : 0;
        sum += c[k];
    }
    const int incl = ef_wave_scan_i32(sum);
    if (ef_lane() == EF_WAVE - 1) wave_tot[t / EF_WAVE] = incl;
    __syncthreads();
    int off = incl - sum;
    for (int v = 0; v < t / EF_WAVE; ++v) off += wave_tot[v];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (b0 + k < n_buckets) {
            cursor[b0 + k] = off;
            table[(size_t)blockIdx.x * n_buckets + b0 + k] = (u32)off << 16 | (u32)c[k];
        }
        off += c[k];
    }
    __syncthreads();
    for (int e = t; e < total; e += blockDim.x) {
        const u32 o = offers[e];
        out[atomicAdd(&cursor[o >> (RB + shift)], 1)] = o;
    }
}

// Alg. 4 step 1+2 for short rows: sample_row for 1 << RB rows, the reverse-new offers to the
// block's runs.  LDS: offers [L << RB] words, hist and cursor [n_buckets] int each.
// E: entries per lane of a row's eight lanes (8 E >= K).
template <int E, int RB>
__global__ void __launch_bounds__(1 << RB)
sample_bucket_kernel(u64 *graph, int n, int K, int L, int *__restrict__ nw, int *__restrict__ od,
                     int *__restrict__ nw_c, int *__restrict__ od_c, u32 *worst, int n_buckets, int shift,
                     u32 *__restrict__ offer_runs, u32 *__restrict__ table)
{
    extern __shared__ __align__(16) u32 offer_sm[];
    u32 *offers = offer_sm;
    constexpr int kRows = 1 << RB, kThreads = 1 << RB;
    int *hist = (int *)(offers + (size_t)kRows * L), *cursor = hist + n_buckets;
    __shared__ int fill;
    for (int b = threadIdx.x; b < n_buckets; b += kThreads) hist[b] = 0;
    if (threadIdx.x == 0) fill = 0;
    __syncthreads();
    // (loading the entries of several of a thread's rows ahead of time gains nothing measurable,
    // and beyond 64 registers the second block of a CU is lost)
    // eight lanes with two entries each per row: a wave ranks eight rows with the broadcasts that
    // four rows of sixteen lanes would take (147 -> 93 us on the headline; four or two lanes
    // per row: the same again)
    constexpr int G = 8, kRowsPerPass = kThreads / G;
    for (int pass = 0; pass < kRows / kRowsPerPass; ++pass) {
        const int i = blockIdx.x * kRows + pass * kRowsPerPass + (int)(threadIdx.x / G);
        u64 e[E];
        sample_load<G, E>(graph, i, i < n, K, e);
        sample_row<G, E>(graph, e, i, i < n, K, L, nw, od, nw_c, od_c, worst, [&](bool take, int id) {
            // (an id outside the data, from a graph the library did not write, is not offered:
            // it would index the bucket counters out of bounds)
            offer_append<RB>(take && (unsigned)id < (unsigned)n, ((u32)id << RB) | (u32)(i & (kRows - 1)), shift, offers,
                             hist, &fill);
        });
    }
    __syncthreads();
    offers_flush<RB, 2>(offers, hist, cursor, n_buckets, shift, fill, offer_runs + (size_t)blockIdx.x * kRows * L, table);
}

// The offers of a block's 1 << RB rows to the reverse-old lists of points that join something.  Four ids per thread travel at a
// time, and then four words of the map: the two waits are what a block's time is made of.  (One id at a time:
// six launches of 10^5 points, degree 20 125 -> 104 us, the wait of 10^6 points is for lines of the map, 444 -> 436.)
template <int RB>
__device__ inline void old_offers(const int *__restrict__ od, int n, int K, const u64 *__restrict__ active, int shift, u32 *offers,
                                  int *hist, int *fill)
{
    constexpr int U = 4;
    const int n_thr = (int)blockDim.x, first = blockIdx.x << RB, ids_here = min(1 << RB, n - first) * K;
    for (int f0 = 0; f0 < ids_here; f0 += U * n_thr) {      // all threads take every round
        int id[U];
        bool take[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * n_thr + (int)threadIdx.x;
            id[u] = f < ids_here ? od[(size_t)first * K + f] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            take[u] = id[u] >= 0 && id[u] < n && ((active[id[u] / EF_WAVE] >> (id[u] % EF_WAVE)) & 1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * n_thr + (int)threadIdx.x;
            offer_append<RB>(take[u], ((u32)id[u] << RB) | (u32)(f / K), shift, offers, hist, fill);
        }
    }
}

// Reverse-old offers of 1 << RB rows (to points that join something, as in reverse_old_kernel).
// LDS: offers [K << RB] words, hist and cursor [n_buckets] int each.
template <int RB>
__global__ void __launch_bounds__(1 << RB)
reverse_old_bucket_kernel(const int *__restrict__ od, int n, int K, const u64 *__restrict__ active,
                          int n_buckets, int shift, u32 *__restrict__ offer_runs, u32 *__restrict__ table)
{
    extern __shared__ __align__(16) u32 offer_sm[];
    u32 *offers = offer_sm;
    constexpr int kRows = 1 << RB, kThreads = 1 << RB;
    int *hist = (int *)(offers + (size_t)kRows * K), *cursor = hist + n_buckets;
    __shared__ int fill;
    for (int b = threadIdx.x; b < n_buckets; b += kThreads) hist[b] = 0;
    if (threadIdx.x == 0) fill = 0;
    __syncthreads();
    old_offers<RB>(od, n, K, active, shift, offers, hist, &fill);
    __syncthreads();
    offers_flush<RB, 2>(offers, hist, cursor, n_buckets, shift, fill, offer_runs + (size_t)blockIdx.x * kRows * K, table);
}

// The two for long rows (see wide_lists): a wave per row, 4 << RB threads, E entries per lane.
template <int E, int RB>
__global__ void __launch_bounds__(4 << RB)
sample_wide_kernel(u64 *graph, int n, int K, int L, int *__restrict__ nw, int *__restrict__ od,
                   int *__restrict__ nw_c, int *__restrict__ od_c, u32 *worst, int n_buckets, int shift,
                   u32 *__restrict__ offer_runs, u32 *__restrict__ table)
{
    extern __shared__ __align__(16) u32 offer_sm[];
    u32 *offers = offer_sm;
    constexpr int kRows = 1 << RB, kThreads = 4 << RB, kWaveRows = kRows / (kThreads / EF_WAVE);
    int *hist = (int *)(offers + (size_t)kRows * L), *cursor = hist + n_buckets;
    __shared__ int fill;
    for (int b = threadIdx.x; b < n_buckets; b += kThreads) hist[b] = 0;
    if (threadIdx.x == 0) fill = 0;
    __syncthreads();
    const int i0 = blockIdx.x * kRows + (int)(threadIdx.x / EF_WAVE) * kWaveRows;
    u64 next[E];
    sample_load<EF_WAVE, E>(graph, i0, i0 < n, K, next);
    for (int p = 0; p < kWaveRows; ++p) {      // (the next row travels while this one is ranked)
        const int i = i0 + p;
        u64 e[E];
#pragma unroll
        for (int h = 0; h < E; ++h) e[h] = next[h];
        if (p + 1 < kWaveRows) sample_load<EF_WAVE, E>(graph, i + 1, i + 1 < n, K, next);
        sample_row<EF_WAVE, E>(graph, e, i, i < n, K, L, nw, od, nw_c, od_c, worst, [&](bool take, int id) {
            offer_append<RB>(take && (unsigned)id < (unsigned)n, ((u32)id << RB) | (u32)(i & (kRows - 1)), shift, offers,
                             hist, &fill);
        });
    }
    __syncthreads();
    offers_flush<RB, 4>(offers, hist, cursor, n_buckets, shift, fill, offer_runs + (size_t)blockIdx.x * kRows * L, table);
}

template <int RB>
__global__ void __launch_bounds__(4 << RB)
reverse_old_wide_kernel(const int *__restrict__ od, int n, int K, const u64 *__restrict__ active,
                        int n_buckets, int shift, u32 *__restrict__ offer_runs, u32 *__restrict__ table)
{
    extern __shared__ __align__(16) u32 offer_sm[];
    u32 *offers = offer_sm;
    constexpr int kRows = 1 << RB, kThreads = 4 << RB;
    int *hist = (int *)(offers + (size_t)kRows * K), *cursor = hist + n_buckets;
    __shared__ int fill;
    for (int b = threadIdx.x; b < n_buckets; b += kThreads) hist[b] = 0;
    if (threadIdx.x == 0) fill = 0;
    __syncthreads();
    old_offers<RB>(od, n, K, active, shift, offers, hist, &fill);
    __syncthreads();
    offers_flush<RB, 4>(offers, hist, cursor, n_buckets, shift, fill, offer_runs + (size_t)blockIdx.x * kRows * K, table);
}

// The lists of one bucket.  run_cap: offers per part of an offer block (its rows * L or * K).
// Offers are sorted by target in LDS (histogram, prefix sum, scatter); a list that was offered no more than L
// sources is written as it is, without a hash, and the others choose their L smallest keys: up to 32 offers
// sixteen lanes rank them by row rotations of the hashes, up to 512 a wave finds a bound that L hashes lie below
// bit by bit from ballots, and of more only those below a bound that some L + 6 sqrt(L) hashes lie below
// are sorted at all (all threads of the block look at the popular points' offers).
// Where the offers do not fit the threads' registers they are read twice, and where what is to be sorted cannot be sure to
// fit the LDS, keys enter lists there by the bounded insertion, as many targets at a time as there is room for: ranges of
// popular points side by side, data sorted by norm among them.  (Insertion alone with a scan per offer, before the offers were sorted /
// offers counted first, walked by eight lanes a run, and every key's scan by its own lane / now: 100 000 x 64 sorted by norm, degree 20, four iterations
// 6.33, 9.59 and 5.34 ms; 200 000 x 8, low ids named more often, degree 10, two 4.29, 6.00 and 3.54.  Not made up for: 500 000 x 16 sorted by
// norm, degree 10, 3.91 and 4.2 ms, where two dozen ranges of up to twice what fits make a launch 80 to 150 us instead of 50 to 75, ten of them
// the descriptors and barriers of any launch; room for all lists at once, what is left for the second go moved to the front of its run,
// a scan by every lane for its own offer, and ranges dealt to the chiplets in turn made no difference.)
// What bounds it: instruction issue in the first iterations (10^6 points of degree 10: 3900 -> 3100 wave instructions per
// wave of a launch, half of them choosing), a fixed 25 us of run descriptors and barriers in the last.  All
// sixteen launches of that build 1338 -> 1035 us, with the bounded insertion for all (a list scanned in LDS per offer, again
// whenever another thread was first) before; degree 20, 10^5 points 793 -> 239, where popular points' insertions waited for each other.
// LDS: area words, run_at [n_blocks + 1] (later offs [targets]), hist [targets], order and bound [targets] of 16 bits;
// n_blocks <= twice the threads (four times if WIDE), at least one thread per target.
__host__ __device__ inline size_t bucket_lists_rest(int shift, int n_blocks)
{
    const size_t targets = (size_t)1 << shift, runs = (size_t)n_blocks + 1, most = runs > targets ? runs : targets;
    return most * 4 + targets * 4 + targets * 2 * 2;
}

// Words of a list block for the offers of a bucket: what its threads can hold while they are sorted, 1.6 times what
// there are on average if all rows are full, as far as the LDS goes.
inline int bucket_lists_area(int K, int L, int shift, int n_blocks, int threads, int thread_words)
{
    const size_t most = (160 * 1024 - 512 - bucket_lists_rest(shift, n_blocks)) / 4, avg = (size_t)(K > L ? K : L) << shift;
    size_t words = (size_t)thread_words * threads;
    if (words < avg * 8 / 5) words = avg * 8 / 5;
    return (int)((words < most ? words : most) & ~(size_t)3);
}

// least LDS of a list block: the insertion's lists (what bucketed_lists asks for)
__host__ __device__ inline size_t bucket_lists_lds(int L, int shift, int n_blocks)
{
    return ((size_t)L << shift) * 8 + ((size_t)2 * n_blocks + 2) * 4;
}

// The bucket of a list block: workgroups go to the eight chiplets in turn, and neighbouring buckets, whose runs lie side by
// side in every offer block's part of the array and share its lines, as the words of the table do, go to the same one's L2.
__device__ inline int bucket_of_block()
{
    const int n = (int)gridDim.x, part = blockIdx.x % 8;
    return part * (n / 8) + min(part, n % 8) + (int)(blockIdx.x / 8);
}

struct OfferRun {
    int start, count;      // in its offer block's part of the array
    int place;             // among the bucket's offers
};

// The offers of a bucket by their runs, lanes_bits: log2 of the lanes that walk a run together; run(r): an OfferRun.
// found(run, place, offer word) for every offer.
// U: runs in flight per group of lanes, A: words of what is left of a run in flight per lane.
template <int U, int A, class Run, class Found>
__device__ inline void walk_offers(const u32 *__restrict__ offer_runs, int n_blocks, int run_cap, int lanes_bits, int n_thr,
                                   Run &&run, Found &&found)
{
    const int g = 1 << lanes_bits, gl = threadIdx.x & (g - 1), groups = n_thr >> lanes_bits;
    for (int r0 = threadIdx.x >> lanes_bits; r0 < n_blocks; r0 += U * groups) {
        u32 o[U];
        OfferRun a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * groups;
            a[u] = run(min(r, n_blocks - 1));
            if (r >= n_blocks) a[u].count = 0;
            if (gl < a[u].count) o[u] = offer_runs[(size_t)r * run_cap + a[u].start + gl];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * groups;
            if (gl < a[u].count) found(r, a[u].place + gl, o[u]);
            for (int q0 = gl + g; q0 < a[u].count; q0 += A * g) {
                u32 more[A];
#pragma unroll
                for (int k = 0; k < A; ++k)
                    if (q0 + k * g < a[u].count) more[k] = offer_runs[(size_t)r * run_cap + a[u].start + q0 + k * g];
#pragma unroll
                for (int k = 0; k < A; ++k)
                    if (q0 + k * g < a[u].count) found(r, a[u].place + q0 + k * g, more[k]);
            }
        }
    }
}

// hash of a key (its high half; the low half is the source)
__device__ inline u32 reverse_hash(u64 stream_key, int target, u32 source)
{
    return (u32)(reverse_key(stream_key, target, (int)source) >> 32);
}

// Row rotation T of the sixteen lanes of a group: how many of the rotated hashes are below the own ones.
template <int T, int E>
__device__ inline void rank_round(const u32 (&h)[E], int (&rank)[E])
{
#pragma unroll
    for (int p = 0; p < E; ++p) {
        const u32 o = T ? (u32)EF_ROW_ROR((int)h[p], T ? T : 1) : h[p];
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (T || p != e) rank[e] += o < h[e] ? 1 : 0;
    }
}

// Lists that were offered more than L, but at most 16 E sources: sixteen lanes to a list.
template <int E>
__device__ inline void select_by_group(const u32 *sorted, const int *end, const int *begin, const unsigned short *order,
                                       int n_sel, int first, int L, u64 stream_key, int n_waves, u32 *__restrict__ lists)
{
    const int lane = ef_lane(), gl = lane & 15, shift = lane & 48, wave = threadIdx.x / EF_WAVE;
    for (int q0 = 4 * wave; q0 < n_sel; q0 += 4 * n_waves) {
        const int q = q0 + (lane >> 4);
        const bool ok = q < n_sel;
        const int row = order[ok ? q : n_sel - 1], s0 = begin[row], c = end[row] - s0;
        u32 src[E], h[E];
        int rank[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = gl + 16 * e;
            src[e] = sorted[s0 + min(j, c - 1)];
            h[e] = j < c ? reverse_hash(stream_key, first + row, src[e]) : ~0u;
            rank[e] = 0;
        }
#define EF_RANK(T) rank_round<T>(h, rank);
        EF_RANK(0) EF_RANK(1) EF_RANK(2) EF_RANK(3) EF_RANK(4) EF_RANK(5) EF_RANK(6) EF_RANK(7)
        EF_RANK(8) EF_RANK(9) EF_RANK(10) EF_RANK(11) EF_RANK(12) EF_RANK(13) EF_RANK(14) EF_RANK(15)
#undef EF_RANK
        int place[E], taken = 0;
        auto places = [&]() {
            taken = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const u32 mask = (u32)(__ballot(gl + 16 * e < c && rank[e] < L) >> shift) & 0xFFFFu;
                place[e] = (mask >> gl) & 1 ? taken + __popc(mask & ((1u << gl) - 1)) : -1;
                taken += __popc(mask);
            }
        };
        places();
        if (__ballot(taken > L)) {      // equal hashes around the L-th: the source decides
#pragma unroll
            for (int e = 0; e < E; ++e) rank[e] = 0;
#pragma unroll
            for (int p = 0; p < E; ++p)
                for (int k = 0; k < 16; ++k) {
                    const u32 oh = __shfl(h[p], k, 16), os = __shfl(src[p], k, 16);
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        rank[e] += 16 * p + k < c && (oh < h[e] || (oh == h[e] && os < src[e])) ? 1 : 0;
                }
            places();
        }
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (ok && place[e] >= 0) lists[(size_t)(first + row) * L + place[e]] = src[e];
    }
}

constexpr int kSelect = 8 * EF_WAVE;      // offers to one target that a wave chooses among, at most
constexpr int kRoom = 2 * EF_WAVE;        // room for the offers to a popular point that are left below its bound

// Lists that were offered more than that many: a wave to a list, c offers to `target` in its registers.
template <int N>
__device__ inline void select_by_wave(const u32 *from, int c, int target, int L, u64 stream_key, u32 *__restrict__ out)
{
    const int lane = ef_lane();
    u32 src[N], h[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const int j = lane + EF_WAVE * e;
        src[e] = from[min(j, c - 1)];
        h[e] = reverse_hash(stream_key, target, src[e]);
    }
    auto count = [&](auto &&f) {
        int n = 0;
#pragma unroll
        for (int e = 0; e < N; ++e) n += __popcll(__ballot(lane + EF_WAVE * e < c && f(h[e], src[e])));
        return n;
    };
    // a bound that L hashes lie below: bit by bit, mostly found after some log2(c) + 3 of them
    u32 t = 0, s_max = 0;
    for (u32 bit = 1u << 31; bit; bit >>= 1) {
        const int below = count([&](u32 hash, u32) { return hash < (t | bit); });
        if (below > L) continue;
        t |= bit;
        if (below == L) break;
    }
    const int below = count([&](u32 hash, u32) { return hash < t; });
    if (below < L)      // t is the L-th smallest hash and not the only one of its value: the smallest sources with it
        for (u32 bit = 1u << 31; bit; bit >>= 1)
            if (count([&](u32 hash, u32 s) { return hash == t && s < (s_max | bit); }) <= L - below) s_max |= bit;
    int place = 0;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const bool take = lane + EF_WAVE * e < c && (h[e] < t || (h[e] == t && src[e] < s_max));
        const u64 mask = __ballot(take);
        if (take) out[place + lanes_below(mask)] = src[e];
        place += __popcll(mask);
    }
}

// LT: the list length, if fixed at compile time (else 0); RB: row bits of an offer; shift: log2 of the bucket's targets.
// WIDE: for long rows and lists, one block per CU instead of two: twice the offers and offer blocks per thread.
template <int LT, int RB, bool WIDE>
__global__ void __launch_bounds__(kBktThreads) __attribute__((amdgpu_waves_per_eu(WIDE ? 4 : 8)))
bucket_lists_kernel(const u32 *__restrict__ offer_runs, const u32 *__restrict__ table, int n_blocks,
                    int run_cap, u64 stream_key, int n, int L_, int shift, int area, int g_bits, u32 *__restrict__ lists,
                    int *__restrict__ counts, const int *__restrict__ nw_c, u32 *__restrict__ active, int *work_count)
{
    const int L = LT ? LT : L_;
    constexpr int kWords = WIDE ? 2 * kBktWords : kBktWords, PER = WIDE ? 4 : 2;
    extern __shared__ __align__(16) u64 list_sm[];
    const int targets = 1 << shift, n_thr = (int)blockDim.x;
    const int most = max(n_blocks + 1, targets);
    u32 *words = (u32 *)list_sm;
    u32 *run_at = words + area;      // start << 16 | place among the bucket's offers
    int *offs = (int *)run_at, *hist = offs + most;
    unsigned short *order = (unsigned short *)(hist + targets), *bound = order + targets;
    __shared__ int total_sm, any_many, again;
    __shared__ int wave_tot[kBktThreads / EF_WAVE];
    __shared__ int n_class[3];
    const int bucket = bucket_of_block(), t = threadIdx.x, first = bucket * targets, rows_here = min(targets, n - first);
    const int lane = ef_lane(), wave = t / EF_WAVE, n_waves = n_thr / EF_WAVE;
    for (int f = t; f < targets; f += n_thr) hist[f] = 0;
    if (t < 3) n_class[t] = 0;
    if (t == 0) any_many = 0;
    const u32 *runs = table + bucket;      // (of block r: r * pitch words on)
    const size_t pitch = gridDim.x;
    {
        const int k0 = PER * t;
        u32 r[PER];
        int sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            r[k] = k0 + k < n_blocks ? runs[(k0 + k) * pitch] : 0u;
            sum += (int)(r[k] & 0xFFFFu);
        }
        const int incl = ef_wave_scan_i32(sum);
        if (lane == EF_WAVE - 1) wave_tot[wave] = incl;
        __syncthreads();
        int off = incl - sum;
        for (int v = 0; v < wave; ++v) off += wave_tot[v];
        // (places of 16 bits: only where the offers fit the LDS are they looked at)
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (k0 + k < n_blocks) run_at[k0 + k] = (r[k] & 0xFFFF0000u) | (u32)(off & 0xFFFF);
            off += (int)(r[k] & 0xFFFFu);
        }
        if (t == n_thr - 1) {      // everything before it, and its own
            total_sm = off;
            run_at[n_blocks] = (u32)(off & 0xFFFF);
        }
    }
    __syncthreads();
    const int total = total_sm;
    constexpr u32 kRowMask = (1u << RB) - 1;
    int c = 0;      // filled slots of target t's list
    const bool sorted_by_regs = total <= min(area, kWords * n_thr);
    const bool insert = !sorted_by_regs && total > area && targets * kRoom > area;      // what is to be sorted might not fit
    const int many_bits = total >= 40 * n_blocks ? 6 : g_bits;      // lanes to a run where there are more than usual
    constexpr int SB = 21;      // source bits
    constexpr u32 kNone = ~0u;
    // (places have 16 bits: of more offers only the differences are good, which no run exceeds)
    auto run_of = [&](int r) {
        const u32 here = run_at[r];
        const int place = (int)(here & 0xFFFFu);
        return OfferRun{(int)(here >> 16), (int)((run_at[r + 1] - here) & 0xFFFFu), place};
    };
    auto table_run = [&](int r) { return OfferRun{(int)(runs[r * pitch] >> 16), (int)(runs[r * pitch] & 0xFFFFu), 0}; };
    auto row_of = [&](u32 o) {      // (always inside: runs are filed by bucket)
        const int row = (int)(o >> RB) - first;
        return (unsigned)row < (unsigned)rows_here ? row : -1;
    };
    auto source_of = [&](int run, u32 o) { return ((u32)run << RB) + (o & kRowMask); };
    // ---- the bucket's offers, in any order, as (target inside the bucket, source); offers per target --------------
    if (sorted_by_regs) {
        auto found = [&](int run, int at, u32 o) {
            const int row = row_of(o);
            words[at] = row >= 0 ? (u32)row << SB | source_of(run, o) : kNone;
            if (row >= 0) atomicAdd(&hist[row], 1);
        };
        if (total <= kBktFew * n_thr) {      // few offers: a thread looks for the run of its offer
            for (int j = t; j < total; j += n_thr) {
                int lo = 0, hi = n_blocks;      // place of lo <= j < place of hi
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if ((int)(run_at[mid] & 0xFFFFu) <= j) lo = mid;
                    else hi = mid;
                }
                const OfferRun r = run_of(lo);
                found(lo, j, offer_runs[(size_t)lo * run_cap + r.start + (j - r.place)]);
            }
        } else
            walk_offers<4, 1>(offer_runs, n_blocks, run_cap, g_bits, n_thr, run_of, found);
    } else if (!insert)
        walk_offers<1, 4>(offer_runs, n_blocks, run_cap, many_bits, n_thr, run_of, [&](int, int, u32 o) {
            const int row = row_of(o);
            if (row >= 0) atomicAdd(&hist[row], 1);
        });
    __syncthreads();      // (run_at is free from here on)
    // ---- sorted by target, in place: every word is in a register before the first is written -----------------------
    // (More offers than fit: the offers are walked again, and popular points get room for kRoom of them only.)
    u32 w[kWords];
    if (sorted_by_regs) {
#pragma unroll
        for (int u = 0; u < kWords; ++u)
            if (u * n_thr < total) w[u] = u * n_thr + t < total ? words[u * n_thr + t] : kNone;
    }
    const int mine = t < rows_here ? hist[t] : 0, room = sorted_by_regs ? mine : min(mine, kRoom);
    const bool many = mine > (sorted_by_regs ? kSelect : kRoom);
    const int incl = ef_wave_scan_i32(room);
    if (lane == EF_WAVE - 1) wave_tot[wave] = incl;
    // lists with more than L offers, by what it takes to choose among them
    const int cls = mine <= L ? -1 : mine <= 16 ? 0 : mine <= 32 ? 1 : 2;
    const u64 in0 = __ballot(cls == 0), in1 = __ballot(cls == 1), in2 = __ballot(cls == 2);
    int base = 0;
    if (lane < 3 && (in0 | in1 | in2)) base = atomicAdd(&n_class[lane], __popcll(lane == 0 ? in0 : lane == 1 ? in1 : in2));
    const int place = __shfl(base, max(cls, 0), EF_WAVE) + lanes_below(cls == 0 ? in0 : cls == 1 ? in1 : in2);
    // Popular points (uniformly over the block: is there one?): only those offers with a hash below what some L + 6 sqrt(L) + 12 lie below.
    float share = fminf((float)(L + 12) + 6.0f * __builtin_sqrtf((float)L), 0.875f * kRoom) / (float)max(mine, 1);
    constexpr u32 kAll = 0xFFFFu;
    if (many) any_many = 1;
    if (t < targets) bound[t] = (unsigned short)(many ? (u32)(share * 65535.0f) : kAll);
    __syncthreads();
    int begin = incl - room;
    for (int v = 0; v < wave; ++v) begin += wave_tot[v];
    const int n0 = n_class[0], n1 = n_class[1], n2 = n_class[2];
    const bool popular = any_many;
    bool settled = !insert;      // uniform over the block
    if (settled) {
        if (t < targets) offs[t] = hist[t] = begin;
        if (cls >= 0) order[(cls == 0 ? 0 : cls == 1 ? n0 : n0 + n1) + place] = (unsigned short)t;
        __syncthreads();
        if (sorted_by_regs) {
#pragma unroll
            for (int u = 0; u < kWords; ++u) {
                if (u * n_thr >= total) continue;
                const int row = (int)(w[u] >> SB) & (targets - 1);
                const u32 source = w[u] & ((1u << SB) - 1);
                bool take = w[u] != kNone;
                if (popular) {
                    const u32 most = bound[row];
                    if (__ballot(most != kAll)) take = take && (most == kAll || reverse_hash(stream_key, first + row, source) >> 16 <= most);
                }
                if (take) words[atomicAdd(&offs[row], 1)] = source;
            }
        }
        // (once, but for a popular point that was left with fewer than L or more than kRoom: again with another bound)
        for (int tries = 0;; ++tries) {
            if (popular) {
                if (t == 0) again = 0;
                __syncthreads();
            }
            if (tries > 0 || !sorted_by_regs)
                walk_offers<1, 4>(offer_runs, n_blocks, run_cap, many_bits, n_thr, table_run, [&](int run, int, u32 o) {
                    const int row = row_of(o);
                    if (row < 0) return;
                    const u32 source = source_of(run, o), most = bound[row];
                    if (tries > 0 && most == kAll) return;
                    if (most != kAll && reverse_hash(stream_key, first + row, source) >> 16 > most) return;
                    const int p = atomicAdd(&offs[row], 1);
                    if (most == kAll || p - hist[row] < kRoom) words[p] = source;
                });
            __syncthreads();      // (offs[r] is now the end of target r's sources)
            if (!popular) break;      // (uniform over the block)
            if (t < rows_here && bound[t] != kAll) {
                const int kept = offs[t] - begin;
                if (kept < L || kept > kRoom) {
                    share *= kept < L ? 2.0f : 0.75f;
                    bound[t] = (unsigned short)(fminf(share, 0.99f) * 65535.0f);
                    offs[t] = begin;
                    again = 1;
                } else
                    bound[t] = kAll;
            }
            __syncthreads();
            if (!again) break;
            if (tries == 15) {
                settled = false;
                break;
            }
            __syncthreads();
        }
    }
    if (settled) {
        // ---- the lists -----------------------------------------------------------------------------------------
        for (int q = wave; q < n2; q += n_waves) {
            const int row = __builtin_amdgcn_readfirstlane((int)order[n0 + n1 + q]);
            const int from = __builtin_amdgcn_readfirstlane(hist[row]), cnt = __builtin_amdgcn_readfirstlane(offs[row]) - from;
            u32 *out = lists + (size_t)(first + row) * L;
            if (cnt <= EF_WAVE) select_by_wave<1>(words + from, cnt, first + row, L, stream_key, out);
            else if (cnt <= 2 * EF_WAVE) select_by_wave<2>(words + from, cnt, first + row, L, stream_key, out);
            else if (cnt <= 4 * EF_WAVE) select_by_wave<4>(words + from, cnt, first + row, L, stream_key, out);
            else select_by_wave<8>(words + from, cnt, first + row, L, stream_key, out);
        }
        if (L < 32) select_by_group<2>(words, offs, hist, order + n0, n1, first, L, stream_key, n_waves, lists);
        if (L < 16) select_by_group<1>(words, offs, hist, order, n0, first, L, stream_key, n_waves, lists);
        // (places beyond a list's count are never read)
        for (int f = t; f < rows_here * L; f += n_thr) {
            const int row = LT ? f / LT : f / L, a = f - row * L, from = hist[row], cnt = offs[row] - from;
            if (cnt <= L && a < cnt) lists[(size_t)first * L + f] = words[from + a];
        }
        c = min(mine, L);
    }
    if (!settled) {
        // more offers than are sure to fit, or no bound found: bounded insertion, as many targets at a time as there is room for.
        // A wave walks a run, drops what is above the largest key that was seen in a full list (hist: its high half; keys
        // only ever fall) and puts the others by until they fill its lanes: of the offers to popular points few are
        // left, and a scan of the list costs a wave the same for one of them as for 64.
        __syncthreads();
        u64 *ll = list_sm;
        u32 *put_by = words + area - EF_WAVE * (wave + 1);
        const int step = (area - n_thr) / (2 * L);
        for (int row0 = 0; row0 < rows_here; row0 += step) {
            const int rows = min(step, rows_here - row0);
            for (int f = t; f < rows * L; f += n_thr) ll[f] = ~0ULL;
            if (t < rows) hist[t] = -1;
            __syncthreads();
            auto largest = [&](int row) { return __hip_atomic_load((u32 *)hist + row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
            int fill = 0;      // (the wave's)
            auto wave_sync = [&]() {      // one wave: its LDS operations complete in program order
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            };
            auto drain = [&]() {
                wave_sync();
                if (lane < fill) {
                    const u32 o = put_by[lane];
                    const int row = (int)(o >> SB);
                    const u64 key = reverse_key(stream_key, first + row0 + row, (int)(o & ((1u << SB) - 1)));
                    unsigned long long *list = (unsigned long long *)(ll + row * L);
                    while ((u32)(key >> 32) <= largest(row)) {
                        u64 mx = 0;
                        int ms = 0;
#pragma unroll 4
                        for (int a = 0; a < L; ++a) {
                            const u64 v = __hip_atomic_load(list + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            if (v > mx) {      // the first of equal (empty) slots: lists fill from slot 0 up
                                mx = v;
                                ms = a;
                            }
                        }
                        atomicMin((u32 *)hist + row, (u32)(mx >> 32));
                        if (key >= mx) break;
                        // slots only ever fall: if slot ms still holds mx, it still is the largest
                        if (atomicCAS(list + ms, (unsigned long long)mx, (unsigned long long)key) == mx) break;
                    }
                }
                wave_sync();
                fill = 0;
            };
            auto offer = [&](int run, u32 o) {      // all lanes of the wave together
                const int row = (int)(o >> RB) - first - row0;
                const bool take = (unsigned)row < (unsigned)rows &&
                                  reverse_hash(stream_key, first + row0 + row, source_of(run, o)) <= largest(row);
                const u64 mask = __ballot(take);
                if (!mask) return;
                if (fill + __popcll(mask) > EF_WAVE) drain();
                if (take) put_by[fill + lanes_below(mask)] = (u32)row << SB | source_of(run, o);
                fill += __popcll(mask);
            };
            constexpr int U = 8;      // runs in flight, a piece of 64 of each at a time; lane u knows the u-th
            for (int r0 = wave; r0 < n_blocks; r0 += U * n_waves) {
                const int r = r0 + (lane & (U - 1)) * n_waves, rr = min(r, n_blocks - 1);
                const OfferRun run = insert ? run_of(rr) : table_run(rr);
                const int count = r < n_blocks ? run.count : 0, from = rr * run_cap + run.start;
                for (int q0 = 0; __ballot(q0 < count); q0 += EF_WAVE) {
                    u32 o[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int c = __builtin_amdgcn_readlane(count, u), at = __builtin_amdgcn_readlane(from, u);
                        o[u] = q0 + lane < c ? offer_runs[at + q0 + lane] : ~0u;
                    }
#pragma unroll 1
                    for (int u = 0; u < U; ++u)
                        offer(r0 + u * n_waves, u == 0 ? o[0] : u == 1 ? o[1] : u == 2 ? o[2] : u == 3 ? o[3] : u == 4 ? o[4] : u == 5 ? o[5] : u == 6 ? o[6] : o[7]);
                }
            }
            drain();
            __syncthreads();
            // only the sources are wanted from here on (the keys decided who is in the list)
            for (int f = t; f < rows * L; f += n_thr) lists[(size_t)(first + row0) * L + f] = (u32)ll[f];
            if (t >= row0 && t < row0 + rows)
                for (int a = 0; a < L; ++a) c += ll[(t - row0) * L + a] != ~0ULL ? 1 : 0;
            __syncthreads();
        }
    }
    if (t < rows_here) counts[first + t] = c;
    if (!active) return;
    // The reverse-new lists are complete: who joins anything in this iteration (see active_kernel; 32 points a
    // word, so that the smallest ranges of targets own whole words), and the work lists are empty again.
    const u64 mask = __ballot(t < rows_here && (c > 0 || nw_c[first + t] > 0));
    const int t0 = t & ~(EF_WAVE - 1), half = ef_lane();
    if (half < 2 && t0 + 32 * half < rows_here) active[(first + t0) / 32 + half] = (u32)(mask >> (32 * half));
    if (blockIdx.x == 0 && t < kMaxClasses) work_count[t] = 0;
}

// The same for the shortest lists and the fewest points (insert_lists): every key goes through the bounded insertion; all slots start as the largest
// key, so a list fills from slot 0 up and then keeps its L smallest keys.  Short scans and hardly a barrier: where
// the sorting kernel takes longer (builds of 19 000 x 13, degree 7, lists of 5 / 3000 x 16, degree 3 / 300 000 x 32, degree 32, lists of 5:
// 687 and 714 us, 454 and 473, 8.27 and 8.67 ms).  Lists of 7 take 1 to 3 % less with it from 2 10^5 points on (800 000 x 128, degree 7 8.33 and 8.55 ms) and
// 1 to 6 % more below 10^5 (3000 x 128 655 and 615 us), lists of 8 up to 5 % more.  Up to 256 points of degree 10 the sort's extra barriers are
// 1.3 us of a launch of 4 to 6 (builds of 24, 100, 150 and 256 points 248 and 262 us, 310 and 319, 304 and 314, 329 and 332; of 350 points or of degree 12
// level, 100 points of degree 20, lists of 10 637 and 625).  LDS: lists [bucket's targets * L] u64, scan [n_blocks + 1] and start [n_blocks] int.
template <int LT, int RB>      // (see bucket_lists_kernel)
__global__ void __launch_bounds__(kBktThreads)
bucket_insert_kernel(const u32 *__restrict__ offer_runs, const u32 *__restrict__ table, int n_blocks,
                    int run_cap, u64 stream_key, int n, int L_, int shift, int, int, u32 *__restrict__ lists,
                    int *__restrict__ counts, const int *__restrict__ nw_c, u32 *__restrict__ active, int *work_count)
{
    const int L = LT ? LT : L_;
    extern __shared__ __align__(16) u64 list_sm[];
    u64 *ll = list_sm;
    const int targets = 1 << shift, n_thr = (int)blockDim.x;
    int *scan = (int *)(ll + (size_t)targets * L), *start = scan + n_blocks + 1;
    __shared__ int wave_tot[kBktThreads / EF_WAVE];
    const int bucket = bucket_of_block(), t = threadIdx.x, first = bucket * targets, rows_here = min(targets, n - first);
    for (int f = t; f < targets * L; f += n_thr) ll[f] = ~0ULL;
    const u32 *runs = table + bucket;      // (of block r: r * pitch words on)
    const size_t pitch = gridDim.x;
    {
        const int k0 = 2 * t;
        const u32 r0 = k0 < n_blocks ? runs[k0 * pitch] : 0u, r1 = k0 + 1 < n_blocks ? runs[(k0 + 1) * pitch] : 0u;
        const int c0 = (int)(r0 & 0xffffu), c1 = (int)(r1 & 0xffffu);
        const int incl = ef_wave_scan_i32(c0 + c1);
        if (ef_lane() == EF_WAVE - 1) wave_tot[t / EF_WAVE] = incl;
        __syncthreads();
        int off = incl - (c0 + c1);
        for (int v = 0; v < t / EF_WAVE; ++v) off += wave_tot[v];
        if (k0 < n_blocks) {
            scan[k0] = off;
            start[k0] = (int)(r0 >> 16);
        }
        if (k0 + 1 < n_blocks) {
            scan[k0 + 1] = off + c0;
            start[k0 + 1] = (int)(r1 >> 16);
        }
        if (t == n_thr - 1) scan[n_blocks] = off + c0 + c1;      // everything before it, and its own
    }
    __syncthreads();
    const int total = scan[n_blocks];
    for (int j = t; j < total; j += n_thr) {      // neighbouring threads take neighbouring offers
        int lo = 0, hi = n_blocks;      // scan[lo] <= j < scan[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (scan[mid] <= j) lo = mid;
            else hi = mid;
        }
        const u32 o = offer_runs[(size_t)lo * run_cap + start[lo] + (j - scan[lo])];
        const int target = (int)(o >> RB), source = (lo << RB) + (int)(o & ((1u << RB) - 1));
        const int row = target - first;
        if ((unsigned)row >= (unsigned)rows_here) continue;      // cannot happen: runs are filed by bucket
        const u64 key = reverse_key(stream_key, target, source);
        unsigned long long *list = (unsigned long long *)(ll + row * L);
        for (;;) {
            u64 mx = 0;
            int ms = 0;
            for (int a = 0; a < L; ++a) {
                const u64 v = __hip_atomic_load(list + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (v > mx) {      // the first of equal (empty) slots: lists fill from slot 0 up
                    mx = v;
                    ms = a;
                }
            }
            if (key >= mx) break;
            // slots only ever fall: if slot ms still holds mx, it still is the largest
            if (atomicCAS(list + ms, (unsigned long long)mx, (unsigned long long)key) == mx) break;
        }
    }
    __syncthreads();
    // only the sources are wanted from here on (the keys decided who is in the list)
    for (int f = t; f < rows_here * L; f += n_thr) lists[(size_t)first * L + f] = (u32)ll[f];
    int c = 0;
    if (t < rows_here) {
        for (int a = 0; a < L; ++a) c += ll[t * L + a] != ~0ULL ? 1 : 0;
        counts[first + t] = c;
    }
    if (!active) return;
    // The reverse-new lists are complete: who joins anything in this iteration (see active_kernel; 32 points a
    // word, so that the smallest ranges of targets own whole words), and the work lists are empty again.
    const u64 mask = __ballot(t < rows_here && (c > 0 || nw_c[first + t] > 0));
    const int t0 = t & ~(EF_WAVE - 1), half = ef_lane();
    if (half < 2 && t0 + 32 * half < rows_here) active[(first + t0) / 32 + half] = (u32)(mask >> (32 * half));
    if (blockIdx.x == 0 && t < kMaxClasses) work_count[t] = 0;
}

// Work lists by the number of vectors a join gathers: list c takes the joins of at most
// bound[c] vectors that no earlier list takes (bounds ascending; a bound of 0: no such list).
// Lists 0 and 1 are the register-operand joins (16 and 32 vectors), the others the size classes
// of the LDS-row join: a launch per class with a row buffer of that size, so that small joins
// do not occupy the LDS of the largest one and several blocks fit a CU.
struct JoinClasses {
    int n;
    int bound[kMaxClasses];
};

// the size classes for joins of up to max_rows vectors; reg_ok: lists 0 and 1 are in use
inline JoinClasses join_classes(int max_rows, bool reg_ok)
{
    JoinClasses jc;
    jc.n = 2;
    jc.bound[0] = reg_ok ? 16 : 0;
    jc.bound[1] = reg_ok ? 32 : 0;
    for (int c : {48, 64, 96, 128, 160})
        if (c < max_rows && c > jc.bound[1]) jc.bound[jc.n++] = c;
    jc.bound[jc.n++] = max_rows;
    for (int c = jc.n; c < kMaxClasses; ++c) jc.bound[c] = 0;
    return jc;
}

// End of the kernels below: every thread of the block holds a point (i; class cls, -1 = no join; its pairs and
// vectors) and files it.
__device__ inline void append_points(int cls, int i, int n, int evals, int rows, const JoinClasses &jc,
                                     int *__restrict__ work, int *__restrict__ work_count,
                                     long long *__restrict__ part)
{
    // append to the work lists: ranks inside the block first, then one counter bump per
    // list and block (bumps of one address serialise at about 11 ns each)
    __shared__ int wave_cnt[kMaxClasses][16], block_base[kMaxClasses];
    __shared__ int wave_sum[3][16];
    const int lane = ef_lane(), wave = threadIdx.x / EF_WAVE, n_waves = blockDim.x / EF_WAVE;
    int rank = 0;
    for (int c = 0; c < jc.n; ++c) {
        const u64 mask = __ballot(cls == c);
        if (cls == c) rank = __popcll(mask & ((1ULL << lane) - 1));
        if (lane == 0) wave_cnt[c][wave] = __popcll(mask);
    }
    // the block's share of the counters: pairs evaluated, vectors gathered, vectors gathered by
    // joins of at most rows0 vectors (a block's totals fit 32 bits)
    const int s_ev = ef_wave_sum_i32(evals), s_rw = ef_wave_sum_i32(rows),
              s_r0 = ef_wave_sum_i32(cls == 0 ? rows : 0);
    if (lane == 0) {
        wave_sum[0][wave] = s_ev;
        wave_sum[1][wave] = s_rw;
        wave_sum[2][wave] = s_r0;
    }
    __syncthreads();
    if ((int)threadIdx.x < jc.n) {
        int tot = 0;
        for (int v = 0; v < n_waves; ++v) tot += wave_cnt[threadIdx.x][v];
        block_base[threadIdx.x] = tot ? atomicAdd(&work_count[threadIdx.x], tot) : 0;
    }
    if (threadIdx.x < 3) {
        long long sum = 0;
        for (int v = 0; v < n_waves; ++v) sum += wave_sum[threadIdx.x][v];
        part[(size_t)blockIdx.x * 3 + threadIdx.x] = sum;
    }
    __syncthreads();
    if (cls >= 0) {
        int off = block_base[cls] + rank;
        for (int v = 0; v < wave; ++v) off += wave_cnt[cls][v];
        work[(size_t)cls * n + off] = i;
    }
}

// After sampling and the reverse lists: one thread per point merges its four id lists
// into U_new ++ U_old (Alg. 4: G_new U G_rnew, G_old U G_rold), without duplicates and
// with everything already in U_new left out of U_old, and files the point under one of
// the work lists by the number of vectors its join gathers.
// Points with an empty U_new are dropped.  A thread compares only what can collide:
// ids inside one sampled list are distinct, and so are the sources inside one reverse
// list.  ulist: [n][cap] (written through LDS so that the stores coalesce), ucount: [n]
// (m_new, m); work: [jc.n][n], work_count: [kMaxClasses].
template <class Source>      // of a reverse list's entries: 32 bits, or the key's low half
__global__ void prepare_kernel(const int *__restrict__ nw, const int *__restrict__ od,
                               const int *__restrict__ nw_c, const int *__restrict__ od_c,
                               const Source *__restrict__ rnew, const Source *__restrict__ rold,
                               const int *__restrict__ rnew_c, const int *__restrict__ rold_c,
                               int n, int K, int L, int cap, u32 cap_magic, JoinClasses jc,
                               int *__restrict__ ulist, int2 *__restrict__ ucount,
                               int *__restrict__ work, int *__restrict__ work_count,
                               long long *__restrict__ part)
{
    extern __shared__ int ids_sh[];
    const int pitch = cap | 1;                      // odd: threads hit different banks
    int *mine = ids_sh + threadIdx.x * pitch;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    int cls = -1, m = 0;
    int evals = 0, rows = 0;      // this point's share of the iteration's work counters
    if (i < n) {
        const int c_new = nw_c[i];
        int c_old = od_c[i];
        const int rn = min(rnew_c[i], L), ro = min(rold_c[i], L);
        if (c_new + rn == 0) c_old = 0;      // empty U_new: no join, nothing to list
        for (int a = 0; a < c_new; ++a) mine[m++] = nw[(size_t)i * L + a];
        for (int a = 0; a < rn; ++a) {
            const int id = (int)(u32)rnew[(size_t)i * L + a];
            bool dup = false;
            for (int k = 0; k < c_new; ++k) dup |= mine[k] == id;
            if (!dup) mine[m++] = id;
        }
        const int m_new = m;
        for (int a = 0; a < c_old; ++a) {
            const int id = od[(size_t)i * K + a];
            bool dup = false;
            for (int k = c_new; k < m_new; ++k) dup |= mine[k] == id;      // only reverse-new can collide
            if (!dup) mine[m++] = id;
        }
        const int m_mid = m;
        for (int a = 0; a < ro; ++a) {
            const int id = (int)(u32)rold[(size_t)i * L + a];
            bool dup = false;
            for (int k = 0; k < m_mid; ++k) dup |= mine[k] == id;
            if (!dup) mine[m++] = id;
        }
        ucount[i] = make_int2(m_new, m);
        if (m_new >= 1 && m >= 2) {
            cls = 0;
            while (cls < jc.n - 1 && m > jc.bound[cls]) ++cls;
            evals = m_new * (m_new - 1) / 2 + m_new * (m - m_new);
            rows = m;
        }
    }
    for (int k = m; k < cap; ++k) mine[k] = -1;
    __syncthreads();
    // coalesced write-out of the block's lists
    const int first = blockIdx.x * blockDim.x, rows_here = min((int)blockDim.x, n - first);
    for (int f = threadIdx.x; f < rows_here * cap; f += blockDim.x) {
        const int r = (int)(((u64)(u32)f * cap_magic) >> 32), c = f - r * cap;
        ulist[(size_t)first * cap + f] = ids_sh[r * pitch + c];
    }
    append_points(cls, i, n, evals, rows, jc, work, work_count, part);
}

// The same for short lists (the bucket scheme: K, L <= 32, 32-bit sources), eight lanes per point, E ids
// of every list per lane (8 E >= K, L): all four lists travel together, where a thread that walks
// them alone waits for one id after the other; duplicates are found against the ids already in
// LDS, places come from ballots.  64 points per pass, `passes` (at most 4) per block of 512 threads: a
// block bumps the work lists' counters once (11 ns each, one after the other).  Per launch, before and after: 10^4 points of
// degree 10 23.5 -> 9.3 us, 10^5 of degree 20 50 -> 31, 10^6 of degree 10 108 -> 104.
constexpr int kPrepPoints = 64, kPrepThreads = 8 * kPrepPoints, kPrepMaxPasses = 4;
// LDS for the ids in the kernels that write the join lists: with the arrays they declare (at most 2.8 KB) it
// stays within the 64 KB that a launch gets without asking for more.
constexpr size_t kPrepLds = 64 * 1024 - 4096;
template <int E>
__global__ void __launch_bounds__(kPrepThreads)
prepare_group_kernel(const int *__restrict__ nw, const int *__restrict__ od,
                     const int *__restrict__ nw_c, const int *__restrict__ od_c,
                     const u32 *__restrict__ rnew, const u32 *__restrict__ rold,
                     const int *__restrict__ rnew_c, const int *__restrict__ rold_c,
                     int n, int K, int L, int cap, u32 cap_magic, JoinClasses jc, int passes,
                     int *__restrict__ ulist, int2 *__restrict__ ucount,
                     int *__restrict__ work, int *__restrict__ work_count,
                     long long *__restrict__ part)
{
    extern __shared__ int ids_sh[];
    const int pitch = cap | 1;                      // odd: points hit different banks
    __shared__ int2 sizes[kPrepPoints * kPrepMaxPasses];      // (m_new, m) of every point
    const int tid = threadIdx.x, gl = tid & 7, grp_shift = ef_lane() & 56;
    const int first = blockIdx.x * kPrepPoints * passes;
    auto wave_sync = [&]() {      // one wave: its LDS operations complete in program order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int pass = 0; pass < passes; ++pass) {
        const int p = pass * kPrepPoints + (tid >> 3), i = first + p;
        const bool ok = i < n;
        const size_t row_l = (size_t)(ok ? i : 0) * L, row_k = (size_t)(ok ? i : 0) * K;
        int *mine = ids_sh + p * pitch;
        int c_new = ok ? nw_c[i] : 0, c_old = ok ? od_c[i] : 0, rn = ok ? min(rnew_c[i], L) : 0, ro = ok ? min(rold_c[i], L) : 0;
        int a_new[E], a_rn[E], a_old[E], a_ro[E];
#pragma unroll
        for (int h = 0; h < E; ++h) {      // (entries beyond a list's count are read along)
            const int al = min(gl + 8 * h, L - 1), ak = min(gl + 8 * h, K - 1);
            a_new[h] = nw[row_l + al];
            a_rn[h] = (int)rnew[row_l + al];
            a_old[h] = od[row_k + ak];
            a_ro[h] = (int)rold[row_l + al];
        }
        if (c_new + rn == 0) c_old = ro = 0;      // empty U_new: no join, nothing to list
        // entries [0, cnt) of a list join `mine` behind the m there are, but for those among mine[from .. to)
        int m = 0;
        auto merge = [&](const int (&a)[E], int cnt, int from, int to) {
#pragma unroll
            for (int h = 0; h < E; ++h) {
                bool fresh = gl + 8 * h < cnt;
                if (fresh)
                    for (int k = from; k < to; ++k) fresh &= mine[k] != a[h];
                const int mask = (int)((__ballot(fresh) >> grp_shift) & 0xFF);
                if (fresh) mine[m + __popc(mask & ((1 << gl) - 1))] = a[h];
                m += __popc(mask);
            }
            wave_sync();
        };
        merge(a_new, c_new, 0, 0);
        merge(a_rn, rn, 0, c_new);
        const int m_new = m;
        merge(a_old, c_old, c_new, m_new);      // only reverse-new can collide
        merge(a_ro, ro, 0, m);
        for (int k = m + gl; k < cap; k += 8) mine[k] = -1;
        if (gl == 0) {
            sizes[p] = make_int2(m_new, m);
            if (ok) ucount[i] = make_int2(m_new, m);
        }
    }
    __syncthreads();
    // coalesced write-out of the block's lists
    const int here = min(kPrepPoints * passes, n - first);
    for (int f = tid; f < here * cap; f += kPrepThreads) {
        const int r = (int)(((u64)(u32)f * cap_magic) >> 32), c = f - r * cap;
        ulist[(size_t)first * cap + f] = ids_sh[r * pitch + c];
    }
    int cls = -1, evals = 0, rows = 0;
    if (tid < here) {
        const int m_new = sizes[tid].x, m = sizes[tid].y;
        if (m_new >= 1 && m >= 2) {
            cls = 0;
            while (cls < jc.n - 1 && m > jc.bound[cls]) ++cls;
            evals = m_new * (m_new - 1) / 2 + m_new * (m - m_new);
            rows = m;
        }
    }
    append_points(cls, first + tid, n, evals, rows, jc, work, work_count, part);
}

// ---------------------------------------------------------------------------------------
// Alg. 4 step 3+4: local joins.
//
// Each block walks a work list (grid-strided), one point at a time:
//   0. candidates: the four id lists are merged and de-duplicated through a small LDS
//      hash table into U_new ++ U_old;
//   1. gather: their rows, thresholds and squared norms go to LDS;
//   2. filter: 16x16 blocks of the Gram matrix U_new x U are formed with fp32 MFMA
//      (v_mfma_f32_16x16x4f32); a pair survives if |a|^2 + |b|^2 - 2ab, lowered by a
//      bound on the rounding error of that expression, is not above the larger of
//      the two rows' thresholds.  The bound is conservative, so no pair that the exact
//      test would accept is dropped; most pairs are, at a quarter of the VALU cost;
//   3. survivors get the library's fixed-order distance (one 16-lane group per pair),
//      the exact threshold test, and go to the proposal queue;
//   4. the queue is drained into the graph rows with the lock-free insertion.
// cap_rows: how many vectors the LDS row buffer of this launch holds.

struct JoinLds {
    float *rows;      // [cap_rows][stride], columns d..dpad-1 zero
    int *uid;         // [cap_rows] U_new ++ U_old
    u32 *thr;         // [cap_rows] threshold bits
    float *nrm;       // [cap_rows] squared norms (float32, any order: filter only)
    int *meta;        // [2] updates [3] queue count [4] survivor count
    u32 *surv;        // [s_cap] a | b << 16
    u32 *known;       // [cap_rows][known_words(cap_rows)] bit c of row r: uid[c] is (or was) in the graph row of uid[r]
    int *hkey, *hidx; // [known_slots(cap_rows)] each: open-addressing table id -> place in uid
    Proposal *queue;  // [q_cap]
};

// words per row of the `known` bit table, slots of the id table (a power of two, at most half full)
__host__ __device__ inline int known_words(int cap_rows) { return (cap_rows + 31) >> 5; }
__host__ __device__ inline int known_slots(int cap_rows)
{
    int s = 64;
    while (s < 2 * cap_rows) s <<= 1;
    return s;
}

__host__ __device__ inline size_t join_lds_floats(int cap_rows, int stride, int s_cap)
{
    return (size_t)align4(cap_rows * stride) + align4(3 * cap_rows) + 8 + align4(s_cap) +
           align4(cap_rows * known_words(cap_rows)) + 2 * known_slots(cap_rows);
}

__device__ inline JoinLds join_lds_carve(float *smem, int cap_rows, int stride, int s_cap)
{
    JoinLds l;
    l.rows = smem;
    l.uid = (int *)(smem + align4(cap_rows * stride));
    l.thr = (u32 *)(l.uid + cap_rows);
    l.nrm = (float *)(l.thr + cap_rows);
    l.meta = l.uid + align4(3 * cap_rows);
    l.surv = (u32 *)(l.meta + 8);
    l.known = l.surv + align4(s_cap);
    l.hkey = (int *)(l.known + align4(cap_rows * known_words(cap_rows)));
    l.hidx = l.hkey + known_slots(cap_rows);
    l.queue = (Proposal *)(l.hidx + known_slots(cap_rows));
    return l;
}

template <bool WIDE>      // WIDE: graph rows of fifty entries or more, sixteen threads per proposal
__global__ void __launch_bounds__(512) join_kernel(const float *__restrict__ X, const float *__restrict__ norms, int d,
                            int dpad, int stride, u32 q4_magic, int K, u32 k_magic,
                            const int *__restrict__ work, const int *__restrict__ work_count,
                            int cap_rows, int s_cap, int q_cap, float margin_rel, float thr_scale,
                            const int *__restrict__ ulist, const int2 *__restrict__ ucount,
                            int ucap, u64 *graph, u32 *worst, int *__restrict__ upd_block, int mode)
{
    extern __shared__ __align__(16) float smem[];
    const JoinLds lds = join_lds_carve(smem, cap_rows, stride, s_cap);
    const int mark = mode != 2;      // (modes: see join_reg_kernel)
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & (EF_WAVE - 1), wave = tid / EF_WAVE, n_waves = nthr / EF_WAVE;
    const int grp = tid >> 4, gl = tid & 15, n_grp = nthr >> 4;
    const int count = *work_count;
    const int kw = known_words(cap_rows), hslots = known_slots(cap_rows), hshift = 32 - (31 - __clz(hslots));
    int block_updates = 0;      // thread 0: insertions made by this block
    for (int w = blockIdx.x; w < count; w += gridDim.x) {
        const int i = work[w];
        // ---- 0. the point's U_new ++ U_old ------------------------------------------------
        const int2 mc = ucount[i];
        const int m_new = mc.x, m = mc.y;
        for (int r = tid; r < m; r += nthr) lds.uid[r] = ulist[(size_t)i * ucap + r];
        if (tid < 8) lds.meta[tid] = 0;
        for (int f = tid; f < m * kw; f += nthr) lds.known[f] = 0u;
        for (int f = tid; f < hslots; f += nthr) lds.hkey[f] = -1;
        __syncthreads();
        // ---- 1. gather -------------------------------------------------------------------
        for (int r = tid; r < m; r += nthr) {
            const int id = lds.uid[r];
            lds.thr[r] = ef_load_coherent(worst + id);
            lds.nrm[r] = norms[id];
            // the members' places by id (ids of a list are distinct: every one finds a free slot)
            int h = (int)(((u32)id * 0x9E3779B1u) >> hshift);
            while (atomicCAS(&lds.hkey[h], -1, id) != -1) h = (h + 1) & (hslots - 1);
            lds.hidx[h] = r;
        }
        gather_rows(X, d, stride, q4_magic, lds.uid, m, lds.rows, tid, nthr);
        __syncthreads();      // the id table is complete
        // Which members already know which: the graph rows of all members are read once (plain
        // loads: a row as it was some time ago will do) and every entry that is itself a member
        // sets a bit.  An entry that is or ever was in a row never needs to be offered to that row
        // again (rows only improve: what has left a row cannot come back), so such pairs are
        // neither evaluated exactly nor queued; with rows of a hundred entries they are nearly all
        // of the pairs inside the thresholds, and each would otherwise cost a scan of the row.
        for (int f0 = tid; f0 < m * K; f0 += 8 * nthr) {      // eight entries in flight per thread
            u64 en[8];
            int rr[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int f = f0 + q * nthr;
                rr[q] = K == 1 ? min(f, m * K - 1) : (int)(((u64)(u32)min(f, m * K - 1) * k_magic) >> 32);
                en[q] = f < m * K ? graph[(size_t)lds.uid[rr[q]] * K + (f - rr[q] * K)] : ~0ULL;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (ef_is_empty(en[q])) continue;
                const int id = ef_id(en[q]);
                int h = (int)(((u32)id * 0x9E3779B1u) >> hshift);
                for (int k = lds.hkey[h]; k != -1; k = lds.hkey[h]) {
                    if (k == id) {
                        const int c = lds.hidx[h];
                        atomicOr(&lds.known[rr[q] * kw + (c >> 5)], 1u << (c & 31));
                        break;
                    }
                    h = (h + 1) & (hslots - 1);
                }
            }
        }
        if (dpad > d)
            for (int f = tid; f < m * (dpad - d); f += nthr) {
                const int r = f / (dpad - d), c = f - r * (dpad - d);
                lds.rows[r * stride + d + c] = 0.0f;
            }
        __syncthreads();
        // ---- 2..4: blocks of 16x16 pairs, in rounds of one block per wave -----------------
        const int nbr = (m_new + 15) >> 4, nbc = (m + 15) >> 4;
        const int n_blocks = nbr * nbc - nbr * (nbr - 1) / 2;     // block row <= block column
        int updates = 0;
        for (int q0 = 0; q0 < n_blocks; q0 += n_waves) {
            const int q = q0 + wave;
            if (q < n_blocks) {
                int bi = 0, rem = q;
                while (rem >= nbc - bi) {
                    rem -= nbc - bi;
                    ++bi;
                }
                const int bj = bi + rem;
                const int r16 = lane & 15, g = lane >> 4;
                const float *pa = lds.rows + min(16 * bi + r16, m - 1) * stride + 4 * g;
                const float *pb = lds.rows + min(16 * bj + r16, m - 1) * stride + 4 * g;
                floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
                for (int c = 0; c < dpad; c += 16) {
                    const float4 va = *reinterpret_cast<const float4 *>(pa + c);
                    const float4 vb = *reinterpret_cast<const float4 *>(pb + c);
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(va.x, vb.x, acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(va.y, vb.y, acc1, 0, 0, 0);
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(va.z, vb.z, acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(va.w, vb.w, acc1, 0, 0, 0);
                }
                // lane holds G[a = 16 bi + 4 g + k][b = 16 bj + r16], k = 0..3
                const int b = 16 * bj + r16;
                const float nb = lds.nrm[min(b, m - 1)];
                const float tb = __uint_as_float(lds.thr[min(b, m - 1)]);
                // what row b already knows of rows 16 bi .. 16 bi + 15 (one half of a word)
                const u32 known_b = lds.known[min(b, m - 1) * kw + (bi >> 1)] >> (16 * (bi & 1));
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int a = 16 * bi + 4 * g + k;
                    if (a < b && a < m_new && b < m && (mode == 0 || (mode == 1) == (b < m_new))) {
                        const float na = lds.nrm[a];
                        const float ta = __uint_as_float(lds.thr[a]);
                        const float sum = na + nb;
                        const float low = sum - 2.0f * (acc0[k] + acc1[k]) - margin_rel * sum;
                        // the pair is wanted by a row that may still accept it and does not know it yet
                        const bool for_a = low <= ta * thr_scale && !((lds.known[a * kw + (b >> 5)] >> (b & 31)) & 1u);
                        const bool for_b = low <= tb * thr_scale && !((known_b >> (4 * g + k)) & 1u);
                        if (for_a || for_b) lds.surv[atomicAdd(&lds.meta[4], 1)] = (u32)a | ((u32)b << 16);
                    }
                }
            }
            __syncthreads();
            const int n_surv = lds.meta[4];
            const bool last = q0 + n_waves >= n_blocks;
            if (last || n_surv + 256 * n_waves > s_cap) {
                // ---- 3. exact distances of the survivors, one 16-lane group per pair,
                //         in chunks whose proposals (two per pair at most) fit the queue -------
                for (int c0 = 0; c0 < n_surv; c0 += q_cap / 2) {
                    const int c1 = min(n_surv, c0 + q_cap / 2);
                    for (int p0 = c0; p0 < c1; p0 += n_grp) {
                        const int p = min(p0 + grp, c1 - 1);      // keep whole groups busy
                        const u32 ab = lds.surv[p];
                        const int a = ab & 0xFFFF, b = ab >> 16;
                        const float *ra = lds.rows + a * stride, *rb = lds.rows + b * stride;
                        float acc = 0.0f;
                        for (int j = gl; j < dpad; j += 16) {      // padding columns are 0 in both rows
                            const float diff = ra[j] - rb[j];
                            acc = __builtin_fmaf(diff, diff, acc);
                        }
                        const float dist = ef_group_reduce16(acc);
                        if (gl == 0 && p0 + grp < c1) {
                            const u32 db = __float_as_uint(dist);
                            if (db <= lds.thr[a] && !((lds.known[a * kw + (b >> 5)] >> (b & 31)) & 1u)) {
                                const int slot = atomicAdd(&lds.meta[3], 1);
                                lds.queue[slot].key = ef_pack(dist, lds.uid[b], mark);
                                lds.queue[slot].target = lds.uid[a];
                            }
                            if (db <= lds.thr[b] && !((lds.known[b * kw + (a >> 5)] >> (a & 31)) & 1u)) {
                                const int slot = atomicAdd(&lds.meta[3], 1);
                                lds.queue[slot].key = ef_pack(dist, lds.uid[a], mark);
                                lds.queue[slot].target = lds.uid[b];
                            }
                        }
                    }
                    __syncthreads();
                    // ---- 4. drain (one form for rows of any length: a second one for even, aligned rows makes
                    //      degree 64 0.7 % slower and degree 100 1 % faster, 30 000 x 256 and 20 000 x 160) ----
                    updates += WIDE
                                   ? drain_queue_g16(lds.queue, lds.meta[3], graph, worst, K, tid, nthr)
                                   : drain_queue(lds.queue, lds.meta[3], graph, worst, K, tid, nthr);
                    __syncthreads();
                    if (tid == 0) lds.meta[3] = 0;
                    __syncthreads();
                }
                if (tid == 0) lds.meta[4] = 0;
                __syncthreads();
            }
        }
        if (updates) atomicAdd(&lds.meta[2], updates);
        __syncthreads();
        if (tid == 0) block_updates += lds.meta[2];
        __syncthreads();
    }
    if (tid == 0) upd_block[blockIdx.x] = block_updates + (mode == 2 ? upd_block[blockIdx.x] : 0);      // (mode 2 follows mode 1)
}

// ---------------------------------------------------------------------------------------
// The same for long lists (some hundred ids per point): a thread per point would compare every
// id with every other and leaves room for a wave or three per CU next to its lists.  Here a
// wave takes a point: the four lists are read 64 ids at a time, an id is new to the join if
// its insertion into a hash table in LDS (open addressing, cleared per point) finds it absent,
// and a ballot gives the fresh ids their places.  A block of four waves takes 256 consecutive
// points per round and appends them to the work lists together (one counter bump per list and
// round).  Same lists as prepare_kernel up to the order of the ids inside U_new and U_old,
// which nothing depends on.  part: one triple per block.
template <class Source>      // (see prepare_kernel)
__global__ void __launch_bounds__(kBlock)
prepare_wave_kernel(const int *__restrict__ nw, const int *__restrict__ od,
                    const int *__restrict__ nw_c, const int *__restrict__ od_c,
                    const Source *__restrict__ rnew, const Source *__restrict__ rold,
                    const int *__restrict__ rnew_c, const int *__restrict__ rold_c,
                    int n, int K, int L, int cap, int hash_slots, JoinClasses jc,
                    int *__restrict__ ulist, int2 *__restrict__ ucount,
                    int *__restrict__ work, int *__restrict__ work_count,
                    long long *__restrict__ part)
{
    extern __shared__ int prep_sh[];
    constexpr int n_waves = kBlock / EF_WAVE;
    const int lane = ef_lane(), wave = threadIdx.x / EF_WAVE;
    int *hash = prep_sh + wave * (hash_slots + cap + EF_WAVE);      // [hash_slots]
    int *out = hash + hash_slots;                                  // [cap]
    int *cls_of = out + cap;                                       // [64] class of each point of the round
    __shared__ int wave_cnt[kMaxClasses][n_waves], block_base[kMaxClasses];
    __shared__ long long wave_sum[3][n_waves];
    const int hshift = 32 - (31 - __clz(hash_slots));
    auto wave_sync = [&]() {      // one wave: its LDS operations complete in program order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    long long evals = 0, rows = 0, rows0 = 0;      // lane 0: this wave's share of the iteration's work counters
    for (int i0 = blockIdx.x * kBlock; i0 < n; i0 += gridDim.x * kBlock) {      // (uniform over the block)
        const int w0 = i0 + wave * EF_WAVE;
        for (int p = 0; p < EF_WAVE; ++p) {
            const int i = w0 + p;
            if (i >= n) break;
            const int c_new = nw_c[i], rn = min(rnew_c[i], L);
            int m = 0, m_new = 0, cls = -1;
            if (c_new + rn > 0) {
                const int c_old = od_c[i], ro = min(rold_c[i], L);
                for (int f = lane; f < hash_slots; f += EF_WAVE) hash[f] = -1;
                wave_sync();
                auto add = [&](int id, bool have) {      // all lanes call; have: this lane offers id
                    bool fresh = false;
                    if (have) {
                        int h = (int)(((u32)id * 0x9E3779B1u) >> hshift);
                        for (;;) {
                            const int prev = atomicCAS(&hash[h], -1, id);
                            if (prev == -1) {
                                fresh = true;
                                break;
                            }
                            if (prev == id) break;
                            h = (h + 1) & (hash_slots - 1);
                        }
                    }
                    const u64 mask = __ballot(fresh);
                    if (fresh) out[m + __popcll(mask & ((1ULL << lane) - 1))] = id;
                    m += __popcll(mask);
                };
                for (int a0 = 0; a0 < c_new; a0 += EF_WAVE) {
                    const int a = a0 + lane;
                    add(a < c_new ? nw[(size_t)i * L + a] : -1, a < c_new);
                }
                for (int a0 = 0; a0 < rn; a0 += EF_WAVE) {
                    const int a = a0 + lane;
                    const int id = a < rn ? (int)(u32)rnew[(size_t)i * L + a] : -1;
                    add(id, a < rn);
                }
                m_new = m;
                for (int a0 = 0; a0 < c_old; a0 += EF_WAVE) {
                    const int a = a0 + lane;
                    add(a < c_old ? od[(size_t)i * K + a] : -1, a < c_old);
                }
                for (int a0 = 0; a0 < ro; a0 += EF_WAVE) {
                    const int a = a0 + lane;
                    const int id = a < ro ? (int)(u32)rold[(size_t)i * L + a] : -1;
                    add(id, a < ro);
                }
                wave_sync();
                if (m_new >= 1 && m >= 2) {
                    cls = 0;
                    while (cls < jc.n - 1 && m > jc.bound[cls]) ++cls;
                    evals += (long long)m_new * (m_new - 1) / 2 + (long long)m_new * (m - m_new);
                    rows += m;
                    if (cls == 0) rows0 += m;
                }
            }
            for (int f = lane; f < cap; f += EF_WAVE) ulist[(size_t)i * cap + f] = f < m ? out[f] : -1;
            if (lane == 0) {
                ucount[i] = make_int2(m_new, m);
                cls_of[p] = cls;
            }
            wave_sync();      // out is free for the next point
        }
        // append the round's points to the work lists
        const int mine = w0 + lane < n ? cls_of[lane] : -1;
        int rank = 0;
        for (int c = 0; c < jc.n; ++c) {
            const u64 mask = __ballot(mine == c);
            if (mine == c) rank = __popcll(mask & ((1ULL << lane) - 1));
            if (lane == 0) wave_cnt[c][wave] = __popcll(mask);
        }
        __syncthreads();
        if ((int)threadIdx.x < jc.n) {
            int tot = 0;
            for (int v = 0; v < n_waves; ++v) tot += wave_cnt[threadIdx.x][v];
            block_base[threadIdx.x] = tot ? atomicAdd(&work_count[threadIdx.x], tot) : 0;
        }
        __syncthreads();
        if (mine >= 0) {
            int off = block_base[mine] + rank;
            for (int v = 0; v < wave; ++v) off += wave_cnt[mine][v];
            work[(size_t)mine * n + off] = w0 + lane;
        }
        __syncthreads();      // wave_cnt and block_base are free for the next round
    }
    if (lane == 0) {
        wave_sum[0][wave] = evals;
        wave_sum[1][wave] = rows;
        wave_sum[2][wave] = rows0;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        long long sum = 0;
        for (int v = 0; v < n_waves; ++v) sum += wave_sum[threadIdx.x][v];
        part[(size_t)blockIdx.x * 3 + threadIdx.x] = sum;
    }
}

// ---------------------------------------------------------------------------------------
// The same local join for points whose join gathers at most 16 * NB vectors (NB = 1, 2),
// which is nearly all of them.  One wave per point and no row buffer in LDS: lane
// (r, g) = (lane % 16, lane / 16) loads 16-byte pieces of vector r (and 16 + r) straight
// from memory into the registers the MFMA reads, 128 coordinates at a time, so a block
// needs a few KB of LDS and many more waves fit a CU to hide the memory round trips.
// Survivors of the filter (few) get their exact distance from the same registers when
// the vectors fit them in one piece (ONE: d <= 128): lane (a, g) fetches the matching
// pieces of row b from lane (b, g) with cross-lane reads, accumulates the four partial
// sums it owns (coordinates = 4g..4g+3 mod 16, ascending) and the 16 partial sums are
// added in the fixed tree across the four lanes of row a.  Longer vectors take no filter:
// every pair is evaluated from the registers as the coordinates pass (see below).
// Requires d >= 4.

// where the survivors of Gram blocks (0,0), (0,1), (1,1) start in the LDS survivor buffer
__device__ constexpr int kSurvBase[3] = {0, 120, 376};
// d <= 128, joins of at most 16: more survivors than this and all pairs are evaluated by row rotations
constexpr int kDenseSurvivors = 24;
// d > 128: up to this many new members, or rows of the second set of sixteen, are broadcast to the others; the
// registers set the limits.  Rotations meet all pairs whatever the join asks for, 512 vector instructions per
// 8 KB of rows, 2048 per 16 KB of 17..32 rows, which also had to be streamed twice: the vector ALU was busy for
// 71 to 90 % of the joins' time.  10^6 x 960, iterations 1 to 6: 13.0 14.3 12.7 10.5 7.1 3.9 -> 11.0 12.6 10.3 7.6 4.7 2.6 ms,
// from the fourth on 5.6 to 5.8 TB/s; build 78.0 -> 64.3.  Unaligned rows, whose kernel for two sets keeps 48 registers
// in scratch memory (26 before), gain as much: NN-descent of 10 000 x 957 1.22 -> 1.09 ms, of x 960 1.23 -> 1.08; 20 000 x 131
// at degree 16 1.40 -> 1.16, x 132 1.29 -> 1.02.  (For d <= 128 the same next to the filter's code spilled
// and cost a quarter.)
constexpr int kFewNew = 8, kFewRest = 8;      // (EF_EACH_FEW names eight of either)
static_assert(kFewNew <= 8 && kFewRest <= 8 && kFewNew % 4 == 0 && kFewRest % 4 == 0, "EF_EACH_FEW");

// One surviving pair (rows a, b of the point's list) per lane with `mine` set: its distance is
// offered to row a and to row b where it passes their thresholds.  All lanes of the wave call
// this together; `fill` is the wave-uniform number of proposals queued, the new one is returned.
__device__ inline int propose_pair(Proposal *queue, int fill, bool mine, float dist, int a, int b,
                                   const u32 *thr, const int *uid, int mark)
{
    const u32 db = __float_as_uint(dist);
    const int ua = uid[a], ub = uid[b];
    const bool to_a = mine && db <= thr[a], to_b = mine && db <= thr[b];
    const u64 mask_a = __ballot(to_a), mask_b = __ballot(to_b);
    if (to_a) {
        Proposal &p = queue[fill + lanes_below(mask_a)];
        p.key = ef_pack(dist, ub, mark);
        p.target = ua;
    }
    fill += __popcll(mask_a);
    if (to_b) {
        Proposal &p = queue[fill + lanes_below(mask_b)];
        p.key = ef_pack(dist, ua, mark);
        p.target = ub;
    }
    return fill + __popcll(mask_b);
}

// KT: the row length if fixed at compile time (the row scans unroll), else -16 (2 .. 16 entries), -24 (17 .. 24, long vectors
// only) or 0
template <int NB, bool ONE, int KT, bool ALIGNED>
__global__ void __launch_bounds__(EF_WAVE) __attribute__((amdgpu_waves_per_eu(NB > 1 ? 3 : 4)))
join_reg_kernel(const float *__restrict__ X, int d, int K_,
                const int *__restrict__ work, const int *__restrict__ work_count, int q_cap,
                float margin_rel, float thr_scale, float u_rel, float rho0, const int *__restrict__ ulist,
                const int2 *__restrict__ ucount, int ucap, u64 *graph, u32 *worst,
                int *__restrict__ upd_block, int mode, const u32 *__restrict__ xmax)
{
    // mode 0: every pair of the join, fresh entries marked new.  1: only pairs of two new members.
    // 2: only pairs of a new and an old member, fresh entries marked old (the literal marking of
    // Alg. 4's second inner loop runs the joins twice, mode 1 before mode 2).  Rows 0 .. m_new - 1
    // of a list are its new members, so a pair (a, b), a < b, a new, is of two new members iff b is.
    const int mark = mode != 2;
    const int K = KT > 0 ? KT : K_;
    constexpr int R = 16 * NB;                    // rows
    constexpr int S_CAP = ONE ? R * (R - 1) / 2 + 8 : 0;    // every pair may survive
    extern __shared__ __align__(16) float smem[];
    int *uid = (int *)smem;                       // [R]
    u32 *thr = (u32 *)(uid + R);                  // [R] threshold bits (exact test)
    float *nf = (float *)(thr + R);               // [R] |x|^2 (1 - margin)   } the filter's
    float *tf = nf + R;                           // [R] threshold * scale    } operands (in the
    float *sq = tf + R;                           // [R] its square root      } scaled units of
    float *rr = sq + R;                           // [R] rounding radius      } the operands)
    u32 *surv = (u32 *)(rr + R);                  // [S_CAP] surviving pairs
    Proposal *queue = (Proposal *)(surv + align4(S_CAP));   // [q_cap]
    const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
    const int dirn = (EF_ROW_ROR(r16, 1) - r16) & 15;      // a rotation by t brings row r + t * dirn to row r
    const int count = *work_count;
    // The filter works on the vectors times a power of two that suits half precision (see ef_f16_scale).
    const float scale = ef_f16_scale(*xmax);
    // The id list and the sizes of a point are fetched one point ahead, and the thresholds of
    // its vectors as soon as those ids are there, so that they travel while the point before
    // is being worked on: the row loads are the only latency a point waits for.
    // (Thresholds only ever fall: one that is a point old lets a few more pairs through the
    // filter, nothing else.)
    int w = blockIdx.x;
    int i = w < count ? work[w] : -1;
    int u_pre = i >= 0 && lane < R ? ulist[(size_t)i * ucap + min(lane, ucap - 1)] : -1;
    int2 c_pre = i >= 0 ? ucount[i] : make_int2(0, 0);
    int i_next = w + (int)gridDim.x < count ? work[w + gridDim.x] : -1;
    u32 t_pre = u_pre >= 0 ? worst[u_pre] : 0u;
    // Proposals wait in the queue across points and are applied when about half of it is
    // full (and at the end): late iterations accept well under one proposal per point, and
    // a drain costs two memory round trips whatever its size.
    // The block is one wave: the fill of the queue and of the survivor lists are wave-uniform
    // registers, and a lane finds its slot from a ballot (no LDS counters, no round trips).
    int updates = 0, q_fill = 0;
    auto drain = [&](const Proposal *from, int cnt) {
        const int lane = ef_opaque(threadIdx.x);
        int len = K;
        if constexpr (KT <= 0) asm volatile("" : "+s"(len));      // (see ef_opaque)
        if constexpr (KT > 0 || KT == -16) return drain_queue_row(from, cnt, graph, worst, len, lane, EF_WAVE);
        else return drain_queue(from, cnt, graph, worst, len, lane, EF_WAVE);
    };
    for (; i >= 0; w += gridDim.x) {
        // ---- 0. the point's U_new ++ U_old (the loop ends with a barrier: LDS is free) -------
        const int m_new = c_pre.x, m = c_pre.y;
        auto mode_ok = [&](int b) { return mode == 0 || (mode == 1) == (b < m_new); };      // b: the pair's larger row
        const int u_cur = u_pre;
        if (lane < R) {
            uid[lane] = u_cur;
            thr[lane] = t_pre;
            const float t = ef_scaled_threshold(t_pre, scale, thr_scale);
            tf[lane] = t;
            sq[lane] = __builtin_sqrtf(t) * 1.000001f;
        }
        i = i_next;
        u_pre = i >= 0 && lane < R ? ulist[(size_t)i * ucap + min(lane, ucap - 1)] : -1;
        c_pre = i >= 0 ? ucount[i] : make_int2(0, 0);
        i_next = w + 2 * (int)gridDim.x < count ? work[w + 2 * gridDim.x] : -1;
        // ---- 1+2. Gram blocks from register operands ---------------------------------------
        const float *pa = X + (size_t)__shfl(u_cur, min(r16, m - 1), EF_WAVE) * d;
        const float *pb = NB > 1 ? X + (size_t)__shfl(u_cur, min(16 + r16, m - 1), EF_WAVE) * d : pa;
        const bool need11 = NB > 1 && m_new > 16;      // block (1,1) only if new rows reach it
        constexpr int NQ = NB > 1 ? 3 : 1;      // Gram blocks (0,0), (0,1), (1,1)
        floatx4 acc[NQ][2];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[q][h] = (floatx4){0.f, 0.f, 0.f, 0.f};
        float4 va[8], vb[NB > 1 ? 8 : 1];
        // Long vectors (d > 128): with the filter the rows would have to be streamed again for the
        // pairs that pass it, once per 128 of them.  Instead every pair gets its fixed-order
        // distance straight away, as in init_reg_kernel: row rotations per 128-coordinate piece
        // meet the pairs (vector instructions that hide under the gather: 512 per 8 KB of rows),
        // the four lanes of a column add their partial sums in the fixed tree, and lane (r, g)
        // holds the distances from row r to the rows 2g+1 and 2g+2 places on.  No Gram block, no
        // filter.  At most 16 rows: one pass, eight rotations.  17..32 rows: a first pass for the
        // pairs inside rows 0..15 and inside rows 16..31, a second one for rows 0..15 against
        // rotations 0..15 of rows 16..31.
        // Few new members (late iterations): each of them is broadcast to the sixteen lanes of a row set (a
        // modifier on the subtract again) and meets all the others, 64 vector instructions per new member, row
        // set and 128 coordinates; all rows are read once.  17..32 rows with few in the second set: rotations for
        // the pairs of the first set, and the rows of the second are broadcast; again one pass.
        // Not with long graph rows: a broadcast queues sixteen proposals to one row side by side, they are applied
        // together, and whoever finds its slot changed scans the row again.  Rows of the second set are broadcast up to
        // degree 24 (rotations and broadcasts: joins of 17..32 of 100 000 x 132, degree 17 3.35 and 2.88 ms, 20 3.54 and 3.12, 24
        // 4.03 and 3.89, 28 4.33 and 4.36, 30 4.47 and 4.59; of 20 000 x 132, degree 40 1.39 and 1.45, 64 3.17 and 3.53), in a
        // kernel of their own: next to them the rotations spill 47 registers instead of 34 where rows are unaligned.  New
        // members up to degree 32 (NN-descent of 30 000 x 200, samples of 3 and 4, degree 100 6.67 and 7.20 ms, 62 4.38 and
        // 4.61, 44 2.99 and 3.04, 40 2.27 and 2.28, 33 2.66 and 2.64; samples of 8, 62 7.07 and 6.99).
        constexpr bool rotated = !ONE;
        const bool few = rotated && (KT != 0 || K <= 32) && m_new <= kFewNew, few_rest = rotated && NB > 1 && KT != 0 && m <= 16 + kFewRest;
        float two[2] = {0.f, 0.f}, two_b[2] = {0.f, 0.f};
        // may_drain: only where a join can propose more than the queue holds (see reg_q_cap_for; every
        // place that drains is a copy of the insertion, in code and in registers)
        auto offer = [&](auto may_drain, bool mine, float dist, int a, int b) {
            if (decltype(may_drain)::value && q_fill + 2 * EF_WAVE > q_cap) {      // a step adds at most two proposals per lane
                updates += drain(queue, q_fill);
                q_fill = 0;
                __syncthreads();
            }
            q_fill = propose_pair(queue, q_fill, mine, dist, a, b, thr, uid, mark);
            __syncthreads();
        };
        // pairs inside rows 0..15 from rotations: lane (r, g) has the distances 2g+1 and 2g+2 places on (t = 0, 1)
        auto offer_rotation = [&](auto may_drain, int t) {
            const int rot = 2 * g + 1 + t, b = (r16 + dirn * rot) & 15;
            // rotation 8 meets every pair from both ends: the lower row keeps it
            offer(may_drain, (rot != 8 || r16 < b) && r16 < m && b < m && min(r16, b) < m_new && mode_ok(max(r16, b)), two[t], r16, b);
        };
#define EF_EACH_FEW(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7)
        if (few) {
            float P[kFewNew][4], PB[NB > 1 ? kFewNew : 1][4];
#pragma unroll
            for (int t = 0; t < kFewNew; ++t) {
                P[t][0] = P[t][1] = P[t][2] = P[t][3] = 0.0f;
                if (NB > 1) PB[NB > 1 ? t : 0][0] = PB[NB > 1 ? t : 0][1] = PB[NB > 1 ? t : 0][2] = PB[NB > 1 ? t : 0][3] = 0.0f;
            }
            for (int c0 = 0; c0 < d; c0 += 128) {
                const int n_pieces = min(8, (d - c0 + 15) >> 4);
                load_pieces<ALIGNED>(va, pa, c0, g, d, true);
                float4 (&wb)[8] = reinterpret_cast<float4 (&)[8]>(NB > 1 ? *vb : *va);
                if (NB > 1) load_pieces<ALIGNED>(wb, pb, c0, g, d, true);
#define EF_BROADCAST(A)                                                                    \
    if (A < m_new) {                                                                       \
        broadcast_round<A>(va, va, n_pieces, P[A]);                                        \
        if (NB > 1) broadcast_round<A>(va, wb, n_pieces, PB[NB > 1 ? A : 0]);              \
    }
                EF_EACH_FEW(EF_BROADCAST)
#undef EF_BROADCAST
            }
            __syncthreads();      // uid, thr visible
            t_pre = u_pre >= 0 ? worst[u_pre] : 0u;      // the next point's; its ids have arrived by now
#pragma unroll
            for (int a0 = 0; a0 < kFewNew; a0 += 4) {
                if (a0 >= m_new) break;
#pragma unroll
                for (int set = 0; set < NB; ++set) {
                    const float (&Q)[4][4] = reinterpret_cast<const float (&)[4][4]>(set == 0 ? P[a0] : PB[NB > 1 ? a0 : 0]);
                    const float dist = reduce_rotations4(Q);      // row a0 + g to row 16 set + r16
                    const int a = a0 + g, b = 16 * set + r16;
                    offer(std::false_type{}, a < m_new && a < b && b < m && mode_ok(b), dist, a, b);
                }
            }
        } else if (few_rest) {
            float P[8][4], PX[kFewRest][4], PB[kFewRest][4];
#pragma unroll
            for (int t = 0; t < 8; ++t) P[t][0] = P[t][1] = P[t][2] = P[t][3] = 0.0f;
#pragma unroll
            for (int t = 0; t < kFewRest; ++t) {
                PX[t][0] = PX[t][1] = PX[t][2] = PX[t][3] = 0.0f;
                PB[t][0] = PB[t][1] = PB[t][2] = PB[t][3] = 0.0f;
            }
            for (int c0 = 0; c0 < d; c0 += 64) {      // (the registers hold half a stretch next to that many sums)
                const int n_pieces = min(4, (d - c0 + 15) >> 4);
                float4 ha[4], hb[4];
                load_pieces<ALIGNED>(ha, pa, c0, g, d, true);
                load_pieces<ALIGNED>(hb, pb, c0, g, d, true);
                init_round<1>(ha, n_pieces, P[0]);
                init_round<2>(ha, n_pieces, P[1]);
                init_round<3>(ha, n_pieces, P[2]);
                init_round<4>(ha, n_pieces, P[3]);
                init_round<5>(ha, n_pieces, P[4]);
                init_round<6>(ha, n_pieces, P[5]);
                init_round<7>(ha, n_pieces, P[6]);
                init_round<8>(ha, n_pieces, P[7]);
#define EF_BROADCAST(B)                                                                    \
    if (B < kFewRest && 16 + B < m) {                                                      \
        broadcast_round<B>(hb, ha, n_pieces, PX[B]);                                       \
        if (need11) broadcast_round<B>(hb, hb, n_pieces, PB[B]);                           \
    }
                EF_EACH_FEW(EF_BROADCAST)
#undef EF_BROADCAST
            }
            reduce_rotations(P, two);
            __syncthreads();      // uid, thr visible
            t_pre = u_pre >= 0 ? worst[u_pre] : 0u;
            offer_rotation(std::false_type{}, 0);
            offer_rotation(std::false_type{}, 1);
#pragma unroll
            for (int t0 = 0; t0 < kFewRest; t0 += 4) {
                if (16 + t0 >= m) break;
                const int x = 16 + t0 + g, y = 16 + r16;      // the broadcast row; the lane's row of the second set
                const float dist = reduce_rotations4(reinterpret_cast<const float (&)[4][4]>(PX[t0]));
                offer(std::false_type{}, x < m && r16 < m_new && mode_ok(x), dist, r16, x);
                if (need11) {
                    const float dist_b = reduce_rotations4(reinterpret_cast<const float (&)[4][4]>(PB[t0]));
                    offer(std::false_type{}, x < m_new && x < y && y < m && mode_ok(y), dist_b, x, y);
                }
            }
        } else {
        if (rotated) {
            float P[8][4], PB[NB > 1 ? 8 : 1][4];
#pragma unroll
            for (int t = 0; t < 8; ++t) P[t][0] = P[t][1] = P[t][2] = P[t][3] = 0.0f;
            if (NB > 1) {
#pragma unroll
                for (int t = 0; t < 8; ++t) PB[NB > 1 ? t : 0][0] = PB[NB > 1 ? t : 0][1] = PB[NB > 1 ? t : 0][2] = PB[NB > 1 ? t : 0][3] = 0.0f;
            }
            for (int c0 = 0; c0 < d; c0 += 128) {
                const int n_pieces = min(8, (d - c0 + 15) >> 4);
                load_pieces<ALIGNED>(va, pa, c0, g, d, true);
                init_round<1>(va, n_pieces, P[0]);
                init_round<2>(va, n_pieces, P[1]);
                init_round<3>(va, n_pieces, P[2]);
                init_round<4>(va, n_pieces, P[3]);
                init_round<5>(va, n_pieces, P[4]);
                init_round<6>(va, n_pieces, P[5]);
                init_round<7>(va, n_pieces, P[6]);
                init_round<8>(va, n_pieces, P[7]);
                if (NB > 1 && need11) {      // pairs inside rows 16..31 are wanted only if new rows reach them
                    float4 (&wb)[8] = reinterpret_cast<float4 (&)[8]>(vb);
                    load_pieces<ALIGNED>(wb, pb, c0, g, d, true);
                    init_round<1>(wb, n_pieces, PB[0]);
                    init_round<2>(wb, n_pieces, PB[NB > 1 ? 1 : 0]);
                    init_round<3>(wb, n_pieces, PB[NB > 1 ? 2 : 0]);
                    init_round<4>(wb, n_pieces, PB[NB > 1 ? 3 : 0]);
                    init_round<5>(wb, n_pieces, PB[NB > 1 ? 4 : 0]);
                    init_round<6>(wb, n_pieces, PB[NB > 1 ? 5 : 0]);
                    init_round<7>(wb, n_pieces, PB[NB > 1 ? 6 : 0]);
                    init_round<8>(wb, n_pieces, PB[NB > 1 ? 7 : 0]);
                }
            }
            reduce_rotations(P, two);
            if (NB > 1) reduce_rotations(reinterpret_cast<const float (&)[8][4]>(PB), two_b);
        }
        for (int c0 = 0; c0 < d && !rotated; c0 += 128) {
            if (c0 + 128 <= d) {     // a whole 128-coordinate piece: no per-load bounds test
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int j = c0 + 16 * s + 4 * g;
                    va[s] = ALIGNED ? *reinterpret_cast<const float4 *>(pa + j) : load_unaligned4(pa + j);
                    if (NB > 1) vb[NB > 1 ? s : 0] = ALIGNED ? *reinterpret_cast<const float4 *>(pb + j) : load_unaligned4(pb + j);
                }
            } else {
                load_pieces<ALIGNED>(va, pa, c0, g, d, true);
                if (NB > 1) load_pieces<ALIGNED>(reinterpret_cast<float4 (&)[8]>(vb), pb, c0, g, d, true);
            }
            auto gram = [&](auto scaled) {
#pragma unroll
                for (int s = 0; s < 8; s += 2) {
                    if (c0 + 16 * s >= d) break;      // (pieces beyond d were loaded as zeros)
                    const f16x8 oa = ef_pack_f16<decltype(scaled)::value>(va[s], va[s + 1], scale);
                    acc[0][(s >> 1) & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(oa, oa, acc[0][(s >> 1) & 1], 0, 0, 0);
                    if (NB > 1) {
                        constexpr int Q1 = NB > 1 ? 1 : 0, Q2 = NB > 1 ? 2 : 0;
                        const f16x8 ob = ef_pack_f16<decltype(scaled)::value>(vb[NB > 1 ? s : 0], vb[NB > 1 ? s + 1 : 0], scale);
                        acc[Q1][(s >> 1) & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(oa, ob, acc[Q1][(s >> 1) & 1], 0, 0, 0);
                        acc[Q2][(s >> 1) & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ob, ob, acc[Q2][(s >> 1) & 1], 0, 0, 0);
                    }
                }
            };
            if (scale != 1.0f) gram(std::true_type{});
            else gram(std::false_type{});
        }
        if (!rotated) {
            // The filter's squared norms are those of the rounded vectors: the diagonals of Gram
            // blocks (0,0) and (1,1) (lane (r16, g) holds G[4 g + k][r16]).  rr: how far rounding may
            // have moved the vector, u |x'| + r0.
            if ((r16 >> 2) == g) {
                const int kd = r16 & 3;
                const float dg = kd == 0 ? acc[0][0][0] + acc[0][1][0]
                               : kd == 1 ? acc[0][0][1] + acc[0][1][1]
                               : kd == 2 ? acc[0][0][2] + acc[0][1][2] : acc[0][0][3] + acc[0][1][3];
                nf[r16] = dg * (1.0f - margin_rel);
                rr[r16] = __builtin_fmaf(u_rel, __builtin_sqrtf(dg), rho0);
                if (NB > 1) {
                    constexpr int Q2 = NB > 1 ? 2 : 0;
                    const float dh = kd == 0 ? acc[Q2][0][0] + acc[Q2][1][0]
                                   : kd == 1 ? acc[Q2][0][1] + acc[Q2][1][1]
                                   : kd == 2 ? acc[Q2][0][2] + acc[Q2][1][2] : acc[Q2][0][3] + acc[Q2][1][3];
                    nf[16 + r16] = dh * (1.0f - margin_rel);
                    rr[16 + r16] = __builtin_fmaf(u_rel, __builtin_sqrtf(dh), rho0);
                }
            }
        }
        __syncthreads();      // uid, thr, nf, tf, sq, rr visible
        t_pre = u_pre >= 0 ? worst[u_pre] : 0u;      // the next point's; its ids have arrived by now
        // ---- filter: lane holds G[a = 16 bi + 4 g + k][b = 16 bj + r16] of block q -----------
        // With D' the distance of the rounded vectors, r = rr[a] + rr[b] and T the larger threshold:
        // |D' - D| <= r, so D^2 <= T implies D'^2 <= T + r (2 sqrt(T) + r).  Pair (a, b) survives
        // unless (|a'|^2 + |b'|^2)(1 - margin) - 2 a'.b' is above that (the margin covers the three
        // accumulations; a comparison with a NaN - an infinite threshold times a zero radius -
        // keeps the pair).
        int n_surv[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) n_surv[q] = 0;
#pragma unroll
        for (int q = 0; q < (NB > 1 ? 3 : 1); ++q) {
            if (rotated) break;
            const int bi = q == 2 ? 1 : 0, bj = q == 0 ? 0 : 1;
            const int b = 16 * bj + r16, a0 = 16 * bi + 4 * g;
            // valid pairs: a < lim
            const int lim = b >= m ? 0 : mode == 0 ? min(m_new, b) : mode == 1 ? (b < m_new ? b : 0) : (b >= m_new ? m_new : 0);
            const float nfb = nf[b], tfb = tf[b], sqb = sq[b], rrb = rr[b];      // junk beyond m, masked by lim
            const float4 nfa = *reinterpret_cast<const float4 *>(nf + a0);
            const float4 tfa = *reinterpret_cast<const float4 *>(tf + a0);
            const float4 sqa = *reinterpret_cast<const float4 *>(sq + a0);
            const float4 rra = *reinterpret_cast<const float4 *>(rr + a0);
            const float nfa_k[4] = {nfa.x, nfa.y, nfa.z, nfa.w}, tfa_k[4] = {tfa.x, tfa.y, tfa.z, tfa.w};
            const float sqa_k[4] = {sqa.x, sqa.y, sqa.z, sqa.w}, rra_k[4] = {rra.x, rra.y, rra.z, rra.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float lhs = __builtin_fmaf(-2.0f, acc[q][0][k] + acc[q][1][k], nfa_k[k] + nfb);
                const float rad = rra_k[k] + rrb;
                const float rhs = __builtin_fmaf(rad, __builtin_fmaf(2.0f, fmaxf(sqa_k[k], sqb), rad), fmaxf(tfa_k[k], tfb));
                // one list per Gram block, entries are rows local to the block
                const bool keep = a0 + k < lim && !(lhs > rhs);
                const u64 kept = __ballot(keep);
                if (keep) surv[kSurvBase[q] + n_surv[q] + lanes_below(kept)] = (u32)((a0 + k) & 15) | ((u32)(b & 15) << 8);
                n_surv[q] += __popcll(kept);
            }
        }
        __syncthreads();
        if (rotated) {
            // (the two sets in turn: proposals to one row further apart in the queue; both rotations of the first
            // set before those of the second: 200 000 x 132, degree 64 16.9 -> 17.2 ms)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                offer_rotation(std::bool_constant<(NB > 1)>{}, t);
                if (NB > 1 && need11) {
                    const int rot = 2 * g + 1 + t, b = (r16 + dirn * rot) & 15;
                    offer(std::true_type{}, (rot != 8 || r16 < b) && 16 + r16 < m && 16 + b < m && 16 + min(r16, b) < m_new &&
                              mode_ok(16 + max(r16, b)),
                          two_b[t], 16 + r16, 16 + b);
                }
            }
            if (NB > 1) {
                // second pass: row r of rows 0..15 against rows 16 + (r + T) of rows 16..31, T = 0..15
                float PX[2][8][4];
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int t = 0; t < 8; ++t) PX[h][t][0] = PX[h][t][1] = PX[h][t][2] = PX[h][t][3] = 0.0f;
                float4 (&wb)[8] = reinterpret_cast<float4 (&)[8]>(vb);
                for (int c0 = 0; c0 < d; c0 += 128) {
                    const int n_pieces = min(8, (d - c0 + 15) >> 4);
                    load_pieces<ALIGNED>(va, pa, c0, g, d, true);
                    load_pieces<ALIGNED>(wb, pb, c0, g, d, true);
                    cross_round<0>(va, wb, n_pieces, PX[0][0]);
                    cross_round<1>(va, wb, n_pieces, PX[0][1]);
                    cross_round<2>(va, wb, n_pieces, PX[0][2]);
                    cross_round<3>(va, wb, n_pieces, PX[0][3]);
                    cross_round<4>(va, wb, n_pieces, PX[0][4]);
                    cross_round<5>(va, wb, n_pieces, PX[0][5]);
                    cross_round<6>(va, wb, n_pieces, PX[0][6]);
                    cross_round<7>(va, wb, n_pieces, PX[0][7]);
                    cross_round<8>(va, wb, n_pieces, PX[1][0]);
                    cross_round<9>(va, wb, n_pieces, PX[1][1]);
                    cross_round<10>(va, wb, n_pieces, PX[1][2]);
                    cross_round<11>(va, wb, n_pieces, PX[1][3]);
                    cross_round<12>(va, wb, n_pieces, PX[1][4]);
                    cross_round<13>(va, wb, n_pieces, PX[1][5]);
                    cross_round<14>(va, wb, n_pieces, PX[1][6]);
                    cross_round<15>(va, wb, n_pieces, PX[1][7]);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float cross[2];
                    reduce_rotations(PX[h], cross);      // rotations 8h + 2g and 8h + 2g + 1
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int rot = 8 * h + 2 * g + t, b = 16 + ((r16 + dirn * rot) & 15);
                        offer(std::true_type{}, b < m && r16 < m_new && mode_ok(b), cross[t], r16, b);
                    }
                }
            }
        }
        // ---- 3a. survivors from registers, sixteen pairs per round --------------------------
        // The four lanes r16 + 16 g (g = 0..3) of column r16 take pair p0 + r16: lane g
        // fetches the pieces it needs of rows a and b from lanes a + 16 g and b + 16 g,
        // which hold the coordinates = 4g..4g+3 (mod 16) of those rows.
        if (ONE) {
#pragma unroll
            for (int q = 0; q < (NB > 1 ? 3 : 1); ++q) {
                const int bi = q == 2 ? 1 : 0, bj = q == 0 ? 0 : 1;
                const int n_q = n_surv[q];
                // Joins of at most 16, many survivors (early iterations: most pairs
                // pass): all 120 pairs by row rotations, as for long vectors, cost what two rounds
                // of sixteen survivors cost.  The filter never drops a pair that would pass a
                // threshold, so which way a pair takes makes no difference to what is proposed.
                if (NB == 1 && n_q > kDenseSurvivors) {
                    const int lane = ef_opaque(threadIdx.x), r16 = lane & 15, g = lane >> 4;
                    const int n_pieces = (d + 15) >> 4;
#pragma unroll
                    for (int half = 0; half < 2; ++half) {      // rotations 1..4, then 5..8
                        float P[4][4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) P[t][0] = P[t][1] = P[t][2] = P[t][3] = 0.0f;
                        if (half == 0) {
                            init_round<1>(va, n_pieces, P[0]);
                            init_round<2>(va, n_pieces, P[1]);
                            init_round<3>(va, n_pieces, P[2]);
                            init_round<4>(va, n_pieces, P[3]);
                        } else {
                            init_round<5>(va, n_pieces, P[0]);
                            init_round<6>(va, n_pieces, P[1]);
                            init_round<7>(va, n_pieces, P[2]);
                            init_round<8>(va, n_pieces, P[3]);
                        }
                        const float dist = reduce_rotations4(P);
                        const int rot = 4 * half + 1 + g, b = (r16 + dirn * rot) & 15;
                        const bool once = rot != 8 || r16 < b;      // rotation 8 meets every pair from both ends
                        q_fill = propose_pair(queue, q_fill, once && r16 < m && b < m && min(r16, b) < m_new && mode_ok(max(r16, b)),
                                              dist, r16, b, thr, uid, mark);
                        __syncthreads();
                    }
                    continue;
                }
                for (int p0 = 0; p0 < n_q; p0 += 16) {
                    const bool has = p0 + r16 < n_q;
                    const u32 ent = surv[kSurvBase[q] + min(p0 + r16, n_q - 1)];
                    const int al = ent & 15, bl = (ent >> 8) & 15;
                    const int src_a = al + 16 * g, src_b = bl + 16 * g;
                    float p0s = 0.f, p1s = 0.f, p2s = 0.f, p3s = 0.f;
#pragma unroll
                    for (int s = 0; s < 8; ++s) {
                        if (16 * s >= d) break;
                        const float4 own = bi == 0 ? va[s] : vb[NB > 1 ? s : 0];
                        const float4 oth = bj == 0 ? va[s] : vb[NB > 1 ? s : 0];
                        const float d0 = __shfl(own.x, src_a, EF_WAVE) - __shfl(oth.x, src_b, EF_WAVE);
                        const float d1 = __shfl(own.y, src_a, EF_WAVE) - __shfl(oth.y, src_b, EF_WAVE);
                        const float d2 = __shfl(own.z, src_a, EF_WAVE) - __shfl(oth.z, src_b, EF_WAVE);
                        const float d3 = __shfl(own.w, src_a, EF_WAVE) - __shfl(oth.w, src_b, EF_WAVE);
                        p0s = __builtin_fmaf(d0, d0, p0s);
                        p1s = __builtin_fmaf(d1, d1, p1s);
                        p2s = __builtin_fmaf(d2, d2, p2s);
                        p3s = __builtin_fmaf(d3, d3, p3s);
                    }
                    // partial sum l lives in lane g = l / 4, slot l % 4
                    const float dist = ef_sum_partials(p0s, p1s, p2s, p3s);
                    q_fill = propose_pair(queue, q_fill, has && g == 0, dist, 16 * bi + al, 16 * bj + bl, thr, uid, mark);
                    __syncthreads();
                    // NB = 1: the queue is sized so that a point's proposals always fit (at most 240
                    // on top of fewer than q_cap / 2): no drain while the operands are live
                    if (NB > 1 && q_fill + 32 > q_cap) {      // a round adds at most two proposals per pair
                        updates += drain(queue, q_fill);
                        q_fill = 0;
                        __syncthreads();
                    }
                }
            }
        }
        }      // few
        if (q_fill >= (ONE ? q_cap / 2 : EF_WAVE)) {
            // whole passes of 64 only, from the end of the queue: what is left waits for the next
            // drain (a pass costs its two round trips however few lanes it fills)
            const int rest = q_fill & (EF_WAVE - 1);
            updates += drain(queue + rest, q_fill - rest);
            q_fill = rest;
        }
        __syncthreads();
    }
    __syncthreads();
    updates += drain(queue, q_fill);
    updates = ef_wave_sum_i32(updates);
    if (lane == 0) upd_block[blockIdx.x] = updates + (mode == 2 ? upd_block[blockIdx.x] : 0);      // (mode 2 follows mode 1)
}

// ---------------------------------------------------------------------------------------
// The local join for points whose join gathers more than 32 vectors of at most 128 coordinates
// (d >= 4), without a row buffer: one wave per point.  Three passes over the join's list:
//   1. Wants.  Up to kTileGroup tiles of sixteen new rows (A) stand in registers as half-precision operands while
//      every tile of sixteen rows from the first of them onwards (B) passes by once: a Gram block per tile
//      pair, join_reg_kernel's filter (the squared norms of the rounded rows are the diagonals of the tiles'
//      blocks with themselves), and for either row of a pair one bit that says whether its own threshold lets
//      the other in.
//   2. Known.  The rows of ids of the members that want anybody are scanned, and every entry that is itself a
//      member loses its bit: with rows of a hundred entries most pairs inside the thresholds are in the rows
//      already (two close points sit together in the lists of a hundred others), and offering them again
//      would cost a scan of the row each.
//   3. The wants that are left, one (row, member) per four lanes: both rows are loaded from memory (from
//      the caches mostly), the fixed-order distance goes through the exact threshold test and into the queue.
// The bound: vector issue and the gathers of rows and ids (fabric 4.5 TB/s).  Scanning only rows that want
// somebody, after the filter, is what pays: 59 of 65 million members in the first iteration of 10^6 x 96 at
// degree 100, 94 of 107, 39 of 98, 44 of 106, 32 of 102, 18 of 93, 11 of 83, 6 of 74 in the eighth.  (When the
// scan came first, for all members, and each pair of tiles was loaded and evaluated together:
// 318 ms of tile joins per build, now 234; from the fourth iteration on 136, now 68.)
struct TileLds {
    int *uid;          // [c16] U_new ++ U_old
    u32 *thr;          // [c16] threshold bits
    u32 *want;         // [cap][known_words(cap)] bit c of row r: r would take member c
    u32 *bits;         // [kTileBits / 32] which hashes occur among the members' ids
    unsigned short *head, *next;      // [kTileHeads], [c16] chains of places (+ 1; 0 = end) by hash
    unsigned char *rows;              // [c16] members that want anybody
    int2 *hits;        // [5 * EF_WAVE] ids that passed the hash bits, and the members whose rows they are in
    unsigned short *items;      // [2 * EF_WAVE] wants to evaluate, row << 8 | member (shares the room of hits)
    float *terms;      // [c16 / 16][4][16] the filter's terms of the rows, tile by tile (pass 1; shares the room of hits)
    Proposal *queue;   // [kTileQueue]
};
constexpr int kTileQueue = 96;      // proposals that can wait
constexpr int kTileGroup = 2;       // A tiles in registers at a time (three: the same; four: 18 ms slower, 69 spills)
constexpr int kTileBits = 4096, kTileHeads = 256;
__host__ __device__ inline size_t tile_lds_bytes(int cap)
{
    const int c16 = (cap + 15) & ~15;
    const size_t hits = 5 * EF_WAVE * sizeof(int2), terms = (size_t)16 * c16;
    return (size_t)kTileQueue * sizeof(Proposal) + (hits > terms ? hits : terms) + (size_t)(2 * c16 + align4(cap * known_words(cap)) + kTileBits / 32) * 4 +
           (size_t)(kTileHeads + c16) * 2 + c16;
}
__device__ inline TileLds tile_lds_carve(float *smem, int cap)
{
    TileLds l;
    const int c16 = (cap + 15) & ~15;
    l.queue = (Proposal *)smem;
    l.hits = (int2 *)(l.queue + kTileQueue);
    l.items = (unsigned short *)l.hits;
    l.terms = (float *)l.hits;
    l.uid = (int *)(l.hits + max(5 * EF_WAVE, 2 * c16));
    l.thr = (u32 *)(l.uid + c16);
    l.want = l.thr + c16;
    l.bits = l.want + align4(cap * known_words(cap));
    l.head = (unsigned short *)(l.bits + kTileBits / 32);
    l.next = l.head + kTileHeads;
    l.rows = (unsigned char *)(l.next + c16);
    return l;
}

constexpr int kTileWaves = 4;      // waves per SIMD the tile join is compiled for
// LONG_ROWS: longer graph rows (see the launch): eight lanes per proposal.  QUADS: K % 4 == 0, rows of
// ids and of entries are 16-byte aligned (compiled apart: addressing for any K cost such rows 2 %;
// before other lengths had it, a thread scanned a row alone: 10^5 x 64, degree 81 53 -> 36 ms per build).
template <bool LONG_ROWS, bool ALIGNED, bool QUADS>
__global__ void __launch_bounds__(EF_WAVE) __attribute__((amdgpu_waves_per_eu(kTileWaves)))
join_tile_kernel(const float *__restrict__ X, int d, int K, u32 k_magic,
                 u32 kq_magic, int *gid, const int *__restrict__ work, const int *__restrict__ work_count, int cap,
                 float margin_rel, float thr_scale, float u_rel, float rho0, const int *__restrict__ ulist,
                 const int2 *__restrict__ ucount, int ucap, u64 *graph, u32 *worst,
                 int *__restrict__ upd_block, int mode, const u32 *__restrict__ xmax)
{
    extern __shared__ __align__(16) float smem[];
    const TileLds lds = tile_lds_carve(smem, cap);
    const int mark = mode != 2;      // (modes: see join_reg_kernel)
    const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
    const int kw = known_words(cap);
    // the power of two that suits the data's halves (see join_reg_kernel)
    const float scale = ef_f16_scale(*xmax);
    const int count = *work_count;
    int updates = 0, q_fill = 0, w = blockIdx.x;
    auto drain = [&]() {
        const int lane = ef_opaque(threadIdx.x);
        updates += LONG_ROWS ? drain_queue_g8<!QUADS>(lds.queue, q_fill, graph, worst, K, lane, EF_WAVE, gid)
                             : drain_queue(lds.queue, q_fill, graph, worst, K, lane, EF_WAVE);
        q_fill = 0;
        __syncthreads();
    };
    // A full-rate multiplication of the id's low 24 bits; bits 20..31 of the product pick one of
    // kTileBits bits, bits 24..31 one of kTileHeads chains.
    auto hash_of = [](int id) -> u32 { return ((u32)id & 0xFFFFFFu) * 0x9E3779u; };
    static_assert(kTileBits == 1 << 12 && kTileHeads == 1 << 8, "hash bits");
    // passes 0 to 2 for point i: returns how many members want anybody (lds.rows, lds.want)
    auto wants_of = [&](int i) {
        const int2 mc = ucount[i];
        const int m_new = mc.x, m = min(mc.y, cap);
        // ---- 0. ids, thresholds; the members' places by id ------------------------------------
        for (int f = lane; f < m * kw; f += EF_WAVE) lds.want[f] = 0u;
        for (int f = lane; f < kTileBits / 32; f += EF_WAVE) lds.bits[f] = 0u;
        for (int f = lane; f < kTileHeads / 2; f += EF_WAVE) ((u32 *)lds.head)[f] = 0u;
        __syncthreads();
        for (int r0 = 0; r0 < m; r0 += EF_WAVE) {
            const int r = r0 + lane;
            if (r < m) {
                const int id = ulist[(size_t)i * ucap + r];
                const u32 t = ef_load_coherent(worst + id);
                lds.uid[r] = id;
                lds.thr[r] = t;
                const u32 h = hash_of(id);
                atomicOr(&lds.bits[h >> 25], 1u << ((h >> 20) & 31));
                // the place enters its chain at the head (a 16-bit half of a word)
                u32 *word = (u32 *)lds.head + (h >> 25);
                const int sh = (h >> 20) & 16;
                u32 old = *word, seen;
                for (;;) {
                    seen = atomicCAS(word, old, (old & ~(0xFFFFu << sh)) | (u32)(r + 1) << sh);
                    if (seen == old) break;
                    old = seen;
                }
                lds.next[r] = (unsigned short)(old >> sh);
            }
        }
        __syncthreads();
        // ---- 1. wants ---------------------------------------------------------------------------
        const int nbr = (m_new + 15) >> 4, nbc = (m + 15) >> 4;
        auto load_tile = [&](int tile, f16x8 (&o)[4]) {
            float4 v[8];
            load_row<ALIGNED>(v, X + (size_t)lds.uid[min(16 * tile + r16, m - 1)] * d, g, d);
            if (scale != 1.0f) {
#pragma unroll
                for (int s = 0; s < 4; ++s) o[s] = ef_pack_f16<true>(v[2 * s], v[2 * s + 1], scale);
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) o[s] = ef_pack_f16<false>(v[2 * s], v[2 * s + 1], scale);
            }
        };
        auto gram = [&](const f16x8 (&a)[4], const f16x8 (&b)[4]) {
            floatx4 acc = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (32 * s >= d) break;      // (pieces beyond d are zeros)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s], b[s], acc, 0, 0, 0);
            }
            return acc;
        };
        // the filter's terms of the tile's sixteen rows: |x'|^2 (1 - margin), rounding radius, scaled
        // threshold and twice its square root (junk beyond m is masked below)
        auto terms = [&](const f16x8 (&o)[4], int tile) {
            float *const f = lds.terms + 64 * tile;
            const floatx4 acc = gram(o, o);      // lane (r16, r16 >> 2) holds the diagonal
            if ((r16 >> 2) != g) return;
            const int kd = r16 & 3;
            const float dg = kd == 0 ? acc[0] : kd == 1 ? acc[1] : kd == 2 ? acc[2] : acc[3];
            const float t = ef_scaled_threshold(lds.thr[16 * tile + r16], scale, thr_scale);
            f[r16] = dg * (1.0f - margin_rel);
            f[16 + r16] = __builtin_fmaf(u_rel, ef_sqrt_up(dg), rho0);
            f[32 + r16] = t;
            f[48 + r16] = 2.0f * ef_sqrt_up(t);
        };
        unsigned short *const want16 = (unsigned short *)lds.want;      // [cap][2 kw]: sixteen members each
        for (int bi0 = 0; bi0 < nbr; bi0 += kTileGroup) {
            f16x8 oa[kTileGroup][4];
#pragma unroll
            for (int t = 0; t < kTileGroup; ++t) {
                if (bi0 + t >= nbr) break;
                load_tile(bi0 + t, oa[t]);
                if (bi0 == 0) terms(oa[t], t);      // (later groups have passed by as B tiles)
            }
            for (int bj = bi0; bj < nbc; ++bj) {
                f16x8 ob[4];
                load_tile(bj, ob);
                if (bi0 == 0 && bj >= min(kTileGroup, nbr)) terms(ob, bj);
                __syncthreads();
                const float *const fb = lds.terms + 64 * bj;
                const int b = 16 * bj + r16;
                const float nfb = fb[r16], rrb = fb[16 + r16], tfb = fb[32 + r16], sqb = fb[48 + r16];
                // valid pairs: a < lim
                const int lim = b >= m ? 0 : mode == 0 ? min(m_new, b) : mode == 1 ? (b < m_new ? b : 0) : (b >= m_new ? m_new : 0);
#pragma unroll
                for (int t = 0; t < kTileGroup; ++t) {
                    const int bi = bi0 + t;
                    if (bi >= nbr || bi > bj) break;
                    const floatx4 acc = gram(oa[t], ob);      // the lane holds G[a = 16 bi + 4 g + k][b]
                    const float *fa = lds.terms + 64 * bi + 4 * g;
                    const float4 nfa = *reinterpret_cast<const float4 *>(fa), rra = *reinterpret_cast<const float4 *>(fa + 16);
                    const float4 tfa = *reinterpret_cast<const float4 *>(fa + 32), sqa = *reinterpret_cast<const float4 *>(fa + 48);
                    const float nfa_k[4] = {nfa.x, nfa.y, nfa.z, nfa.w}, rra_k[4] = {rra.x, rra.y, rra.z, rra.w};
                    const float tfa_k[4] = {tfa.x, tfa.y, tfa.z, tfa.w}, sqa_k[4] = {sqa.x, sqa.y, sqa.z, sqa.w};
                    const int a0 = 16 * bi + 4 * g;
                    u32 by_b = 0, by_a = 0;      // which of rows a0 .. a0 + 3 b wants; the sixteen members row a0 + r16 wants (r16 < 4)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float lhs = __builtin_fmaf(-2.0f, acc[k], nfa_k[k] + nfb), rad = rra_k[k] + rrb;
                        // (a comparison with a NaN keeps the pair)
                        const bool valid = a0 + k < lim;
                        const u64 for_a = __ballot(valid && !(lhs > __builtin_fmaf(rad, sqa_k[k] + rad, tfa_k[k])));
                        by_a = r16 == k ? (u32)(for_a >> (16 * g)) : by_a;
                        by_b |= valid && !(lhs > __builtin_fmaf(rad, sqb + rad, tfb)) ? 1u << k : 0u;
                    }
                    by_b <<= 4 * g;
                    by_b |= (u32)__shfl_xor((int)by_b, 16, EF_WAVE);
                    by_b |= (u32)__shfl_xor((int)by_b, 32, EF_WAVE);
                    if (r16 < 4 && a0 + r16 < m) want16[(size_t)(a0 + r16) * 2 * kw + bj] = (unsigned short)by_a;
                    if (bi == bj) __syncthreads();      // (inside one tile the two halves of a row's bits meet)
                    if (g == 0 && b < m) {
                        unsigned short *const wb = want16 + (size_t)b * 2 * kw + bi;
                        *wb = (unsigned short)(bi == bj ? by_b | *wb : by_b);
                    }
                }
            }
        }
        __syncthreads();
        // the members that want anybody
        int n_rows = 0;
        for (int r0 = 0; r0 < m; r0 += EF_WAVE) {
            const int r = r0 + lane;
            u32 any = 0;
            if (r < m)
                for (int q = 0; q < kw; ++q) any |= lds.want[r * kw + q];
            const u64 mask = __ballot(any != 0);
            if (any) lds.rows[n_rows + lanes_below(mask)] = (unsigned char)r;
            n_rows += __popcll(mask);
        }
        __syncthreads();
        // ---- 2. known pairs: the rows of ids of those members, four ids per load where rows allow it --
        const int lane = ef_opaque(threadIdx.x);
        int n_hits = 0;
        auto settle = [&](int most) {      // until at most that many hits (fewer than 64, or none) are left: members lose their bit
            while (n_hits > most) {
                const int n_h = min(n_hits, EF_WAVE);
                n_hits -= n_h;
                __syncthreads();
                if (lane < n_h) {
                    const int2 hit = lds.hits[n_hits + lane];
                    const int id = hit.x, row = hit.y;
                    for (int p = lds.head[hash_of(id) >> 24]; p != 0; p = lds.next[p - 1])
                        if (lds.uid[p - 1] == id) {
                            atomicAnd(&lds.want[row * kw + ((p - 1) >> 5)], ~(1u << ((p - 1) & 31)));
                            break;
                        }
                }
                __syncthreads();
            }
        };
        auto probe = [&](int id, int row, u32 word) {      // word: the id's word of hash bits
            const bool hit = (word >> ((hash_of(id) >> 20) & 31)) & 1u;
            const u64 mask = __ballot(hit);
            if (hit) lds.hits[n_hits + lanes_below(mask)] = make_int2(id, row);
            n_hits += __popcll(mask);
        };
        auto bits_of = [&](int id) { return lds.bits[hash_of(id) >> 25]; };
        if (QUADS || K >= 4) {      // (rows at any multiple of four bytes; the last load of a row may repeat ids)
            const int kq = QUADS ? K >> 2 : (K + 3) >> 2, total = n_rows * kq;
            for (int f0 = lane; f0 - lane < total; f0 += 8 * EF_WAVE) {
                int4 four[8];
                int rr[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int f = min(f0 + q * EF_WAVE, total - 1);
                    const int at = kq == 1 ? f : (int)(((u64)(u32)f * kq_magic) >> 32);
                    rr[q] = lds.rows[at];
                    const int *row = gid + (size_t)lds.uid[rr[q]] * K;
                    if (QUADS) {
                        four[q] = *reinterpret_cast<const int4 *>(row + 4 * (f - at * kq));
                    } else {
                        const ef_i32x4_u v = *reinterpret_cast<const ef_i32x4_u *>(row + min(4 * (f - at * kq), K - 4));
                        four[q] = make_int4(v.x, v.y, v.z, v.w);
                    }
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    if (f0 - lane + q * EF_WAVE >= total) break;
                    // (lanes beyond the end have the last load again: its hits are settled twice, to the same effect)
                    const int id4[4] = {four[q].x, four[q].y, four[q].z, four[q].w};
                    u32 word[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) word[t] = bits_of(id4[t]);
#pragma unroll
                    for (int t = 0; t < 4; ++t) probe(id4[t], rr[q], word[t]);
                    settle(EF_WAVE - 1);
                }
            }
        } else {
            for (int f0 = lane; f0 - lane < n_rows * K; f0 += EF_WAVE) {
                const int f = min(f0, n_rows * K - 1), at = K == 1 ? f : (int)(((u64)(u32)f * k_magic) >> 32), row = lds.rows[at];
                const int id = gid[(size_t)lds.uid[row] * K + (f - at * K)];
                probe(id, row, bits_of(id));
                settle(EF_WAVE - 1);
            }
        }
        settle(0);
        return n_rows;
    };
    // (one place that drains the queue: a copy of the insertion per place cost registers in all of the kernel)
    for (bool end = false; !end;) {
        end = w >= count;      // (one turn more: what is left in the queue)
        const int n_rows = end ? 0 : wants_of(work[w]);
        w += gridDim.x;
        const int lane = ef_opaque(threadIdx.x), r16 = lane & 15, g = lane >> 4;
        // ---- 3. what is left: sixteen wants per round, four lanes each -----------------------------
        int n_items = 0;
        auto round = [&](int first, int n_r) {      // wants first .. first + n_r - 1 (at most sixteen)
            const bool mine = r16 < n_r && g == 0;
            const u32 ent = lds.items[first + min(r16, n_r - 1)];
            const int a = ent >> 8, b = ent & 255;
            const int ia = lds.uid[a], ib = lds.uid[b];
            float4 va[8], vb[8];
            load_row<ALIGNED>(va, X + (size_t)ia * d, g, d);
            load_row<ALIGNED>(vb, X + (size_t)ib * d, g, d);
            float p[4] = {0.f, 0.f, 0.f, 0.f};
            accumulate_pair(va, vb, (d + 15) >> 4, p);
            // partial sum l lives in lane g = l / 4, slot l % 4 (see join_reg_kernel)
            const float dist = ef_sum_partials(p[0], p[1], p[2], p[3]);
            const bool take = mine && __float_as_uint(dist) <= lds.thr[a];
            const u64 mask = __ballot(take);
            if (take) {
                Proposal &pr = lds.queue[q_fill + lanes_below(mask)];
                pr.key = ef_pack(dist, ib, mark);
                pr.target = ia;
            }
            q_fill += __popcll(mask);
            __syncthreads();
        };
        bool more = true;
        for (int f0 = 0; more; f0 += EF_WAVE) {
            more = f0 + EF_WAVE < n_rows * kw;
            const int f = f0 + lane, at = f / kw, c0 = 32 * (f - at * kw);
            int row = 0;
            u32 left = 0;
            if (f < n_rows * kw) {
                row = lds.rows[at];
                left = lds.want[row * kw + (f - at * kw)];
            }
            for (u64 mask = ~0ULL; mask != 0;) {      // a bit per lane at a time
                mask = __ballot(left != 0);
                if (left) {
                    lds.items[n_items + lanes_below(mask)] = (unsigned short)(row << 8 | (c0 + __ffs(left) - 1));
                    left &= left - 1;
                }
                n_items += __popcll(mask);
                __syncthreads();
                const int keep = more || mask ? EF_WAVE - 1 : 0;
                for (;;) {
                    if (q_fill > (end ? 0 : kTileQueue - 16)) drain();      // (a round adds at most one proposal per want)
                    if (n_items <= keep) break;
                    const int n_r = min(n_items, 16);
                    n_items -= n_r;
                    round(n_items, n_r);
                }
            }
        }
        __syncthreads();
    }
    updates = ef_wave_sum_i32(updates);
    if (lane == 0) upd_block[blockIdx.x] = updates + (mode == 2 ? upd_block[blockIdx.x] : 0);      // (mode 2 follows mode 1)
}

// The ids of all graph entries (-1 for an empty slot), written once per iteration after the
// sampling: the tile join looks for pairs that already know each other in these, at half the
// bytes of the entries themselves, and notes the ids it inserts there as well.  An id that is or
// was in a row is all the table of known pairs asks for: the mirror may lag behind the rows.
__global__ void __launch_bounds__(kBlock) graph_ids_kernel(const u64 *__restrict__ graph, size_t total, int *__restrict__ gid)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (size_t)gridDim.x * kBlock) {
        const u64 e = graph[i];
        gid[i] = ef_is_empty(e) ? -1 : ef_id(e);
    }
}

// squared norms in float32 (only the LDS join's filter uses them; any summation order will do).
// A group of sixteen lanes per point, points strided over the grid.
__global__ void __launch_bounds__(kBlock)
norms_kernel(const float *__restrict__ X, int n, int d, float *__restrict__ norms)
{
    const int gl = threadIdx.x & 15;
    const size_t n_groups = (size_t)gridDim.x * (kBlock / 16);
    for (size_t g = ((size_t)blockIdx.x * kBlock + threadIdx.x) >> 4; g < (size_t)n; g += n_groups) {
        const float *a = X + g * d;
        float acc = 0.0f;
        for (int j = gl; j < d; j += 16) acc = __builtin_fmaf(a[j], a[j], acc);
        acc = ef_group_reduce16(acc);
        if (gl == 0) norms[g] = acc;
    }
}

// Only the bits of the largest |coordinate|, for the joins that take their norms from Gram diagonals: one
// pass at full width (the norms took 151 us for 10^6 x 128, this 93).  xmax is zeroed beforehand.
__global__ void __launch_bounds__(kBlock)
xmax_kernel(const float *__restrict__ X, size_t total, u32 *xmax)
{
    const size_t step = (size_t)gridDim.x * kBlock, quads = total / 4;
    float m = 0.f;
    for (size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x; q < quads; q += 4 * step) {
        float4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            v[k] = load_unaligned4(X + 4 * min(q + k * step, quads - 1));
#pragma unroll
        for (int k = 0; k < 4; ++k) m = fmaxf(fmaxf(fmaxf(m, fabsf(v[k].x)), fmaxf(fabsf(v[k].y), fabsf(v[k].z))), fabsf(v[k].w));
    }
    if (blockIdx.x == 0 && threadIdx.x < (total & 3)) m = fmaxf(m, fabsf(X[4 * quads + threadIdx.x]));
    u32 b = __float_as_uint(m);
    for (int o = 32; o >= 1; o >>= 1) b = max(b, (u32)__shfl_xor((int)b, o, EF_WAVE));
    __shared__ u32 wave_max[kBlock / EF_WAVE];
    if (ef_lane() == 0) wave_max[threadIdx.x / EF_WAVE] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < kBlock / EF_WAVE; ++v) b = max(b, wave_max[v]);
        atomicMax(xmax, b);
    }
}

// per-iteration counters from the per-block partial sums: part[b] = (pairs evaluated, vectors
// gathered, vectors gathered by the smallest join class) of prepare block b; upd_block: insertions
// per join block
// (a block of 1024 threads per 2048 partial sums, 64 blocks at most - 33 for 10^6 points of degree 10: with 16 blocks of
// 256 a thread had thirty loads one after the other, 12 us for 10^6 points)
constexpr int kStatsThreads = 1024;
__global__ void __launch_bounds__(kStatsThreads)
stats_kernel(const long long *__restrict__ part, int n_part, const int *__restrict__ upd_block, int n_upd_block, u64 *stats)
{
    long long sum[4] = {0, 0, 0, 0};      // pairs, insertions, vectors, vectors of the smallest class
    const int t = blockIdx.x * kStatsThreads + threadIdx.x, nt = gridDim.x * kStatsThreads;
    for (int b = t; b < n_part; b += nt) {
        sum[0] += part[(size_t)b * 3];
        sum[2] += part[(size_t)b * 3 + 1];
        sum[3] += part[(size_t)b * 3 + 2];
    }
    for (int b = t; b < n_upd_block; b += nt) sum[1] += upd_block[b];
    __shared__ long long wave_sum[4][kStatsThreads / EF_WAVE];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        sum[q] = ef_wave_sum_i64(sum[q]);
        if (ef_lane() == 0) wave_sum[q][threadIdx.x / EF_WAVE] = sum[q];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        long long all = 0;
        for (int v = 0; v < kStatsThreads / EF_WAVE; ++v) all += wave_sum[threadIdx.x][v];
        atomicAdd(stats + threadIdx.x, (u64)all);
    }
}

// number of graph entries carrying the new mark (early termination)
__global__ void __launch_bounds__(kBlock) count_new_kernel(const u64 *__restrict__ graph, size_t total, u64 *out)
{
    __shared__ int wave_cnt[kBlock / EF_WAVE];
    int mine = 0;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (size_t)gridDim.x * kBlock) {
        const u64 e = graph[i];
        mine += (e & 1) && !ef_is_empty(e) ? 1 : 0;
    }
    mine = ef_wave_sum_i32(mine);
    if (ef_lane() == 0) wave_cnt[threadIdx.x / EF_WAVE] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int w = 0; w < kBlock / EF_WAVE; ++w) tot += wave_cnt[w];
        if (tot) atomicAdd(out, (u64)tot);
    }
}

__global__ void zero_u64_kernel(u64 *p, int count)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

// ---------------------------------------------------------------------------------------
// rows in and out

__global__ void __launch_bounds__(kBlock)
get_graph_kernel(const u64 *__restrict__ graph, int n, int K, int *__restrict__ ids,
                 float *__restrict__ dists, unsigned char *__restrict__ flags)
{
    __shared__ u64 keys_sh[kBlock / EF_WAVE][2 * EF_WAVE];
    const int wave = threadIdx.x / EF_WAVE, lane = ef_lane();
    const int i = blockIdx.x * (kBlock / EF_WAVE) + wave;
    u64 *keys = keys_sh[wave];
    u64 e[2] = {~0ULL, ~0ULL};
    if (i < n) {
        if (lane < K) e[0] = graph[(size_t)i * K + lane];
        if (lane + EF_WAVE < K) e[1] = graph[(size_t)i * K + lane + EF_WAVE];
    }
    keys[lane] = e[0];
    keys[lane + EF_WAVE] = e[1];
    __syncthreads();
    if (i >= n) return;
    int rank[2] = {0, 0};
    for (int k = 0; k < K; ++k) {
        const u64 o = keys[k];
        rank[0] += o < e[0] ? 1 : 0;
        rank[1] += o < e[1] ? 1 : 0;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (lane + h * EF_WAVE >= K) continue;
        const size_t dst = (size_t)i * K + rank[h];
        const bool empty = ef_is_empty(e[h]);
        ids[dst] = empty ? -1 : ef_id(e[h]);
        dists[dst] = empty ? __uint_as_float(EF_INF_BITS) : __uint_as_float(ef_dist_bits(e[h]));
        if (flags) flags[dst] = empty ? 0 : (unsigned char)(e[h] & 1);
    }
}

// Rows of at most G entries: a group of G lanes per row, ranks by broadcast inside the group.
template <int G>
__global__ void __launch_bounds__(kBlock)
get_graph_group_kernel(const u64 *__restrict__ graph, int n, int K, int *__restrict__ ids,
                       float *__restrict__ dists, unsigned char *__restrict__ flags)
{
    const int gl = threadIdx.x & (G - 1);
    const size_t i = ((size_t)blockIdx.x * kBlock + threadIdx.x) / G;
    const bool mine = i < (size_t)n && gl < K;
    const u64 e = mine ? graph[i * K + gl] : ~0ULL;
    int rank = 0;
    for (int k = 0; k < K; ++k) rank += __shfl(e, k, G) < e ? 1 : 0;
    if (!mine) return;
    const size_t dst = i * K + rank;
    const bool empty = ef_is_empty(e);
    ids[dst] = empty ? -1 : ef_id(e);
    dists[dst] = empty ? __uint_as_float(EF_INF_BITS) : __uint_as_float(ef_dist_bits(e));
    if (flags) flags[dst] = empty ? 0 : (unsigned char)(e & 1);
}

// Rows hold distinct entries: the ranks of sampling and of get_graph, and the insertions, rely on it (two entries
// of one key have the same rank, and the place after it would keep what was there before).  A random start may
// draw an id twice, so an id that an earlier slot of the row names leaves its slot empty.  A thread per slot of the
// block's kBlock / K rows; the threads of a row walk its slots together, in LDS.  (Without and with the walk: 10^6 rows
// of 10 35 and 52 us, of 100 0.38 and 1.09 ms, vector instructions.  Four ids per LDS read, or eight reads in
// flight: 1.4 ms and 1.3.)
__global__ void __launch_bounds__(kBlock)
set_graph_kernel(u64 *graph, size_t n, int K, const int *__restrict__ ids, const float *__restrict__ dists,
                 const unsigned char *__restrict__ flags)
{
    __shared__ int id_sh[kBlock];
    const int t = threadIdx.x, rows = kBlock / K, r = t / K, slot = t - r * K;
    const size_t i = (size_t)blockIdx.x * rows + r;
    const bool mine = r < rows && i < n;
    const int id = mine ? ids[i * K + slot] : -1;
    id_sh[t] = id;
    __syncthreads();
    if (!mine) return;
    bool ok = id >= 0 && (size_t)id < n;
    for (int s = 0; s < slot; ++s) ok &= id_sh[r * K + s] != id;
    graph[i * K + slot] = ok ? ef_pack(dists[i * K + slot], id, flags ? flags[i * K + slot] : 1) : ef_empty_entry(slot);
}

__global__ void pair_distances_kernel(const float *__restrict__ X, int d,
                                      const int *__restrict__ a_ids, const int *__restrict__ b_ids,
                                      size_t m, float *__restrict__ out)
{
    const size_t g = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
    const int gl = threadIdx.x & 15;
    const size_t gc = g < m ? g : m - 1;   // keep every lane of a group active
    const float *a = X + (size_t)a_ids[gc] * d, *b = X + (size_t)b_ids[gc] * d;
    float acc = 0.0f;
    for (int j = gl; j < d; j += 16) {
        float diff = a[j] - b[j];
        acc = __builtin_fmaf(diff, diff, acc);
    }
    acc = ef_group_reduce16(acc);
    if (g < m && gl == 0) out[g] = acc;
}

struct NndWs {
    int *nw, *od, *nw_c, *od_c, *work, *work_count, *rnew_c, *rold_c, *ovf_count, *ulist, *upd_block;
    int2 *ucount;
    void *overflow;
    u64 *rnew, *rold, *list_max, *active, *fresh;
    u32 *offer_runs, *run_table;
    int *gid;      // ids of all graph entries (joins of more than 32 vectors)
    long long *part;
    u32 *worst;
    float *norms;
    u32 *xmax;      // bits of the largest |coordinate| of the data
    size_t bytes;
};

NndWs carve_nnd(void *ws, int64_t n, int K, int L)
{
    char *p = (char *)ws;
    size_t off = 0;
    NndWs w;
    auto take = [&](size_t bytes) {
        char *r = p ? p + off : nullptr;
        off += align_up(bytes);
        return r;
    };
    w.nw = (int *)take((size_t)n * L * 4);
    w.od = (int *)take((size_t)n * K * 4);
    w.nw_c = (int *)take((size_t)n * 4);
    w.od_c = (int *)take((size_t)n * 4);
    w.part = (long long *)take(((size_t)n / EF_WAVE + 1) * 3 * 8);      // prepare blocks hold >= 64 points
    const int n_lists = join_classes(K + 2 * L, true).n;      // (without the register joins there are no more lists)
    w.work = (int *)take((size_t)n * n_lists * 4);
    w.work_count = (int *)take(kMaxClasses * 4);     // list sizes
    w.rnew_c = (int *)take((size_t)n * 4);
    w.rold_c = (int *)take((size_t)n * 4);
    // reverse lists: either the overflow queues of the counter scheme or the offer runs and
    // their table of the bucket scheme
    const bool bkt = bucketed_lists(n, K, L);
    const size_t n_bkt = (size_t)(n + kBktRows - 1) / kBktRows, n_buckets = (size_t)((n - 1) >> bucket_shift(L)) + 1;
    w.overflow = take(bkt ? 0 : ovf_region_for(n, K) * kOvfQueues * sizeof(Overflow));
    w.offer_runs = (u32 *)take(bkt ? n_bkt * kBktRows * (size_t)(K > L ? K : L) * 4 : 0);
    w.run_table = (u32 *)take(bkt ? n_buckets * n_bkt * 4 : 0);
    w.ovf_count = (int *)take((size_t)kOvfQueues * kOvfCounterPitch * 4);
    w.ulist = (int *)take((size_t)n * (K + 2 * L) * 4);
    w.ucount = (int2 *)take((size_t)n * 8);
    w.upd_block = (int *)take((size_t)(2 * kRegGrid + (n_lists - 2) * kMaxLargeGrid) * 4);
    w.rnew = (u64 *)take((size_t)n * L * 8);
    w.rold = (u64 *)take((size_t)n * L * 8);
    // (32-bit sources fill the first half; the table of many small runs lies behind them)
    if (bkt && bucket_shape(n, K, L).table_behind) w.run_table = (u32 *)w.rold + (size_t)n * L;
    BucketShape wide;
    if (wide_lists(n, K, L, &wide)) {
        w.offer_runs = (u32 *)w.overflow;
        w.run_table = w.offer_runs + (((size_t)(K > L ? K : L) << wide.row_bits) * wide.blocks);
    }
    w.list_max = (u64 *)take((size_t)n * 2 * 8);
    w.active = (u64 *)take((size_t)(n + 63) / 64 * 8);
    w.fresh = (u64 *)take(8);
    w.worst = (u32 *)take((size_t)n * 4);
    w.norms = (float *)take((size_t)n * 4);
    w.xmax = (u32 *)take(8);
    w.gid = (int *)take(K + 2 * L > 32 ? (size_t)n * K * 4 : 0);
    w.bytes = off;
    return w;
}

constexpr size_t kLdsLimit = 160 * 1024;

inline u32 q4_magic_for(int d)
{
    const u64 q4 = (u64)((d + 3) >> 2);
    return q4 == 1 ? 0xFFFFFFFFu : (u32)(((1ULL << 32) + q4 - 1) / q4);
}

inline int grid_for(size_t total, int block) { return (int)((total + block - 1) / block); }

}  // namespace

extern "C" const char *efanna_status_string(int status)
{
    switch (status) {
    case EFANNA_OK: return "ok";
    case EFANNA_EINVAL: return "invalid argument";
    case EFANNA_EWORKSPACE: return "workspace missing, misaligned or too small";
    case EFANNA_EINPUT: return "input holds a non-finite value or |x| >= 2^20";
    case EFANNA_EHIP: return "HIP runtime error";
    case EFANNA_ECAPACITY: return "more leaves than max_leaves";
    case EFANNA_EUNSUPPORTED: return "shape not supported by this build";
    case EFANNA_ESCRATCH: return "input needs more scratch memory than the library's fixed array holds";
    default: return "unknown status";
    }
}

extern "C" size_t efanna_init_workspace_bytes(int64_t n, int32_t levels)
{
    if (n < 1) return 0;
    // one leaf index per point and visited level above the leaves
    return levels > 0 ? align_up((size_t)n * (size_t)levels * 4) : 256;
}

extern "C" int efanna_init_graph(const float *X, int64_t n, int32_t d, const int32_t *perm,
                                 const int32_t *leaf_off, int32_t max_leaves,
                                 const int32_t *n_leaves, const efanna_node *nodes,
                                 const int32_t *leaf_up, int32_t tree_depth,
                                 int32_t conquer_depth, int32_t n_trees,
                                 int32_t leaf_size, int32_t k, efanna_entry *graph_, void *ws,
                                 size_t ws_bytes, void *stream)
{
    if (!X || !perm || !leaf_off || !n_leaves || !graph_ || (!nodes) != (!leaf_up)) return EFANNA_EINVAL;
    if (nodes && conquer_depth < 0) return EFANNA_EINVAL;
    if (n < 2 || d < 1 || n_trees < 1 || n_trees > EFANNA_MAX_TREES || leaf_size < 1 ||
        leaf_size > EFANNA_MAX_LEAF || k < 1 || k > EFANNA_MAX_K || k >= n || max_leaves < 1 ||
        n >= 2147483647LL - 256)
        return EFANNA_EINVAL;
    // levels above the leaves that the conquer step visits (none without nodes)
    const int levels = nodes ? (tree_depth - conquer_depth + 1 > 64 ? 64 : tree_depth - conquer_depth + 1) : 0;
    if (nodes && tree_depth - conquer_depth + 1 > 64) return EFANNA_EUNSUPPORTED;
    if (!ws || ((uintptr_t)ws & 255) || ws_bytes < efanna_init_workspace_bytes(n, levels))
        return EFANNA_EWORKSPACE;
    if (n * (int64_t)k >= 2147483647LL) return EFANNA_EINVAL;   // LDS row indices are 32-bit
    for (int t = 0; t < n_trees; ++t)
        if (n_leaves[t] < 1 || n_leaves[t] > max_leaves) return EFANNA_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    u64 *const graph = (u64 *)graph_;
    const int stride = d + kRowPad;
    const size_t lds = (size_t)(align4(leaf_size * stride) + align4(leaf_size * leaf_size)) * 4 +
                       (size_t)leaf_size * k * 8 + (size_t)leaf_size * (leaf_size + 1) * 8 +
                       (size_t)leaf_size * 8;
    // (a block per leaf and, with leaves of 64 and rows of 100, one block per CU: sixteen waves
    // of it keep the CU busy through the loads of the rows)
    const int block_threads = 4 * EF_WAVE * ((leaf_size + 15) / 16);
    // Leaves of at most 16 points: rows in registers, with 16-byte loads at any multiple of four
    // bytes where rows are not aligned.  (Below four coordinates a row is shorter than a load.)
    const bool aligned = d % 4 == 0 && ((uintptr_t)X & 15) == 0;
    const bool reg_ok = leaf_size <= 16 && (aligned || d >= 4);
    if (leaf_size > EF_WAVE) return EFANNA_EUNSUPPORTED;
    if (!aligned && lds > kLdsLimit) return EFANNA_EUNSUPPORTED;      // (the documented limit of unaligned rows)
    if (reg_ok) {
        const size_t reg_lds = (size_t)16 * k * 8 + (size_t)16 * kCandPitch * 8 + 16 * 4;
        const size_t conquer_lds = (size_t)2 * 16 * k * 8 + (size_t)16 * kCandPitch * 8 + 16 * 16 * 4;
        const size_t conquer_tile_lds = (size_t)2 * 16 * k * 8 + (size_t)16 * kCandPitch * 8 + (64 + 32 + 16 + 16) * 4 + 512;
        for (int t = 0; t < n_trees; ++t) {
            const int32_t *perm_t = perm + (size_t)t * n, *off_t = leaf_off + (size_t)t * (max_leaves + 1);
            if (aligned)
                init_reg_kernel<true><<<min(n_leaves[t], kLeafGrid), EF_WAVE, reg_lds, st>>>(
                    X, d, perm_t, off_t, n_leaves[t], k, graph, t == 0);
            else
                init_reg_kernel<false><<<min(n_leaves[t], kLeafGrid), EF_WAVE, reg_lds, st>>>(
                    X, d, perm_t, off_t, n_leaves[t], k, graph, t == 0);
            if (levels > 0) {
                int *etab = (int *)ws;
                classify_kernel<<<min(grid_for((size_t)n_leaves[t], kBlock / EF_WAVE), 256 * 8), kBlock, 0, st>>>(
                    X, d, perm_t, off_t, n_leaves[t], nodes + (size_t)t * (max_leaves + 1),
                    leaf_up + (size_t)t * (max_leaves + 1), conquer_depth, levels, etab);
                const int grid = min(n_leaves[t], kLeafGrid);
                if (d <= 128 && aligned)
                    conquer_tile_kernel<true><<<grid, EF_WAVE, conquer_tile_lds, st>>>(
                        X, d, perm_t, off_t, n_leaves[t], etab, levels, k, f16_filter(d), graph);
                else if (d <= 128)
                    conquer_tile_kernel<false><<<grid, EF_WAVE, conquer_tile_lds, st>>>(
                        X, d, perm_t, off_t, n_leaves[t], etab, levels, k, f16_filter(d), graph);
                else if (aligned)
                    conquer_kernel<true><<<grid, EF_WAVE, conquer_lds, st>>>(
                        X, d, perm_t, off_t, n_leaves[t], etab, levels, k, graph);
                else
                    conquer_kernel<false><<<grid, EF_WAVE, conquer_lds, st>>>(
                        X, d, perm_t, off_t, n_leaves[t], etab, levels, k, graph);
            }
        }
        EF_HIP_CHECK(hipGetLastError());
        return EFANNA_OK;
    }
    if (lds > kLdsLimit) return EFANNA_EUNSUPPORTED;
    EF_HIP_CHECK(hipFuncSetAttribute((const void *)init_tree_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const size_t any_lds = (size_t)(kBlock / EF_WAVE) * (2 * k + EF_WAVE) * 8;
    for (int t = 0; t < n_trees; ++t) {
        const int32_t *perm_t = perm + (size_t)t * n, *off_t = leaf_off + (size_t)t * (max_leaves + 1);
        init_tree_kernel<<<n_leaves[t], block_threads, lds, st>>>(
            X, d, stride, q4_magic_for(d), leaf_size, perm_t, off_t, k, graph, t == 0);
        if (levels > 0) {      // above the leaves: the general kernels (any leaf size up to 64, any d)
            int *etab = (int *)ws;
            classify_any_kernel<<<min(grid_for((size_t)n_leaves[t], kBlock / EF_WAVE), 256 * 8), kBlock, 0, st>>>(
                X, d, perm_t, off_t, n_leaves[t], nodes + (size_t)t * (max_leaves + 1),
                leaf_up + (size_t)t * (max_leaves + 1), conquer_depth, levels, etab);
            conquer_any_kernel<<<min(n_leaves[t], 256 * 64), kBlock, any_lds, st>>>(
                X, d, perm_t, off_t, n_leaves[t], etab, levels, k, graph);
        }
    }
    EF_HIP_CHECK(hipGetLastError());
    return EFANNA_OK;
}

extern "C" size_t efanna_nndescent_workspace_bytes(int64_t n, int32_t k, int32_t sample_L)
{
    if (n < 1 || k < 1 || sample_L < 1) return 0;
    return carve_nnd(nullptr, n, k, sample_L).bytes;
}

namespace {

// Scratch of the entry point that allocates nothing: device memory that the code object
// brings along, one copy per GPU.  Host code never uses the array's name as an address (on
// the host it is only a handle for hipGetSymbolAddress): the address on each device is
// looked up once, with that device current, and kept.
__device__ __align__(256) unsigned char noalloc_scratch[EFANNA_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::atomic<void *> noalloc_scratch_ptr[kMaxDevices];

// The scratch array's address on the current device (nullptr and a status on failure).
int noalloc_scratch_address(void **out)
{
    *out = nullptr;
    int dev = -1;
    EF_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return EFANNA_EUNSUPPORTED;
    void *p = noalloc_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        EF_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc_scratch)));
        if (!p) return EFANNA_EHIP;
        noalloc_scratch_ptr[dev].store(p, std::memory_order_release);      // racing callers store the same address
    }
    *out = p;
    return EFANNA_OK;
}

int nndescent_run(const float *X, int64_t n, int32_t d, int32_t k, efanna_entry *graph_, int32_t iters,
                  int32_t sample_L, uint64_t seed, int32_t first_iter, float delta, int32_t cross_old,
                  int32_t *iters_done, uint64_t *stats_, float *phase_ms, void *ws, size_t ws_bytes, void *stream);

}  // namespace

extern "C" int efanna_nndescent(const float *X, int64_t n, int32_t d, int32_t k,
                                efanna_entry *graph_, int32_t iters, int32_t sample_L,
                                uint64_t seed, int32_t first_iter, float delta, int32_t cross_old,
                                int32_t *iters_done, uint64_t *stats_, float *phase_ms, void *ws,
                                size_t ws_bytes, void *stream)
{
    return nndescent_run(X, n, d, k, graph_, iters, sample_L, seed, first_iter, delta, cross_old, iters_done,
                         stats_, phase_ms, ws, ws_bytes, stream);
}

extern "C" int efanna_nndescent_noalloc(const float *X, int64_t n, int32_t d, int32_t k,
                                        efanna_entry *graph_, int32_t iters, int32_t sample_L,
                                        uint64_t seed, int32_t first_iter, uint64_t *stats_,
                                        void *stream)
{
    if (n < 1 || k < 1 || sample_L < 1) return EFANNA_EINVAL;
    if (efanna_nndescent_workspace_bytes(n, k, sample_L) > (size_t)EFANNA_NOALLOC_SCRATCH_BYTES)
        return EFANNA_ESCRATCH;
    void *scratch = nullptr;
    const int rc = noalloc_scratch_address(&scratch);
    if (rc != EFANNA_OK) return rc;
    // no early termination (it reads a counter back after every iteration) and no phase timing
    // (it creates events): neither allocates device memory, but both make the call wait
    return nndescent_run(X, n, d, k, graph_, iters, sample_L, seed, first_iter, 0.0f, 0, nullptr, stats_,
                         nullptr, scratch, (size_t)EFANNA_NOALLOC_SCRATCH_BYTES, stream);
}

namespace {

int nndescent_run(const float *X, int64_t n, int32_t d, int32_t k, efanna_entry *graph_, int32_t iters,
                  int32_t sample_L, uint64_t seed, int32_t first_iter, float delta, int32_t cross_old,
                  int32_t *iters_done, uint64_t *stats_, float *phase_ms, void *ws, size_t ws_bytes, void *stream)
{
    if (iters_done) *iters_done = 0;
    if (!X || !graph_ || !(delta >= 0.0f)) return EFANNA_EINVAL;
    u64 *const graph = (u64 *)graph_;
    u64 *const stats = (u64 *)stats_;
    if (n < 2 || d < 1 || k < 1 || k > EFANNA_MAX_K || k >= n || iters < 0 || sample_L < 1 ||
        sample_L > EFANNA_MAX_SAMPLE || first_iter < 0 || n >= 2147483647LL - 256)
        return EFANNA_EINVAL;
    if (!ws || ((uintptr_t)ws & 255) || ws_bytes < efanna_nndescent_workspace_bytes(n, k, sample_L))
        return EFANNA_EWORKSPACE;
    const int K = k, L = sample_L;
    const int dpad = (d + 15) & ~15;
    const int stride = dpad + kRowPad;
    // a join gathers at most K + 2L vectors: new and old sets together come from one row
    // of K entries, each reverse list adds at most L
    const int max_rows = K + 2 * L;
    // work lists: joins of at most 16 and at most 32 vectors run from register operands, the rest
    // tile by tile or through LDS row buffers, one launch per size class
    const bool aligned = (d & 3) == 0 && ((uintptr_t)X & 15) == 0;
    const bool reg_ok = aligned || d >= 4;
    const int rows1 = reg_ok ? 32 : 0;
    const JoinClasses jc = join_classes(max_rows, reg_ok);
    // (a work list has n entries at most: of few points more blocks would only start and end)
    // (Vectors of at most 160 coordinates, up to 2^17 points: half the blocks, where starting them is what late
    // iterations take.  Joins of at most 32, all blocks and half: 50 000 x 32, degree 10 522 and 495 us, 131 072 x 32 982 and
    // 948, 131 072 x 128 1255 and 1242, degree 20 2989 and 2980, 10^5 x 133, degree 7 966 and 938; beyond, 250 000 x 32 1605
    // both, 250 000 x 128 2124 and 2135, degree 20 5314 and 5358.  Longer vectors: 10^5 x 200, degree 12 1601 and 1607,
    // 50 000 x 960, degree 10 2140 and 2168, 10^5 x 960 4170 and 4220, degree 4 1651 and 1736.)
    const int reg_grid = (int)min(n, (int64_t)(d <= 160 && n <= (1 << 17) ? kRegGrid / 2 : kRegGrid));
    struct Shape {
        int cap_rows, threads, s_cap, q_cap, grid;
        size_t lds;
    };
    auto shape_for = [&](int cap_rows) {
        Shape sh;
        sh.cap_rows = cap_rows;
        const long blocks = (long)((cap_rows + 15) / 16) * ((cap_rows + 15) / 16);
        sh.threads = blocks <= 2 ? 64 : (blocks <= 9 ? 128 : (blocks <= 36 ? 256 : 512));
        const long pairs = (long)cap_rows * (cap_rows - 1) / 2;
        for (bool fits = false; !fits; sh.threads /= 2) {
            const int n_waves = sh.threads / EF_WAVE;
            // a round of blocks adds at most 256 survivors per wave, and the list is emptied
            // whenever the next round might not fit; more room means fewer drains
            sh.s_cap = 256 * n_waves;
            if (pairs > sh.s_cap && pairs <= 1024) sh.s_cap = align4((int)pairs);
            if (cap_rows <= 16) sh.s_cap = 128;     // a single block of at most 120 pairs
            // (pairs that a row already knows are not queued: a few hundred proposals per join at most)
            for (sh.q_cap = min(4 * sh.threads, 512); sh.q_cap >= 128 && !fits; sh.q_cap /= 2) {
                sh.lds = join_lds_floats(cap_rows, stride, sh.s_cap) * 4 +
                         (size_t)sh.q_cap * sizeof(Proposal);
                fits = sh.lds <= kLdsLimit;
                if (fits) break;
            }
            if (fits || sh.threads == EF_WAVE) break;
        }
        const int n_waves = sh.threads / EF_WAVE;
        // persistent grid: as many blocks as fit the 256 CUs at once, twice over
        long per_cu = (long)(kLdsLimit / sh.lds);
        const long by_waves = 32 / n_waves;
        if (per_cu > by_waves) per_cu = by_waves;
        if (per_cu < 1) per_cu = 1;
        sh.grid = (int)(256 * per_cu * 2);
        return sh;
    };
    Shape large[kMaxClasses];
    size_t large_lds = 0;
    for (int c = 2; c < jc.n; ++c) {
        large[c] = shape_for(jc.bound[c]);
        large_lds = large[c].lds > large_lds ? large[c].lds : large_lds;
    }
    // joins of more than 32 vectors: register tiles for vectors of at most 128 coordinates, else rows in LDS
    const bool tiles = reg_ok && d <= 128;
    if (!tiles && max_rows > rows1 && large_lds > kLdsLimit) return EFANNA_EUNSUPPORTED;
    if (!aligned && shape_for(max_rows).lds > kLdsLimit) return EFANNA_EUNSUPPORTED;      // (the documented limit of unaligned rows)
    // joins of at most 16 vectors from registers (d <= 128): room for a whole point's proposals
    // (240) above the drain mark; joins of 17..32 drain between rounds as well (256 entries measured 3 % faster
    // than 128, 512 no better).  Long vectors: room on top of a pass for the 240 proposals of 16 vectors, and for
    // the 552 of 24 vectors or the 440 of eight new members and 24 others; only the rest drains in between.
    auto reg_q_cap_for = [&](int R) { return R == 16 ? (d <= 128 ? 512 : 320) : (d <= 128 ? 256 : 640); };
    static_assert(EF_WAVE + (16 + kFewRest) * (15 + kFewRest) <= 640 && EF_WAVE + kFewNew * (kFewNew - 1 + 2 * (32 - kFewNew)) <= 640 &&
                  EF_WAVE + 16 * 15 <= 320, "queue");
    auto reg_lds = [&](int R) {
        const int reg_q_cap = reg_q_cap_for(R);
        return (size_t)(6 * R + (d <= 128 ? align4(R * (R - 1) / 2 + 8) : 0)) * 4 +
               (size_t)reg_q_cap * sizeof(Proposal);
    };
    // prepare: one thread per point with max_rows ids of LDS each
    int prep_threads = (int)(kPrepLds / ((size_t)(max_rows | 1) * 4)) / EF_WAVE * EF_WAVE;
    prep_threads = prep_threads > kBlock ? kBlock : (prep_threads < EF_WAVE ? EF_WAVE : prep_threads);
    const size_t prep_lds = (size_t)prep_threads * (max_rows | 1) * 4;
    // long lists: a wave per point with a hash table of at least twice the longest list
    const bool prep_wave = max_rows > 96;
    int prep_hash = 128;
    while (prep_hash < 2 * max_rows) prep_hash <<= 1;
    const size_t prep_wave_lds = (size_t)(kBlock / EF_WAVE) * (prep_hash + max_rows + EF_WAVE) * 4;
    const int prep_wave_grid = min(grid_for((size_t)n, kBlock), 256 * 8);
    // short lists: eight lanes per point, as many points per block as keep a thousand blocks busy
    const bool prep_group = bucketed_lists(n, K, L);
    int prep_passes = 1;
    while (prep_passes < kPrepMaxPasses && n > (int64_t)kPrepPoints * prep_passes * 512 &&
           (size_t)kPrepPoints * 2 * prep_passes * (max_rows | 1) * 4 <= kPrepLds)
        prep_passes *= 2;
    const size_t prep_group_lds = (size_t)kPrepPoints * prep_passes * (max_rows | 1) * 4;
    const int n_part = prep_group  ? grid_for((size_t)n, kPrepPoints * prep_passes)
                       : prep_wave ? prep_wave_grid
                                   : grid_for((size_t)n, prep_threads);
    // filter margins: Gram-form rounding error <= (2*dpad + 4) u (|a|^2 + |b|^2), u = 2^-24,
    // doubled; the fixed-order distance is within (d/16 + 8) u of the true one, doubled twice
    const float margin_rel = (float)((4.0 * dpad + 16.0) * 5.9604644775390625e-08);
    const float thr_scale = (float)(1.0 + 4.0 * (d / 16.0 + 8.0) * 5.9604644775390625e-08);
    // The register joins filter with Gram blocks of the vectors in half precision, rounded towards
    // zero after a scaling by a power of two that keeps them below 2^15: a coordinate moves by at
    // most 2^-10 of itself or, below 2^-14, by 2^-24.  The blocks' diagonals are the rounded
    // vectors' squared norms, so the filter's left side is the squared distance D'^2 of the rounded
    // vectors up to the accumulation error, and |D' - D| <= r(a) + r(b) with
    // r(x) = u |x'| + r0, u = 2^-10 / (1 - 2^-10) (+ slack for the square root and the norm's own
    // error), r0 = 1.01 sqrt(d) 2^-24.  The margin on the norms pays for the three accumulations in
    // single precision: four times (dpad + 4) 2^-23, a bound that holds whether the matrix unit
    // rounds or truncates its partial sums.
    const F16Filter f16 = f16_filter(d);
    const float margin_f16 = f16.margin, thr_scale_f16 = f16.thr_scale, u_f16 = f16.u, rho0_f16 = f16.rho0;
    hipStream_t st = (hipStream_t)stream;
    NndWs w = carve_nnd(ws, n, K, L);
    // reverse lists by buckets (short rows and lists): LDS of an offer block (words) or a list
    // block (keys) with `per_row` of them per row, and one int per bucket or offer block twice over
    BucketShape bs;
    const bool wide = wide_lists(n, K, L, &bs), bkt = wide || bucketed_lists(n, K, L);
    if (!wide) bs = bucket_shape(n, K, L);
    const int bkt_rows = 1 << bs.row_bits;
    const bool bkt_small = bs.row_bits != 10;
    auto bkt_lds = [&](int per_row) { return (size_t)bkt_rows * per_row * 4 + ((size_t)2 * bs.buckets + 4) * 4; };
    // (degree 20, 100 000 x 64 sorted by norm, four iterations: 6.2 ms with 256 threads, 5.3 with the LDS of 512, 4.9 with 512; 100 000 x 128, not
    // sorted: 4.27, 4.27 and 4.30)
    const bool roomy = !wide && bs.row_bits == 10 && bs.shift == 7 && (K > 10 || L > 10);
    const int lists_area = bkt ? bucket_lists_area(K, L, bs.shift, bs.blocks, bs.threads, wide || roomy ? 2 * kBktWords : kBktWords) : 0;
    const size_t lists_lds = !bkt ? 0 : insert_lists(n, K, L) && !wide ? bucket_lists_lds(L, bs.shift, bs.blocks)
                                   : (size_t)lists_area * 4 + bucket_lists_rest(bs.shift, bs.blocks);
    // lanes that walk a run of `per` offers per row together
    auto run_lanes = [&](int per) {
        const int64_t mean = n * per / ((int64_t)bs.blocks * bs.buckets);
        return mean <= 6 ? 3 : mean <= 14 ? 4 : mean <= 40 ? 5 : 6;
    };
    typedef void (*SampleKernel)(u64 *, int, int, int, int *, int *, int *, int *, u32 *, int, int, u32 *, u32 *);
    typedef void (*ReverseOldKernel)(const int *, int, int, const u64 *, int, int, u32 *, u32 *);
    typedef void (*ListsKernel)(const u32 *, const u32 *, int, int, u64, int, int, int, int, int, u32 *, int *, const int *, u32 *, int *);
    const bool few_rows = bs.row_bits == 6;      // (of a wide offer block)
    const SampleKernel bkt_sample = wide ? (K <= 64 ? (few_rows ? sample_wide_kernel<1, 6> : sample_wide_kernel<1, 8>)
                                                    : (few_rows ? sample_wide_kernel<2, 6> : sample_wide_kernel<2, 8>))
                                    : bkt_small ? (K <= 16 ? sample_bucket_kernel<2, 8> : sample_bucket_kernel<4, 8>)
                                                : (K <= 16 ? sample_bucket_kernel<2, 10> : sample_bucket_kernel<4, 10>);
    const ReverseOldKernel bkt_old = wide ? (few_rows ? reverse_old_wide_kernel<6> : reverse_old_wide_kernel<8>)
                                          : bkt_small ? reverse_old_bucket_kernel<8> : reverse_old_bucket_kernel<10>;
    const ListsKernel bkt_lists =
        wide ? (few_rows ? bucket_lists_kernel<0, 6, true> : bucket_lists_kernel<0, 8, true>)
        : insert_lists(n, K, L) ? (!bkt_small ? bucket_insert_kernel<0, 10> : L == 10 ? bucket_insert_kernel<10, 8> : bucket_insert_kernel<0, 8>)
        : bkt_small ? (L == 10 ? bucket_lists_kernel<10, 8, false> : bucket_lists_kernel<0, 8, false>)
                    : (L == 10 ? bucket_lists_kernel<10, 10, false> : bucket_lists_kernel<0, 10, false>);
    const int offer_threads = wide ? 4 * bkt_rows : bkt_rows;
    if (bkt) {
        EF_HIP_CHECK(hipFuncSetAttribute((const void *)bkt_sample, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bkt_lds(L)));
        EF_HIP_CHECK(hipFuncSetAttribute((const void *)bkt_old, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bkt_lds(K)));
        EF_HIP_CHECK(hipFuncSetAttribute((const void *)bkt_lists, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lists_lds));
    }
    if (max_rows > rows1 && !tiles)
        EF_HIP_CHECK(hipFuncSetAttribute(K >= 2 * EF_WIDE_PIECES ? (const void *)join_kernel<true>
                                                                 : (const void *)join_kernel<false>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)large_lds));
    zero_u64_kernel<<<1, EF_WAVE, 0, st>>>((u64 *)w.xmax, 1);
    // the half-precision filters want the data's magnitude, the joins with rows in LDS its norms, the joins of
    // up to 32 long vectors neither (10^6 x 960: a pass of 1.08 ms less)
    if (tiles) xmax_kernel<<<(int)min((size_t)grid_for((size_t)n * d / 4 + 1, 4 * kBlock), (size_t)256 * 8), kBlock, 0, st>>>(X, (size_t)n * d, w.xmax);
    else if (max_rows > rows1)
        norms_kernel<<<min(grid_for((size_t)n * 16, kBlock), 256 * 8), kBlock, 0, st>>>(X, (int)n, d, w.norms);
    if (stats) zero_u64_kernel<<<grid_for((size_t)iters * 4 + 1, kBlock), kBlock, 0, st>>>(stats, iters * 4);
    // optional phase timing: events around the sampling and the join of every iteration
    struct PhaseEvents {      // destroyed on every way out of the call
        std::vector<hipEvent_t> list;
        ~PhaseEvents()
        {
            for (hipEvent_t e : list) (void)hipEventDestroy(e);
        }
    } events;
    hipEvent_t *ev = nullptr;
    if (phase_ms && iters > 0) {
        events.list.reserve((size_t)iters * 5);
        for (int e = 0; e < iters * 5; ++e) {
            hipEvent_t one;
            EF_HIP_CHECK(hipEventCreate(&one));
            events.list.push_back(one);
        }
        ev = events.list.data();
    }
    int done = 0;
    for (int it = 0; it < iters; ++it) {
        const int g = first_iter + it;
        if (ev) EF_HIP_CHECK(hipEventRecord(ev[5 * it], st));
        // (the bucket scheme writes every list count itself and empties the work lists on the way)
        if (!bkt)
            fill_reverse_kernel<<<grid_for((size_t)n, kBlock), kBlock, 0, st>>>(w.rnew_c, w.rold_c, w.list_max, (size_t)n,
                                                                                w.work_count, w.ovf_count);
        {
            const u64 kn = ef_stream_key(seed, 2 * g), ko = ef_stream_key(seed, 2 * g + 1);
            Overflow *ovf = (Overflow *)w.overflow;
            const size_t ovf_region = ovf_region_for(n, K);
#define EF_SAMPLE(G, E)                                                                          \
    sample_kernel<G, E><<<grid_for((size_t)n * G, kBlock), kBlock, 0, st>>>(                     \
        graph, (int)n, K, L, kn, w.nw, w.od, w.nw_c, w.od_c, w.rnew, w.rnew_c, ovf,              \
        ovf_region, w.ovf_count, w.worst)
#define EF_REVERSE_OLD(G)                                                                        \
    reverse_old_kernel<G><<<grid_for((size_t)n * G, kBlock), kBlock, 0, st>>>(                   \
        w.od, (int)n, K, L, ko, w.active, w.rold, w.rold_c, ovf, ovf_region, w.ovf_count)
            if (bkt) {
                bkt_sample<<<bs.blocks, offer_threads, bkt_lds(L), st>>>(graph, (int)n, K, L, w.nw, w.od, w.nw_c, w.od_c, w.worst,
                                                                   bs.buckets, bs.shift, w.offer_runs, w.run_table);
                bkt_lists<<<bs.buckets, bs.threads, lists_lds, st>>>(w.offer_runs, w.run_table, bs.blocks, bkt_rows * L, kn,
                                                                    (int)n, L, bs.shift, lists_area, run_lanes(L), (u32 *)w.rnew, w.rnew_c, w.nw_c,
                                                                    (u32 *)w.active, w.work_count);
            } else if (K <= 16) EF_SAMPLE(16, 1);
            else if (K <= 32) EF_SAMPLE(32, 1);
            else if (K <= 64) EF_SAMPLE(64, 1);
            else EF_SAMPLE(64, 2);
            if (!bkt) active_kernel<<<grid_for((size_t)n, kBlock), kBlock, 0, st>>>(w.nw_c, w.rnew_c, (int)n, w.active);
            if (bkt) {
                bkt_old<<<bs.blocks, offer_threads, bkt_lds(K), st>>>(w.od, (int)n, K, w.active, bs.buckets, bs.shift, w.offer_runs,
                                                                w.run_table);
                bkt_lists<<<bs.buckets, bs.threads, lists_lds, st>>>(w.offer_runs, w.run_table, bs.blocks, bkt_rows * K, ko,
                                                                    (int)n, L, bs.shift, lists_area, run_lanes(K), (u32 *)w.rold, w.rold_c, nullptr,
                                                                    nullptr, nullptr);
            } else if (K <= 16) EF_REVERSE_OLD(16);
            else if (K <= 32) EF_REVERSE_OLD(32);
            else EF_REVERSE_OLD(64);
#undef EF_SAMPLE
#undef EF_REVERSE_OLD
            if (bkt) {
            } else if (L >= 2 * EF_WIDE_PIECES)
                reverse_overflow_kernel<true><<<dim3(kOvfBlocksPerQueue, kOvfQueues), kBlock, 0, st>>>(
                    ovf, ovf_region, w.ovf_count, (size_t)n, w.rnew, w.rold, w.list_max, L);
            else
                reverse_overflow_kernel<false><<<dim3(kOvfBlocksPerQueue, kOvfQueues), kBlock, 0, st>>>(
                    ovf, ovf_region, w.ovf_count, (size_t)n, w.rnew, w.rold, w.list_max, L);
        }
        const u32 rows_magic = (u32)(((1ULL << 32) + max_rows - 1) / max_rows);
#define EF_PREPARE_GROUP(E)                                                                        \
    prepare_group_kernel<E><<<n_part, kPrepThreads, prep_group_lds, st>>>(                          \
        w.nw, w.od, w.nw_c, w.od_c, (const u32 *)w.rnew, (const u32 *)w.rold, w.rnew_c, w.rold_c,   \
        (int)n, K, L, max_rows, rows_magic, jc, prep_passes, w.ulist, w.ucount, w.work,            \
        w.work_count, w.part)
        if (prep_group) {
            if (K <= 16 && L <= 16) EF_PREPARE_GROUP(2);
            else EF_PREPARE_GROUP(4);
        } else if (prep_wave) {
            auto go = [&](auto kernel, auto *rnew, auto *rold) {
                kernel<<<prep_wave_grid, kBlock, prep_wave_lds, st>>>(
                    w.nw, w.od, w.nw_c, w.od_c, rnew, rold, w.rnew_c, w.rold_c, (int)n, K, L, max_rows, prep_hash, jc,
                    w.ulist, w.ucount, w.work, w.work_count, w.part);
            };
            if (wide) go(prepare_wave_kernel<u32>, (const u32 *)w.rnew, (const u32 *)w.rold);
            else go(prepare_wave_kernel<u64>, (const u64 *)w.rnew, (const u64 *)w.rold);
        } else {
            auto go = [&](auto kernel, auto *rnew, auto *rold) {
                kernel<<<n_part, prep_threads, prep_lds, st>>>(
                    w.nw, w.od, w.nw_c, w.od_c, rnew, rold, w.rnew_c, w.rold_c, (int)n, K, L, max_rows, rows_magic, jc,
                    w.ulist, w.ucount, w.work, w.work_count, w.part);
            };
            if (wide) go(prepare_kernel<u32>, (const u32 *)w.rnew, (const u32 *)w.rold);
            else go(prepare_kernel<u64>, (const u64 *)w.rnew, (const u64 *)w.rold);
        }
#undef EF_PREPARE_GROUP
        if (ev) EF_HIP_CHECK(hipEventRecord(ev[5 * it + 1], st));
        if (tiles && max_rows > rows1)
            graph_ids_kernel<<<min(grid_for((size_t)n * K, kBlock), 256 * 64), kBlock, 0, st>>>(graph, (size_t)n * K, w.gid);
        // One pass over the joins; with cross_old two, all pairs of two new members of every join
        // before any pair of a new and an old one (the phase events are recorded in the last pass:
        // the split by join size then says little).
        const int n_pass = cross_old ? 2 : 1;
        int n_upd = 0;
        for (int pass = 0; pass < n_pass; ++pass) {
        const int mode = cross_old ? 1 + pass : 0;
        n_upd = 0;      // (the joins' counts of insertions, one launch's blocks after the other's)
        const bool timed = ev && pass == n_pass - 1;
        if (reg_ok) {
#define EF_JOIN_REG_K(NB, ONE, LIST, KT, ALIGNED)                                                  \
    join_reg_kernel<NB, ONE, KT, ALIGNED><<<reg_grid, EF_WAVE, reg_lds(16 * NB), st>>>(                     \
        X, d, K, w.work + (size_t)(LIST) * n, w.work_count + (LIST), reg_q_cap_for(16 * NB), \
        (ONE) ? margin_f16 : margin_rel, (ONE) ? thr_scale_f16 : thr_scale, u_f16, rho0_f16,       \
        w.ulist, w.ucount, max_rows, graph, w.worst, w.upd_block + n_upd, mode,                    \
        w.xmax)
    // (a row length of 10 is compiled in: 3 % off the joins of 17..32 vectors; rows of up to sixteen entries in general go
    // in one piece, see ef_bounded_insert_row; -24: see kFewRest's use)
#define EF_JOIN_REG_A(NB, ONE, LIST, ALIGNED)                                                       \
    do {                                                                                           \
        if (K == 10) EF_JOIN_REG_K(NB, ONE, LIST, 10, ALIGNED);                                    \
        else if (!(ONE) && (NB) > 1 && K > 16 && K <= 24) EF_JOIN_REG_K(NB, ONE, LIST, (ONE) || (NB) == 1 ? 0 : -24, ALIGNED); \
        else if (K > 16 || K < 2) EF_JOIN_REG_K(NB, ONE, LIST, 0, ALIGNED);                        \
        else EF_JOIN_REG_K(NB, ONE, LIST, -16, ALIGNED);                                           \
    } while (0)
#define EF_JOIN_REG(NB, ONE, LIST)                                                                 \
    do {                                                                                           \
        if (aligned) EF_JOIN_REG_A(NB, ONE, LIST, true);                                           \
        else EF_JOIN_REG_A(NB, ONE, LIST, false);                                                  \
        n_upd += reg_grid;                                                                         \
    } while (0)
            if (d <= 128) EF_JOIN_REG(1, true, 0);
            else EF_JOIN_REG(1, false, 0);
            if (timed) EF_HIP_CHECK(hipEventRecord(ev[5 * it + 2], st));
            if (max_rows > 16) {
                if (d <= 128) EF_JOIN_REG(2, true, 1);
                else EF_JOIN_REG(2, false, 1);
            }
#undef EF_JOIN_REG
#undef EF_JOIN_REG_A
#undef EF_JOIN_REG_K
        } else if (timed) {
            EF_HIP_CHECK(hipEventRecord(ev[5 * it + 2], st));
        }
        if (timed) EF_HIP_CHECK(hipEventRecord(ev[5 * it + 3], st));
#define EF_JOIN_LARGE(WIDE, C)                                                                     \
    join_kernel<WIDE><<<large[C].grid, large[C].threads, large[C].lds, st>>>(                      \
        X, w.norms, d, dpad, stride, q4_magic_for(d), K, (u32)(((1ULL << 32) + K - 1) / K),       \
        w.work + (size_t)(C) * n, w.work_count + (C),                                              \
        large[C].cap_rows, large[C].s_cap, large[C].q_cap, margin_rel, thr_scale, w.ulist,         \
        w.ucount, max_rows, graph, w.worst, w.upd_block + n_upd, mode)
        // the larger classes first: their blocks run longest
        for (int c = jc.n - 1; c >= 2 && max_rows > rows1; --c) {
            if (tiles) {      // vectors of at most 128 coordinates pass through registers
                const size_t tl = tile_lds_bytes(jc.bound[c]);
                long per_cu = (long)(kLdsLimit / tl);
                per_cu = per_cu > 4 * kTileWaves ? 4 * kTileWaves : (per_cu < 1 ? 1 : per_cu);      // by registers
                const int tgrid = (int)min((long)n, 256 * per_cu * 4);
                int *upd = w.upd_block + n_upd;
                n_upd += tgrid;
                const u32 km = (u32)(((1ULL << 32) + K - 1) / K);
                const u32 kqm = (u32)(((1ULL << 32) + ((K + 3) >> 2) - 1) / ((K + 3) >> 2));
#define EF_JOIN_TILE(LONG_ROWS, ALIGNED, QUADS)                                                            \
    join_tile_kernel<LONG_ROWS, ALIGNED, QUADS><<<tgrid, EF_WAVE, tl, st>>>(                               \
        X, d, K, km, kqm, w.gid, w.work + (size_t)c * n, w.work_count + c, jc.bound[c],                    \
        margin_f16, thr_scale_f16, u_f16, rho0_f16, w.ulist, w.ucount, max_rows, graph, w.worst, upd,      \
        mode, w.xmax)
                const bool quads = K % 4 == 0 && ((uintptr_t)graph & 15) == 0;
                // (odd rows of up to 32 entries: 64 threads scanning a row each are the better ones still,
                // 300 000 x 112, degree 23: 15.3 ms per build against 15.7)
                if (K <= 16 || (K <= 32 && (K & 1))) {
                    if (aligned) EF_JOIN_TILE(false, true, false);
                    else EF_JOIN_TILE(false, false, false);
                } else if (aligned) {
                    if (quads) EF_JOIN_TILE(true, true, true);
                    else EF_JOIN_TILE(true, true, false);
                } else {
                    if (quads) EF_JOIN_TILE(true, false, true);
                    else EF_JOIN_TILE(true, false, false);
                }
#undef EF_JOIN_TILE
            } else {
                if (K >= 2 * EF_WIDE_PIECES) EF_JOIN_LARGE(true, c);
                else EF_JOIN_LARGE(false, c);
                n_upd += large[c].grid;
            }
        }
#undef EF_JOIN_LARGE
        }      // pass
        if (ev) EF_HIP_CHECK(hipEventRecord(ev[5 * it + 4], st));
        if (stats)
            stats_kernel<<<max(1, min(64, (n_part + n_upd) / (2 * kStatsThreads))), kStatsThreads, 0, st>>>(
                w.part, n_part, w.upd_block, n_upd, stats + 4 * it);
        done = it + 1;
        if (delta > 0.0f) {      // early termination: the host looks at the count after every iteration
            u64 fresh = 0;
            zero_u64_kernel<<<1, kBlock, 0, st>>>(w.fresh, 1);
            count_new_kernel<<<1024, kBlock, 0, st>>>(graph, (size_t)n * K, w.fresh);
            EF_HIP_CHECK(hipMemcpyAsync(&fresh, w.fresh, 8, hipMemcpyDeviceToHost, st));
            EF_HIP_CHECK(hipStreamSynchronize(st));
            if ((double)fresh < (double)delta * (double)n * (double)K) break;
        }
    }
    if (iters_done) *iters_done = done;
    EF_HIP_CHECK(hipGetLastError());
    if (ev) {
        EF_HIP_CHECK(hipStreamSynchronize(st));
        for (int it = 0; it < iters; ++it) {
            for (int ph = 0; ph < 4; ++ph) {
                if (it < done)
                    EF_HIP_CHECK(hipEventElapsedTime(&phase_ms[4 * it + ph], ev[5 * it + ph], ev[5 * it + ph + 1]));
                else
                    phase_ms[4 * it + ph] = 0.0f;
            }
        }
    }
    return EFANNA_OK;
}

}  // namespace

extern "C" int efanna_get_graph(const efanna_entry *graph_, int64_t n, int32_t k, int32_t *ids,
                                float *dists, uint8_t *flags, void *stream)
{
    const u64 *const graph = (const u64 *)graph_;
    if (!graph || !ids || !dists || n < 1 || k < 1 || k > EFANNA_MAX_K) return EFANNA_EINVAL;
    if (k <= 16)
        get_graph_group_kernel<16><<<grid_for((size_t)n * 16, kBlock), kBlock, 0, (hipStream_t)stream>>>(
            graph, (int)n, k, ids, dists, flags);
    else if (k <= 32)
        get_graph_group_kernel<32><<<grid_for((size_t)n * 32, kBlock), kBlock, 0, (hipStream_t)stream>>>(
            graph, (int)n, k, ids, dists, flags);
    else
        get_graph_kernel<<<grid_for((size_t)n, kBlock / EF_WAVE), kBlock, 0, (hipStream_t)stream>>>(
            graph, (int)n, k, ids, dists, flags);
    EF_HIP_CHECK(hipGetLastError());
    return EFANNA_OK;
}

extern "C" int efanna_set_graph(efanna_entry *graph_, int64_t n, int32_t k, const int32_t *ids,
                                const float *dists, const uint8_t *flags, void *stream)
{
    u64 *const graph = (u64 *)graph_;
    if (!graph || !ids || !dists || n < 1 || k < 1 || k > EFANNA_MAX_K) return EFANNA_EINVAL;
    set_graph_kernel<<<grid_for((size_t)n, kBlock / k), kBlock, 0, (hipStream_t)stream>>>(
        graph, (size_t)n, k, ids, dists, flags);
    EF_HIP_CHECK(hipGetLastError());
    return EFANNA_OK;
}

extern "C" int efanna_pair_distances(const float *X, int64_t n, int32_t d, const int32_t *a_ids,
                                     const int32_t *b_ids, int64_t m, float *out, void *stream)
{
    if (!X || !a_ids || !b_ids || !out || n < 1 || d < 1 || m < 0) return EFANNA_EINVAL;
    if (m == 0) return EFANNA_OK;
    pair_distances_kernel<<<grid_for((size_t)m * 16, kBlock), kBlock, 0, (hipStream_t)stream>>>(
        X, d, a_ids, b_ids, (size_t)m, out);
    EF_HIP_CHECK(hipGetLastError());
    return EFANNA_OK;
}
