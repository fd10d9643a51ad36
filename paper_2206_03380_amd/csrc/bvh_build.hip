// Device BVH construction for the shadow-ray mesh (rebuilt whenever the mesh
// changes: the paper re-extracts its mesh every optimisation iteration).
//
// Linear BVH: 63-bit Morton codes of triangle centroids (under a top bit that
// puts the mesh's big triangles first, see morton()), a radix sort, the
// binary radix tree of the sorted codes built in parallel (one lane per
// internal node, Karras 2012), box fitting and the counts of the nodes that
// survive collapsing subtrees of <= kLeafMax triangles (1 among the big ones) into
// leaves, and a final pass that writes every surviving node at its depth-first
// pre-order index with a skip link, so traversal needs no stack.
//
// Fitting has no dependency chain: every internal node's box is a range of the
// sorted triangles' boxes, found by two overlapping power-of-two ranges of a
// sparse table (min and max are idempotent).  Blocks of 256 triangles hold
// their table in LDS and fit the nodes inside them; super-blocks of 256 blocks
// do the same with the blocks' boxes, and one table holds the super-blocks'.
// A node spanning blocks is the union of the suffix box of its first block,
// the prefix box of its last block and the whole blocks between.  A node's
// surviving-node count is 2 L - 1 for the L leaves in its range, read from a
// prefix sum of leaf marks (every surviving internal node has two surviving
// children).
//
// Statistics (deepest node, leaf areas) are reduced per workgroup and summed by
// one last workgroup: atomics on one address from every wavefront took 13 ns
// each, 400 us of the emission and 100 us of the areas at 1.0M triangles.
#include <hip/hip_runtime.h>
#include <cstring>
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "mcdi_internal.h"

namespace mcdi {
namespace {

__device__ __forceinline__ int ord_key(float f) {
    const int i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7FFFFFFF;
}
__device__ __forceinline__ float ord_val(int i) { return __int_as_float(i >= 0 ? i : i ^ 0x7FFFFFFF); }

__device__ __forceinline__ float wave_min(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

constexpr int kFitBlock = 256;   // triangles per fitting block (= workgroup size of the block passes)
constexpr int kFitLevels = 9;    // 2^8 = kFitBlock

// fetch vertices, replace bad triangles by a degenerate one; centroid bounds
// of the workgroup's triangles to part[6 * blockIdx.x] (min xyz, max xyz)
__global__ __launch_bounds__(256) void tri_prep(const float* verts, int64_t nv, const int32_t* tris, int64_t nt,
                                                float4* tmp, float* part, DeviceSceneInfo* info) {
    __shared__ float sb[4][6];
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float cx = INFINITY, cy = INFINITY, cz = INFINITY, Cx = -INFINITY, Cy = -INFINITY, Cz = -INFINITY;
    if (f < nt) {
        float4 v[3];
        bool ok = true;
        for (int c = 0; c < 3; ++c) {
            const int32_t id = tris[3 * f + c];
            if (id < 0 || id >= nv) { ok = false; v[c] = make_float4(0, 0, 0, 0); continue; }
            v[c] = make_float4(verts[3 * (size_t)id], verts[3 * (size_t)id + 1], verts[3 * (size_t)id + 2], 0.0f);
            ok = ok && isfinite(v[c].x) && isfinite(v[c].y) && isfinite(v[c].z);
        }
        if (!ok) {
            atomicAdd(&info->bad_tris, 1);
            v[0] = v[1] = v[2] = make_float4(0, 0, 0, 0);
        }
        tmp[3 * f] = v[0];
        tmp[3 * f + 1] = v[1];
        tmp[3 * f + 2] = v[2];
        const float x = (v[0].x + v[1].x + v[2].x) * (1.0f / 3.0f);
        const float y = (v[0].y + v[1].y + v[2].y) * (1.0f / 3.0f);
        const float z = (v[0].z + v[1].z + v[2].z) * (1.0f / 3.0f);
        cx = Cx = x; cy = Cy = y; cz = Cz = z;
    }
    cx = wave_min(cx); cy = wave_min(cy); cz = wave_min(cz);
    Cx = wave_max(Cx); Cy = wave_max(Cy); Cz = wave_max(Cz);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sb[w][0] = cx; sb[w][1] = cy; sb[w][2] = cz;
        sb[w][3] = Cx; sb[w][4] = Cy; sb[w][5] = Cz;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int k = threadIdx.x;
        float v = sb[0][k];
        for (int j = 1; j < 4; ++j) v = k < 3 ? fminf(v, sb[j][k]) : fmaxf(v, sb[j][k]);
        part[6 * (size_t)blockIdx.x + k] = v;
    }
}

// scene centroid bounds from the per-workgroup parts, as order-preserving
// integer keys (one workgroup)
__global__ __launch_bounds__(256) void bounds_reduce(const float* part, int nb, int* cb) {
    __shared__ float sb[4][6];
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nb; b += 256)
        for (int k = 0; k < 6; ++k) v[k] = k < 3 ? fminf(v[k], part[6 * (size_t)b + k]) : fmaxf(v[k], part[6 * (size_t)b + k]);
    for (int k = 0; k < 3; ++k) { v[k] = wave_min(v[k]); v[3 + k] = wave_max(v[3 + k]); }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < 6; ++k) sb[w][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 6) {
        const int k = threadIdx.x;
        float r = sb[0][k];
        for (int j = 1; j < 4; ++j) r = k < 3 ? fminf(r, sb[j][k]) : fmaxf(r, sb[j][k]);
        cb[k] = ord_key(r);
    }
}

__device__ __forceinline__ uint64_t spread3(uint64_t x) {
    x &= 0x1FFFFFull;
    x = (x | (x << 32)) & 0x1F00000000FFFFull;
    x = (x | (x << 16)) & 0x1F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Key of a triangle: bit 63 clear for a big triangle (its box's longest side
// at least 1/kBigTriDiv of the centroid bounds' longest side), set for the
// others, above the 63-bit Morton code of its centroid.  A mesh with both
// kinds splits at the root into the big triangles (first) and the rest: a
// room's walls, say, stop most shadow rays leaving the geometry inside it,
// and under the Morton order alone each wall triangle widens the box of every
// node it shares with the small triangles around its centroid.  The big ones
// are counted into info->n_big.
__global__ __launch_bounds__(256) void morton(const float4* tmp, int64_t nt, const int* cb, uint64_t* keys,
                                              uint32_t* vals, DeviceSceneInfo* info) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool big = false;
    if (f < nt) {
        const float4 a = tmp[3 * f], b = tmp[3 * f + 1], c = tmp[3 * f + 2];
        const float p[3] = {(a.x + b.x + c.x) * (1.0f / 3.0f), (a.y + b.y + c.y) * (1.0f / 3.0f),
                            (a.z + b.z + c.z) * (1.0f / 3.0f)};
        const float sx = fmaxf(a.x, fmaxf(b.x, c.x)) - fminf(a.x, fminf(b.x, c.x));
        const float sy = fmaxf(a.y, fmaxf(b.y, c.y)) - fminf(a.y, fminf(b.y, c.y));
        const float sz = fmaxf(a.z, fmaxf(b.z, c.z)) - fminf(a.z, fminf(b.z, c.z));
        uint64_t code = 0;
        float cext = 0.0f;
        for (int k = 0; k < 3; ++k) {
            const float lo = ord_val(cb[k]), hi = ord_val(cb[3 + k]);
            const float ext = hi - lo;
            cext = fmaxf(cext, ext);
            float u = ext > 0.0f ? (p[k] - lo) / ext : 0.5f;
            u = fminf(fmaxf(u, 0.0f), 1.0f);
            const uint64_t q = (uint64_t)fminf(u * 2097152.0f, 2097151.0f);
            code |= spread3(q) << (2 - k);
        }
        big = fmaxf(sx, fmaxf(sy, sz)) * kBigTriDiv >= cext;
        keys[f] = big ? code : (code | (1ull << 63));
        vals[f] = (uint32_t)f;
    }
    const uint64_t m = __ballot(big);
    if ((threadIdx.x & 63) == 0 && m != 0) atomicAdd(&info->n_big, (int)__popcll(m));
}

// The big triangles' subtree by the surface area heuristic (one workgroup,
// after the sort; at most kBigSah of them, beyond that they keep their Morton
// keys).  Every shadow ray of a scene with walls walks this subtree first, and
// under the Morton order one wall's triangles are spread over several nodes
// whose boxes span the room.  The split of least cost (areas times counts over
// every triangle's centroid as the plane, all three axes) is found level by
// level for all nodes at once, and a triangle's path is written into its key
// as the radix tree reads it: each level takes the next bit down whose place
// stands for the split's axis, set for the upper side.  Paths that run out of
// bits, and equal centroids, are split by index as equal keys are.
// 36 walls of a room of 1.0M triangles: 6.1 -> 4.6 node visits a shadow ray
// (studied on the CPU), shadow rays 7.1 -> 5.4 ms.
//
// A thread to each place of three lists, in which a node's triangles are
// neighbours, by centroid along the list's axis: the boxes on both sides of
// every plane are a prefix and a suffix box within the node, and a split moves
// each list's upper side behind its lower one.  The scans run in rows of 16
// lanes by data-parallel moves and take the other rows' ends from LDS.  Bound by
// the latency of a level's LDS accesses and its five barriers.
// (Each triangle's thread visiting all triangles for its planes, twice a level,
// made a build's time with 12, 36, 80 and 128 big triangles beside 600 small ones
// 104, 160, 261 and 350 us, now 91, 99, 110 and 114; 79 without any.  Scans by shuffles, two
// places a lane: 99, 110, 131 and 146; in LDS with a barrier a step: 92, 102, 114
// and 118.)
constexpr int kBigSah = 128;

// a box while it is scanned: 16 + 8 bytes
struct ScanBox {
    float4 a;   // lo.x, lo.y, lo.z, hi.x
    float2 b;   // hi.y, hi.z
    __device__ __forceinline__ void grow(const float4& oa, const float2& ob) {
        a = make_float4(fminf(a.x, oa.x), fminf(a.y, oa.y), fminf(a.z, oa.z), fmaxf(a.w, oa.w));
        b = make_float2(fmaxf(b.x, ob.x), fmaxf(b.y, ob.y));
    }
    __device__ __forceinline__ float area() const {   // half of it
        const float dx = a.w - a.x, dy = b.x - a.y, dz = b.y - a.z;
        return fmaf(dz, dx, fmaf(dx, dy, dy * dz));
    }
};

// the value of the lane O before (row_shr) or behind (row_shl) in its row of 16
// lanes; undefined where the row has none
template <int CTRL>
__device__ __forceinline__ float row_move(float x) {
    const int v = __builtin_bit_cast(int, x);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ ScanBox row_move(const ScanBox& s) {
    return ScanBox{make_float4(row_move<CTRL>(s.a.x), row_move<CTRL>(s.a.y), row_move<CTRL>(s.a.z), row_move<CTRL>(s.a.w)),
                   make_float2(row_move<CTRL>(s.b.x), row_move<CTRL>(s.b.y))};
}
// one step of the scans within a row: of places [begin, p], and of (p, end)
template <int O>
__device__ __forceinline__ void row_scan(int p, int begin, int end, ScanBox& pre, ScanBox& suf) {
    const ScanBox before = row_move<0x110 + O>(pre), behind = row_move<0x100 + O>(suf);
    if ((p & 15) >= O && p - O >= begin) pre.grow(before.a, before.b);
    if ((p & 15) + O < 16 && p + O < end) suf.grow(behind.a, behind.b);
}

__global__ __launch_bounds__(3 * kBigSah) void big_sah(const float4* tmp, int nt, uint64_t* keys, uint32_t* vals,
                                                       const DeviceSceneInfo* info) {
    constexpr int T = 3 * kBigSah;
    __shared__ float4 s_boxa[kBigSah];
    __shared__ float2 s_boxb[kBigSah];
    __shared__ ScanBox s_pre[T / 16], s_suf[T / 16];         // by row: its last place's prefix, its first one's suffix
    __shared__ float s_ctr[3][kBigSah];           // by triangle, as are s_box, s_code and s_bit
    __shared__ unsigned long long s_code[kBigSah];
    __shared__ int s_bit[kBigSah];                // its node's next key bit, -1: not split any more
    __shared__ int s_list[3][kBigSah];
    __shared__ int s_begin[kBigSah], s_end[kBigSah];         // the places of the node a place is in
    __shared__ uint32_t s_cost[kBigSah], s_plane[kBigSah];   // at the node's first place: the least cost, its plane
    __shared__ unsigned long long s_upper[T / 64];
    __shared__ int s_largest[2];                  // by the level's parity
    const int n = info->n_big;
    if (n < 3 || n > kBigSah || n >= nt) return;
    const int p = threadIdx.x % kBigSah, axis = threadIdx.x / kBigSah;
    const bool on = p < n, first = axis == 0 && on;          // one thread of each place
    uint32_t val = 0;
    if (first) {
        val = vals[p];
        const float4* t = tmp + 3 * (size_t)val;
        const float4 a = t[0], b = t[1], c = t[2];
        s_boxa[p] = make_float4(fminf(a.x, fminf(b.x, c.x)), fminf(a.y, fminf(b.y, c.y)), fminf(a.z, fminf(b.z, c.z)),
                                fmaxf(a.x, fmaxf(b.x, c.x)));
        s_boxb[p] = make_float2(fmaxf(a.y, fmaxf(b.y, c.y)), fmaxf(a.z, fmaxf(b.z, c.z)));
        s_ctr[0][p] = (a.x + b.x + c.x) * (1.0f / 3.0f);
        s_ctr[1][p] = (a.y + b.y + c.y) * (1.0f / 3.0f);
        s_ctr[2][p] = (a.z + b.z + c.z) * (1.0f / 3.0f);
        s_code[p] = 0ull;
        s_bit[p] = 62;
        s_begin[p] = 0;
        s_end[p] = n;
        s_cost[p] = s_plane[p] = ~0u;
    }
    __syncthreads();
    if (on) {
        // (of equal centroids the lowest index comes last, where their plane is)
        const float c = s_ctr[axis][p];
        int place = 0;
        for (int j = 0; j < n; ++j) {
            const float o = s_ctr[axis][j];
            place += (o < c || (o == c && j > p)) ? 1 : 0;
        }
        s_list[axis][place] = p;
    }
    int largest = n;     // triangles of the level's largest node that may be split
    __syncthreads();
    for (int level = 0; largest > 1; ++level) {              // (every level takes a bit of 63)
        int t = 0, begin = 0, end = 0, bit = -1;
        ScanBox pre{}, suf{};    // of the node's triangles up to this place, and behind it
        float next = 0.0f;       // the centroid behind it
        if (on) {
            t = s_list[axis][p];
            begin = s_begin[p];
            end = s_end[p];
            bit = s_bit[t];
            pre.a = s_boxa[t];
            pre.b = s_boxb[t];
            suf.a = make_float4(INFINITY, INFINITY, INFINITY, -INFINITY);
            suf.b = make_float2(-INFINITY, -INFINITY);
            if (p + 1 < end) {
                const int t1 = s_list[axis][p + 1];
                suf.a = s_boxa[t1];
                suf.b = s_boxb[t1];
                next = s_ctr[axis][t1];
            }
        }
        if (threadIdx.x == 0) s_largest[level & 1] = 0;
        row_scan<1>(p, begin, end, pre, suf);
        if (largest > 2) row_scan<2>(p, begin, end, pre, suf);
        if (largest > 4) row_scan<4>(p, begin, end, pre, suf);
        if (largest > 8) row_scan<8>(p, begin, end, pre, suf);
        const int row = threadIdx.x >> 4;
        if ((p & 15) == 15) s_pre[row] = pre;
        if ((p & 15) == 0) s_suf[row] = suf;
        __syncthreads();
        if (bit >= 0) {
            const int row0 = row - (p >> 4);     // the list's first
            for (int r = row0 + (begin >> 4); r < row; ++r) pre.grow(s_pre[r].a, s_pre[r].b);
            for (int r = row + 1; 16 * (r - row0) < end - 1; ++r) suf.grow(s_suf[r].a, s_suf[r].b);
        }
        // the plane at this place's triangle: the least cost of its node, then
        // of the planes that have it the one of the lowest axis and index
        uint32_t mine = ~0u;
        if (bit >= 0 && p + 1 < end && next > s_ctr[axis][t]) {
            // (written out: the same two sets along several axes are told apart
            // by its rounding, which the compiler's choice of fusions would change)
            const float cost = fmaf(suf.area(), (float)(end - p - 1), pre.area() * (float)(p + 1 - begin));
            if (cost >= 0.0f) {
                mine = __float_as_uint(cost);
                atomicMin(&s_cost[begin], mine);
            }
        }
        __syncthreads();
        if (mine != ~0u && mine == s_cost[begin]) atomicMin(&s_plane[begin], (uint32_t)(axis << 8 | t));
        __syncthreads();
        int at = -1;         // the bit the node's split takes
        bool upper = false;
        if (bit >= 0) {
            const uint32_t b = s_plane[begin];
            if (b != ~0u) {
                const int a = (int)(b >> 8), pivot = (int)(b & 255u);
                at = bit;
                while (at >= 0 && 2 - at % 3 != a) --at;
                upper = at >= 0 && s_ctr[a][t] > s_ctr[a][pivot];
            }
        }
        const unsigned long long mask = __ballot(upper);
        if ((threadIdx.x & 63) == 0) s_upper[threadIdx.x >> 6] = mask;
        __syncthreads();
        if (at >= 0) {
            // upper ones of the list before place q
            const unsigned long long m0 = s_upper[2 * axis], m1 = s_upper[2 * axis + 1];
            auto uppers = [&](int q) {
                return q < 64 ? __popcll(m0 & ((1ull << q) - 1ull))
                              : __popcll(m0) + (q < 128 ? __popcll(m1 & ((1ull << (q - 64)) - 1ull)) : __popcll(m1));
            };
            const int u0 = uppers(begin), u = uppers(p) - u0, middle = end - (uppers(end) - u0);
            const int place = upper ? middle + u : p - u;
            s_list[axis][place] = t;
            if (axis == 0) {
                s_begin[place] = upper ? middle : begin;
                s_end[place] = upper ? end : middle;
                if (upper) s_code[t] |= 1ull << at;
                s_bit[t] = at - 1;
                if (p == begin) atomicMax(&s_largest[level & 1], max(middle - begin, end - middle));
            }
        } else if (first) {
            s_bit[t] = -1;
        }
        if (first) s_cost[p] = s_plane[p] = ~0u;
        __syncthreads();
        largest = s_largest[level & 1];      // (uniform: the next level writes the other one)
    }
    // the nodes stand in the order of their codes; triangles of one keep theirs
    if (first) s_list[1][s_list[0][p]] = p;                  // a triangle's place
    __syncthreads();
    if (first) {
        const int q = s_list[1][p], begin = s_begin[q], end = s_end[q];
        int rank = begin;
        for (int j = begin; j < end; ++j) rank += s_list[0][j] < p ? 1 : 0;
        keys[rank] = s_code[p];
        vals[rank] = val;
    }
}

struct Tree {
    int32_t* parent;   // [2nt-1]
    int32_t* left;     // [nt-1] node ids (leaf k = nt-1+k)
    int32_t* right;
    int32_t* first;    // [nt-1] sorted-primitive range
    int32_t* last;
    int32_t* axis;     // [nt-1] the axis the node's Morton split separates its children on
    int32_t* cnt;      // [2nt-1] surviving nodes in the subtree
    float4* box;       // [2*(2nt-1)]
    // block fitting (blocks of kFitBlock sorted triangles)
    int32_t* mark;     // [nt] 1 at the first triangle of every leaf
    int32_t* mark_pre; // [nt] exclusive prefix of mark within the block
    float4* pre;       // [2nt] box of the block's triangles up to k (inclusive)
    float4* suf;       // [2nt] box of the block's triangles from k to the block end
    // super-blocks of kFitBlock blocks
    int32_t* blk_mark; // [nb] leaf marks of each block
    int32_t* blk_base; // [nb] leaf marks before each block within its super-block
    float4* blk_pre;   // [2nb] box of the super-block's blocks up to b (inclusive)
    float4* blk_suf;   // [2nb] box of the super-block's blocks from b on
    float4* st;        // [kFitLevels][nb][2] box of blocks [b, b + 2^j) within the super-block
    // the whole mesh
    int32_t* sup_mark; // [ns] leaf marks of each super-block
    int32_t* sup_base; // [ns + 1] leaf marks before each super-block, then all
    float4* sup_st;    // [sup_levels][ns][2] sparse table of super-block boxes
    const int32_t* nbig;   // the big triangles' count (sorted first)
    int nb, ns, sup_levels;
};

// Most triangles a leaf holds: kLeafMax, and kBigLeafMax inside the big
// triangles' subtree (sorted range [0, n_big)) of a mesh that has both kinds.
// Every node but the root lies entirely on one side of n_big.
__device__ __forceinline__ int leaf_cap(const Tree& T, int nt, int last) {
    const int nb = *T.nbig;
    return (nb < nt && last < nb) ? kBigLeafMax : kLeafMax;
}

__device__ __forceinline__ int prefix_len(const uint64_t* keys, int nt, int a, int b) {
    if (b < 0 || b >= nt) return -1;
    const uint64_t ka = keys[a], kb = keys[b];
    if (ka == kb) return 64 + __clz((uint32_t)(a ^ b));
    return __clzll((long long)(ka ^ kb));
}

__global__ __launch_bounds__(256) void radix_tree(const uint64_t* keys, int nt, Tree T, int32_t* gflag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt - 1) return;
    // cleared for the passes that set some of their entries
    T.mark[i] = 0;
    gflag[i] = 0;
    gflag[nt - 1 + i] = 0;
    if (i == 0) {
        T.mark[nt - 1] = 0;
        gflag[2 * nt - 2] = 0;
    }
    const int d = prefix_len(keys, nt, i, i + 1) > prefix_len(keys, nt, i, i - 1) ? 1 : -1;
    const int dmin = prefix_len(keys, nt, i, i - d);
    int lmax = 2;
    while (prefix_len(keys, nt, i, i + lmax * d) > dmin) lmax <<= 1;
    int l = 0;
    for (int t = lmax >> 1; t >= 1; t >>= 1)
        if (prefix_len(keys, nt, i, i + (l + t) * d) > dmin) l += t;
    const int j = i + l * d;
    const int dnode = prefix_len(keys, nt, i, j);
    int s = 0, t = l;
    do {
        t = (t + 1) >> 1;
        if (prefix_len(keys, nt, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int g = i + s * d + (d < 0 ? -1 : 0);
    const int lo = min(i, j), hi = max(i, j);
    const int L = (lo == g) ? (nt - 1 + g) : g;
    const int R = (hi == g + 1) ? (nt - 1 + g + 1) : g + 1;
    T.left[i] = L;
    T.right[i] = R;
    T.first[i] = lo;
    T.last[i] = hi;
    // the split is at the first bit the range's codes differ in, bit 63 - dnode
    // (x, y, z interleaved from bit 62 down: bit b is x, y or z as b % 3 is 2,
    // 1 or 0); the left child holds the codes with a 0 there, the lower side;
    // equal codes (split by index) take x.  A split at bit 63 (the root of a
    // mesh with big and small triangles) is 3: no axis, the left child (the
    // big triangles) first for every ray
    T.axis[i] = dnode == 0 ? 3 : dnode < 64 ? 2 - (63 - dnode) % 3 : 0;
    T.parent[L] = i;
    T.parent[R] = i;
    if (i == 0) T.parent[0] = -1;
}

__device__ __forceinline__ void tri_box(const float4* t, float4& lo, float4& hi) {
    lo = make_float4(fminf(t[0].x, fminf(t[1].x, t[2].x)), fminf(t[0].y, fminf(t[1].y, t[2].y)),
                     fminf(t[0].z, fminf(t[1].z, t[2].z)), 0.0f);
    hi = make_float4(fmaxf(t[0].x, fmaxf(t[1].x, t[2].x)), fmaxf(t[0].y, fmaxf(t[1].y, t[2].y)),
                     fmaxf(t[0].z, fmaxf(t[1].z, t[2].z)), 0.0f);
}

// rows (v0, v1, v2, 0) of x, y and z from vertices, or vertices from rows
__device__ __forceinline__ void transpose_tri(const float4* t, float4* out) {
    const float4 a = t[0], b = t[1], c = t[2];
    out[0] = make_float4(a.x, b.x, c.x, 0.0f);
    out[1] = make_float4(a.y, b.y, c.y, 0.0f);
    out[2] = make_float4(a.z, b.z, c.z, 0.0f);
}

// leaf marks: a node of <= leaf_cap triangles whose parent has more is a
// leaf of the collapsed tree (the root, when the whole mesh fits in one)
__global__ __launch_bounds__(256) void mark_leaves(int nt, Tree T) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= 2 * nt - 1) return;
    const bool prim = x >= nt - 1;
    const int first = prim ? x - (nt - 1) : T.first[x];
    const int last = prim ? first : T.last[x];
    const int size = last - first + 1;
    if (size > leaf_cap(T, nt, last)) return;
    if (x != 0) {
        const int p = T.parent[x];
        if (p < 0 || p >= nt - 1 || T.last[p] - T.first[p] + 1 <= leaf_cap(T, nt, T.last[p])) return;
    }
    if (first >= 0 && first < nt) T.mark[first] = 1;
}

// Boxes of 256 consecutive elements with their sparse table in LDS: level j
// holds the box of elements [t, t + 2^j) (clamped at the last).
struct FitTable {
    float lo[kFitLevels][3][kFitBlock], hi[kFitLevels][3][kFitBlock];
};

__device__ __forceinline__ void table_put(FitTable& S, int j, int t, float4 lo, float4 hi) {
    S.lo[j][0][t] = lo.x; S.lo[j][1][t] = lo.y; S.lo[j][2][t] = lo.z;
    S.hi[j][0][t] = hi.x; S.hi[j][1][t] = hi.y; S.hi[j][2][t] = hi.z;
}

// levels 1.. from level 0 (thread t its own column; ends with a barrier)
__device__ void table_build(FitTable& S, int t) {
    __syncthreads();
    for (int j = 1; j < kFitLevels; ++j) {
        const int u = min(t + (1 << (j - 1)), kFitBlock - 1);
        for (int a = 0; a < 3; ++a) {
            S.lo[j][a][t] = fminf(S.lo[j - 1][a][t], S.lo[j - 1][a][u]);
            S.hi[j][a][t] = fmaxf(S.hi[j - 1][a][t], S.hi[j - 1][a][u]);
        }
        __syncthreads();
    }
}

// box of elements [f, l], 0 <= f <= l < kFitBlock
__device__ __forceinline__ void table_range(const FitTable& S, int f, int l, float4& lo, float4& hi) {
    const int j = 31 - __clz(l - f + 1), u = l + 1 - (1 << j);
    lo = make_float4(fminf(S.lo[j][0][f], S.lo[j][0][u]), fminf(S.lo[j][1][f], S.lo[j][1][u]),
                     fminf(S.lo[j][2][f], S.lo[j][2][u]), 0.0f);
    hi = make_float4(fmaxf(S.hi[j][0][f], S.hi[j][0][u]), fmaxf(S.hi[j][1][f], S.hi[j][1][u]),
                     fmaxf(S.hi[j][2][f], S.hi[j][2][u]), 0.0f);
}

// exclusive prefix over the workgroup's kFitBlock threads; *total the sum
__device__ int block_prefix(int v, int* s_wave, int* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        incl += lane >= o ? u : 0;
    }
    if (lane == 63) s_wave[w] = incl;
    __syncthreads();
    int before = 0, sum = 0;
    for (int k = 0; k < kFitBlock / 64; ++k) {
        before += k < w ? s_wave[k] : 0;
        sum += s_wave[k];
    }
    *total = sum;
    return before + incl - v;
}

// Block pass (workgroup b = sorted triangles [256 b, 256 b + 256)): the
// triangles' rows in sorted order, leaf boxes, the block's prefix and suffix
// boxes and leaf-mark prefix, and box and surviving-node count of every node
// inside the block (node i is one end of its range, so it belongs to block
// i / 256).  (Fitting bottom-up inside the block instead, the second child to
// arrive taking the parent, and two more scans took 52 us at 296k triangles
// and 21 us at 590, now 20 and 8.)
__global__ __launch_bounds__(kFitBlock) void fit_block(const float4* tmp, const uint32_t* vals, int nt, Tree T,
                                                       float4* tris_out) {
    __shared__ FitTable S;
    __shared__ int s_pre[kFitBlock], s_wave[kFitBlock / 64];
    const int t = threadIdx.x;
    const int lo = blockIdx.x * kFitBlock;
    const int hi = min(nt, lo + kFitBlock) - 1;
    const int k = lo + t;
    const bool valid = k <= hi;
    float4 blo = make_float4(INFINITY, INFINITY, INFINITY, 0.0f), bhi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.0f);
    int m = 0;
    if (valid) {
        const float4* tri = tmp + 3 * (size_t)vals[k];
        tri_box(tri, blo, bhi);
        transpose_tri(tri, tris_out + 3 * (size_t)k);
        const int leaf = nt - 1 + k;
        T.box[2 * leaf] = blo;
        T.box[2 * leaf + 1] = bhi;
        T.cnt[leaf] = 1;
        m = T.mark[k];
    }
    table_put(S, 0, t, blo, bhi);
    table_build(S, t);
    int total = 0;
    const int mp = block_prefix(m, s_wave, &total);
    s_pre[t] = mp;
    __syncthreads();
    float4 al, ah;
    if (valid) {
        table_range(S, 0, t, al, ah);
        T.pre[2 * (size_t)k] = al;
        T.pre[2 * (size_t)k + 1] = ah;
        T.mark_pre[k] = mp;
        if (k == hi) {
            T.st[2 * (size_t)blockIdx.x] = al;
            T.st[2 * (size_t)blockIdx.x + 1] = ah;
            T.blk_mark[blockIdx.x] = total;
        }
        table_range(S, t, kFitBlock - 1, al, ah);   // (past the last triangle: empty boxes)
        T.suf[2 * (size_t)k] = al;
        T.suf[2 * (size_t)k + 1] = ah;
    }
    if (k < nt - 1) {
        const int f = T.first[k], l = T.last[k];
        if (f >= lo && l <= hi && f < l) {
            table_range(S, f - lo, l - lo, al, ah);
            T.box[2 * (size_t)k] = al;
            T.box[2 * (size_t)k + 1] = ah;
            const int leaves = (l < hi ? s_pre[l + 1 - lo] : total) - s_pre[f - lo];
            T.cnt[k] = l - f + 1 <= leaf_cap(T, nt, l) ? 1 : 2 * leaves - 1;
        }
    }
}

// The same over the boxes of a super-block's blocks.
__global__ __launch_bounds__(kFitBlock) void fit_super(Tree T) {
    __shared__ FitTable S;
    __shared__ int s_wave[kFitBlock / 64];
    const int t = threadIdx.x;
    const int b = blockIdx.x * kFitBlock + t;
    const int last = min(T.nb, (int)(blockIdx.x + 1) * kFitBlock) - 1;
    const bool valid = b <= last;
    float4 lo = make_float4(INFINITY, INFINITY, INFINITY, 0.0f), hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.0f);
    int m = 0;
    if (valid) {
        lo = T.st[2 * (size_t)b];
        hi = T.st[2 * (size_t)b + 1];
        m = T.blk_mark[b];
    }
    table_put(S, 0, t, lo, hi);
    table_build(S, t);
    int total = 0;
    const int mp = block_prefix(m, s_wave, &total);
    if (!valid) return;
    T.blk_base[b] = mp;
    for (int j = 1; j < kFitLevels; ++j) {
        float4* st = T.st + 2 * ((size_t)j * T.nb + b);
        st[0] = make_float4(S.lo[j][0][t], S.lo[j][1][t], S.lo[j][2][t], 0.0f);
        st[1] = make_float4(S.hi[j][0][t], S.hi[j][1][t], S.hi[j][2][t], 0.0f);
    }
    table_range(S, 0, t, lo, hi);
    T.blk_pre[2 * (size_t)b] = lo;
    T.blk_pre[2 * (size_t)b + 1] = hi;
    if (b == last) {
        T.sup_st[2 * (size_t)blockIdx.x] = lo;
        T.sup_st[2 * (size_t)blockIdx.x + 1] = hi;
        T.sup_mark[blockIdx.x] = total;
        if (T.ns == 1) {
            T.sup_base[0] = 0;
            T.sup_base[1] = total;
        }
    }
    table_range(S, t, kFitBlock - 1, lo, hi);
    T.blk_suf[2 * (size_t)b] = lo;
    T.blk_suf[2 * (size_t)b + 1] = hi;
}

// Over the super-blocks (one workgroup; at most 1024 of them, 2^26 triangles):
// scan of their leaf marks and the sparse table of their boxes.
__global__ __launch_bounds__(1024) void fit_mesh(Tree T) {
    __shared__ int s[1024];
    const int t = threadIdx.x, ns = T.ns;
    const int v = t < ns ? T.sup_mark[t] : 0;
    s[t] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int a = t >= o ? s[t - o] : 0;
        __syncthreads();
        s[t] += a;
        __syncthreads();
    }
    if (t < ns) T.sup_base[t] = s[t] - v;
    if (t == 0) T.sup_base[ns] = s[1023];
    for (int j = 1; j < T.sup_levels; ++j) {
        const float4* prev = T.sup_st + 2 * (size_t)(j - 1) * ns;
        float4* cur = T.sup_st + 2 * (size_t)j * ns;
        if (t < ns) {
            const int u = min(t + (1 << (j - 1)), ns - 1);
            const float4 al = prev[2 * t], ah = prev[2 * t + 1], bl = prev[2 * u], bh = prev[2 * u + 1];
            cur[2 * t] = make_float4(fminf(al.x, bl.x), fminf(al.y, bl.y), fminf(al.z, bl.z), 0.0f);
            cur[2 * t + 1] = make_float4(fmaxf(ah.x, bh.x), fmaxf(ah.y, bh.y), fmaxf(ah.z, bh.z), 0.0f);
        }
        __syncthreads();
    }
}

__device__ __forceinline__ void grow(float4& lo, float4& hi, const float4* b) {
    lo = make_float4(fminf(lo.x, b[0].x), fminf(lo.y, b[0].y), fminf(lo.z, b[0].z), 0.0f);
    hi = make_float4(fmaxf(hi.x, b[1].x), fmaxf(hi.y, b[1].y), fmaxf(hi.z, b[1].z), 0.0f);
}

// leaves before sorted position i (i in [0, nt])
__device__ __forceinline__ int leaves_before(const Tree& T, int nt, int i) {
    if (i >= nt) return T.sup_base[T.ns];
    const int b = i / kFitBlock;
    return T.sup_base[b / kFitBlock] + T.blk_base[b] + T.mark_pre[i];
}

// every internal node spanning blocks: box and surviving-node count directly
__global__ __launch_bounds__(256) void fit_top(int nt, Tree T) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nt - 1) return;
    const int f = T.first[p], l = T.last[p];
    if (f < 0 || l >= nt || f > l) return;
    const int bf = f / kFitBlock, bl = l / kFitBlock;
    if (bf == bl) return;   // fitted by its block
    float4 lo = T.suf[2 * (size_t)f], hi = T.suf[2 * (size_t)f + 1];
    grow(lo, hi, T.pre + 2 * (size_t)l);
    const int b0 = bf + 1, b1 = bl - 1;   // whole blocks strictly between
    if (b0 <= b1) {
        const int s0 = b0 / kFitBlock, s1 = b1 / kFitBlock;
        if (s0 == s1) {
            const int j = 31 - __clz(b1 - b0 + 1);
            grow(lo, hi, T.st + 2 * ((size_t)j * T.nb + b0));
            grow(lo, hi, T.st + 2 * ((size_t)j * T.nb + (b1 + 1 - (1 << j))));
        } else {
            grow(lo, hi, T.blk_suf + 2 * (size_t)b0);
            grow(lo, hi, T.blk_pre + 2 * (size_t)b1);
            const int n = s1 - s0 - 1;    // whole super-blocks between
            if (n > 0) {
                const int j = 31 - __clz(n);
                grow(lo, hi, T.sup_st + 2 * ((size_t)j * T.ns + s0 + 1));
                grow(lo, hi, T.sup_st + 2 * ((size_t)j * T.ns + (s1 - (1 << j))));
            }
        }
    }
    T.box[2 * (size_t)p] = lo;
    T.box[2 * (size_t)p + 1] = hi;
    T.cnt[p] = 2 * (leaves_before(T, nt, l + 1) - leaves_before(T, nt, f)) - 1;
}

// Quantisation frame of the scene from its root box: the box's middle rounded
// to FP32, and a step such that mid -/+ 2^15 step lie outside the box with a
// pad of 2^-20 of the largest extent, rounded up to FP32.
__device__ void qframe_of(float4 rlo, float4 rhi, QFrame& F) {
    const double ext = fmax(fmax((double)rhi.x - rlo.x, (double)rhi.y - rlo.y), (double)rhi.z - rlo.z);
    const double pad = fmax(ext * 0x1p-20, 1e-30);
    const double lo[3] = {rlo.x, rlo.y, rlo.z}, hi[3] = {rhi.x, rhi.y, rhi.z};
    for (int a = 0; a < 3; ++a) {
        F.mid[a] = (float)(0.5 * (lo[a] + hi[a]));
        const double reach = fmax(hi[a] - (double)F.mid[a], (double)F.mid[a] - lo[a]) + pad;
        F.step[a] = __double2float_ru(reach * 0x1p-15);
    }
}

// Bits of the largest half <= x (|x| <= 2^15): x in units of its half's last
// place, rounded down (subnormals below 2^-14 have a last place of 2^-24).
__device__ uint32_t half_down(double x) {
    if (x == 0.0) return 0u;
    int e = 0;
    (void)frexp(fabs(x), &e);
    const int k = max(e - 11, -24);
    const double v = ldexp(floor(ldexp(x, -k)), k);
    return __builtin_bit_cast(uint16_t, (_Float16)(float)v);
}
__device__ double half_value(uint32_t h) { return (double)(float)__builtin_bit_cast(_Float16, (uint16_t)h); }

// Outward quantisation: the plane of lo is at or below v.  A non-finite
// coordinate gives the end of the range.  (The plane is formed in FP64 and
// stepped down while the division's rounding left it above v.)
__device__ uint32_t quant_lo(float v, double mid, float step) {
    constexpr uint32_t kEnd = 0xF800u;   // -2^15
    if (!isfinite(v)) return kEnd;
    uint32_t h = half_down(fmin(fmax(((double)v - mid) / step, -0x1p15), 0x1p15));
    for (int k = 0; k < 4 && h != kEnd && mid + half_value(h) * (double)step > (double)v; ++k)
        h = (h & 0x7FFFu) == 0u ? 0x8001u : ((h & 0x8000u) ? h + 1u : h - 1u);
    return h;
}
// the plane of hi is at or above v
__device__ uint32_t quant_hi(float v, double mid, float step) { return quant_lo(-v, -mid, step) ^ 0x8000u; }

__device__ QNode quantise(const QFrame& F, const Node& nd) {
    uint32_t l[3], h[3];
    for (int a = 0; a < 3; ++a) {
        l[a] = quant_lo(nd.lo[a], F.mid[a], F.step[a]);
        h[a] = quant_hi(nd.hi[a], F.mid[a], F.step[a]);
    }
    QNode q;
    q.x = l[0] | (l[1] << 16);
    q.y = l[2] | (h[0] << 16);
    q.z = h[1] | (h[2] << 16);
    q.w = nd.payload != 0 ? leaf_ref((uint32_t)nd.payload >> 3, (uint32_t)nd.payload & 7u) : (uint32_t)nd.escape;
    return q;
}

__device__ __forceinline__ double box_area(const Node& nd) {
    const double dx = fmax((double)nd.hi[0] - nd.lo[0], 0.0), dy = fmax((double)nd.hi[1] - nd.lo[1], 0.0),
                 dz = fmax((double)nd.hi[2] - nd.lo[2], 0.0);
    return 2.0 * (dx * dy + dy * dz + dz * dx);
}

// a workgroup's share of the statistics
struct EmitPart {
    double leaf_area;
    int32_t max_depth;
};

// one surviving node x at its pre-order index, with its depth and, of a leaf,
// its box's area
__device__ __forceinline__ void emit_node(int x, int nt, const Tree& T, Node* out, QNode* qout, QFrame* frame,
                                          int32_t* gflag, int32_t* naxis, int& max_depth, double& area) {
    const bool is_prim = x >= nt - 1;
    if (x != 0) {
        const int p = T.parent[x];
        if (p < 0 || p >= nt - 1) return;                       // not linked (never for a valid tree)
        if (T.last[p] - T.first[p] + 1 <= leaf_cap(T, nt, T.last[p])) return;  // inside a collapsed leaf
    }
    int idx = 0, depth = 0, cur = x;
    while (cur != 0 && depth < 4096) {
        const int p = T.parent[cur];
        if (p < 0 || p >= nt - 1) return;
        const int l = T.left[p];
        idx += (cur == l) ? 1 : 1 + T.cnt[l];
        cur = p;
        ++depth;
    }
    if (idx < 0 || idx >= 2 * nt - 1) return;
    int payload = 0;
    if (is_prim) {
        payload = ((x - (nt - 1)) << 3) | 1;
    } else {
        const int size = T.last[x] - T.first[x] + 1;
        if (size <= leaf_cap(T, nt, T.last[x])) payload = (T.first[x] << 3) | size;
    }
    const float4 lo = T.box[2 * x], hi = T.box[2 * x + 1];
    Node nd;
    nd.lo[0] = lo.x; nd.lo[1] = lo.y; nd.lo[2] = lo.z;
    nd.hi[0] = hi.x; nd.hi[1] = hi.y; nd.hi[2] = hi.z;
    nd.escape = idx + T.cnt[x];
    nd.payload = payload;
    out[idx] = nd;
    naxis[idx] = is_prim ? 0 : T.axis[x];
    // the root's box (internal node 0) sets the frame, the same for every thread
    QFrame F;
    qframe_of(T.box[0], T.box[1], F);
    qout[idx] = quantise(F, nd);
    if (idx == 0) *frame = F;
    // a wide node for the root and for every internal node at even depth
    gflag[idx] = (idx == 0 || (payload == 0 && (depth & 1) == 0)) ? 1 : 0;
    if (payload != 0) area = box_area(nd);
    max_depth = depth;
}

__global__ __launch_bounds__(256) void emit(int nt, Tree T, Node* out, QNode* qout, QFrame* frame,
                                            int32_t* gflag, int32_t* naxis, EmitPart* part) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    int depth = -1;
    double area = 0.0;
    if (x < 2 * nt - 1) emit_node(x, nt, T, out, qout, frame, gflag, naxis, depth, area);
    __shared__ int s_depth[4];
    __shared__ double s_area[4];
    for (int o = 32; o > 0; o >>= 1) {
        depth = max(depth, __shfl_xor(depth, o));
        area += __shfl_xor(area, o);
    }
    if ((threadIdx.x & 63) == 0) {
        s_depth[threadIdx.x >> 6] = depth;
        s_area[threadIdx.x >> 6] = area;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        part[blockIdx.x] = EmitPart{s_area[0] + s_area[1] + s_area[2] + s_area[3],
                                    max(max(s_depth[0], s_depth[1]), max(s_depth[2], s_depth[3]))};
}

__global__ __launch_bounds__(256) void tri_vertices(const float4* rows, int64_t n, float4* verts) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < n) transpose_tri(rows + 3 * k, verts + 3 * k);
}

// The 4-wide hierarchy of the shadow-ray traversal, collapsed from the binary
// one: a wide node for the root and for every internal node N at even depth,
// whose up to four children are N's children, a child that is internal being
// replaced by its own two children.  Slots 0-1 hold what N's first child
// contributes (itself when it is a leaf, else its two children), slots 2-3
// what the second contributes; a child record is the quantised box of that
// binary node with w = its wide node's index (internal) or its leaf reference,
// and an unused slot holds an empty record (lo > hi: no ray hits it).
// Wide nodes are numbered in the binary pre-order of their nodes (an
// exclusive scan of the flags), so the wide hierarchy is in pre-order too.
//
// The records' words also carry the axes of the up to three binary splits a
// wide node covers.  A ray takes each split's child farther along the ray on
// the split's axis first (the Morton order puts the lower side left), and at
// the split that separates the big triangles (axis 3) their child first.
__device__ __forceinline__ QNode empty_record() {
    QNode q;
    q.x = 0x7BFF7BFFu;   // lo = 65504, the largest half, hi = -65504
    q.y = 0xFBFF7BFFu;
    q.z = 0xFBFFFBFFu;
    q.w = kEmptyRef;     // tests nothing, should it ever be taken
    return q;
}

__device__ __forceinline__ QNode child_record(const Node* out, const QNode* qout, const int32_t* gidx, int x) {
    QNode q = qout[x];
    if (out[x].payload == 0) q.w = (uint32_t)gidx[x];
    return q;
}

__global__ __launch_bounds__(256) void wide_groups(const Node* out, const QNode* qout, const int32_t* gflag,
                                                   const int32_t* gidx, const int32_t* naxis, int n_max,
                                                   QNode* groups, DeviceSceneInfo* info) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n_max) return;
    const int n_nodes = out[0].escape;            // surviving binary nodes
    if (x >= n_nodes || !gflag[x]) return;
    const int self = gidx[x];
    QNode g[4];
    for (int k = 0; k < 4; ++k) g[k] = empty_record();
    uint32_t axis[3] = {0u, 0u, 0u};
    if (out[x].payload != 0) {                    // a root that is a leaf
        g[0] = child_record(out, qout, gidx, x);
    } else {
        const int c[2] = {x + 1, out[x + 1].escape};
        axis[0] = (uint32_t)naxis[x];
        for (int i = 0; i < 2; ++i) {
            const int y = c[i];
            if (y <= x || y >= n_nodes) continue;    // never for a valid tree
            if (out[y].payload != 0) {
                g[2 * i] = child_record(out, qout, gidx, y);
            } else {
                axis[1 + i] = (uint32_t)naxis[y];
                const int d[2] = {y + 1, out[y + 1].escape};
                for (int j = 0; j < 2; ++j)
                    if (d[j] > y && d[j] < n_nodes) g[2 * i + j] = child_record(out, qout, gidx, d[j]);
            }
        }
    }
    // the walk's termination rests on this: every internal child reference
    // lies past its parent and inside the node array (pre-order numbering);
    // a violation (never for a valid tree) sends the scene to the binary walk
    const int n_groups = gidx[n_max - 1] + gflag[n_max - 1];
    for (int i = 0; i < 4; ++i) {
        const uint32_t w = g[i].w;
        if (!(w & kQLeaf) && ((int)w <= self || (int)w >= n_groups)) atomicOr(&info->wide_bad, 1);
        g[i].w = (w & kRefMask) | kRefLive | (i < 3 ? axis[i] << kRefAxisShift : 0u);
        groups[4 * (size_t)self + i] = g[i];
    }
}

// Hoisted nodes (one wavefront): breadth-first from the root, one level a
// step with a lane to each of its nodes, until kTopNodes are taken.  Only as
// many levels as a full 4-ary tree needs twice over: what a thinner tree
// leaves out stays in the node array.
constexpr int kTopLevels = 6;
// (A reference that failed the builder's check, never for a valid tree, is read
// inside the array, whose capacity this is, and no walk takes the wide nodes.)
__global__ __launch_bounds__(64) void hoist_top(const QNode* groups, uint32_t capacity, QNode* top) {
    static_assert(kTopNodes <= 64, "a lane to each node of a level");
    __shared__ uint32_t s_list[kTopNodes];
    const int t = threadIdx.x;
    int begin = 0, end = 1;
    if (t == 0) s_list[0] = 0u;
    __syncthreads();
    for (int level = 0; begin < end; ++level) {
        const bool mine = begin + t < end;
        QNode g[4];
        int n = 0;
        if (mine) {
            const QNode* src = groups + 4 * (size_t)s_list[begin + t];
            for (int k = 0; k < 4; ++k) {
                g[k] = src[k];
                n += (g[k].w & kQLeaf) ? 0 : 1;
            }
        }
        // internal children before this lane's on the level
        int incl = n;
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            incl += t >= o ? v : 0;
        }
        int at = end + incl - n;
        const int total = __shfl(incl, 63);
        const int next_end = level + 1 < kTopLevels ? min(end + total, kTopNodes) : end;
        if (mine) {
            for (int k = 0; k < 4; ++k) {
                if (!(g[k].w & kQLeaf)) {
                    if (at < next_end) {
                        s_list[at] = min(g[k].w & (kRefTop - 1u), capacity - 1u);
                        g[k].w = (g[k].w & ~(kRefTop - 1u)) | kRefTop | (uint32_t)at;
                    }
                    ++at;
                }
                top[4 * (begin + t) + k] = g[k];
            }
        }
        begin = end;
        end = next_end;
        __syncthreads();
    }
}

__global__ void tiny_scene(const float4* tmp, int nt, Node* out, float4* tris_out, QNode* qout, QFrame* frame,
                           DeviceSceneInfo* info, QNode* groups, QNode* top) {
    Node nd;
    if (nt == 0) {
        for (int k = 0; k < 3; ++k) { nd.lo[k] = 0.0f; nd.hi[k] = 0.0f; }
        nd.escape = 0;  // loop bound read by traversal: no nodes
        nd.payload = 0;
        info->n_nodes = 0;
    } else {
        float4 lo, hi;
        tri_box(tmp, lo, hi);
        nd.lo[0] = lo.x; nd.lo[1] = lo.y; nd.lo[2] = lo.z;
        nd.hi[0] = hi.x; nd.hi[1] = hi.y; nd.hi[2] = hi.z;
        nd.escape = 1;
        nd.payload = (0 << 3) | 1;
        transpose_tri(tmp, tris_out);
        info->n_nodes = 1;
    }
    out[0] = nd;
    QFrame F;
    qframe_of(make_float4(nd.lo[0], nd.lo[1], nd.lo[2], 0.0f), make_float4(nd.hi[0], nd.hi[1], nd.hi[2], 0.0f), F);
    qout[0] = quantise(F, nd);
    *frame = F;
    info->max_depth = 0;
    groups[0] = nt == 0 ? empty_record() : qout[0];
    for (int k = 1; k < 4; ++k) groups[k] = empty_record();
    for (int k = 0; k < 4; ++k) {
        groups[k].w |= kRefLive;
        top[k] = groups[k];
    }
    info->n_groups = 1;
}

__global__ void init_info(DeviceSceneInfo* info) {
    info->n_nodes = 0;
    info->max_depth = 0;
    info->bad_tris = 0;
    info->n_groups = 0;
    info->wide = 0;
    info->wide_bad = 0;
    info->n_big = 0;
    info->depth_complexity = 0.0f;
}

// Node counts, depth, and the depth complexity with the class it selects (one
// workgroup; the areas are summed in a fixed order).
__global__ __launch_bounds__(256) void finish_info(const Node* out, const EmitPart* part, int n_part, const int32_t* gflag,
                                                   const int32_t* gidx, int n_max, DeviceSceneInfo* info) {
    __shared__ double s_area[256];
    __shared__ int s_depth[256];
    const int t = threadIdx.x;
    double a = 0.0;
    int d = 0;
    for (int k = t; k < n_part; k += 256) {
        a += part[k].leaf_area;
        d = max(d, part[k].max_depth);
    }
    s_area[t] = a;
    s_depth[t] = d;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o) {
            s_area[t] += s_area[t + o];
            s_depth[t] = max(s_depth[t], s_depth[t + o]);
        }
        __syncthreads();
    }
    if (t != 0) return;
    const double root = box_area(out[0]);
    const double c = root > 0.0 ? s_area[0] / root : 0.0;
    info->n_nodes = out[0].escape;
    info->max_depth = s_depth[0];
    info->n_groups = gidx[n_max - 1] + gflag[n_max - 1];
    info->depth_complexity = (float)c;
    info->wide = (c >= (double)kWideDepthComplexity && info->wide_bad == 0) ? 1 : 0;
}

inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_tri_vertices(const float4* rows, int64_t n, float4* verts, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(tri_vertices, dim3(nblk(n)), dim3(256), 0, s, rows, n, verts);
    return hipGetLastError();
}

hipError_t build_bvh(const float* verts, int64_t nv, const int32_t* tris, int64_t nt64, Node* nodes_out,
                     float4* tris_out, QNode* qnodes_out, QFrame* frame_out, QNode* groups_out,
                     DeviceSceneInfo* info, const TempAlloc& ta, hipStream_t s, int* oom) {
    *oom = 0;
    const int nt = (int)nt64;
    hipLaunchKernelGGL(init_info, dim3(1), dim3(1), 0, s, info);
    const size_t n_nodes = nt > 0 ? (size_t)(2 * nt - 1) : 1;
    // temporary storage (one block, carved)
    size_t sort_bytes = 0;
    if (nt > 1) {
        hipError_t e = rocprim::radix_sort_pairs(nullptr, sort_bytes, (uint64_t*)nullptr, (uint64_t*)nullptr,
                                                 (uint32_t*)nullptr, (uint32_t*)nullptr, (size_t)nt, 0, 64, s);
        if (e != hipSuccess) return e;
    }
    size_t scan_bytes = 0;
    if (nt > 1) {
        hipError_t e = rocprim::exclusive_scan(nullptr, scan_bytes, (const int32_t*)nullptr, (int32_t*)nullptr, 0,
                                               n_nodes, rocprim::plus<int32_t>(), s);
        if (e != hipSuccess) return e;
    }
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t ntm = nt > 0 ? (size_t)nt : 1;
    const int nb = (int)((ntm + kFitBlock - 1) / kFitBlock);
    const int ns = (nb + kFitBlock - 1) / kFitBlock;   // super-blocks
    int sup_levels = 1;
    while ((1 << sup_levels) <= ns) ++sup_levels;      // 2^(sup_levels-1) <= ns < 2^sup_levels
    const unsigned n_part = nblk((int64_t)n_nodes);
    const size_t sz_tmp = al(sizeof(float4) * 3 * ntm), sz_keys = al(sizeof(uint64_t) * ntm),
                 sz_vals = al(sizeof(uint32_t) * ntm), sz_i = al(sizeof(int32_t) * n_nodes),
                 sz_box = al(sizeof(float4) * 2 * n_nodes), sz_cb = al(sizeof(int) * 8), sz_sort = al(sort_bytes),
                 sz_part = al(sizeof(float) * 6 * (size_t)nblk(ntm)), sz_nt = al(sizeof(int32_t) * ntm),
                 sz_nb = al(sizeof(int32_t) * (size_t)nb), sz_pre = al(sizeof(float4) * 2 * ntm),
                 sz_bpre = al(sizeof(float4) * 2 * (size_t)nb), sz_st = al(sizeof(float4) * 2 * (size_t)nb * kFitLevels),
                 sz_ns = al(sizeof(int32_t) * (size_t)(ns + 1)),
                 sz_sst = al(sizeof(float4) * 2 * (size_t)ns * (size_t)sup_levels), sz_ep = al(sizeof(EmitPart) * n_part);
    const size_t sz_scan = al(scan_bytes);
    const size_t total = sz_tmp + 2 * sz_keys + 2 * sz_vals + 10 * sz_i + sz_box + sz_cb + sz_sort + sz_part + 2 * sz_nt +
                         2 * sz_nb + 2 * sz_pre + 2 * sz_bpre + sz_st + 2 * sz_ns + sz_sst + sz_ep + sz_scan;
    char* base = (char*)ta.alloc(ta.ctx, total, s);
    if (!base) { *oom = 1; return hipErrorOutOfMemory; }
    char* p = base;
    auto take = [&](size_t b) { char* r = p; p += b; return r; };
    float4* tmp = (float4*)take(sz_tmp);
    uint64_t* keys = (uint64_t*)take(sz_keys);
    uint64_t* keys2 = (uint64_t*)take(sz_keys);
    uint32_t* vals = (uint32_t*)take(sz_vals);
    uint32_t* vals2 = (uint32_t*)take(sz_vals);
    Tree T;
    T.parent = (int32_t*)take(sz_i);
    T.left = (int32_t*)take(sz_i);
    T.right = (int32_t*)take(sz_i);
    T.first = (int32_t*)take(sz_i);
    T.last = (int32_t*)take(sz_i);
    T.axis = (int32_t*)take(sz_i);
    T.cnt = (int32_t*)take(sz_i);
    T.box = (float4*)take(sz_box);
    int* cb = (int*)take(sz_cb);
    void* sort_tmp = take(sz_sort);
    float* part = (float*)take(sz_part);
    T.mark = (int32_t*)take(sz_nt);
    T.mark_pre = (int32_t*)take(sz_nt);
    T.pre = (float4*)take(sz_pre);
    T.suf = (float4*)take(sz_pre);
    T.blk_mark = (int32_t*)take(sz_nb);
    T.blk_base = (int32_t*)take(sz_nb);
    T.blk_pre = (float4*)take(sz_bpre);
    T.blk_suf = (float4*)take(sz_bpre);
    T.st = (float4*)take(sz_st);
    T.sup_mark = (int32_t*)take(sz_ns);
    T.sup_base = (int32_t*)take(sz_ns);
    T.sup_st = (float4*)take(sz_sst);
    EmitPart* eparts = (EmitPart*)take(sz_ep);
    int32_t* gflag = (int32_t*)take(sz_i);
    int32_t* gidx = (int32_t*)take(sz_i);
    int32_t* naxis = (int32_t*)take(sz_i);
    void* scan_tmp = take(sz_scan);
    // the hoisted nodes follow the wide nodes in the same allocation
    QNode* top = groups_out + 4 * ntm;
    T.nb = nb;
    T.ns = ns;
    T.sup_levels = sup_levels;
    T.nbig = &info->n_big;
    hipError_t err = hipSuccess;
    if (nt > 0) {
        hipLaunchKernelGGL(tri_prep, dim3(nblk(nt)), dim3(256), 0, s, verts, nv, tris, (int64_t)nt, tmp, part, info);
        hipLaunchKernelGGL(bounds_reduce, dim3(1), dim3(256), 0, s, part, (int)nblk(nt), cb);
    }
    if (nt <= 1) {
        hipLaunchKernelGGL(tiny_scene, dim3(1), dim3(1), 0, s, tmp, nt, nodes_out, tris_out, qnodes_out, frame_out,
                           info, groups_out, top);
    } else {
        hipLaunchKernelGGL(morton, dim3(nblk(nt)), dim3(256), 0, s, tmp, (int64_t)nt, cb, keys, vals, info);
        err = rocprim::radix_sort_pairs(sort_tmp, sort_bytes, keys, keys2, vals, vals2, (size_t)nt, 0, 64, s);
        if (err == hipSuccess) {
            hipLaunchKernelGGL(big_sah, dim3(1), dim3(3 * kBigSah), 0, s, tmp, nt, keys2, vals2, info);
            hipLaunchKernelGGL(radix_tree, dim3(nblk(nt - 1)), dim3(256), 0, s, keys2, nt, T, gflag);
            hipLaunchKernelGGL(mark_leaves, dim3(nblk(2 * nt - 1)), dim3(256), 0, s, nt, T);
            hipLaunchKernelGGL(fit_block, dim3((unsigned)nb), dim3(kFitBlock), 0, s, tmp, vals2, nt, T, tris_out);
            hipLaunchKernelGGL(fit_super, dim3((unsigned)ns), dim3(kFitBlock), 0, s, T);
            if (ns > 1) hipLaunchKernelGGL(fit_mesh, dim3(1), dim3(1024), 0, s, T);
            if (nb > 1) hipLaunchKernelGGL(fit_top, dim3(nblk(nt - 1)), dim3(256), 0, s, nt, T);
            hipLaunchKernelGGL(emit, dim3(n_part), dim3(256), 0, s, nt, T, nodes_out, qnodes_out, frame_out, gflag, naxis,
                               eparts);
            err = rocprim::exclusive_scan(scan_tmp, scan_bytes, gflag, gidx, 0, (size_t)(2 * nt - 1),
                                          rocprim::plus<int32_t>(), s);
        }
        if (err == hipSuccess) {
            hipLaunchKernelGGL(wide_groups, dim3(nblk(2 * nt - 1)), dim3(256), 0, s, nodes_out, qnodes_out, gflag,
                               gidx, naxis, 2 * nt - 1, groups_out, info);
            hipLaunchKernelGGL(hoist_top, dim3(1), dim3(64), 0, s, groups_out, (uint32_t)nt, top);
            hipLaunchKernelGGL(finish_info, dim3(1), dim3(256), 0, s, nodes_out, eparts, (int)n_part, gflag, gidx,
                               2 * nt - 1, info);
        }
    }
    if (err == hipSuccess) err = hipGetLastError();
    ta.free(ta.ctx, base, s);
    return err;
}

}  // namespace mcdi
