// Cell build: the cells of section 3.1 of the Swift paper.
//
// Particles are binned into a uniform top grid per box whose cells are at
// least as wide as the largest search radius in the box (so every neighbour of
// a particle lies in the same or one of the 26 adjacent top cells, Fig. 1),
// then each top cell is refined as an octree: a cell is split when it holds
// more than leaf_target particles and at most one in eight of them has
// cell_ratio times its search radius wider than half the cell (the mesh
// "needs to be adaptive", section 3.1; pairs of cells are then found by box
// distance with each cell's own largest radius, so the few wide particles
// only give their small cells a longer reach). Leaves hold contiguous ranges
// of the Morton-sorted particles. For every leaf the tree is walked from the 27 surrounding top
// cells to collect each leaf within reach -- the cell-pair tasks, found with a
// tree as the end of section 3.1 describes -- with the periodic image of each.
//
// All of it runs on the GPU: integer keys, a radix sort, one pass of small
// kernels per tree level, and one walk per leaf over a stack of nodes in LDS. The
// host only reads back counts to size buffers.
#include "common.h"
#include "tiles.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int BS = 256;

__device__ __forceinline__ uint64_t spread3(uint32_t v)
{
    uint64_t x = v & 0x1fffffu;
    x = (x | x << 32) & 0x1f00000000ffffull;
    x = (x | x << 16) & 0x1f0000ff0000ffull;
    x = (x | x << 8) & 0x100f00f00f00f00full;
    x = (x | x << 4) & 0x10c30c30c30c30c3ull;
    x = (x | x << 2) & 0x1249249249249249ull;
    return x;
}

__device__ __forceinline__ uint32_t compact3(uint64_t x)
{
    x &= 0x1249249249249249ull;
    x = (x ^ (x >> 2)) & 0x10c30c30c30c30c3ull;
    x = (x ^ (x >> 4)) & 0x100f00f00f00f00full;
    x = (x ^ (x >> 8)) & 0x1f0000ff0000ffull;
    x = (x ^ (x >> 16)) & 0x1f00000000ffffull;
    x = (x ^ (x >> 32)) & 0x1fffffull;
    return (uint32_t)x;
}

struct KeyLayout {
    int bits_top;  // bits of the top-cell index
    int levels;    // octree levels below the top grid (3 key bits each)
    int low;       // key bits below the top-cell index: 3 levels of Morton bits, or
                   // (the first sort) the fine cell in z
};

// Raise base[key] to v over a workgroup of WBS threads (valid lanes only).
// Each wavefront reduces first; when every wavefront of the group holds one
// key (a single box, or the inside of a box) a single atomic per group
// remains, otherwise each wavefront adds its own. Same-address atomics
// serialise at the L2, so one per 64 lanes still cost tens of microseconds
// for a million particles. Every thread of the group must call it.
constexpr int WBS = 1024;
__device__ __forceinline__ void block_atomic_max_u32(unsigned* base, int key, unsigned v, bool valid)
{
    __shared__ int wkey[WBS / 64];
    __shared__ unsigned wmax[WBS / 64];
    __shared__ int wstate[WBS / 64];  // 0: no valid lane, 1: one key, 2: several keys
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    const bool any = __any(valid);
    const int kref = __shfl(valid ? key : 0x7fffffff, __ffsll((unsigned long long)__ballot(valid)) - 1, 64);
    const bool uni = __all(!valid || key == kref);
    unsigned m = valid ? v : 0u;
    for (int o = 32; o >= 1; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o, 64));
    if (lane == 0) {
        wkey[w] = kref;
        wmax[w] = m;
        wstate[w] = !any ? 0 : (uni ? 1 : 2);
    }
    __syncthreads();
    bool one = true;  // every wavefront with a valid lane holds one and the same key
    int k0 = -1;
    unsigned mm = 0u;
    for (int q = 0; q < nw; ++q) {
        if (wstate[q] == 0) continue;
        if (wstate[q] == 2 || (k0 >= 0 && wkey[q] != k0)) one = false;
        k0 = k0 < 0 ? wkey[q] : k0;
        mm = max(mm, wmax[q]);
    }
    if (one) {
        if (threadIdx.x == 0 && k0 >= 0) atomicMax(&base[k0], mm);
    } else if (uni) {
        if (lane == 0 && any) atomicMax(&base[kref], m);
    } else if (valid) {
        atomicMax(&base[key], v);
    }
}

__global__ void k_wrap(int64_t n, const double* __restrict__ pos, const int64_t* __restrict__ box_first,
                       int n_boxes, const double* __restrict__ box_len, const float* __restrict__ hg,
                       double* __restrict__ pos_w, float* __restrict__ hg_copy,
                       unsigned* __restrict__ box_hmax, float margin, int64_t* __restrict__ ctr)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool in_range = p < n;
    int b = 0;
    bool bad = false;
    float h = 0.0f;
    if (in_range) {
        b = box_of(box_first, n_boxes, p);
        const double L = box_len[b];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double x = pos[3 * p + a];
            bad |= !isfinite(x);
            double y = x - L * floor(x / L);
            if (!(y < L) || !(y >= 0.0)) y = 0.0;
            pos_w[3 * p + a] = y;
        }
        h = hg[p];
        bad |= !(h > 0.0f) || !isfinite(h);
        hg_copy[p] = h;
        if (bad) atomicAdd((unsigned long long*)&ctr[CT_BAD_INPUT], 1ull);
    }
    block_atomic_max_u32(box_hmax, b, __float_as_uint(margin * h), in_range && !bad);
}

// Largest search radius per box from the stored (caller-order) h guesses.
__global__ void k_box_hmax(int64_t n, const int64_t* __restrict__ box_first, int n_boxes,
                           const float* __restrict__ hg, unsigned* __restrict__ box_hmax, float margin,
                           int64_t* __restrict__ ctr)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool in_range = p < n;
    float h = 0.0f;
    int b = 0;
    bool ok = false;
    if (in_range) {
        h = hg[p];
        b = box_of(box_first, n_boxes, p);
        ok = (h > 0.0f) && isfinite(h);
        if (!ok) atomicAdd((unsigned long long*)&ctr[CT_BAD_INPUT], 1ull);
    }
    block_atomic_max_u32(box_hmax, b, __float_as_uint(margin * h), ok);
}

// Sort keys: box, top cell, and below it the Morton code of the particle's
// place (fzb < 0) or its fine cell, one of 2^fzb slices of the top cell in z.
__global__ void k_keys(int64_t n, const double* __restrict__ pos_w, const int64_t* __restrict__ box_first,
                       int n_boxes, const double* __restrict__ box_len, const int* __restrict__ box_G,
                       KeyLayout kl, int fzb, uint64_t* __restrict__ keys, uint32_t* __restrict__ vals)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int b = box_of(box_first, n_boxes, p);
    const int G = box_G[b];
    const double wtop = box_len[b] / G;
    const uint32_t nsub = fzb >= 0 ? 1u << fzb : 1u << kl.levels;
    uint32_t tc[3], sc[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double y = pos_w[3 * p + a];
        double c = floor(y / wtop);
        int ci = (int)c;
        ci = ci < 0 ? 0 : (ci >= G ? G - 1 : ci);
        double s = (y - ci * wtop) / wtop * (double)nsub;
        long si = (long)floor(s);
        si = si < 0 ? 0 : (si >= (long)nsub ? (long)nsub - 1 : si);
        tc[a] = (uint32_t)ci;
        sc[a] = (uint32_t)si;
    }
    const uint64_t top = ((uint64_t)tc[0] * G + tc[1]) * G + tc[2];
    const uint64_t below = fzb >= 0 ? (uint64_t)sc[2] : (spread3(sc[0]) << 2) | (spread3(sc[1]) << 1) | spread3(sc[2]);
    keys[p] = ((uint64_t)b << (kl.bits_top + kl.low)) | (top << kl.low) | below;
    vals[p] = (uint32_t)p;
}

// ---- the grid layout (no top cell split) -----------------------------------------------
// Particles sorted by box, column of top cells (x, y), z in fine cells. Work
// items take them 16 at a time along each column, whatever cells they are in:
// cells of a grid one search radius wide hold 8 to 27 particles, and items of
// single cells left a third of the lanes without a particle (a pass over 256
// boxes: 4.97 ms with one wavefront per cell, 5.12 ms with cells in items of at
// most 16, 3.47 ms along columns; gravity 1.20, 1.36 and 0.72 ms).

// Positions are 32-bit fractions of the box, or, from 16 cells a side, of one of its
// 2^k equal pieces, k so that a piece is 8 to 15 cells wide. What a frame holds lies
// within 3.5 cells of its centre (two of an item, one on either side, and the
// drift), so that differences wrap around a piece as they would around the box, and
// the fraction stays below 2^-28 of a cell's width: fractions of the whole box would
// be coarser than FP32 offsets from the cells' centres from about 128 cells a side
// on (2^-24 of the width at 256).
__host__ __device__ inline int piece_bits(int G)
{
    int k = 0;
    while (G >> (k + 1) >= 8) ++k;
    return k;
}

// First particle of every fine cell (starts[n_fine] = n): the thread of a
// particle that begins a cell also fills the empty cells before it, up to FINE_ALONE
// of them; longer stretches are filled by the whole workgroup. (Around a cylinder of
// 456,000 particles, 47 cells a side, one thread alone held a build up to 5.2 ms;
// 0.31 ms here.)
constexpr int FINE_ALONE = 16;

__global__ void __launch_bounds__(BS) k_fine_starts(int64_t n, const uint64_t* __restrict__ keys, KeyLayout kl,
                                                    const int64_t* __restrict__ box_top_base, int64_t n_fine,
                                                    int* __restrict__ starts)
{
    __shared__ int lo[BS + 1], hi[BS + 1], val[BS + 1];  // stretches [lo, hi]
    __shared__ int n_long;
    if (threadIdx.x == 0) n_long = 0;
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * BS + threadIdx.x;
    auto fine = [&](uint64_t k) {
        const int b = (int)(k >> (kl.bits_top + kl.low));
        return (int)((box_top_base[b] << kl.low) + (int64_t)(k & ((1ull << (kl.bits_top + kl.low)) - 1)));
    };
    auto fill = [&](int c0, int c1, int v) {
        if (c1 - c0 < FINE_ALONE) {
            for (int c = c0; c <= c1; ++c) starts[c] = v;
        } else {
            const int q = atomicAdd(&n_long, 1);
            lo[q] = c0;
            hi[q] = c1;
            val[q] = v;
        }
    };
    if (p < n) {
        const uint64_t k = keys[p];
        if (p == 0 || k != keys[p - 1]) fill(p == 0 ? 0 : fine(keys[p - 1]) + 1, fine(k), (int)p);
        if (p == n - 1) fill(fine(k) + 1, (int)n_fine, (int)n);
    }
    __syncthreads();
    for (int q = 0; q < n_long; ++q)
        for (int c = lo[q] + (int)threadIdx.x; c <= hi[q]; c += BS) starts[c] = val[q];
}

// Columns of box b: [col_base[b], col_base[b + 1]).
__device__ __forceinline__ int box_of_col(const int* col_base, int n_boxes, int r)
{
    int lo = 0, hi = n_boxes - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (col_base[mid] <= r) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// A column of top cells (one wavefront): its box, place and particles, and the
// fine cell in z of a particle.
struct Column {
    int b, G, gz, x, y, p0, p1;
    int64_t base, f;         // first fine cell of the box, of the column
    const uint64_t* keys;
    uint64_t mask;
    __device__ __forceinline__ int z(int p) const { return (int)((keys[p] & mask) - (uint64_t)(f - base)); }
};

__device__ __forceinline__ Column column_of(int r, int n_boxes, const int* col_base, const int* box_G,
                                            const int64_t* box_top_base, KeyLayout kl, const int* starts,
                                            const uint64_t* keys)
{
    Column c;
    c.b = box_of_col(col_base, n_boxes, r);
    c.G = box_G[c.b];
    c.gz = c.G << kl.low;
    const int xy = r - col_base[c.b];
    c.x = xy / c.G;
    c.y = xy % c.G;
    c.base = box_top_base[c.b] << kl.low;
    c.f = c.base + (int64_t)xy * c.gz;
    c.p0 = starts[c.f];
    c.p1 = starts[c.f + c.gz];
    c.keys = keys;
    c.mask = (1ull << (kl.bits_top + kl.low)) - 1;
    return c;
}

// A column's items are its particles 16 at a time; 16 that lie over more than
// ITEM_CELLS top cells (a sparse column) are cut into items that do not. FP32
// coordinates from an item's centre hold separations as well as offsets from the
// cells' centres do up to there and worse beyond (rms error of a separation over
// that of cell-centred offsets, 16 cells a side, along z and over the three axes:
// 0.95 and 0.95 at one cell, 1.11 and 1.01 at two, 1.50 and 1.16 at three, 2.64 and
// 1.71 at six). No cell is then the candidate of an item twice, with four cells per
// side or more. Whole columns in pieces of two cells instead: sedov 64^3 192 -> 200
// us a pass, for 2% of the runs are too long there, and a piece holds 19 particles.
constexpr int ITEM_CELLS = 2;

// Calls f(first, end) for the items of the particles [i0, i1) of a column, i1 - i0
// <= 16, and returns their number.
template <class F>
__device__ __forceinline__ int column_run(const Column& c, int fzb, int i0, int i1, F f)
{
    if (i0 >= i1) return 0;
    int n = 0, first = i0, z0 = c.z(i0);
    if (c.z(i1 - 1) - z0 >= ITEM_CELLS << fzb) {
        for (int i = i0 + 1; i < i1; ++i) {
            const int z = c.z(i);
            if (z - z0 < ITEM_CELLS << fzb) continue;
            f(n++, first, i);
            first = i;
            z0 = z;
        }
    }
    f(n++, first, i1);
    return n;
}

__global__ void __launch_bounds__(256) k_col_count(int n_cols, int n_boxes, const int* __restrict__ col_base,
                                                   const int* __restrict__ box_G,
                                                   const int64_t* __restrict__ box_top_base, KeyLayout kl,
                                                   const int* __restrict__ starts, const uint64_t* __restrict__ keys,
                                                   uint32_t* __restrict__ it_cnt)
{
    const int r = (int)(((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= n_cols) return;  // whole wavefronts
    const Column c = column_of(r, n_boxes, col_base, box_G, box_top_base, kl, starts, keys);
    int n = 0;
    for (int i0 = c.p0 + 16 * lane; i0 < c.p1; i0 += 16 * 64)
        n += column_run(c, kl.low, i0, min(i0 + 16, c.p1), [](int, int, int) {});
    for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o, 64);
    if (lane == 0) it_cnt[r] = (uint32_t)n;
}

// The items of each column (one wavefront per column) and the first item of
// each box.
__global__ void __launch_bounds__(256) k_col_items(int n_cols, int n_boxes, const int* __restrict__ col_base,
                                                   const int* __restrict__ box_G, const double* __restrict__ box_len,
                                                   const int64_t* __restrict__ box_top_base, KeyLayout kl,
                                                   const int* __restrict__ starts, const uint64_t* __restrict__ keys,
                                                   const uint32_t* __restrict__ it_start, int4* __restrict__ cells,
                                                   int* __restrict__ box_item)
{
    const int r = (int)(((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= n_cols) return;  // whole wavefronts
    const Column c = column_of(r, n_boxes, col_base, box_G, box_top_base, kl, starts, keys);
    const double pieces = 4294967296.0 * (double)(1 << piece_bits(c.G));
    const double unit = box_len[c.b] / pieces;
    const float sh = (float)unit, sl = (float)(unit - (double)sh);
    const unsigned step = (unsigned)(pieces / c.G);
    int64_t it = it_start[r];
    if (lane == 0) {
        if (c.x == 0 && c.y == 0) box_item[c.b] = (int)it;
        if (r == n_cols - 1) box_item[n_boxes] = (int)it_start[n_cols];
    }
    for (int i = c.p0; i < c.p1; i += 16 * 64) {
        const int i0 = i + 16 * lane, i1 = min(i0 + 16, c.p1);
        int all;
        const int64_t k = it + wave_excl_scan(column_run(c, kl.low, i0, i1, [](int, int, int) {}), all);
        column_run(c, kl.low, i0, i1, [&](int q, int a, int b) {
            cells[2 * (k + q)] = make_int4(a, (b - a) | (c.G << 8), c.x | (c.y << 16), c.z(a) | (c.z(b - 1) << 16));
            cells[2 * (k + q) + 1] = make_int4((int)c.base, __float_as_int(sh), __float_as_int(sl), (int)step);
        });
        it += all;
    }
}

// Positions as 32-bit fractions (piece_bits), sorted: differences are exact and
// wrap around the box by themselves.
__global__ void k_fix_fill(int64_t n, const uint32_t* __restrict__ perm, const double* __restrict__ pos_w,
                           const int64_t* __restrict__ box_first, int n_boxes, const double* __restrict__ box_len,
                           const int* __restrict__ box_G, int4* __restrict__ xfix)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t o = perm[p];
    const int b = box_of(box_first, n_boxes, o);
    const double s = 4294967296.0 * (double)(1 << piece_bits(box_G[b])) / box_len[b];
    int v[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = (int)(unsigned)(unsigned long long)llrint(pos_w[3 * o + a] * s);
    xfix[p] = make_int4(v[0], v[1], v[2], 0);
}

// As k_cell_pbox for a grid layout: the box's centre in 32-bit fractions. The
// particles are measured from the middle of the item's cells, which no particle is
// half the box away from: differences from one of the particles would wrap in an item
// longer than half the box, and the frame around the wrapped box would tear its pairs
// apart.
__global__ void __launch_bounds__(256) k_fix_pbox(int64_t n_items, const int4* __restrict__ cells, int fzb,
                                                  const int4* __restrict__ xfix, const float* __restrict__ Hs,
                                                  float4* __restrict__ pbox)
{
    const int64_t it = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
    const int sub = threadIdx.x & 15;
    const bool live = it < n_items;
    const int4 c0 = live ? cells[2 * it] : make_int4(0, 0, 0, 0);
    const int ni = c0.y & 0xff;
    unsigned x0[3] = {0u, 0u, 0u};
    if (live) {
        const unsigned step = (unsigned)cells[2 * it + 1].w, fstep = step >> fzb;  // width of a cell, of a fine one
        const unsigned z0 = (unsigned)(c0.w & 0xffff), z1 = (unsigned)(c0.w >> 16) + 1u;
        x0[0] = (unsigned)(c0.z & 0xffff) * step + (step >> 1);
        x0[1] = (unsigned)(c0.z >> 16) * step + (step >> 1);
        x0[2] = z0 * fstep + (((z1 - z0) * fstep) >> 1);
    }
    // (lanes past the item's particles repeat its first)
    const int4 x = live ? xfix[c0.x + (sub < ni ? sub : 0)] : make_int4(0, 0, 0, 0);
    int lo[3], hi[3];
    lo[0] = hi[0] = (int)((unsigned)x.x - x0[0]);
    lo[1] = hi[1] = (int)((unsigned)x.y - x0[1]);
    lo[2] = hi[2] = (int)((unsigned)x.z - x0[2]);
    float H = live && sub < ni ? Hs[c0.x + sub] : 0.0f;
    for (int o = 8; o >= 1; o >>= 1) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = min(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = max(hi[a], __shfl_xor(hi[a], o, 64));
        }
        H = fmaxf(H, __shfl_xor(H, o, 64));
    }
    if (live && sub == 0) {
        const int4 c1 = cells[2 * it + 1];
        const double u = (double)__int_as_float(c1.y) + (double)__int_as_float(c1.z);
        unsigned o[3];
        float h[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const long long mid = ((long long)lo[a] + (long long)hi[a]) >> 1;
            o[a] = x0[a] + (unsigned)mid;
            h[a] = (float)((double)((long long)hi[a] - mid) * u) * 1.00001f;
        }
        pbox[2 * it] = make_float4(__int_as_float((int)o[0]), __int_as_float((int)o[1]), __int_as_float((int)o[2]), H);
        pbox[2 * it + 1] = make_float4(h[0], h[1], h[2], 0.0f);
    }
}

// Sorted search radii; also no drift yet (sph_ctx::drift: bound, step maximum,
// smallest search radius before its minimum, non-finite flag).
__global__ void k_sorted_H(int64_t n, const uint32_t* __restrict__ perm, const float* __restrict__ hg,
                           float margin, float* __restrict__ Hs, int* __restrict__ leaf_tmp,
                           unsigned* __restrict__ drift)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < 4) drift[p] = p == 2 ? 0x7f800000u : 0u;
    if (p >= n) return;
    Hs[p] = margin * hg[perm[p]];
    if (leaf_tmp) leaf_tmp[p] = -1;
}

__global__ void k_lvl_head(int64_t n, const uint64_t* __restrict__ keys, const int* __restrict__ leaf_tmp,
                           int shift, uint32_t* __restrict__ head)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    uint32_t h = 0;
    if (leaf_tmp[p] < 0) {
        h = (p == 0) || (leaf_tmp[p - 1] >= 0) || ((keys[p] >> shift) != (keys[p - 1] >> shift));
    }
    head[p] = h;
}

// Node of every unassigned particle at level l; node start, count, largest
// search radius, and the number of particles whose search radius is too wide
// for half the node (cell_ratio * H > w / 2).
__global__ void k_lvl_nodes(int64_t n, const uint64_t* __restrict__ keys, const int* __restrict__ leaf_tmp,
                            const uint32_t* __restrict__ head, const uint32_t* __restrict__ excl,
                            const float* __restrict__ Hs, int level, KeyLayout kl, int64_t node_base,
                            int* __restrict__ nid, int* __restrict__ nd_start, int* __restrict__ nd_count,
                            unsigned* __restrict__ nd_hmax, int* __restrict__ nd_wide, int* __restrict__ nd_box,
                            int* __restrict__ nd_level, int* __restrict__ nd_coord,
                            const int* __restrict__ box_G, const double* __restrict__ box_len, float cell_ratio)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = p < n && leaf_tmp[p] < 0;
    int id = -1;
    unsigned hb = 0u;
    int wide = 0;
    if (valid) {
        id = (int)(node_base + (int64_t)excl[p] + head[p] - 1);
        nid[p] = id;
        const uint64_t k = keys[p];
        const int b = (int)(k >> (kl.bits_top + kl.low));
        const double w = box_len[b] / box_G[b] / (double)(1u << level);
        const float H = Hs[p];
        hb = __float_as_uint(H);
        wide = (double)(cell_ratio * H) > 0.5 * w ? 1 : 0;
    }
    // The particles of a node are consecutive among the valid lanes (sorted
    // order; lanes of assigned particles only sit between nodes), so a scan
    // that combines equal ids gives each run's totals in its last lane, and
    // one atomic per run and array remains instead of one per particle.
    const int lane = threadIdx.x & 63;
    int cnt = valid ? 1 : 0, wsum = wide;
    unsigned hmx = hb;
    for (int o = 1; o < 64; o <<= 1) {
        const int id_o = __shfl_up(id, o, 64);
        const int c_o = __shfl_up(cnt, o, 64);
        const int w_o = __shfl_up(wsum, o, 64);
        const unsigned h_o = (unsigned)__shfl_up((int)hmx, o, 64);
        if (valid && lane >= o && id_o == id) {
            cnt += c_o;
            wsum += w_o;
            hmx = max(hmx, h_o);
        }
    }
    const int id_next = __shfl_down(id, 1, 64);
    if (valid && (lane == 63 || id_next != id)) {
        atomicAdd(&nd_count[id], cnt);
        atomicMax(&nd_hmax[id], hmx);
        if (wsum) atomicAdd(&nd_wide[id], wsum);
    }
    if (valid && head[p]) {
        const uint64_t k = keys[p];
        const int b = (int)(k >> (kl.bits_top + kl.low));
        const uint64_t top = (k >> kl.low) & ((1ull << kl.bits_top) - 1);
        const int G = box_G[b];
        const uint64_t pre = level > 0 ? (k & ((1ull << kl.low) - 1)) >> (3 * (kl.levels - level)) : 0;
        const uint32_t mx = compact3(pre >> 2), my = compact3(pre >> 1), mz = compact3(pre);
        const uint32_t tz = (uint32_t)(top % G), ty = (uint32_t)((top / G) % G), tx = (uint32_t)(top / ((uint64_t)G * G));
        nd_start[id] = (int)p;
        nd_box[id] = b;
        nd_level[id] = level;
        nd_coord[3 * id + 0] = (int)((tx << level) | mx);
        nd_coord[3 * id + 1] = (int)((ty << level) | my);
        nd_coord[3 * id + 2] = (int)((tz << level) | mz);
    }
}

// A node is split when it holds more than leaf_target particles and at most
// one in eight of them has a search radius too wide for half its width. The
// wide few then sit in small cells with a long reach (pairs are found by box
// distance with each cell's own largest radius), instead of a few outliers
// keeping every particle of a dense region in one huge cell.
// The per-level kernels below run over a bound on the level's node count
// that the host knows (the launch), and take the count itself (*dM) from the
// device: slots k in [*dM, bound) hold no node.
// The sums of a level's nodes; at the first level also the table of top cells.
__global__ void k_lvl_clear(int64_t node_base, int64_t bound, int* __restrict__ nd_count,
                            unsigned* __restrict__ nd_hmax, int* __restrict__ nd_wide, int64_t n_top,
                            int* __restrict__ top)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n_top) top[k] = -1;
    if (k >= bound) return;
    nd_count[node_base + k] = 0;
    nd_hmax[node_base + k] = 0u;
    nd_wide[node_base + k] = 0;
}

__global__ void k_lvl_decide(int64_t bound, const uint32_t* __restrict__ dM, int64_t node_base, int level,
                             int max_level, int leaf_target, const int* __restrict__ nd_count,
                             const int* __restrict__ nd_wide, uint32_t* __restrict__ nflag,
                             int* __restrict__ nd_child0, int* __restrict__ nd_child1)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= bound) return;
    if (k >= (int64_t)*dM) {  // no node: not a leaf either (the scan of nflag counts the leaves)
        nflag[k] = 0u;
        return;
    }
    const int64_t id = node_base + k;
    const int cnt = nd_count[id];
    const bool split = level < max_level && cnt > leaf_target && 8 * nd_wide[id] <= cnt;
    nflag[k] = split ? 0u : 1u;
    nd_child0[id] = -1;
    nd_child1[id] = -1;
}

__global__ void k_lvl_leaves(int64_t bound, const uint32_t* __restrict__ dM, int64_t node_base, int64_t leaf_base,
                             const uint32_t* __restrict__ nflag, const uint32_t* __restrict__ nscan,
                             int* __restrict__ nd_leaf, int* __restrict__ lo2node)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= bound || k >= (int64_t)*dM) return;
    const int64_t id = node_base + k;
    if (nflag[k]) {
        const int64_t lo = leaf_base + nscan[k];
        nd_leaf[id] = (int)lo;
        lo2node[lo] = (int)id;
    } else {
        nd_leaf[id] = -1;
    }
}

__global__ void k_lvl_assign(int64_t n, const int* __restrict__ nid, const int* __restrict__ nd_leaf,
                             int* __restrict__ leaf_tmp)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n || leaf_tmp[p] >= 0) return;
    const int lf = nd_leaf[nid[p]];
    if (lf >= 0) leaf_tmp[p] = lf;
}

// Children of the split nodes of the previous level: the level-l nodes holding
// the first and last particle of each split parent (level-l nodes are
// numbered in particle order, so a parent's children are the ids between).
__global__ void k_lvl_children(int64_t Mprev, int64_t base_prev, const int* __restrict__ nd_leaf,
                               const int* __restrict__ nd_start, const int* __restrict__ nd_count,
                               const int* __restrict__ nid, int* __restrict__ nd_child0,
                               int* __restrict__ nd_child1)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= Mprev) return;
    const int64_t id = base_prev + k;
    if (nd_leaf[id] >= 0) return;
    const int s = nd_start[id];
    const int c0 = nid[s], c1 = nid[s + nd_count[id] - 1];
    nd_child0[id] = c0;
    nd_child1[id] = c1;
}

__global__ void k_top_table(int64_t bound, const uint32_t* __restrict__ dM, const int* __restrict__ nd_box,
                            const int* __restrict__ nd_coord, const int* __restrict__ box_G,
                            const int64_t* __restrict__ box_top_base, int* __restrict__ top)
{
    int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= bound || id >= (int64_t)*dM) return;
    const int b = nd_box[id];
    const int G = box_G[b];
    const int64_t t = ((int64_t)nd_coord[3 * id] * G + nd_coord[3 * id + 1]) * G + nd_coord[3 * id + 2];
    top[box_top_base[b] + t] = (int)id;
}

__global__ void k_leaf_head(int64_t n, const int* __restrict__ leaf_tmp, uint32_t* __restrict__ head)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    head[p] = (p == 0) || (leaf_tmp[p] != leaf_tmp[p - 1]);
}

__global__ void k_leaf_fill(int64_t n, const uint32_t* __restrict__ head, const uint32_t* __restrict__ excl,
                            const int* __restrict__ leaf_tmp, const int* __restrict__ lo2node,
                            int* __restrict__ leaf_of, int* __restrict__ lf_start, int* __restrict__ lf_node)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int L = (int)(excl[p] + head[p]) - 1;
    leaf_of[p] = L;
    if (head[p]) {
        lf_start[L] = (int)p;
        lf_node[L] = lo2node[leaf_tmp[p]];
    }
}

// First item of each box (tree): leaves follow the sorted particles, whose
// boxes are contiguous blocks, and items the leaves.
__global__ void k_box_item(int n_boxes, int64_t n, int64_t nl, const int64_t* __restrict__ box_first,
                           const int* __restrict__ leaf_of, const uint32_t* __restrict__ it_start,
                           int* __restrict__ box_item)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b > n_boxes) return;
    const int64_t p = box_first[b];
    box_item[b] = (int)it_start[p < n ? leaf_of[p] : nl];
}

__global__ void k_leaf_fix(int64_t nl, const int* __restrict__ lf_node, const int* __restrict__ nd_count,
                           const unsigned* __restrict__ nd_hmax, int* __restrict__ nd_leaf,
                           int* __restrict__ lf_count, float* __restrict__ lf_hmax)
{
    int64_t L = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (L >= nl) return;
    const int id = lf_node[L];
    nd_leaf[id] = (int)L;
    lf_count[L] = nd_count[id];
    lf_hmax[L] = __uint_as_float(nd_hmax[id]);
}

// The leaves where no top cell splits: they are the level-0 nodes, whose order is
// the particles' already (nid: the node of each particle), so one kernel stands
// for the renumbering, its scan and the packing of the tree (seven launches; a
// leapfrog step with a rebuild at 48^3 particles 261 -> 249 us).
__global__ void k_leaf_top(int64_t n, int64_t nl, const int* __restrict__ nid, const int* __restrict__ nd_start,
                           const int* __restrict__ nd_count, const unsigned* __restrict__ nd_hmax,
                           const int* __restrict__ nd_coord, int* __restrict__ leaf_of, int* __restrict__ lf_start,
                           int* __restrict__ lf_node, int* __restrict__ lf_count, float* __restrict__ lf_hmax,
                           int4* __restrict__ nodes)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) leaf_of[p] = nid[p];
    if (p >= nl) return;
    const int cnt = nd_count[p];
    const unsigned h = nd_hmax[p];
    lf_start[p] = nd_start[p];
    lf_node[p] = (int)p;
    lf_count[p] = cnt;
    lf_hmax[p] = __uint_as_float(h);
    nodes[2 * p] = make_int4(nd_coord[3 * p], nd_coord[3 * p + 1], nd_coord[3 * p + 2], 0);
    nodes[2 * p + 1] = make_int4((int)h, (int)p, cnt, 0);
}

// Centre and width of a node with integer coordinates (x, y, z) and level w.
__device__ __forceinline__ void node_box(int4 n, double wtop, double c[3], double& w)
{
    w = ldexp(wtop, -n.w);
    c[0] = ((double)n.x + 0.5) * w;
    c[1] = ((double)n.y + 0.5) * w;
    c[2] = ((double)n.z + 0.5) * w;
}

// The 27 top cells around a leaf's own, in the order its partner list visits
// them: three classes of (dx + dy + dz) mod 3, nine cells each, every class
// spread over the whole 3x3x3 block. The hot kernels stage a list in
// consecutive chunks, and a chunk that samples the whole neighbourhood gives
// every particle a similar share of its neighbours (even lane lists).
__constant__ signed char NB27[27][3] = {
    {-1, -1, -1}, {-1, 0, 1}, {-1, 1, 0}, {0, -1, 1}, {0, 0, 0}, {0, 1, -1}, {1, -1, 0}, {1, 0, -1}, {1, 1, 1},
    {-1, -1, 0}, {-1, 0, -1}, {-1, 1, 1}, {0, -1, -1}, {0, 0, 1}, {0, 1, 0}, {1, -1, 1}, {1, 0, 0}, {1, 1, -1},
    {-1, -1, 1}, {-1, 0, 0}, {-1, 1, -1}, {0, -1, 0}, {0, 0, -1}, {0, 1, 1}, {1, -1, -1}, {1, 0, 1}, {1, 1, 0}};

// The tree as the walks below read it, two words of 16 bytes per node: integer
// centre and level; largest search radius (bits), leaf or -1 - first child,
// particles of a leaf or number of children (their ids are consecutive), -.
struct TreeView {
    const int4* nodes;
    int n_nodes;
};

__global__ void k_tree_pack(int64_t n_nodes, const int* __restrict__ nd_coord, const int* __restrict__ nd_level,
                            const unsigned* __restrict__ nd_hmax, const int* __restrict__ nd_leaf,
                            const int* __restrict__ nd_child0, const int* __restrict__ nd_child1,
                            const int* __restrict__ lf_count,
                            int4* __restrict__ nodes)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= n_nodes) return;
    const int lf = nd_leaf[id];
    nodes[2 * id] = make_int4(nd_coord[3 * id], nd_coord[3 * id + 1], nd_coord[3 * id + 2], nd_level[id]);
    nodes[2 * id + 1] = make_int4((int)nd_hmax[id], lf >= 0 ? lf : -1 - nd_child0[id],
                                  lf >= 0 ? lf_count[lf] : nd_child1[id] - nd_child0[id] + 1, 0);
}

struct RecordOut {
    int* p_leaf;
    float4* p_shift;
    uint8_t* p_code;
    int2* p_rec;
    const int* lf_start;
    const int* lf_count;
    const uint32_t* it_start;  // null: no items
};

// Sums over the 32 lanes of a half-wavefront.
__device__ __forceinline__ uint32_t half_sum(uint32_t v)
{
    for (int o = 16; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Exclusive prefix sum over the 32 lanes of a half-wavefront.
__device__ __forceinline__ uint32_t half_excl_scan(uint32_t v)
{
    const int q = threadIdx.x & 31;
    uint32_t s = v;
    for (int o = 1; o < 32; o <<= 1) {
        const uint32_t t = __shfl_up(s, o, 32);
        if (q >= o) s += t;
    }
    return s - v;
}

constexpr int PBS = 256;

// Counters k0 + k of the workgroup's values v[k]: the total for k < n_sum,
// the largest value for the others. One atomic per counter and workgroup,
// into its spread slot (one per wavefront would be 10^5 atomics on a few
// cache lines for the largest sets). Every thread of the group must call it.
template <int NV>
__device__ __forceinline__ void block_counters(const int64_t (&v)[NV], int64_t (&red)[NV][PBS / 64],
                                               int64_t* __restrict__ ctr, int k0, int n_sum)
{
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        int64_t x = v[k];
        for (int o = 32; o >= 1; o >>= 1) {
            const int64_t y = __shfl_xor(x, o, 64);
            x = k < n_sum ? x + y : max(x, y);
        }
        if ((threadIdx.x & 63) == 0) red[k][w] = x;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        const int k = threadIdx.x;
        int64_t x = red[k][0];
        for (int q = 1; q < PBS / 64; ++q) x = k < n_sum ? x + red[k][q] : max(x, red[k][q]);
        unsigned long long* slot = (unsigned long long*)&ctr_slot(ctr)[k0 + k];
        if (k < n_sum) {
            if (x != 0) atomicAdd(slot, (unsigned long long)x);
        } else {
            atomicMax(slot, (unsigned long long)x);
        }
    }
}

// Work items of the hot kernels: the particles of a leaf in runs of at most
// ITEM_N, one wavefront each. A wavefront takes ITEM_N particles at a time
// (four lanes per particle), so a leaf of more would be a serial loop: as
// separate items its runs go to several wavefronts (a box of 16^3 particles
// has 125 leaves of 27 to 64 particles for 1024 SIMDs). item_range.h says which
// particles an item holds.
constexpr int ITEM_N = 16;

__global__ void k_item_count(int64_t nl, const int* __restrict__ lf_count, uint32_t* __restrict__ it_cnt)
{
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a < nl) it_cnt[a] = (uint32_t)((lf_count[a] + ITEM_N - 1) / ITEM_N);
}

// The cell-pair tasks (section 3.1: the neighbouring cells of each leaf, found
// with a tree), one half-wavefront per leaf a: every leaf whose box lies within
// max(HA, its own largest radius) of a's box, HA the largest radius in a. fill ==
// 0 counts each leaf's records (all into p_cnt, the density's into p_cntd). fill
// == 1 writes the list at p_start[a], in two parts: first the leaves within HA
// (p_cntd[a] of them), then those that reach a only with their own radius. The
// density of a's particles (a gather over j inside h_i <= HA) needs only the
// first part; the force (pairs inside max(h_i, h_j)) takes both. The count also
// adds up the build's shape counters (CT_B_*). The fill also writes (it_start !=
// null) the leaf of each of its work items and the item's schedule key (sk !=
// null), its cost particles x candidates as 12 bits of its float (exponent and
// four bits of mantissa) in decreasing order, prefixed with the XCD whose Morton
// range holds the item when xcd_local.
//
// The nodes still to be tested, at first the 27 surrounding top cells, wait on a
// stack in LDS, and every step tests its uppermost 32 at once: a walk visits
// hundreds of nodes where the set is clustered, most of them below two or three
// of the top cells, so a lane per top cell left the rest idle behind the longest
// walk and took a memory latency per node (clustered 2^20: 1.10 ms a call, 0.23
// here; log-normal 2^24: 11 ms and 1.7; 0.73 with the packed nodes alone). The
// order is fixed, so the lists have the same records in the same order in every
// build. A step takes fewer nodes where their children could overrun
// PSTACK; single nodes add at most seven per level after that.
constexpr int PSTACK = 256;
constexpr int MAX_LEVELS = 10;
constexpr int PSTACK_ALL = PSTACK + 7 * MAX_LEVELS + 2;

__global__ void __launch_bounds__(PBS) k_partners(int64_t nl, int fill, const int* __restrict__ lf_node,
                                                  TreeView tv, const int* __restrict__ nd_box,
                                                  const int* __restrict__ top,
                                                  const int64_t* __restrict__ box_top_base,
                                                  const int* __restrict__ box_G, const double* __restrict__ box_len,
                                                  uint32_t* __restrict__ p_cnt, uint32_t* __restrict__ p_cntd,
                                                  const uint32_t* __restrict__ p_start, RecordOut ro,
                                                  const uint32_t* __restrict__ it_start, int64_t n_items,
                                                  int* __restrict__ it_leaf, uint64_t* __restrict__ sk,
                                                  uint32_t* __restrict__ sv, int xcd_local, int64_t* __restrict__ ctr)
{
    const int q = threadIdx.x & 31, half = threadIdx.x >> 5, upper = threadIdx.x & 32;
    const int64_t a = ((int64_t)blockIdx.x * PBS + threadIdx.x) >> 5;
    const bool leaf_ok = a < nl;
    __shared__ int st_node[PBS / 32][PSTACK_ALL];
    __shared__ uint8_t st_code[PBS / 32][PSTACK_ALL];
    __shared__ int64_t red[5][PBS / 64];
    int* const sn = st_node[half];
    uint8_t* const sc = st_code[half];
    auto half_ballot = [&](bool v) { return (uint32_t)(__ballot(v) >> upper); };
    const uint32_t below = (1u << q) - 1u;
    double cA[3] = {0.0, 0.0, 0.0}, wA = 0.0, wtop = 1.0, L = 0.0;
    float HA = 0.0f;
    int T = -1, code = 0;
    if (leaf_ok) {
        const int A = lf_node[a];
        const int b = nd_box[A];
        const int G = box_G[b];
        L = box_len[b];
        wtop = L / G;
        const int4 nA = tv.nodes[2 * (int64_t)A];
        node_box(nA, wtop, cA, wA);
        HA = __int_as_float(tv.nodes[2 * (int64_t)A + 1].x);
        if (q < 27) {
            const int tA[3] = {nA.x, nA.y, nA.z};
            int t[3], s[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                t[k] = (tA[k] >> nA.w) + NB27[q][k];
                s[k] = 0;
                if (t[k] < 0) { t[k] += G; s[k] = -1; }
                else if (t[k] >= G) { t[k] -= G; s[k] = 1; }
            }
            T = top[box_top_base[b] + ((int64_t)t[0] * G + t[1]) * G + t[2]];
            code = image_code(s[0], s[1], s[2]);
        }
    }
    const double eps = 1e-9 * wtop, HA2 = (double)HA * (double)HA;
    int size = 0;  // of the half's stack
    {
        const uint32_t m = half_ballot(T >= 0);
        if (T >= 0) {
            const int d = __popc(m & below);
            sn[d] = T;
            sc[d] = (uint8_t)code;
        }
        size = __popc(m);
    }
    uint32_t nd = 0, nf = 0;  // records so far
    int nj = 0;               // particles of this lane's
    const uint32_t od = fill && leaf_ok ? p_start[a] : 0u, of = fill && leaf_ok ? od + p_cntd[a] : 0u;
    for (int64_t steps = 0; __any(size > 0); ++steps) {
        if (steps > 27 * (int64_t)tv.n_nodes) {  // (whole wavefront) more than any tree has
            if ((threadIdx.x & 63) == 0) atomicAdd((unsigned long long*)&ctr[CT_BAD_INPUT], 1ull);
            break;
        }
        wave_sync_lds();
        const int m = min(min(32, size), max(1, (PSTACK - size) / 7));
        size -= m;
        bool dens = false, far = false;
        int kids = 0, child = 0, lf = 0, cnt = 0, img = 0;
        float4 sh = make_float4(0.f, 0.f, 0.f, 0.f);
        if (q < m) {
            const int64_t X = sn[size + q];
            img = sc[size + q];
            const int4 na = tv.nodes[2 * X], nb = tv.nodes[2 * X + 1];
            double cX[3], wX;
            node_box(na, wtop, cX, wX);
            const double S[3] = {image_shift(img, 0, L), image_shift(img, 1, L), image_shift(img, 2, L)};
            double d2 = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                double g = fabs(cX[k] + S[k] - cA[k]) - 0.5 * (wA + wX) - eps;
                g = g > 0.0 ? g : 0.0;
                d2 += g * g;
            }
            const double R = (double)fmaxf(HA, __int_as_float(nb.x));
            if (d2 < R * R) {
                if (nb.y < 0) {
                    child = -1 - nb.y;
                    kids = nb.z;
                } else {
                    lf = nb.y;
                    cnt = nb.z;
                    nj += cnt;
                    dens = d2 < HA2;
                    far = !dens;
                    sh = make_float4((float)(cX[0] + S[0] - cA[0]), (float)(cX[1] + S[1] - cA[1]),
                                     (float)(cX[2] + S[2] - cA[2]), 0.0f);
                }
            }
        }
        const uint32_t md = half_ballot(dens), mf = half_ballot(far);
        if (fill && (dens || far)) {
            const uint32_t o = dens ? od + nd + __popc(md & below) : of + nf + __popc(mf & below);
            sh.w = __int_as_float(ro.it_start ? (int)ro.it_start[lf] : 0);
            ro.p_leaf[o] = lf;
            ro.p_rec[o] = make_int2(ro.lf_start[lf], cnt);
            ro.p_shift[o] = sh;
            ro.p_code[o] = (uint8_t)img;
        }
        nd += __popc(md);
        nf += __popc(mf);
        // the children, on the stack
        const uint32_t at = half_excl_scan((uint32_t)kids);
        wave_sync_lds();  // every lane has read its node
        for (int k = 0; k < kids; ++k) {
            sn[size + at + k] = child + k;
            sc[size + at + k] = (uint8_t)img;
        }
        size += __shfl((int)at + kids, 31, 32);
    }
    if (!fill) {
        const int tj = (int)half_sum((uint32_t)nj);
        const bool lead = leaf_ok && q == 0;
        if (lead) {
            p_cnt[a] = nd + nf;
            p_cntd[a] = nd;
        }
        // the build's shape: the candidate pairs and the records of all leaves
        // (in 64 bits: the list offsets are a 32-bit scan), then the maxima
        const int ni = leaf_ok ? ro.lf_count[a] : 0;
        const int64_t r[5] = {lead ? (int64_t)ni * tj : 0, lead ? (int64_t)(nd + nf) : 0, lead ? ni : 0,
                              lead ? (int64_t)(nd + nf) : 0, lead ? tj : 0};
        block_counters<5>(r, red, ctr, CT_B_CAND_PAIRS, 2);
        return;
    }
    if (!it_start) return;
    nj = (int)half_sum((uint32_t)nj);
    if (leaf_ok) {
        // the leaf's work items, one lane each
        const int ni = ro.lf_count[a];
        const int t0 = (int)it_start[a], nt = (int)it_start[a + 1] - t0;
        for (int t = q; t < nt; t += 32) {
            const int it = t0 + t;
            it_leaf[it] = (int)a;
            if (!sk) continue;
            const float cost = (float)(item_first(ni, nt, t + 1) - item_first(ni, nt, t)) * (float)nj;
            uint64_t x = 0;
            if (xcd_local)
                while (x < 7 && it >= sph::xcd_start(n_items, (int)x + 1)) ++x;
            sk[it] = (x << 12) | (uint64_t)(0xfffu - (__float_as_uint(cost) >> 19));
            sv[it] = (uint32_t)it;
        }
    }
}

// Schedule slots, one per work item. by_cost != null and deal: the item of
// cost rank r goes to slot xcd_start(n, r % 8) + r / 8. by_cost != null, no
// deal: slot r holds the item of rank r (the ranks already group each XCD's
// range). by_cost == null: slot r holds item r (Morton order, so each XCD
// takes a contiguous range of neighbouring cells).
__global__ void k_sched_fill(int64_t n_items, const uint32_t* __restrict__ by_cost, int deal,
                             const int* __restrict__ it_leaf, const uint32_t* __restrict__ it_start,
                             const int* __restrict__ lf_start, const int* __restrict__ lf_count,
                             const uint32_t* __restrict__ p_start, const uint32_t* __restrict__ p_cntd,
                             int4* __restrict__ cells, int* __restrict__ cell_item, int4* __restrict__ cells_d)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_items) return;
    const int it = by_cost ? (int)by_cost[r] : (int)r;
    const int64_t slot = by_cost && deal ? sph::xcd_start(n_items, (int)(r & 7)) + (r >> 3) : r;
    const int a = it_leaf[it];
    const int t0 = (int)it_start[a], nt = (int)it_start[a + 1] - t0;
    const int i0 = item_first(lf_count[a], nt, it - t0), ni = item_first(lf_count[a], nt, it - t0 + 1) - i0;
    cells[slot] = make_int4(lf_start[a] + i0, ni, (int)p_start[a], (int)(p_start[a + 1] - p_start[a]));
    cells_d[slot] = make_int4(lf_start[a] + i0, ni, (int)p_start[a], (int)p_cntd[a]);
    cell_item[slot] = it;
}

// Bounding box of each item's particles at their current offsets (sixteen
// lanes per schedule slot), for the culling of candidates, by slot and by item:
// centre and the item's largest search radius, then the half widths, rounded up by a
// relative 1e-6 of the coordinates so that the FP32 centre and widths still
// contain every particle.
__global__ void __launch_bounds__(256) k_cell_pbox(int64_t n_items, const int4* __restrict__ cells,
                                                   const int* __restrict__ cell_item,
                                                   const float4* __restrict__ xrel, const float* __restrict__ Hs,
                                                   float4* __restrict__ pbox, float4* __restrict__ ibox)
{
    // every lane takes part in the shuffles, a group past the last item with no data
    const int64_t slot = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
    const int sub = threadIdx.x & 15;
    const bool live = slot < n_items;
    const int4 ci = live ? cells[slot] : make_int4(0, 0, 0, 0);
    const float BIG = 3.0e38f;
    float lx = BIG, ly = BIG, lz = BIG, hx = -BIG, hy = -BIG, hz = -BIG, H = 0.0f;
    if (sub < ci.y) {
        const float4 x = xrel[ci.x + sub];
        H = Hs[ci.x + sub];
        lx = hx = x.x;
        ly = hy = x.y;
        lz = hz = x.z;
    }
    for (int o = 8; o >= 1; o >>= 1) {  // within the group of 16
        lx = fminf(lx, __shfl_xor(lx, o, 64));
        ly = fminf(ly, __shfl_xor(ly, o, 64));
        lz = fminf(lz, __shfl_xor(lz, o, 64));
        hx = fmaxf(hx, __shfl_xor(hx, o, 64));
        hy = fmaxf(hy, __shfl_xor(hy, o, 64));
        hz = fmaxf(hz, __shfl_xor(hz, o, 64));
        H = fmaxf(H, __shfl_xor(H, o, 64));
    }
    if (live && sub == 0) {
        const float4 c = make_float4(0.5f * (lx + hx), 0.5f * (ly + hy), 0.5f * (lz + hz), H);
        const float4 h = make_float4(0.5f * (hx - lx) * 1.000001f + 1.0e-6f * fmaxf(fabsf(lx), fabsf(hx)),
                                     0.5f * (hy - ly) * 1.000001f + 1.0e-6f * fmaxf(fabsf(ly), fabsf(hy)),
                                     0.5f * (hz - lz) * 1.000001f + 1.0e-6f * fmaxf(fabsf(lz), fabsf(hz)), 0.0f);
        const int64_t it = cell_item[slot];
        pbox[2 * slot] = c;
        pbox[2 * slot + 1] = h;
        ibox[2 * it] = c;
        ibox[2 * it + 1] = h;
    }
}

// Sorted FP32 offsets from the centre of each particle's leaf, or (xrel null) FP64
// positions.
__global__ void k_sorted_fill(int64_t n, const uint32_t* __restrict__ perm, const double* __restrict__ pos_w,
                              const int* __restrict__ leaf_of, const int* __restrict__ lf_node,
                              const int* __restrict__ nd_coord, const int* __restrict__ nd_level,
                              const int* __restrict__ nd_box, const int* __restrict__ box_G,
                              const double* __restrict__ box_len, double* __restrict__ pos_s,
                              float4* __restrict__ xrel)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint32_t o = perm[p];
    const int id = lf_node[leaf_of[p]];
    const int b = nd_box[id];
    double c[3], w;
    node_box(make_int4(nd_coord[3 * id], nd_coord[3 * id + 1], nd_coord[3 * id + 2], nd_level[id]),
             box_len[b] / box_G[b], c, w);
    const double L = box_len[b];
    double d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // the image of the particle nearest its leaf: itself at a build; after
        // a drift across the box boundary, the one on the leaf's side
        const double x = pos_w[3 * (int64_t)o + a];
        const double img = L * rint((x - c[a]) / L);
        if (!xrel) pos_s[3 * p + a] = x - img;
        d[a] = (x - c[a]) - img;
    }
    if (xrel) xrel[p] = make_float4((float)d[0], (float)d[1], (float)d[2], 0.0f);
}

// Smallest search radius (float bits; non-negative floats order like their bits).
__global__ void __launch_bounds__(BS) k_min_H(int64_t n, const float* __restrict__ Hs, unsigned* __restrict__ out)
{
    __shared__ float wm[BS / 64];
    float m = INFINITY;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x)
        m = fminf(m, Hs[p]);
    for (int o = 32; o >= 1; o >>= 1) m = fminf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {  // one atomic per workgroup
        for (int q = 1; q < BS / 64; ++q) m = fminf(m, wm[q]);
        atomicMin(out, __float_as_uint(m));
    }
}

// The tables of boxes between host and device, by kernels on pinned memory: a
// copy of a few words costs 5 to 10 us each, and a build had eight of them.
struct BoxTables {
    int64_t* first;     // n_boxes + 1
    double* len;        // n_boxes
    int64_t* top_base;  // n_boxes + 1
    int64_t* bad;       // 1
    unsigned* hmax;     // n_boxes
    int* G;             // n_boxes
    int* col_base;      // n_boxes + 1
    uint32_t* level;    // LEVEL_WORDS: a level's nodes and leaves (CT_TOTAL), the grid's items
};
constexpr int LEVEL_WORDS = 3;

// At the start of a build: the boxes (len null: as they are), and zero maxima and
// counters.
__global__ void k_build_begin(int nb, BoxTables h, int64_t* __restrict__ box_first, double* __restrict__ box_len,
                              unsigned* __restrict__ box_hmax, int64_t* __restrict__ ctr)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (box_len) {
        if (k <= nb) box_first[k] = h.first[k];
        if (k < nb) box_len[k] = h.len[k];
    }
    if (k < nb) box_hmax[k] = 0u;
    if (k < CT_COUNT) ctr[k] = 0;
}

__global__ void k_hmax_out(int nb, const unsigned* __restrict__ box_hmax, const int64_t* __restrict__ ctr, BoxTables h)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nb) h.hmax[k] = box_hmax[k];
    if (k == 0) *h.bad = ctr[CT_BAD_INPUT];
}

__global__ void k_box_tables(int nb, BoxTables h, int* __restrict__ box_G, int64_t* __restrict__ top_base,
                             int* __restrict__ col_base)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nb) box_G[k] = h.G[k];
    if (k <= nb) {
        top_base[k] = h.top_base[k];
        col_base[k] = h.col_base[k];
    }
}

// n_items: of a grid layout (null: none made)
__global__ void k_level_out(const uint32_t* __restrict__ d, const uint32_t* __restrict__ n_items, BoxTables h)
{
    if (threadIdx.x < 2) h.level[threadIdx.x] = d[threadIdx.x];
    if (threadIdx.x == 2) h.level[2] = n_items ? *n_items : 0u;
}

// The build's shape counters folded over their spread slots, and the
// smallest search radius, into out (BUILD_OUT_WORDS words of pinned host memory,
// read after the next synchronisation).
__global__ void k_build_out(const int64_t* __restrict__ ctr, const unsigned* __restrict__ hmin,
                            int64_t* __restrict__ out)
{
    const int k = threadIdx.x;  // CT_B_CAND_PAIRS + k
    if (k < 5) {
        int64_t v = ctr[CT_B_CAND_PAIRS + k];
        for (int sl = 0; sl < CT_SPREAD_SLOTS; ++sl) {
            const int64_t x = ctr[CT_SPREAD + sl * CT_SUMS + CT_B_CAND_PAIRS + k];
            v = k < 2 ? v + x : max(v, x);
        }
        out[k] = v;
    } else if (k == 5) {
        out[5] = (int64_t)*hmin;
    }
}

int ceil_log2(uint64_t v)
{
    int b = 0;
    while ((1ull << b) < v) ++b;
    return b;
}

}  // namespace

namespace sph {

// The pinned tables, for the context's number of boxes. Nothing of an earlier build
// still reads what the next one writes here: k_build_begin's part is read before the
// wait for k_hmax_out, k_box_tables' before the wait for the first level's counts
// or, if the build ended early, before the next wait for k_hmax_out.
static BoxTables box_tables(sph_ctx* c)
{
    const size_t nb = (size_t)c->n_boxes;
    if (c->h_boxes_cap < nb) {
        if (c->h_boxes) SPH_HIP(hipHostFree(c->h_boxes));
        c->h_boxes = nullptr;
        c->h_boxes_cap = 0;
        SPH_HIP(hipHostMalloc((void**)&c->h_boxes, (nb + 1) * 36 + LEVEL_WORDS * 4, hipHostMallocDefault));
        c->h_boxes_cap = nb;
    }
    const size_t m = c->h_boxes_cap + 1;
    BoxTables t;
    t.first = reinterpret_cast<int64_t*>(c->h_boxes);
    t.top_base = t.first + m;
    t.len = reinterpret_cast<double*>(t.top_base + m);  // the last word of each: spare, or `bad`
    t.bad = reinterpret_cast<int64_t*>(t.len + m - 1);
    t.hmax = reinterpret_cast<unsigned*>(t.len + m);
    t.G = reinterpret_cast<int*>(t.hmax + m);
    t.col_base = t.G + m;
    t.level = reinterpret_cast<uint32_t*>(t.col_base + m);
    return t;
}

static void build_begin(sph_ctx* c, const BoxTables& bt, int64_t* box_first, double* box_len, unsigned* box_hmax,
                        int64_t* ctr, hipStream_t s)
{
    k_build_begin<<<blocks_for(std::max<int64_t>(c->n_boxes + 1, CT_COUNT), BS), BS, 0, s>>>(
        c->n_boxes, bt, box_first, box_len, box_hmax, ctr);
    SPH_HIP(hipGetLastError());
}

static TreeView tree_view(sph_ctx* c)
{
    return TreeView{static_cast<int4*>(c->nd_pack.p), (int)c->n_nodes};
}

// Offsets of the leaves' partner lists from their counts (p_cnt); sets n_pairs
// (from the counters of the build under way; later builds' read-back has set
// it: known). Synchronises the stream.
static void list_offsets(sph_ctx* c, bool known, hipStream_t s)
{
    const int64_t nl = c->n_leaves;
    uint32_t* p_start = ensure<uint32_t>(c, c->p_start, nl + 1);
    scan_exclusive(c, static_cast<uint32_t*>(c->p_cnt.p), p_start, nl, p_start + nl, s);
    uint32_t np = 0;
    SPH_HIP(hipMemcpyAsync(&np, p_start + nl, 4, hipMemcpyDeviceToHost, s));
    int64_t np64 = c->n_pairs;
    if (known) {
        SPH_HIP(hipStreamSynchronize(s));
    } else {
        const int64_t* hc = read_counters(c, s);  // synchronises: np is in
        np64 = hc[CT_B_PAIRS64];
        SPH_REQUIRE(hc[CT_BAD_INPUT] == 0, SPH_E_HIP,
                    "inconsistent cell tree: a walk took more steps than the tree has nodes");
    }
    SPH_REQUIRE(np64 <= (int64_t)UINT32_MAX && (int64_t)np == np64, SPH_E_ARG,
                std::to_string(np64) + " (cell, neighbour cell) records: more than 2^32 - 1 cannot be indexed");
    c->n_pairs = np;
}

// The partner lists at those offsets (and the items' leaves and schedule keys).
static void fill_lists(sph_ctx* c, const uint32_t* it_start, int64_t n_items, int* it_leaf, uint64_t* sk, uint32_t* sv,
                       int xcd_local, hipStream_t s)
{
    const int64_t nl = c->n_leaves, np = c->n_pairs;
    int* p_leaf = ensure<int>(c, c->p_leaf, np);
    float4* p_shift = ensure<float4>(c, c->p_shift, np);
    uint8_t* p_code = ensure<uint8_t>(c, c->p_code, np);
    int2* p_rec = ensure<int2>(c, c->p_rec, np);
    k_partners<<<(unsigned)blocks_for(nl * 32, PBS), PBS, 0, s>>>(
        nl, 1, static_cast<int*>(c->lf_node.p), tree_view(c), static_cast<int*>(c->nd_box.p),
        static_cast<int*>(c->top.p), static_cast<int64_t*>(c->box_top_base.p), static_cast<int*>(c->box_G.p),
        static_cast<double*>(c->box_len.p), static_cast<uint32_t*>(c->p_cnt.p), static_cast<uint32_t*>(c->p_cntd.p),
        static_cast<uint32_t*>(c->p_start.p),
        RecordOut{p_leaf, p_shift, p_code, p_rec, static_cast<int*>(c->lf_start.p), static_cast<int*>(c->lf_count.p),
                  it_start},
        it_start, n_items, it_leaf, sk, sv, xcd_local, static_cast<int64_t*>(c->counters.p));
    SPH_HIP(hipGetLastError());
    c->lists_built = true;
}

static void sorted_fill(sph_ctx* c, double* pos_s, float4* xrel, hipStream_t s)
{
    const int64_t n = c->n;
    k_sorted_fill<<<blocks_for(n, BS), BS, 0, s>>>(
        n, static_cast<uint32_t*>(c->perm.p), static_cast<double*>(c->pos_w.p), static_cast<int*>(c->leaf_of.p),
        static_cast<int*>(c->lf_node.p), static_cast<int*>(c->nd_coord.p), static_cast<int*>(c->nd_level.p),
        static_cast<int*>(c->nd_box.p), static_cast<int*>(c->box_G.p), static_cast<double*>(c->box_len.p), pos_s, xrel);
    SPH_HIP(hipGetLastError());
}

void partner_lists(sph_ctx* c, hipStream_t s)
{
    if (!c->lists_built) {
        finish_build_read(c);
        list_offsets(c, true, s);
        fill_lists(c, nullptr, 0, nullptr, nullptr, nullptr, 0, s);
    }
    if (!c->pos_built) sorted_fill(c, ensure<double>(c, c->pos_s, 3 * c->n), nullptr, s);
    c->pos_built = true;
}

// Everything after the positions are wrapped: keys, sort, tree, leaves, lists.
// allow_grid: take the grid layout where it serves.
static void build_layout(sph_ctx* c, bool allow_grid, hipStream_t s)
{
    const int64_t n = c->n;
    const int nb = c->n_boxes;
    const float margin = (float)c->prm.h_margin;
    int64_t* ctr = static_cast<int64_t*>(c->counters.p);

    // ---- largest search radius per box (k_wrap / k_box_hmax ran) -> top grid --------
    unsigned* box_hmax = static_cast<unsigned*>(c->box_hmax.p);
    const BoxTables bt = box_tables(c);
    k_hmax_out<<<blocks_for(nb, BS), BS, 0, s>>>(nb, box_hmax, ctr, bt);
    SPH_HIP(hipGetLastError());
    SPH_HIP(hipStreamSynchronize(s));
    SPH_REQUIRE(*bt.bad == 0, SPH_E_ARG, "non-finite position or non-positive/non-finite h_guess");
    c->h_box_G.assign(nb, 0);
    c->h_box_top_base.assign(nb + 1, 0);
    uint64_t maxG3 = 1;
    for (int b = 0; b < nb; ++b) {
        const int64_t cnt = c->h_box_first[b + 1] - c->h_box_first[b];
        float H;
        std::memcpy(&H, &bt.hmax[b], 4);
        const double L = c->h_box_len[b];
        int G = 3;
        if (cnt > 0) {
            SPH_REQUIRE(3.0 * (double)H <= L, SPH_E_H_TOO_LARGE,
                        "box " + std::to_string(b) + ": search radius " + std::to_string(H) +
                            " exceeds a third of the box side " + std::to_string(L));
            G = (int)std::floor(L / (double)H);
            // a top cell exactly one radius wide must still hold the radius after rounding
            while (G > 3 && L / G < (double)H) --G;
            G = std::max(3, std::min(G, 256));
        }
        c->h_box_G[b] = G;
        c->h_box_top_base[b + 1] = c->h_box_top_base[b] + (int64_t)G * G * G;
        maxG3 = std::max<uint64_t>(maxG3, (uint64_t)G * G * G);
    }
    c->n_top = c->h_box_top_base[nb];
    // from here on the last cells are taken apart: none to compute on until these are whole
    c->built = false;
    // columns of top cells of each box, for a grid layout, which needs at least
    // four cells per side (the frame of an item reaches a cell and a half from
    // its centre, and with three the cells on both sides are the same ones) and a
    // table of fine cells in proportion to the particles. Where a top cell splits
    // the radii differ so much that the columns would hold many candidates for
    // nothing: with the top cells kept whole a pass over 32768 clustered particles
    // takes 607 us, split (the tree) 558; a log-normal set of 64000 268 and 190
    bool grid_ok = allow_grid;
    bt.col_base[0] = 0;
    bt.top_base[0] = 0;
    for (int b = 0; b < nb; ++b) {
        bt.col_base[b + 1] = bt.col_base[b] + c->h_box_G[b] * c->h_box_G[b];
        bt.top_base[b + 1] = c->h_box_top_base[b + 1];
        bt.G[b] = c->h_box_G[b];
        if (c->h_box_first[b + 1] > c->h_box_first[b] && c->h_box_G[b] < 4) grid_ok = false;
    }
    c->bits_box = nb > 1 ? ceil_log2((uint64_t)nb) : 0;
    c->bits_top = std::max(1, ceil_log2(maxG3));
    c->levels = std::min(MAX_LEVELS, (63 - c->bits_box - c->bits_top) / 3);
    SPH_REQUIRE(c->levels >= 1, SPH_E_ARG, "too many boxes or top cells for the key layout");
    int* box_G = ensure<int>(c, c->box_G, nb);
    int64_t* box_top_base = ensure<int64_t>(c, c->box_top_base, nb + 1);
    int* col_base = ensure<int>(c, c->col_base, nb + 1);
    k_box_tables<<<blocks_for(nb + 1, BS), BS, 0, s>>>(nb, bt, box_G, box_top_base, col_base);
    SPH_HIP(hipGetLastError());

    // ---- keys and sort -------------------------------------------------------------------
    // Sorted by box, top cell and fine cell in z first (as many fine cells, up to
    // eight, as the last 8-bit pass of the sort has bits for, or four): all a
    // grid layout needs. Where a top cell splits, the particles are sorted again
    // by the whole Morton key after level 0, below.
    {
        const int base = c->bits_box + c->bits_top;
        c->fzb = base % 8 == 0 ? 2 : std::min(3, 8 - base % 8);
    }
    const int64_t n_fine = c->n_top << c->fzb;
    grid_ok = grid_ok && n_fine <= 16 * n + 4096 && n_fine < (int64_t)1 << 30;
    const int n_cols = bt.col_base[nb];
    KeyLayout kl{c->bits_top, c->levels, c->fzb};
    uint64_t* keys = ensure<uint64_t>(c, c->keys, n);
    uint64_t* keys_alt = ensure<uint64_t>(c, c->keys_alt, n);
    uint32_t* perm = ensure<uint32_t>(c, c->perm, n);
    uint32_t* perm_alt = ensure<uint32_t>(c, c->perm_alt, n);
    const int64_t* box_first = static_cast<int64_t*>(c->box_first.p);
    const double* box_len = static_cast<double*>(c->box_len.p);
    k_keys<<<blocks_for(n, BS), BS, 0, s>>>(n, static_cast<double*>(c->pos_w.p), box_first, nb, box_len,
                                            box_G, kl, c->fzb, keys, perm);
    SPH_HIP(hipGetLastError());
    radix_sort(c, keys, perm, keys_alt, perm_alt, n, c->bits_box + c->bits_top + c->fzb, s);

    // ---- the number of items of a grid layout (made if no top cell splits) -----------------------
    int* starts = nullptr;
    uint32_t* col_start = nullptr;
    if (grid_ok) {
        starts = ensure<int>(c, c->starts, (size_t)n_fine + 1);
        col_start = ensure<uint32_t>(c, c->it_start, (size_t)n_cols + 1);
        k_fine_starts<<<blocks_for(n, BS), BS, 0, s>>>(n, keys, kl, box_top_base, n_fine, starts);
        SPH_HIP(hipGetLastError());
        k_col_count<<<blocks_for((int64_t)n_cols * 64, 256), 256, 0, s>>>(n_cols, nb, col_base, box_G, box_top_base, kl,
                                                                          starts, keys, col_start);
        SPH_HIP(hipGetLastError());
        scan_exclusive(c, col_start, col_start, n_cols, col_start + n_cols, s);
    }

    float* Hs = ensure<float>(c, c->Hs, n);
    int* leaf_tmp = ensure<int>(c, c->lf_tmp, n);
    unsigned* drift = ensure<unsigned>(c, c->drift, 4);
    k_sorted_H<<<blocks_for(n, BS), BS, 0, s>>>(n, perm, static_cast<float*>(c->hguess.p), margin, Hs,
                                                leaf_tmp, drift);
    SPH_HIP(hipGetLastError());

    // ---- tree, level by level ---------------------------------------------------------------
    // One read-back per level: its node count M and leaf count K (the two
    // halves of one counter word). The level's kernels run over a bound the
    // host already has: the top cells at level 0, eight children per split
    // node of the level above after that.
    uint32_t* head = ensure<uint32_t>(c, c->head, n + 1);
    uint32_t* excl = ensure<uint32_t>(c, c->scan1, n + 1);
    int* nid = ensure<int>(c, c->nid, n);
    uint32_t* d_M = reinterpret_cast<uint32_t*>(&ctr[CT_TOTAL]);
    uint32_t* d_K = d_M + 1;
    int* top = ensure<int>(c, c->top, (size_t)c->n_top);

    int64_t node_base = 0, leaf_base = 0, prev_base = 0, prev_M = 0;
    int64_t bound = std::min<int64_t>(n, c->n_top);
    // level-order leaf id -> node; parked in lf_start's buffer until the leaves
    // are renumbered in Morton order
    int* lo2node = ensure<int>(c, c->lf_start, n + 1);
    for (int level = 0; level <= c->levels && bound > 0; ++level) {
        const int shift = level == 0 ? kl.low : 3 * (c->levels - level);
        k_lvl_head<<<blocks_for(n, BS), BS, 0, s>>>(n, keys, leaf_tmp, shift, head);
        SPH_HIP(hipGetLastError());
        scan_exclusive(c, head, excl, n, d_M, s);
        const int64_t need = node_base + bound;
        // node ids are int and index 3 ints of nd_coord each
        SPH_REQUIRE(need <= (int64_t)(INT32_MAX / 3), SPH_E_ARG,
                    "the cell tree needs more than " + std::to_string(INT32_MAX / 3) + " nodes");
        if (need > c->node_cap) {
            const int64_t cap = std::max<int64_t>(need + need / 2, 1024);
            grow_keep<int>(c, c->nd_start, cap, node_base, s);
            grow_keep<int>(c, c->nd_count, cap, node_base, s);
            grow_keep<unsigned>(c, c->nd_hmax, cap, node_base, s);
            grow_keep<int>(c, c->nd_wide, cap, node_base, s);
            grow_keep<int>(c, c->nd_child0, cap, node_base, s);
            grow_keep<int>(c, c->nd_child1, cap, node_base, s);
            grow_keep<int>(c, c->nd_leaf, cap, node_base, s);
            grow_keep<int>(c, c->nd_box, cap, node_base, s);
            grow_keep<int>(c, c->nd_level, cap, node_base, s);
            grow_keep<int>(c, c->nd_coord, 3 * cap, 3 * node_base, s);
            c->node_cap = cap;
        }
        int* nd_start = static_cast<int*>(c->nd_start.p);
        int* nd_count = static_cast<int*>(c->nd_count.p);
        unsigned* nd_hmax = static_cast<unsigned*>(c->nd_hmax.p);
        int* nd_wide = static_cast<int*>(c->nd_wide.p);
        int* nd_child0 = static_cast<int*>(c->nd_child0.p);
        int* nd_child1 = static_cast<int*>(c->nd_child1.p);
        int* nd_leaf = static_cast<int*>(c->nd_leaf.p);
        int* nd_box = static_cast<int*>(c->nd_box.p);
        int* nd_level = static_cast<int*>(c->nd_level.p);
        int* nd_coord = static_cast<int*>(c->nd_coord.p);
        const unsigned gb = (unsigned)blocks_for(bound, BS);
        const int64_t n_clear = level == 0 ? c->n_top : 0;
        k_lvl_clear<<<(unsigned)blocks_for(std::max(bound, n_clear), BS), BS, 0, s>>>(node_base, bound, nd_count, nd_hmax,
                                                                                      nd_wide, n_clear, top);
        SPH_HIP(hipGetLastError());
        k_lvl_nodes<<<blocks_for(n, BS), BS, 0, s>>>(n, keys, leaf_tmp, head, excl, Hs, level, kl, node_base,
                                                     nid, nd_start, nd_count, nd_hmax, nd_wide, nd_box, nd_level,
                                                     nd_coord, box_G, box_len, (float)c->prm.cell_ratio);
        SPH_HIP(hipGetLastError());
        if (level == 0) {
            k_top_table<<<gb, BS, 0, s>>>(bound, d_M, nd_box, nd_coord, box_G, box_top_base, top);
            SPH_HIP(hipGetLastError());
        } else {
            k_lvl_children<<<blocks_for(prev_M, BS), BS, 0, s>>>(prev_M, prev_base, nd_leaf, nd_start,
                                                                 nd_count, nid, nd_child0, nd_child1);
            SPH_HIP(hipGetLastError());
        }
        uint32_t* nflag = ensure<uint32_t>(c, c->nflag, bound + 1);
        uint32_t* nscan = ensure<uint32_t>(c, c->nscan, bound + 1);
        k_lvl_decide<<<gb, BS, 0, s>>>(bound, d_M, node_base, level, c->levels, c->prm.leaf_target, nd_count,
                                       nd_wide, nflag, nd_child0, nd_child1);
        SPH_HIP(hipGetLastError());
        scan_exclusive(c, nflag, nscan, bound, d_K, s);
        k_lvl_leaves<<<gb, BS, 0, s>>>(bound, d_M, node_base, leaf_base, nflag, nscan, nd_leaf, lo2node);
        SPH_HIP(hipGetLastError());
        k_lvl_assign<<<blocks_for(n, BS), BS, 0, s>>>(n, nid, nd_leaf, leaf_tmp);
        SPH_HIP(hipGetLastError());
        k_level_out<<<1, 64, 0, s>>>(d_M, level == 0 && grid_ok ? col_start + n_cols : nullptr, bt);
        SPH_HIP(hipGetLastError());
        SPH_HIP(hipStreamSynchronize(s));
        const int64_t M = bt.level[0], K = bt.level[1];
        if (level == 0) {
            c->uni = grid_ok && K == M;
            if (c->uni) {
                c->n_items = bt.level[2];
                int* box_item = ensure<int>(c, c->box_item, nb + 1);
                int4* cells = ensure<int4>(c, c->cells, 2 * (size_t)c->n_items);
                k_col_items<<<blocks_for((int64_t)n_cols * 64, 256), 256, 0, s>>>(n_cols, nb, col_base, box_G, box_len,
                                                                                  box_top_base, kl, starts, keys,
                                                                                  col_start, cells, box_item);
                SPH_HIP(hipGetLastError());
            }
        }
        // every particle not yet in a leaf heads or joins a node of this level,
        // so the bound (its parents' children) holds them; a larger count is a bug
        SPH_REQUIRE(M <= bound && K <= M, SPH_E_HIP, "cell tree level outside its bound");
        if (level == 0 && K < M) {
            // A top cell splits: order the particles by the whole key. Every top
            // cell keeps its range, so the level-0 nodes, their sums and each
            // particle's node and leaf stay as they are; only the keys and the
            // sorted search radii follow the new order.
            kl.low = 3 * c->levels;
            k_keys<<<blocks_for(n, BS), BS, 0, s>>>(n, static_cast<double*>(c->pos_w.p), box_first, nb, box_len,
                                                    box_G, kl, -1, keys, perm);
            SPH_HIP(hipGetLastError());
            radix_sort(c, keys, perm, keys_alt, perm_alt, n, c->bits_box + c->bits_top + 3 * c->levels, s);
            k_sorted_H<<<blocks_for(n, BS), BS, 0, s>>>(n, perm, static_cast<float*>(c->hguess.p), margin, Hs,
                                                        nullptr, drift);
            SPH_HIP(hipGetLastError());
        }
        prev_base = node_base;
        prev_M = M;
        node_base += M;
        leaf_base += K;
        bound = std::min<int64_t>(8 * (M - K), n);  // children of this level's split nodes
    }
    c->n_nodes = node_base;

    // ---- leaves in Morton (particle) order ---------------------------------------------------
    const int64_t nl = leaf_base;  // the leaves of all levels, one per run of leaf_tmp
    c->n_leaves = nl;
    int* leaf_of = ensure<int>(c, c->leaf_of, n);
    int* lf_node = ensure<int>(c, c->lf_node, nl);
    int* lf_count = ensure<int>(c, c->lf_count, nl);
    float* lf_hmax = ensure<float>(c, c->lf_hmax, nl);
    int4* nodes = ensure<int4>(c, c->nd_pack, 2 * c->n_nodes);
    int* lf_start = static_cast<int*>(c->lf_start.p);  // (lo2node's buffer: n + 1)
    if (c->n_nodes == nl) {
        k_leaf_top<<<blocks_for(n, BS), BS, 0, s>>>(
            n, nl, nid, static_cast<int*>(c->nd_start.p), static_cast<int*>(c->nd_count.p),
            static_cast<unsigned*>(c->nd_hmax.p), static_cast<int*>(c->nd_coord.p), leaf_of, lf_start, lf_node, lf_count,
            lf_hmax, nodes);
        SPH_HIP(hipGetLastError());
    } else {
        k_leaf_head<<<blocks_for(n, BS), BS, 0, s>>>(n, leaf_tmp, head);
        SPH_HIP(hipGetLastError());
        scan_exclusive(c, head, excl, n, nullptr, s);
        // lo2node lives in lf_start's buffer; move it aside before lf_start is written
        int* lo2 = ensure<int>(c, c->nid, std::max<int64_t>(n, nl));
        SPH_HIP(hipMemcpyAsync(lo2, lo2node, (size_t)nl * 4, hipMemcpyDeviceToDevice, s));
        k_leaf_fill<<<blocks_for(n, BS), BS, 0, s>>>(n, head, excl, leaf_tmp, lo2, leaf_of, lf_start, lf_node);
        SPH_HIP(hipGetLastError());
        k_leaf_fix<<<blocks_for(nl, BS), BS, 0, s>>>(nl, lf_node, static_cast<int*>(c->nd_count.p),
                                                     static_cast<unsigned*>(c->nd_hmax.p),
                                                     static_cast<int*>(c->nd_leaf.p), lf_count, lf_hmax);
        SPH_HIP(hipGetLastError());
        k_tree_pack<<<blocks_for(c->n_nodes, BS), BS, 0, s>>>(
            c->n_nodes, static_cast<int*>(c->nd_coord.p), static_cast<int*>(c->nd_level.p),
            static_cast<unsigned*>(c->nd_hmax.p), static_cast<int*>(c->nd_leaf.p), static_cast<int*>(c->nd_child0.p),
            static_cast<int*>(c->nd_child1.p), lf_count, nodes);
        SPH_HIP(hipGetLastError());
    }

    // ---- partner lists: their number, and in a tree layout the lists and the items ------------
    uint32_t* p_cnt = ensure<uint32_t>(c, c->p_cnt, nl + 1);
    uint32_t* p_cntd = ensure<uint32_t>(c, c->p_cntd, nl + 1);
    const TreeView tv = tree_view(c);
    k_partners<<<(unsigned)blocks_for(nl * 32, PBS), PBS, 0, s>>>(
        nl, 0, lf_node, tv, static_cast<int*>(c->nd_box.p), top, box_top_base, box_G, box_len, p_cnt, p_cntd, nullptr,
        RecordOut{nullptr, nullptr, nullptr, nullptr, lf_start, lf_count, nullptr}, nullptr, 0, nullptr, nullptr, nullptr, 0,
        ctr);
    SPH_HIP(hipGetLastError());
    c->lists_built = false;
    if (!c->uni) {
        uint32_t* it_start = ensure<uint32_t>(c, c->it_start, nl + 1);
        k_item_count<<<blocks_for(nl, BS), BS, 0, s>>>(nl, lf_count, it_start);
        SPH_HIP(hipGetLastError());
        scan_exclusive(c, it_start, it_start, nl, it_start + nl, s);
        uint32_t nit = 0;
        SPH_HIP(hipMemcpyAsync(&nit, it_start + nl, 4, hipMemcpyDeviceToHost, s));
        list_offsets(c, false, s);  // synchronises: nit is in
        const int64_t ni = nit;
        c->n_items = ni;
        int* box_item = ensure<int>(c, c->box_item, nb + 1);
        k_box_item<<<blocks_for(nb + 1, BS), BS, 0, s>>>(nb, n, nl, box_first, leaf_of, it_start, box_item);
        SPH_HIP(hipGetLastError());
        // the schedule: items by decreasing cost dealt out to the XCDs, Morton ranges, or Morton
        // ranges each ordered by decreasing cost
        const int order = c->prm.cell_order;
        const bool by_cost = order != 1;
        // (in what the particles' keys and scans leave free: no more items than particles)
        int* it_leaf = reinterpret_cast<int*>(excl);
        uint64_t* sk = by_cost ? keys : nullptr;
        uint32_t* sv = by_cost ? perm_alt : nullptr;
        fill_lists(c, it_start, ni, it_leaf, sk, sv, order == 2 ? 1 : 0, s);
        if (by_cost) radix_sort(c, sk, sv, keys_alt, head, ni, order == 2 ? 15 : 12, s);
        int4* cells = ensure<int4>(c, c->cells, ni);
        int* cell_item = ensure<int>(c, c->cell_item, ni);
        int4* cells_d = ensure<int4>(c, c->cells_d, ni);
        k_sched_fill<<<blocks_for(ni, BS), BS, 0, s>>>(ni, sv, order == 0 ? 1 : 0, it_leaf, it_start, lf_start,
                                                       lf_count, static_cast<uint32_t*>(c->p_start.p), p_cntd, cells,
                                                       cell_item, cells_d);
        SPH_HIP(hipGetLastError());
    }

    // ---- sorted particle streams ------------------------------------------------------------------
    refresh_offsets(c, s);
    // the smallest search radius bounds how far the particles may drift before
    // the cells are rebuilt
    k_min_H<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>(blocks_for(n, BS), 256)), BS, 0, s>>>(n, Hs,
                                                                                                 drift + 2);
    SPH_HIP(hipGetLastError());
    // the shape counters and the smallest radius come back behind an event;
    // the next synchronisation (or finish_build_read) picks them up
    k_build_out<<<1, 64, 0, s>>>(ctr, drift + 2, c->h_build);
    SPH_HIP(hipGetLastError());
    SPH_HIP(hipEventRecord(c->ev_build, s));
    c->build_read_pending = true;
    c->binfo.n_cells = nl;
    c->built = true;
    ++c->tm.builds;
    c->drift_pending = false;
    c->vsig_valid = false;  // signal velocities belong to the cells of the last force pass
    c->bal_valid = false;
    c->div_valid = false;   // and the divergences to its particle order
    ++c->layout_serial;  // cell arrays and grid sizes changed
    c->density_done = false;
    c->density64_done = false;
}

// The build. Where memory runs out with a grid's tables (held for this build or
// kept from an earlier one) those are given back and the cells made as a tree, so that
// what the tree alone has room for is accepted.
static void build_from_wrapped(sph_ctx* c, hipStream_t s)
{
    try {
        build_layout(c, true, s);
    } catch (const Error& e) {
        if (e.code != SPH_E_NOMEM || !c->starts.p) throw;
        SPH_HIP(hipDeviceSynchronize());
        for (Buf* b : {&c->starts, &c->xfix, &c->it_start, &c->cells, &c->cell_pbox}) free_buf(c, *b);
        fill_u32(c->counters.p, 0u, 2 * (int64_t)CT_COUNT, s);
        build_layout(c, false, s);
    }
}

void finish_build_read(sph_ctx* c)
{
    if (!c->build_read_pending) return;
    SPH_HIP(hipEventSynchronize(c->ev_build));
    c->build_read_pending = false;
    const int64_t* hb = c->h_build;
    c->binfo.candidate_pairs = hb[0];
    c->binfo.n_pairs = c->n_pairs = hb[1];
    c->binfo.max_cell_particles = hb[2];
    c->binfo.max_neighbour_cells = hb[3];
    c->binfo.max_candidates = hb[4];
    const uint32_t bits = (uint32_t)hb[5];
    std::memcpy(&c->h_min, &bits, 4);
}

void build_cells(sph_ctx* c, int32_t n_boxes, const int64_t* box_first, const double* box_len, int64_t n,
                 const double* pos, const float* h_guess, hipStream_t s)
{
    c->built = false;
    c->density_done = false;
    c->density64_done = false;
    c->n = n;
    c->n_boxes = n_boxes;
    c->h_box_first.assign(box_first, box_first + n_boxes + 1);
    c->h_box_len.assign(box_len, box_len + n_boxes);
    int64_t* bf = ensure<int64_t>(c, c->box_first, n_boxes + 1);
    double* bl = ensure<double>(c, c->box_len, n_boxes);
    ensure<int64_t>(c, c->counters, CT_COUNT);
    double* pw = ensure<double>(c, c->pos_w, 3 * n);
    float* hg = ensure<float>(c, c->hguess, n);
    unsigned* box_hmax = ensure<unsigned>(c, c->box_hmax, n_boxes);
    int64_t* ctr = static_cast<int64_t*>(c->counters.p);
    const BoxTables bt = box_tables(c);
    std::copy(box_first, box_first + n_boxes + 1, bt.first);
    std::copy(box_len, box_len + n_boxes, bt.len);
    build_begin(c, bt, bf, bl, box_hmax, ctr, s);
    k_wrap<<<blocks_for(n, WBS), WBS, 0, s>>>(n, pos, bf, n_boxes, bl, h_guess, pw, hg, box_hmax,
                                            (float)c->prm.h_margin, ctr);
    SPH_HIP(hipGetLastError());
    c->rebuilds = 0;
    build_from_wrapped(c, s);
}

// The sorted positions (32-bit fractions, or offsets from the leaf centres) and
// the items' boxes from the current positions, keeping the cells: at a build and
// after a drift.
void refresh_offsets(sph_ctx* c, hipStream_t s)
{
    c->pos_built = false;
    if (c->uni) {
        int4* xfix = ensure<int4>(c, c->xfix, c->n);
        k_fix_fill<<<blocks_for(c->n, BS), BS, 0, s>>>(c->n, static_cast<uint32_t*>(c->perm.p),
                                                      static_cast<double*>(c->pos_w.p),
                                                      static_cast<int64_t*>(c->box_first.p), c->n_boxes,
                                                      static_cast<double*>(c->box_len.p),
                                                      static_cast<int*>(c->box_G.p), xfix);
        SPH_HIP(hipGetLastError());
    } else {
        sorted_fill(c, nullptr, ensure<float4>(c, c->xrel, c->n), s);
    }
    cell_boxes(c, s);
}

// The particle boxes of every work item from the current offsets.
void cell_boxes(sph_ctx* c, hipStream_t s)
{
    const int64_t ni = c->n_items;
    float4* pbox = ensure<float4>(c, c->cell_pbox, 2 * ni);
    if (ni == 0) return;
    if (c->uni)
        k_fix_pbox<<<blocks_for(16 * ni, 256), 256, 0, s>>>(ni, static_cast<int4*>(c->cells.p), c->fzb,
                                                           static_cast<int4*>(c->xfix.p),
                                                           static_cast<float*>(c->Hs.p), pbox);
    else
        k_cell_pbox<<<blocks_for(16 * ni, 256), 256, 0, s>>>(
            ni, static_cast<int4*>(c->cells.p), static_cast<int*>(c->cell_item.p), static_cast<float4*>(c->xrel.p),
            static_cast<float*>(c->Hs.p), pbox, ensure<float4>(c, c->item_box, 2 * ni));
    SPH_HIP(hipGetLastError());
}

// Rebuild around new smoothing lengths (caller order) keeping the positions.
void rebuild_cells(sph_ctx* c, const float* h_caller, hipStream_t s)
{
    float* hg = static_cast<float*>(c->hguess.p);
    unsigned* box_hmax = static_cast<unsigned*>(c->box_hmax.p);
    int64_t* ctr = static_cast<int64_t*>(c->counters.p);
    if (h_caller && h_caller != hg)  // null: the guesses of the last build
        SPH_HIP(hipMemcpyAsync(hg, h_caller, (size_t)c->n * 4, hipMemcpyDeviceToDevice, s));
    build_begin(c, box_tables(c), nullptr, nullptr, box_hmax, ctr, s);
    k_box_hmax<<<blocks_for(c->n, WBS), WBS, 0, s>>>(c->n, static_cast<int64_t*>(c->box_first.p), c->n_boxes, hg,
                                                   box_hmax, (float)c->prm.h_margin, ctr);
    SPH_HIP(hipGetLastError());
    build_from_wrapped(c, s);
}

}  // namespace sph
