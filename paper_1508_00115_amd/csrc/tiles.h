// Wavefront-level helpers shared by the hot kernels: the per-XCD work queues,
// the work items with their frames and candidates, and the matrix-core filter of
// the pairs.
#pragma once

#include "common.h"
#include "item_range.h"

// Work sources of the hot kernels. Items are schedule slots: either work items
// ranked by decreasing cost (particles x candidates) and dealt out to the 8
// XCDs (xcd_start), so the longest start first and every XCD gets an equal
// share of each cost class, or items in Morton order (a grid layout: in the
// order of its columns, always), so each XCD runs a contiguous range of
// neighbouring items whose particles its L2 keeps.
//   hardware dispatch: one item per wavefront; consecutive workgroups are
//     placed round-robin on the 8 XCDs and workgroup b is remapped to the next
//     slot of its XCD's run, which is rank b;
//   persistent: a grid sized to the machine pops batches of items from eight
//     per-XCD queues (one atomic per batch) and steals from the other queues
//     when its own is empty.
// Queue q covers items [xcd_start(n_items, q), xcd_start(n_items, q + 1)).
struct WorkSched {
    int persistent;   // 0: hardware dispatch, 1: per-XCD queues
    int batch;        // items per pop (persistent)
    int n_items;
};

// The kernel's argument block (its only argument, a T), through a pointer the
// compiler cannot see through: fields read from it are loaded where they are
// used. Arguments by value all live in scalar registers from the start; the hot
// loops' wave-uniform values then spill over into vector registers.
template <class T>
using KernArgs = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ KernArgs<T> late_args()
{
    KernArgs<T> p = (KernArgs<T>)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// Workgroup index with the XCD round-robin undone: blocks that land on the
// same XCD get consecutive indices.
__device__ __forceinline__ int xcd_block_index()
{
    const int nb = gridDim.x;
    const int q = nb / 8, r = nb % 8;
    const int x = blockIdx.x % 8, l = blockIdx.x / 8;
    return x * q + min(x, r) + l;
}

// Next item range [a, a_end) of this wavefront; false when the work is done.
__device__ __forceinline__ bool next_items(const WorkSched& W, int64_t* ctr, int waves_per_block, int& state,
                                           int& a, int& a_end)
{
    if (!W.persistent) {
        if (state) return false;
        state = 1;
        a = xcd_block_index() * waves_per_block + (int)(threadIdx.x >> 6);
        a_end = min(a + 1, W.n_items);
        return a < a_end;
    }
    int lo = -1, hi = -1;
    if ((threadIdx.x & 63) == 0) {
        const int xcd = blockIdx.x & 7;
        while (state < 8) {
            const int q = (xcd + state) & 7;
            const int begin = (int)sph::xcd_start(W.n_items, q);
            const int size = (int)sph::xcd_start(W.n_items, q + 1) - begin;
            const int64_t k = atomicAdd((unsigned long long*)&ctr[CT_QUEUE + 8 * q], (unsigned long long)W.batch);
            if (k < size) {
                lo = begin + (int)k;
                hi = begin + (int)min<int64_t>(k + W.batch, size);
                break;
            }
            ++state;
        }
    }
    a = __shfl(lo, 0, 64);
    a_end = __shfl(hi, 0, 64);
    state = __shfl(state, 0, 64);
    return a >= 0;
}

__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A 32-bit value of another lane of the same row of 16, by a DPP pattern:
// 0xB1 = quad_perm [1,0,3,2], 0x4E = quad_perm [2,3,0,1], 0x141 =
// row_half_mirror (lane i of 8 reads 7 - i), 0x140 = row_mirror (lane i of
// 16 reads 15 - i). Every lane of the row must be active.
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v)
{
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}

// Sum over aligned groups of lpi lanes (1, 2, 4, 8 or 16), returned to every
// lane of the group; the whole wavefront must be active. The two quad
// patterns add the partners at distance 1 and 2; once each quad holds its
// sum, the half-row mirror brings in the other quad of the 8 and the row
// mirror the other half of the 16. The partners of a group add the same two
// values at every step, so every lane ends with the same bits (the same sums
// as exchanges at distance 1, 2, 4 and 8). One VALU operation per step.
__device__ __forceinline__ float group_sum(float v, int lpi)
{
    if (lpi >= 2) v += dpp_f<0xB1>(v);
    if (lpi >= 4) v += dpp_f<0x4E>(v);
    if (lpi >= 8) v += dpp_f<0x141>(v);
    if (lpi >= 16) v += dpp_f<0x140>(v);
    return v;
}
// Largest value over aligned groups of lpi lanes, with the same patterns.
__device__ __forceinline__ float group_max(float v, int lpi)
{
    if (lpi >= 2) v = fmaxf(v, dpp_f<0xB1>(v));
    if (lpi >= 4) v = fmaxf(v, dpp_f<0x4E>(v));
    if (lpi >= 8) v = fmaxf(v, dpp_f<0x141>(v));
    if (lpi >= 16) v = fmaxf(v, dpp_f<0x140>(v));
    return v;
}
__device__ __forceinline__ int group_sum_i(int v, int lpi)
{
    if (lpi >= 2) v += dpp_i<0xB1>(v);
    if (lpi >= 4) v += dpp_i<0x4E>(v);
    if (lpi >= 8) v += dpp_i<0x141>(v);
    if (lpi >= 16) v += dpp_i<0x140>(v);
    return v;
}

// Number of lanes for which c holds (a scalar bit count of the ballot).
__device__ __forceinline__ int wave_count(bool c)
{
    return __popcll(__ballot(c));
}

// Lanes of the wavefront below this one whose bit is set in mask.
__device__ __forceinline__ int lanes_below(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Culling of staged candidates. A candidate farther from a box than every
// search radius of the particles inside it (and, for the force, than its own
// h) pairs with none of them: the 3x3x3 block of cells is a cube, the region
// within reach of a cell a rounded box about a quarter smaller, and that of an
// item's particles smaller still. An axis-aligned box in the item's frame.
struct CullBox {
    float cx, cy, cz, hx, hy, hz;
};

// A value every active lane holds alike, moved to a scalar register: it then
// costs no vector register while it stays live across a loop.
__device__ __forceinline__ float uniform_f(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ float wave_min(float v)
{
    for (int o = 32; o >= 1; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}

// Largest v over the wavefront (every lane active).
__device__ __forceinline__ float wave_max(float v)
{
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Bounding box of the positions of the lanes with `in` set (every lane must
// take part). The half widths are rounded up by a relative 1e-6 of the
// coordinates, so that the FP32 centre and widths still contain every
// position; the cull's reach has its own margin.
__device__ __forceinline__ CullBox pass_box(float x, float y, float z, bool in)
{
    const float BIG = 3.0e38f;
    const float lx = wave_min(in ? x : BIG), hx = wave_max(in ? x : -BIG);
    const float ly = wave_min(in ? y : BIG), hy = wave_max(in ? y : -BIG);
    const float lz = wave_min(in ? z : BIG), hz = wave_max(in ? z : -BIG);
    CullBox b;
    b.cx = uniform_f(0.5f * (lx + hx));
    b.cy = uniform_f(0.5f * (ly + hy));
    b.cz = uniform_f(0.5f * (lz + hz));
    b.hx = uniform_f(0.5f * (hx - lx) * 1.000001f + 1.0e-6f * fmaxf(fabsf(lx), fabsf(hx)));
    b.hy = uniform_f(0.5f * (hy - ly) * 1.000001f + 1.0e-6f * fmaxf(fabsf(ly), fabsf(hy)));
    b.hz = uniform_f(0.5f * (hz - lz) * 1.000001f + 1.0e-6f * fmaxf(fabsf(lz), fabsf(hz)));
    return b;
}

__device__ __forceinline__ float box_dist2(float x, float y, float z, const CullBox& b)
{
    const float gx = fmaxf(fabsf(x - b.cx) - b.hx, 0.0f), gy = fmaxf(fabsf(y - b.cy) - b.hy, 0.0f),
                gz = fmaxf(fabsf(z - b.cz) - b.hz, 0.0f);
    return fmaf(gx, gx, fmaf(gy, gy, gz * gz));
}

// Margin of the box test: FP32 positions in the item's frame carry relative
// errors near 1e-7, so the radii grow by 1e-5 (a candidate near the reach is
// kept, never dropped).
__device__ __forceinline__ float cull_reach2(float reach) { return (reach * 1.00001f) * (reach * 1.00001f); }

// ---- the matrix-core pair filter of the density and force loops ------------------------
//
// A work item has at most 16 particles, and its candidates wait in an LDS
// tile. Which candidate lies within which particle's radius is a table of
// |x_i|^2 + |x_j|^2 - 2 x_i . x_j, a product of inner size four: the 16 blocks
// of one v_mfma_f32_4x4x4_16b_f16 hold it for 16 particles x 16 candidates
// (8 cycles for 256 pairs, where the difference form takes 6 vector
// operations per pair and lane, 64 cycles). With C = |x_i|^2 - R_i^2 the sign
// bit of a result is the test, and one v_alignbit per pair gathers the signs of
// a lane's candidates into a word.
//
// Half precision only proposes pairs: the loops recompute every proposed pair
// from the FP32 differences. Coordinates are taken from the centre of the
// item's box and scaled so that its half width and reach together make
// FILTER_SCALE. Rounded toward zero they are off by at most u = 2^-10 of
// themselves, so 2 x_i . x_j is off by at most (2 u + u^2) (|x_i|^2 + |x_j|^2);
// the squares are lowered by FILTER_EPS (a little more than that), the radii
// raised by it and by FILTER_ABS (inputs below the normal range of half
// precision), so no pair inside its radius is missed. On a cell one search
// radius wide about 1.5% of the proposed pairs are outside.
//
// Lane l is column l % 16 (a particle); of each 16 candidates its results are
// rows 4 (l / 16) ... + 3 of the table, which the inputs make candidates 4 r +
// l / 16, r = 0 ... 3: lane group g meets candidates g, g + 4, g + 8, ... of
// the tile, in order, so neighbours in the candidate list go to different
// groups (even word counts). Lane l feeds candidate 4 (l % 4) + l / 16.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef __fp16 f16x2_ __attribute__((ext_vector_type(2)));

constexpr float FILTER_SCALE = 32.0f;
constexpr float FILTER_EPS = 2.1e-3f;   // > 2^-9 + 2^-20
constexpr float FILTER_ABS = 0.02f;     // scaled units: 2e-5 of the frame's square
constexpr float FILTER_FAR = 60000.0f;  // |x_j|^2 of an unused slot; also the most a slot may hold

__device__ __forceinline__ uint32_t pack_f16(float a, float b)
{
    const f16x2_ v = __builtin_amdgcn_cvt_pkrtz(a, b);
    uint32_t r;
    __builtin_memcpy(&r, &v, 4);
    return r;
}

__device__ __forceinline__ f16x4 f16x4_of(uint32_t lo, uint32_t hi)
{
    const uint2 v = make_uint2(lo, hi);
    f16x4 r;
    __builtin_memcpy(&r, &v, 8);
    return r;
}

// The filter's particle input (every k of the column): -2 x_i, 1.
__device__ __forceinline__ f16x4 filter_column(float ax, float ay, float az)
{
    return f16x4_of(pack_f16(-2.0f * ax, -2.0f * ay), pack_f16(-2.0f * az, 1.0f));
}

// Tests of word k (of 32) of a lane's hit words for nk staged candidates: 16
// or 32 (the tile is padded to a multiple of 64). Test t of the word is bit
// n - 1 - t and candidate 128 k + 4 t + l / 16.
__device__ __forceinline__ int word_tests(int nk, int k) { return min(32, (nk - 128 * k + 63) / 64 * 16); }

// The bits of word k that belong to the 64 candidates `part` of the tile.
__device__ __forceinline__ unsigned hit_part(unsigned word, int nk, int k, int part)
{
    if (k != part >> 1) return 0u;
    return word & (word_tests(nk, k) - 16 * (part & 1) == 32 ? 0xffff0000u : 0x0000ffffu);
}

// Exclusive prefix sum over the wavefront, with the total on every lane, by
// DPP (no LDS): sums within rows of 16, then the row totals broadcast on.
__device__ __forceinline__ int wave_excl_scan(int x, int& total)
{
    int v = x;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false); // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false); // row_bcast:31 into rows 2 and 3
    total = __builtin_amdgcn_readlane(v, 63);
    return v - x;
}

// Largest v >= 0 over the wavefront, in the same steps.
__device__ __forceinline__ int wave_max_u(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// ---- work items: their particles, frames and candidates ----------------------------------
//
// Two layouts. A grid layout (UNI: no top cell split, see the cell build)
// keeps the particles of every column of top cells in order of z, so an item is
// 16 consecutive particles of one column whatever cells they are in, and its
// candidates are at most 18 runs of consecutive particles: the z range within
// reach of the item's own, in its column and the eight around it, and what
// wraps around the box. Positions are 32-bit fractions of the box or of an equal
// piece of it (piece_bits in the cell build), whose
// differences are exact and periodic, so there are no frames to shift between.
// A tree layout's items are runs of one leaf's particles, its candidates the
// leaf's records (neighbour leaf and frame shift), its positions FP32 offsets
// from their leaf's centre.
struct CellArgs {
    const int4* cells;       // per slot, tree: first particle, count, first record, records. Grid, two per slot:
                             // first particle, count | G << 8, x | y << 16 of the column, first | last << 16 of
                             // its fine cells in z; first fine cell of the box, the box's unit of length
                             // (two floats, high and low part), width of a cell in 32-bit fractions
    const float4* pbox;      // per slot, 2: centre of the box around its particles (grid: 32-bit fractions) and
                             // largest search radius; half widths, -
    const int2* p_rec;       // tree: per record, first particle and count of the neighbour leaf
    const float4* p_shift;   // tree: its frame shift, first item (bits)
    const float4* ibox;      // tree: pbox by item rather than by slot
    const int* starts;       // grid: first particle of each fine cell
    int fzb;                 // grid: fine cells in z per top cell, logarithm
};

inline CellArgs cell_args(sph_ctx* c, const int4* cells)
{
    CellArgs g;
    g.cells = cells;
    g.pbox = static_cast<float4*>(c->cell_pbox.p);
    g.p_rec = static_cast<int2*>(c->p_rec.p);
    g.p_shift = static_cast<float4*>(c->p_shift.p);
    g.ibox = static_cast<float4*>(c->item_box.p);
    g.starts = static_cast<int*>(c->starts.p);
    g.fzb = c->fzb;
    return g;
}

template <bool UNI>
struct Item {
    int i0, ni;              // particles
    int ox, oy, oz;          // grid: the frame's origin, the box centre
    float sh, sl;            // grid: unit of length
    float bx, by, bz;        // box centre in the frame (grid: 0)
    float hx, hy, hz, H;     // half widths; largest search radius
};

// x of a particle in the item's frame from its stored coordinate.
template <bool UNI>
__device__ __forceinline__ float item_coord(float v, int o, float sh, float sl, float shift)
{
    if constexpr (UNI) {
        const float d = (float)(int)((unsigned)__float_as_int(v) - (unsigned)o);
        return fmaf(d, sh, d * sl);
    } else {
        return v + shift;
    }
}

// The candidates of an item, walked in order, 64 U per step: its runs (grid), or
// its records' leaves (tree). Of a neighbour leaf only the items whose boxes are
// within reach of this item's box are walked, from the first of them to the
// last: a leaf within reach of a leaf has many particles that are not (force
// loop, where the reach may be the neighbour's: 726 -> 607 us on the clustered
// 2^20 set, 9.9 -> 8.3 ms on the log-normal 2^24 set). The
// runs left, up to 64 at a time, are rows of an LDS table (first particle minus
// offset, and the shift), where each candidate slot reads its own; the row of a
// slot is found from marks at the first slots of the rows, made for 256 slots at
// a time.
template <bool UNI>
struct CandWalk {
    int pb0, np;            // tree: first record, records
    int b0;                 // tree: first record not in the table yet
    int nj;                 // candidates of the table
    int c;                  // next of them
    int q;                  // row holding the last slot before the marks' next 64
    int off;                // candidates before row `lane` (no such row: out of range)
    float reach;            // tree: an item is in reach within this, or (own) its own largest radius
    bool own;
};

constexpr int WALK_MARKS = 256;
template <bool UNI>
constexpr int WALK_LDS = 64 * (UNI ? 4 : 16) + WALK_MARKS;  // table and marks

constexpr int WALK_NO_ROW = 0x40000000;

// The marks of the 256 slots from w.c (a multiple of 256) on.
template <bool UNI>
__device__ __forceinline__ void walk_marks(CandWalk<UNI>& w, char* lds)
{
    const int lane = threadIdx.x & 63;
    uint8_t* mk = reinterpret_cast<uint8_t*>(lds + 64 * (UNI ? 4 : 16));
    wave_sync_lds();
    reinterpret_cast<uint32_t*>(mk)[lane] = 0;
    wave_sync_lds();
    const int s = w.off - w.c;
    if (s >= 0 && s < WALK_MARKS) mk[s] = 1;
    w.q = __popcll(__ballot(w.off < w.c)) - 1;
    wave_sync_lds();
}

// The table of the next records (tree), as many blocks of 64 as fit in its rows.
__device__ __forceinline__ void walk_fill(CandWalk<false>& w, const CellArgs& G, const Item<false>& it, char* lds)
{
    const int lane = threadIdx.x & 63;
    int* offs = reinterpret_cast<int*>(lds + 64 * 16);  // (in the place of the marks)
    int rows = 0;
    wave_sync_lds();
    w.nj = 0;
    do {
        const int r = w.b0 + lane;
        int cnt = 0, first = 0;
        float4 sh = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r < w.np) {
            const int2 rec = G.p_rec[w.pb0 + r];
            sh = G.p_shift[w.pb0 + r];
            const int nt = (rec.y + 15) >> 4;
            first = rec.x;
            cnt = rec.y;
            if (nt <= 4) {
                const float4* b = G.ibox + 2 * (int64_t)__float_as_int(sh.w);
                int lo = 4, hi = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int k = 2 * min(t, nt - 1);
                    const float4 c = b[k], h = b[k + 1];
                    const float gx = fmaxf(fabsf(sh.x + c.x - it.bx) - (it.hx + h.x), 0.0f),
                                gy = fmaxf(fabsf(sh.y + c.y - it.by) - (it.hy + h.y), 0.0f),
                                gz = fmaxf(fabsf(sh.z + c.z - it.bz) - (it.hz + h.z), 0.0f);
                    const float R = w.own ? fmaxf(w.reach, c.w) : w.reach;
                    if (fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < cull_reach2(R)) {
                        lo = min(lo, t);
                        hi = t + 1;
                    }
                }
                hi = min(hi, nt);
                const int a = lo < hi ? item_first_small(rec.y, nt, lo) : 0;
                first += a;
                cnt = lo < hi ? item_first_small(rec.y, nt, hi) - a : 0;
            }
        }
        const uint64_t m = __ballot(cnt > 0);
        const int k = __popcll(m);
        if (rows + k > 64) break;
        int n;
        const int off = w.nj + wave_excl_scan(cnt, n);
        if (cnt > 0) {
            const int row = rows + lanes_below(m);
            reinterpret_cast<float4*>(lds)[row] = make_float4(sh.x, sh.y, sh.z, __int_as_float(first - off));
            offs[row] = off;
        }
        rows += k;
        w.nj += n;
        w.b0 += 64;
    } while (w.b0 < w.np);
    wave_sync_lds();
    w.off = lane < rows ? offs[lane] : WALK_NO_ROW;
    w.c = 0;
    walk_marks(w, lds);
}

// Order of the nine columns: centre and corners, then edges, so a chunk of the
// list samples the whole neighbourhood (even lists).
__constant__ signed char COL9[9][2] = {{0, 0}, {-1, -1}, {1, 1}, {-1, 0}, {0, 1}, {1, -1}, {-1, 1}, {1, 0}, {0, -1}};

template <bool UNI>
__device__ __forceinline__ void item_load(Item<UNI>& it, CandWalk<UNI>& w, const CellArgs& G, int slot, char* lds)
{
    const float4 b0 = G.pbox[2 * (int64_t)slot], b1 = G.pbox[2 * (int64_t)slot + 1];
    it.hx = uniform_f(b1.x);
    it.hy = uniform_f(b1.y);
    it.hz = uniform_f(b1.z);
    it.H = uniform_f(b0.w);
    if constexpr (UNI) {
        const int4 c0 = G.cells[2 * (int64_t)slot], c1 = G.cells[2 * (int64_t)slot + 1];
        it.i0 = __builtin_amdgcn_readfirstlane(c0.x);
        it.ni = __builtin_amdgcn_readfirstlane(c0.y & 0xff);
        it.ox = __builtin_amdgcn_readfirstlane(__float_as_int(b0.x));
        it.oy = __builtin_amdgcn_readfirstlane(__float_as_int(b0.y));
        it.oz = __builtin_amdgcn_readfirstlane(__float_as_int(b0.z));
        it.sh = uniform_f(__int_as_float(c1.y));
        it.sl = uniform_f(__int_as_float(c1.z));
        it.bx = it.by = it.bz = 0.0f;
        // lane q < 9: the run of column q inside the box; q + 9: what wraps around it
        const int lane = threadIdx.x & 63;
        const int g = c0.y >> 8, gz = g << G.fzb, reach = 1 << G.fzb;
        const bool wrap = lane >= 9;
        const int q = lane < 9 ? lane : lane < 18 ? lane - 9 : 0;
        int x = (c0.z & 0xffff) + COL9[q][0], y = (c0.z >> 16) + COL9[q][1];
        x += x < 0 ? g : x >= g ? -g : 0;
        y += y < 0 ? g : y >= g ? -g : 0;
        const int lo = (c0.w & 0xffff) - reach, hi = (c0.w >> 16) + reach;
        int a, b;  // fine cells [a, b)
        if (!wrap) {
            a = max(lo, 0);
            b = min(hi + 1, gz);
        } else {
            a = lo < 0 ? lo + gz : 0;
            b = lo < 0 ? gz : max(hi + 1 - gz, 0);
        }
        int cnt = 0, first = 0;
        if (lane < 18 && a < b) {
            const int64_t col = (int64_t)c1.x + (int64_t)(x * g + y) * gz;
            first = G.starts[col + a];
            cnt = G.starts[col + b] - first;
        }
        // rows in the order of the lanes; runs with no particle are left out
        const uint64_t m = __ballot(cnt > 0);
        const int off = wave_excl_scan(cnt, w.nj), row = lanes_below(m), rows = __popcll(m);
        int* offs = reinterpret_cast<int*>(lds + 64 * 4);  // (in the place of the marks)
        wave_sync_lds();
        if (cnt > 0) {
            reinterpret_cast<int*>(lds)[row] = first - off;
            offs[row] = off;
        }
        wave_sync_lds();
        w.off = lane < rows ? offs[lane] : WALK_NO_ROW;
    } else {
        const int4 c0 = G.cells[slot];
        it.i0 = __builtin_amdgcn_readfirstlane(c0.x);
        it.ni = __builtin_amdgcn_readfirstlane(c0.y);
        it.ox = it.oy = it.oz = 0;
        it.sh = it.sl = 0.0f;
        it.bx = uniform_f(b0.x);
        it.by = uniform_f(b0.y);
        it.bz = uniform_f(b0.z);
        w.pb0 = __builtin_amdgcn_readfirstlane(c0.z);
        w.np = __builtin_amdgcn_readfirstlane(c0.w);
        w.b0 = 0;
    }
}

// To the first candidate, of those within reach of the item's box (tree; own:
// or of their own largest search radius).
template <bool UNI>
__device__ __forceinline__ void walk_start(CandWalk<UNI>& w, const CellArgs& G, const Item<UNI>& it, char* lds,
                                           float reach, bool own)
{
    if constexpr (!UNI) {
        w.b0 = 0;
        w.reach = reach;
        w.own = own;
        walk_fill(w, G, it, lds);
    } else {
        w.c = 0;
        walk_marks(w, lds);
    }
}

// The next 64 U candidates (U 1, 2 or 4), U slots per lane: false when none is
// left. ok: there is one; src: its particle (a valid index in any case); sh: its
// shift into the item's frame (tree).
template <int U>
struct Slots {
    bool ok[U];
    int src[U];
    float3 sh[U];
};

template <int U, bool UNI>
__device__ __forceinline__ bool walk_next(CandWalk<UNI>& w, const CellArgs& G, const Item<UNI>& it, char* lds,
                                          Slots<U>& S)
{
    static_assert(WALK_MARKS % (64 * U) == 0, "a step stays inside one set of marks");
    const int lane = threadIdx.x & 63;
    if (w.c >= w.nj) {
        if constexpr (UNI) {
            return false;
        } else {
            do {
                if (w.b0 >= w.np) return false;
                walk_fill(w, G, it, lds);
            } while (w.nj == 0);
        }
    } else if ((w.c & (WALK_MARKS - 1)) == 0 && w.c > 0) {
        walk_marks(w, lds);
    }
    const uint8_t* mk = reinterpret_cast<const uint8_t*>(lds + 64 * (UNI ? 4 : 16)) + (w.c & (WALK_MARKS - 1));
    bool start[U];
#pragma unroll
    for (int u = 0; u < U; ++u) start[u] = mk[64 * u + lane] != 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t m = __ballot(start[u]);
        const int row = w.q + lanes_below(m) + (start[u] ? 1 : 0);
        w.q += __popcll(m);
        const int c = w.c + 64 * u + lane;
        S.ok[u] = c < w.nj;
        const int t = min(c, w.nj - 1);
        if constexpr (UNI) {
            S.src[u] = reinterpret_cast<const int*>(lds)[row] + t;
            S.sh[u] = make_float3(0.f, 0.f, 0.f);
        } else {
            const float4 r = reinterpret_cast<const float4*>(lds)[row];
            S.src[u] = __float_as_int(r.w) + t;
            S.sh[u] = make_float3(r.x, r.y, r.z);
        }
    }
    w.c += 64 * U;
    return true;
}

// The sum over the four lanes of a column (lanes l, l ^ 16, l ^ 32, l ^ 48) and
// the share of the lower groups, for counts. Row and half swaps give both
// partners' values in two registers each, with no trip through LDS.
__device__ __forceinline__ int column_excl_scan(int n, int& total)
{
    const int lane = threadIdx.x & 63;
    const auto r = __builtin_amdgcn_permlane16_swap(n, n, false, false);  // rows (0, 0, 2, 2), (1, 1, 3, 3)
    const int p = (int)(r[0] + r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(p, p, false, false);  // lower half, upper half
    total = (int)(h[0] + h[1]);
    return ((lane & 16) ? (int)r[0] : 0) + ((lane & 32) ? (int)h[0] : 0);
}
