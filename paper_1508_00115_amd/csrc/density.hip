// FP32 density loop with the smoothing-length solve (section 2, Eq. 1 of the
// Swift paper, and the choice of h for a fixed weighted neighbour number).
//
// Work unit: an item of at most 16 particles (tiles.h), handled by one
// wavefront. Its candidates, the particles of the cells within reach (the self
// task and the pair tasks of section 3.1), are staged through the wavefront's
// LDS tile in the item's FP32 frame, the next 64 in flight meanwhile.
//
// Two phases (k_density):
//   A. the matrix cores propose the candidates inside each particle's search
//      radius (the filter of tiles.h); the distances of those, from FP32
//      differences, go to the particle's list in LDS;
//   B. the four lanes of a particle hold its list in registers and run
//      Newton's method on h against it: the density sums of a particle depend
//      only on its own h and the fixed positions, so the whole iteration stays
//      inside the wavefront: no global sweep and no ghost pass between
//      iterations.
// With a margin above LIST_WIDE the lists at first reach LIST_GROW times the
// starting h rather than the H the cells were built for: a third fewer entries
// at the default margin of 1.26, and a particle whose root lies beyond gets a
// second list out to H. (With a narrow margin H is the better guide: cells
// rebuilt around converged radii are often met with poorer starting values.)
// Particles whose lists did not fit are taken again, four at a time with four
// times the room. Lists hold distances only, so items whose candidates do not
// all share one mass (checked on the staged candidates) take one more sweep
// over them for the mass-weighted sums at the final h. A particle with more
// neighbours than even that room holds is left to k_density_scan: k_density
// queues its item, and the re-scanning kernel (launched after it on the same
// stream, idle when the queue is empty) solves it over longer lists of distances
// and masses, or by re-testing every candidate, 16 lanes per particle. A
// particle whose root lies beyond its search radius H is flagged; the host
// rebuilds the cells around a larger guess and solves it again.
//
// What bounds it: the issue of vector instructions, about 145 per particle on a
// grid, where one leaves every 4.0 cycles of a SIMD (they cost 2.6 to 4.4 by kind)
// with four wavefronts there; a wavefront's cycles go 14% to staging, 30% to the
// filter and the lists, 21% to Newton and a third to the item's start and end. In a
// tree (265 per particle, three wavefronts, by LDS) one leaves every 6: the walk of the candidates
// takes 38%. Measured, here / with one wavefront per cell and no matrix cores:
// 256 boxes of 20^3 to 40^3 particles, 6.9 million in all, 1.64 / 2.60 ms, clustered
// 2^20 0.75 / 1.01 ms, log-normal 2^24 11.3 / 11.8 ms (the last two with the re-scans,
// which the older form left more of); bench.py's 7.2 million in 256 boxes 1.77 ms. Tiles of 256, 192 and
// 128 candidates: 2.09, 1.91 and 1.72 ms on the 6.9 million (occupancy), 64: 1.95.
#include "common.h"
#include "tiles.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

constexpr int BS = 64;         // one wavefront per block (finest LDS allocation)
constexpr int WAVES = BS / 64;
constexpr int DCAP = 128;      // candidates per LDS tile (list kernel)
constexpr int SCAP = 512;      // candidates per LDS tile (re-scanning kernel)
constexpr float LIST_GROW = 1.12f;  // first list radius over the starting h, where the margin is wide
constexpr double LIST_WIDE = 1.2;   // h_margin from which lists start at LIST_GROW

struct DensArgs {
    const float4* jd;        // sorted (x, y, z) as the layout stores them, m
    const float* Hs;         // sorted search radii
    float* hs;               // sorted h: in, start value; out, result
    float* rhos;
    float* fs;
    uint8_t* st_s;           // sorted state
    const uint32_t* perm;    // sorted index -> caller index
    float* h_out;            // caller order: h (on an overflow, the larger guess
                             // the rebuild starts from)
    float* rho_out;
    float* f_out;
    float* nw_out;           // weighted neighbour count (null: not wanted)
    uint8_t* status;         // caller order
    CellArgs cell;           // the items, their frames and candidates (tree: the records within the leaf's
                             // largest search radius, a prefix of its list: the density needs no others)
    int64_t* ctr;
    int* scan_cells;         // schedule slots queued for k_density_scan (ctr[CT_SCAN_CELLS] of them)
    WorkSched W;             // which wavefront takes which cell
    float target;            // S0 = sum w(q) at the root: 3 n_ngb / 32
    float inv_target;        // 1 / target
    float tol;               // on |S0 / target - 1|
    int max_iter;
    // ghost step fused into the outputs (null jf: not fused): the force
    // loop's three float4 per particle from the final h, rho, f and the
    // caller-order velocity and u
    const float* vel_in;
    const float* u_in;
    float4* jf;
    float gamma;
    const float* drift;      // [0]: bound on the drift since the build (search Hs - 2 drift)
    float grow;              // first list radius over the starting h
    int list_room;           // (HALF) room of a list at which an item is taken whole
    int scan_lists;          // the re-scanning kernel's lists hold more than a second round of the list kernel
    int detail;              // count the list-building tests and the listed candidates
                             // (sph_params.timing = 2; the list kernel's DETAIL instance)
};

// Sorted copies of position (bits as the layout stores it), mass, h and state. fresh: every
// particle starts active; otherwise the caller-order state of the previous
// pass is kept (an overflowed particle starts again). The pass's fused ghost
// step reads velocity and u itself, by caller index, where it writes the
// particle's force streams: copying them here would gather them once more.
__global__ void __launch_bounds__(256) k_dens_prologue(int64_t n, const uint32_t* __restrict__ perm,
                                                       const int4* __restrict__ xs,
                                                       const float* __restrict__ mass,
                                                       const float* __restrict__ h_in,
                                                       const uint8_t* __restrict__ status, int fresh,
                                                       int4* __restrict__ jd, float* __restrict__ hs,
                                                       uint8_t* __restrict__ st_s, int64_t* __restrict__ ctr)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    if (p < n) {
        const uint32_t o = perm[p];
        const float m = mass[o];
        const float h = h_in[o];
        const int4 x = xs[p];
        jd[p] = make_int4(x.x, x.y, x.z, __float_as_int(m));
        hs[p] = h;
        const uint8_t st = fresh ? (uint8_t)ST_ACTIVE : status[o];
        st_s[p] = st == ST_OVERFLOW ? (uint8_t)ST_ACTIVE : st;
        bad = !((m > 0.0f) && isfinite(m) && (h > 0.0f) && isfinite(h));
    }
    // one count per block instead of per-particle atomics on a shared counter
    const int n_bad = __syncthreads_count(bad);
    if (threadIdx.x == 0 && n_bad) atomicAdd((unsigned long long*)&ctr_slot(ctr)[CT_BAD_INPUT], (unsigned long long)n_bad);
}

// Sorted copies of the final h, rho and f after the cells were rebuilt (the
// caller-order outputs hold every particle's final values).
__global__ void k_dens_regather(int64_t n, const uint32_t* __restrict__ perm, const float* __restrict__ h,
                                const float* __restrict__ rho, const float* __restrict__ f,
                                float* __restrict__ hs, float* __restrict__ rhos, float* __restrict__ fs)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint32_t o = perm[p];
    hs[p] = h[o];
    rhos[p] = rho[o];
    fs[p] = f[o];
}

// Newton state of one particle's h.
struct HSolve {
    float h, lo, hi, Hi;
    bool hi_known, done;
    uint8_t state;
    int nev;
};

__device__ __forceinline__ HSolve hsolve_init(float h, float Hi, bool done, uint8_t st0)
{
    HSolve s;
    s.Hi = Hi;
    s.h = (!(h > 0.0f) || h > Hi) ? Hi : h;
    s.lo = 0.0f;
    s.hi = Hi;
    s.hi_known = false;
    s.done = done;
    s.state = st0;
    s.nev = 0;
    return s;
}

// One Newton update from the sums at the current h: bracketed step on ln S0
// against ln h (exact where S0 ~ h^slope), bisection when the step leaves the
// bracket. Stops on |S0/target - 1| <= tol, on a step below FP32 resolution of
// h, on a root beyond the search radius (overflow) or after max_iter.
// Quotients use the hardware reciprocal (1 ulp): they only steer the steps,
// and the tests above are far coarser.
__device__ __forceinline__ void hsolve_step(HSolve& s, float S0, float S1, float inv_target, float tol, int max_iter)
{
    ++s.nev;
    const float ratio = S0 * inv_target;
    if (fabsf(ratio - 1.0f) <= tol) {
        s.done = true;
        s.state = ST_DONE;
        return;
    }
    if (ratio < 1.0f) {
        s.lo = s.h;
    } else {
        s.hi = s.h;
        s.hi_known = true;
    }
    if (ratio < 1.0f && s.h >= s.Hi) {
        s.done = true;
        s.state = ST_OVERFLOW;
        return;
    }
    const float slope = -S1 * __builtin_amdgcn_rcpf(S0);  // d ln S0 / d ln h
    float hn = slope > 0.05f ? s.h * __expf(-__logf(ratio) * __builtin_amdgcn_rcpf(slope)) : 2.0f * s.h;
    // a step to Hi is always evaluated there: however short, the root may lie beyond
    const bool edge = hn >= s.hi && !s.hi_known;
    if (hn >= s.hi) hn = s.hi_known ? 0.5f * (s.h + s.hi) : s.Hi;
    if (hn <= s.lo) hn = 0.5f * (s.lo + s.h);
    if (!edge && fabsf(hn - s.h) <= 2.5e-7f * s.h) {
        s.done = true;  // the next step is below FP32 resolution of h: h is the root
        s.state = ST_DONE;
        return;
    }
    if (s.nev >= max_iter) {
        s.done = true;
        s.state = ST_UNCONVERGED;
        return;
    }
    s.h = hn;
}

// Outputs of one particle at its final h (sums M0 = sum m w, M1 = sum m q w'):
// sorted copies for the force loop, caller-order outputs at o = perm[i]
// (loaded with the particle, so the stores wait for nothing). SORTED_STATE
// false leaves the sorted state as it is: the re-scanning kernel's wavefronts
// that share a cell number its flagged particles from it, and nothing reads it
// after that kernel (the caller-order state carries over to the next pass).
template <bool SORTED_STATE = true>
__device__ __forceinline__ void write_result(KernArgs<DensArgs> A, int i, uint32_t o, const HSolve& s, float S0,
                                             float M0, float M1)
{
    float h_report = s.h;
    if (s.state == ST_OVERFLOW) {
        // propose the radius at which a uniform density would hold the target
        // (the rebuild starts this particle from there)
        h_report = s.h * fmaxf(cbrtf(A->target / S0), 1.0f) * 1.05f;
    }
    // (rare: counted at once rather than in registers that live through the kernel)
    if (s.state == ST_OVERFLOW) atomicAdd((unsigned long long*)&ctr_slot(A->ctr)[CT_OVERFLOW], 1ull);
    if (s.state == ST_UNCONVERGED) atomicAdd((unsigned long long*)&ctr_slot(A->ctr)[CT_UNCONV], 1ull);
    const float hinv = __builtin_amdgcn_rcpf(s.h);
    const float rho = (8.0f / SPH_PI_F) * M0 * hinv * hinv * hinv;
    const float f = M1 < 0.0f ? -3.0f * M0 * __builtin_amdgcn_rcpf(M1) : 1.0f;
    A->hs[i] = s.h;
    A->rhos[i] = rho;
    A->fs[i] = f;
    if (SORTED_STATE) A->st_s[i] = s.state;
    A->h_out[o] = h_report;
    A->rho_out[o] = rho;
    A->f_out[o] = f;
    if (A->nw_out) A->nw_out[o] = (32.0f / 3.0f) * S0;
    A->status[o] = s.state;
    if (A->jf) {
        // the ghost step of this particle (the same arithmetic as the force
        // loop's ghost kernel, so both give the same bits), with the checks
        // of its velocity and u: every particle of the pass passes here once
        const float4 x = A->jd[i];
        const float h = s.h;
        const float uu = A->u_in[o];
        const float vx = A->vel_in[3 * (int64_t)o], vy = A->vel_in[3 * (int64_t)o + 1],
                    vz = A->vel_in[3 * (int64_t)o + 2];
        if (!(uu >= 0.0f) || !isfinite(uu) || !isfinite(vx) || !isfinite(vy) || !isfinite(vz))
            atomicAdd((unsigned long long*)&ctr_slot(A->ctr)[CT_BAD_INPUT], 1ull);
        const float gamma = A->gamma;
        const float P = (gamma - 1.0f) * rho * uu;
        const float c = sqrtf(gamma * (gamma - 1.0f) * uu);
        const float phi = f * P / (rho * rho);
        A->jf[3 * (int64_t)i + 0] = make_float4(x.x, x.y, x.z, h * h);
        A->jf[3 * (int64_t)i + 1] = make_float4(vx, vy, vz, x.w);
        A->jf[3 * (int64_t)i + 2] = make_float4(rho, phi, c, 1.0f / h);
    }
}

// The wavefront's totals (every argument wave-uniform).
__device__ __forceinline__ void flush_counters(KernArgs<DensArgs> A, int64_t cand_acc, int64_t list_acc,
                                               int64_t inter_acc, int64_t sweep_acc, int max_ev, int64_t n_scan,
                                               int64_t listed_acc)
{
    ctr_add_uniform(A->ctr, CT_DENS_CAND, cand_acc + list_acc);
    if (A->detail) {
        ctr_add_uniform(A->ctr, CT_DENS_TESTS, cand_acc);
        ctr_add_uniform(A->ctr, CT_DENS_LISTED, listed_acc);
    }
    ctr_add_uniform(A->ctr, CT_DENS_INTER, inter_acc);
    ctr_add_uniform(A->ctr, CT_DENS_SWEEP_INTER, sweep_acc);
    ctr_add_uniform(A->ctr, CT_NEED_SCAN, n_scan);
    if ((threadIdx.x & 63) == 0) atomicMax((unsigned long long*)&ctr_slot(A->ctr)[CT_SWEEPS], (unsigned long long)max_ev);
}

// Queue schedule slot `slot` for the re-scanning kernel when any lane flagged
// a particle of its cell.
__device__ __forceinline__ void enqueue_scan(KernArgs<DensArgs> A, int slot, int n_flag)
{
    if (__any(n_flag > 0) && (threadIdx.x & 63) == 0) {
        const int64_t k = (int64_t)atomicAdd((unsigned long long*)&A->ctr[CT_SCAN_CELLS], 1ull);
        A->scan_cells[k] = slot;
    }
}

// ---- the list kernel ----------------------------------------------------------------

// One wavefront per item. LCAP: list entries of a particle, LCAP / 4 per lane in
// registers. UNI: a grid layout (no culling of the candidates there: a cell one
// search radius wide loses only the block's corners, which costs about what it
// saves; a tree layout keeps the candidates within reach of the box around the
// item's particles). DETAIL: also count the candidates inside H
// (sph_params.timing = 2).
//
// Rounds: the first takes all of the item's particles, four lanes each; those
// whose list did not fit, or whose root lies beyond it, are taken up to four at
// a time after that, 16 lanes and four times the room each. HALF, for more neighbours
// than 16 lists hold with two wavefronts on a SIMD: the item's particles still at
// once where they are so few that each has room for list_room entries, else eight at a
// time, eight lanes and twice the room each.
template <int LCAP, bool HALF, bool UNI, bool DETAIL>
__global__ void __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(4))) k_density(DensArgs A)
{
    static_assert(LCAP % 16 == 0, "a lane reads its list four entries at a time");
    constexpr int SEG = LCAP + 4;    // (skewed against bank conflicts)
    constexpr int TOT = 16 * SEG;    // LDS entries of the lists
    constexpr int NR = HALF && LCAP < 300 ? 28 : LCAP / 16;  // float4 of a lane's entries
    constexpr int NW = (DCAP + 127) / 128;
    constexpr int U = 2;             // candidates per lane and step
    constexpr float FAR2 = 1.0e30f;  // r^2 of an empty entry
    __shared__ float4 t0[DCAP];      // x, y, z, m
    __shared__ uint2 fa[DCAP];       // filter input: x, y; z, |x|^2 (half precision)
    __shared__ float4 list4[16 * SEG / 4];
    __shared__ float4 scratch4[WALK_LDS<UNI> / 16];
    float* list = reinterpret_cast<float*>(list4);
    char* scratch = reinterpret_cast<char*>(scratch4);
    const int lane = threadIdx.x & 63;
    const int pc = lane & 15, gc = lane >> 4;  // column (particle) and lane group of the filter
    const int fin = 4 * (lane & 3) + gc;       // the candidate (of 16) this lane feeds to the filter
    const float two_delta = 2.0f * A.drift[0];  // the cells are searched to Hs - 2 drift
    int wstate = 0, a_cur = 0, a_end = 0;
    int64_t cand_acc = 0, inter_acc = 0, sweep_acc = 0, listed_acc = 0, list_acc = 0;  // wave-uniform
    int n_scan = 0, max_ev = 0;                                                        // wave-uniform

    for (;;) {
        if (a_cur >= a_end && !next_items(A.W, A.ctr, WAVES, wstate, a_cur, a_end)) break;
        const int slot = __builtin_amdgcn_readfirstlane(a_cur);
        ++a_cur;
        Item<UNI> it;
        CandWalk<UNI> w;
        item_load(it, w, A.cell, slot, scratch);
        const int i0 = it.i0, ni = it.ni;
        // this lane's column
        const int ic = i0 + min(pc, ni - 1);
        const float4 jc = A.jd[ic];
        const float Hc = A.Hs[ic] - two_delta, hc = A.hs[ic];
        const float m0 = uniform_f(jc.w);  // the mass of the item's first particle
        const float xc = item_coord<UNI>(jc.x, it.ox, it.sh, it.sl, 0.0f),
                    yc = item_coord<UNI>(jc.y, it.oy, it.sh, it.sl, 0.0f),
                    zc = item_coord<UNI>(jc.z, it.oz, it.sh, it.sl, 0.0f);
        // masks over the item's particles: unsolved; those to be listed out to H; left to the re-scan
        unsigned todo = (unsigned)__ballot(lane < ni && A.st_s[ic] == ST_ACTIVE);
        unsigned wide = 0u, scan = 0u;
        unsigned again = 0u;  // those whose candidates are walked more than once (rescanned_density)
        int n_flag = 0;
        if constexpr (DETAIL) {
            // the candidates inside H (the lists need not reach it): a walk of its own
            const float Hp = (todo >> pc) & 1u ? Hc : 0.0f, H2 = Hp * Hp;
            int inside = 0, all;
            Slots<1> S;
            walk_start(w, A.cell, it, scratch, uniform_f(group_max(Hp, 16)), false);
            while (walk_next<1>(w, A.cell, it, scratch, S)) {
                const float4 v = A.jd[S.src[0]];
                wave_sync_lds();
                t0[lane] = S.ok[0] ? make_float4(item_coord<UNI>(v.x, it.ox, it.sh, it.sl, S.sh[0].x),
                                                 item_coord<UNI>(v.y, it.oy, it.sh, it.sl, S.sh[0].y),
                                                 item_coord<UNI>(v.z, it.oz, it.sh, it.sl, S.sh[0].z), 0.0f)
                                   : make_float4(1.0e15f, 0.0f, 0.0f, 0.0f);
                wave_sync_lds();
                for (int k = 0; k < 16; ++k) {
                    const float4 q = t0[4 * k + gc];
                    const float dx = xc - q.x, dy = yc - q.y, dz = zc - q.z;
                    inside += fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < H2 ? 1 : 0;
                }
            }
            wave_excl_scan(inside, all);
            listed_acc += all;
        }

        unsigned big = 0u;  // (HALF) those to be taken with the most room
        for (int round = 0; todo; ++round) {
            // ---- this round's particles, and which one this lane works for -------------------
            const bool first = HALF ? (todo & ~big) != 0u : round == 0;
            const unsigned pool = HALF && first ? todo & ~big : todo;
            const bool whole = HALF && first && A.list_room <= 16 * NR && __popc(pool) * (A.list_room + 4) <= TOT;
            const int lg = first ? (HALF && !whole ? 3 : 2) : 4, lpp = 1 << lg;
            const int sub = lane & (lpp - 1);
            unsigned batch = pool;
            int pq = lane >> lg;
            if (HALF || !first) {
                unsigned rest = pool;
                int pk = 0;
#pragma unroll
                for (int k = 0; k < (HALF ? 16 : 4); ++k) {
                    if (k < 64 >> lg) {
                        pk = pq == k && rest ? __builtin_ctz(rest) : pk;
                        rest &= rest - 1;
                    }
                }
                batch = pool & ~rest;
                const bool any = pq < __popc(batch);
                pq = any ? pk : 31;
            }
            const bool mine = (batch >> pq) & 1u;
            const int iq = i0 + (mine ? pq : 0);
            // column pc: its list segment, and the first lane of its particle
            const bool inb = (batch >> pc) & 1u;
            const int rank = HALF || !first ? __popc(batch & ((1u << pc) - 1u)) : pc;
            const int lane_c = (rank << lg) & 63;
            // (a list's stride and room)
            const int stride = whole ? min(16 * NR, (TOT / __popc(pool) - 4) & ~15) + 4 : (lpp >> 2) * SEG;
            const int seg = stride * rank;
            const int room = whole ? stride - 4 : (lpp >> 2) * LCAP;
            const float h_start = A.hs[iq], H = A.Hs[iq] - two_delta;
            HSolve s = hsolve_init(h_start, H, !mine, ST_ACTIVE);
            {
                const float R = (wide >> pq) & 1u ? H : fminf(H, A.grow * s.h);
                s.h = fminf(s.h, R);
                s.Hi = s.hi = R;
            }
            const bool cut = s.Hi < H;  // the list may miss the root
            bool solved = false;
            bool mixed = false;         // wave-uniform: masses differ
            float fS0 = 0.f, fS1 = 0.f, M0 = 0.f, M1 = 0.f;
            for (int acc = 0;; acc = 1) {
                // ---- sweep the candidates: lists inside R, or (acc) the sums inside h ---------------
                float Rc;
                if (acc) {
                    Rc = __shfl(solved ? s.h : 0.0f, lane_c, 64);
                } else {
                    const float h0 = !(hc > 0.0f) || hc > Hc ? Hc : hc;
                    Rc = (wide >> pc) & 1u ? Hc : fminf(Hc, A.grow * h0);
                }
                if (!inb) Rc = 0.0f;
                const float R2 = Rc * Rc;
                const float hic = __builtin_amdgcn_rcpf(Rc > 0.0f ? Rc : 1.0f);
                const float reach = uniform_f(group_max(Rc, 16));
                const float reach2 = cull_reach2(reach);
                const float fs = FILTER_SCALE / (fmaxf(fmaxf(it.hx, it.hy), it.hz) + reach);
                f16x4 fcol;
                f32x4 C;
                {
                    const float ux = (xc - it.bx) * fs, uy = (yc - it.by) * fs, uz = (zc - it.bz) * fs;
                    const float n2 = fmaf(ux, ux, fmaf(uy, uy, uz * uz)) * (1.0f - FILTER_EPS) - FILTER_ABS;
                    fcol = filter_column(ux, uy, uz);
                    const float c = Rc > 0.0f ? fmaf(R2 * (fs * fs), -(1.0f + FILTER_EPS), n2) : 1.0e9f;
                    C = {c, c, c, c};
                }
                int T = 0, kept = 0, nk = 0;  // entries of this column's particle; candidates kept; in the tile
                bool differs = false;
                float cM0t = 0.f, cM0u = 0.f, cM1t = 0.f, cM1u = 0.f;
                Slots<U> S;
                float4 p0[U];
                auto fetch = [&]() -> bool {
                    if (!walk_next<U>(w, A.cell, it, scratch, S)) return false;
#pragma unroll
                    for (int u = 0; u < U; ++u) p0[u] = A.jd[S.src[u]];
                    return true;
                };
                walk_start(w, A.cell, it, scratch, reach, false);
                bool more = fetch();
                for (;;) {
                    // ---- stage, while the tile has room ------------------------------------------------
                    bool full = !more;
                    if (more) {
                        float x[U], y[U], z[U];
                        uint64_t m[U];
                        int n = 0;
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            x[u] = item_coord<UNI>(p0[u].x, it.ox, it.sh, it.sl, S.sh[u].x);
                            y[u] = item_coord<UNI>(p0[u].y, it.oy, it.sh, it.sl, S.sh[u].y);
                            z[u] = item_coord<UNI>(p0[u].z, it.oz, it.sh, it.sl, S.sh[u].z);
                            bool keep = S.ok[u];
                            if constexpr (!UNI) {
                                const float gx = fmaxf(fabsf(x[u] - it.bx) - it.hx, 0.0f),
                                            gy = fmaxf(fabsf(y[u] - it.by) - it.hy, 0.0f),
                                            gz = fmaxf(fabsf(z[u] - it.bz) - it.hz, 0.0f);
                                keep = keep && fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < reach2;
                            }
                            m[u] = __ballot(keep);
                            n += __popcll(m[u]);
                        }
                        // A grid keeps every candidate, so its tile is one step; a tree about a
                        // third of them, so a step that does not fit is taken again after the tile
                        // (never one that does not fit an empty tile: boxes 1757 -> 1725 us; in a
                        // tree whole steps alone fill the tile less: clustered 764 -> 777 us).
                        full = UNI || nk + n > DCAP;
                        if (UNI || !full) {
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                differs |= S.ok[u] && p0[u].w != m0;
                                if ((m[u] >> lane) & 1u) {
                                    const int d = nk + lanes_below(m[u]);
                                    const float fx = (x[u] - it.bx) * fs, fy = (y[u] - it.by) * fs,
                                                fz = (z[u] - it.bz) * fs;
                                    const float n2 = fmaf(fx, fx, fmaf(fy, fy, fz * fz)) * (1.0f - FILTER_EPS);
                                    fa[d] = make_uint2(pack_f16(fx, fy), pack_f16(fz, n2));
                                    t0[d] = make_float4(x[u], y[u], z[u], p0[u].w);
                                }
                                nk += __popcll(m[u]);
                            }
                            more = fetch();
                        }
                    }
                    if (!full) continue;
                    kept += nk;
                    if (nk + lane < ((nk + 63) & ~63)) fa[nk + lane] = make_uint2(0u, pack_f16(0.0f, FILTER_FAR));
                    wave_sync_lds();

                    // ---- filter --------------------------------------------------------------------------
                    unsigned hit[NW];
#pragma unroll
                    for (int k = 0; k < NW; ++k) hit[k] = 0u;
#pragma unroll
                    for (int q = 0; q < DCAP / 64; ++q) {
                        if (64 * q < nk) {
                            unsigned m = hit[q >> 1];
#pragma unroll
                            for (int b = 4 * q; b < 4 * q + 4; ++b) {
                                const uint2 a = fa[16 * b + fin];
                                const f32x4 D =
                                    __builtin_amdgcn_mfma_f32_4x4x4f16(f16x4_of(a.x, a.y), fcol, C, 0, 0, 0);
#pragma unroll
                                for (int r = 0; r < 4; ++r) m = __builtin_amdgcn_alignbit(m, __float_as_uint(D[r]), 31);
                            }
                            hit[q >> 1] = m;
                        }
                    }
                    if (acc) {
                        // the mass-weighted sums at the final h (zero from r = h on)
#pragma unroll
                        for (int k = 0; k < NW; ++k) {
                            unsigned m = hit[k];
                            const int top = 128 * k + 4 * (word_tests(nk, k) - 1) + gc;
                            while (m) {
                                const int bit = __builtin_ctz(m);
                                m &= m - 1;
                                const float4 q = t0[top - 4 * bit];
                                const float dx = xc - q.x, dy = yc - q.y, dz = zc - q.z;
                                const float r = __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
                                const float t = __builtin_amdgcn_fmed3f(fmaf(-r, hic, 1.0f), 0.0f, 1.0f);
                                const float u = __builtin_amdgcn_fmed3f(fmaf(-r, hic, 0.5f), 0.0f, 1.0f);
                                const float mt = q.w * t * t, mu = q.w * u * u;
                                cM0t = fmaf(mt, t, cM0t);
                                cM0u = fmaf(mu, u, cM0u);
                                cM1t = fmaf(r * hic, mt, cM1t);
                                cM1u = fmaf(r * hic, mu, cM1u);
                            }
                        }
                    } else {
                        int n = 0, tot = 0;
#pragma unroll
                        for (int k = 0; k < NW; ++k) n += __popc(hit[k]);
                        const int pre = column_excl_scan(n, tot);
                        float* lp = list + seg + T + pre;
                        T += tot;
                        const bool fits = T <= room;
#pragma unroll
                        for (int k = 0; k < NW; ++k) {
                            unsigned m = fits ? hit[k] : 0u;
                            const int top = 128 * k + 4 * (word_tests(nk, k) - 1) + gc;
                            while (m) {
                                const int bit = __builtin_ctz(m);
                                m &= m - 1;
                                const float4 q = t0[top - 4 * bit];
                                const float dx = xc - q.x, dy = yc - q.y, dz = zc - q.z;
                                const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                                // (the filter's margin lets a few through: kept as empty entries)
                                *lp++ = r2 < R2 ? r2 : FAR2;
                            }
                        }
                    }
                    wave_sync_lds();
                    nk = 0;
                    if (!more) break;
                }
                mixed |= __any(differs);
                cand_acc += (int64_t)__popc((unsigned)__ballot(Rc > 0.0f) & 0xffffu) * kept;
                if (acc) {
                    // the column's lanes, then over to the particle's
                    float t = cM0t, u = cM0u, v = cM1t, x = cM1u;
#pragma unroll
                    for (int o = 16; o <= 32; o <<= 1) {
                        t += __shfl_xor(t, o, 64);
                        u += __shfl_xor(u, o, 64);
                        v += __shfl_xor(v, o, 64);
                        x += __shfl_xor(x, o, 64);
                    }
                    M0 = __shfl(fmaf(2.0f, t, -8.0f * u), pq & 15, 64);
                    M1 = __shfl(fmaf(24.0f, x, -6.0f * v), pq & 15, 64);
                    break;
                }

                // ---- the lists that fit, in registers: entries 4 (j lpp + sub) ... + 3 -----------------
                const unsigned over = (unsigned)__ballot(inb && T > room) & 0xffffu;
                if (!first) scan |= over;  // (no room here either)
                const int Tq = __shfl(T, pq & 15, 64);
                solved = mine && Tq <= room;
                const int len = solved ? Tq : 0;
                const int nj4 = (wave_max_u(len) + 4 * lpp - 1) >> (lg + 2);
                // (lane groups without a particle have no list: they read the first and write none)
                float* lq = list + (mine ? stride * (lane >> lg) : 0);
                for (int e = len + sub; mine && e < 4 * lpp * nj4; e += lpp) lq[e] = FAR2;
                wave_sync_lds();
                float4 r4[NR];
#pragma unroll
                for (int j = 0; j < NR; ++j) {
                    r4[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (j < nj4) {
                        const float4 v = *reinterpret_cast<const float4*>(lq + 4 * (j * lpp + sub));
                        r4[j] = make_float4(__builtin_amdgcn_sqrtf(v.x), __builtin_amdgcn_sqrtf(v.y),
                                            __builtin_amdgcn_sqrtf(v.z), __builtin_amdgcn_sqrtf(v.w));
                    }
                }

                // ---- phase B: Newton's method on h. w(q) = 2 t^3 - 8 u^3 and q w'(q) = q (24 u^2 - 6
                //      t^2) with t = max(1 - q, 0), u = max(1/2 - q, 0): the cubic spline as truncated
                //      powers, no branch and no select ------------------------------------------------
                bool run = solved;
                int inside_h = 0, swept = 0;
                while (__any(run)) {
                    const float hinv = __builtin_amdgcn_rcpf(s.h);
                    float At = 0.f, Au = 0.f, Bt = 0.f, Bu = 0.f;
                    int cnt = 0;  // this lane's entries inside h
                    auto entry = [&](float r) {
                        const float q = r * hinv;
                        const float t = __builtin_amdgcn_fmed3f(fmaf(-r, hinv, 1.0f), 0.0f, 1.0f);
                        const float u = __builtin_amdgcn_fmed3f(fmaf(-r, hinv, 0.5f), 0.0f, 1.0f);
                        const float t2 = t * t, u2 = u * u;
                        At = fmaf(t2, t, At);
                        Au = fmaf(u2, u, Au);
                        Bt = fmaf(q, t2, Bt);
                        Bu = fmaf(q, u2, Bu);
                        cnt += t > 0.0f ? 1 : 0;  // r < h
                    };
#pragma unroll
                    for (int j = 0; j < NR; ++j) {
                        if (j < nj4) {
                            entry(r4[j].x);
                            entry(r4[j].y);
                            entry(r4[j].z);
                            entry(r4[j].w);
                        }
                    }
                    const float S0 = group_sum(fmaf(2.0f, At, -8.0f * Au), lpp);
                    const float S1 = group_sum(fmaf(24.0f, Bu, -6.0f * Bt), lpp);
                    if (run) {
                        inside_h = cnt;
                        swept += cnt;
                        fS0 = S0;
                        fS1 = S1;
                        hsolve_step(s, S0, S1, A.inv_target, A.tol, A.max_iter);
                        run = !s.done;
                    }
                }
                {
                    // evaluations: their most, the entries they read and those inside h, and the
                    // interactions at the final h, which is the last one evaluated (less the
                    // particle itself)
                    while (__any(solved && s.nev > max_ev)) ++max_ev;
                    int a, b, d;
                    wave_excl_scan(solved && sub == 0 ? s.nev * len : 0, a);
                    wave_excl_scan(swept, b);
                    wave_excl_scan(solved && s.state == ST_DONE ? inside_h - (sub == 0 ? 1 : 0) : 0, d);
                    list_acc += a;
                    sweep_acc += b;
                    inter_acc += d;
                }
                // a root beyond a list that stopped short of H: once more, out to H
                const bool beyond = solved && s.state == ST_OVERFLOW && cut;
                if (beyond) solved = false;
                const bool beyond_c = __shfl(beyond ? 1 : 0, lane_c, 64) != 0;
                const unsigned bm = (unsigned)__ballot(inb && beyond_c) & 0xffffu;
                wide |= bm;
                again |= over | bm;
                big |= over | bm;
                todo &= ~(batch & ~bm & (first ? ~over : ~0u));
                if (!mixed || !__any(solved)) break;
            }
            if (mixed) again |= batch;
            if (solved && sub == 0) {
                if (!mixed) {
                    M0 = m0 * fS0;
                    M1 = m0 * fS1;
                }
                const KernArgs<DensArgs> K = late_args<DensArgs>();
                write_result(K, iq, K->perm[iq], s, fS0, M0, M1);
            }
        }
        n_scan += __popc(again);
        if ((scan >> lane) & 1u && lane < 16) {
            late_args<DensArgs>()->st_s[i0 + lane] = ST_SCAN;
            n_flag = 1;
        }
        enqueue_scan(late_args<DensArgs>(), slot, n_flag);
    }
    flush_counters(late_args<DensArgs>(), cand_acc, list_acc, inter_acc, sweep_acc, max_ev, n_scan, listed_acc);
}

// ---- the re-scanning kernel: particles flagged ST_SCAN -------------------------------
// Persistent wavefronts take the queued items one at a time (or, when the
// queue is short, a share of an item's groups: see `split`); a wavefront with
// no queued item left exits at once, so the launch costs little when nothing
// was queued. The flagged particles of an item are compacted and taken four at
// a time, RLPI = 16 lanes each. Phase A walks the item's candidates once and
// appends the distance and the mass of every hit inside the search radius to
// the lane's lists (room for RLPI * RSLOTS hits per particle); phase B runs
// Newton's method over the lists with mass-weighted sums. A particle with still more
// hits re-tests every candidate at each evaluation (rewalk_solve); where the list
// kernel's second round has as much room, that is all of them, and nothing is listed.
constexpr int RLPI = 16;
constexpr int RSLOTS = 32;
constexpr int GP = 64 / RLPI;  // particles per group

// One evaluation over a lane's list (r and m at stride 64) at 1/h = hinv:
// S0 = sum w, S1 = sum q w', M0 = sum m w, M1 = sum m q w', and the entries
// inside h. The cubic spline as truncated powers, as in the list kernel:
// w = 2 t^3 - 8 u^3 and q w' = q (24 u^2 - 6 t^2).
struct ListSums {
    float S0, S1, M0, M1;
    int cnt;
};

__device__ __forceinline__ ListSums list_sums(const float* lr, const float* lm, int len, float hinv)
{
    float At = 0.f, Au = 0.f, Bt = 0.f, Bu = 0.f, mAt = 0.f, mAu = 0.f, mBt = 0.f, mBu = 0.f;
    int cnt = 0;
    for (int e = 0; e < len; ++e) {
        const float r = lr[e * 64];
        const float m = lm[e * 64];
        const float q = r * hinv;
        const float t = __builtin_amdgcn_fmed3f(fmaf(-r, hinv, 1.0f), 0.0f, 1.0f);
        const float u = __builtin_amdgcn_fmed3f(fmaf(-r, hinv, 0.5f), 0.0f, 1.0f);
        const float t2 = t * t, u2 = u * u;
        const float a = t2 * t, b = u2 * u, c = q * t2, d = q * u2;
        At += a;
        Au += b;
        Bt += c;
        Bu += d;
        mAt = fmaf(m, a, mAt);
        mAu = fmaf(m, b, mAu);
        mBt = fmaf(m, c, mBt);
        mBu = fmaf(m, d, mBu);
        cnt += t > 0.0f ? 1 : 0;
    }
    ListSums L;
    L.S0 = fmaf(2.0f, At, -8.0f * Au);
    L.S1 = fmaf(24.0f, Bu, -6.0f * Bt);
    L.M0 = fmaf(2.0f, mAt, -8.0f * mAu);
    L.M1 = fmaf(24.0f, mBu, -6.0f * mBt);
    L.cnt = cnt;
    return L;
}

// The candidates of an item within reach2 of a group's box, SCAP at a time (x,
// y, z in the item's frame, m): a particle of the group pairs with no other.
// Returns how many were staged; more: there are others.
template <bool UNI>
struct RescanItem {
    Item<UNI> it;
    CandWalk<UNI> w;
};

template <bool UNI>
__device__ __forceinline__ int rescan_stage(const DensArgs& A, RescanItem<UNI>& I, float4* tile, char* scratch,
                                            bool first, bool& more, const CullBox& box, float reach2)
{
    int nk = 0;
    if (first) walk_start(I.w, A.cell, I.it, scratch, I.it.H, false);
    do {
        Slots<1> S;
        more = walk_next<1>(I.w, A.cell, I.it, scratch, S);
        if (!more) break;
        float4 a = A.jd[S.src[0]];
        a.x = item_coord<UNI>(a.x, I.it.ox, I.it.sh, I.it.sl, S.sh[0].x);
        a.y = item_coord<UNI>(a.y, I.it.oy, I.it.sh, I.it.sl, S.sh[0].y);
        a.z = item_coord<UNI>(a.z, I.it.oz, I.it.sh, I.it.sl, S.sh[0].z);
        const bool keep = S.ok[0] && box_dist2(a.x, a.y, a.z, box) < reach2;
        const uint64_t m = __ballot(keep);
        if (keep) tile[nk + lanes_below(m)] = a;
        nk += __popcll(m);
    } while (nk + 64 <= SCAP);
    wave_sync_lds();
    return nk;
}

// Newton's method re-testing every candidate at each evaluation, for the
// lanes whose particle (active) has more hits than its lists hold.
template <bool UNI, class N>
__device__ __forceinline__ void rewalk_solve(const DensArgs& A, RescanItem<UNI>& I, float4* tile, char* scratch,
                                             bool active, int i, float4 xi, int sub, const CullBox& box, float reach2,
                                             int64_t& cand_acc, N& inter_acc, N& sweep_acc, int& max_ev)
{
    HSolve s = hsolve_init(A.hs[i], A.Hs[i] - 2.0f * A.drift[0], !active, ST_ACTIVE);
    float S0 = 0.f, S1 = 0.f, M0 = 0.f, M1 = 0.f;
    int cnt = 0;
    while (__any(!s.done)) {
        const float h2 = s.h * s.h;
        const float hinv = __builtin_amdgcn_rcpf(s.h);
        S0 = S1 = M0 = M1 = 0.f;
        cnt = 0;
        const int groups_now = wave_count(!s.done && sub == 0);
        int kept_tot = 0;
        bool more = true;
        for (bool head = true; more; head = false) {
            const int kept = rescan_stage(A, I, tile, scratch, head, more, box, reach2);
            kept_tot += kept;
            for (int k = sub; k < kept; k += RLPI) {
                const float4 pj = tile[k];
                const float dx = xi.x - pj.x, dy = xi.y - pj.y, dz = xi.z - pj.z;
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                const bool in = r2 < h2;
                const float q = in ? __builtin_amdgcn_sqrtf(r2) * hinv : 1.0f;
                float w, dw;
                spline_w_dw(q, w, dw);
                const float qdw = q * dw;
                S0 += w;
                S1 += qdw;
                M0 = fmaf(pj.w, w, M0);
                M1 = fmaf(pj.w, qdw, M1);
                cnt += in ? 1 : 0;
            }
            wave_sync_lds();
        }
        cand_acc += (int64_t)groups_now * kept_tot;
        S0 = group_sum(S0, RLPI);
        S1 = group_sum(S1, RLPI);
        M0 = group_sum(M0, RLPI);
        M1 = group_sum(M1, RLPI);
        cnt = group_sum_i(cnt, RLPI);
        if (s.done) continue;
        if (sub == 0) sweep_acc += cnt;
        hsolve_step(s, S0, S1, A.inv_target, A.tol, A.max_iter);
    }
    if (active && sub == 0) {
        if (s.state == ST_DONE) inter_acc += cnt - 1;
        max_ev = max(max_ev, s.nev);
        write_result<false>(late_args<DensArgs>(), i, A.perm[i], s, S0, M0, M1);
    }
}

template <bool UNI>
__global__ void __launch_bounds__(BS) k_density_scan(DensArgs A)
{
    __shared__ float4 tile[SCAP];
    __shared__ float lr_all[(RSLOTS + 1) * 64];
    __shared__ float lm_all[(RSLOTS + 1) * 64];
    __shared__ int pidx[16];
    __shared__ float4 scratch4[WALK_LDS<UNI> / 16];
    char* scratch = reinterpret_cast<char*>(scratch4);
    const int lane = threadIdx.x & 63;
    const int g = lane / RLPI, sub = lane & (RLPI - 1);
    float* lr = lr_all + lane;
    float* lm = lm_all + lane;
    char* br = reinterpret_cast<char*>(lr_all);
    char* bm = reinterpret_cast<char*>(lm_all);
    const unsigned o_lane = 4u * (unsigned)lane, o_cap = o_lane + 256u * RSLOTS;
    const float two_delta = 2.0f * A.drift[0];
    int64_t cand_acc = 0;  // wave-uniform
    int list_acc = 0, inter_acc = 0, sweep_acc = 0;
    int max_ev = 0;
    const int n_queued = (int)A.ctr[CT_SCAN_CELLS];  // final: written by the list kernel
    // A short queue leaves most wavefronts idle while a few take items with
    // thousands of candidates, groups taken one after another. Each queued item
    // then goes to `split` wavefronts (an item has at most four groups). A group's
    // arithmetic does not depend on which wavefront runs it, so the results keep
    // their bits.
    const int n_waves = (int)gridDim.x * WAVES;
    int split = 1;
    while (split < 16 / GP && (int64_t)n_queued * split * 2 <= n_waves) split *= 2;
    const int n_items = n_queued * split;
    if ((int)blockIdx.x * WAVES + (int)(threadIdx.x >> 6) >= n_items) return;

    for (;;) {
        int k = 0;
        if (lane == 0) k = (int)atomicAdd((unsigned long long*)&A.ctr[CT_SCAN_POP], 1ull);
        k = __shfl(k, 0, 64);
        if (k >= n_items) break;
        const int kc = k / split, part = k - kc * split;
        const int slot = A.scan_cells[kc];
        RescanItem<UNI> I;
        item_load(I.it, I.w, A.cell, slot, scratch);
        const int i0 = I.it.i0, ni = I.it.ni;
        // the item's flagged particles, compacted into pidx
        const bool flag = lane < ni && A.st_s[i0 + lane] == ST_SCAN;
        const uint64_t fm = __ballot(flag);
        const int nflag = __popcll(fm);
        wave_sync_lds();  // the previous item's reads of pidx are done
        if (flag) pidx[lanes_below(fm)] = lane;
        wave_sync_lds();
        // this wavefront's groups of them: those whose number is part modulo split
        for (int p0 = GP * part; p0 < nflag; p0 += GP * split) {
            const bool valid = p0 + g < nflag;
            const int i = i0 + pidx[valid ? p0 + g : p0];
            float4 xi = A.jd[i];
            xi.x = item_coord<UNI>(xi.x, I.it.ox, I.it.sh, I.it.sl, 0.0f);
            xi.y = item_coord<UNI>(xi.y, I.it.oy, I.it.sh, I.it.sl, 0.0f);
            xi.z = item_coord<UNI>(xi.z, I.it.oz, I.it.sh, I.it.sl, 0.0f);
            HSolve s = hsolve_init(A.hs[i], A.Hs[i] - two_delta, !valid, ST_ACTIVE);

            // ---- phase A: every candidate once, hits inside H listed ----------
            const float H2 = valid ? s.Hi * s.Hi : -1.0f;
            // the staged candidates any particle of this group can pair with:
            // within its largest search radius of the box around the group
            const CullBox gbox = pass_box(xi.x, xi.y, xi.z, valid);
            const float greach2 = uniform_f(cull_reach2(wave_max(valid ? s.Hi : 0.0f)));
            unsigned o = o_lane;
            int kept_tot = 0;
            bool more = A.scan_lists != 0;
            for (bool head = true; more; head = false) {
                const int kept = rescan_stage(A, I, tile, scratch, head, more, gbox, greach2);
                kept_tot += kept;
                for (int kk = sub; kk < kept; kk += RLPI) {
                    const float4 pj = tile[kk];
                    const float dx = xi.x - pj.x, dy = xi.y - pj.y, dz = xi.z - pj.z;
                    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                    const unsigned oo = min(o, o_cap);
                    *reinterpret_cast<float*>(br + oo) = r2;
                    *reinterpret_cast<float*>(bm + oo) = pj.w;
                    o += r2 < H2 ? 256u : 0u;
                }
                wave_sync_lds();
            }
            cand_acc += (int64_t)wave_count(valid && sub == 0) * kept_tot;
            const int nl = (int)((o - o_lane) >> 8);
            const bool fits = A.scan_lists && group_sum_i(nl > RSLOTS ? 1 : 0, RLPI) == 0;

            // ---- phase B: Newton's method over the lists ---------------------
            const bool listed = valid && fits;
            if (!listed) s.done = true;
            const int len_l = listed ? nl : 0;
            for (int e = 0; e < len_l; ++e) lr[e * 64] = __builtin_amdgcn_sqrtf(lr[e * 64]);
            float fS0 = 0.f, fM0 = 0.f, fM1 = 0.f;
            int fcnt = 0;
            while (__any(!s.done)) {
                const float hinv = __builtin_amdgcn_rcpf(s.h);
                const int len_e = s.done ? 0 : len_l;
                const ListSums L = list_sums(lr, lm, len_e, hinv);
                list_acc += len_e;
                const float S0 = group_sum(L.S0, RLPI);
                const float S1 = group_sum(L.S1, RLPI);
                const float M0 = group_sum(L.M0, RLPI);
                const float M1 = group_sum(L.M1, RLPI);
                const int cnt = group_sum_i(L.cnt, RLPI);
                if (s.done) continue;
                if (sub == 0) sweep_acc += cnt;
                fS0 = S0;
                fM0 = M0;
                fM1 = M1;
                fcnt = cnt;
                hsolve_step(s, S0, S1, A.inv_target, A.tol, A.max_iter);
            }
            if (listed && sub == 0) {
                if (s.state == ST_DONE) inter_acc += fcnt - 1;
                max_ev = max(max_ev, s.nev);
                write_result<false>(late_args<DensArgs>(), i, A.perm[i], s, fS0, fM0, fM1);
            }

            // ---- lists too short: re-test every candidate per evaluation -------
            const bool rewalk = valid && !fits;
            if (__any(rewalk))
                rewalk_solve(A, I, tile, scratch, rewalk, i, xi, sub, gbox, greach2, cand_acc, inter_acc, sweep_acc,
                             max_ev);
        }
    }
    int64_t inter = inter_acc, swept = sweep_acc, listed = list_acc;  // to wavefront totals
    for (int o = 32; o >= 1; o >>= 1) {
        inter += __shfl_xor(inter, o, 64);
        swept += __shfl_xor(swept, o, 64);
        listed += __shfl_xor(listed, o, 64);
        max_ev = max(max_ev, __shfl_xor(max_ev, o, 64));
    }
    flush_counters(late_args<DensArgs>(), cand_acc, listed, inter, swept, max_ev, 0, 0);
}

}  // namespace

namespace sph {

// Work schedule of a hot kernel over n_items cells and the grid to launch:
// one wavefront per cell under hardware dispatch, or a machine-sized grid of
// persistent wavefronts popping batches from the per-XCD queues.
int make_sched(sph_ctx* c, int64_t n_items, int waves_per_block, int blocks_per_cu, WorkSched& W)
{
    W.persistent = c->prm.schedule == 1 ? 1 : 0;
    W.batch = c->prm.queue_batch > 0 ? c->prm.queue_batch : 4;
    W.n_items = (int)n_items;
    const int64_t all = (n_items + waves_per_block - 1) / waves_per_block;
    int64_t grid = all;
    if (W.persistent) grid = std::min<int64_t>(all, (int64_t)c->n_cu * blocks_per_cu);
    return (int)std::max<int64_t>(grid, 1);
}

void density_enqueue(sph_ctx* c, const float* mass, float* h, float* rho, float* f, float* nw, bool fresh,
                     bool events, hipStream_t s, const float* ghost_vel, const float* ghost_u)
{
    const int64_t n = c->n;
    int64_t* ctr = static_cast<int64_t*>(c->counters.p);
    uint8_t* status = static_cast<uint8_t*>(c->status.p);
    float4* jd = static_cast<float4*>(c->jd.p);
    float* hs = static_cast<float*>(c->hs.p);
    float* rhos = static_cast<float*>(c->rhos.p);
    float* fs = static_cast<float*>(c->fs.p);
    uint8_t* st_s = static_cast<uint8_t*>(c->st_s.p);
    const bool ghost = ghost_vel && ghost_u;
    float4* jf = ghost ? static_cast<float4*>(c->jf.p) : nullptr;
    fill_u32(ctr, 0u, 2 * (int64_t)CT_COUNT, s);  // sums, spread slots, queue heads
    k_dens_prologue<<<blocks_for(n, 256), 256, 0, s>>>(n, static_cast<uint32_t*>(c->perm.p),
                                                        static_cast<int4*>(c->uni ? c->xfix.p : c->xrel.p), mass, h,
                                                        status, fresh ? 1 : 0, static_cast<int4*>(c->jd.p), hs, st_s,
                                                        ctr);
    SPH_HIP(hipGetLastError());
    DensArgs A;
    A.jd = jd;
    A.Hs = static_cast<float*>(c->Hs.p);
    A.hs = hs;
    A.rhos = rhos;
    A.fs = fs;
    A.st_s = st_s;
    A.perm = static_cast<uint32_t*>(c->perm.p);
    A.h_out = h;
    A.rho_out = rho;
    A.f_out = f;
    A.nw_out = nw;
    A.status = status;
    A.cell = cell_args(c, static_cast<int4*>(c->uni ? c->cells.p : c->cells_d.p));
    A.ctr = ctr;
    A.target = (float)(3.0 * c->prm.n_ngb / 32.0);
    A.inv_target = (float)(32.0 / (3.0 * c->prm.n_ngb));
    A.tol = (float)c->prm.n_tol;
    A.max_iter = c->prm.max_iter;
    A.scan_cells = static_cast<int*>(c->scan_cells.p);
    A.vel_in = ghost ? ghost_vel : nullptr;
    A.u_in = ghost ? ghost_u : nullptr;
    A.jf = jf;
    A.gamma = (float)c->prm.gamma;
    A.drift = static_cast<float*>(c->drift.p);
    A.detail = c->prm.timing == 2 ? 1 : 0;
    const int grid = make_sched(c, c->n_items, WAVES, 16, A.W);
    // re-scan grid: enough wavefronts for a full queue; the surplus exits at once
    const int scan_grid = (int)std::max<int64_t>(std::min<int64_t>(c->n_items, (int64_t)c->n_cu * 8), 1);
    if (events) ev_record(c, EV_DENS_K0, s);
    // Room of the lists. A good guess finds about x = n_ngb g^3 candidates inside its
    // first radius (g the smaller of h_margin and LIST_GROW): a third more on a
    // grid, where the guesses of a lattice are good, nearly twice that in a tree,
    // where a particle that needs a second list costs its item a second sweep
    // (log-normal 2^24: 96 entries, 27 of 1000 particles, 11.9 ms; 128, 3 of 1000,
    // 11.5 ms). Longer lists cost LDS and registers, so wavefronts: the clustered
    // 2^20 set with 48 neighbours and the default margin, which just fits 128,
    // takes 936 us with 128 entries and 1291 us with 240. 240 serve to x = 235 on a
    // grid and 200 in a tree. Beyond, longer lists for all of an item leave one
    // wavefront on a SIMD (448 entries; one and a half with 320): half an item at a time,
    // or a small one (a tree's leaf of nine) whole, with the same LDS, is better (ms: a
    // list per cell of old / 448 / 320 / so): 64^3, 170 neighbours, margin 1.26: 0.74 /
    // 0.90 / 0.59 / 0.49; 100^3, 250 and 1.05: 1.94 / 4.5 / 2.85 / 2.29; 100^3, 300 and
    // 1.05: 2.37 / 4.2 / - / 3.1; clustered 2^20, 200 and 1.26: 55 / 9.6 / 9.8 / 7.6;
    // log-normal 2^21, 200 and 1.05: 6.9 / 8.9 / 7.3 / 6.1. Above x = 470 the halves'
    // lists have room for 640: 100^3, 400 and 1.26, x = 562: 24.7 / 17.8 / 10.9 / 5.6.
    const bool wide = c->prm.h_margin > LIST_WIDE;
    const double g = wide ? (double)LIST_GROW : c->prm.h_margin;
    A.grow = wide ? LIST_GROW : 1.0e30f;
    const double x = c->prm.n_ngb * g * g * g;
    const double want = (c->uni ? 1.35 : 1.85) * x;
    auto launch = [&](auto lcap, auto half) {
        constexpr int L = decltype(lcap)::value;
        constexpr bool H = decltype(half)::value;
        A.scan_lists = 4 * L < RLPI * RSLOTS ? 1 : 0;
        if (c->uni)
            A.detail ? k_density<L, H, true, true><<<grid, BS, 0, s>>>(A)
                     : k_density<L, H, true, false><<<grid, BS, 0, s>>>(A);
        else
            A.detail ? k_density<L, H, false, true><<<grid, BS, 0, s>>>(A)
                     : k_density<L, H, false, false><<<grid, BS, 0, s>>>(A);
    };
    A.list_room = (int)std::min(1.08 * x + 23.0, 1.0e6) & ~15;
    using Whole = std::false_type;
    using Half = std::true_type;
    if (want <= 80.0)
        launch(std::integral_constant<int, 80>{}, Whole{});
    else if (want <= 96.0)
        launch(std::integral_constant<int, 96>{}, Whole{});
    else if (want <= 128.0)
        launch(std::integral_constant<int, 128>{}, Whole{});
    else if (x <= (c->uni ? 235.0 : 200.0))
        launch(std::integral_constant<int, 240>{}, Whole{});
    else if (x <= 470.0)
        launch(std::integral_constant<int, 240>{}, Half{});
    else
        launch(std::integral_constant<int, 320>{}, Half{});
    SPH_HIP(hipGetLastError());
    if (events) ev_record(c, EV_DENS_KM, s);
    if (c->uni)
        k_density_scan<true><<<scan_grid, BS, 0, s>>>(A);
    else
        k_density_scan<false><<<scan_grid, BS, 0, s>>>(A);
    SPH_HIP(hipGetLastError());
    if (events) ev_record(c, EV_DENS_K1, s);
}

void density_buffers(sph_ctx* c)
{
    const int64_t n = c->n;
    ensure<uint8_t>(c, c->status, n);
    ensure<float4>(c, c->jd, n);
    ensure<float>(c, c->hs, n);
    ensure<float>(c, c->rhos, n);
    ensure<float>(c, c->fs, n);
    ensure<uint8_t>(c, c->st_s, n);
    ensure<int>(c, c->scan_cells, (size_t)c->n_items);
}

void density_f32(sph_ctx* c, const float* mass, float* h, float* rho, float* f, float* nw, sph_stats* st,
                 hipStream_t s)
{
    SPH_REQUIRE(c->built, SPH_E_STATE, "sph_density before sph_build_cells");
    SPH_REQUIRE(mass && h && rho && f, SPH_E_ARG, "null mass/h/rho/f");
    check_drift(c, h, s);
    int64_t tot_inter = 0, tot_cand = 0, tot_sweep_inter = 0, tot_scan = 0, tot_tests = 0, tot_listed = 0;
    int32_t sweeps = 0;
    c->rebuilds = 0;
    c->density_done = false;
    c->vsig_valid = c->bal_valid = c->div_valid = false;  // all belong to the h this call replaces
    c->tm.density_kernel_ms = 0.0;
    c->tm.density_rescan_ms = 0.0;
    c->tm.density_launches = 0;
    ev_record(c, EV_DENS_C0, s);
    for (;;) {
        density_buffers(c);
        // the first pass starts every particle afresh; after a rebuild the
        // particles solved earlier keep their results
        density_enqueue(c, mass, h, rho, f, nw, c->rebuilds == 0, true, s);
        const int64_t* hc = read_counters(c, s);
        c->tm.density_kernel_ms += ev_ms(c, EV_DENS_K0, EV_DENS_K1);
        c->tm.density_rescan_ms += ev_ms(c, EV_DENS_KM, EV_DENS_K1);
        c->tm.density_launches += 2;
        SPH_REQUIRE(hc[CT_BAD_INPUT] == 0, SPH_E_ARG, "non-positive or non-finite mass or h");
        tot_scan += hc[CT_NEED_SCAN];
        tot_inter += hc[CT_DENS_INTER];
        tot_cand += hc[CT_DENS_CAND];
        tot_tests += hc[CT_DENS_TESTS];
        tot_listed += hc[CT_DENS_LISTED];
        tot_sweep_inter += hc[CT_DENS_SWEEP_INTER];
        sweeps = std::max<int32_t>(sweeps, (int32_t)hc[CT_SWEEPS]);
        if (hc[CT_OVERFLOW] == 0) {
            if (st) {
                st->sweeps = sweeps;
                st->rebuilds = c->rebuilds;
                st->unconverged = hc[CT_UNCONV];
                st->interactions_density = tot_inter;
                st->interactions_force = 0;
                st->candidates_density = tot_cand;
                st->candidates_force = 0;
                st->sweep_interactions_density = tot_sweep_inter;
                st->rescanned_density = tot_scan;
                st->tests_density = tot_tests;
                st->listed_density = tot_listed;
                st->n_cells = c->n_leaves;
                finish_build_read(c);
                st->n_pairs = c->n_pairs;
            }
            if (c->rebuilds > 0) {
                // sorted copies of every particle's final values (those solved
                // before the last rebuild were not touched by its pass)
                k_dens_regather<<<blocks_for(c->n, 256), 256, 0, s>>>(
                    c->n, static_cast<uint32_t*>(c->perm.p), h, rho, f, static_cast<float*>(c->hs.p),
                    static_cast<float*>(c->rhos.p), static_cast<float*>(c->fs.p));
                SPH_HIP(hipGetLastError());
            }
            ev_record(c, EV_DENS_C1, s);
            c->tm.density_call_ms = ev_ms(c, EV_DENS_C0, EV_DENS_C1);
            SPH_REQUIRE(hc[CT_UNCONV] == 0, SPH_E_NOT_CONVERGED,
                        std::to_string(hc[CT_UNCONV]) + " smoothing lengths did not converge");
            c->density_done = true;
            return;
        }
        SPH_REQUIRE(c->rebuilds < 16, SPH_E_NOT_CONVERGED, "smoothing lengths keep outgrowing their cells");
        // cells around the current h (the overflowed particles report a larger
        // guess); converged particles keep their results and are skipped
        rebuild_cells(c, h, s);
        c->rebuilds += 1;
    }
}

}  // namespace sph
