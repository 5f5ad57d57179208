// Near-field gravity, particle-particle: Newton's pull of section 2, Eq. 3 of
// the Swift paper, summed directly over the pairs of neighbouring cells, the
// part that the tree code of section 3.2 evaluates particle by particle:
//
//   g_i = -G sum_{j != i} m_j r_ij (r_ij^2 + eps^2)^(-3/2) S(r_ij / r_cut),
//
// r_ij the minimum image of x_i - x_j, eps a Plummer softening and
// S(x) = (1 - x^2)^2 below 1, 0 beyond: the window takes the pull to zero
// with zero slope at the cutoff, so the sum is continuous in the positions
// (the remaining 1 - S belongs to a far field of multipoles, not computed
// here). Coincident pairs add nothing.
//
// Work unit: an item of at most 16 particles per wavefront (tiles.h), as in the
// density loop. Its candidates are the particles of the cells within its search
// radii, which the cutoff may not exceed, so every pair inside r_cut is among
// them. They are staged through LDS, keeping only those within r_cut of the
// bounding box of the item's particles (the cutoff is usually well inside the
// search radius); the matrix cores propose the pairs inside r_cut (the filter of
// tiles.h) and the four lanes of a particle sum every fourth of them. It is a
// gather: each particle sums its own pairs, so there are no atomics and the
// result has the same bits on every run. Measured, here / with one wavefront per
// cell and every candidate tested on the vector units: 0.67 / 1.14 ms on 256
// boxes of 20^3 to 40^3 particles (6.9 million), bound by the issue of vector
// instructions.
#include <cmath>

#include "common.h"
#include "tiles.h"

namespace {

constexpr int GBS = 64;    // one wavefront per block
constexpr int GCAP = 128;  // candidates per LDS tile
constexpr int GLCAP = 80;  // entries of a particle's list (64 candidates always fit)
constexpr int GLSEG = GLCAP;

struct GravArgs {
    const float4* jg;       // sorted (x, y, z) as the layout stores them, m
    const uint32_t* perm;   // sorted index -> caller index
    CellArgs cell;          // the items, their frames and candidates (within the search radii)
    float* acc;             // caller order, 3 per particle
    int64_t* ctr;
    int n_slots;
    float G, eps2, rc, rc2, inv_rc2;
};

// Sorted copies of position (bits as the layout stores it) and mass; counts non-positive or
// non-finite masses.
__global__ void __launch_bounds__(256) k_grav_prologue(int64_t n, const uint32_t* __restrict__ perm,
                                                       const int4* __restrict__ xs,
                                                       const float* __restrict__ mass, int4* __restrict__ jg,
                                                       int64_t* __restrict__ ctr)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    if (p < n) {
        const float m = mass[perm[p]];
        const int4 x = xs[p];
        jg[p] = make_int4(x.x, x.y, x.z, __float_as_int(m));
        bad = !(m > 0.0f) || !isfinite(m);
    }
    const int n_bad = __syncthreads_count(bad);
    if (threadIdx.x == 0 && n_bad) atomicAdd((unsigned long long*)&ctr_slot(ctr)[CT_BAD_INPUT], (unsigned long long)n_bad);
}

template <bool UNI>
__global__ void __launch_bounds__(GBS) __attribute__((amdgpu_waves_per_eu(4))) k_gravity(GravArgs A)
{
    constexpr int NW = (GCAP + 127) / 128;
    __shared__ float4 t0[GCAP];  // x, y, z, m
    __shared__ uint2 fa[GCAP];   // filter input: x, y; z, |x|^2 (half precision)
    __shared__ uint8_t lists[16 * GLSEG];  // of the particles: candidate numbers of one tile
    __shared__ float4 scratch4[WALK_LDS<UNI> / 16];
    char* scratch = reinterpret_cast<char*>(scratch4);
    const int lane = threadIdx.x & 63;
    const int pc = lane & 15, gc = lane >> 4;  // column (particle) and lane group of the filter
    const int pq = lane >> 2, sub = lane & 3;  // particle and lane of the pair loop
    const int fin = 4 * (lane & 3) + gc;       // the candidate (of 16) this lane feeds to the filter
    const int slot = xcd_block_index();        // each XCD takes its own run of slots
    if (slot >= A.n_slots) return;             // whole wavefront
    Item<UNI> it;
    CandWalk<UNI> w;
    item_load(it, w, A.cell, slot, scratch);
    const int i0 = it.i0, ni = it.ni;
    auto frame = [&](float4 v, float3 sh) {
        return make_float4(item_coord<UNI>(v.x, it.ox, it.sh, it.sl, sh.x),
                           item_coord<UNI>(v.y, it.oy, it.sh, it.sl, sh.y),
                           item_coord<UNI>(v.z, it.oz, it.sh, it.sl, sh.z), v.w);
    };
    const float3 none = make_float3(0.f, 0.f, 0.f);
    const float reach2 = cull_reach2(A.rc);
    const float fs = FILTER_SCALE / (fmaxf(fmaxf(it.hx, it.hy), it.hz) + A.rc);
    f16x4 fcol;
    f32x4 C;
    {
        const float4 xc = frame(A.jg[i0 + min(pc, ni - 1)], none);
        const float ux = (xc.x - it.bx) * fs, uy = (xc.y - it.by) * fs, uz = (xc.z - it.bz) * fs;
        const float n2 = fmaf(ux, ux, fmaf(uy, uy, uz * uz)) * (1.0f - FILTER_EPS) - FILTER_ABS;
        fcol = filter_column(ux, uy, uz);
        const float c = pc < ni ? fmaf(A.rc2 * (fs * fs), -(1.0f + FILTER_EPS), n2) : 1.0e9f;
        C = {c, c, c, c};
    }
    const bool valid = pq < ni;
    const int i = i0 + (valid ? pq : 0);
    const float4 xi = frame(A.jg[i], none);
    float ax = 0.0f, ay = 0.0f, az = 0.0f;
    int pairs = 0;  // this lane's
    int kept = 0;
    bool ok = false;
    int src = 0;
    float3 sh = none;
    float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f);
    auto fetch = [&]() -> bool {
        Slots<1> S;
            if (!walk_next<1>(w, A.cell, it, scratch, S)) return false;
            ok = S.ok[0];
            src = S.src[0];
            sh = S.sh[0];
        p0 = A.jg[src];
        return true;
    };
    walk_start(w, A.cell, it, scratch, A.rc, false);
    bool more = fetch();
    while (more) {
        // stage the candidates within r_cut of the item's box
        int nk = 0;
        do {
            const float4 q = frame(p0, sh);
            const float ux = UNI ? q.x : q.x - it.bx, uy = UNI ? q.y : q.y - it.by, uz = UNI ? q.z : q.z - it.bz;
            const float gx = fmaxf(fabsf(ux) - it.hx, 0.0f), gy = fmaxf(fabsf(uy) - it.hy, 0.0f),
                        gz = fmaxf(fabsf(uz) - it.hz, 0.0f);
            const bool keep = ok && fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < reach2;
            const uint64_t m = __ballot(keep);
            if (keep) {
                const int d = nk + lanes_below(m);
                const float fx = ux * fs, fy = uy * fs, fz = uz * fs;
                const float n2 = fmaf(fx, fx, fmaf(fy, fy, fz * fz)) * (1.0f - FILTER_EPS);
                fa[d] = make_uint2(pack_f16(fx, fy), pack_f16(fz, n2));
                t0[d] = q;
            }
            nk += __popcll(m);
            more = fetch();
        } while (more && nk + 64 <= GCAP);
        kept += nk;
        if (nk + lane < ((nk + 63) & ~63)) fa[nk + lane] = make_uint2(0u, pack_f16(0.0f, FILTER_FAR));
        wave_sync_lds();
        unsigned hit[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) hit[k] = 0u;
#pragma unroll
        for (int q = 0; q < GCAP / 64; ++q) {
            if (64 * q < nk) {
                unsigned m = hit[q >> 1];
#pragma unroll
                for (int b = 4 * q; b < 4 * q + 4; ++b) {
                    const uint2 a = fa[16 * b + fin];
                    const f32x4 D = __builtin_amdgcn_mfma_f32_4x4x4f16(f16x4_of(a.x, a.y), fcol, C, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) m = __builtin_amdgcn_alignbit(m, __float_as_uint(D[r]), 31);
                }
                hit[q >> 1] = m;
            }
        }
        // the words become lists and the lists pairs: the whole tile at once, or (a
        // list would not fit) 64 candidates at a time
        int n_all = 0, tot = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) n_all += __popc(hit[k]);
        int pre = column_excl_scan(n_all, tot);
        const bool whole = !__any(tot > GLCAP);
        for (int part = 0; part < (whole ? 1 : (nk + 63) / 64); ++part) {
            unsigned now[NW];
#pragma unroll
            for (int k = 0; k < NW; ++k) now[k] = whole ? hit[k] : hit_part(hit[k], nk, k, part);
            if (!whole) {
                int n_part = 0;
#pragma unroll
                for (int k = 0; k < NW; ++k) n_part += __popc(now[k]);
                pre = column_excl_scan(n_part, tot);
            }
            uint8_t* lp = lists + pc * GLSEG + pre;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                unsigned m = now[k];
                const int top = 128 * k + 4 * (word_tests(nk, k) - 1) + gc;
                while (m) {
                    const int bit = __builtin_ctz(m);
                    m &= m - 1;
                    *lp++ = (uint8_t)(top - 4 * bit);
                }
            }
            wave_sync_lds();
            const int nl = __shfl(tot, pq, 64);
            const uint8_t* lst = lists + pq * GLSEG;
            for (int e = sub; e < nl; e += 4) {
                // the pull on i is -m_j S (r^2 + eps^2)^(-3/2) r_ij per pair inside r_cut
                const float4 q = t0[lst[e]];
                const float dx = xi.x - q.x, dy = xi.y - q.y, dz = xi.z - q.z;
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                const bool in = r2 < A.rc2 && r2 > 0.0f;
                const float s = fmaf(-r2, A.inv_rc2, 1.0f);              // 1 - x^2
                const float inv = __builtin_amdgcn_rsqf(r2 + A.eps2);    // (r^2 + eps^2)^(-1/2)
                const float f = in ? q.w * (s * s) * (inv * inv * inv) : 0.0f;
                ax = fmaf(-f, dx, ax);
                ay = fmaf(-f, dy, ay);
                az = fmaf(-f, dz, az);
                pairs += in ? 1 : 0;
            }
            wave_sync_lds();  // every lane is done with the lists and the tile
        }
    }
    ax = group_sum(ax, 4);
    ay = group_sum(ay, 4);
    az = group_sum(az, 4);
    if (valid && sub < 3)  // three lanes of a particle store a component each
        A.acc[3 * (int64_t)A.perm[i] + sub] = A.G * (sub == 0 ? ax : sub == 1 ? ay : az);
    // the gravity call has the counters to itself
    ctr_wave_add(A.ctr, CT_FORCE_INTER, pairs);
    ctr_add_uniform(A.ctr, CT_FORCE_CAND, (int64_t)ni * kept);
}

}  // namespace

namespace sph {

void gravity_p2p(sph_ctx* c, const float* mass, double G, double eps, double r_cut, float* acc,
                 int64_t* counts, hipStream_t s)
{
    SPH_REQUIRE(c->built, SPH_E_STATE, "sph_gravity_p2p before sph_build_cells");
    SPH_REQUIRE(mass && acc, SPH_E_ARG, "null mass or acc");
    SPH_REQUIRE(std::isfinite(G) && std::isfinite(eps) && eps >= 0.0, SPH_E_ARG,
                "G must be finite and eps finite and >= 0");
    SPH_REQUIRE(std::isfinite(r_cut) && r_cut > 0.0, SPH_E_ARG, "r_cut must be finite and > 0");
    // after drifts that used up the margin of the cells, rebuild them around
    // the guesses of the last build (as the density would)
    check_drift(c, nullptr, s);
    finish_build_read(c);  // the smallest search radius of the build
    // the lists hold every pair closer than the search radius less twice the
    // distance the particles may have moved since the build. A search radius
    // is at most a third of its box (a build condition), so no two periodic
    // images of one particle both lie inside r_cut.
    unsigned w[4] = {0u, 0u, 0u, 0u};
    SPH_HIP(hipMemcpyAsync(w, c->drift.p, sizeof(w), hipMemcpyDeviceToHost, s));
    SPH_HIP(hipStreamSynchronize(s));
    float delta;
    std::memcpy(&delta, &w[0], 4);
    SPH_REQUIRE(r_cut + 2.0 * (double)delta <= (double)c->h_min, SPH_E_ARG,
                "r_cut " + std::to_string(r_cut) + " exceeds the smallest search radius of the cells (" +
                    std::to_string(c->h_min) + ", less twice the drift since the build)");
    const int64_t n = c->n;
    int64_t* ctr = static_cast<int64_t*>(c->counters.p);
    int4* jg = ensure<int4>(c, c->jg, n);
    fill_u32(ctr, 0u, 2 * (int64_t)CT_COUNT, s);
    k_grav_prologue<<<blocks_for(n, 256), 256, 0, s>>>(n, static_cast<uint32_t*>(c->perm.p),
                                                       static_cast<int4*>(c->uni ? c->xfix.p : c->xrel.p), mass,
                                                       jg, ctr);
    SPH_HIP(hipGetLastError());
    GravArgs A;
    A.jg = static_cast<float4*>(c->jg.p);
    A.perm = static_cast<uint32_t*>(c->perm.p);
    A.cell = cell_args(c, static_cast<int4*>(c->uni ? c->cells.p : c->cells_d.p));
    A.acc = acc;
    A.ctr = ctr;
    A.n_slots = (int)c->n_items;
    A.G = (float)G;
    A.eps2 = (float)(eps * eps);
    A.rc = (float)r_cut;
    A.rc2 = (float)(r_cut * r_cut);
    A.inv_rc2 = (float)(1.0 / (r_cut * r_cut));
    ev_record(c, EV_GRAV_K0, s);
    const unsigned grid = (unsigned)std::max<int64_t>(c->n_items, 1);
    if (c->uni)
        k_gravity<true><<<grid, GBS, 0, s>>>(A);
    else
        k_gravity<false><<<grid, GBS, 0, s>>>(A);
    SPH_HIP(hipGetLastError());
    ev_record(c, EV_GRAV_K1, s);
    const int64_t* hc = read_counters(c, s);
    SPH_REQUIRE(hc[CT_BAD_INPUT] == 0, SPH_E_ARG, "non-positive or non-finite mass");
    if (counts) {
        counts[0] = hc[CT_FORCE_INTER];
        counts[1] = hc[CT_FORCE_CAND];
    }
    c->tm.gravity_kernel_ms = ev_ms(c, EV_GRAV_K0, EV_GRAV_K1);
}

}  // namespace sph
