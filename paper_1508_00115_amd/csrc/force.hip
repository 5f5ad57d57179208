// FP32 force loop: the pressure-gradient sum of the Swift paper (section 2,
// Eq. 2) in the grad-h form of Gadget-2 that Swift implements, with a
// signal-velocity artificial viscosity, in the internal-energy variable.
//
// The ghost step (after the density, section 3.1's dependency) turns rho, f
// and u into the per-particle pressure term Phi = f P / rho^2 and sound speed,
// packed with position, h^2, velocity, mass and 1/h into three float4 per
// particle: (x, y, z, h^2), (v, m), (rho, Phi, c, 1/h); x, y, z as the cell
// layout stores them (see Item in tiles.h).
// The loop then runs one wavefront per item of at most 16 particles like the
// density loop: the candidates are staged into an LDS tile, the matrix cores
// propose the pairs inside max(h_i, h_j) (two tables, one per radius), and the
// four lanes of a particle gather the terms of every fourth pair of its list.
// The gather form evaluates each pair from both sides, so no two waves write the
// same particle and the result does not depend on scheduling. Per-box momentum
// and energy rates are summed in FP64: each wave stores its item's share (plain
// stores, no atomics) and a second kernel adds the shares of each box's items in a
// fixed order, so the sums are also reproducible.
//
// What bounds it: the issue of vector instructions (one per 3.6 cycles of a SIMD on
// a grid, 4.4 in a tree), most of them in the pair loop, whose lists' lengths
// differ between particles. Measured, here / with one wavefront per cell and
// every candidate tested on the vector units: 256 boxes of 20^3 to 40^3 particles,
// 6.9 million in all, 1.57 / 2.25 ms, clustered 2^20 0.62 / 0.85 ms, log-normal 2^24
// 8.2 / 10.8 ms; bench.py's 7.2 million in 256 boxes 1.73 ms. Tiles of 192 candidates
// instead of 128: 1.91 against 1.64 ms on the boxes (LDS holds fewer wavefronts).
//
// With the Balsara switch (not in the paper; the Gadget-2 form) the same loop
// first runs in a gather mode that sums the velocity divergence and curl of
// each particle over its neighbours inside h_i (staging only position and
// velocity, testing only r < h_i) and stores the factor
// B = |div v| / (|div v| + |curl v| + 1e-4 c / h) in place of 1/h in the
// particle's third float4, (rho, Phi, c, B); the force loop then takes 1/h
// from h^2 (a reciprocal square root) and scales each pair's viscosity by
// (B_i + B_j) / 2.
//
// sph_params.force_form = 1 swaps the grad-h pressure terms for the sum the
// paper prints as its illustration (Eq. 2): (P_i / rho_i^2 + P_j / rho_j^2)
// times the gradient of particle i's kernel, with no grad-h factor (the
// prologue then stores Phi = P / rho^2).
#include <type_traits>

#include "common.h"
#include "tiles.h"

namespace {

constexpr int BS = 64;     // one wavefront per block (finest LDS allocation)
constexpr int WAVES = BS / 64;
constexpr int FCAP = 128;  // candidates per LDS tile
constexpr int LCAP = 80;   // entries of a particle's list (64 candidates always fit)
constexpr int LSEG = LCAP;  // (20 words: the lists of 16 particles start in different banks)
constexpr int NWORDS = (FCAP + 127) / 128;  // hit words per lane
static_assert(FCAP % 64 == 0 && FCAP <= 256, "whole steps of the filter; byte-sized candidate numbers");

__global__ void k_force_prologue(int64_t n, const uint32_t* __restrict__ perm, const float4* __restrict__ jd,
                                 const float* __restrict__ hs, const float* __restrict__ rhos,
                                 const float* __restrict__ fs, const float* __restrict__ vel,
                                 const float* __restrict__ u, float gamma, int with_f,
                                 float4* __restrict__ jf, int64_t* __restrict__ ctr)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint32_t o = perm[p];
    const float4 x = jd[p];
    const float h = hs[p];
    const float rho = rhos[p];
    const float uu = u[o];
    const float vx = vel[3 * (int64_t)o], vy = vel[3 * (int64_t)o + 1], vz = vel[3 * (int64_t)o + 2];
    if (!(uu >= 0.0f) || !isfinite(uu) || !isfinite(vx) || !isfinite(vy) || !isfinite(vz))
        atomicAdd((unsigned long long*)&ctr_slot(ctr)[CT_BAD_INPUT], 1ull);
    const float P = (gamma - 1.0f) * rho * uu;
    const float c = sqrtf(gamma * (gamma - 1.0f) * uu);
    const float phi = (with_f ? fs[p] : 1.0f) * P / (rho * rho);
    jf[3 * p + 0] = make_float4(x.x, x.y, x.z, h * h);
    jf[3 * p + 1] = make_float4(vx, vy, vz, x.w);
    jf[3 * p + 2] = make_float4(rho, phi, c, 1.0f / h);
}

struct ForceArgs {
    const float4* jf;
    float4* jf_w;             // the same array, written by the divergence pass (B in place of 1/h)
    CellArgs cell;         // the items, their frames and candidates
    const int* cell_item;  // per schedule slot: work item (null: the slot's number)
    const uint32_t* perm;
    float* acc;
    float* dudt;
    double* cons_part;  // 4 per item, may be null
    float* vsig;        // sorted: signal velocity per particle (k_force<true> only)
    float* divv;        // sorted: velocity divergence per particle (k_force<true> only)
    float* bal;         // sorted: Balsara factor per particle (written in the FM_DIVCURL mode)
    int64_t* ctr;
    WorkSched W;
    float alpha;
};

// What a pass of k_force computes: the force; the force with the Balsara
// switch (4 float4 per particle); the Balsara factors (3 float4 per particle,
// no force, no counters); the force in the Eq. 2 form.
enum { FM_FORCE = 0, FM_BALSARA = 1, FM_DIVCURL = 2, FM_EQ2 = 3 };
// With FM_BALSARA the third float4 of a particle holds (rho, Phi, c, B).

// Input-order copy of the sorted Balsara factors.
__global__ void k_unsort_f32(int64_t n, const uint32_t* __restrict__ perm, const float* __restrict__ src,
                             float* __restrict__ dst)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) dst[perm[p]] = src[p];
}

// VSIG: also record each particle's signal velocity max(c_i, max_j (c_i +
// c_j - 3 w_ij)) over its pairs, for the Courant time step, and its velocity
// divergence, rho_i div v_i = -sum_j m_j (v_i - v_j) . grad_i W(r_ij, h_i)
// (the pairs inside h_i; grad_i W = D_i rhat), from which the next step's
// smoothing length is predicted (continuity: dh/dt = h div v / 3).
// UNI: a grid layout.
//
// An item's candidates are staged FCAP at a time, keeping those within the
// item's largest h, or their own, of the box around its particles; the next 64
// are in flight meanwhile. The matrix cores filter the pairs inside max(h_i,
// h_j): two tables, one with each radius, a pair where either sign is set. The
// lanes that hold a particle's hit words write the candidates they name to the
// particle's list in LDS, and the pair loop gives the four lanes of a particle
// every fourth entry: its trip count follows the item's longest list over
// four, where lanes that kept their own candidates' hits waited for the longest
// of 64 short lists.
template <bool VSIG, int MODE, bool UNI>
__global__ void __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(4))) k_force(ForceArgs A)
{
    constexpr bool DC = MODE == FM_DIVCURL;
    __shared__ float4 t0[FCAP];                 // x, y, z, 48 / (pi h^4) (0 in the Balsara mode's stead: h^2)
    __shared__ float4 t1[FCAP];                 // v, m
    __shared__ float4 t2[DC ? 1 : FCAP];        // rho, Phi, c, 1/h
    __shared__ uint2 fa[FCAP];                  // filter input: x, y; z, |x|^2 (half precision)
    __shared__ uint32_t fb[DC ? 1 : FCAP];      // z, |x|^2 - h^2
    __shared__ uint8_t lists[16 * LSEG];  // of the particles: candidate numbers of one tile
    __shared__ float4 scratch4[WALK_LDS<UNI> / 16];
    char* scratch = reinterpret_cast<char*>(scratch4);
    const int lane = threadIdx.x & 63;
    const int pc = lane & 15, gc = lane >> 4;  // column (particle) and lane group of the filter
    const int pq = lane >> 2, sub = lane & 3;  // particle and lane of the pair loop
    const int fin = 4 * (lane & 3) + gc;       // the candidate (of 16) this lane feeds to the filter
    int wstate = 0, a_cur = 0, a_end = 0;
    int64_t cand_acc = 0;  // wave-uniform
    int inter_acc = 0;     // this lane's pairs
    const float K6 = 6.0f * 8.0f / SPH_PI_F;  // w'(q) = 6 (U^2 - t^2), U = max(1 - 2 q, 0), t = max(1 - q, 0)

    for (;;) {
        if (a_cur >= a_end && !next_items(A.W, A.ctr, WAVES, wstate, a_cur, a_end)) break;
        const int slot = __builtin_amdgcn_readfirstlane(a_cur);
        ++a_cur;
        Item<UNI> it;
        CandWalk<UNI> w;
        item_load(it, w, A.cell, slot, scratch);
        const int i0 = it.i0, ni = it.ni;
        // coordinates of a particle's first float4 in the item's frame
        auto frame = [&](float4 v, float3 sh) {
            return make_float4(item_coord<UNI>(v.x, it.ox, it.sh, it.sl, sh.x),
                               item_coord<UNI>(v.y, it.oy, it.sh, it.sl, sh.y),
                               item_coord<UNI>(v.z, it.oz, it.sh, it.sl, sh.z), v.w);
        };
        const float3 none = make_float3(0.f, 0.f, 0.f);
        // the filter's particle
        const bool vc = pc < ni;
        const float4 xc = frame(A.jf[3 * (int64_t)(i0 + min(pc, ni - 1)) + 0], none);
        const float reach = uniform_f(sqrtf(group_max(vc ? xc.w : 0.0f, 16)));
        const float reach2 = cull_reach2(reach);
        const float fs = FILTER_SCALE / (fmaxf(fmaxf(it.hx, it.hy), it.hz) + reach);
        const float fs2 = fs * fs;
        f16x4 fcol;
        f32x4 C1, C2;
        {
            const float ux = (xc.x - it.bx) * fs, uy = (xc.y - it.by) * fs, uz = (xc.z - it.bz) * fs;
            const float n2 = fmaf(ux, ux, fmaf(uy, uy, uz * uz)) * (1.0f - FILTER_EPS) - FILTER_ABS;
            fcol = filter_column(ux, uy, uz);
            const float c1 = vc ? fmaf(xc.w * fs2, -(1.0f + FILTER_EPS), n2) : 1.0e9f, c2 = vc ? n2 : 1.0e9f;
            C1 = {c1, c1, c1, c1};
            C2 = {c2, c2, c2, c2};
        }
        // the pair loop's particle
        const bool valid = pq < ni;
        const int i = i0 + (valid ? pq : 0);
        const float4 i0v = frame(A.jf[3 * (int64_t)i + 0], none);
        const float4 i1v = A.jf[3 * (int64_t)i + 1];
        const float4 i2v = A.jf[3 * (int64_t)i + 2];
        const uint32_t o_i = DC ? 0u : A.perm[i];  // loaded here so the stores wait for nothing
        const float bal_i = MODE == FM_BALSARA ? i2v.w : 1.0f;
        const float hinv_i = MODE == FM_BALSARA ? __builtin_amdgcn_rsqf(i0v.w) : i2v.w;
        const float hinv2_i = hinv_i * hinv_i;
        const float Ki = K6 * hinv2_i * hinv2_i;
        const float rho_i = i2v.x, phi_i = i2v.y, c_i = i2v.z;
        // sums over the pairs (the force: a; s1 = sum m D_i v.rhat, s2 = sum m
        // visc / 2 (D_i + D_j) v.rhat, du/dt = Phi_i s1 + s2 / 2)
        float ax = 0.f, ay = 0.f, az = 0.f, s1 = 0.f, s2 = 0.f;
        float vmax = 0.f;  // (VSIG) largest c_i + c_j - 3 w_ij of this lane's pairs
        const float visc_k = -0.5f * A.alpha;
        int kept = 0;      // candidates kept by the box test

        // the next 64 candidates, in flight
        bool ok = false;
        int src = 0;
        float3 sh = make_float3(0.f, 0.f, 0.f);
        float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f), p1 = p0, p2 = p0;
        auto fetch = [&]() -> bool {
            Slots<1> S;
            if (!walk_next<1>(w, A.cell, it, scratch, S)) return false;
            ok = S.ok[0];
            src = S.src[0];
            sh = S.sh[0];
            p0 = A.jf[3 * (int64_t)src + 0];
            p1 = A.jf[3 * (int64_t)src + 1];
            if (!DC) p2 = A.jf[3 * (int64_t)src + 2];
            return true;
        };
        walk_start(w, A.cell, it, scratch, reach, !DC);
        bool more = fetch();
        while (more) {
            // ---- stage up to FCAP candidates ------------------------------------------
            int nk = 0;
            do {
                const float4 xj = frame(p0, sh);
                const float x = xj.x, y = xj.y, z = xj.z, h2 = xj.w;
                const float ux = UNI ? x : x - it.bx, uy = UNI ? y : y - it.by, uz = UNI ? z : z - it.bz;
                const float gx = fmaxf(fabsf(ux) - it.hx, 0.0f), gy = fmaxf(fabsf(uy) - it.hy, 0.0f),
                            gz = fmaxf(fabsf(uz) - it.hz, 0.0f);
                const bool keep = ok && fmaf(gx, gx, fmaf(gy, gy, gz * gz)) <
                                            (DC ? reach2 : fmaxf(reach2, h2 * 1.00002f));
                const uint64_t m = __ballot(keep);
                if (keep) {
                    const int d = nk + lanes_below(m);
                    float fx = ux * fs, fy = uy * fs, fz = uz * fs;
                    float n1 = fmaf(fx, fx, fmaf(fy, fy, fz * fz)) * (1.0f - FILTER_EPS);
                    const float hs2 = h2 * fs2 * (1.0f + FILTER_EPS);
                    float n2 = n1 - hs2;
                    if (!DC && fmaxf(n1, hs2) > FILTER_FAR) {  // beyond half precision: propose every pair
                        fx = fy = fz = 0.0f;
                        n1 = n2 = -FILTER_FAR;
                    }
                    fa[d] = make_uint2(pack_f16(fx, fy), pack_f16(fz, n1));
                    if constexpr (!DC) {
                        fb[d] = pack_f16(fz, n2);
                        // (the third float4 holds 1/h, or B in the Balsara mode)
                        const float hinv = MODE == FM_BALSARA ? __builtin_amdgcn_rsqf(h2) : p2.w;
                        const float hinv2 = hinv * hinv;
                        t0[d] = make_float4(x, y, z, MODE == FM_BALSARA ? h2 : K6 * hinv2 * hinv2);
                        t2[d] = p2;
                    } else {
                        t0[d] = make_float4(x, y, z, h2);
                    }
                    t1[d] = p1;
                }
                nk += __popcll(m);
                more = fetch();
            } while (more && nk + 64 <= FCAP);
            kept += nk;
            // unused slots up to a multiple of 64
            if (nk + lane < ((nk + 63) & ~63)) {
                fa[nk + lane] = make_uint2(0u, pack_f16(0.0f, FILTER_FAR));
                if constexpr (!DC) fb[nk + lane] = pack_f16(0.0f, FILTER_FAR);
            }
            wave_sync_lds();

            // ---- filter: the lane's hit words --------------------------------------------
            unsigned hit[NWORDS];
#pragma unroll
            for (int k = 0; k < NWORDS; ++k) hit[k] = 0u;
#pragma unroll
            for (int q = 0; q < FCAP / 64; ++q) {
                if (64 * q < nk) {
                    unsigned m = hit[q >> 1];
#pragma unroll
                    for (int b = 4 * q; b < 4 * q + 4; ++b) {
                        const uint2 a = fa[16 * b + fin];
                        f32x4 D = __builtin_amdgcn_mfma_f32_4x4x4f16(f16x4_of(a.x, a.y), fcol, C1, 0, 0, 0);
                        f32x4 E = D;
                        if constexpr (!DC)
                            E = __builtin_amdgcn_mfma_f32_4x4x4f16(f16x4_of(a.x, fb[16 * b + fin]), fcol, C2, 0, 0, 0);
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            m = __builtin_amdgcn_alignbit(m, __float_as_uint(D[r]) | __float_as_uint(E[r]), 31);
                    }
                    hit[q >> 1] = m;
                }
            }

            // ---- the words become lists, and the lists pairs: the whole tile at once, or
            //      (a list would not fit) 64 candidates at a time --------------------------------
            int n_all = 0, tot = 0;
#pragma unroll
            for (int k = 0; k < NWORDS; ++k) n_all += __popc(hit[k]);
            int pre = column_excl_scan(n_all, tot);
            const bool whole = !__any(tot > LCAP);
            for (int part = 0; part < (whole ? 1 : (nk + 63) / 64); ++part) {
                unsigned now[NWORDS];
#pragma unroll
                for (int k = 0; k < NWORDS; ++k) now[k] = whole ? hit[k] : hit_part(hit[k], nk, k, part);
                if (!whole) {
                    int n_part = 0;
#pragma unroll
                    for (int k = 0; k < NWORDS; ++k) n_part += __popc(now[k]);
                    pre = column_excl_scan(n_part, tot);
                }
                uint8_t* lp = lists + pc * LSEG + pre;
#pragma unroll
                for (int k = 0; k < NWORDS; ++k) {
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
                const uint8_t* lst = lists + pq * LSEG;
                // (not unrolled: the lists' lengths differ, and a second copy of
                // the body measured slower)
#pragma unroll 1
                for (int e = sub; e < nl; e += 4) {
                    const int k = lst[e];
                    const float4 q0 = t0[k], q1 = t1[k];
                    const float dx = i0v.x - q0.x, dy = i0v.y - q0.y, dz = i0v.z - q0.z;
                    float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                    // a coincident pair (the particle itself among them) adds nothing: far away
                    r2 = r2 > 0.0f ? r2 : 1.0e30f;
                    const float rinv = __builtin_amdgcn_rsqf(r2);
                    const float r = r2 * rinv;
                    const float r_2 = 2.0f * r;
                    // w'(q) of both kernels as truncated powers: t is 0 from q = 1 on, so a
                    // pair the filter's margin let through adds exactly nothing
                    const float ti = __builtin_amdgcn_fmed3f(fmaf(-r, hinv_i, 1.0f), 0.0f, 1.0f);
                    const float ui = __builtin_amdgcn_fmed3f(fmaf(-r_2, hinv_i, 1.0f), 0.0f, 1.0f);
                    const float Di = Ki * fmaf(ui, ui, -(ti * ti));
                    const float wx = i1v.x - q1.x, wy = i1v.y - q1.y, wz = i1v.z - q1.z;
                    if constexpr (DC) {
                        // rho_i div v_i = -sum m_j D_i (v_i - v_j) . rhat, rho_i curl v_i =
                        // sum m_j D_i (v_i - v_j) x rhat; D_i is 0 from r = h_i on
                        const float mD = q1.w * Di * rinv;
                        s1 = fmaf(mD, fmaf(wx, dx, fmaf(wy, dy, wz * dz)), s1);
                        ax = fmaf(mD, wy * dz - wz * dy, ax);
                        ay = fmaf(mD, wz * dx - wx * dz, ay);
                        az = fmaf(mD, wx * dy - wy * dx, az);
                        continue;
                    }
                    const float4 q2 = t2[DC ? 0 : k];
                    float hinv_j = q2.w, Kj = q0.w;
                    if constexpr (MODE == FM_BALSARA) {
                        hinv_j = __builtin_amdgcn_rsqf(q0.w);
                        const float hinv2_j = hinv_j * hinv_j;
                        Kj = K6 * hinv2_j * hinv2_j;
                    }
                    const float tj = __builtin_amdgcn_fmed3f(fmaf(-r, hinv_j, 1.0f), 0.0f, 1.0f);
                    const float uj = __builtin_amdgcn_fmed3f(fmaf(-r_2, hinv_j, 1.0f), 0.0f, 1.0f);
                    const float Dj = Kj * fmaf(uj, uj, -(tj * tj));
                    const bool in = ti + tj > 0.0f;
                    inter_acc += in ? 1 : 0;
                    const float vr = fmaf(wx, dx, fmaf(wy, dy, wz * dz)) * rinv;
                    const float wv = fminf(vr, 0.0f);
                    const float vsig = fmaf(-3.0f, wv, c_i + q2.z);
                    float v2 = visc_k * (vsig * wv) * __builtin_amdgcn_rcpf(rho_i + q2.x);  // Pi / 2
                    if constexpr (MODE == FM_BALSARA) v2 *= 0.5f * (bal_i + q2.w);
                    if constexpr (VSIG) vmax = fmaxf(vmax, in ? vsig : 0.0f);
                    // G = Phi_i D_i + Phi_j D_j + Pi (D_i + D_j) / 2; Eq. 2: (Phi_i + Phi_j) D_i + Pi (...) / 2
                    const float Ds = Di + Dj;
                    const float G = MODE == FM_EQ2 ? fmaf(phi_i + q2.y, Di, v2 * Ds)
                                                   : fmaf(phi_i + v2, Di, (q2.y + v2) * Dj);
                    const float mGr = q1.w * G * rinv;
                    ax = fmaf(-mGr, dx, ax);
                    ay = fmaf(-mGr, dy, ay);
                    az = fmaf(-mGr, dz, az);
                    const float mvr = q1.w * vr;
                    s1 = fmaf(mvr, Di, s1);
                    s2 = fmaf(mvr * v2, Ds, s2);
                }
                // every lane is done with the lists and the tile
                wave_sync_lds();
            }
            }
        ax = group_sum(ax, 4);
        ay = group_sum(ay, 4);
        az = group_sum(az, 4);
        s1 = group_sum(s1, 4);
        if constexpr (DC) {
            if (valid && sub == 0) {
                const float ad = fabsf(s1) / rho_i;
                const float den = ad + sqrtf(fmaf(ax, ax, fmaf(ay, ay, az * az))) / rho_i + 1.0e-4f * c_i * hinv_i;
                const float B = den > 0.0f ? ad / den : 0.0f;  // no motion and no sound: no viscosity
                A.bal[i] = B;
                // B replaces 1/h in the particle's third float4 for the force
                // pass (the candidates of this pass read only the first two)
                A.jf_w[3 * (int64_t)i + 2] = make_float4(rho_i, phi_i, c_i, B);
            }
            continue;
        }
        const float du = fmaf(phi_i, s1, 0.5f * group_sum(s2, 4));
        if constexpr (VSIG) vmax = group_max(vmax, 4);
        cand_acc += (int64_t)ni * kept;
        if (valid) {
            // the four lanes of a particle store ax, ay, az and du/dt
            float* dst = sub == 3 ? A.dudt + o_i : A.acc + 3 * (int64_t)o_i + sub;
            *dst = sub == 0 ? ax : sub == 1 ? ay : sub == 2 ? az : du;
            if constexpr (VSIG) {
                if (sub == 0) {
                    A.vsig[i] = fmaxf(vmax, c_i);
                    A.divv[i] = -s1 / rho_i;
                }
            }
        }
        if (A.cons_part) {
            // lane `sub` of each particle takes component `sub` of the item's
            // share; then the particles in a fixed order
            const double m = i1v.w;
            double cm = sub == 0   ? m * ax
                        : sub == 1 ? m * ay
                        : sub == 2 ? m * az
                                   : m * ((double)i1v.x * ax + (double)i1v.y * ay + (double)i1v.z * az + (double)du);
            if (!valid) cm = 0.0;
            for (int o = 32; o >= 4; o >>= 1) cm += __shfl_xor(cm, o, 64);
            if (lane < 4) A.cons_part[4 * (int64_t)(A.cell_item ? A.cell_item[slot] : slot) + lane] = cm;
        }
    }
    if constexpr (!DC) {
        ctr_wave_add(A.ctr, CT_FORCE_INTER, inter_acc);
        ctr_add_uniform(A.ctr, CT_FORCE_CAND, cand_acc);  // already a wavefront total
    }
}

// Per-box sums of the items' shares: block b adds the shares of its items
// [box_item[b], box_item[b + 1]) in a fixed order (strided partial sums, then
// a tree in LDS), so the result does not depend on scheduling.
constexpr int CR_BS = 1024;

__global__ void __launch_bounds__(CR_BS) k_cons_reduce(const int* __restrict__ box_item,
                                                       const double* __restrict__ cons_part, double* __restrict__ cons)
{
    __shared__ double red[4][CR_BS];
    const int b = blockIdx.x;
    const int t = threadIdx.x;
    const int l0 = box_item[b], l1 = box_item[b + 1];
    // two partial sums per thread (items t, t + 2 CR_BS, ... and t + CR_BS,
    // t + 3 CR_BS, ...): two loads in flight, one fixed order
    double v[4] = {0.0, 0.0, 0.0, 0.0}, w[4] = {0.0, 0.0, 0.0, 0.0};
    for (int l = l0 + t; l < l1; l += 2 * CR_BS) {
        const bool second = l + CR_BS < l1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] += cons_part[4 * (int64_t)l + k];
            w[k] += second ? cons_part[4 * (int64_t)(l + CR_BS) + k] : 0.0;
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) red[k][t] = v[k] + w[k];
    __syncthreads();
    for (int half = CR_BS / 2; half >= 1; half >>= 1) {
        if (t < half) {
#pragma unroll
            for (int k = 0; k < 4; ++k) red[k][t] += red[k][t + half];
        }
        __syncthreads();
    }
    if (t < 4) cons[4 * (int64_t)b + t] = red[t][0];
}

}  // namespace

namespace sph {

int make_sched(sph_ctx* c, int64_t n_items, int waves_per_block, int blocks_per_cu, WorkSched& W);

void mark_force_outputs(sph_ctx* c)
{
    c->vsig_valid = c->prm.signal_velocity != 0;
    c->div_valid = c->prm.signal_velocity != 0;
    c->bal_valid = c->prm.balsara != 0 && c->prm.alpha_visc > 0;
}

void force_enqueue(sph_ctx* c, const float* vel, const float* u, float* acc, float* dudt, double* cons_d,
                   bool clear_all, bool events, hipStream_t s, bool prologue)
{
    const int64_t n = c->n;
    int64_t* ctr = static_cast<int64_t*>(c->counters.p);
    float4* jf = static_cast<float4*>(c->jf.p);
    // all counters, or (after a density pass whose counters are still to be
    // read) only the work-queue heads, which only the persistent schedule uses
    if (clear_all)
        fill_u32(ctr, 0u, 2 * (int64_t)CT_COUNT, s);
    else if (c->prm.schedule == 1)
        fill_u32(ctr + CT_QUEUE, 0u, 2 * 64, s);
    const bool eq2 = c->prm.force_form == 1;
    if (prologue || eq2) {  // else the density kernels wrote the streams (ghost step fused)
        k_force_prologue<<<blocks_for(n, 256), 256, 0, s>>>(n, static_cast<uint32_t*>(c->perm.p),
                                                             static_cast<float4*>(c->jd.p),
                                                             static_cast<float*>(c->hs.p),
                                                             static_cast<float*>(c->rhos.p),
                                                             static_cast<float*>(c->fs.p), vel, u,
                                                             (float)c->prm.gamma, eq2 ? 0 : 1, jf, ctr);
        SPH_HIP(hipGetLastError());
    }
    ForceArgs A;
    A.jf = jf;
    A.jf_w = jf;
    A.cell = cell_args(c, static_cast<int4*>(c->cells.p));
    A.cell_item = c->uni ? nullptr : static_cast<int*>(c->cell_item.p);
    A.perm = static_cast<uint32_t*>(c->perm.p);
    A.acc = acc;
    A.dudt = dudt;
    A.cons_part = cons_d ? static_cast<double*>(c->cons_part.p) : nullptr;
    const bool vsig = c->prm.signal_velocity != 0;
    A.vsig = vsig ? static_cast<float*>(c->vsig_s.p) : nullptr;
    A.divv = vsig ? static_cast<float*>(c->divv_s.p) : nullptr;
    A.bal = static_cast<float*>(c->bal_s.p);
    A.ctr = ctr;
    const int grid = make_sched(c, c->n_items, WAVES, 16, A.W);
    A.alpha = c->prm.alpha_visc > 0 ? (float)c->prm.alpha_visc : 0.0f;
    if (events) ev_record(c, EV_FORCE_K0, s);
    const bool bal = c->prm.balsara != 0 && A.alpha > 0.0f;
    auto go = [&](auto vs, auto md) {
        constexpr bool V = decltype(vs)::value;
        constexpr int M = decltype(md)::value;
        if (c->uni)
            k_force<V, M, true><<<grid, BS, 0, s>>>(A);
        else
            k_force<V, M, false><<<grid, BS, 0, s>>>(A);
    };
    using T = std::true_type;
    using F = std::false_type;
    if (bal) {
        go(F{}, std::integral_constant<int, FM_DIVCURL>{});
        SPH_HIP(hipGetLastError());
        if (c->prm.schedule == 1) fill_u32(ctr + CT_QUEUE, 0u, 2 * 64, s);  // the force pass pops the queues again
        if (vsig)
            go(T{}, std::integral_constant<int, FM_BALSARA>{});
        else
            go(F{}, std::integral_constant<int, FM_BALSARA>{});
    } else if (eq2) {
        if (vsig)
            go(T{}, std::integral_constant<int, FM_EQ2>{});
        else
            go(F{}, std::integral_constant<int, FM_EQ2>{});
    } else if (vsig) {
        go(T{}, std::integral_constant<int, FM_FORCE>{});
    } else {
        go(F{}, std::integral_constant<int, FM_FORCE>{});
    }
    SPH_HIP(hipGetLastError());
    if (events) ev_record(c, EV_FORCE_K1, s);
    if (cons_d) {
        k_cons_reduce<<<c->n_boxes, CR_BS, 0, s>>>(static_cast<int*>(c->box_item.p), A.cons_part, cons_d);
        SPH_HIP(hipGetLastError());
    }
}

double* force_buffers(sph_ctx* c, bool cons)
{
    SPH_REQUIRE(c->prm.force_form == 0 || c->prm.force_form == 1, SPH_E_ARG, "sph_params.force_form must be 0 or 1");
    SPH_REQUIRE(!(c->prm.force_form == 1 && c->prm.balsara), SPH_E_ARG,
                "the Eq. 2 force form (force_form = 1) has no Balsara switch");
    ensure<float4>(c, c->jf, 3 * c->n);
    if (c->prm.signal_velocity) {
        ensure<float>(c, c->vsig_s, c->n);
        ensure<float>(c, c->divv_s, c->n);
    }
    if (c->prm.balsara) ensure<float>(c, c->bal_s, c->n);
    if (!cons) return nullptr;
    ensure<double>(c, c->cons_part, (size_t)4 * c->n_items);
    return ensure<double>(c, c->cons_d, (size_t)4 * c->n_boxes);
}

void force_f32(sph_ctx* c, const float* vel, const float* u, float* acc, float* dudt, double* cons,
               sph_stats* st, hipStream_t s)
{
    SPH_REQUIRE(c->built && c->density_done, SPH_E_STATE, "sph_force needs a successful sph_density first");
    SPH_REQUIRE(vel && u && acc && dudt, SPH_E_ARG, "null vel/u/acc/dudt");
    double* cons_d = force_buffers(c, cons != nullptr);
    // the sorted signal velocities and Balsara factors are rewritten below:
    // they are valid again only once this pass has succeeded
    c->vsig_valid = c->bal_valid = c->div_valid = false;
    ev_record(c, EV_FORCE_C0, s);
    force_enqueue(c, vel, u, acc, dudt, cons_d, true, true, s);
    if (cons || st) {
        const int64_t* hc = read_counters(c, s, cons_d, cons);
        SPH_REQUIRE(hc[CT_BAD_INPUT] == 0, SPH_E_ARG, "negative or non-finite u, or non-finite velocity");
        if (st) {
            st->interactions_force = hc[CT_FORCE_INTER];
            st->candidates_force = hc[CT_FORCE_CAND];
            st->n_cells = c->n_leaves;
            finish_build_read(c);
            st->n_pairs = c->n_pairs;
        }
    }
    mark_force_outputs(c);
    ev_record(c, EV_FORCE_C1, s);
    if (c->prm.timing) {
        c->tm.force_kernel_ms = ev_ms(c, EV_FORCE_K0, EV_FORCE_K1);
        c->tm.force_call_ms = ev_ms(c, EV_FORCE_C0, EV_FORCE_C1);
    }
}

void balsara_unsort(sph_ctx* c, float* out, hipStream_t s)
{
    SPH_REQUIRE(out, SPH_E_ARG, "null output");
    SPH_REQUIRE(c->built && c->bal_valid, SPH_E_STATE,
                "sph_get_balsara needs a force pass with sph_params.balsara (and viscosity) since the last build or drift");
    if (c->n == 0) return;
    k_unsort_f32<<<blocks_for(c->n, 256), 256, 0, s>>>(c->n, static_cast<uint32_t*>(c->perm.p),
                                                      static_cast<float*>(c->bal_s.p), out);
    SPH_HIP(hipGetLastError());
}

}  // namespace sph
