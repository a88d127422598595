// Adjoint of the derivative sums (sph_forces) with the neighbour lists held
// fixed: the pair loops, for the smoothing kernel SPH_KERNEL_KIND (compiled
// once per kernel, every formulation / laminar term / diffusion instance of
// that kernel in both kernel forms).
//
// Forward pair term of central c and neighbour n (r < 2h), x = x_c - x_n,
// u = u_c - u_n, w = u.x:
//   a_c    += -m_n (S_p + Pi) F x  [+ Lm u]  [+ Lk x]
//   Drho_c += W_c m_n F w           [+ density diffusion]
//   S_p = p_c + p_n (p = P/rho^2), W_c = 1 (golden rule, eq. mass-cont-sph1,
//         eq. ns-sph1) or S_p = (P_c + P_n)/(rho_c rho_n), W_c = rho_c/rho_n
//         (Landrini-Morris, eq. mass-cont-sph2, eq. ns-sph2)
//   Pi = K min(w, 0) / (r^2 + eps h^2),  K = -alpha h (c_c + c_n)/(rho_c + rho_n)
//   Lm = 4 nu m_n F/(rho_c + rho_n)  (Morris),
//   Lk = 4 K' nu m_n F w/((rho_c + rho_n)(r^2 + eps h^2))  (Monaghan's K form)
// (with the readings of the design notes).
//
// Atomic-free gather: the list is symmetric (the float32 predicate gives
// x_ji = -x_ij bit for bit), so particle i visits each partner j once and
// collects both its role as central (upstream abar_i, dbar_i) and its role as
// neighbour of j (upstream abar_j, dbar_j).  With
//   da = m_j abar_i - m_i abar_j,  dA = da.x,  dU = da.u,
//   sD = m_j W_i dbar_i + m_i W_j dbar_j   (W_i = rho_i/rho_j, W_j = rho_j/rho_i, or 1)
// the two roles combine into
//   dL/do_i   += -S F da - dA (S F'/r x + F act K (u/d - 2 w x/d^2)) + sD (F u + w F'/r x)
//                [+ 4 nu F'/(rs r) dU x]  [+ Q da + dA kr ((F'/r w - 2 F w/d) x + F u)]
//   dL/du_i   += -F act K/d dA x + sD F x                       [+ 4 nu F/rs da]  [+ dA kr F x]
//   dL/drho_i += -F (dS_p/drho_i + dPi/drho_i) dA               [- 4 nu F/rs^2 dU]  [- Q dA/rs]
//                [+ w F (dbar_i m_j/rho_j - dbar_j m_i rho_j/rho_i^2)  (Landrini-Morris)]
// with S = S_p + Pi, d = r^2 + eps h^2, rs = rho_i + rho_j, act = (w < 0),
// kr = 4 K' nu/(rs d), Q = kr F w.
// Parameter derivatives are taken from the central role only:
//   dL/dalpha += abar_i.x (-m_j F) Pi/alpha,  dL/dc0 += abar_i.x (-m_j F)(2 S_p + Pi)/c0,
//   dL/dnu    += abar_i.u 4 m_j F/rs  or  abar_i.x 4 K' m_j F w/(rs d).
#include <hip/hip_runtime.h>
#include <math.h>

#include "backward_common.h"
#include "brick_items.h"

#ifndef SPH_KERNEL_KIND
#error "compile with SPH_KERNEL_KIND set to one of the SPH_KERNEL_* values"
#endif

using namespace sph;

namespace {

constexpr int kThreads = 256;

struct BackAcc {
    float ox, oy, oz, ux, uy, uz, r;
    float galpha, gc0, gnu;
};

// aux: xi = (p or P, c, dp/drho or dP/drho, dc/drho) of the central; xj = (p
// or P, c) of the neighbour.  pair_fluid: both are fluid (density diffusion).
// in: 1 inside the list, 0 past its end.
// MASKED: a pair outside the support or past the list has F and F'/r set to
// zero and is accumulated anyway (every term is a finite factor times one of
// them, so it adds +-0; the LDS loop only stages real particles, so every
// factor is finite); otherwise a branch skips it.  The LDS loop takes the
// masked form except with density diffusion, whose longer pair body spills
// when it runs for every slot.  For the Wendland kernel the mask is the clamp
// to [0, 1] of t = in - r/(2h), which is 1 - q/2 inside the list: F = -8 c t^3
// and F'/r = (12 c t^2/h)/r vanish with it.
template <int MODEL, bool MASKED>
__device__ __forceinline__ void pair_adjoint_core(BackAcc &G, float xx, float xy, float xz, float mi,
                                                  const float4 &vi, const float4 &xi, const float4 &gi, float mj,
                                                  const float4 &vj, const float2 &xj, const float4 &gj, float in,
                                                  bool pair_fluid, const BackConst &C)
{
    constexpr int KER = model_kernel(MODEL);
    // (the Wendland masked form has no decision on r^2: fused, and kept off
    // zero, so that a slot past the list that holds the central itself gives
    // zeros and not 0 x inf; the others round it as the list predicate does)
    constexpr bool CLAMPED = MASKED && KER == SPH_KERNEL_WENDLAND;
    float r2;
    if constexpr (CLAMPED) {
        r2 = fmaxf(fmaf(xx, xx, fmaf(xy, xy, xz * xz)), 1e-30f);
    } else {
#pragma clang fp contract(off)
        r2 = (xx * xx + xy * xy) + xz * xz;
    }
    bool inter = in > 0.0f && r2 < C.lim2;
    if constexpr (KER == SPH_KERNEL_QUADRATIC) inter = inter && r2 > 0.0f;  // its F is unbounded at r = 0
    // 1/r from one reciprocal square root, r = r^2/r
    const float inv_r = __builtin_amdgcn_rsqf(r2);
    const float r = r2 * inv_r;
    float F, Fp_r;  // F and F'(r)/r
    if constexpr (CLAMPED) {
        const float t = __builtin_amdgcn_fmed3f(fmaf(r, C.neg_inv_2h, in), 0.0f, 1.0f), t2 = t * t;
        F = t2 * (t * C.minus_8c);
        Fp_r = (t2 * C.c12_h) * inv_r;  // (12 c/h times 1e15 may exceed float32: the mask comes first)
    } else {
        kernel_F_dF<KER>(C.fcoeff, r, r2, inv_r, C.inv_h, C.inv_h2, F, Fp_r);
        if (MASKED) {
            F = inter ? F : 0.0f;
            Fp_r = inter ? Fp_r : 0.0f;
        }
    }
    const float ux = vi.x - vj.x, uy = vi.y - vj.y, uz = vi.z - vj.z;
    const float w = fmaf(ux, xx, fmaf(uy, xy, uz * xz));
    const float rs = vi.w + vj.w;
    const float dd = r2 + C.eps_h2;
    // 1/rs and 1/d from one reciprocal (a quarter-rate operation) of their
    // product (rs d >= 2 rho eps h^2, far from the float range's ends)
    const float inv_rsd = __builtin_amdgcn_rcpf(rs * dd);
    const float inv_rs = dd * inv_rsd;
    const float inv_d = rs * inv_rsd;
    const float csum = xi.y + xj.y;
    // Pi = -alpha h min(w, 0)/d (c_i + c_j)/rs = -alpha h (m/d) B with m =
    // min(w, 0) (zero for w >= 0, and so are Pi and its derivatives) and B =
    // csum/rs; act/d: 1/d for w < 0, else 0
    const float act_d = w < 0.0f ? inv_d : 0.0f;
    const float mwd = w * act_d;
    const float B = csum * inv_rs;
    const float mB = mwd * B;
    const float Pi = -C.alpha_h * mB;
    // dPi/drho_i = -alpha h (m/d) (dc_i/drho_i - B)/rs
    const float dPi_dri = -C.alpha_h * mwd * (xi.w - B) * inv_rs;
    // 1/(rho_i rho_j), 1/rho_i and 1/rho_j from one reciprocal (Landrini-Morris;
    // the density diffusion alone takes them in its branch)
    [[maybe_unused]] float inv_rr = 0.0f, iri = 0.0f, irj = 0.0f;
    if constexpr (MODEL & kLandrini) {
        inv_rr = __builtin_amdgcn_rcpf(vi.w * vj.w);
        iri = vj.w * inv_rr;
        irj = vi.w * inv_rr;
    }
    // pressure factor S_p and dS_p/drho_i
    float Sp, dSp;
    if constexpr (MODEL & kLandrini) {
        Sp = (xi.x + xj.x) * inv_rr;
        dSp = (xi.z - Sp * vj.w) * inv_rr;  // (c_i^2 - S_p rho_j)/(rho_i rho_j)
    } else {
        Sp = xi.x + xj.x;
        dSp = xi.z;
    }
    const float S = Sp + Pi;
    // combined upstream of the two roles
    const float dax = mj * gi.x - mi * gj.x;
    const float day = mj * gi.y - mi * gj.y;
    const float daz = mj * gi.z - mi * gj.z;
    const float dA = fmaf(dax, xx, fmaf(day, xy, daz * xz));
    float sD;
    [[maybe_unused]] float inv_ri = 0.0f, inv_rj = 0.0f, wj = 0.0f;
    if constexpr (MODEL & kLandrini) {
        inv_ri = iri;
        inv_rj = irj;
        wj = vj.w * inv_ri;
        sD = fmaf(mj * gi.w, vi.w * inv_rj, mi * gj.w * wj);
    } else {
        sD = fmaf(mj, gi.w, mi * gj.w);
    }
    // d/do_i = ka da + kx x + ku u, d/du_i = ku x (+ the laminar terms)
    const float t = w * inv_d;
    const float cu = F * (-C.alpha_h * B * act_d);
    const float cx = fmaf(-2.0f * t, cu, S * Fp_r);  // S F'/r - 2 F act K w/d^2
    float kx = fmaf(-dA, cx, sD * w * Fp_r);
    float ku = fmaf(-dA, cu, sD * F);
    float ka = -S * F;
    [[maybe_unused]] float kr = 0.0f, Q = 0.0f, duu = 0.0f;
    if constexpr (model_visc(MODEL) == kMonaghanK) {
        kr = C.k_four_nu * inv_rs * inv_d;
        Q = kr * F * w;
        ka += Q;
        kx = fmaf(dA * kr, fmaf(Fp_r, w, -2.0f * F * t), kx);
        ku = fmaf(dA * kr, F, ku);
    }
    if constexpr (model_visc(MODEL) == kMorris) {
        duu = fmaf(dax, ux, fmaf(day, uy, daz * uz));
        kx = fmaf(C.four_nu * Fp_r * inv_rs, duu, kx);
    }
    // d/drho_i
    float gr = F * (dSp + dPi_dri) * -dA;
    if constexpr (model_visc(MODEL) == kMorris) gr = fmaf(-C.four_nu * F * inv_rs * inv_rs, duu, gr);
    if constexpr (model_visc(MODEL) == kMonaghanK) gr = fmaf(-Q * inv_rs, dA, gr);
    if constexpr (MODEL & kLandrini) gr = fmaf(w * F, fmaf(gi.w * mj, inv_rj, -gj.w * mi * wj * inv_ri), gr);
    // parameters (central role)
    const float AmF = fmaf(gi.x, xx, fmaf(gi.y, xy, gi.z * xz)) * (-mj * F);
    const float ga = AmF * mB;                 // (times -h: scale_parameters)
    float gc = AmF * fmaf(2.0f, Sp, Pi);       // (times 1/c0)
    float gn = 0.0f;
    if constexpr (model_visc(MODEL) == kMorris) gn = fmaf(gi.x, ux, fmaf(gi.y, uy, gi.z * uz)) * 4.0f * mj * F * inv_rs;
    if constexpr (model_visc(MODEL) == kMonaghanK)
        gn = fmaf(gi.x, xx, fmaf(gi.y, xy, gi.z * xz)) * (4.0f * kMonaghanKFactor) * mj * F * w * inv_rs * inv_d;
    if constexpr (MODEL & kDiffusion) {
        // density diffusion, term_ij = c m_j (rho_i - rho_j)/rho_j Gd(r) with
        // Gd = F r^2/(r^2 + eps h^2), c = 2 delta h c0; both roles combined:
        //   do_i   += c Gd'/r (rho_i - rho_j)(dbar_i m_j/rho_j - dbar_j m_i/rho_i) x
        //   drho_i += c Gd (dbar_i m_j/rho_j - dbar_j m_i rho_j/rho_i^2)
        //   dc0    += dbar_i term_ij / c0   (central role)
        if (pair_fluid) {
            if constexpr (!(MODEL & kLandrini)) {
                inv_rr = __builtin_amdgcn_rcpf(vi.w * vj.w);
                iri = vj.w * inv_rr;
                irj = vi.w * inv_rr;
            }
            const float Gd = F * r2 * inv_d;
            const float Gd_r = Fp_r * r2 * inv_d + 2.0f * F * C.eps_h2 * inv_d * inv_d;
            const float w1 = gi.w * mj * irj, w2 = gj.w * mi * iri;
            const float dr = vi.w - vj.w;
            kx = fmaf(C.diff * Gd_r * dr, w1 - w2, kx);
            gr = fmaf(C.diff * Gd, w1 - w2 * vj.w * iri, gr);
            gc = fmaf(w1 * C.diff * dr, Gd, gc);
        }
    }
    if (MASKED || inter) {
        G.ox = fmaf(ka, dax, fmaf(kx, xx, fmaf(ku, ux, G.ox)));
        G.oy = fmaf(ka, day, fmaf(kx, xy, fmaf(ku, uy, G.oy)));
        G.oz = fmaf(ka, daz, fmaf(kx, xz, fmaf(ku, uz, G.oz)));
        G.ux = fmaf(ku, xx, G.ux);
        G.uy = fmaf(ku, xy, G.uy);
        G.uz = fmaf(ku, xz, G.uz);
        if constexpr (model_visc(MODEL) == kMorris) {
            const float la = C.four_nu * F * inv_rs;
            G.ux = fmaf(la, dax, G.ux);
            G.uy = fmaf(la, day, G.uy);
            G.uz = fmaf(la, daz, G.uz);
        }
        G.r += gr;
        G.galpha += ga;
        G.gc0 += gc;
        G.gnu += gn;
    }
}

// The common factors of the parameter sums, applied once per central.
__device__ __forceinline__ void scale_parameters(BackAcc &G, const BackConst &C)
{
    G.galpha *= -C.h;
    G.gc0 *= C.inv_c0;
}

template <int MODEL>
__device__ __forceinline__ void pair_adjoint(BackAcc &G, uint32_t e, const float4 &pi, const float4 &vi,
                                             const float4 &xi, const float4 &gi, const float4 &pj,
                                             const float4 &vj, const float4 &xj, const float4 &gj, bool valid,
                                             bool pair_fluid, const BackConst &C)
{
    const float xx = fmaf(entry_k(e, 0), C.csx, pi.x - pj.x);
    const float xy = fmaf(entry_k(e, 1), C.csy, pi.y - pj.y);
    const float xz = fmaf(entry_k(e, 2), C.csz, pi.z - pj.z);
    pair_adjoint_core<MODEL, false>(G, xx, xy, xz, pi.w, vi, xi, gi, pj.w, vj, make_float2(xj.x, xj.y), gj,
                                       valid ? 1.0f : 0.0f, pair_fluid, C);
}

template <int MODEL>
__global__ __launch_bounds__(kThreads) void k_forces_backward(
    int n, const float4 *__restrict__ pos, const float4 *__restrict__ vel, const float4 *__restrict__ aux,
    const float4 *__restrict__ gforce, const uint32_t *__restrict__ neibs, const uint32_t *__restrict__ count,
    const uint32_t *__restrict__ info, float4 *__restrict__ gpos, float4 *__restrict__ gvel,
    double *__restrict__ partial, int accumulate, BackConst C)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x % kWave;
    const int ii = min(i, n - 1);
    const int M = C.max_neibs;
    const uint32_t cnt = i < n ? count[i] : 0u;
    const int nf = min((int)(cnt & 0xFFFFu), M);
    const int nt = min(nf + (int)(cnt >> 16), M);
    const int last = max(nt - 1, 0);
    const int ntw = __builtin_amdgcn_readfirstlane(wave_max(nt));
    const uint32_t jmax = (uint32_t)(n - 1);
    BackAcc G = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (ntw > 0) {
        const int tile_id = __builtin_amdgcn_readfirstlane(i / kWave);
        const uint32_t *tile = neibs + (size_t)tile_id * (kWave * M);
        const float4 pi = pos[ii], vi = vel[ii], xi = aux[ii], gi = gforce[ii];
        const bool central_fluid = (MODEL & kDiffusion) ? ptype(info[ii]) != kBoundary : true;
        uint32_t eA = tile[list_slot(0, nf, last, M) * kWave + lane];
        uint32_t eNext = tile[list_slot(1, nf, last, M) * kWave + lane];
        uint32_t jA = min(eA & kIndexMask, jmax);
        float4 pA = pos[jA], vA = vel[jA], xA = aux[jA], gA = gforce[jA];
        for (int k = 0; k < ntw; k += 2) {
            const uint32_t eN2 = tile[list_slot(k + 2, nf, last, M) * kWave + lane];
            const uint32_t eB = eNext;
            const uint32_t jB = min(eB & kIndexMask, jmax);
            const float4 pB = pos[jB], vB = vel[jB], xB = aux[jB], gB = gforce[jB];
            pair_adjoint<MODEL>(G, eA, pi, vi, xi, gi, pA, vA, xA, gA, k < nt, central_fluid && k < nf, C);
            eNext = tile[list_slot(k + 3, nf, last, M) * kWave + lane];
            eA = eN2;
            jA = min(eA & kIndexMask, jmax);
            pA = pos[jA];
            vA = vel[jA];
            xA = aux[jA];
            gA = gforce[jA];
            pair_adjoint<MODEL>(G, eB, pi, vi, xi, gi, pB, vB, xB, gB, k + 1 < nt, central_fluid && k + 1 < nf,
                               C);
        }
    }
    if (i < n) {
        float4 po = make_float4(G.ox, G.oy, G.oz, 0.0f);
        float4 vo = make_float4(G.ux, G.uy, G.uz, G.r);
        if (nt == 0) po = vo = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (accumulate) {
            const float4 p0 = gpos[i], v0 = gvel[i];
            po = make_float4(p0.x + po.x, p0.y + po.y, p0.z + po.z, p0.w);
            vo = make_float4(v0.x + vo.x, v0.y + vo.y, v0.z + vo.z, v0.w + vo.w);
        } else {
            po.w = gpos[i].w;
        }
        gpos[i] = po;
        gvel[i] = vo;
    }
    // parameter derivatives: per-block partial sums in double, fixed order
    scale_parameters(G, C);
    double a = nt > 0 ? (double)G.galpha : 0.0, c = nt > 0 ? (double)G.gc0 : 0.0,
           v = nt > 0 ? (double)G.gnu : 0.0;
    if (i >= n) a = c = v = 0.0;
    a = wave_sum(a);
    c = wave_sum(c);
    v = wave_sum(v);
    __shared__ double red[3][kThreads / kWave];
    const int w = threadIdx.x / kWave;
    if (lane == 0) {
        red[0][w] = a;
        red[1][w] = c;
        red[2][w] = v;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double s = 0.0;
        for (int k = 0; k < kThreads / kWave; ++k) s += red[threadIdx.x][k];
        partial[3 * (size_t)blockIdx.x + threadIdx.x] = s;
    }
}

// ---------------------------------------------------------------------------
// Cell-brick form of the adjoint (the cell perspective of section "Changing
// perspective: from the particle to the cell", as in sph_forces).  The work
// items are those of the derivative kernel (brick_items.h); per staged
// particle 56 bytes go to LDS (brick-relative position and mass, velocity and
// density, P/rho^2 and c, the upstream adjoint), which holds the halo of half
// a 3 x 4 x 3 brick at the lattice density, so its items are halves.  A run
// that does not fit even as a single row reads the global lists and arrays as
// k_forces_backward does.  The sums per pair are those of k_forces_backward;
// the separation is taken from brick-relative positions (rounding differs from
// the gather kernel at the ulp level).
//
// What bounds it is VALU issue: 92 instructions per pair (99 before the masks
// went into the clamp, r^2 was fused and the parameter sums' common factors
// left the loop), four lanes per central.  1.62M-particle dam break 382 -> 305
// us, the 169k one with Morris viscosity 90 -> 51 us (its 120 bricks were one
// item each, two halves one after the other).
#ifndef SPH_BACK_RING
#define SPH_BACK_RING 2
#endif
constexpr int kBackThreads = 1024;
constexpr int kBackCap = 2624;
constexpr int kBackPairTime = 86;  // of a whole brick, in half microseconds (brick_split)

// The staged arrays of a run.
template <int CAP>
struct StagedBack {
    float4 P[CAP];  // brick-relative offset, mass
    float4 V[CAP];  // velocity, density
    float4 G[CAP];  // upstream adjoint
    float2 X[CAP];  // equation-of-state terms
};

// Pairs of one central's brick-local list, read from LDS, shared by kLanes
// lanes as in the derivative kernel (which says why the two runs of entries
// take turns).
template <int MODEL, int CAP>
__device__ __forceinline__ void brick_adjoint_lds(BackAcc &G, const uint4 *lg, Entries ea, Entries eb, int h, int nt,
                                                  uint32_t lo2, uint32_t max2, const StagedBack<CAP> &L,
                                                  const float4 &pi, const float4 &vi, const float4 &xi,
                                                  const float4 &gi, const BackConst &C)
{
    // pairs of staged data in flight; one for the longest pair bodies
    // (Landrini-Morris with density diffusion and a laminar term), which
    // would otherwise exceed the 128 registers of a 1024-lane workgroup
    constexpr bool kHeaviest = (MODEL & kLandrini) && (MODEL & kDiffusion) && model_visc(MODEL) != 0;
    constexpr int R = kHeaviest ? 1 : SPH_BACK_RING;
    const int runs = (nt + kEntries - 1) / kEntries;
    const uint32_t baseP = lds_address(L.P), baseG = lds_address(L.G), baseX = lds_address(L.X);
    float4 P[R], V[R], Gj[R];
    float2 X[R];
    auto fetch = [&](const Entries &e, int s) {
        const uint32_t w = staged_slots(e[s >> 1], lo2, max2), a = slot_address(w, s & 1, 16, baseP);
        const int r = s % R;
        P[r] = lds_float4(a, 0);
        V[r] = lds_float4(a, CAP);
        Gj[r] = lds_float4(slot_address(w, s & 1, 16, baseG), 0);
        X[r] = lds_float2(slot_address(w, s & 1, 8, baseX));
    };
#pragma unroll
    for (int s = 0; s < R; ++s) fetch(ea, s);
    float rem = (float)(nt - h * kEntries);  // entries of the list from this lane's run on
    int g = h;
    auto run = [&](Entries &e, const Entries &f) {
#pragma unroll
        for (int s = 0; s < kEntries; ++s) {
            const int r = s % R, s2 = s + R;
            // staged w = +-m_j, negative for boundary particles
            pair_adjoint_core<MODEL, !(MODEL & kDiffusion)>(
                G, pi.x - P[r].x, pi.y - P[r].y, pi.z - P[r].z, fabsf(pi.w), vi, xi, gi, fabsf(P[r].w), V[r], X[r],
                Gj[r], __builtin_amdgcn_fmed3f(rem - (float)s, 0.0f, 1.0f), pi.w > 0.0f && P[r].w > 0.0f, C);
            if (s2 < kEntries)
                fetch(e, s2);
            else
                fetch(f, s2 - kEntries);
            if (s2 == kEntries - 1) e = list_entries(lg, min(g + 2 * kLanes, runs - 1));
        }
        g += kLanes;
        rem -= (float)(kLanes * kEntries);
    };
    while (g < runs) {
        run(ea, eb);
        if (g >= runs) break;
        run(eb, ea);
    }
}

// One particle of a staged row on its way to LDS.
struct BackChunk {
    float4 p, v, g;
    int cx;  // cell along x from the brick's centre cell
    uint32_t info;
};
template <int MODEL, typename Rows, typename Scans>
__device__ __forceinline__ BackChunk load_chunk(const Rows &rows, const Scans &B, int k, int t,
                                                const float4 *__restrict__ pos, const float4 *__restrict__ vel,
                                                const float4 *__restrict__ gforce, const uint32_t *__restrict__ info)
{
    BackChunk q;
    const int j = rows.particle(B, k, t, q.cx);
    q.p = load_at(pos, j);
    q.v = load_at(vel, j);
    q.g = load_at(gforce, j);
    q.info = (MODEL & kDiffusion) ? load_at(info, j) : 0u;
    return q;
}
template <int MODEL, typename Rows, int CAP>
__device__ __forceinline__ void store_chunk(StagedBack<CAP> &L, const Rows &rows, const BackChunk &q, int k, int t,
                                            const BackConst &C)
{
    if (t >= rows.len[k]) return;
    const int l = rows.slot[k] + t;
    // mass negated for boundary particles when the diffusion needs the type
    L.P[l] = rows.brick_relative(q.p, k, q.cx, C.csx, C.csy, C.csz,
                                 (MODEL & kDiffusion) && ptype(q.info) == kBoundary ? -q.p.w : q.p.w);
    L.V[l] = q.v;
    L.G[l] = q.g;
    // equation-of-state terms (P/rho^2 or P, c) from the staged density
    const float4 x = eos_grad_terms(q.v.w, C);
    L.X[l] = make_float2(x.x, x.y);
}

// Output of one particle's adjoint by two lanes, h = 0 the position's and h =
// 1 the velocity's and density's (overwrite or accumulate; grad_pos.w is left
// as it is).
__device__ __forceinline__ void store_adjoint(int i, int h, const BackAcc &A, float4 *__restrict__ gpos,
                                              float4 *__restrict__ gvel, int accumulate)
{
    if (h == 0) {
        const float4 p = load_at(gpos, i);
        store_at(gpos, i, accumulate ? make_float4(p.x + A.ox, p.y + A.oy, p.z + A.oz, p.w)
                                     : make_float4(A.ox, A.oy, A.oz, p.w));
    } else if (h == 1) {
        float4 v = make_float4(A.ux, A.uy, A.uz, A.r);
        if (accumulate) {
            const float4 v0 = load_at(gvel, i);
            v = make_float4(v0.x + v.x, v0.y + v.y, v0.z + v.z, v0.w + v.w);
        }
        store_at(gvel, i, v);
    }
}

// One resident workgroup per CU takes the items; the order of their stages is
// that of k_forces_brick.  The parameter derivatives are summed in double in a
// fixed order: over the centrals of a group by its wave, over the groups of an
// item, over the items in the order of the build's table.
template <int MODEL, int BX, int BY, int BZ, int NT, int NC, int CAP>
__global__ __launch_bounds__(NT) void k_forces_backward_brick(
    int n, const float4 *__restrict__ pos, const float4 *__restrict__ vel,
    const float4 *__restrict__ gforce, const uint32_t *__restrict__ neibs, const uint16_t *__restrict__ neibs_brick,
    const uint32_t *__restrict__ count, const int32_t *__restrict__ cell_start, const int32_t *__restrict__ cell_end,
    const int32_t *__restrict__ table, int cap_ids, int32_t *__restrict__ next,
    const uint32_t *__restrict__ info,
    float4 *__restrict__ gpos, float4 *__restrict__ gvel, double *__restrict__ partial,
    double *__restrict__ grad_params, int accumulate, BackConst C, BrickGrid G)
{
    constexpr int NW = NT / kWave, LEAST = BY == 4 ? 2 : 1;
    // a wave takes QG consecutive centrals of the table at a time
    constexpr int QG = kWave / kLanes, MAXG = NC / QG;
    static_assert(MAXG == kWave, "one lane per group in the sum over groups");
    __shared__ StagedBack<CAP> L;
    __shared__ BrickScans<BX, BY, BZ> Q[3];  // this item's, the next one's and the one after
    __shared__ CentralTable<NC, NT, false> T[2];        // this item's and the next one's
    __shared__ double par[3][MAXG];          // parameter sums of each group
    __shared__ double red[3][NW];
    __shared__ int sGroup;  // groups of centrals claimed in the item
    __shared__ int sLast;
    using Rows = StagedRows<BX, BY, BZ, NW>;
    constexpr int SUB = 2;        // chunks of kWave particles of a row carried to the next item
    constexpr int PREP = NW - 1;  // the wave that prepares items
    const int M = C.max_neibs;
    BackChunk chunk[Rows::ROWS][SUB];
    auto load_chunks = [&](const BrickScans<BX, BY, BZ> &N, int wave, int lane) {
        // (always loads, so that no chunk is kept from one item to the next)
        Rows rows;
        rows.locate(N, wave);
#pragma unroll
        for (int k = 0; k < Rows::ROWS; ++k)
#pragma unroll
            for (int u = 0; u < SUB; ++u)
                chunk[k][u] = load_chunk<MODEL>(rows, N, k, u * kWave + lane, pos, vel, gforce, info);
    };
    // The first item (prepared, staging loads under way, table made) and the
    // second (prepared).  Meanwhile particles with an empty list (in no table
    // of centrals; also those the build dropped) get a zero adjoint when the
    // call overwrites (grad_pos.w is kept): no other lane writes them.
    {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
        if (threadIdx.x == 0) Q[2].d = BrickItem{};
        __syncthreads();
        if (wave == PREP)
            prepare_item<BX, BY, BZ, NC, CAP, kBackPairTime, LEAST>(Q[0], Q[2].d, true, lane, table, cap_ids, next,
                                                                    cell_start, cell_end, G);
        else if (!accumulate)
            for (int i = blockIdx.x * (PREP * kWave) + threadIdx.x; i < n; i += gridDim.x * (PREP * kWave))
                if (count[i] == 0u) {
                    gpos[i] = make_float4(0.0f, 0.0f, 0.0f, gpos[i].w);
                    gvel[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
        __syncthreads();
        TableMaker<BX, BY, BZ, NC, NT, false> maker;
        maker.request(Q[0], wave, lane, count);
        load_chunks(Q[0], wave, lane);
        maker.tally(T[0], wave, lane, M);
        __syncthreads();
        maker.place(T[0], wave, lane);
        if (wave == PREP)
            prepare_item<BX, BY, BZ, NC, CAP, kBackPairTime, LEAST>(Q[1], Q[0].d, false, lane, table, cap_ids, next,
                                                                    cell_start, cell_end, G);
        __syncthreads();
    }
    int cur = 0;
    double item_sum = 0.0;  // (waves 0 .. 2) over the runs of the current item
    for (int k = 0;; ++k) {
        const int nxt = cur == 2 ? 0 : cur + 1, far = nxt == 2 ? 0 : nxt + 1;
        // the thread index is re-read per item (an empty asm hides that it is
        // the same), so nothing derived from it is kept live across the pair loop
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
        const BrickScans<BX, BY, BZ> &B = Q[cur];
        const CentralTable<NC, NT, false> &D = T[k & 1];
        CentralTable<NC, NT, false> &DN = T[(k & 1) ^ 1];
        if (__builtin_amdgcn_readfirstlane(B.d.item) < 0) break;
        const int s_lo = __builtin_amdgcn_readfirstlane(B.d.s_lo), span = __builtin_amdgcn_readfirstlane(B.d.span);
        const bool use_lds = __builtin_amdgcn_readfirstlane(B.d.lds) != 0;
        const int nc = __builtin_amdgcn_readfirstlane(use_lds ? D.used : B.d.nc);
        TableMaker<BX, BY, BZ, NC, NT, false> maker;
        maker.request(Q[nxt], wave, lane, count);
        const int h = lane % kLanes;
        const uint32_t lo2 = (uint32_t)s_lo * 0x10001u, max2 = (uint32_t)(span - 1) * 0x10001u;
        int g = wave;
        if (tid == 0) sGroup = NW;  // read after the staging barrier
        if (tid < 3 * MAXG) (&par[0][0])[tid] = 0.0;
        if (use_lds) {
            // the item's particles into LDS: the chunks requested at the end of
            // the last item, then what is left of rows longer than those
            Rows rows;
            rows.locate(B, wave);
#pragma unroll
            for (int r = 0; r < Rows::ROWS; ++r)
#pragma unroll
                for (int u = 0; u < SUB; ++u) store_chunk<MODEL>(L, rows, chunk[r][u], r, u * kWave + lane, C);
#pragma unroll
            for (int r = 0; r < Rows::ROWS; ++r)
                for (int t = SUB * kWave + lane; t - lane < rows.len[r]; t += kWave)
                    store_chunk<MODEL>(L, rows, load_chunk<MODEL>(rows, B, r, t, pos, vel, gforce, info), r, t, C);
        }
        maker.tally(DN, wave, lane, M);
        __syncthreads();
        if (wave == PREP) {
            // (few instructions in a long chain of latencies: it goes first)
            __builtin_amdgcn_s_setprio(3);
            prepare_item<BX, BY, BZ, NC, CAP, kBackPairTime, LEAST>(Q[far], Q[nxt].d, false, lane, table, cap_ids,
                                                                    next, cell_start, cell_end, G);
            __builtin_amdgcn_s_setprio(0);
        }
        while (g * QG < nc) {  // wave-uniform
            const int q = g * QG + lane / kLanes;
            BackAcc A = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            int i, nt;
            if (use_lds) {
                const uint32_t e = D.entry(min(q, nc - 1));
                const int si = (int)(e & kCenSlotMask);
                nt = q < nc ? (int)(e >> kCenCountShift) : 0;
                i = min(si + B.row_shift[e >> kCenRowShift & 15u], n - 1);
                if (nt > 0) {
                    const uint4 *lg = list_groups(neibs_brick, i, brick_groups(M));
                    const int last = (nt - 1) / kEntries;
                    const Entries ea = list_entries(lg, min(h, last)), eb = list_entries(lg, min(h + kLanes, last));
                    const float4 vi = L.V[si];
                    brick_adjoint_lds<MODEL, CAP>(A, lg, ea, eb, h, nt, lo2, max2, L, L.P[si], vi,
                                                  eos_grad_terms(vi.w, C), L.G[si], C);
                }
            } else {
                // more particles than LDS holds: the global lists and arrays, the
                // lanes of a central taking every kLanes-th entry
                i = item_central(B, min(q, nc - 1));
                const uint32_t cw = q < nc ? count[i] : 0u;
                const int nf = min((int)(cw & 0xFFFFu), M);
                nt = min(nf + (int)(cw >> 16), M);
                const int ntw = __builtin_amdgcn_readfirstlane(wave_max(nt));
                const uint32_t *tile = neibs + (size_t)(i / kWave) * (kWave * M) + (i % kWave);
                const float4 pi = pos[i], vi = vel[i], gi = gforce[i];
                const float4 xi = eos_grad_terms(vi.w, C);
                const bool central_fluid = (MODEL & kDiffusion) ? ptype(info[i]) != kBoundary : true;
                const int last = max(nt - 1, 0);
                for (int t = h; t < ntw; t += kLanes) {
                    const uint32_t e = tile[list_slot(t, nf, last, M) * kWave];
                    const uint32_t j = min(e & kIndexMask, (uint32_t)(n - 1));
                    const float4 vj = vel[j];
                    pair_adjoint<MODEL>(A, e, pi, vi, xi, gi, pos[j], vj, eos_grad_terms(vj.w, C), gforce[j], t < nt,
                                        central_fluid && t < nf, C);
                }
                if (nt == 0) A = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            }
            A.ox = lanes_sum(A.ox);
            A.oy = lanes_sum(A.oy);
            A.oz = lanes_sum(A.oz);
            A.ux = lanes_sum(A.ux);
            A.uy = lanes_sum(A.uy);
            A.uz = lanes_sum(A.uz);
            A.r = lanes_sum(A.r);
            A.galpha = lanes_sum(A.galpha);
            A.gc0 = lanes_sum(A.gc0);
            A.gnu = lanes_sum(A.gnu);
            if (nt > 0) store_adjoint(i, h, A, gpos, gvel, accumulate);
            scale_parameters(A, C);
            // parameter sums: lane h of every central takes one of the three,
            // summed in double over the wave's centrals
            double s = (double)(h == 0 ? A.galpha : h == 1 ? A.gc0 : A.gnu);
#pragma unroll
            for (int o = kLanes; o < kWave; o <<= 1) s += __shfl_xor(s, o);
            if (use_lds) {
                if (lane < 3) par[lane][g] = s;
                int c = 0;
                if (lane == 0) c = atomicAdd(&sGroup, 1);
                g = __builtin_amdgcn_readfirstlane(c);
            } else {
                // (such an item may have more groups than slots: dealt to the
                // waves in turn, each adds up its own)
                if (lane < 3) par[lane][wave] += s;
                g += NW;
            }
        }
        // (in the time that waves without a group wait for the others)
        maker.place(DN, wave, lane);
        load_chunks(Q[nxt], wave, lane);
        __syncthreads();  // the next item reuses the LDS
        if (wave < 3) {  // (the same wave clears par[wave] for the next item)
            const double v = wave_sum(par[wave][lane]);
            item_sum += v;
            if (lane == 0 && B.d.yb == B.d.yend) partial[3 * (size_t)B.d.item + wave] = item_sum;
            if (B.d.yb == B.d.yend) item_sum = 0.0;
        }
        cur = nxt;
    }
    // The last workgroup to finish sums the partials of all items in a fixed
    // order: each workgroup makes its partials visible device-wide before it
    // counts itself finished (next[1]), and the last one takes that count's
    // view of memory before it reads them.
    // (the thread index is hidden from the compiler here as in the loop, so
    // that nothing derived from it is computed before the loop and kept live)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    __syncthreads();
    if (tid == 0) {
        __threadfence();
        sLast = atomicAdd(&next[1], 1) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (sLast) {  // uniform
        __threadfence();
        sum_partials<NT>(tid, item_split<BX, BY, BZ, kBackPairTime, LEAST>(table, cap_ids, G).items, partial, grad_params,
                         accumulate, red);
    }
}

template <int MODEL>
void launch_backward_brick(const BackArgs &a, const BackConst &C, hipStream_t s)
{
    with_shape(a.shape, [&]<int BX, int BY, int BZ>() {
        const BrickGrid G = brick_grid<BX, BY, BZ>(a.grid->ncell, a.grid->periodic);
        const unsigned blocks = (unsigned)G.nbx * G.nby * G.nbz;
        // (the counters were cleared before the launch; the table of bricks
        // with a pair is the build's)
        k_forces_backward_brick<MODEL, BX, BY, BZ, kBackThreads, kBackThreads, kBackCap>
            <<<brick_workgroups(blocks, BY), kBackThreads, 0, s>>>(
                a.n, a.pos, a.vel, a.gforce, a.neibs, a.neibs_brick, a.count, a.cell_start, a.cell_end, a.table,
                a.cap_ids, a.next, a.info, a.gpos, a.gvel, a.partial, a.grad_params, a.accumulate, C, G);
    });
}

}  // namespace

#define SPH_BACK_FN_(k) backward_pairs_kernel##k
#define SPH_BACK_FN(k) SPH_BACK_FN_(k)

bool sph::SPH_BACK_FN(SPH_KERNEL_KIND)(int model, const BackArgs &a, const BackConst &C, hipStream_t s,
                                      int &n_partials)
{
    if (model < 0 || model_kernel(model) != SPH_KERNEL_KIND) return false;
    return with_model<SPH_KERNEL_KIND>(model & kModelLowBits, [&]<int M>() {
        if (a.bricks) {
            // cell ranges and brick-local lists of the last build: LDS bricks
            // (the kernel sums its own partials)
            launch_backward_brick<M>(a, C, s);
            n_partials = 0;
        } else {
            const unsigned blocks = sph_blocks(a.n, kThreads);
            n_partials = (int)blocks;
            k_forces_backward<M><<<blocks, kThreads, 0, s>>>(a.n, a.pos, a.vel, a.aux, a.gforce, a.neibs, a.count,
                                                            a.info, a.gpos, a.gvel, a.partial, a.accumulate, C);
        }
    });
}
