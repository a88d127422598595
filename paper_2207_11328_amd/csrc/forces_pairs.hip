// Pair loops of the time derivatives ("forces"): continuity, pressure
// gradient, artificial and laminar viscosity, density diffusion, for the
// smoothing kernel SPH_KERNEL_KIND (arXiv:2207.11328, eq. mass-cont-sph1,
// eq. ns-sph1, eq. mass-cont-sph2, eq. ns-sph2, section "Minimizing
// complexity", listing l:ktemplate).  This file is compiled once per kernel;
// each object holds every formulation / laminar term / diffusion instance of
// its kernel, in both kernel forms (global gather and LDS brick).
//
// Layout of the work on gfx950:
// * One lane per central particle; the list is neighbour-major inside tiles
//   of 64 particles, so slot k of a wave is one contiguous 256-byte row and
//   its address is one 32-bit offset from the lane's tile base.
// * The trip count is the wave's largest list (a scalar), lanes past their
//   own count are masked, and fluid and boundary segments are walked in one
//   loop (slot k < nf from the front, the rest from the back), so there is
//   no divergent control flow in the pair loop.
// * Loads are software-pipelined: list entries two pairs ahead, neighbour
//   data one pair ahead, so each wave keeps several gathers in flight.
#include <hip/hip_runtime.h>
#include <math.h>

#include "brick_items.h"
#include "forces_common.h"

#ifndef SPH_KERNEL_KIND
#error "compile with SPH_KERNEL_KIND set to one of the SPH_KERNEL_* values"
#endif

using namespace sph;

namespace {

constexpr int kThreads = 256;
// pairs in flight per lane in the derivative loop
#ifndef SPH_FORCES_DEPTH
#define SPH_FORCES_DEPTH 4
#endif
constexpr int kDepth = SPH_FORCES_DEPTH;

struct PairAcc {
    float ax, ay, az, dr;
};

// One pair (i, j) of the derivative sums, branch-free; contributes only when
// it is inside i's list and r < 2h.  mcj = m_j times the kernel coefficient c
// of F = c f(q); ai.y, aj.y = alpha h c / 2 (so the mean of the sound speeds
// and the min(u.x, 0) of Monaghan's term come out of one sum and one
// subtraction: (ai.y + aj.y)(w - |w|) = alpha h (c_i + c_j) min(w, 0));
// ai.x, aj.x = P/rho^2 (golden rule) or P (Landrini-Morris).
// pair_fluid: both particles are fluid (density diffusion applies).
// in: 1 inside the list, 0 past its end.
// LDS: the form of the LDS brick loop, where a pair outside the support or
// past the list has m_j F set to zero and every term is computed (no branch,
// fewer registers); the global-gather loop keeps per-term selects, which the
// compiler turns into a branch that skips the term arithmetic and keeps more
// gathers in flight.  Both give the same values (the zeroed terms add +-0).
// For the Wendland kernel the mask costs one instruction instead of four: F
// = -8 c t^3 with t = 1 - q/2, and the clamp of t to [0, 1] (a modifier of
// the multiply-add) is the support test; `in` takes the place of the 1.  A
// pair at r = 2h within rounding then weighs t^3 ~ 1e-21 on either side.
template <int MODEL, bool LDS>
__device__ __forceinline__ void pair_core(PairAcc &A, float xx, float xy, float xz, const float4 &vi,
                                          const float2 &ai, float mcj, const float4 &vj, const float2 &aj,
                                          float in, bool pair_fluid, const ForceConst &C)
{
    constexpr int KER = model_kernel(MODEL);
    const float r2 = fmaf(xx, xx, fmaf(xy, xy, xz * xz));
    const float r = __builtin_amdgcn_sqrtf(r2);
    // m_j F_ij; in the LDS form zero for a pair outside the support or past
    // the list (every term below is a finite factor times mF)
    bool inter = true;
    float mF;
    if constexpr (LDS && KER == SPH_KERNEL_WENDLAND) {
        const float t = __builtin_amdgcn_fmed3f(fmaf(r, C.neg_inv_2h, in), 0.0f, 1.0f);
        mF = -(t * t) * (t * mcj);  // (mcj holds 8 c m_j: fcoeff_brick)
    } else {
        inter = in > 0.0f && r2 < C.lim2;
        if constexpr (KER == SPH_KERNEL_QUADRATIC) inter = inter && r2 > 0.0f;  // its F is unbounded at r = 0
        const float mF0 = kernel_mF<KER>(mcj, r, r2, C.inv_h, C.inv_h2);
        mF = LDS ? (inter ? mF0 : 0.0f) : mF0;
    }
    const float ux = vi.x - vj.x;
    const float uy = vi.y - vj.y;
    const float uz = vi.z - vj.z;
    const float udx = fmaf(ux, xx, fmaf(uy, xy, uz * xz));
    float pres;
    if constexpr (MODEL & kLandrini) {
        // (P_i + P_j)/(rho_i rho_j) and the continuity weight rho_i/rho_j
        const float inv_rj = __builtin_amdgcn_rcpf(vj.w);
        pres = (ai.x + aj.x) * (inv_rj * __builtin_amdgcn_rcpf(vi.w));
        A.dr = (LDS || inter) ? fmaf(mF * (vi.w * inv_rj), udx, A.dr) : A.dr;
    } else {
        pres = ai.x + aj.x;
        A.dr = (LDS || inter) ? fmaf(mF, udx, A.dr) : A.dr;
    }
    // Monaghan: Pi = -alpha h (c_i + c_j)/2 min(u.x, 0) / ((rho_i + rho_j)/2 (r^2 + eps h^2))
    const float d2 = r2 + C.eps_h2;
    const float den = (vi.w + vj.w) * d2;
    float vnum = -(ai.y + aj.y) * (udx - fabsf(udx));
    // laminar K form: + 4 K nu m_j F (u.x) / ((rho_i + rho_j)(r^2 + eps h^2)) x, the same denominator
    if constexpr (model_visc(MODEL) == kMonaghanK) vnum = fmaf(-C.k_four_nu, udx, vnum);
    const float inv_den = __builtin_amdgcn_rcpf(den);
    const float visc = vnum * inv_den;
    const float coef = (LDS || inter) ? -mF * (pres + visc) : 0.0f;
    A.ax = fmaf(coef, xx, A.ax);
    A.ay = fmaf(coef, xy, A.ay);
    A.az = fmaf(coef, xz, A.az);
    if constexpr (model_visc(MODEL) == kMorris) {
        // 1/(rho_i + rho_j) = (r^2 + eps h^2)/den: no second reciprocal
        const float lam = (LDS || inter) ? C.four_nu * mF * (d2 * inv_den) : 0.0f;
        A.ax = fmaf(lam, ux, A.ax);
        A.ay = fmaf(lam, uy, A.ay);
        A.az = fmaf(lam, uz, A.az);
    }
    if constexpr (MODEL & kDiffusion) {
        // Molteni-Colagrossi: 2 delta h c0 (rho_i - rho_j) m_j F r^2 / ((r^2 + eps h^2) rho_j)
        const float dd = C.diff * (vi.w - vj.w) * mF * r2 * __builtin_amdgcn_rcpf((r2 + C.eps_h2) * vj.w);
        A.dr = ((LDS || inter) && pair_fluid) ? A.dr + dd : A.dr;
    }
}

template <int MODEL>
__device__ __forceinline__ void pair_terms(PairAcc &A, uint32_t e, const float4 &pi, const float4 &vi,
                                           const float2 &ai, const float4 &pj, const float4 &vj, const float2 &aj,
                                           bool valid, bool pair_fluid, const ForceConst &C)
{
    // separation x = k cs + (o_i - o_j), each component bit-identical to the
    // list predicate's; r^2 is then formed with fused multiply-adds, so the
    // r < 2h decision can differ from an exactly rounded one by a rounding
    // of r^2
    const float xx = fmaf(entry_k(e, 0), C.csx, pi.x - pj.x);
    const float xy = fmaf(entry_k(e, 1), C.csy, pi.y - pj.y);
    const float xz = fmaf(entry_k(e, 2), C.csz, pi.z - pj.z);
    pair_core<MODEL, false>(A, xx, xy, xz, vi, ai, pj.w * C.fcoeff, vj, aj, valid ? 1.0f : 0.0f, pair_fluid, C);
}

// Pairs of one lane's list gathered from global memory, in list order.
// Software pipeline over a ring of D pair slots, unrolled by D: slot s holds
// the neighbour data of pair k + s (requested D pairs before it is used) and
// the list entry of pair k + s + D (requested 2 D pairs ahead).  Neighbour
// data registers are only ever written by loads, so the loop carries no copy
// of an in-flight value.
// aux == nullptr: the neighbours' equation-of-state terms are evaluated from
// their densities (eos_terms, bit-identical to the gather form's prologue).
template <int MODEL, int D>
__device__ __forceinline__ void gather_pairs(PairAcc &A, const uint32_t *tile, int nf, int nt, int ntw, int M,
                                             uint32_t jmax, const float4 *__restrict__ pos,
                                             const float4 *__restrict__ vel, const float2 *__restrict__ aux,
                                             const int32_t *__restrict__ cell, const float4 &pi, const float4 &vi,
                                             const float2 &ai, bool central_fluid, const ForceConst &C)
{
    const int last = max(nt - 1, 0);
    uint32_t e[D], en[D];
    float4 P[D], V[D];
    float2 X[D];
    auto terms = [&](uint32_t j, const float4 &v) {
        return aux ? aux[j] : eos_terms<(MODEL & kLandrini) != 0>(v.w, alpha_h_of((int)j, cell, C), C);
    };
#pragma unroll
    for (int s = 0; s < D; ++s) {
        e[s] = tile[list_slot(s, nf, last, M) * kWave];
        en[s] = tile[list_slot(s + D, nf, last, M) * kWave];
    }
#pragma unroll
    for (int s = 0; s < D; ++s) {
        const uint32_t j = min(e[s] & kIndexMask, jmax);
        P[s] = pos[j];
        V[s] = vel[j];
        X[s] = terms(j, V[s]);
    }
    for (int k = 0; k < ntw; k += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            pair_terms<MODEL>(A, e[s], pi, vi, ai, P[s], V[s], X[s], k + s < nt, central_fluid && k + s < nf, C);
            e[s] = en[s];
            const uint32_t j = min(e[s] & kIndexMask, jmax);
            P[s] = pos[j];
            V[s] = vel[j];
            X[s] = terms(j, V[s]);
            en[s] = tile[list_slot(k + s + 2 * D, nf, last, M) * kWave];
        }
    }
}

template <int MODEL>
__global__ __launch_bounds__(kThreads) void k_forces(int n, const float4 *__restrict__ pos,
                                                     const float4 *__restrict__ vel,
                                                     const float2 *__restrict__ aux,
                                                     const uint32_t *__restrict__ neibs,
                                                     const uint32_t *__restrict__ count,
                                                     const uint32_t *__restrict__ info,
                                                     float4 *__restrict__ out, ForceConst C, Corrector K)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    const float tau = K.d_dt && !K.cell_scene ? (float)*K.d_dt : 0.0f;  // (the corrector's step)
    corrector_clock(K);
    const int lane = threadIdx.x % kWave;
    const int ii = min(i, n - 1);  // lanes past the end load in bounds and store nothing
    const int M = C.max_neibs;
    const uint32_t cnt = i < n ? count[i] : 0u;
    // counts and indices are clamped: a stale or foreign list gives wrong
    // numbers but never an out-of-bounds access
    const int nf = min((int)(cnt & 0xFFFFu), M);
    const int nt = min(nf + (int)(cnt >> 16), M);
    const int ntw = __builtin_amdgcn_readfirstlane(wave_max(nt));
    if (ntw == 0) {
        if (i < n) {
            const float4 z = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (out) out[i] = z;
            if (K.d_dt && K.cell[i] >= 0) corrector_at(i, z, vel[i], tau, K);
        }
        return;
    }
    // a wave is exactly one 64-particle tile of the list (wave-uniform base)
    const int tile_id = __builtin_amdgcn_readfirstlane(i / kWave);
    const uint32_t *tile = neibs + (size_t)tile_id * (kWave * M);
    const uint32_t jmax = (uint32_t)(n - 1);

    const float4 pi = pos[ii];
    const float4 vi = vel[ii];
    const float2 ai = aux[ii];
    PairAcc A = {0.0f, 0.0f, 0.0f, 0.0f};

    const bool central_fluid = (MODEL & kDiffusion) ? ptype(info[ii]) != kBoundary : true;
    gather_pairs<MODEL, kDepth>(A, tile + lane, nf, nt, ntw, M, jmax, pos, vel, aux, nullptr, pi, vi, ai,
                                central_fluid, C);
    if (i < n) {
        const float4 f = nt > 0 ? make_float4(A.ax, A.ay, A.az, A.dr) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (out) out[i] = f;
        if (K.d_dt && K.cell[i] >= 0) corrector_at(i, f, vi, tau, K);
    }
}

// ---------------------------------------------------------------------------
// Cell-brick variant of the derivative kernel (the cell perspective of section
// "Changing perspective: from the particle to the cell" applied to the
// derivatives).  A workgroup owns a brick of cells; it first copies
// the particles of the brick and of its one-cell halo (every possible
// neighbour of its particles) from HBM/L2 into LDS with coalesced loads, one
// contiguous cell range after another, then four lanes share the list of one
// central particle of the brick and read the neighbour data from LDS.  The
// 64 lanes of a wave read neighbours scattered over dozens of cache lines,
// which the global-gather kernel pays in L1/L2 request throughput.
//
// The lists are the brick-local ones of the build: entry k is the
// neighbour's LDS slot itself (uint16, fluid then boundary contiguous), so a
// pair costs no index decoding.  Staged positions are relative to the centre
// cell of the brick, o + s cs with s in {-2, ..., 2} per axis, so the
// separation is one subtraction: its rounding error is a few ulp of 2.5 cs,
// not of cs (the list predicate, which must be exact, is not evaluated here).
// The r < 2h mask may therefore differ from an exactly rounded one for a
// pair within that error of the support edge: for the Wendland, cubic-spline
// and quadratic kernels such a pair weighs ~(q - 2)^2 or less, i.e. nothing
// in float32; the truncated Gaussian's F does not vanish at r = 2h, so there
// such a pair carries a finite weight and is counted by one side and not
// the other.  A brick whose halo does not fit in LDS reads the global
// lists and the global state with the arithmetic of k_forces.

// Pairs of one central's brick-local list, read from LDS, shared by kLanes
// lanes: lane h takes the groups of 8 entries h, h + kLanes, h + 2 kLanes, ...
// A group is one 16-byte load for 8 pairs; the staged data of pair k + R is
// requested while pair k is computed (a ring of R slots, R dividing 8 so the
// ring phase is the same in every group).  Two lanes run the loop as fast, but
// their work items are twice as long, and the waves of a brick then wait 5.1
// instead of 3.3 us for the last one (1.62M-particle dam break).
//
// What bounds the loop is VALU issue (85% busy over the whole kernel at 1.62M
// particles): 36 instructions per pair, the method's own 31 (two of them at half
// rate) and 5 for slot, address and list end; the waves wait for LDS in 4% of
// their cycles, and its bank conflicts (half of its accesses' cycles) cost
// nothing measurable.
#ifndef SPH_BRICK_RING
#define SPH_BRICK_RING 2
#endif
constexpr int kRing = SPH_BRICK_RING;
constexpr int kPairTime = 32;  // of a whole brick, in half microseconds (brick_split)
static_assert(kBrickGroup % kRing == 0, "ring must divide the group");

// The staged arrays of a brick.  P and V are read with one address register
// (V's distance fits the 16-bit offset of an LDS read), A with a second one.
template <int CAP>
struct Staged {
    float4 P[CAP];  // brick-relative offset, mass x kernel coefficient
    float4 V[CAP];  // velocity, density
    float2 A[CAP];  // equation-of-state terms
};

// Lane h of a central's kLanes lanes takes the runs of kEntries entries h, h +
// kLanes, ... of its list; ea and eb are its first two.  The two take turns:
// each is loaded again as soon as its last slot is read, so that no loaded
// value is copied (a copy would wait for it) and a run has eight pairs' time
// to arrive.
template <int MODEL, int CAP>
__device__ __forceinline__ void brick_pairs_lds(PairAcc &A, const uint4 *lg, Entries ea, Entries eb, int h, int nt,
                                                uint32_t lo2, uint32_t max2, const Staged<CAP> &L, const float4 &pi,
                                                const float4 &vi, const float2 &ai, const ForceConst &C)
{
    const int runs = (nt + kEntries - 1) / kEntries;
    const uint32_t baseP = lds_address(L.P), baseA = lds_address(L.A);
    float4 P[kRing], V[kRing];
    float2 X[kRing];
    auto fetch = [&](const Entries &e, int s) {
        const uint32_t w = staged_slots(e[s >> 1], lo2, max2), a = slot_address(w, s & 1, 16, baseP);
        const int r = s % kRing;
        P[r] = lds_float4(a, 0);
        V[r] = lds_float4(a, CAP);
        X[r] = lds_float2(slot_address(w, s & 1, 8, baseA));
    };
#pragma unroll
    for (int s = 0; s < kRing; ++s) fetch(ea, s);
    float rem = (float)(nt - h * kEntries);  // entries of the list from this lane's run on
    int g = h;
    auto run = [&](Entries &e, const Entries &f) {
#pragma unroll
        for (int s = 0; s < kEntries; ++s) {
            const int r = s % kRing, s2 = s + kRing;
            // staged w = +-(m_j x kernel coefficient), negative for boundary particles
            pair_core<MODEL, true>(A, pi.x - P[r].x, pi.y - P[r].y, pi.z - P[r].z, vi, ai, fabsf(P[r].w), V[r], X[r],
                                   __builtin_amdgcn_fmed3f(rem - (float)s, 0.0f, 1.0f), pi.w > 0.0f && P[r].w > 0.0f,
                                   C);
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
struct Chunk {
    float4 p, v;
    float ah;  // alpha h
    int cx;    // cell along x from the brick's centre cell
    uint32_t info;
};

template <int MODEL, typename Rows, typename Scans>
__device__ __forceinline__ Chunk load_chunk(const Rows &rows, const Scans &B, int k, int t,
                                            const float4 *__restrict__ pos, const float4 *__restrict__ vel,
                                            const int32_t *__restrict__ cell, const uint32_t *__restrict__ info,
                                            const ForceConst &C)
{
    Chunk q;
    const int j = rows.particle(B, k, t, q.cx);
    q.p = load_at(pos, j);
    q.v = load_at(vel, j);
    q.ah = alpha_h_of(j, cell, C);
    q.info = (MODEL & kDiffusion) ? load_at(info, j) : 0u;
    return q;
}
template <int MODEL, typename Rows, int CAP>
__device__ __forceinline__ void store_chunk(Staged<CAP> &L, const Rows &rows, const Chunk &q, int k, int t,
                                            const ForceConst &C)
{
    if (t >= rows.len[k]) return;
    const int l = rows.slot[k] + t;
    // w = m x kernel coefficient, negated for boundary particles when the
    // density diffusion needs the type
    const float mf = q.p.w * C.fcoeff_brick;
    L.P[l] = rows.brick_relative(q.p, k, q.cx, C.csx, C.csy, C.csz,
                                 (MODEL & kDiffusion) && ptype(q.info) == kBoundary ? -mf : mf);
    L.V[l] = q.v;
    // equation-of-state terms from the staged density
    L.A[l] = eos_terms<(MODEL & kLandrini) != 0>(q.v.w, q.ah, C);
}

// Particles with an empty list (in no table of centrals; also those the build
// dropped) get zero derivatives, by the first T lanes of every workgroup
// while the last wave walks the chain of loads of the first item: no other
// lane writes them.
template <int T>
__device__ __forceinline__ void empty_lists(int n, const uint32_t *__restrict__ count, const float4 *__restrict__ vel,
                                            float4 *__restrict__ out, float tau, const Corrector &K)
{
    constexpr int U = 4;  // counts in flight per lane
    const int stride = gridDim.x * T;
    for (int i0 = blockIdx.x * T + threadIdx.x; i0 < n; i0 += U * stride) {
        uint32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = count[min(i0 + u * stride, n - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * stride;
            if (i < n && c[u] == 0u) {
                const float4 z = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (out) out[i] = z;
                if (K.d_dt && K.cell[i] >= 0) corrector_at(i, z, vel[i], tau, K);
            }
        }
    }
}

// One resident workgroup per CU (its LDS is the CU's) takes items, bricks or
// runs of their rows, one after the other (brick_items.h).  In the time of
// item k:
//   * the staging loads of item k, requested before its turn, are turned into
//     staged particles; the first lists of its centrals and the list counts of
//     item k + 1 are on their way;
//   * after a barrier, the pairs: a wave takes 16 centrals at a time, wave w
//     group w first, then the next unclaimed group (LDS counter) as it finishes
//     one; the lists of a group are requested one group ahead.  One wave first
//     prepares item k + 2;
//   * a wave without a group writes its part of the table of item k + 1 and
//     requests its share of that item's particles.
// 1.62M-particle dam break, 5.9 items per CU: a full brick (800 to 972 centrals)
// takes 3.0 us to the end of the barrier after its staging and 22.4 us from
// there to its last wave, one of 100 to 300 centrals 1.7 and 6.4 us; the first
// item starts 13 to 16 us into the kernel.
template <int MODEL, int BX, int BY, int BZ, int NT, int NC, int CAP>
__global__ __launch_bounds__(NT) void k_forces_brick(int n, const float4 *__restrict__ pos,
                                                     const float4 *__restrict__ vel,
                                                     const int32_t *__restrict__ cell,
                                                     const uint32_t *__restrict__ neibs,
                                                     const uint16_t *__restrict__ neibs_brick,
                                                     const uint32_t *__restrict__ count,
                                                     const int32_t *__restrict__ cell_start,
                                                     const int32_t *__restrict__ cell_end,
                                                     const int32_t *__restrict__ table, int cap_ids,
                                                     int32_t *__restrict__ next,
                                                     const uint32_t *__restrict__ info,
                                                     float4 *__restrict__ out, ForceConst C, BrickGrid G,
                                                     Corrector K)
{
    using St = Staging<BX, BY, BZ>;
    constexpr int NI = St::NI, NW = NT / kWave;
    constexpr bool SHORT = NC < NT;  // entries of the table of centrals
    __shared__ Staged<CAP> L;
    __shared__ BrickScans<BX, BY, BZ> Q[3];  // this item's, the next one's and the one after
    __shared__ CentralTable<NC, NT, SHORT> T[2];        // this item's and the next one's
    __shared__ int sGroup;  // groups of centrals claimed in the item
    // (corrector with a step per scene) each inner cell's scene (-1: none) and step
    __shared__ int sSc[NI];
    __shared__ float sTau[NI];

    const int M = C.max_neibs;
    const float tau = K.d_dt && !K.cell_scene ? (float)*K.d_dt : 0.0f;  // (the corrector's step)
    corrector_clock(K);
    using Rows = StagedRows<BX, BY, BZ, NW>;
    constexpr int SUB = 2;          // chunks of kWave particles of a row carried to the next item
    constexpr int PREP = NW - 1;    // the wave that prepares items
    Chunk chunk[Rows::ROWS][SUB];
    auto load_chunks = [&](const BrickScans<BX, BY, BZ> &N, int wave, int lane) {
        // (always loads, so that no chunk is kept from one item to the next)
        Rows rows;
        rows.locate(N, wave);
#pragma unroll
        for (int k = 0; k < Rows::ROWS; ++k)
#pragma unroll
            for (int u = 0; u < SUB; ++u)
                chunk[k][u] = load_chunk<MODEL>(rows, N, k, u * kWave + lane, pos, vel, cell, info, C);
    };
    // The first item (prepared, staging loads under way, table made) and the second (prepared)
    {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
        if (threadIdx.x == 0) Q[2].d = BrickItem{};
        __syncthreads();
        if (wave == PREP)
            prepare_item<BX, BY, BZ, NC, CAP, kPairTime, 1>(Q[0], Q[2].d, true, lane, table, cap_ids, next, cell_start, cell_end, G);
        else
            empty_lists<PREP * kWave>(n, count, vel, out, tau, K);
        __syncthreads();
        TableMaker<BX, BY, BZ, NC, NT, SHORT> maker;
        maker.request(Q[0], wave, lane, count);
        load_chunks(Q[0], wave, lane);
        if (wave == PREP)  // (while the others' loads arrive)
            prepare_item<BX, BY, BZ, NC, CAP, kPairTime, 1>(Q[1], Q[0].d, false, lane, table, cap_ids, next, cell_start, cell_end, G);
        maker.tally(T[0], wave, lane, M);
        __syncthreads();
        maker.place(T[0], wave, lane);
        __syncthreads();
    }
    int cur = 0;
    for (int k = 0;; ++k) {
        const int nxt = cur == 2 ? 0 : cur + 1, far = nxt == 2 ? 0 : nxt + 1;
        // the thread index is re-read per item (an empty asm hides that it is
        // the same), so nothing derived from it is kept live across the pair loop
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
        const BrickScans<BX, BY, BZ> &B = Q[cur];
        const CentralTable<NC, NT, SHORT> &D = T[k & 1];
        CentralTable<NC, NT, SHORT> &DN = T[(k & 1) ^ 1];
        if (__builtin_amdgcn_readfirstlane(B.d.item) < 0) break;
        const int s_lo = __builtin_amdgcn_readfirstlane(B.d.s_lo), span = __builtin_amdgcn_readfirstlane(B.d.span);
        const bool use_lds = __builtin_amdgcn_readfirstlane(B.d.lds) != 0;
        const int nc = __builtin_amdgcn_readfirstlane(use_lds ? D.used : B.d.nc);
        TableMaker<BX, BY, BZ, NC, NT, SHORT> maker;
        maker.request(Q[nxt], wave, lane, count);

        // a wave takes QG consecutive centrals of the table at a time
        constexpr int QG = kWave / kLanes;
        const int h = lane % kLanes;
        // this lane's central of group g: particle, list length (0: none),
        // table entry, and the first of its list entries, requested here (one
        // group of centrals ahead of its use; the item's first one before the
        // staging)
        struct Central {
            int i, nt;
            uint32_t e;
            const uint4 *lg;
            Entries list, more;
        };
        const uint32_t lo2 = (uint32_t)s_lo * 0x10001u, max2 = (uint32_t)(span - 1) * 0x10001u;
        // (without a branch, so that no loaded value is copied: past the table,
        // or where there is none, a lane loads some particle's list.  An empty
        // table may hold any bits: particle and group are kept inside the lists)
        auto take = [&](int g) {
            Central c;
            const int q = g * QG + lane / kLanes;
            c.e = D.entry(max(min(q, nc - 1), 0));
            const uint32_t i = (c.e & kCenSlotMask) + (uint32_t)B.row_shift[c.e >> kCenRowShift & 15u];
            c.i = (int)min(i, (uint32_t)(n - 1));
            const int len = D.length(c.e, c.i, count, M);
            c.nt = q < nc ? len : 0;
            c.lg = list_groups(neibs_brick, c.i, brick_groups(M));
            const int last = min(max(len - 1, 0) / kEntries, brick_groups(M) - 1);
            c.list = list_entries(c.lg, min(h, last));
            c.more = list_entries(c.lg, min(h + kLanes, last));
            return c;
        };
        int g = wave;
        Central now = take(g);
        if (K.cell_scene && tid < NI) {
            // the step of each inner cell's scene, for the corrector of its
            // centrals (read after the staging barrier)
            const int b = B.d.brick;
            const int cx = (b % G.nbx) * BX + St::ix_of(tid), cy = ((b / G.nbx) % G.nby) * BY + St::iy_of(tid),
                      cz = (b / (G.nbx * G.nby)) * BZ + St::iz_of(tid);
            int sc = -1;
            if (cx < G.nx && cy < G.ny && cz < G.nz) {
                sc = K.cell_scene[cx + G.nx * (cy + G.ny * cz)];
                if ((unsigned)sc >= (unsigned)K.n_scenes) sc = -1;
            }
            sSc[tid] = sc;
            sTau[tid] = sc >= 0 ? (float)K.d_dt[sc] : 0.0f;
        }
        if (tid == 0) sGroup = NW;  // read after the staging barrier
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
                    store_chunk<MODEL>(L, rows, load_chunk<MODEL>(rows, B, r, t, pos, vel, cell, info, C), r, t, C);
        }
        maker.tally(DN, wave, lane, M);
        __syncthreads();
        auto claim = [&]() {
            int c = 0;
            if (lane == 0) c = atomicAdd(&sGroup, 1);
            return __builtin_amdgcn_readfirstlane(c);
        };
        if (wave == PREP) {
            // (few instructions in a long chain of latencies: it goes first)
            __builtin_amdgcn_s_setprio(3);
            prepare_item<BX, BY, BZ, NC, CAP, kPairTime, 1>(Q[far], Q[nxt].d, false, lane, table, cap_ids, next, cell_start, cell_end,
                                              G);
            __builtin_amdgcn_s_setprio(0);
        }
        if (use_lds) {
            while (g * QG < nc) {  // wave-uniform
                const int gn = claim();
                Central c = now;
                now = take(gn);
                const int si = (int)(c.e & kCenSlotMask);
                PairAcc A = {0.0f, 0.0f, 0.0f, 0.0f};
                if (c.nt > 0)
                    brick_pairs_lds<MODEL, CAP>(A, c.lg, c.list, c.more, h, c.nt, lo2, max2, L, L.P[si], L.V[si],
                                                L.A[si], C);
                A.ax = lanes_sum(A.ax);
                A.ay = lanes_sum(A.ay);
                A.az = lanes_sum(A.az);
                A.dr = lanes_sum(A.dr);
                if (h == 0 && c.nt > 0) {
                    const float4 f = make_float4(A.ax, A.ay, A.az, A.dr);
                    if (out) store_at(out, c.i, f);
                    if (K.d_dt) {
                        const float4 ustar = L.V[si];
                        if (!K.cell_scene) {
                            corrector_apply(c.i, f, ustar, tau, K);
                        } else {
                            // the central's inner cell: its place in its row
                            const int r = (int)(c.e >> kCenRowShift & 15u);
                            const int t0 = St::cell(1, r / BZ + 1, r % BZ + 1);
                            int u = r * BX;
#pragma unroll
                            for (int m = 1; m < BX; ++m) u += si + s_lo >= B.base[t0 + m] ? 1 : 0;
                            if (sSc[u] >= 0) corrector_apply(c.i, f, ustar, sTau[u], K);
                        }
                    }
                }
                g = gn;
            }
        } else {
            // more particles than LDS holds: the global lists and state with the
            // arithmetic of k_forces, one lane per central (a shallow pipeline:
            // this path shares the register budget of the LDS path).  0.9M
            // particles at h = 1.5 dp: 1021 us, and 1093 with half the lanes of a
            // wave, 1679 with a quarter
            while (g * kWave < nc) {  // wave-uniform
                const int q = g * kWave + lane;
                const int i = item_central(B, min(q, nc - 1));
                const uint32_t cw = q < nc ? count[i] : 0u;
                const int nf = min((int)(cw & 0xFFFFu), M), nt = min(nf + (int)(cw >> 16), M);
                const int ntw = __builtin_amdgcn_readfirstlane(wave_max(nt));
                if (ntw > 0) {
                    const bool central_fluid = (MODEL & kDiffusion) ? ptype(info[i]) != kBoundary : true;
                    const float4 vi = vel[i];
                    PairAcc A = {0.0f, 0.0f, 0.0f, 0.0f};
                    gather_pairs<MODEL, 2>(A, neibs + (size_t)(i / kWave) * (kWave * M) + (i % kWave), nf, nt, ntw, M,
                                           (uint32_t)(n - 1), pos, vel, nullptr, cell, pos[i], vi,
                                           eos_terms<(MODEL & kLandrini) != 0>(vi.w, alpha_h_of(i, cell, C), C), central_fluid, C);
                    if (nt > 0) {
                        const float4 f = make_float4(A.ax, A.ay, A.az, A.dr);
                        if (out) out[i] = f;
                        if (K.d_dt) corrector_at(i, f, vi, tau, K);
                    }
                }
                g = claim();
            }
        }
        // (in the time that waves without a group wait for the others)
        maker.place(DN, wave, lane);
        load_chunks(Q[nxt], wave, lane);
        __syncthreads();  // the next item reuses the LDS
        cur = nxt;
    }
}

// A workgroup has the LDS of a CU to itself whatever the brick shape: 40
// bytes per staged particle, 10.5 KB of scans and tables.  The halo of a brick at the h =
// 1.3 dp, r_s = 2.86 dp lattice density holds up to about 27 particles per
// staged cell (3 x 4 x 3: 150 cells, at most 15 x 17 x 15 = 3825 lattice places
// in the 1.62M dam break and in tanks of 0.1 to 0.4M, and 9 x 12 x 9 = 972
// centrals); bricks beyond the capacity are taken in runs of fewer rows.  In
// a call of one round of bricks the last one is waited for: tank of 107k particles, 148
// bricks, 33.2 us, and 40.7 with room for 3760 (1% of its bricks cut).  The smaller
// shapes hold at most 3375 at that density and keep the plain table (3 x 2 x 3,
// cubic spline, 1.38M particles: 208 us, and 212 with the short one).
constexpr int kBrickThreads = 1024;
constexpr int brick_centrals(int cells) { return cells >= 36 ? 976 : kBrickThreads; }
constexpr int brick_cap(int cells) { return cells >= 36 ? 3828 : 3760; }

template <int MODEL>
void launch_brick(const ForceArgs &a, const ForceConst &C, hipStream_t s)
{
    with_shape(a.shape, [&]<int BX, int BY, int BZ>() {
        const BrickGrid G = brick_grid<BX, BY, BZ>(a.grid->ncell, a.grid->periodic);
        const unsigned blocks = (unsigned)G.nbx * G.nby * G.nbz;
        // (the item counter, if used, was zeroed before the launch; the table of
        // bricks with a pair is the build's; at most one item per row of a brick)
        const unsigned wgs = brick_workgroups(blocks, BY);
        k_forces_brick<MODEL, BX, BY, BZ, kBrickThreads, brick_centrals(BX * BY * BZ), brick_cap(BX * BY * BZ)><<<wgs, kBrickThreads, 0, s>>>(
            a.n, a.pos, a.vel, a.cell, a.neibs, a.neibs_brick, a.count, a.cell_start, a.cell_end, a.table,
            a.cap_ids, a.next, a.info, a.out, C, G, a.K);
    });
}

}  // namespace

#define SPH_PAIRS_FN_(k) forces_pairs_kernel##k
#define SPH_PAIRS_FN(k) SPH_PAIRS_FN_(k)

bool sph::SPH_PAIRS_FN(SPH_KERNEL_KIND)(int model, const ForceArgs &a, const ForceConst &C, hipStream_t s)
{
    if (model < 0 || model_kernel(model) != SPH_KERNEL_KIND) return false;
    return with_model<SPH_KERNEL_KIND>(model & kModelLowBits, [&]<int M>() {
        if (a.bricks) {
            // cell ranges and brick-local lists of the last build: LDS cell-brick
            // kernel (it writes the derivatives of every particle, those with an
            // empty list and those dropped by the build while it prepares its first item)
            launch_brick<M>(a, C, s);
        } else {
            k_forces<M><<<sph_blocks(a.n, kThreads), kThreads, 0, s>>>(a.n, a.pos, a.vel, a.aux, a.neibs, a.count,
                                                                       a.info, a.out, C, a.K);
        }
    });
}
