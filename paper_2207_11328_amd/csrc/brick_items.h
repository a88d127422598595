// Work items of the persistent brick kernels (derivatives and adjoint): the
// claiming of bricks, the cell scans of a brick and the table of its central
// particles, all by one wave, ahead of the workgroup.
//
// One resident workgroup per CU takes the bricks of the build's table one
// after the other (heavy ones first: brick_at).  What a brick needs before
// its pairs can be summed is a chain of dependent loads (brick id, cell
// ranges, list counts, lists), several microseconds of latency and hardly any
// arithmetic.  So the items are pipelined: while the workgroup sums the pairs
// of item k, one wave walks the chain up to the cell ranges of item k + 2
// (prepare_item), and every wave has the counts of 64 centrals of item k + 1
// in flight with its staging loads and makes its part of that item's table of
// centrals (TableMaker).  At the start of an item every wave then knows its
// centrals and requests their lists together with the staging loads.
//
// The table leaves out the central particles with an empty list.  (Grouping
// the others by list length, in classes of 24 entries, fills 89% of the lanes
// of the pair loop instead of 87% on the 1.62M-particle dam break, but
// scatters the list loads: measured slower, 155.6 against 153.3 us.)
//
// An item is a run of y rows of a brick.  The staging order has y outermost,
// so the staged cells of a run (its rows and one halo row on each side) are
// one contiguous range of staging slots, and the brick-local lists index into
// it unchanged.  Whole bricks stage the fewest particles per central one;
// they are cut into parts where the grid's bricks would leave CUs idle
// (brick_split), and where a brick holds somewhat more particles than LDS or
// more centrals than lanes.
#pragma once

#include <type_traits>

#include "sph_device.h"

namespace sph {

// How the bricks of the table are cut into items, by their place in it: all but
// `cut` of them, which come after the first `whole` (the larger ones), into
// `first` parts each, then those into `rest`.
struct BrickSplit {
    int whole, cut, first, rest, uncut, items;  // uncut: items of the first kind
};

// The split of n bricks, `heavy` of them heavy ones, for wgs workgroups.
// Less than a round of bricks: all of them into the parts whose rounds, times
// the cost of an item, cost least: about 5 us of staging and latency for a whole
// brick, 4 for a half, 3.5 for a row, and PAIRS halves of a microsecond for the
// pairs of a full 3 x 4 x 3 brick.  Tank of 15.5k particles (27 bricks with a
// pair): 16.9 us in rows against 30.0 with whole bricks; 169k dam break (120,
// cubic spline, Landrini-Morris, Morris viscosity, diffusion): 34.1 us in halves
// against 51.4.
// One to three rounds of heavy bricks: whole ones, and the heavy ones left over
// by the last whole round in the smallest parts that keep all items within one
// round more; the light ones are short and fill the gaps whole, before the
// parts.  Tank of 320 bricks, 280 of them heavy: 55.6 us
// with the 24 left over in rows against 64.5 whole; 378, 325 heavy: 56.5 us in halves
// against 63.8, and 66.3 in rows (three rounds of items); batch of 497, 364 heavy: 64.6 us
// whole against 78.7 in halves (as many rounds more); tank of 567, 564 heavy: 70.6 us in rows
// against 78.1.  From three rounds on what is left over is small against
// them: no split of 770 to 1030 bricks was faster than whole ones.
// FIRST: the parts below which no item would fit in LDS, limit: the most items
// (there are slots for).
template <int BX, int BY, int BZ, int PAIRS, int FIRST>
__device__ __forceinline__ BrickSplit brick_split(int n, int heavy, int wgs, int limit)
{
    constexpr int P = PAIRS * BX * BY * BZ / 36;
    constexpr auto cost = [](int parts) { return (parts == 1 ? 10 : parts == BY ? 7 : 8) + P / parts; };
    constexpr int HALF = BY % 2 == 0 && BY > 2 ? 2 : FIRST;
    if (n * FIRST > limit) return {n, 0, 1, 1, n, n};
    BrickSplit best = {n, 0, FIRST, FIRST, n * FIRST, n * FIRST};
    if (n * FIRST < wgs) {
        int least = INT32_MAX;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int parts = k == 0 ? FIRST : k == 1 ? HALF : BY;
            if (k == 1 && HALF == FIRST) continue;
            int c = 0;
            for (int i = n * parts; i > 0; i -= wgs) c += cost(parts);  // (BY rounds at most)
            if (c < least && n * parts <= limit) {
                best = {n, 0, parts, parts, n * parts, n * parts};
                least = c;
            }
        }
    } else if (heavy * FIRST > wgs && heavy * FIRST < 3 * wgs) {
        const int rounds = heavy * FIRST < 2 * wgs ? 1 : 2, whole = rounds * wgs / FIRST, left = heavy - whole;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int parts = k == 0 ? HALF : BY, items = (n - left) * FIRST + left * parts;
            if (parts > FIRST && items <= (rounds + 1) * wgs && items <= limit)
                best = {whole, left, FIRST, parts, (n - left) * FIRST, items};
        }
    }
    return best;
}

template <int BX, int BY, int BZ, int PAIRS, int FIRST>
__device__ __forceinline__ BrickSplit item_split(const int32_t *__restrict__ table, int cap_ids, const BrickGrid &G)
{
    const int heavy = table[0], n = heavy + table[cap_ids + 1];
    return brick_split<BX, BY, BZ, PAIRS, FIRST>(n, heavy, gridDim.x, G.nx * G.ny * G.nz);
}

// Descriptor of an item.
struct BrickItem {
    int item;    // index in the claim order, -1: none left
    int brick;
    int ya, yb;  // inner y rows
    int yend;    // end of the part of the brick that was claimed (rows yb .. yend follow)
    int s_lo;    // first staged slot, in the staging order of the whole brick
    int span;    // staged particles
    int nc;      // central particles in the rows (with an empty list included)
    int lds;     // the run fits in LDS
};

// Bricks with more staged particles than this (1.4 times the lattice density
// in a 3 x 4 x 3 brick) are not cut into runs but read the global lists, with
// the bits of the gather form.
constexpr int kRunTotal = 4800;

// Entry of the table: staged slot (from s_lo) | inner row << 12 | list length << 16.
constexpr int kCenRowShift = 12, kCenCountShift = 16;
constexpr uint32_t kCenSlotMask = (1u << kCenRowShift) - 1u;

template <int BX, int BY, int BZ>
struct BrickScans {
    using St = Staging<BX, BY, BZ>;
    static constexpr int NR = BY * BZ;  // inner rows (x-consecutive cells: one particle range each)
    static_assert(NR <= 16, "a row id fits its field of a table entry");
    int base[St::S + 1];  // staged slot of each staged cell
    int delta[St::S];     // slot minus particle index
    int row_first[16];      // centrals before each inner row of the item (past the last row: all ones)
    int row_index[16];      // particle index of its first central
    int row_shift[16];      // particle index minus staged slot (from s_lo)
    BrickItem d;
};

// Lane k's value of an inclusive sum over the first 2^STEPS lanes.
template <int STEPS>
__device__ __forceinline__ int lanes_scan(int v, int lane)
{
#pragma unroll
    for (int o = 1; o < (1 << STEPS); o <<= 1) {
        const int t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    return v;
}

// The next item into Q, by one wave: the rows left of item prev, else the next
// part of a brick from the counter.  CAP: staged particles that fit in LDS;
// NC: centrals that fit in the table.
template <int BX, int BY, int BZ, int NC, int CAP, int PAIRS, int LEAST>
__device__ __forceinline__ void prepare_item(BrickScans<BX, BY, BZ> &Q, const BrickItem &prev, bool first, int lane,
                                             const int32_t *__restrict__ table, int cap_ids,
                                             int32_t *__restrict__ next, const int32_t *__restrict__ cell_start,
                                             const int32_t *__restrict__ cell_end, const BrickGrid &G)
{
    using St = Staging<BX, BY, BZ>;
    constexpr int SX = St::SX, SZ = St::SZ, S = St::S, ROW = SX * SZ, NR = BY * BZ;
    static_assert(CAP <= (int)kCenSlotMask + 1, "a staged slot fits its field of a table entry");
    const int pb = __builtin_amdgcn_readfirstlane(prev.yb), pe = __builtin_amdgcn_readfirstlane(prev.yend);
    int item, b, ya, yend;
    if (pb < pe) {
        item = __builtin_amdgcn_readfirstlane(prev.item);
        b = __builtin_amdgcn_readfirstlane(prev.brick);
        ya = pb;
        yend = pe;
    } else {
        // the first item of a workgroup is its index; the others come from the
        // counter (zeroed before the launch), or, without one, rounds of
        // workgroups take the items, which are ordered by size, forwards and
        // backwards in turn
        const int heavy = table[0];
        const int guess = first ? table[1 + min((int)blockIdx.x, cap_ids - 1)] : 0;  // (sent for with the counts)
        const BrickSplit B = item_split<BX, BY, BZ, PAIRS, LEAST>(table, cap_ids, G);
        const int items = B.items, last = __builtin_amdgcn_readfirstlane(prev.item);
        item = items;
        if (first) {
            item = blockIdx.x;
        } else if (!next) {
            if (last >= 0) {
                const int g = gridDim.x, round = last / g + 1;
                item = round * g + (round & 1 ? g - 1 - (int)blockIdx.x : (int)blockIdx.x);
            }
        } else if (last >= 0 && items > (int)gridDim.x) {
            int k = 0;
            if (lane == 0) k = atomicAdd(next, 1);
            item = __builtin_amdgcn_readfirstlane(k) + gridDim.x;
        }
        if (item >= items) {
            if (lane == 0) {
                Q.d = BrickItem{};
                Q.d.item = -1;
            }
            return;
        }
        const bool piece = item >= B.uncut;
        const int parts = piece ? B.rest : B.first, of = piece ? item - B.uncut : item;
        const int quot = parts == 1 ? of : parts == 2 ? of / 2 : parts == 3 ? of / 3 : of / 4;
        static_assert(BY <= 4, "parts of a brick");
        const int place = piece ? B.whole + quot : quot < B.whole ? quot : quot + B.cut;
        b = first && place == (int)blockIdx.x && place < heavy ? guess : brick_at(table, cap_ids, place);
        const int rows = parts == 1 ? BY : parts == BY ? 1 : BY / 2;
        ya = (of - quot * parts) * rows;
        yend = ya + rows;
    }
    const int cx0 = (b % G.nbx) * BX, cy0 = ((b / G.nbx) % G.nby) * BY, cz0 = (b / (G.nbx * G.nby)) * BZ;
    // ranges of the staged cells (empty outside a non-periodic grid edge) and
    // their slots in the staging order of the whole brick
    constexpr int NCH = (S + kWave - 1) / kWave;
    int st[NCH], ct[NCH], total = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int t = c * kWave + lane;
        st[c] = 0;
        ct[c] = 0;
        if (t < S) {
            int gx = cx0 - 1 + St::sx_of(t), gy = cy0 - 1 + St::sy_of(t), gz = cz0 - 1 + St::sz_of(t);
            const bool ok = wrap_axis(gx, G.nx, G.periodic & 1u) && wrap_axis(gy, G.ny, (G.periodic >> 1) & 1u) &&
                            wrap_axis(gz, G.nz, (G.periodic >> 2) & 1u);
            if (ok) {
                const int lin = gx + G.nx * (gy + G.ny * gz);
                st[c] = cell_start[lin];
                ct[c] = cell_end[lin] - st[c];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int t = c * kWave + lane, inc = lanes_scan<6>(ct[c], lane), ex = total + inc - ct[c];
        if (t < S) {
            Q.base[t] = ex;
            Q.delta[t] = ex - st[c];
        }
        total += __builtin_amdgcn_readlane(inc, kWave - 1);
    }
    if (lane == 0) Q.base[S] = total;
    wave_fence();  // (read below by other lanes than wrote them)
    // the inner rows, one per lane (inner cells past the grid edge hold no
    // centrals: on a periodic axis the staged copy is the wrapped cell, owned
    // by another brick)
    const int iy = lane / BZ, iz = lane % BZ;
    const bool row = lane < NR && cy0 + iy < G.ny && cz0 + iz < G.nz;
    const int t0 = St::cell(1, row ? iy + 1 : 1, row ? iz + 1 : 1), bxn = min(BX, G.nx - cx0);
    const int slot0 = Q.base[t0], all = row ? Q.base[t0 + bxn] - slot0 : 0, dl = Q.delta[t0];
    // the longest run of rows that fits (of a brick that takes runs at all)
    const int s_lo = __builtin_amdgcn_readfirstlane(Q.base[ya * ROW]);
    int yb = yend, span = 0, nc = 0;
    for (;; --yb) {
        span = __builtin_amdgcn_readfirstlane(Q.base[(yb + 2) * ROW]) - s_lo;
        nc = lanes_scan<4>(iy >= ya && iy < yb ? all : 0, lane);
        nc = __builtin_amdgcn_readlane(nc, 15);
        if (yb == ya + 1 || total > kRunTotal || (span <= CAP && nc <= NC)) break;
    }
    const bool lds = span <= CAP && nc <= NC && total <= kRunTotal;
    const int cnt = iy >= ya && iy < yb ? all : 0;
    const int inc = lanes_scan<4>(cnt, lane);
    if (lane < 16) Q.row_first[lane] = lane < NR ? inc - cnt : INT32_MAX;
    if (lane < NR) {
        Q.row_index[lane] = slot0 - dl;
        Q.row_shift[lane] = s_lo - dl;
    }
    if (lane == 0) {
        Q.d.item = item;
        Q.d.brick = b;
        Q.d.ya = ya;
        Q.d.yb = yb;
        Q.d.yend = yend;
        Q.d.s_lo = s_lo;
        Q.d.span = span;
        Q.d.nc = nc;
        Q.d.lds = lds ? 1 : 0;
    }
}

// Inner row of central q of the item (sorted order): the last one whose first
// central is q or before (the others of the same first central are empty).
template <int BX, int BY, int BZ>
__device__ __forceinline__ int central_row(const BrickScans<BX, BY, BZ> &Q, int q)
{
    int r = 0;
#pragma unroll
    for (int step = 8; step; step >>= 1) r = Q.row_first[r + step] <= q ? r + step : r;
    return r;
}

// Particle index of central q, for items that do not fit in LDS.
template <int BX, int BY, int BZ>
__device__ __forceinline__ int item_central(const BrickScans<BX, BY, BZ> &Q, int q)
{
    const int r = central_row(Q, q);
    return Q.row_index[r] + (q - Q.row_first[r]);
}

// p[i] by a 32-bit byte offset from a scalar base (per-particle arrays have at
// most 2^26 entries): one address register and no 64-bit arithmetic.
template <typename T>
__device__ __forceinline__ T load_at(const T *__restrict__ p, int i)
{
    return *(const T *)((const char *)p + (uint32_t)i * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void store_at(T *__restrict__ p, int i, const T &v)
{
    *(T *)((char *)p + (uint32_t)i * (uint32_t)sizeof(T)) = v;
}

// The table of centrals of an item, made by all waves of the workgroup, 64
// centrals each: request() sends for the list counts, tally() leaves how many
// of the wave's centrals have a list, and after a barrier place() writes the
// entries, in sorted order.
// NC: centrals that fit.  SHORT: an entry takes 3 bytes instead of 4, its list
// length 8 bits, where kLongList stands for that many or more (length() reads
// the count again): the 2 KB hold 51 more staged particles.
constexpr int kLongList = 255;
template <int NC, int NT, bool SHORT>
struct CentralTable {
    typename std::conditional<SHORT, uint16_t, uint32_t>::type cen[NC];
    uint8_t len[SHORT ? NC : 1];
    int tally[NT / kWave];
    int used;  // entries: centrals with a list

    __device__ __forceinline__ uint32_t entry(int q) const
    {
        return SHORT ? cen[q] | (uint32_t)len[q] << kCenCountShift : cen[q];
    }
    // list length of entry e, particle i (M: list slots per particle)
    __device__ __forceinline__ static int length(uint32_t e, int i, const uint32_t *__restrict__ count, int M)
    {
        int n = (int)(e >> kCenCountShift);
        if (SHORT && M >= kLongList && n == kLongList) {
            const uint32_t cw = load_at(count, i);
            n = min(min((int)(cw & 0xFFFFu), M) + (int)(cw >> 16), M);
        }
        return n;
    }
    __device__ __forceinline__ void set(int q, uint32_t slot_row, int n)
    {
        if constexpr (SHORT) {
            cen[q] = (uint16_t)slot_row;
            len[q] = (uint8_t)min(n, kLongList);
        } else {
            cen[q] = slot_row | (uint32_t)n << kCenCountShift;
        }
    }
};

template <int BX, int BY, int BZ, int NC, int NT, bool SHORT>
struct TableMaker {
    uint32_t entry;  // slot and row
    uint32_t cw;     // list count
    int len;

    __device__ __forceinline__ void request(const BrickScans<BX, BY, BZ> &Q, int wave, int lane,
                                            const uint32_t *__restrict__ count)
    {
        const int nc = __builtin_amdgcn_readfirstlane(Q.d.nc);
        entry = 0u;
        cw = 0u;
        if (__builtin_amdgcn_readfirstlane(Q.d.item) < 0 || !__builtin_amdgcn_readfirstlane(Q.d.lds) ||
            wave * kWave >= nc)
            return;  // uniform
        const int q = min(wave * kWave + lane, nc - 1);
        const int r = central_row(Q, q);
        const int i = Q.row_index[r] + (q - Q.row_first[r]);
        entry = (uint32_t)(i - Q.row_shift[r]) | (uint32_t)r << kCenRowShift;
        cw = load_at(count, i);
        if (wave * kWave + lane >= nc) cw = 0u;
    }

    // M: list slots per particle
    __device__ __forceinline__ void tally(CentralTable<NC, NT, SHORT> &T, int wave, int lane, int M)
    {
        // (clamped: a stale or foreign list gives wrong numbers but never an
        // access outside the lists)
        const int nf = min((int)(cw & 0xFFFFu), M);
        len = min(nf + (int)(cw >> 16), M);
        const int some = (int)__popcll(__builtin_amdgcn_ballot_w64(len > 0));
        if (lane == 0) T.tally[wave] = some;
    }

    __device__ __forceinline__ void place(CentralTable<NC, NT, SHORT> &T, int wave, int lane)
    {
        constexpr int NW = NT / kWave;
        const int inc = lanes_scan<4>(lane < NW ? T.tally[min(lane, NW - 1)] : 0, lane);
        if (wave == 0 && lane == NW - 1) T.used = inc;
        const int before = wave == 0 ? 0 : __builtin_amdgcn_readlane(inc, wave - 1);
        const unsigned long long m = __builtin_amdgcn_ballot_w64(len > 0);
        const int p = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)before));
        if (len > 0) T.set(p, entry, len);
    }
};

// ---- reading a brick's lists and staged particles ----------------------------

// LDS by address (a 32-bit offset in the workgroup's LDS).
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef float vf2 __attribute__((ext_vector_type(2)));
template <typename T>
using Lds = __attribute__((address_space(3))) T;
template <typename T>
__device__ __forceinline__ uint32_t lds_address(const T *p)
{
    return (uint32_t)(uintptr_t)(Lds<const T> *)p;
}
__device__ __forceinline__ float4 lds_float4(uint32_t a, int index)
{
    const vf4 v = ((Lds<const vf4> *)(uintptr_t)a)[index];
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float2 lds_float2(uint32_t a)
{
    const vf2 v = *(Lds<const vf2> *)(uintptr_t)a;
    return make_float2(v.x, v.y);
}

// base + scale x (the 16-bit slot in half `hi` of w): one instruction, the
// unpacking included.
__device__ __forceinline__ uint32_t slot_address(uint32_t w, int hi, int scale, uint32_t base)
{
    uint32_t a;
    if (scale == 16) {
        if (hi) asm("v_mad_u32_u16 %0, %1, 16, %2 op_sel:[1,0,0,0]" : "=v"(a) : "v"(w), "s"(base));
        else asm("v_mad_u32_u16 %0, %1, 16, %2" : "=v"(a) : "v"(w), "s"(base));
    } else {
        if (hi) asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[1,0,0,0]" : "=v"(a) : "v"(w), "s"(base));
        else asm("v_mad_u32_u16 %0, %1, 8, %2" : "=v"(a) : "v"(w), "s"(base));
    }
    return a;
}

// Lanes per central, and the entries one of them takes at a time.
constexpr int kLanes = 4, kEntries = kBrickGroup;
typedef uint32_t Entries __attribute__((ext_vector_type(4)));
// group e of a brick-local list, lg its group 0
__device__ __forceinline__ Entries list_entries(const uint4 *lg, int e)
{
    return load_at((const Entries *)lg, e * kWave);
}
// Two slots of a list relative to the first staged one, kept inside the staged
// range (a stale list gives wrong numbers but no access past it).
__device__ __forceinline__ uint32_t staged_slots(uint32_t w, uint32_t lo2, uint32_t max2)
{
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    const us2 d = __builtin_elementwise_sub_sat(__builtin_bit_cast(us2, w), __builtin_bit_cast(us2, lo2));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(d, __builtin_bit_cast(us2, max2)));
}

// The sum of a value over the lanes of a central, in all of them.
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float lanes_sum(float v)
{
    v += dpp<0xB1>(v);  // quad lanes 1, 0, 3, 2
    v += dpp<0x4E>(v);  // quad lanes 2, 3, 0, 1
    return v;
}

// The brick-local list of particle i (brick_entry(i, 0, groups)): group g at
// [g * kWave].
__device__ __forceinline__ const uint4 *list_groups(const uint16_t *__restrict__ neibs_brick, int i, uint32_t groups)
{
    const uint32_t u = (uint32_t)i;
    return (const uint4 *)((const char *)neibs_brick + (uint64_t)(u / kWave) * (groups * (kWave * 16u)) +
                           (u % kWave) * 16u);
}

// Staged rows of cells of an item (SX x-consecutive cells: one contiguous LDS
// range and, away from a periodic seam, one contiguous global range): wave w
// takes rows w and w + NW.
template <int BX, int BY, int BZ, int NW>
struct StagedRows {
    using St = Staging<BX, BY, BZ>;
    static constexpr int SX = St::SX, SZ = St::SZ, ROWS = 2;
    static_assert(St::SY * SZ <= ROWS * NW, "two rows per wave hold every row");
    int row[ROWS], slot[ROWS], len[ROWS];  // row, its first slot (from s_lo), its particles

    __device__ __forceinline__ void locate(const BrickScans<BX, BY, BZ> &B, int wave)
    {
        const bool staged = __builtin_amdgcn_readfirstlane(B.d.item) >= 0 && __builtin_amdgcn_readfirstlane(B.d.lds);
        const int R0 = __builtin_amdgcn_readfirstlane(B.d.ya * SZ), R1 = __builtin_amdgcn_readfirstlane((B.d.yb + 2) * SZ);
#pragma unroll
        for (int k = 0; k < ROWS; ++k) {
            row[k] = min(R0 + wave + k * NW, R1 - 1);
            const int b0 = __builtin_amdgcn_readfirstlane(B.base[row[k] * SX]);
            slot[k] = b0 - __builtin_amdgcn_readfirstlane(B.d.s_lo);
            const int l = __builtin_amdgcn_readfirstlane(B.base[row[k] * SX + SX]) - b0;
            len[k] = staged && R0 + wave + k * NW < R1 ? l : 0;
        }
    }
    // Index of particle t of row k, and its cell along x from the brick's
    // centre cell (t past the row's end: particle 0).
    __device__ __forceinline__ int particle(const BrickScans<BX, BY, BZ> &B, int k, int t, int &cx) const
    {
        const int *base = B.base + row[k] * SX, *delta = B.delta + row[k] * SX;
        const int s = base[0] + t;
        int d = delta[0];
        cx = -2;
#pragma unroll
        for (int m = 1; m < SX; ++m) {
            const bool past = s >= base[m];
            cx += past ? 1 : 0;
            d = past ? delta[m] : d;
        }
        return t < len[k] ? s - d : 0;
    }
    // Position of a particle of row k relative to the centre cell of the whole
    // brick (cx along x).
    __device__ __forceinline__ float4 brick_relative(const float4 &p, int k, int cx, float csx, float csy, float csz,
                                                     float w) const
    {
        return make_float4(fmaf((float)cx, csx, p.x), fmaf((float)(row[k] / SZ - 2), csy, p.y),
                           fmaf((float)(row[k] % SZ - 2), csz, p.z), w);
    }
};

// Workgroups of a persistent brick kernel over a grid of `blocks` bricks of BY
// rows: one per CU (at most one item per row of a brick).
inline unsigned brick_workgroups(unsigned blocks, unsigned BY)
{
    const unsigned cus = (unsigned)sph_device_cus();
    return blocks < (cus + BY - 1) / BY ? blocks * BY : cus;
}

}  // namespace sph
