// Neighbour search: re-bin, counting sort by cell with an in-cell sort by
// (type, id), reorder, cell ranges and split neighbour lists.
//
// Sort order is cell, then particle type, then particle id (section
// "Changing perspective: from the particle to the cell").  Instead of a
// multi-pass radix sort of 64-bit keys, the cell index is used directly as
// a single radix digit: a histogram over cells, an exclusive scan (which is
// also the cell-start array) and a scatter put every particle in its cell's
// range; each particle then ranks itself among the few of its cell by their
// (type, id) words, which makes the permutation unique, and is copied to its
// final place.
//
// Lists are split (fluid from the front, boundary from the back) and stored
// neighbour-major (section "Efficient split neighbors list").
#include <hip/hip_runtime.h>

#include "sph_device.h"

using namespace sph;

namespace {

constexpr int kThreads = 256;
constexpr int kScanItems = 4;                       // per thread
constexpr int kScanTile = kThreads * kScanItems;    // elements per block
// blocks up to which every block of the scan adds up the sums before it
// itself (1M cells: at most 4 loads per lane; beyond, the re-reading grows with
// the square of the grid)
constexpr int kFewPartials = 1024;

struct BuildLayout {
    size_t cnt, hist, start, partials, keys, index, t_cell, t_pos, t_vel, place, active, classes, total;
};

size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

BuildLayout build_layout(int64_t capacity, int64_t n_cells)
{
    const int64_t nb = n_cells + 1;  // one extra bucket for dropped particles
    const int64_t nparts = (nb + kScanTile - 1) / kScanTile;
    BuildLayout L;
    size_t o = 0;
    L.cnt = o;      o = align_up(o + sizeof(int32_t) * nb);
    // (a histogram of 64 classes per 1024 bricks, and at most one brick per
    // cell: within nb words, or within the 64 of the alignment)
    L.hist = o;     o = align_up(o + sizeof(int32_t) * nb);
    L.start = o;    o = align_up(o + sizeof(int32_t) * (nb + 1));
    L.partials = o; o = align_up(o + sizeof(int32_t) * (nparts + 1));
    L.keys = o;     o = align_up(o + sizeof(uint32_t) * capacity);
    L.index = o;    o = align_up(o + sizeof(uint32_t) * capacity);
    L.t_cell = o;   o = align_up(o + sizeof(int32_t) * capacity);
    L.t_pos = o;    o = align_up(o + sizeof(float4) * capacity);
    L.t_vel = o;    o = align_up(o + sizeof(float4) * capacity);
    L.place = o;    o = align_up(o + sizeof(uint32_t) * capacity);
    L.active = o;   o = align_up(o + sizeof(int32_t) * (n_cells + 1));
    L.classes = o;  o = align_up(o + (size_t)n_cells + 4);
    L.total = o;
    return L;
}

// Everything the build counts into starts at zero, in one launch (a kernel,
// not a memset, so that a captured graph holds no memset node): the bucket
// counts (nb), the status words, the size classes of the bricks with a pair
// (key_words int32 words, none without brick lists) and the counter of the
// active-brick list.
__global__ void k_build_zero(int64_t nb, int32_t *__restrict__ cnt, int32_t *__restrict__ status, int64_t key_words,
                             int32_t *__restrict__ keys, int32_t *__restrict__ active)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = t; i < nb; i += stride) cnt[i] = 0;
    for (int64_t i = t; i < key_words; i += stride) keys[i] = 0;
    if (t < SPH_STATUS_WORDS) status[t] = 0;
    if (t == 0) *active = 0;
}

// atomicAdd(&cnt[key], 1) for every valid lane of a wave, combined over runs
// of consecutive lanes with the same key (particles come in the order of the
// last build, sorted by cell, so a run is typically a whole cell's part of
// the wave): one atomic per run.  Returns the value the lane's own atomic
// could have returned (the run's base plus the lane's rank in the run).
// Every lane of the wave must call it.
__device__ __forceinline__ int run_atomic_inc(int32_t *cnt, int key, bool valid)
{
    const int lane = threadIdx.x % kWave;
    const int prev = __shfl(key, lane > 0 ? lane - 1 : 0);
    const unsigned long long vmask = __ballot(valid);
    const bool prev_valid = lane > 0 && ((vmask >> (lane - 1)) & 1ull);
    const bool first = valid && (!prev_valid || prev != key);
    // run boundaries: run starts and invalid lanes
    const unsigned long long bounds = __ballot(first) | ~vmask;
    const unsigned long long upto = bounds & (~0ull >> (kWave - 1 - lane));  // bits <= lane
    const int rs = kWave - 1 - __clzll(upto | 1ull);
    const unsigned long long above = lane == kWave - 1 ? 0ull : bounds & (~0ull << (lane + 1));
    const int re = above ? __ffsll((long long)above) - 1 : kWave;
    int base = 0;
    if (first) base = atomicAdd(&cnt[key], re - rs);
    base = __shfl(base, rs);
    return base + (lane - rs);
}

// Re-bin offsets into [-cs/2, cs/2) (float32, at most 4 cells per axis) and
// count particles per cell.  Particles that leave a non-periodic axis, or
// whose offsets are not finite, become dropped (cell = -1, last bucket).  The
// re-binned state goes to the workspace, from where k_sort_gather brings it
// back in sorted order (so the state is read and written twice in all), with
// each particle's place among its cell's as the counting met it.  Also counts the
// particles whose offset, mass, velocity or density is not finite (one atomic
// per wave), so that a state that blew up is reported by the status word.
__global__ __launch_bounds__(kThreads) void k_rebin_count(
    int n, const int32_t *__restrict__ cell, const float4 *__restrict__ pos, const float4 *__restrict__ vel,
    CellDims dims, float csx, float csy, float csz, int cell_base, int n_cells, int32_t *__restrict__ cnt,
    int32_t *__restrict__ t_cell, float4 *__restrict__ t_pos, float4 *__restrict__ t_vel,
    uint32_t *__restrict__ place, int32_t *__restrict__ status)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    const bool valid = i < n;
    int c = valid ? cell[i] : -1;
    int bucket = n_cells;
    bool bad = false;
    if (valid) {
        float4 p = pos[i];
        const float4 v = vel[i];
        t_vel[i] = v;
        int moved = c;
        if (c >= 0) {
            int cc[3];
            cell_coords(c - cell_base, dims, cc[0], cc[1], cc[2]);
            float o[3] = {p.x, p.y, p.z};
            const float cs[3] = {csx, csy, csz};
            const int nd[3] = {dims.nx, dims.ny, dims.nz};
            bool ok = true;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const float half = 0.5f * cs[d];
                float w = o[d];
                for (int it = 0; it < 4; ++it) {
                    if (w >= half) { w = w - cs[d]; cc[d] += 1; }
                    else if (w < -half) { w = w + cs[d]; cc[d] -= 1; }
                    else break;
                }
                if (!(w >= -half && w < half)) ok = false;
                if ((dims.periodic >> d) & 1u) {
                    cc[d] %= nd[d];
                    if (cc[d] < 0) cc[d] += nd[d];
                } else if (cc[d] < 0 || cc[d] >= nd[d]) {
                    ok = false;
                }
                o[d] = w;
            }
            p = make_float4(o[0], o[1], o[2], p.w);
            if (ok) {
                const int lc = cc[0] + dims.nx * (cc[1] + dims.ny * cc[2]);
                moved = lc + cell_base;
                bucket = lc;
            } else {
                moved = -1;
            }
        }
        t_cell[i] = moved;
        t_pos[i] = p;
        bad = !(isfinite(p.x) && isfinite(p.y) && isfinite(p.z) && isfinite(p.w) && isfinite(v.x) &&
                isfinite(v.y) && isfinite(v.z) && isfinite(v.w));
    }
    const int r = run_atomic_inc(cnt, bucket, valid);
    if (valid) place[i] = (uint32_t)r;
    const unsigned long long m = __ballot(bad);
    if (m && (threadIdx.x % kWave) == 0) atomicAdd(&status[SPH_STATUS_NONFINITE], (int)__popcll(m));
}

// ---- exclusive scan of cnt[0..m) into start[0..m], start[m] = total --------
__device__ __forceinline__ int block_exclusive_scan(int v, int &total)
{
    __shared__ int wsum[kThreads / kWave];
    const int lane = threadIdx.x % kWave;
    const int w = threadIdx.x / kWave;
    int inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    if (lane == kWave - 1) wsum[w] = inc;
    __syncthreads();
    int off = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < kThreads / kWave; ++k) {
        if (k < w) off += wsum[k];
        total += wsum[k];
    }
    __syncthreads();
    return off + inc - v;
}

__global__ __launch_bounds__(kThreads) void k_scan_reduce(const int32_t *__restrict__ in, int m,
                                                          int32_t *__restrict__ partials)
{
    const int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    int s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < m) s += in[base + k];
    int total;
    (void)block_exclusive_scan(s, total);
    if (threadIdx.x == 0) partials[blockIdx.x] = total;
}

__global__ __launch_bounds__(kThreads) void k_scan_partials(int32_t *__restrict__ partials, int np)
{
    int carry = 0;
    for (int base = 0; base < np; base += kThreads) {
        const int i = base + threadIdx.x;
        const int v = i < np ? partials[i] : 0;
        int total;
        const int ex = block_exclusive_scan(v, total);
        if (i < np) partials[i] = carry + ex;
        carry += total;
    }
}

// ... in[0..m) is the bucket counts (m = n_cells + 1, the last bucket the
// dropped particles): also writes the cell ranges and, from the last bucket,
// the particles in cells and the dropped ones to the status words.  FEW: the
// partials are the blocks' sums, not yet scanned (few enough for every block
// to add up those before it, which saves the launch between).
template <bool FEW>
__global__ __launch_bounds__(kThreads) void k_scan_apply(const int32_t *__restrict__ in, int m,
                                                         const int32_t *__restrict__ partials,
                                                         int32_t *__restrict__ out, int32_t *__restrict__ cell_start,
                                                         int32_t *__restrict__ cell_end, int32_t *__restrict__ status)
{
    const int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    int before = 0;
    if constexpr (FEW) {
        int p = 0;
        for (int k = threadIdx.x; k < (int)blockIdx.x; k += kThreads) p += partials[k];
        (void)block_exclusive_scan(p, before);
    } else {
        before = partials[blockIdx.x];
    }
    int v[kScanItems];
    int s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = base + k < m ? in[base + k] : 0;
        s += v[k];
    }
    int total;
    int ex = block_exclusive_scan(s, total) + before;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int c = base + k;
        if (c < m) out[c] = ex;
        if (c < m - 1) {
            cell_start[c] = ex;
            cell_end[c] = ex + v[k];
        } else if (c == m - 1) {
            out[m] = ex + v[k];
            status[SPH_STATUS_N_ACTIVE] = ex;
            status[SPH_STATUS_DROPPED] = v[k];
        }
        ex += v[k];
    }
}

// Place every particle's (type, id) word and index in its bucket's range
// (order inside a bucket as the counting met them).
__global__ __launch_bounds__(kThreads) void k_scatter(int n, const int32_t *__restrict__ cell,
                                                      int cell_base, int n_cells,
                                                      const int32_t *__restrict__ start,
                                                      const uint32_t *__restrict__ place,
                                                      const uint32_t *__restrict__ info,
                                                      uint32_t *__restrict__ keys, uint32_t *__restrict__ index)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int c = cell[i];
    const int b = c >= 0 ? c - cell_base : n_cells;
    const int slot = start[b] + (int)place[i];
    keys[slot] = info[i];
    index[slot] = (uint32_t)i;
}

// Every particle ranks itself in its bucket by its info word (type << 30 |
// id) and is copied to its final position.  Ids are unique; equal words
// (invalid input) are ranked by their slot so the result is a permutation in
// every case.  One lane per position of the scattered order, which is grouped
// by bucket: the lanes of a bucket (about 24) read the same keys at the same
// time.  1.62M particles: 36 us with the copy, against 46 us for a wave per
// bucket and 46 us for a gather and a copy back.
__global__ __launch_bounds__(kThreads) void k_sort_gather(int n, const int32_t *__restrict__ cell, int cell_base,
                                                          int n_cells, const int32_t *__restrict__ start,
                                                          const uint32_t *__restrict__ keys,
                                                          const uint32_t *__restrict__ index,
                                                          const float4 *__restrict__ pos,
                                                          const float4 *__restrict__ vel,
                                                          int32_t *__restrict__ o_cell, float4 *__restrict__ o_pos,
                                                          float4 *__restrict__ o_vel, uint32_t *__restrict__ o_info,
                                                          uint32_t *__restrict__ perm_out,
                                                          uint32_t *__restrict__ neib_count)
{
    const int p = blockIdx.x * kThreads + threadIdx.x;
    if (p >= n) return;
    const uint32_t src = index[p], key = keys[p];
    const int c = cell[src];
    const int b = c >= 0 ? c - cell_base : n_cells;
    const float4 x = pos[src], v = vel[src];
    const int s = start[b], e = start[b + 1];
    int rank = 0;
    for (int t = s; t < e; ++t) {
        const uint32_t k = keys[t];
        rank += (k < key || (k == key && t < p)) ? 1 : 0;
    }
    const int k = s + rank;
    o_cell[k] = c;
    o_pos[k] = x;
    o_vel[k] = v;
    o_info[k] = key;
    if (perm_out) perm_out[k] = src;
    if (c < 0) neib_count[k] = 0u;  // (dropped: in no brick, no neighbours)
}

// The table of bricks with a pair, in order of size (the particles of their
// inner cells), large ones first, bricks of one size class in order of their
// ids: the persistent kernels that take them in that order end with the cheap
// ones, and their work is dealt the same way after every build of the same
// state.  A counting sort over kClasses size classes: per block of bricks a
// histogram, then every block finds its bricks' places from all histograms.  A
// block takes kOrderThreads bricks, or a run of as many tiles of them that
// kOrderBlocks blocks take all: every block reads the histograms of all.
// keys[b]: 0 for a brick without a pair, else 1 + min(particles / width, 62)
// (brick_class); a brick is heavy from class 27 on (12 particles per cell).
// The derivatives of the 1.62M-particle dam break are 2.5% faster in this order
// than with the heavy and the light bricks each in an arbitrary one.
constexpr int kClasses = 64, kHeavyClass = 27, kOrderThreads = 1024, kOrderBlocks = 256;
template <int BX, int BY, int BZ>
__device__ __forceinline__ int brick_class(int particles)
{
    // width of a class: heavy means 12 particles per inner cell
    constexpr int W = 12 * BX * BY * BZ / kHeavyClass;
    static_assert(W * kHeavyClass == 12 * BX * BY * BZ);
    return 1 + min(particles / W, kClasses - 2);
}

__global__ __launch_bounds__(kOrderThreads) void k_order_count(int nb, int tiles, const uint8_t *__restrict__ keys,
                                                               int32_t *__restrict__ hist)
{
    __shared__ int h[kClasses];
    if (threadIdx.x < kClasses) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * tiles * kOrderThreads + threadIdx.x;
    for (int t = 0; t < tiles; ++t) {
        const int64_t b = b0 + (int64_t)t * kOrderThreads;
        const int key = b < nb ? keys[b] : 0;
        if (key) atomicAdd(&h[key], 1);
    }
    __syncthreads();
    if (threadIdx.x < kClasses) hist[blockIdx.x * kClasses + threadIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(kOrderThreads) void k_order_place(int nb, int tiles, const uint8_t *__restrict__ keys,
                                                               const int32_t *__restrict__ hist,
                                                               int32_t *__restrict__ table, int cap_ids)
{
    constexpr int NW = kOrderThreads / kWave;
    static_assert(kClasses == kWave, "one lane per class");
    __shared__ int all[NW][kClasses], before[NW][kClasses], own[NW][kClasses];
    __shared__ int at[kClasses];  // place of the first brick of each class, heavy bricks
    __shared__ int heavy;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    // class `lane`: the bricks of all blocks and of those before this one
    int a = 0, f = 0;
    for (int k = w; k < (int)gridDim.x; k += NW) {
        const int v = hist[k * kClasses + lane];
        a += v;
        f += k < (int)blockIdx.x ? v : 0;
    }
    all[w][lane] = a;
    before[w][lane] = f;
    __syncthreads();
    if (w == 0) {
        int total = 0, first = 0;
        for (int k = 0; k < NW; ++k) {
            total += all[k][lane];
            first += before[k][lane];
        }
        // large classes first: the bricks of the classes above
        int above = total;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int v = __shfl_down(above, o);
            if (lane + o < kWave) above += v;
        }
        at[lane] = above - total + first;
        if (lane == 1 + kHeavyClass) heavy = above;
        if (blockIdx.x == 0) {
            if (lane == 1 + kHeavyClass) table[0] = above;
            const int h = __shfl(above, 1 + kHeavyClass);
            if (lane == 1) table[cap_ids + 1] = above - h;
        }
    }
    for (int t = 0; t < tiles; ++t) {  // uniform
        const int64_t b = ((int64_t)blockIdx.x * tiles + t) * kOrderThreads + threadIdx.x;
        const int key = b < nb ? keys[b] : 0;
        // lanes of the wave with the same class
        unsigned long long same = ~0ull;
#pragma unroll
        for (int bit = 1; bit < kClasses; bit <<= 1) {
            const unsigned long long m = __ballot((key & bit) != 0);
            same &= (key & bit) ? m : ~m;
        }
        own[w][lane] = 0;
        __syncthreads();
        const unsigned long long below = same & ((1ull << lane) - 1ull);
        if (key && below == 0ull) own[w][key] = (int)__popcll(same);
        __syncthreads();
        if (key) {
            int p = at[key] + (int)__popcll(below);
            for (int k = 0; k < w; ++k) p += own[k][key];
            if (p < heavy) table[1 + p] = (int)b;
            else table[cap_ids - (p - heavy)] = (int)b;
        }
        if (t + 1 == tiles) break;  // uniform
        __syncthreads();
        if (w == 0) {  // the places of the next tile
            int sum = 0;
            for (int k = 0; k < NW; ++k) sum += own[k][lane];
            at[lane] += sum;
        }
        __syncthreads();
    }
}

// Neighbour lists, cell-brick form (section "Changing perspective: from the
// particle to the cell": a group of work-items per cell, neighbour data shared
// through on-chip memory).  A workgroup owns a brick of BX x BY x BZ cells, or
// a run of its rows; its work items are the fluid and the boundary centrals of
// each inner cell (inside a cell fluid particles precede boundary ones, so
// boundary centrals, which take no boundary neighbours, have the fluid prefix
// of each cell as candidates).  A wave takes items from a counter.
//
// For its item a wave lists the candidates: the particles of the 27 cells of
// the Moore neighbourhood (z, y, x from -1 to +1), each cell in sorted order.
// The distances of 16 centrals to 16 candidates are a 16 x 4 by 4 x 16 product
// in float32,
//   |o_i|^2 - r_s^2 + |p_j|^2 - 2 o_i . p_j,
// with the offset o_i and the candidate's position p_j = o_j + d cs in the
// frame of the central's cell: one matrix instruction instead of 11 vector
// ones per 64 pairs, and the hit is the sign of the result.  The list predicate
// is a float32 expression of its own (predicate_r2), so a result within a slack
// of zero decides nothing: that pair is evaluated with the predicate itself.
// Both differ from the real r^2 - r_s^2 by rounding: with u = 2^-24,
// S = |cs|^2, |o|^2 <= S/4 and |p|^2 <= 9/4 S,
//   shift of p (1/2 ulp of it, twice)                    6 u S
//   |p|^2, |o|^2 - r_s^2 (3 roundings each)              9 u S
//   four products and sums of at most 4 S                32 u S
//   the predicate: x to 2.5 u |cs|, its square and sum   8 u S
// less than 64 u S together; kSlack = 128 u S.  (Every particle in a cell has
// its offset in that cell, or re-binning has dropped it.)  Places without a
// candidate lie farther away than any r_s whose square is a float.
//
// Lanes 16 g .. 16 g + 15 take quarter g of the candidate list, each lane for
// one central: row 4 g + r of the candidate operand is candidate g Q + 4 t + r
// in tile t, so the four results of a lane are consecutive candidates of its
// quarter, and their signs are shifted into its hit words.  A central's entries
// are then the hits of its four lanes one after the other: after a count over
// the four, each lane writes its own to LDS in scan order, and from there the
// four lanes write both lists in rows of 16 centrals.  Two groups of centrals
// share a candidate operand.  Fluid entries fill the split list from the front
// and boundary entries from the back, in scan order, until M entries are
// written.
//
// The brick-local form of the same lists is for the derivative kernels: entry k
// is the neighbour's slot in the staging order of the central particle's brick
// (cells of the brick and its halo in the Staging order, particles of a cell in
// sorted order), uint16 (slots beyond 65535 as 65535), in scan order with fluid and
// boundary neighbours interleaved as found (entries 0 .. nf+nb-1), stored in groups of 8 per
// particle (brick_entry).
//
// Bound by VALU issue and the latencies between the steps: of the 530 us that
// the scan of the 1.62M-particle dam break takes (92 neighbours a particle, 0.9 GB of
// lists), the vector ALU issues for 330; the lists alone would take 175 at the
// rate of a large copy.  Taking away in turn the writing of the lists, the
// collecting of entries, the products and the positions leaves 450, 335, 215
// and 180 us.  Before, a wave took one central and 64 candidates at a time from
// a brick staged in LDS, with a ballot per central: 721 us (still-water tank of
// 15.5k particles, 27 bricks: 141, now 45; 169k dam break: 180, now 98).
//
// Candidates are listed kList at a time and their positions laid out by
// component kTilesPage tiles at a time.  Rows of a quarter are kRow apart: the
// 64 operands of a tile (16 candidates by 4 components) then lie in 64 places
// of distinct banks, two passes of 32.  Entries are collected kWindow at a time
// (kOut apart per central) in the memory of the positions.
constexpr int kList = 640, kWords = kList / 4 / 32, kTilesPage = 16, kRow = 4 * kTilesPage + 4;
constexpr int kWindow = 128, kOut = kWindow + 8;
constexpr float kSlack = 0x1p-17f, kFarAway = 3e38f;  // (times |cs|^2; |p|^2)
typedef float vf4 __attribute__((ext_vector_type(4)));

template <int BX, int BY, int BZ, int NW>
struct ScanTables {
    static constexpr int S = Staging<BX, BY, BZ>::S, NI = Staging<BX, BY, BZ>::NI;
    struct Wave {
        int4 cell[27];  // of the neighbour cells with candidates: slot of a candidate - its place,
                        // end of the fluid prefix, image code - delta
        alignas(16) union {
            float page[4][4 * kRow];  // x, y, z, |p|^2
            uint16_t out[16][kOut];   // places of a central's neighbours, times 4
        };
        // by place: entry of the split list, slot; [kList]: 0, for the rest of a group
        uint32_t code[kList + 4];
        uint16_t slot[kList + 8];
        alignas(8) uint32_t marks[kList / 32];  // first candidates of a cell, then boundary candidates
    } wave[NW];
    float4 shift[64];  // by the image code: the shift d cs of a candidate
    int base[S + 1], delta[S];  // first slot of each staged cell, slot - particle index
    int fluid_end[S];           // end of the fluid prefix of each staged cell (slot)
    int first[NI + 1];          // first central of each inner cell
    int wsum[NW];
    int item;                 // work items taken
    int most, over;             // most neighbours found, centrals with more than max_neibs
};

struct ScanArgs {
    const float4 *__restrict__ pos;
    float csx, csy, csz, rs2;
    int M;
    uint32_t *__restrict__ neibs;
    uint16_t *__restrict__ neibs_brick;
    uint32_t *__restrict__ neib_count;
};

// The lists of the centrals of one work item (bound: the boundary centrals) of
// staged cell tc: centrals slots q_begin .. q_begin + nq - 1.
template <int BX, int BY, int BZ, int NW>
__device__ __forceinline__ void scan_item(ScanTables<BX, BY, BZ, NW> &T, const ScanArgs &A, int tc, bool bound,
                                          int q_begin, int nq, int &most, int &over)
{
    using St = Staging<BX, BY, BZ>;
    // (opaque: what follows from the lane is computed for each item, not kept in registers across them)
    unsigned lane_bits = threadIdx.x;
    asm volatile("" : "+v"(lane_bits));
    const int lane = lane_bits % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int quarter = lane / 16, m = lane % 16, M = A.M, G = brick_groups(M);
    auto &W = T.wave[wave];
    const float slack = kSlack * (A.csx * A.csx + A.csy * A.csy + A.csz * A.csz);
    const int to_index = __builtin_amdgcn_readfirstlane(-T.delta[tc]);

    auto of_quarter = [&](int v, int q) { return __builtin_amdgcn_ds_bpermute(4 * (16 * q + m), v); };

    // candidate ranges of the 27 cells, lane k < 27 (k = 9 (dz+1) + 3 (dy+1) + dx+1);
    // tables of those that have any, in order
    int beg = 0, len = 0;
    const int dx = lane % 3 - 1, dy = (lane / 3) % 3 - 1, dz = lane / 9 - 1;
    const int t_cell = lane < 27 ? tc + St::step(dx, dy, dz) : tc;
    if (lane < 27) {
        beg = T.base[t_cell];
        len = (bound ? T.fluid_end[t_cell] : T.base[t_cell + 1]) - beg;
    }
    int inc = len;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
        const int v = __builtin_amdgcn_ds_bpermute(4 * (lane - o), inc);
        if (lane >= o) inc += v;
    }
    const int ex = inc - len;
    const int n_cand = __builtin_amdgcn_readlane(inc, 26);
    const int self0 = __builtin_amdgcn_readlane(ex, 13) - __builtin_amdgcn_readlane(beg, 13);  // place - slot
    const uint64_t some = __builtin_amdgcn_ballot_w64(len > 0);
    if (len > 0) {
        const int r = (int)__popcll(some & ((1ull << lane) - 1ull));
        W.cell[r] = make_int4(beg - ex, T.fluid_end[t_cell], (int)(pack_neib(0u, -dx, -dy, -dz) - (uint32_t)T.delta[t_cell]), 0);
    }
    if (lane == 0) W.code[kList] = W.slot[kList] = 0;
    wave_fence();
    bool mixed = false;  // boundary particles among the candidates

    for (int q0 = 0; q0 < nq; q0 += 32) {  // uniform: two groups of 16 centrals
        const bool two = nq - q0 > 16;
        // this lane's central of each group: its index, operand, counts of
        // neighbours found and of fluid ones kept
        int index[2], found[2] = {0, 0}, fluid[2] = {0, 0};
        float bop[2], c_init[2];
        bool has[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int q = q0 + 16 * c + m;
            has[c] = q < nq;
            index[c] = q_begin + min(q, nq - 1) + to_index;
            const float4 o = A.pos[index[c]];
            bop[c] = quarter == 0 ? -2.0f * o.x : quarter == 1 ? -2.0f * o.y : quarter == 2 ? -2.0f * o.z : 1.0f;
            c_init[c] = fmaf(o.x, o.x, fmaf(o.y, o.y, fmaf(o.z, o.z, -A.rs2)));
        }
        for (int pg = 0; pg < n_cand; pg += kList) {  // uniform
            const int np = min(n_cand - pg, kList);
            const int tiles = 4 * ((np + 63) / 64), Q = 4 * tiles;  // of a quarter: Q candidates
            if (q0 == 0 || n_cand > kList) {
                // 1. the list: a mark at the first candidate of each cell but
                //    the first; a candidate's cell is the count of marks up to it
                if (lane < kList / 32) W.marks[lane] = 0u;
                wave_fence();
                const int mark = ex - pg;
                if (len > 0 && mark > 0 && mark < kList) atomicOr(&W.marks[mark >> 5], 1u << (mark & 31));
                wave_fence();
                const uint32_t marks = lane < kList / 32 ? W.marks[lane] : 0u;
                int before = (int)__popcll(__builtin_amdgcn_ballot_w64(len > 0 && mark <= 0)) - 1;
                for (int ch = 0; ch < Q / 16; ++ch) {  // uniform
                    const uint32_t lo = __builtin_amdgcn_readlane(marks, 2 * ch);
                    const uint32_t hi = __builtin_amdgcn_readlane(marks, 2 * ch + 1);
                    const uint64_t mm = ((uint64_t)hi << 32 | lo) >> 1;
                    const int k = __builtin_amdgcn_mbcnt_hi((uint32_t)(mm >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mm, before + (int)(lo & 1u)));
                    before += __popc(lo) + __popc(hi);
                    const int f = 64 * ch + lane;
                    const int4 c = W.cell[k];
                    const int sl = f + pg + c.x;
                    const uint64_t b = __builtin_amdgcn_ballot_w64(f < np && sl >= c.y);
                    mixed |= b != 0;
                    W.code[f] = (uint32_t)(sl + c.z);
                    W.slot[f] = (uint16_t)min(sl, 0xFFFF);
                    if (lane == 0) *(uint64_t *)&W.marks[2 * ch] = b;
                }
                wave_fence();
            }
            // 2. hit words
            uint32_t w[2][kWords];
            const float *mine = &W.page[quarter][m / 4 * kRow + m % 4];
#pragma unroll
            for (int k = 0; k < kWords; ++k) {
                w[0][k] = 0u;
                w[1][k] = 0u;
                if (8 * k >= tiles) continue;  // uniform
                if (k % 2 == 0) {
                    // the positions of the next kTilesPage tiles
                    const int f0 = 32 * k + lane;
                    float4 p[4];
                    uint32_t code[4];
                    bool there[4];  // (no code is free to say so: all 32 bits of an entry are in use)
                    wave_fence();
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int f = g * Q + f0;
                        there[g] = f0 < Q && f < np;
                        code[g] = there[g] ? W.code[f] : 0u;
                        p[g] = there[g] ? A.pos[code[g] & kIndexMask] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    }
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float4 d = T.shift[code[g] >> 26];
                        const float x = p[g].x + d.x, y = p[g].y + d.y, z = p[g].z + d.z;
                        W.page[0][g * kRow + lane] = x;
                        W.page[1][g * kRow + lane] = y;
                        W.page[2][g * kRow + lane] = z;
                        W.page[3][g * kRow + lane] = there[g] ? fmaf(x, x, fmaf(y, y, z * z)) : kFarAway;
                    }
                    wave_fence();
                }
                constexpr int kHalf = 4 * kTilesPage / 2;  // candidates of a quarter in a word
                const float *word = mine + (k % 2) * kHalf;
                float least[2] = {kFarAway, kFarAway};
                const int part = min(tiles - 8 * k, 8);  // 4 or 8
#pragma unroll 1
                for (int b = 0; b < part; b += 4) {      // uniform
                    float aop[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) aop[t] = word[4 * (b + t)];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        if (c == 1 && !two) continue;  // uniform
                        const vf4 c4 = {c_init[c], c_init[c], c_init[c], c_init[c]};
                        vf4 r[4];  // (all four under way before the first is read)
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            r[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[t], bop[c], c4, 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                w[c][k] = __builtin_amdgcn_alignbit(w[c][k], __float_as_uint(r[t][e]), 31);
                            least[c] = fminf(fminf(least[c], fabsf(r[t].x)), fabsf(r[t].y));
                            least[c] = fminf(fminf(least[c], fabsf(r[t].z)), fabsf(r[t].w));
                        }
                    }
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if (c == 1 && !two) continue;  // uniform
                    if (__builtin_amdgcn_ballot_w64(has[c] && least[c] < slack)) {  // uniform, rare
                        // the candidates of the word that are that near
                        const vf4 c4 = {c_init[c], c_init[c], c_init[c], c_init[c]};
                        uint32_t near = 0u;
#pragma unroll 1
                        for (int t = 0; t < part; ++t) {
                            const vf4 r = __builtin_amdgcn_mfma_f32_16x16x4f32(word[4 * t], bop[c], c4, 0, 0, 0);
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                near = __builtin_amdgcn_alignbit(near, __float_as_uint(fabsf(r[e]) - slack), 31);
                        }
                        if (!has[c]) near = 0u;
                        const float4 o = A.pos[index[c]];
                        auto listed = [&](uint32_t bit) {
                            const uint32_t e = W.code[quarter * Q + 32 * k + 4 * part - __ffs((int)bit)];
                            const float4 d = T.shift[e >> 26], p = A.pos[e & kIndexMask];
                            return predicate_r2(o.x, o.y, o.z, p.x, p.y, p.z, -d.x, -d.y, -d.z) < A.rs2 ? bit : 0u;
                        };
                        while (near) {  // two at a time
                            const uint32_t b0 = near & (0u - near), rest = near ^ b0, b1 = rest ? rest & (0u - rest) : b0;
                            near = rest & ~b1;
                            const uint32_t h0 = listed(b0), h1 = listed(b1);
                            w[c][k] = (w[c][k] & ~(b0 | b1)) | h0 | h1;
                        }
                    }
                    if (part == 4) w[c][k] <<= 16;  // (the first candidate of a word is its top bit)
                }
            }
            // 3. entries
#pragma unroll 1
            for (int c = 0; c < (two ? 2 : 1); ++c) {  // uniform
                const int i = c ? index[1] : index[0];
                // the central itself is no neighbour (its place in this
                // quarter; a boundary central is not among its candidates)
                const int self = bound ? -1 : i - to_index + self0 - pg - quarter * Q;
                uint32_t hits[kWords];
                int mine_n = 0;
#pragma unroll
                for (int k = 0; k < kWords; ++k) {
                    hits[k] = c ? w[1][k] : w[0][k];
                    if (self >= 0 && self < Q && self >> 5 == k) hits[k] &= ~(0x80000000u >> (self & 31));
                    if (!(c ? has[1] : has[0])) hits[k] = 0u;
                    mine_n += __popc(hits[k]);
                }
                const int n0 = of_quarter(mine_n, 0), n1 = of_quarter(mine_n, 1), n2 = of_quarter(mine_n, 2),
                          n3 = of_quarter(mine_n, 3);
                const int f0 = c ? found[1] : found[0], f1 = f0 + n0 + n1 + n2 + n3;
                const int from = f0 + (quarter > 0 ? n0 : 0) + (quarter > 1 ? n1 : 0) + (quarter > 2 ? n2 : 0);
                int fluid_c = c ? fluid[1] : fluid[0];
                const int kept = min(f1, M);  // entries f0 .. kept - 1 are written
                uint32_t *tile = A.neibs + (size_t)(i / kWave) * kWave * M + (i % kWave);
                uint4 *lt = A.neibs_brick ? (uint4 *)(A.neibs_brick + brick_entry(i, 0, G)) : nullptr;
                // windows of kWindow entries (one, but for long lists)
                for (int win = f0 & ~(kBrickGroup - 1); __builtin_amdgcn_ballot_w64(win < kept); win += kWindow) {
                    wave_fence();
                    uint16_t *out = &W.out[m][0];
                    if (!__builtin_amdgcn_ballot_w64(f1 - win > kWindow || from < win)) {  // uniform: all in this one
                        uint16_t *to = out + (from - win);
#pragma unroll
                        for (int k = 0; k < kWords; ++k) {
                            const int place = 4 * (quarter * Q + 32 * k);
                            for (uint32_t left = __brev(hits[k]); left; left &= left - 1u)
                                *to++ = (uint16_t)(place + 4 * __builtin_ctz(left));
                        }
                    } else {
                        int at = from - win;
#pragma unroll 1
                        for (int f = 0; f < 32 * kWords; ++f) {
                            uint32_t h = hits[0];
#pragma unroll
                            for (int k = 1; k < kWords; ++k) h = f >> 5 == k ? hits[k] : h;
                            if (!(h << (f & 31) >> 31)) continue;
                            if ((unsigned)at < (unsigned)kWindow) out[at] = (uint16_t)(4 * (quarter * Q + f));
                            ++at;
                        }
                    }
                    wave_fence();
                    // the rest of the last group
                    const int end = kept - win;
                    if (end >= 0 && end < kWindow) {
                        for (int e = end + quarter; e < ((end + kBrickGroup - 1) & ~(kBrickGroup - 1)); e += 4)
                            out[e] = 4 * kList;
                    }
                    wave_fence();
                    const bool plain = !mixed && pg == 0;  // uniform: fluid entries from the first
                    if (plain) fluid_c = kept;
                    const char *codes = (const char *)W.code, *slots = (const char *)W.slot;
#pragma unroll 1
                    for (int g0 = 0; g0 < kWindow; g0 += 4 * kBrickGroup) {
                        if (!__builtin_amdgcn_ballot_w64(win + g0 < kept)) break;  // uniform
                        const int e0 = win + g0 + quarter * kBrickGroup;  // this lane's group of entries
                        const int lo = max(f0 - e0, 0), hi = min(kept - e0, kBrickGroup);  // those of it to write
                        const uint4 grp = *(const uint4 *)(out + g0 + quarter * kBrickGroup);
                        const uint32_t pairs[4] = {grp.x, grp.y, grp.z, grp.w};
                        if (plain) {
                            if (hi > 0) {
                                uint32_t e[kBrickGroup], v[kBrickGroup / 2];
#pragma unroll
                                for (int x = 0; x < kBrickGroup; ++x)
                                    e[x] = *(const uint32_t *)(codes + (x & 1 ? pairs[x / 2] >> 16 : pairs[x / 2] & 0xFFFFu));
                                if (lt) {
#pragma unroll
                                    for (int x = 0; x < kBrickGroup / 2; ++x)
                                        v[x] = *(const uint16_t *)(slots + ((pairs[x] & 0xFFFFu) >> 1)) |
                                               (uint32_t) * (const uint16_t *)(slots + (pairs[x] >> 17)) << 16;
                                    lt[(size_t)(e0 / kBrickGroup) * kWave] = make_uint4(v[0], v[1], v[2], v[3]);
                                }
                                uint32_t *to = tile + (size_t)e0 * kWave;
                                if (__builtin_amdgcn_ballot_w64(hi < kBrickGroup)) {  // uniform
#pragma unroll
                                    for (int x = 0; x < kBrickGroup; ++x)
                                        if (x < hi) to[x * kWave] = e[x];
                                } else {
#pragma unroll
                                    for (int x = 0; x < kBrickGroup; ++x) to[x * kWave] = e[x];
                                }
                            }
                            continue;
                        }
                        uint32_t e[kBrickGroup], v[kBrickGroup / 2] = {}, b_bits = 0u;
#pragma unroll
                        for (int x = 0; x < kBrickGroup; ++x) {
                            const bool in = x >= lo && x < hi;
                            const uint32_t pl = in ? (x & 1 ? pairs[x / 2] >> 16 : pairs[x / 2] & 0xFFFFu) : 4u * kList;
                            e[x] = *(const uint32_t *)(codes + pl);
                            v[x / 2] |= (uint32_t) * (const uint16_t *)(slots + pl / 2) << (x % 2 * 16);
                            b_bits |= (in ? W.marks[pl / 128] >> (pl / 4 % 32) & 1u : 0u) << x;
                        }
                        // boundary entries and entries of the quarters before this one
                        const int nb = __popc(b_bits), nn = max(hi - lo, 0);
                        const int both = nn << 16 | nb;
                        const int s0 = of_quarter(both, 0), s1 = of_quarter(both, 1), s2 = of_quarter(both, 2),
                                  s3 = of_quarter(both, 3);
                        const int pre = (quarter > 0 ? s0 : 0) + (quarter > 1 ? s1 : 0) + (quarter > 2 ? s2 : 0);
                        const int sum = s0 + s1 + s2 + s3;
                        int fl = fluid_c + (pre >> 16) - (pre & 0xFFFF);             // fluid entries before
                        int bo = e0 + lo - fl;                                       // boundary entries before
                        fluid_c += (sum >> 16) - (sum & 0xFFFF);
                        if (hi > lo) {
                            if (lt) {
                                uint4 *to = lt + (size_t)(e0 / kBrickGroup) * kWave;
                                if (lo == 0) {
                                    *to = make_uint4(v[0], v[1], v[2], v[3]);
                                } else {  // the group's first entries are from the page before
#pragma unroll
                                    for (int x = 1; x < kBrickGroup; ++x)
                                        if (x >= lo) ((uint16_t *)to)[x] = (uint16_t)(v[x / 2] >> (x % 2 * 16));
                                }
                            }
#pragma unroll
                            for (int x = 0; x < kBrickGroup; ++x) {
                                if (x < lo || x >= hi) continue;
                                const bool b = b_bits >> x & 1u;
                                tile[(size_t)(b ? M - 1 - bo : fl) * kWave] = e[x];
                                bo += b ? 1 : 0;
                                fl += b ? 0 : 1;
                            }
                        }
                    }
                }
                if (c) {
                    found[1] = f1;
                    fluid[1] = fluid_c;
                } else {
                    found[0] = f1;
                    fluid[0] = fluid_c;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (!has[c] || quarter != 0) continue;
            const int kept = min(found[c], M);
            A.neib_count[index[c]] = (uint32_t)fluid[c] | (uint32_t)(kept - fluid[c]) << 16;
            most = max(most, found[c]);
            over += found[c] > M;
        }
    }
}

// Workgroups of 4 waves, four to a CU (127 VGPRs, 38 KB of LDS), so that the
// ranges of one are read while the others scan.
constexpr int kBuildThreads = 256, kBuildResident = 4;

// The inner cells per workgroup for n bricks of NI cells: a multiple of the 4
// waves that share them, 12, or fewer while two rounds of workgroups take them
// all.  The whole build, by cells per workgroup: 1.62M-particle dam break, 3464
// bricks of 36 cells with a particle: 736 us (36), 671 (18), 641 (12), 687 (9), 719
// (6); 169k dam break, 672 bricks of 18 cells, ten steps with a build: 826
// (18), 777 (9), 759 (6), 758 (3); tank of 27 bricks: 575 (9), 548 (6), 525 (4), 522 (3).
template <int NI>
__device__ __forceinline__ int scan_cells(int n, int resident)
{
    int cells = 12;
    if (n * ((NI + 7) / 8) <= 2 * resident) cells = 8;
    if (n * ((NI + 3) / 4) <= 2 * resident) cells = 4;
    return cells;
}

// One workgroup per part of a brick.
template <int BX, int BY, int BZ, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(kBuildResident))) void k_build_brick(
    ScanArgs A, const uint32_t *__restrict__ info, const int32_t *__restrict__ start, BrickGrid G,
    const int32_t *__restrict__ active, int resident, int32_t *__restrict__ status,
    uint8_t *__restrict__ keys)
{
    using St = Staging<BX, BY, BZ>;
    constexpr int SX = St::SX, SZ = St::SZ, S = St::S, NI = St::NI, IROW = BX * BZ;
    static_assert(S <= NT && NI <= NT, "one thread per cell");
    __shared__ ScanTables<BX, BY, BZ, NT / kWave> T;

    const int tid = threadIdx.x;
    const int cells = scan_cells<NI>(active[0], resident), parts = (NI + cells - 1) / cells;
    if ((int)blockIdx.x >= active[0] * parts) return;
    const int b = active[1 + blockIdx.x / parts];
    const int cx0 = (b % G.nbx) * BX, cy0 = ((b / G.nbx) % G.nby) * BY, cz0 = (b / (G.nbx * G.nby)) * BZ;

    if (tid < 64) {
        auto offset = [](int bits) { return (float)(-((bits & 3) - (bits & 2) * 2)); };
        T.shift[tid] = make_float4(offset(tid) * A.csx, offset(tid >> 2) * A.csy, offset(tid >> 4) * A.csz, 0.0f);
    }

    // ranges of the staged cells and their slots in the brick's staging order
    int st = 0, cnt = 0;
    if (tid < S) {
        int gx = cx0 - 1 + St::sx_of(tid), gy = cy0 - 1 + St::sy_of(tid), gz = cz0 - 1 + St::sz_of(tid);
        const bool ok = wrap_axis(gx, G.nx, G.periodic & 1u) && wrap_axis(gy, G.ny, (G.periodic >> 1) & 1u) &&
                        wrap_axis(gz, G.nz, (G.periodic >> 2) & 1u);
        if (ok) {
            const int lin = gx + G.nx * (gy + G.ny * gz);
            st = start[lin];
            cnt = start[lin + 1] - st;
        }
    }
    int total;
    const int ex = block_scan<NT>(cnt, total, T.wsum);
    if (tid < S) {
        T.base[tid] = ex;
        T.delta[tid] = ex - st;
        T.fluid_end[tid] = ex + cnt;  // lowered below where the cell holds boundary particles
    }
    if (tid == 0) {
        T.base[S] = total;
        T.item = T.most = T.over = 0;
    }
    __syncthreads();
    int icnt = 0;
    // inner cells past the grid edge hold no centrals (on a periodic axis the
    // staged copy would be the wrapped cell, owned by another brick)
    if (tid < NI && cx0 + St::ix_of(tid) < G.nx && cy0 + St::iy_of(tid) < G.ny && cz0 + St::iz_of(tid) < G.nz) {
        const int t = St::inner(tid);
        icnt = T.base[t + 1] - T.base[t];
    }
    int nc;
    const int iex = block_scan<NT>(icnt, nc, T.wsum);
    if (tid < NI) T.first[tid] = iex;
    if (tid == 0) T.first[NI] = nc;

    // the part's inner cells; the fluid prefix of the cells of their rows and
    // the halo of these, half a wave per cell
    const int u0 = (int)blockIdx.x % parts * cells, u1 = min(u0 + cells, NI);
    const int t_end = ((u1 - 1) / IROW + 3) * SX * SZ;
#pragma unroll 4
    for (int t = u0 / IROW * SX * SZ + tid / 32; t < t_end; t += NT / 32) {
        const int s0 = T.base[t], s1 = T.base[t + 1], delta = T.delta[t];
        for (int s2 = s0 + tid % 32; s2 < s1; s2 += 32)
            if (ptype(info[s2 - delta]) == kBoundary) atomicMin(&T.fluid_end[t], s2);
    }
    __syncthreads();

    int most = 0, over = 0;
    for (;;) {
        int item = 0;
        if (tid % kWave == 0) item = atomicAdd(&T.item, 1);
        item = __builtin_amdgcn_readfirstlane(item);
        if (item >= 2 * (u1 - u0)) break;  // uniform
        const int u = u0 + item / 2, tc = St::inner(u);
        const bool bound = item & 1;  // the cell's boundary centrals
        const int all = __builtin_amdgcn_readfirstlane(T.first[u + 1] - T.first[u]);
        if (all == 0) continue;  // uniform
        const int c0 = __builtin_amdgcn_readfirstlane(T.base[tc]), cf = __builtin_amdgcn_readfirstlane(T.fluid_end[tc]);
        const int nq = bound ? c0 + all - cf : cf - c0;
        if (nq > 0) scan_item(T, A, tc, bound, bound ? cf : c0, nq, most, over);
    }

    // the workgroup's share of the status, and the brick's class where it has
    // a pair (one atomic a workgroup: all of them are to the same word)
    if (most) atomicMax(&T.most, most);
    if (over) atomicAdd(&T.over, over);
    __syncthreads();
    if (tid == 0) {
        if (T.most) atomicMax(&status[SPH_STATUS_MAX_NEIBS], T.most);
        if (T.over) atomicAdd(&status[SPH_STATUS_OVERFLOW], T.over);
        if (keys && T.most) keys[b] = (uint8_t)brick_class<BX, BY, BZ>(nc);
    }
}

bool grid_ok(const sph_grid *g, float r_search)
{
    for (int d = 0; d < 3; ++d) {
        if (g->ncell[d] < 1) return false;
        if (!(g->cell_size[d] >= r_search)) return false;
        if (((g->periodic >> d) & 1u) && g->ncell[d] < 3) return false;
    }
    const int64_t nc = (int64_t)g->ncell[0] * g->ncell[1] * g->ncell[2];
    if (nc + 2 > INT32_MAX || g->cell_base < 0 || nc + g->cell_base > INT32_MAX) return false;
    return true;
}

}  // namespace

extern "C" size_t sph_neib_list_entries(int32_t capacity, int32_t max_neibs)
{
    if (capacity < 0 || max_neibs < 0) return 0;
    return (size_t)((capacity + kWave - 1) / kWave) * kWave * (size_t)max_neibs;
}

extern "C" size_t sph_neib_brick_entries(int32_t capacity, int32_t max_neibs)
{
    if (capacity < 0 || max_neibs < 0) return 0;
    // the lists, then the table of bricks with a pair (int32 words)
    return brick_list_entries(capacity, max_neibs) + 2 * brick_table_words(capacity);
}

extern "C" size_t sph_build_workspace_bytes(int32_t capacity, int32_t n_cells)
{
    if (capacity < 0 || n_cells < 0) return 0;
    return build_layout(capacity, n_cells).total;
}

extern "C" int32_t sph_brick_shapes(int32_t *shapes, int32_t max_shapes)
{
    if (shapes)
        for (int k = 0; k < kShapes && k < max_shapes; ++k)
            for (int d = 0; d < 3; ++d) shapes[3 * k + d] = kShapeTable[k][d];
    return kShapes;
}

extern "C" sph_status sph_build_neighbors(const sph_grid *grid, const sph_params *params,
                                          sph_particles *parts, uint32_t *neibs, uint32_t *neib_count,
                                          int32_t max_neibs, int32_t *cell_start, int32_t *cell_end,
                                          int32_t *d_status, uint32_t *perm_out, uint16_t *neibs_brick,
                                          void *workspace, size_t workspace_bytes, void *stream)
{
    if (!grid || !params || !parts || !neibs || !neib_count || !cell_start || !cell_end || !d_status)
        return SPH_ERR_ARG;
    if (parts->n < 0 || parts->capacity < parts->n || parts->capacity > SPH_MAX_CAPACITY) return SPH_ERR_ARG;
    if (parts->capacity > 0 && (!parts->cell || !parts->pos || !parts->vel || !parts->info)) return SPH_ERR_ARG;
    if (max_neibs < 1 || max_neibs > 65535) return SPH_ERR_ARG;
    if (neibs_brick && ((uintptr_t)neibs_brick & 15u)) return SPH_ERR_ARG;  // written in 16-byte groups
    if (!(params->r_search > 0.0f) || !grid_ok(grid, params->r_search)) return SPH_ERR_ARG;
    const int shape = brick_shape_index(grid->brick);
    if (shape < 0) return SPH_ERR_ARG;
    const int n = parts->n;
    const int cap = parts->capacity;
    const int n_cells = grid->ncell[0] * grid->ncell[1] * grid->ncell[2];
    const BuildLayout L = build_layout(cap, n_cells);
    if (!workspace || workspace_bytes < L.total) return SPH_ERR_WORKSPACE;

    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    int32_t *cnt = (int32_t *)(ws + L.cnt);
    int32_t *hist = (int32_t *)(ws + L.hist);
    int32_t *start = (int32_t *)(ws + L.start);
    int32_t *partials = (int32_t *)(ws + L.partials);
    uint32_t *keys = (uint32_t *)(ws + L.keys);
    uint32_t *index = (uint32_t *)(ws + L.index);
    int32_t *t_cell = (int32_t *)(ws + L.t_cell);
    float4 *t_pos = (float4 *)(ws + L.t_pos);
    float4 *t_vel = (float4 *)(ws + L.t_vel);
    uint32_t *place = (uint32_t *)(ws + L.place);
    float4 *pos = (float4 *)parts->pos;
    float4 *vel = (float4 *)parts->vel;

    const CellDims dims{grid->ncell[0], grid->ncell[1], grid->ncell[2], grid->periodic};
    const int nbk = n_cells + 1;

    const int cap_ids = brick_table_cap(cap);
    int32_t *table = neibs_brick ? brick_table(reinterpret_cast<int32_t *>(neibs_brick), cap, max_neibs) : nullptr;
    uint8_t *classes = neibs_brick ? (uint8_t *)(ws + L.classes) : nullptr;
    int32_t *active = (int32_t *)(ws + L.active);
    const int64_t class_words = neibs_brick ? (n_cells + 3) / 4 : 0;  // (at most one brick per cell)
    const unsigned fill_blocks = sph_blocks(nbk, kThreads) < 4096u ? sph_blocks(nbk, kThreads) : 4096u;
    k_build_zero<<<fill_blocks, kThreads, 0, s>>>(nbk, cnt, d_status, class_words, (int32_t *)classes, active);
    SPH_CHECK_LAUNCH();
    if (n > 0) {
        k_rebin_count<<<sph_blocks(n, kThreads), kThreads, 0, s>>>(
            n, parts->cell, pos, vel, dims, grid->cell_size[0], grid->cell_size[1], grid->cell_size[2],
            grid->cell_base, n_cells, cnt, t_cell, t_pos, t_vel, place, d_status);
        SPH_CHECK_LAUNCH();
    }
    const int np = (nbk + kScanTile - 1) / kScanTile;
    k_scan_reduce<<<np, kThreads, 0, s>>>(cnt, nbk, partials);
    if (np <= kFewPartials) {
        k_scan_apply<true><<<np, kThreads, 0, s>>>(cnt, nbk, partials, start, cell_start, cell_end, d_status);
    } else {
        k_scan_partials<<<1, kThreads, 0, s>>>(partials, np);
        k_scan_apply<false><<<np, kThreads, 0, s>>>(cnt, nbk, partials, start, cell_start, cell_end, d_status);
    }
    SPH_CHECK_LAUNCH();
    if (n > 0) {
        k_scatter<<<sph_blocks(n, kThreads), kThreads, 0, s>>>(n, t_cell, grid->cell_base, n_cells, start, place,
                                                                parts->info, keys, index);
        k_sort_gather<<<sph_blocks(n, kThreads), kThreads, 0, s>>>(n, t_cell, grid->cell_base, n_cells, start, keys,
                                                                   index, t_pos, t_vel, parts->cell, pos, vel,
                                                                   parts->info, perm_out, neib_count);
        SPH_CHECK_LAUNCH();
        const float rs2 = params->r_search * params->r_search;
        with_shape(shape, [&]<int BX, int BY, int BZ>() {
            const BrickGrid G = brick_grid<BX, BY, BZ>(grid->ncell, grid->periodic);
            const unsigned bricks = (unsigned)G.nbx * G.nby * G.nbz;
            // a workgroup per part of a brick: which bricks have work (at most
            // one per particle), and so the parts, is known on the device
            constexpr int NI = BX * BY * BZ;
            const int resident = kBuildResident * sph_device_cus(), most = min((int)bricks, n);
            const int items = max(most * ((NI + 11) / 12), min(most * ((NI + 3) / 4), 2 * resident));
            k_active_bricks<BX, BY, BZ><<<sph_blocks(bricks, 256), 256, 0, s>>>(cell_start, cell_end, G, active);
            k_build_brick<BX, BY, BZ, kBuildThreads><<<items, kBuildThreads, 0, s>>>(
                ScanArgs{pos, grid->cell_size[0], grid->cell_size[1], grid->cell_size[2], rs2, max_neibs, neibs,
                         neibs_brick, neib_count},
                parts->info, start, G, active, resident, d_status, classes);
        });
        SPH_CHECK_LAUNCH();
    }
    if (neibs_brick) {
        // the table of bricks with a pair behind the brick-local lists, for
        // the derivative kernels
        with_shape(shape, [&]<int BX, int BY, int BZ>() {
            const BrickGrid G = brick_grid<BX, BY, BZ>(grid->ncell, grid->periodic);
            const int bricks = G.nbx * G.nby * G.nbz;
            const int tiles = ((int)sph_blocks(bricks, kOrderThreads) + kOrderBlocks - 1) / kOrderBlocks;
            const unsigned blocks = sph_blocks(bricks, tiles * kOrderThreads);
            k_order_count<<<blocks, kOrderThreads, 0, s>>>(bricks, tiles, classes, hist);
            k_order_place<<<blocks, kOrderThreads, 0, s>>>(bricks, tiles, classes, hist, table, cap_ids);
        });
        SPH_CHECK_LAUNCH();
    }
    return SPH_OK;
}
