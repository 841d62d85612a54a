// Cell grid and re-sort kernels (Sec. 2.2 GridList, Sec. 3.3 re-sort).
//
// GridList on the GPU: a thread per slot labels it with its cell and takes a
// rank inside the cell with an integer atomic; a scan turns the per-cell counts
// into pointers; ranks place the slots; finally each slot counts the smaller
// ones of its cell, whose number is its stable place, which makes the result
// identical to the sequential counting sort that visits particles in index
// order.
// All passes are integer work and read/write each array once, so they are
// bound by HBM bandwidth.

#include <type_traits>

#include "md_internal.h"

namespace md {

__global__ void k_fill_i32(int32_t* __restrict__ p, int32_t v, int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)ceil_div(count, kStreamBlock)), dim3(kStreamBlock),
                       0, s, p, v, count);
    return hipGetLastError();
}

// Several arrays cleared in one launch.
__global__ __launch_bounds__(kStreamBlock) void k_clear(ClearList l)
{
    int64_t i = (int64_t)blockIdx.x * kStreamBlock + threadIdx.x;
    for (int k = 0; k < ClearList::kMost; ++k) {
        if (i < l.words[k]) {
            l.p[k][i] = 0;
            return;
        }
        i -= l.words[k];
    }
}

hipError_t launch_clear(const ClearList& l, hipStream_t s)
{
    int64_t total = 0;
    for (int k = 0; k < ClearList::kMost; ++k) total += l.words[k];
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear, dim3((unsigned)ceil_div(total, kStreamBlock)), dim3(kStreamBlock), 0, s, l);
    return hipGetLastError();
}

// ---- label + count ---------------------------------------------------------
// Groups of equal cells that a wave looks for.  k_label, us, 1.15 million shuffled
// particles mixed / 62 thousand shuffled / 32 million in cell order: 24 groups 51 /
// 9.7 / 239, 16: 50 / 8.9 / 248, 8: 50 / 8.4 / 300, all (up to 64) 58 / 12.3 / 239.
// Beyond that the atomics bound a shuffled pass, 23 a nanosecond.
constexpr int kLabelGroups = 24;
__global__ __launch_bounds__(kStreamBlock) void k_label(Geo g, const double4* __restrict__ pos,
                                                        int32_t* __restrict__ cell_of,
                                                        int32_t* __restrict__ cell_xyz,
                                                        int32_t* __restrict__ count,
                                                        int32_t* __restrict__ rank,
                                                        int64_t* __restrict__ err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    const double4 p = pos[i];
    const bool inside = p.x >= 0.0 && p.x < g.L[0] && p.y >= 0.0 && p.y < g.L[1] && p.z >= 0.0 &&
                        p.z < g.L[2];
    if (!inside) atomicOr((unsigned long long*)err, 2ull);
    const int cx = cell_coord(p.x, g.inv[0], g.nc[0]);
    const int cy = cell_coord(p.y, g.inv[1], g.nc[1]);
    const int cz = cell_coord(p.z, g.inv[2], g.nc[2]);
    const int32_t c = (cx * g.nc[1] + cy) * g.nc[2] + cz;
    cell_of[i] = c;
    cell_xyz[i] = cx | (cy << 10) | (cz << 20);
    // Slots in cell order (after a re-sort) put runs of equal cells in one
    // wave: the lanes are grouped by cell first, then the first lane of each
    // group adds the group's size with one atomic, all groups' atomics issued
    // together; ranks follow lane order inside a group (the order within a
    // cell is made stable afterwards by k_sort_cells).  Slots in other orders
    // put up to 64 cells in a wave: after kLabelGroups groups the lanes that
    // are left add for themselves.
    uint64_t todo = __ballot(1);
    int leader_of = (int)lane_id();
    uint64_t group = 1ull << leader_of;
    for (int k = 0; todo && k < kLabelGroups; ++k) {
        const int leader = __ffsll((unsigned long long)todo) - 1;
        const int32_t cl = __builtin_amdgcn_readlane(c, leader);
        const uint64_t same = __ballot(c == cl);
        if (c == cl) {
            leader_of = leader;
            group = same;
        }
        todo &= ~same;
    }
    int32_t base = 0;
    if ((int)lane_id() == leader_of) base = atomicAdd(&count[c], (int32_t)__popcll(group));
    base = __shfl(base, leader_of, 64);
    rank[i] = base + (int32_t)mbcnt64(group);
}

// ---- three-phase exclusive scan of int32 (block: 256 threads x 4 items) -----
__device__ __forceinline__ int32_t block_excl_scan_256(int32_t v, int32_t* total)
{
    // inclusive wave scan
    __shared__ int32_t s_wave[kStreamBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    int32_t wbase = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kStreamBlock / 64; ++w) {
        const int32_t t = s_wave[w];
        if (w < wave) wbase += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return wbase + x - v;
}

__global__ __launch_bounds__(kStreamBlock) void k_scan_partial(const int32_t* __restrict__ in, int64_t m,
                                                               int32_t* __restrict__ bsum)
{
    const int64_t base = (int64_t)blockIdx.x * kScanItems + threadIdx.x * 4;
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (base + k < m) s += in[base + k];
    int32_t tot;
    block_excl_scan_256(s, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// one block: exclusive scan of the block sums in place, total into bsum[nb]
__global__ __launch_bounds__(kStreamBlock) void k_scan_bsums(int32_t* __restrict__ bsum, int64_t nb)
{
    const int64_t per = ceil_div(nb, kStreamBlock);
    const int64_t b0 = threadIdx.x * per;
    int32_t s = 0;
    for (int64_t k = 0; k < per; ++k)
        if (b0 + k < nb) s += bsum[b0 + k];
    int32_t tot;
    int32_t run = block_excl_scan_256(s, &tot);
    for (int64_t k = 0; k < per; ++k)
        if (b0 + k < nb) {
            const int32_t v = bsum[b0 + k];
            bsum[b0 + k] = run;
            run += v;
        }
    if (threadIdx.x == 0) bsum[nb] = tot;
}

__global__ __launch_bounds__(kStreamBlock) void k_scan_final(const int32_t* __restrict__ in, int64_t m,
                                                             const int32_t* __restrict__ bsum,
                                                             int64_t nb, int32_t* __restrict__ out)
{
    const int64_t base = (int64_t)blockIdx.x * kScanItems + threadIdx.x * 4;
    int32_t v[4];
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = (base + k < m) ? in[base + k] : 0;
        s += v[k];
    }
    int32_t tot;
    int32_t run = block_excl_scan_256(s, &tot) + bsum[blockIdx.x];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (base + k < m) out[base + k] = run;
        run += v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[m] = bsum[nb];
}

// The same scan in one launch of one block, for grids of up to kScanOneCells, whose
// counts one block reads in one turn (3375 cells: 4.5 us against three launches
// and their gaps; 28^3 cells in three turns 22 us, three launches 13).
constexpr int kScanOneThreads = 1024;
constexpr int kScanOneItems = 8;              // per thread
constexpr int64_t kScanOneCells = kScanOneThreads * kScanOneItems;
__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(const int32_t* __restrict__ in, int m,
                                                              int32_t* __restrict__ out)
{
    __shared__ int32_t s_wave[kScanOneThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int base = (int)threadIdx.x * kScanOneItems;
    int32_t v[kScanOneItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kScanOneItems; ++k) v[k] = base + k < m ? in[base + k] : 0;
#pragma unroll
    for (int k = 0; k < kScanOneItems; ++k) sum += v[k];
    int32_t x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    int32_t run = x - sum, tot = 0;
    for (int w = 0; w < kScanOneThreads / 64; ++w) {
        const int32_t t = s_wave[w];
        if (w < wave) run += t;
        tot += t;
    }
#pragma unroll
    for (int k = 0; k < kScanOneItems; ++k) {
        if (base + k < m) out[base + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0) out[m] = tot;
}

// ---- place + per-cell sort ---------------------------------------------------
__global__ __launch_bounds__(kStreamBlock) void k_scatter(int64_t n, const int32_t* __restrict__ cell_of,
                                                          const int32_t* __restrict__ rank,
                                                          const int32_t* __restrict__ start,
                                                          int32_t* __restrict__ order)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    order[start[cell_of[i]] + rank[i]] = (int32_t)i;
}

// Stable order of each cell's slots (the scatter leaves the groups of different
// waves in atomic order).  The cells of a block, CELLS of them, are
// contiguous in `order`: when their slots fit, they are loaded into LDS, and
// each slot's place in its cell is the number of smaller ones in it (a thread
// per slot, ~11 reads each at rho = 0.5); otherwise the block takes its cells one
// after another (sort_by_cell).  Few cells per block on small grids, which
// otherwise have too few blocks (28^3 cells at 11.7 particles, 64, 32, 16, 8 per
// block: 6.4, 5.1, 4.1, 5.7 us; an insertion sort by a thread per cell of 256
// 17.5), more on larger ones, where a block's three waits cost more (71^3 cells,
// 128 per block 21 us, the insertion sort 23.5; 142^3 cells: 16, 32, 64, 128 per
// block 211, 167, 127, 118 us, the insertion sort 99, which grids of more than
// kSortManyCells therefore take).
constexpr int64_t kSortFewCells = 131072;
constexpr int64_t kSortManyCells = 1048576;
constexpr int kSortLds = 4096;   // slots of one block's cells sorted in LDS

// The same for the cells of a block that are too crowded together (a cutoff of
// ten diameters puts a thousand particles in a cell), by the whole block: a cell
// that fits is ordered in LDS, a larger one from a copy of it in tmp, which a block
// reads through LDS in parts, each thread counting for kSortItems slots at a
// time.  (20,000 particles in 27 cells: 1.6 ms a call of md_bin_cells; an
// insertion sort in global memory by a thread per cell 40.)
constexpr int kSortItems = 4;
__device__ void sort_by_cell(int64_t c0, int nc, const int32_t* __restrict__ start, int32_t* __restrict__ order,
                             int32_t* __restrict__ tmp, int32_t* s_o)
{
    const int tid = threadIdx.x;
    for (int c = 0; c < nc; ++c) {
        const int32_t b = start[c0 + c], len = start[c0 + c + 1] - b;
        if (len < 2) continue;
        __syncthreads();     // the cell before is read
        if (len <= kSortLds) {
            for (int t = tid; t < len; t += kStreamBlock) s_o[t] = order[b + t];
            __syncthreads();
            for (int t = tid; t < len; t += kStreamBlock) {
                const int32_t x = s_o[t];
                int r = 0;
                for (int q = 0; q < len; ++q) r += s_o[q] < x;
                order[b + r] = x;
            }
            continue;
        }
        for (int t = tid; t < len; t += kStreamBlock) tmp[b + t] = order[b + t];
        __syncthreads();
        for (int t0 = 0; t0 < len; t0 += kStreamBlock * kSortItems) {
            int32_t x[kSortItems], r[kSortItems];
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) {
                const int t = t0 + k * kStreamBlock + tid;
                x[k] = tmp[b + (t < len ? t : len - 1)];
                r[k] = 0;
            }
            for (int p0 = 0; p0 < len; p0 += kSortLds) {
                const int part = len - p0 < kSortLds ? len - p0 : kSortLds;
                __syncthreads();
                for (int t = tid; t < part; t += kStreamBlock) s_o[t] = tmp[b + p0 + t];
                __syncthreads();
                for (int q = 0; q < part; ++q) {
                    const int32_t y = s_o[q];
#pragma unroll
                    for (int k = 0; k < kSortItems; ++k) r[k] += y < x[k];
                }
            }
#pragma unroll
            for (int k = 0; k < kSortItems; ++k)
                if (t0 + k * kStreamBlock + tid < len) order[b + r[k]] = x[k];
        }
    }
}

template <int CELLS>
__global__ __launch_bounds__(kStreamBlock) void k_sort_cells(int64_t ncell, const int32_t* __restrict__ start,
                                                             int32_t* __restrict__ order, int32_t* __restrict__ tmp)
{
    __shared__ int32_t s_o[kSortLds];
    __shared__ uint8_t s_c[kSortLds];
    __shared__ int32_t s_start[CELLS + 1];
    const int64_t c0 = (int64_t)blockIdx.x * CELLS;
    const int nc = (int)(c0 + CELLS < ncell ? CELLS : ncell - c0);
    const int tid = threadIdx.x;
    if (tid <= nc) s_start[tid] = start[c0 + tid];
    __syncthreads();
    const int32_t b0 = s_start[0], len = s_start[nc] - b0;
    if (len > kSortLds) {
        sort_by_cell(c0, nc, start, order, tmp, s_o);
        return;
    }
    for (int t = tid; t < len; t += kStreamBlock) s_o[t] = order[b0 + t];
    // kMark threads per cell mark its slots
    constexpr int kMark = kStreamBlock / CELLS;
    const int cm = tid / kMark;
    if (cm < nc)
        for (int t = s_start[cm] - b0 + tid % kMark; t < s_start[cm + 1] - b0; t += kMark) s_c[t] = (uint8_t)cm;
    __syncthreads();
    for (int t = tid; t < len; t += kStreamBlock) {
        const int32_t x = s_o[t];
        const int c = s_c[t], q0 = s_start[c] - b0, q1 = s_start[c + 1] - b0;
        int r = 0;
        for (int q = q0; q < q1; ++q) r += s_o[q] < x;
        order[b0 + q0 + r] = x;
    }
}

// A thread per cell, which sorts its slots in LDS by insertion (the groups that
// the scatter leaves are nearly in order).
__device__ __forceinline__ void insertion_sort(int32_t* v, int32_t len)
{
    for (int32_t k = 1; k < len; ++k) {
        const int32_t x = v[k];
        int32_t p = k;
        bool more = true;
        while (more) {
            const int32_t y = v[p - 1];
            more = y > x;
            if (more) v[p] = y;
            p -= more ? 1 : 0;
            more &= p > 0;
        }
        v[p] = x;
    }
}

__global__ __launch_bounds__(kStreamBlock) void k_sort_cells_by_thread(int64_t ncell, const int32_t* __restrict__ start,
                                                                       int32_t* __restrict__ order,
                                                                       int32_t* __restrict__ tmp)
{
    __shared__ int32_t s_o[kSortLds];
    const int64_t c0 = (int64_t)blockIdx.x * kStreamBlock;
    const int64_t c1 = c0 + kStreamBlock < ncell ? c0 + kStreamBlock : ncell;
    const int64_t c = c0 + threadIdx.x;
    const int32_t b0 = start[c0], len = start[c1] - b0;
    if (len > kSortLds) {
        sort_by_cell(c0, (int)(c1 - c0), start, order, tmp, s_o);
        return;
    }
    for (int32_t t = threadIdx.x; t < len; t += kStreamBlock) s_o[t] = order[b0 + t];
    __syncthreads();
    if (c < c1) insertion_sort(s_o + (start[c] - b0), start[c + 1] - start[c]);
    __syncthreads();
    for (int32_t t = threadIdx.x; t < len; t += kStreamBlock) order[b0 + t] = s_o[t];
}

// ---- the same for small systems in one block --------------------------------
// Label, count (LDS atomics), exclusive scan, place and the stable order in one
// launch of one block: the same count, start, cell_of, cell_xyz and
// order as the kernels above, without their launches, which dominate
// a rebuild of a few thousand particles.  Cells and ranks stay in registers, the
// unsorted order in LDS.  (4,000 particles: 23 us with ranks and order in global
// memory and an insertion sort there, 8 here; beyond kBinSmallN one compute
// unit is too few: 62,000 particles took 196 us so.)
constexpr int kBinSmallThreads = 1024;
constexpr int64_t kBinSmallN = 16384;
constexpr int64_t kBinSmallCells = 4096;

template <int ITEMS>
__global__ __launch_bounds__(kBinSmallThreads) void k_bin_small(Geo g, const double4* __restrict__ pos,
                                                                int32_t* __restrict__ cell_of,
                                                                int32_t* __restrict__ cell_xyz,
                                                                int32_t* __restrict__ count,
                                                                int32_t* __restrict__ start,
                                                                int32_t* __restrict__ order,
                                                                int64_t* __restrict__ err)
{
    static_assert(kBinSmallCells <= 4096 && ITEMS * kBinSmallThreads <= 65536, "cell and rank share a word");
    __shared__ int32_t s_cnt[kBinSmallCells + 1];
    __shared__ int32_t s_wave[kBinSmallThreads / 64];
    __shared__ uint16_t s_ord[ITEMS * kBinSmallThreads];
    const int tid = threadIdx.x;
    const int nc = (int)g.ncell;
    const int n = (int)g.n;
    for (int c = tid; c < nc; c += kBinSmallThreads) s_cnt[c] = 0;
    __syncthreads();
    bool outside = false;
    uint32_t item[ITEMS];     // cell | rank << 12
    constexpr int B = 4;      // positions in flight per thread
#pragma unroll
    for (int k0 = 0; k0 < ITEMS; k0 += B) {
        double4 p[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const int i = tid + (k0 + k) * kBinSmallThreads;
            p[k] = pos[i < n ? i : n - 1];
        }
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const int i = tid + (k0 + k) * kBinSmallThreads;
            item[k0 + k] = 0;
            if (i >= n) continue;
            outside |= !(p[k].x >= 0.0 && p[k].x < g.L[0] && p[k].y >= 0.0 && p[k].y < g.L[1] && p[k].z >= 0.0 &&
                         p[k].z < g.L[2]);
            const int cx = cell_coord(p[k].x, g.inv[0], g.nc[0]);
            const int cy = cell_coord(p[k].y, g.inv[1], g.nc[1]);
            const int cz = cell_coord(p[k].z, g.inv[2], g.nc[2]);
            const int32_t c = (cx * g.nc[1] + cy) * g.nc[2] + cz;
            cell_of[i] = c;
            cell_xyz[i] = cx | (cy << 10) | (cz << 20);
            item[k0 + k] = (uint32_t)c | (uint32_t)atomicAdd(&s_cnt[c], 1) << 12;
        }
    }
    if (outside) atomicOr((unsigned long long*)err, 2ull);
    __syncthreads();
    // exclusive scan of the counts: each thread takes a contiguous run of
    // cells, then a scan of the runs' totals over the block
    const int per = (nc + kBinSmallThreads - 1) / kBinSmallThreads;
    const int c0 = min(tid * per, nc), c1 = min(c0 + per, nc);
    int32_t run = 0;
    for (int c = c0; c < c1; ++c) run += s_cnt[c];
    const int lane = tid & 63, wave = tid >> 6;
    int32_t x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    int32_t base = x - run;
    for (int w2 = 0; w2 < wave; ++w2) base += s_wave[w2];
    for (int c = c0; c < c1; ++c) {
        const int32_t v = s_cnt[c];
        count[c] = v;
        start[c] = base;
        s_cnt[c] = base;
        base += v;
    }
    if (tid == 0) {
        start[nc] = n;
        s_cnt[nc] = n;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = tid + k * kBinSmallThreads;
        if (i < n) s_ord[s_cnt[item[k] & 4095u] + (int)(item[k] >> 12)] = (uint16_t)i;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = tid + k * kBinSmallThreads;
        if (i >= n) continue;
        const int q0 = s_cnt[item[k] & 4095u], q1 = s_cnt[(item[k] & 4095u) + 1];
        int r = 0;
        for (int q = q0; q < q1; ++q) r += (int)s_ord[q] < i;
        order[q0 + r] = i;
    }
}

bool bin_clears_counts(const Geo& g) { return !(g.n <= kBinSmallN && g.ncell <= kBinSmallCells); }

hipError_t launch_bin(const Geo& g, const double* pos, const md_cells& cells, void* ws,
                      const WsLayout& L, int64_t* err_flags, hipStream_t s)
{
    char* w = (char*)ws;
    int32_t* rank = (int32_t*)(w + L.rank);
    int32_t* bsum = (int32_t*)(w + L.bsum);
    if (!bin_clears_counts(g)) {
        if (g.n <= 4 * kBinSmallThreads)
            hipLaunchKernelGGL((k_bin_small<4>), dim3(1), dim3(kBinSmallThreads), 0, s, g, (const double4*)pos,
                               cells.cell_of, cells.cell_xyz, cells.count, cells.start, cells.order, err_flags);
        else
            hipLaunchKernelGGL((k_bin_small<16>), dim3(1), dim3(kBinSmallThreads), 0, s, g, (const double4*)pos,
                               cells.cell_of, cells.cell_xyz, cells.count, cells.start, cells.order, err_flags);
        return hipGetLastError();
    }
    const unsigned nbn = (unsigned)ceil_div(g.n, kStreamBlock);
    hipLaunchKernelGGL(k_label, dim3(nbn), dim3(kStreamBlock), 0, s, g, (const double4*)pos,
                       cells.cell_of, cells.cell_xyz, cells.count, rank, err_flags);
    if (g.ncell <= kScanOneCells) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanOneThreads), 0, s, (const int32_t*)cells.count, (int)g.ncell,
                           cells.start);
    } else {
        const int64_t nbs = ceil_div(g.ncell, kScanItems);
        hipLaunchKernelGGL(k_scan_partial, dim3((unsigned)nbs), dim3(kStreamBlock), 0, s,
                           (const int32_t*)cells.count, g.ncell, bsum);
        hipLaunchKernelGGL(k_scan_bsums, dim3(1), dim3(kStreamBlock), 0, s, bsum, nbs);
        hipLaunchKernelGGL(k_scan_final, dim3((unsigned)nbs), dim3(kStreamBlock), 0, s,
                           (const int32_t*)cells.count, g.ncell, (const int32_t*)bsum, nbs, cells.start);
    }
    hipLaunchKernelGGL(k_scatter, dim3(nbn), dim3(kStreamBlock), 0, s, g.n,
                       (const int32_t*)cells.cell_of, (const int32_t*)rank,
                       (const int32_t*)cells.start, cells.order);
    auto sort = [&](auto cells_per_block) {
        constexpr int CELLS = decltype(cells_per_block)::value;
        hipLaunchKernelGGL((k_sort_cells<CELLS>), dim3((unsigned)ceil_div(g.ncell, CELLS)), dim3(kStreamBlock), 0, s,
                           g.ncell, (const int32_t*)cells.start, cells.order, rank);   // (ranks are read)
    };
    if (g.ncell <= kSortFewCells) sort(std::integral_constant<int, 16>());
    else if (g.ncell <= kSortManyCells) sort(std::integral_constant<int, 128>());
    else
        hipLaunchKernelGGL(k_sort_cells_by_thread, dim3((unsigned)ceil_div(g.ncell, kStreamBlock)), dim3(kStreamBlock),
                           0, s, g.ncell, (const int32_t*)cells.start, cells.order, rank);
    return hipGetLastError();
}

// ---- local (cell-corner) coordinates for the mixed-precision force -----------
// l = x - c * cs, taken as the periodic image nearest the cell, rounded to FP32.
__device__ __forceinline__ float local_coord(double x, int c, double cs, double L, double invL)
{
    double l = x - (double)c * cs;
    l -= L * rint((l - 0.5 * cs) * invL);
    return (float)l;
}

// ---- re-sort: gather every per-particle array into cell order ---------------
__global__ __launch_bounds__(kStreamBlock) void k_resort(Geo g, const int32_t* __restrict__ order,
                                                         const double4* __restrict__ pos,
                                                         const double* __restrict__ vel,
                                                         const int32_t* __restrict__ id,
                                                         double4* __restrict__ pos_alt,
                                                         double* __restrict__ vel_alt,
                                                         int32_t* __restrict__ id_alt,
                                                         double* __restrict__ pos_ref,
                                                         float4* __restrict__ pos32,
                                                         int32_t* __restrict__ cell_of,
                                                         int32_t* __restrict__ cell_xyz)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= g.n) return;
    const int64_t n = g.n;
    const int64_t src = order[k];
    const double4 p = pos[src];
    pos_alt[k] = p;
    vel_alt[k] = vel[src];
    vel_alt[n + k] = vel[n + src];
    vel_alt[2 * n + k] = vel[2 * n + src];
    id_alt[k] = id[src];
    pos_ref[k] = p.x;
    pos_ref[n + k] = p.y;
    pos_ref[2 * n + k] = p.z;
    const int cx = cell_coord(p.x, g.inv[0], g.nc[0]);
    const int cy = cell_coord(p.y, g.inv[1], g.nc[1]);
    const int cz = cell_coord(p.z, g.inv[2], g.nc[2]);
    cell_of[k] = (cx * g.nc[1] + cy) * g.nc[2] + cz;
    cell_xyz[k] = cx | (cy << 10) | (cz << 20);
    if (pos32) {
        pos32[k] = make_float4(local_coord(p.x, cx, g.cs[0], g.L[0], g.invL[0]),
                               local_coord(p.y, cy, g.cs[1], g.L[1], g.invL[1]),
                               local_coord(p.z, cz, g.cs[2], g.L[2], g.invL[2]),
                               __int_as_float(cx | (cy << 10) | (cz << 20)));
    }
}

hipError_t launch_resort(const Geo& g, const int32_t* order, const double* pos, const double* vel,
                         const int32_t* id, double* pos_alt, double* vel_alt, int32_t* id_alt,
                         double* pos_ref, float* pos32, int32_t* cell_of, int32_t* cell_xyz,
                         hipStream_t s)
{
    hipLaunchKernelGGL(k_resort, dim3((unsigned)ceil_div(g.n, kStreamBlock)), dim3(kStreamBlock), 0, s, g,
                       order, (const double4*)pos, vel, id, (double4*)pos_alt, vel_alt, id_alt, pos_ref,
                       (float4*)pos32, cell_of, cell_xyz);
    return hipGetLastError();
}

// ---- user [n][3] coordinates -> [n][4] slots, folded into the box ------------
__device__ __forceinline__ double fold(double x, double L, double invL)
{
    double y = x - L * floor(x * invL);
    if (y >= L) y -= L;
    if (y < 0.0) y += L;
    return y;
}

__global__ __launch_bounds__(kStreamBlock) void k_pack(Geo g, const double* __restrict__ q,
                                                       double4* __restrict__ pos)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    pos[i] = make_double4(fold(q[3 * i], g.L[0], g.invL[0]), fold(q[3 * i + 1], g.L[1], g.invL[1]),
                          fold(q[3 * i + 2], g.L[2], g.invL[2]), 0.0);
}

hipError_t launch_pack(const Geo& g, const double* q, double* pos, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack, dim3((unsigned)ceil_div(g.n, kStreamBlock)), dim3(kStreamBlock), 0, s, g, q,
                       (double4*)pos);
    return hipGetLastError();
}

// ---- order of the slots ------------------------------------------------------
// By one block: how far apart in space slots lie that follow one another, as the
// squared distance of their cells (periodic, at most 64), summed over
// kSpreadSamples pairs spread over the slots.
__device__ void sample_spread(const Geo& g, const int32_t* __restrict__ cell_xyz, int64_t* out)
{
    __shared__ int s_sum[kStreamBlock / 64];
    auto gap = [](int a, int b, int nc) {
        const int d = abs(a - b);
        return min(d, nc - d);
    };
    int sum = 0;
#pragma unroll
    for (int t = 0; t < kSpreadSamples / kStreamBlock; ++t) {
        const int64_t i = (int64_t)(t * kStreamBlock + (int)threadIdx.x) * (g.n - 1) / kSpreadSamples;
        const int32_t a = cell_xyz[i], b = cell_xyz[i + 1 < g.n ? i + 1 : i];
        const int dx = gap(a & 1023, b & 1023, g.nc[0]), dy = gap((a >> 10) & 1023, (b >> 10) & 1023, g.nc[1]);
        const int dz = gap((a >> 20) & 1023, (b >> 20) & 1023, g.nc[2]);
        sum += min(dx * dx + dy * dy + dz * dz, 64);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        sum = 0;
        for (int w = 0; w < kStreamBlock / 64; ++w) sum += s_sum[w];
        out[0] = sum;
    }
}

// the same, and a flag word cleared
__global__ __launch_bounds__(kStreamBlock) void k_spread(Geo g, const int32_t* __restrict__ cell_xyz,
                                                         int64_t* __restrict__ flag, int64_t* __restrict__ out)
{
    if (threadIdx.x == 0) flag[0] = 0;
    sample_spread(g, cell_xyz, out);
}

hipError_t launch_spread(const Geo& g, const int32_t* cell_xyz, int64_t* flag, int64_t* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_spread, dim3(1), dim3(kStreamBlock), 0, s, g, cell_xyz, flag, out);
    return hipGetLastError();
}

// ---- reference positions (and local coordinates) without a re-sort ----------
// spread: the order of the slots, too, by the first block (or nullptr)
__global__ __launch_bounds__(kStreamBlock) void k_ref_copy(Geo g, const double4* __restrict__ pos,
                                                           const int32_t* __restrict__ cell_xyz,
                                                           double* __restrict__ pos_ref,
                                                           float4* __restrict__ pos32, int64_t* __restrict__ spread)
{
    if (spread && blockIdx.x == 0) sample_spread(g, cell_xyz, spread);
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= g.n) return;
    const int64_t n = g.n;
    const double4 p = pos[k];
    if (pos_ref) {
        pos_ref[k] = p.x;
        pos_ref[n + k] = p.y;
        pos_ref[2 * n + k] = p.z;
    }
    if (pos32) {
        const int32_t c = cell_xyz[k];
        pos32[k] = make_float4(local_coord(p.x, c & 1023, g.cs[0], g.L[0], g.invL[0]),
                               local_coord(p.y, (c >> 10) & 1023, g.cs[1], g.L[1], g.invL[1]),
                               local_coord(p.z, (c >> 20) & 1023, g.cs[2], g.L[2], g.invL[2]), __int_as_float(c));
    }
}

// Positions of the current slots into a trajectory frame in the particles'
// original order: frame[id[s]] = pos[s] (x, y, z, 0).
__global__ __launch_bounds__(kStreamBlock) void k_record(int64_t n, const double4* __restrict__ pos,
                                                         const int32_t* __restrict__ id, double4* __restrict__ frame,
                                                         RunIo run)
{
    const int64_t s = (int64_t)blockIdx.x * kStreamBlock + threadIdx.x;
    if (run.idx > 0 && (run.slots ? run_stopped(run, run_check_load(run)) : run.gate[0] != 0)) return;
    if (s >= n) return;
    const double4 p = pos[s];
    frame[id[s]] = make_double4(p.x, p.y, p.z, 0.0);
}

hipError_t launch_record(const Geo& g, const double* pos, const int32_t* id, double* frame, hipStream_t s,
                         const RunIo& run)
{
    hipLaunchKernelGGL(k_record, dim3((unsigned)ceil_div(g.n, kStreamBlock)), dim3(kStreamBlock), 0, s, g.n,
                       (const double4*)pos, id, (double4*)frame, run);
    return hipGetLastError();
}

hipError_t launch_ref_copy(const Geo& g, const double* pos, const int32_t* cell_xyz, double* pos_ref,
                           float* pos32, int64_t* spread, hipStream_t s)
{
    hipLaunchKernelGGL(k_ref_copy, dim3((unsigned)ceil_div(g.n, kStreamBlock)), dim3(kStreamBlock), 0, s,
                       g, (const double4*)pos, cell_xyz, pos_ref, (float4*)pos32, spread);
    return hipGetLastError();
}

}  // namespace md
