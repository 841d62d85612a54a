// Pair-list construction (Sec. 2.3 bookkeeping with search length rs; Sec. 2.4
// key-sorted list), one 64-lane wavefront per cell (or, for the tiled list of
// a large grid, per tile of cells built one after another).
//
// The wave stages the particles of the 27 surrounding cells (~300 at
// rho = 0.5) in its registers, one candidate per lane per 64-chunk.  It then
// walks the keys of its own cell: each lane tests its candidates against the
// key with the exact FP64 predicate, a ballot gives the passing lanes, and the
// prefix popcount below each lane gives its output position, so every row is
// written compactly in candidate order (the key's own cell first, then the
// neighbour cells of stencil codes 14 .. 26 and 0 .. 12, each in ascending
// slot) with no atomics.  Rows of one cell are packed one after another into the
// cell's block of the list; the block base is the cell id times a fixed stride,
// so cells never have to wait for each other (tiled lists pool the blocks of a
// tile's cells, below).
//
// The work is ALU bound (about 300 FP64 distance tests per particle at
// rho = 0.5); small grids are bound by one wave's walk over its keys.

#include <cmath>
#include <type_traits>

#include "md_internal.h"

namespace md {

struct BuildArgs {
    const double4* pos;
    const int32_t* start;
    const int32_t* count;
    const int32_t* order;   // nullptr when the slots are already in cell order
    int32_t nc[3];
    int64_t ncell;
    double L[3], invL[3];
    double rs2;
    int32_t exact_all;
    int64_t stride;
    uint32_t* nbr;
    int64_t* offsets;
    int32_t* counts;
    int32_t* cell_rows;
    int64_t* status;
    int32_t tc;                       // tiled: cells per tile along z
    unsigned long long* tile_max;     // tiled: atomic max of the staged count per tile
    FastDiv div_nz;                   // division by nz and by kBuildStrip * ny (cell order decode)
    FastDiv div_strip;
    FastDiv div_tc;                   // tiled: division by tc
    int32_t nt;                       // tiled: tiles per column
    int32_t* tile_used;               // tiled: entries taken so far in each tile's pooled block
    int64_t ntile;                    // tiled: tiles in all
    FastDiv div_nt;                   // tiled: division by nt (tile order decode)
};

// r^2 of the pinned predicate: d = q_j - q_i, optional minimum image,
// r2 = fma(dz, dz, fma(dy, dy, dx * dx)).
template <bool MINIMG>
__device__ __forceinline__ double pair_r2(const BuildArgs& a, double xj, double yj, double zj, double xi,
                                          double yi, double zi)
{
    double dx = xj - xi, dy = yj - yi, dz = zj - zi;
    if (MINIMG) {
        // one component after another (scheduling barriers): interleaved,
        // their temporaries would set the kernel's register count
        dx = dx - a.L[0] * rint(dx * a.invL[0]);
        __builtin_amdgcn_sched_barrier(0);
        dy = dy - a.L[1] * rint(dy * a.invL[1]);
        __builtin_amdgcn_sched_barrier(0);
        dz = dz - a.L[2] * rint(dz * a.invL[2]);
    }
    return __builtin_fma(dz, dz, __builtin_fma(dy, dy, __dmul_rn(dx, dx)));
}

// Inclusive prefix sums by DPP lane moves (no LDS round trips): over each row
// of 16 lanes (Hillis-Steele shifts by 1, 2, 4, 8; lanes shifted in from
// outside the row read 0), and over lanes 0 .. 31 (row 1 then adds lane 15).
constexpr int kDppRowShr = 0x110;     // row_shr:n is kDppRowShr + n
constexpr int kDppRowBcast15 = 0x142;
__device__ __forceinline__ int scan_row16(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 1, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 2, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 4, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 8, 0xF, 0xF, true);
    return v;
}
__device__ __forceinline__ int scan_lanes32(int v)
{
    v = scan_row16(v);
    // rows 1 and 3 take lane 15 of the row below; rows 0 and 2 add nothing
    return v + __builtin_amdgcn_update_dpp(0, v, kDppRowBcast15, 0xA, 0xF, false);
}

// Row header of one key.  When the cell block overflows, the row is clipped to
// the entries actually stored, so an invalid (overflowed) list still only
// references written, in-range entries.
__device__ __forceinline__ void write_row(const BuildArgs& a, int32_t kslot, int64_t base, int64_t used,
                                          int64_t wpos, int64_t cap)
{
    const int64_t start = used < cap ? used : cap;
    const int64_t room = cap - start;
    a.offsets[kslot] = base + start;
    a.counts[kslot] = (int32_t)(wpos < room ? wpos : room);
}

constexpr int kMaxOwn = 64;     // own-cell particles kept in LDS for the key loop (all in the first chunk)

// The neighbour cells in candidate order: rank 0 is the own cell (stencil code
// 13), ranks 1 .. 13 codes 14 .. 26, ranks 14 .. 26 codes 0 .. 12, so that the
// candidates of a half row (own cell, codes 14 .. 26) are the first 14 ranks.
// Code (sx+1)*9 + (sy+1)*3 + (sz+1) for the offsets s in {-1, 0, 1}^3.
__device__ __forceinline__ int code_of_rank(int r) { return r < 14 ? r + 13 : r - 14; }
#ifndef MD_BUILD_STRIP
#define MD_BUILD_STRIP 8
#endif
constexpr int kBuildStrip = MD_BUILD_STRIP;   // x-columns per strip of the cell order

// Tiled (16-bit) rows start at even entries, so the force pass can read two
// entries with one 32-bit load; the entry after a row of odd length holds the
// tile's stand-in partner.  Slot-entry rows are packed.
template <typename E>
__device__ __forceinline__ uint32_t row_start(uint32_t end)
{
    return sizeof(E) == 2 ? (end + 1u) & ~1u : end;
}

#ifndef MD_BUILD_ROWBUF
#define MD_BUILD_ROWBUF 768
#endif
constexpr int kRowBuf = MD_BUILD_ROWBUF;

// Words of a wave's row buffer in LDS.  The cell's buffers first hold the
// candidate table (6 bytes per candidate).  One wave per cell (W = 1): 16-bit
// entries with the smallest register set of candidates sized so that the
// block's LDS stays within 5 KB (32 blocks, 8 waves per SIMD), with the
// larger ones so that the rows of a cell of that neighbourhood usually fit.
// Four waves per cell: a wave's quarter of the keys.
template <int NCH, int W, typename E>
constexpr int rowbuf_words()
{
    if (W > 1) return (NCH <= 8 ? 512 : (NCH <= 12 ? 640 : 960)) * (sizeof(E) == 2 ? 1 : 2);
    if (sizeof(E) == 2) return NCH <= 6 ? 608 : (NCH <= 8 ? kRowBuf : (NCH <= 12 ? 1216 : 1984));
    return NCH * 96 > kRowBuf ? NCH * 96 : kRowBuf;
}
template <int NCH, int W, typename E>
constexpr uint32_t rowbuf_entries()
{
    return (uint32_t)(rowbuf_words<NCH, W, E>() * (4 / sizeof(E)));
}

// Keys of one cell against candidates held in registers: NACT chunks of 64
// (the cell's neighbourhood rounded up; the key loop is instantiated per
// chunk count, so the unrolled chunk sequence carries no branch).  Empty
// candidate slots carry a NaN x coordinate, so r2 < rs2 fails for them in
// both the plain and the minimum-image form of the test.  The own cell's
// particles come first among the candidates, so the key itself is candidate
// self_t < 64 of the first chunk, and only that chunk needs the test that
// drops it.  Output positions come from mbcnt of the row mask, counted on from
// the row's start.
//
// Half rows (HALF): the candidates are the own cell (ascending slots), then
// the cells of codes 14 .. 26, so "partner slot > key slot in the own cell" is
// "candidate number > self_t"; candidates up to self_t are dropped.
//
// Fast form (the key's row surely fits in the LDS row buffer): the row mask is
// the ballot of the distance test (minus the key's own lane in the first
// chunk), and the lanes in it store under that mask as the execution mask, at
// byte offsets formed by one shift-add from mbcnt (the mask moves to the
// scalar unit, which has room here, while the vector unit, which bounds the
// build, saves the select of a spare address per chunk).  The drop test is
// one vector compare of the lane against the key's place (a scalar mask built
// from that place would cost several scalar instructions).
template <bool MINIMG, int NACT, typename E, bool HALF>
__device__ __forceinline__ uint32_t row_staged(const BuildArgs& a, int lane, const double4& kp, int self_t, uint32_t w0,
                                               const double* cx, const double* cy, const double* cz,
                                               const uint32_t* meta, E* s_rows)
{
    constexpr int kShift = sizeof(E) == 2 ? 1 : 2;
    uint32_t wpos = w0;
#pragma unroll
    for (int ch = 0; ch < NACT; ++ch) {
        const double r2 = pair_r2<MINIMG>(a, cx[ch], cy[ch], cz[ch], kp.x, kp.y, kp.z);
        const bool in = r2 < a.rs2;
        uint64_t m = __builtin_amdgcn_ballot_w64(in);
        if (ch == 0) m &= ~__builtin_amdgcn_ballot_w64(HALF ? lane <= self_t : lane == self_t);
        if (__builtin_amdgcn_inverse_ballot_w64(m))
            *(E*)((char*)s_rows + ((mbcnt64(m) << kShift) + (wpos << kShift))) = (E)meta[ch];
        wpos += (uint32_t)__popcll(m);
    }
    return wpos;
}

// The same row past the buffer: counted only (STORE = false), or written to
// dst[w0 ..] where below cap (packed rows of slot entries go to the row buffer
// lds while below room).
template <bool MINIMG, int NACT, typename E, bool HALF, bool STORE>
__device__ __forceinline__ uint32_t row_direct(const BuildArgs& a, int lane, const double4& kp, int self_t, uint32_t w0,
                                               const double* cx, const double* cy, const double* cz,
                                               const uint32_t* meta, E* dst, uint32_t cap, E* lds, uint32_t room)
{
    uint32_t wpos = w0;
#pragma unroll
    for (int ch = 0; ch < NACT; ++ch) {
        const double r2 = pair_r2<MINIMG>(a, cx[ch], cy[ch], cz[ch], kp.x, kp.y, kp.z);
        const bool drop = ch == 0 && (HALF ? lane <= self_t : lane == self_t);
        const bool in = r2 < a.rs2 && !drop;
        const uint64_t m = __builtin_amdgcn_ballot_w64(in);
        if (STORE) {
            const uint32_t w = mbcnt64(m) + wpos;
            if (in) {
                if (lds && w < room) lds[w] = (E)meta[ch];
                else if (w < cap) dst[w] = (E)meta[ch];
            }
        }
        wpos += (uint32_t)__popcll(m);
    }
    return wpos;
}

// A cell's slice of its tile's pool: one atomic add on the tile's counter when
// every cell has waves of its own; when one wave builds the tile's cells one
// after another (SEQ), the slices follow in cell order and the wave keeps the
// running offset itself.
template <bool SEQ>
__device__ __forceinline__ uint32_t reserve_slice(int lane, int32_t* tile_used, uint32_t seq_base, uint32_t used)
{
    if (SEQ) return seq_base;
    uint32_t base = 0;
    if (lane == 0) base = (uint32_t)atomicAdd(tile_used, (int32_t)used);
    return __builtin_amdgcn_readfirstlane(base);
}

// What the row makers need of one cell.
template <typename E>
struct CellRows {
    int lane, wave;
    int T, own_cnt;
    const double4* key;      // the cell's particles, w = slot
    E* rows;                 // this wave's row buffer
    uint32_t* wused;         // W > 1: entries of each wave, then the cell's slice
    E* blk;                  // tiled: the tile's pool; slots: the cell's block
    uint64_t cap;            // entries of it
    int32_t* tile_used;      // tiled: entries taken in the pool
    uint32_t seq_base;       // tiled, SEQ: the cell's slice
    uint32_t pad;            // tiled: the stand-in that follows rows of odd length
};

// Rows of one cell and their headers, by W waves (wave w makes the rows of the
// w-th part of the keys).  A wave stages its rows in LDS while they surely fit
// (a row adds at most T - 1 entries).  With one wave, rows of slot entries past
// the buffer go straight to the cell block.  Otherwise the rest is counted,
// the waves' totals give each its place in the cell's slice, and the rows past
// the buffer are computed again straight into it.  Tiled rows: the cells of a
// tile share one pooled block of tile_cells * cell_stride 16-bit entries (the
// first cell's block and those after it), of which a cell takes a slice once
// its total is known, so the pool has to hold the tile's total rather than
// every cell the largest cell's rows.  Returns the entries the cell takes.
template <bool MINIMG, int NACT, int NCH, typename E, bool HALF, bool SEQ, int W>
__device__ __forceinline__ uint32_t rows_from_registers(const BuildArgs& a, const CellRows<E>& r, const double* cx,
                                                       const double* cy, const double* cz, const uint32_t* meta)
{
    constexpr bool TILED = sizeof(E) == 2;
    constexpr uint32_t ROOM = rowbuf_entries<NCH, W, E>();
    const int lane = r.lane;
    const int per = W > 1 ? (r.own_cnt + W - 1) / W : r.own_cnt;
    const int k0 = W > 1 ? min(r.wave * per, r.own_cnt) : 0, k1 = min(k0 + per, r.own_cnt);
    uint32_t used = 0;
    uint32_t my_end = 0;     // lane j: end of the row of key k0 + j, counted from the first row of the wave
    int kk = k0;
    for (; kk < k1 && used + (uint32_t)r.T <= ROOM; ++kk) {
        used = row_staged<MINIMG, NACT, E, HALF>(a, lane, r.key[kk], kk, used, cx, cy, cz, meta, r.rows);
        my_end = lane == kk - k0 ? used : my_end;
        used = row_start<E>(used);
    }
    const int ks = kk;
    // the stand-ins that follow the staged rows of odd length
    if (TILED && k0 + lane < ks && (my_end & 1u)) r.rows[my_end] = (E)r.pad;
    uint32_t staged = used;
    constexpr bool PACKED = !TILED && W == 1;
    for (; kk < k1; ++kk) {
        used = row_direct<MINIMG, NACT, E, HALF, PACKED>(a, lane, r.key[kk], kk, used, cx, cy, cz, meta, r.blk,
                                                         (uint32_t)r.cap, r.rows, ROOM);
        my_end = lane == kk - k0 ? used : my_end;
        used = row_start<E>(used);
    }
    uint32_t total = used, first = 0, base = 0;
    if constexpr (W > 1) {
        if (lane == 0) r.wused[r.wave] = used;
        __syncthreads();
        total = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t u = r.wused[w];
            if (w < r.wave) first += u;
            total += u;
        }
        if constexpr (TILED) {
            if (r.wave == 0) base = reserve_slice<false>(lane, r.tile_used, 0u, total);
            if (threadIdx.x == 0) r.wused[W] = base;
            __syncthreads();
            base = r.wused[W];
        }
    } else if constexpr (TILED) {
        base = reserve_slice<SEQ>(lane, r.tile_used, r.seq_base, used);
        __syncthreads();
    } else {
        staged = min(used, ROOM);
        __syncthreads();
    }
    const bool fits = (uint64_t)base + total <= r.cap;
    if (TILED && !fits && threadIdx.x == 0) atomicOr((unsigned long long*)&a.status[2], 1ull);
    E* dst = r.blk + base + first;
    const uint32_t room = fits ? total - first : (uint32_t)(r.cap > first ? r.cap - first : 0);   // slots: clipped
    if constexpr (TILED) {
        if (fits) {
            // base, first and staged are even and the pool starts 4-byte aligned
            uint32_t* dst2 = (uint32_t*)dst;
            const uint32_t* src2 = (const uint32_t*)r.rows;
            for (uint32_t t = lane; 2 * t < staged; t += 64) dst2[t] = src2[t];
        }
    } else {
        for (uint32_t t = lane; t < min(staged, room); t += 64) dst[t] = r.rows[t];
    }
    if (!PACKED && (!TILED || fits)) {
        uint32_t w = staged;
        for (int k2 = ks; k2 < k1; ++k2) {
            w = row_direct<MINIMG, NACT, E, HALF, true>(a, lane, r.key[k2], k2, w, cx, cy, cz, meta, dst, room, nullptr,
                                                        0u);
            if (TILED && lane == 0 && (w & 1u)) dst[w] = (E)r.pad;
            w = row_start<E>(w);
        }
    }
    const uint32_t prev = __shfl_up(my_end, 1, 64);
    if (k0 + lane < k1) {
        const int k2 = k0 + lane;
        const uint32_t end = my_end, beg = lane > 0 ? row_start<E>(prev) : 0u;
        const int32_t kslot = (int32_t)__double_as_longlong(r.key[k2].w);
        if constexpr (TILED) {
            // an overflowed cell (list invalid) keeps in-range, empty rows
            a.offsets[kslot] = (int64_t)((fits ? dst : r.blk) - (E*)a.nbr) + (fits ? beg : 0u);
            a.counts[kslot] = fits ? (int32_t)(end - beg) : 0;
        } else {
            write_row(a, kslot, (int64_t)(r.blk - (E*)a.nbr), first + beg, end - beg, (int64_t)r.cap);
        }
    }
    return total;
}

// The key loop for the cell's chunk count nact in [1, NCH], instantiated for
// the chunk counts LOW, LOW + STEP, ... and NCH (the counts that the register
// set's neighbourhoods usually have; chunks past T hold no candidate).
template <int LOW, int STEP, bool MINIMG, int NCH, typename E, bool HALF, bool SEQ, int W>
__device__ __forceinline__ uint32_t rows_for_chunks(int nact, const BuildArgs& a, const CellRows<E>& r,
                                                   const double* cx, const double* cy, const double* cz,
                                                   const uint32_t* meta)
{
    if constexpr (LOW < NCH) {
        if (nact <= LOW) return rows_from_registers<MINIMG, LOW, NCH, E, HALF, SEQ, W>(a, r, cx, cy, cz, meta);
        return rows_for_chunks<LOW + STEP, STEP, MINIMG, NCH, E, HALF, SEQ, W>(nact, a, r, cx, cy, cz, meta);
    } else {
        return rows_from_registers<MINIMG, NCH, NCH, E, HALF, SEQ, W>(a, r, cx, cy, cz, meta);
    }
}

// Same rows, by one wave, candidates re-read from memory for every key
// (neighbourhoods with more than NCH*64 particles or cells with more than 64).
// COUNT: only the rows' total (with the even starts of 16-bit rows) is
// returned, nothing is written.
template <bool MINIMG, typename E, bool HALF, bool COUNT = false>
__device__ __forceinline__ uint32_t rows_from_memory(const BuildArgs& a, E* blk, uint32_t stride, int T, int own_start,
                                     int own_cnt, const int* s_pref, const int* s_nstart, const int* s_lbase,
                                     uint32_t pad)
{
    uint32_t used = 0;
    for (int kk = 0; kk < own_cnt; ++kk) {
        const int kidx = own_start + kk;
        const int32_t kslot = a.order ? a.order[kidx] : kidx;
        const double4 kp = a.pos[kslot];
        uint32_t wpos = 0;
        for (int t0 = 0; t0 < T; t0 += 64) {
            const int t = t0 + (int)lane_id();
            bool pass = false;
            uint32_t meta = 0;
            if (t < T) {
                int q = 0;
#pragma unroll
                for (int h = 16; h > 0; h >>= 1)
                    if (q + h < 27 && s_pref[q + h] <= t) q += h;
                const int idx = s_nstart[q] + (t - s_pref[q]);
                const int32_t slot = a.order ? a.order[idx] : idx;
                const double4 p = a.pos[slot];
                const double r2 = pair_r2<MINIMG>(a, p.x, p.y, p.z, kp.x, kp.y, kp.z);
                // q ranks the neighbour cells (rank 0 the own cell)
                pass = r2 < a.rs2 && (HALF ? (q > 0 || slot > kslot) : slot != kslot);
                meta = s_lbase ? (uint32_t)(s_lbase[q] + (t - s_pref[q])) << 4
                               : (uint32_t)slot | ((uint32_t)code_of_rank(q) << kCodeShift);
            }
            const uint64_t m = __ballot(pass);
            const uint32_t w = used + wpos + mbcnt64(m);
            if (!COUNT && pass && w < stride) blk[w] = (E)meta;
            wpos += (uint32_t)__popcll(m);
        }
        if (!COUNT && lane_id() == 0) {
            write_row(a, kslot, (int64_t)(blk - (E*)a.nbr), used, wpos, stride);
            if (sizeof(E) == 2 && ((used + wpos) & 1u) && used + wpos < stride) blk[used + wpos] = (E)pad;
        }
        used = row_start<E>(used + wpos);
    }
    return used;
}

// What a tiled build takes from the cell's tile: its z range, the pooled block
// of its list (the first cell's block and the blocks after it) and, for lane
// q < 27 (neighbour cell q, in column q / 3 of the tile's 3 x 3 columns), the
// two offsets that turn the start of that neighbour cell into the staged index
// of its first particle in the tile's neighbourhood: the staged layout is the 9
// column runs one after another (exclusive prefix of the run lengths), and a
// run that wraps around the box has a second segment.
struct TileCtx {
    int z0 = 0, z1 = 0, jw = 0;
    int offA = 0, offB = 0;
    uint32_t pad = 0;            // the stand-in partner of the force pass (staged total << 4)
    uint32_t total = 0;          // staged particles of the tile's neighbourhood
    uint16_t* tblk = nullptr;
    uint64_t tcap = 0;
    int32_t* tused = nullptr;    // entries taken so far in the tile's pool
    int64_t tile = 0;
};

// Lanes 0..8 hold the run of column `lane` as tile_run_load gives it.
__device__ __forceinline__ TileCtx tile_ctx(const BuildArgs& a, int cx, int cy, int tz, int z0, int z1,
                                            const TileRun& run)
{
    const int lane = (int)lane_id();
    TileCtx t;
    t.z0 = z0;
    t.z1 = z1;
    t.jw = tile_jw(z0, z1, a.nc[2]);
    const int len = lane < 9 ? run.lenA + run.lenB : 0;
    const int inc = scan_row16(len);
    t.total = (uint32_t)__builtin_amdgcn_readlane(inc, 8);
    const int col = lane < 27 ? code_of_rank(lane) / 3 : 0;
    const int cbase = __shfl(inc - len, col, 64);
    const int sA = __shfl(run.sA, col, 64), lenA = __shfl(run.lenA, col, 64), sB = __shfl(run.sB, col, 64);
    t.offA = cbase - sA;
    t.offB = cbase + lenA - sB;
    t.pad = t.total << 4;
    const int64_t colc = (int64_t)cx * a.nc[1] + cy;
    t.tblk = (uint16_t*)a.nbr + (colc * a.nc[2] + z0) * a.stride;
    t.tcap = (uint64_t)(z1 - z0) * (uint64_t)a.stride;
    t.tile = colc * a.nt + tz;
    t.tused = a.tile_used + t.tile;
    return t;
}

// The rows of one cell (cx, cy, cz), from the starts and counts of its 27
// neighbour cells (lane q < 27 holds those of cell q; half rows use q >= 13
// only).  Tiled: the cell's slice of the tile's pool is reserved by an atomic
// add or, SEQ, starts at seq_base.  Returns the entries the cell takes.
template <int NCH, bool TILED, bool HALF, bool SEQ, int W>
__device__ __forceinline__ uint32_t build_cell(const BuildArgs& a, int cx, int cy, int cz, int st_l, int cnt_l,
                                               const TileCtx& tx, uint32_t seq_base)
{
    using E = typename std::conditional<TILED, uint16_t, uint32_t>::type;
    int lane = (int)lane_id();
    // opaque to the compiler when a wave builds several cells: the per-lane
    // addresses below are then formed per cell instead of being hoisted out of
    // the cell loop into registers that stay live across it
    if (SEQ) asm volatile("" : "+v"(lane));
    const int wave = W > 1 ? (int)(threadIdx.x >> 6) : 0;
    const int nx = a.nc[0], ny = a.nc[1], nz = a.nc[2];
    const int64_t c = ((int64_t)cx * ny + cy) * nz + cz;

    __shared__ int s_nstart[27];
    __shared__ int s_pref[28];
    __shared__ double4 s_key[kMaxOwn];
    // rows of the waves' keys before the block is written (and two words of
    // margin); before that, the candidate table
    constexpr int kRows = rowbuf_words<NCH, W, E>();
    __shared__ __align__(8) uint32_t s_rows[W * kRows + 2];
    __shared__ uint32_t s_wused[W + 1];
    __shared__ int s_lbase[27];
    const bool has_nb = lane < 27 && (!HALF || lane <= 13);
    const int st = has_nb ? st_l : 0, cnt = has_nb ? cnt_l : 0;
    const int incl = scan_lanes32(cnt);
    if (lane < 27) {
        s_nstart[lane] = st;
        s_pref[lane + 1] = incl;
    }
    if (lane == 0) s_pref[0] = 0;
    int lb = 0;   // tiled: staged index of the first particle of this lane's cell
    if (TILED && lane < 27) {
        const int j = cz + code_of_rank(lane) % 3 - tx.z0;   // place of the neighbour cell in its column run
        lb = st + (j < tx.jw ? tx.offA : tx.offB);
        s_lbase[lane] = lb;
    }
    __syncthreads();

    const int T = s_pref[27];
    const uint32_t pad = TILED ? tx.pad : 0u;
    const int own_start = s_nstart[0];
    const int own_cnt = s_pref[1];   // the own cell's particles are the first candidates
    const bool minimg = a.exact_all || cx == 0 || cx == nx - 1 || cy == 0 || cy == ny - 1 || cz == 0 ||
                        cz == nz - 1;
    E* blk = (E*)a.nbr + c * a.stride;
    // capped so that byte offsets (entries << 2) fit in 32 bits
    const uint32_t stride = (uint32_t)(a.stride < (1 << 29) ? a.stride : (1 << 29));
    uint32_t used = 0;

    if (own_cnt > 0 && T <= NCH * 64 && own_cnt <= kMaxOwn) {
        // candidate table: for entry t, the candidate's position in the cell
        // order and (16 bits) its staged index in the tile's neighbourhood
        // (tiled) or its stencil code, written by the lane of its cell; it
        // lives in the row buffer, which is free until the rows are made
        static_assert(NCH * 64 * (sizeof(uint32_t) + sizeof(uint16_t)) <= sizeof(uint32_t) * (W * kRows + 2),
                      "table fits the row buffer");
        uint32_t* s_tpos = s_rows;
        uint16_t* s_tcode = reinterpret_cast<uint16_t*>(s_rows + NCH * 64);
        // two lanes of each wave per neighbour cell (lanes q and q + 32 for
        // q < 27), each writing every other entry of the wave's share of it
        {
            const int q = lane & 31;
            const int t0 = __shfl(incl - cnt, q, 64), stq = __shfl(st, q, 64), cq = __shfl(cnt, q, 64);
            const int eq = TILED ? __shfl(lb, q, 64) : code_of_rank(q);
            if (q < 27) {
                for (int i = (lane >> 5) + 2 * wave; i < cq; i += 2 * W) {
                    s_tpos[t0 + i] = (uint32_t)(stq + i);
                    s_tcode[t0 + i] = (uint16_t)(TILED ? eq + i : eq);
                }
            }
        }
        __syncthreads();
        double px[NCH], py[NCH], pz[NCH];
        uint32_t meta[NCH];
        const double qnan = __longlong_as_double(0x7FF8000000000000LL);
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            px[ch] = py[ch] = pz[ch] = qnan;
            meta[ch] = 0;
            if (ch * 64 >= T) continue;          // uniform: chunk beyond the neighbourhood
            const int tq = ch * 64 + lane;
            const int te = min(tq, T - 1);   // in-range entry; discarded if tq >= T
            const uint32_t ex = s_tpos[te], ey = s_tcode[te];
            const uint32_t slot = a.order ? (uint32_t)a.order[ex] : ex;
            // (slots are below 2^27: a 32-bit byte offset from a uniform base)
            const double4 p = *(const double4*)((const char*)a.pos + (slot << 5));
            // a NaN x alone fails the distance test in both forms of it
            px[ch] = p.x;
            if ((ch + 1) * 64 > T) px[ch] = tq < T ? p.x : qnan;   // (uniform condition)
            py[ch] = p.y;
            pz[ch] = p.z;
            meta[ch] = TILED ? ey << 4 : ((uint32_t)slot | (ey << kCodeShift));
            if (ch == 0 && tq < own_cnt) s_key[tq] = make_double4(p.x, p.y, p.z, __longlong_as_double((long long)slot));
        }
        __syncthreads();
        const int nact = (T + 63) >> 6;
        CellRows<E> r;
        r.lane = lane;
        r.wave = wave;
        r.T = T;
        r.own_cnt = own_cnt;
        r.key = s_key;
        r.rows = reinterpret_cast<E*>(s_rows + wave * kRows);
        r.wused = s_wused;
        r.blk = TILED ? (E*)tx.tblk : blk;
        r.cap = TILED ? tx.tcap : (uint64_t)stride;
        r.tile_used = tx.tused;
        r.seq_base = seq_base;
        r.pad = pad;
        // four waves per cell (small grids, most of whose cells touch the box
        // faces) always take minimum images, which change nothing elsewhere
        constexpr int LOW = NCH <= 6 ? 1 : (NCH <= 8 ? (W > 1 ? 4 : 1) : (NCH <= 12 ? 8 : 14)), STEP = NCH <= 12 ? 1 : 2;
        if (W > 1 || minimg)
            used = rows_for_chunks<LOW, STEP, true, NCH, E, HALF, SEQ, W>(nact, a, r, px, py, pz, meta);
        else
            used = rows_for_chunks<LOW, STEP, W == 1 ? false : true, NCH, E, HALF, SEQ, W>(nact, a, r, px, py, pz, meta);
    } else if (own_cnt > 0 && wave == 0) {
        if constexpr (TILED) {
            // count the rows, take the cell's slice of the tile's pool, write
            const uint32_t total =
                minimg ? rows_from_memory<true, E, false, true>(a, nullptr, 0, T, own_start, own_cnt, s_pref,
                                                                s_nstart, s_lbase, pad)
                       : rows_from_memory<false, E, false, true>(a, nullptr, 0, T, own_start, own_cnt, s_pref,
                                                                 s_nstart, s_lbase, pad);
            const uint32_t base = reserve_slice<SEQ>(lane, tx.tused, seq_base, total);
            const bool fits = (uint64_t)base + total <= tx.tcap;
            if (!fits && lane == 0) atomicOr((unsigned long long*)&a.status[2], 1ull);
            // an overflowed cell writes empty rows (capacity 0)
            E* cblk = (E*)(fits ? tx.tblk + base : tx.tblk);
            const uint32_t cap = fits ? total : 0u;
            if (minimg)
                rows_from_memory<true, E, false>(a, cblk, cap, T, own_start, own_cnt, s_pref, s_nstart, s_lbase, pad);
            else
                rows_from_memory<false, E, false>(a, cblk, cap, T, own_start, own_cnt, s_pref, s_nstart, s_lbase, pad);
            used = total;
        } else {
            used = minimg ? rows_from_memory<true, E, HALF>(a, blk, stride, T, own_start, own_cnt, s_pref, s_nstart,
                                                            nullptr, pad)
                          : rows_from_memory<false, E, HALF>(a, blk, stride, T, own_start, own_cnt, s_pref,
                                                             s_nstart, nullptr, pad);
        }
    }
    if (lane == 0 && wave == 0) {
        a.cell_rows[c] = used > 0x7FFFFFFFu ? 0x7FFFFFFF : (int32_t)used;
        if (!TILED && used > stride) atomicOr((unsigned long long*)&a.status[2], 1ull);
    }
    return used;
}

// Waves per SIMD that the registers must leave room for.  Rebuild's list, us, at
// this bound and at others: wave per tile, 6 chunks (142^3 cells) 7 waves 4880,
// 6 5160, 8 5100, unbounded (92 registers, 5) 5480; wave per cell, 6 chunks
// (71^3) 8 waves 644, 7 664; 8 chunks (28^3) 6 or 7 waves 75, 5 78, and with all
// 8 chunks in use (1M at density 0.8) 298 and 278; 12 chunks (256k at 0.8) 5
// waves 101, 4 105.
template <int NCH, bool SEQ, int W>
constexpr int build_waves_per_simd()
{
    if (NCH == 6) return SEQ ? 7 : 8;
    return NCH == 8 ? 6 : (NCH == 12 && W == 1 ? 5 : 1);
}

// One wave per cell (four on small grids, whose cells alone would leave most of
// the GPU idle while each wave walks its cell's keys), or (SEQ, tiled lists of
// large grids) one wave per tile that builds the tile's cells one after another
// along z: the cells' slices of the tile's pool then follow in cell order with
// no atomic, the tile's runs and staged layout are worked out once, and the next
// cell's neighbour starts and counts load while a cell is built.
template <int NCH, bool TILED, bool HALF, bool SEQ, int W>
__global__ __launch_bounds__(64 * W, (build_waves_per_simd<NCH, SEQ, W>())) void k_build(BuildArgs a)
{
    static_assert(!SEQ || (TILED && !HALF && W == 1), "tile-sequential builds write tiled full rows");
    const int64_t tb = xcd_remap(blockIdx.x, gridDim.x);
    if (tb >= (SEQ ? a.ntile : a.ncell)) return;
    const int lane = (int)(threadIdx.x & 63);
    const int nx = a.nc[0], ny = a.nc[1], nz = a.nc[2];
    // cells (tiles) in strips of kBuildStrip x-columns walked along y (a
    // column's cells consecutive), so that cells built close in time share
    // their neighbour cells in L2 (ids < 2^31: 32-bit arithmetic, divisions
    // by the launch's multiply-shift divisors)
    const uint32_t t = (uint32_t)tb;
    const uint32_t seq = fdiv(t, SEQ ? a.div_nt : a.div_nz);
    const int zi = (int)(t - seq * (uint32_t)(SEQ ? a.nt : nz));   // the tile along z (SEQ), else the cell's z
    const uint32_t strip = fdiv(seq, a.div_strip);
    const uint32_t in = seq - strip * (uint32_t)(kBuildStrip * ny);
    const int sw = min(kBuildStrip, nx - (int)strip * kBuildStrip);
    uint32_t cyu;
    if (sw == kBuildStrip) cyu = in / (uint32_t)kBuildStrip;   // a power of two
    else cyu = in / (uint32_t)sw;                              // the last, narrower strip
    const int cy = (int)cyu, cx = (int)(strip * kBuildStrip + (in - cyu * (uint32_t)sw));

    // Every lane issues its loads before any result is used (a wait inside a
    // branch would serialise them): the neighbour cell of lanes 0..26, and,
    // tiled, the cells at the ends of the tile's column runs (lanes 0..8);
    // lanes without one load cell 0.  Half rows take candidates from the own
    // cell (code 13) and codes 14 .. 26 only: the other 13 cells count as empty.
    const bool has_nb = lane < 27 && (!HALF || lane <= 13);
    const int code = code_of_rank(lane);   // lanes 0 .. 26: the neighbour cells in candidate order
    int colb = 0;                          // first cell of the lane's neighbour column
    if (lane < 27) {
        const int ax = wrap_cell(cx + code / 9 - 1, nx), ay = wrap_cell(cy + (code / 3) % 3 - 1, ny);
        colb = (ax * ny + ay) * nz;
    }
    const int dz = code % 3 - 1;
    const int tz = SEQ ? zi : (TILED ? (int)fdiv((uint32_t)zi, a.div_tc) : 0);
    const int z0 = tz * a.tc, z1 = TILED ? min(z0 + a.tc, nz) : 0;
    const int cz0 = SEQ ? z0 : zi;   // the (first) cell built
    const int nb = has_nb ? colb + wrap_cell(cz0 + dz, nz) : 0;
    TileCells tcl;
    if (TILED) tcl = tile_run_cells(wrap_cell(cx + lane / 3 - 1, nx), wrap_cell(cy + lane % 3 - 1, ny), ny, nz, z0, z1,
                                    lane < 9);
    int st_l = a.start[nb], cnt_l = a.count[nb];
    TileRun run = {0, 0, 0, 0};
    if (TILED) run = tile_run_load(a.start, a.count, tcl);
    TileCtx tx;
    if (TILED) {
        tx = tile_ctx(a, cx, cy, tz, z0, z1, run);
        if (threadIdx.x == 0 && cz0 == z0)
            atomicMax(a.tile_max + (tx.tile & (kTileMaxSlots - 1)), (unsigned long long)tx.total);
    }
    if constexpr (!SEQ) {
        build_cell<NCH, TILED, HALF, false, W>(a, cx, cy, cz0, st_l, cnt_l, tx, 0u);
    } else {
        uint32_t off = 0;
        for (int cz = z0; cz < z1; ++cz) {
            // the next cell's neighbour starts and counts, loaded while this
            // cell is built
            int st_n = 0, cnt_n = 0;
            if (cz + 1 < z1) {
                const int nbn = has_nb ? colb + wrap_cell(cz + 1 + dz, nz) : 0;
                st_n = a.start[nbn];
                cnt_n = a.count[nbn];
            }
            off += build_cell<NCH, true, false, true, 1>(a, cx, cy, cz, st_l, cnt_l, tx, off);
            st_l = st_n;
            cnt_l = cnt_n;
            __syncthreads();
        }
        if (lane == 0) tx.tused[0] = (int32_t)off;
    }
}

// Four waves per cell up to this many cells.  Time of a rebuild's list (build
// and statistics, us, one / four waves per cell): 343 cells at 12 particles
// each 31.0 / 25.5, 343 at 32 each 49.8 / 32.4, 64 at 32 each 69.7 / 37.8;
// 2744 cells at 12 each 36.3 / 39.2, 3375 at 19 each 56.4 / 63.7: beyond about
// a thousand the cells' own waves fill the SIMDs, and four times the candidate
// loads cost more than the shorter key walks save.
constexpr int64_t kWideCells = 1024;


void build_clears(const Geo& g, const md_pairlist& list, void* ws, const WsLayout& L, bool tiled,
                  unsigned long long* tile_max, ClearList& c)
{
    c.add(list.status, 8);
    if (tiled) {
        c.add(tile_max, 2 * kTileMaxSlots);
        c.add((char*)ws + L.tile_used, g.ntile);
    }
}

hipError_t launch_build(const Geo& g, double rs, const double* pos, const md_cells& cells,
                        const md_pairlist& list, void* ws, const WsLayout& L, bool tiled, bool half,
                        unsigned long long* tile_max, int waves, const GatherIo* gather, hipStream_t s)
{
    int32_t* tile_used = (int32_t*)((char*)ws + L.tile_used);
    BuildArgs a;
    a.pos = (const double4*)pos;
    a.start = cells.start;
    a.count = cells.count;
    a.order = cells.sorted ? nullptr : cells.order;
    for (int k = 0; k < 3; ++k) {
        a.nc[k] = g.nc[k];
        a.L[k] = g.L[k];
        a.invL[k] = g.invL[k];
    }
    a.ncell = g.ncell;
    a.rs2 = rs * rs;
    a.exact_all = g.exact_all;
    a.stride = list.cell_stride;
    a.nbr = list.nbr;
    a.offsets = list.offsets;
    a.counts = list.counts;
    a.cell_rows = (int32_t*)((char*)ws + L.cell_rows);
    a.status = list.status;
    a.tc = g.tc;
    a.tile_max = tile_max;
    a.div_nz = make_fastdiv((uint32_t)g.nc[2]);
    a.div_strip = make_fastdiv((uint32_t)(kBuildStrip * g.nc[1]));
    a.div_tc = make_fastdiv((uint32_t)(g.tc > 0 ? g.tc : 1));
    a.nt = g.nt;
    a.tile_used = tile_used;
    a.ntile = g.ntile;
    a.div_nt = make_fastdiv((uint32_t)(g.nt > 0 ? g.nt : 1));
    if (tiled && (half || !cells.sorted || g.tc <= 0 || !tile_max)) return hipErrorInvalidValue;
    // candidates held in registers: the fewest chunks of 64 (fewer registers,
    // more waves per SIMD) that a neighbourhood far in the tail at the mean
    // density needs (4 standard deviations of a Poisson count above the mean,
    // 2 where that takes a larger set than 8 chunks: a liquid dense enough for
    // it fluctuates far less); larger neighbourhoods take the path that
    // re-reads memory for every key (11k particles at density 0.8, 690
    // candidates per cell: 600 us per build on that path, 50 with the set of
    // 12 chunks and one wave per cell; 256k at 0.8: 526 and 113 us; 1M at 0.8,
    // 477 candidates: 303 us with 8 chunks and the few larger cells on that
    // path, 520 with 12 chunks for all)
    const double mean_t = (half ? 14.0 : 27.0) * (double)g.n / (double)g.ncell, dev_t = std::sqrt(mean_t);
    const double most4 = mean_t + 4.0 * dev_t, most2 = mean_t + 2.0 * dev_t;
    const int nch = most4 <= 384.0 ? 6 : (most2 <= 512.0 ? 8 : (most2 <= 768.0 ? 12 : 20));
    // one wave per tile where the tiles alone fill the GPU several times over
    // (below that, the cells' own waves keep more of it busy), and with the
    // smaller register sets
    const bool seq = tiled && (waves == MD_BUILD_TILE_WAVES ||
                               (waves == MD_BUILD_AUTO && g.ntile >= MD_BUILD_TILE_MIN && nch <= 8));
    const dim3 grid((unsigned)(seq ? g.ntile : g.ncell));
    const bool wide = !seq && !half && g.ncell <= kWideCells;
#define MD_BUILD_LAUNCH(N, TILED, HALF, SEQ, W) \
    hipLaunchKernelGGL((k_build<N, TILED, HALF, SEQ, W>), grid, dim3(64 * W), 0, s, a)
    if (seq) {
        if (nch == 6) MD_BUILD_LAUNCH(6, true, false, true, 1);
        else MD_BUILD_LAUNCH(8, true, false, true, 1);
    } else if (half) {
        if (nch == 6) MD_BUILD_LAUNCH(6, false, true, false, 1);
        else MD_BUILD_LAUNCH(8, false, true, false, 1);
    } else if (tiled) {
        if (wide && nch <= 8) MD_BUILD_LAUNCH(8, true, false, false, 4);
        else if (wide && nch == 12) MD_BUILD_LAUNCH(12, true, false, false, 4);
        else if (wide) MD_BUILD_LAUNCH(20, true, false, false, 4);
        else if (nch == 6) MD_BUILD_LAUNCH(6, true, false, false, 1);
        else if (nch == 8) MD_BUILD_LAUNCH(8, true, false, false, 1);
        else if (nch == 12) MD_BUILD_LAUNCH(12, true, false, false, 1);
        else MD_BUILD_LAUNCH(20, true, false, false, 1);
    } else {
        if (wide && nch <= 8) MD_BUILD_LAUNCH(8, false, false, false, 4);
        else if (wide && nch == 12) MD_BUILD_LAUNCH(12, false, false, false, 4);
        else if (wide) MD_BUILD_LAUNCH(20, false, false, false, 4);
        else if (nch == 6) MD_BUILD_LAUNCH(6, false, false, false, 1);
        else if (nch == 8) MD_BUILD_LAUNCH(8, false, false, false, 1);
        else if (nch == 12) MD_BUILD_LAUNCH(12, false, false, false, 1);
        else MD_BUILD_LAUNCH(20, false, false, false, 1);
    }
#undef MD_BUILD_LAUNCH
    if (hipError_t e = hipGetLastError()) return e;
    ListStats st;
    st.cell_rows = a.cell_rows;
    st.ncell = g.ncell;
    st.tile_used = tile_used;
    st.ntile = tiled ? g.ntile : 0;
    st.nt = g.nt;
    st.tc = g.tc;
    st.last_cells = g.nc[2] - (g.nt - 1) * g.tc;
    st.status = list.status;
    st.part = (long long*)((char*)ws + L.red);
    return launch_list_stats(st, gather, s);
}

}  // namespace md
