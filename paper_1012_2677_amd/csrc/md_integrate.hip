// Velocity-Verlet integration (Sec. 4.5: second-order symplectic, periodic on
// all axes) with the half-skin rebuild trigger (Sec. 2.3, search-length figure),
// and the fixed-order FP64 reductions of energy and list statistics.
//
// One thread per slot streams pos, vel, force and pos_ref (SoA, coalesced);
// the kernel is bound by HBM bandwidth.  It runs the first half kick and drift
// at the start of a run and the kinetic energy of a state; inside a run the
// kicks and drift after each force evaluation are fused into the pair kernel.
// Block maxima of the squared displacement since the last build go to one
// atomic max (exact, order independent); kinetic-energy block sums go to a
// partials array reduced later in a fixed order (deterministic).

#include "md_internal.h"

namespace md {

__device__ __forceinline__ double wrap_coord(double x, double L, double invL)
{
    double y = x - L * floor(x * invL);
    if (y >= L) y -= L;
    if (y < 0.0) y += L;
    return y;
}

__device__ __forceinline__ float local_coord_i(double x, int c, double cs, double L, double invL)
{
    double l = x - (double)c * cs;
    l -= L * rint((l - 0.5 * cs) * invL);
    return (float)l;
}

// MODE INT_KD: first half kick and drift of a step (the start of a run, when
// no force evaluation precedes it in the same pass).  MODE INT_KE: kinetic
// energy only.  The kicks that follow a force evaluation run inside the pair
// kernel (launch_force_step).
template <int MODE, bool MIXED>
__global__ __launch_bounds__(kStreamBlock) void k_integrate(Geo g, IntArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = g.n;
    const bool valid = i < n;
    const double h = 0.5 * a.dt;
    constexpr bool DRIFT = MODE == INT_KD;
    constexpr bool KE = MODE == INT_KE;
    double* __restrict__ vel = a.vel;
    double4* __restrict__ P = (double4*)a.pos;
    const double* __restrict__ ref = a.pos_ref;
    double ke = 0.0, d2 = 0.0, v2 = 0.0;
    if (valid) {
        // every input is loaded before anything is stored, so all loads of a
        // thread are in flight together
        double vx = vel[i], vy = vel[n + i], vz = vel[2 * n + i];
        double fx = 0.0, fy = 0.0, fz = 0.0;
        if (DRIFT) {
            if (MIXED) {
                const float* __restrict__ F = (const float*)a.force;
                fx = F[i];
                fy = F[n + i];
                fz = F[2 * n + i];
            } else {
                const double* __restrict__ F = (const double*)a.force;
                fx = F[i];
                fy = F[n + i];
                fz = F[2 * n + i];
            }
        }
        double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
        double rx = 0.0, ry = 0.0, rz = 0.0;
        int32_t c = 0;
        if (DRIFT) {
            p = P[i];
            rx = ref[i];
            ry = ref[n + i];
            rz = ref[2 * n + i];
            if (MIXED) c = a.cell_xyz[i];
        }
        if (KE) ke = vx * vx + vy * vy + vz * vz;
        if (DRIFT) {
            vx = vx + h * fx;
            vy = vy + h * fy;
            vz = vz + h * fz;
            v2 = pinned_len2(vx, vy, vz);
            p.x = wrap_coord(p.x + a.dt * vx, g.L[0], g.invL[0]);
            p.y = wrap_coord(p.y + a.dt * vy, g.L[1], g.invL[1]);
            p.z = wrap_coord(p.z + a.dt * vz, g.L[2], g.invL[2]);
            double ex = p.x - rx, ey = p.y - ry, ez = p.z - rz;
            ex -= g.L[0] * rint(ex * g.invL[0]);
            ey -= g.L[1] * rint(ey * g.invL[1]);
            ez -= g.L[2] * rint(ez * g.invL[2]);
            d2 = pinned_len2(ex, ey, ez);
            P[i] = p;
            if (MIXED) {
                ((float4*)a.pos32)[i] =
                    make_float4(local_coord_i(p.x, c & 1023, g.cs[0], g.L[0], g.invL[0]),
                                local_coord_i(p.y, (c >> 10) & 1023, g.cs[1], g.L[1], g.invL[1]),
                                local_coord_i(p.z, (c >> 20) & 1023, g.cs[2], g.L[2], g.invL[2]),
                                __int_as_float(c));
            }
            vel[i] = vx;
            vel[n + i] = vy;
            vel[2 * n + i] = vz;
        }
    }
    __shared__ double s_v[kStreamBlock / 64], s_u[kStreamBlock / 64];
    if (DRIFT) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            d2 = fmax(d2, __shfl_xor(d2, o, 64));
            v2 = fmax(v2, __shfl_xor(v2, o, 64));
        }
        if ((threadIdx.x & 63) == 0) {
            s_v[threadIdx.x >> 6] = d2;
            s_u[threadIdx.x >> 6] = v2;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double m = 0.0, mv = 0.0;
#pragma unroll
            for (int w = 0; w < kStreamBlock / 64; ++w) {
                m = fmax(m, s_v[w]);
                mv = fmax(mv, s_u[w]);
            }
            atomicMax(max_slot(a.max_d2, blockIdx.x), (unsigned long long)__double_as_longlong(m));
            atomicMax(max_slot(a.max_v2, blockIdx.x), (unsigned long long)__double_as_longlong(mv));
        }
    }
    if (KE) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) ke += __shfl_xor(ke, o, 64);
        if ((threadIdx.x & 63) == 0) s_v[threadIdx.x >> 6] = ke;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < kStreamBlock / 64; ++w) s += s_v[w];
            a.part_ke[blockIdx.x] = 0.5 * s;
        }
    }
}

hipError_t launch_integrate(const Geo& g, IntMode mode, const IntArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)ceil_div(g.n, kStreamBlock)), block(kStreamBlock);
    const bool mixed = a.precision == MD_MIXED;
    if (mode == INT_KD) {
        if (mixed) hipLaunchKernelGGL((k_integrate<INT_KD, true>), grid, block, 0, s, g, a);
        else hipLaunchKernelGGL((k_integrate<INT_KD, false>), grid, block, 0, s, g, a);
    } else {
        if (mixed) hipLaunchKernelGGL((k_integrate<INT_KE, true>), grid, block, 0, s, g, a);
        else hipLaunchKernelGGL((k_integrate<INT_KE, false>), grid, block, 0, s, g, a);
    }
    return hipGetLastError();
}

// ---- fixed-order reductions -------------------------------------------------
__device__ __forceinline__ double block_sum_1024(double v)
{
    __shared__ double s_w[kReduceBlock / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kReduceBlock / 64; ++w) t += s_w[w];
    __syncthreads();
    return t;
}

// energy[0..3] = (KE, PE, W, KE + PE); also into log_row when given.  Two
// fixed-order levels: block b sums its contiguous share of the partials into
// part3[3b .. 3b+2], then one block sums those in block order.  Up to
// kEnergyOne partials one block sums them itself (1000 partials: one launch of
// 4.0 us instead of two of 4.4 and 4.3).
constexpr int kEnergyBlocks = 256;
constexpr int64_t kEnergyOne = 4096;
__global__ __launch_bounds__(kReduceBlock) void k_reduce_energy_part(const double* __restrict__ part_pw, int64_t nbf,
                                                                     const double* __restrict__ part_ke, int64_t nbi,
                                                                     double* __restrict__ part3,
                                                                     const int32_t* __restrict__ gate)
{
    if (gate && gate[0]) return;
    const int64_t cf = (nbf + gridDim.x - 1) / gridDim.x, ci = (nbi + gridDim.x - 1) / gridDim.x;
    const int64_t f0 = (int64_t)blockIdx.x * cf, f1 = min(f0 + cf, nbf);
    const int64_t i0 = (int64_t)blockIdx.x * ci, i1 = min(i0 + ci, nbi);
    double pe = 0.0, w = 0.0, ke = 0.0;
    for (int64_t b = f0 + threadIdx.x; b < f1; b += kReduceBlock) {
        pe += part_pw[2 * b];
        w += part_pw[2 * b + 1];
    }
    for (int64_t b = i0 + threadIdx.x; b < i1; b += kReduceBlock) ke += part_ke[b];
    pe = block_sum_1024(pe);
    w = block_sum_1024(w);
    ke = block_sum_1024(ke);
    if (threadIdx.x == 0) {
        part3[3 * blockIdx.x] = pe;
        part3[3 * blockIdx.x + 1] = w;
        part3[3 * blockIdx.x + 2] = ke;
    }
}

__global__ __launch_bounds__(kReduceBlock) void k_reduce_energy(const double* __restrict__ part3, int nb,
                                                                const double* __restrict__ part_pw, int64_t nbf,
                                                                const double* __restrict__ part_ke, int64_t nbi,
                                                                double* __restrict__ energy,
                                                                double* __restrict__ log_row,
                                                                const int32_t* __restrict__ gate)
{
    if (gate && gate[0]) return;
    double pe = 0.0, w = 0.0, ke = 0.0;
    if (nb == 0) {
        for (int64_t b = threadIdx.x; b < nbf; b += kReduceBlock) {
            pe += part_pw[2 * b];
            w += part_pw[2 * b + 1];
        }
        for (int64_t b = threadIdx.x; b < nbi; b += kReduceBlock) ke += part_ke[b];
    } else if ((int)threadIdx.x < nb) {
        pe = part3[3 * threadIdx.x];
        w = part3[3 * threadIdx.x + 1];
        ke = part3[3 * threadIdx.x + 2];
    }
    pe = block_sum_1024(pe);
    w = block_sum_1024(w);
    ke = block_sum_1024(ke);
    if (threadIdx.x == 0) {
        energy[0] = ke;
        energy[1] = pe;
        energy[2] = w;
        energy[3] = ke + pe;
        if (log_row) {
            log_row[0] = ke;
            log_row[1] = pe;
            log_row[2] = w;
            log_row[3] = ke + pe;
        }
    }
}

hipError_t launch_reduce_energy(const double* part_pw, int64_t nbf, const double* part_ke, int64_t nbi,
                                double* energy, double* log_row, double* scratch, hipStream_t s,
                                const int32_t* gate)
{
    const int64_t most = nbf > nbi ? nbf : nbi;
    int nb = 0;
    if (most > kEnergyOne) {
        nb = (int)std::min<int64_t>(ceil_div(most, kReduceBlock), kEnergyBlocks);
        hipLaunchKernelGGL(k_reduce_energy_part, dim3(nb), dim3(kReduceBlock), 0, s, part_pw, nbf, part_ke, nbi,
                           scratch, gate);
    }
    hipLaunchKernelGGL(k_reduce_energy, dim3(1), dim3(kReduceBlock), 0, s, (const double*)scratch, nb, part_pw, nbf,
                       part_ke, nbi, energy, log_row, gate);
    return hipGetLastError();
}

// out2[k] = scale_k * sum_b part[2b + k]   (or += when accumulating)
__global__ __launch_bounds__(kReduceBlock) void k_reduce_pair(const double* __restrict__ part, int64_t nb,
                                                              double s0, double s1, double* __restrict__ out2,
                                                              int accumulate)
{
    double a = 0.0, b = 0.0;
    for (int64_t k = threadIdx.x; k < nb; k += kReduceBlock) {
        a += part[2 * k];
        b += part[2 * k + 1];
    }
    a = block_sum_1024(a);
    b = block_sum_1024(b);
    if (threadIdx.x == 0) {
        out2[0] = (accumulate ? out2[0] : 0.0) + s0 * a;
        out2[1] = (accumulate ? out2[1] : 0.0) + s1 * b;
    }
}

hipError_t launch_reduce_pair(const double* part, int64_t nb, double scale0, double scale1, double* out2,
                              hipStream_t s, bool accumulate)
{
    hipLaunchKernelGGL(k_reduce_pair, dim3(1), dim3(kReduceBlock), 0, s, part, nb, scale0, scale1, out2,
                       accumulate ? 1 : 0);
    return hipGetLastError();
}

// The flags also to host memory that the device can write, given one: all words
// with the call's number and their seal, in one store of 16 lanes; the host
// polls for a set of words that belong together.
__device__ __forceinline__ void publish_flags(const int64_t* s_out, const GatherIo& io)
{
    if (!io.host) return;
    const int lane = (int)lane_id();
    __builtin_amdgcn_wave_barrier();
    int64_t v = lane < kFlagWords ? s_out[lane] : io.seq;
    int64_t x = lane <= kFlagWords ? (int64_t)seal_mix((uint64_t)v, lane) : 0;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) x ^= (int64_t)__shfl_xor((long long)x, o, 64);
    if (lane == kFlagWords + 1) v = x;
    if (lane < kFlagWords + 2) io.host[lane] = v;
}

// The flags of the state that the host reads, by one wave (FlagGate in
// md_internal.h).
__device__ __forceinline__ void gather_flags(const int64_t status[4], const GatherIo& io, const FlagGate& g)
{
    __shared__ int64_t s_out[kFlagWords];
    // wave-wide maxima over the slots: largest staged tile neighbourhood,
    // largest squared displacement and drift speed (bit patterns of
    // non-negative doubles order like the values)
    const int lane = (int)lane_id();
    const bool step = g.run.gate != nullptr, folded = g.run.slots != nullptr;
    const int32_t stopped = step && (folded || g.run.idx > 1) ? g.run.gate[0] : 0;
    // a run already stopped: leave out (and the slots) as the stopping gather left them
    if (stopped && !folded) {
        if (lane < kFlagWords) s_out[lane] = io.out[lane];
        publish_flags(s_out, io);
        return;
    }
    const int32_t ran = stopped ? g.run.gate[1] : g.run.idx;
    const bool fold = !step || stopped || g.drift;
    int64_t m = 0;
    unsigned long long md = 0, mv = 0;
    for (int k = lane; k < kTileMaxSlots; k += 64) m = max(m, io.tmax[k]);
    if (folded) {
        // the displacements of the last step that ran, set (ran - 1) % 3
        if (lane < kRunSlots) {
            if (fold) md = run_set(g.run, ran + 2)[lane * kMaxSlotStride];
            for (int k = 0; k < 3; ++k)
                *(ulonglong2*)(run_set(g.run, k) + lane * kMaxSlotStride) = make_ulonglong2(0ull, 0ull);
        }
    } else if (fold) {
        for (int k = lane; k < kMaxSlots; k += 64) {
            md = max(md, io.mx[k * kMaxSlotStride]);
            mv = max(mv, io.mx[(kMaxSlots + k) * kMaxSlotStride]);
            if (step) {
                io.mx[k * kMaxSlotStride] = 0;
                io.mx[(kMaxSlots + k) * kMaxSlotStride] = 0;
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        m = max(m, (int64_t)__shfl_xor((long long)m, o, 64));
        md = max(md, (unsigned long long)__shfl_xor((long long)md, o, 64));
        mv = max(mv, (unsigned long long)__shfl_xor((long long)mv, o, 64));
    }
    if (lane == 0) {
        if (fold) {
            io.energy[4] = __longlong_as_double((long long)md);
            io.energy[5] = __longlong_as_double((long long)mv);
        }
        const double d2 = fold ? __longlong_as_double((long long)md) : io.energy[4];
        const double v2 = fold ? __longlong_as_double((long long)mv) : io.energy[5];
        const int32_t stop = step && ((io.flags[0] & 1) != 0 || (fold && d2 > g.run.thr2)) ? 1 : 0;
        for (int k = 0; k < 4; ++k) s_out[k] = status[k];
        s_out[4] = io.err[0];
        s_out[5] = io.err[1];
        s_out[6] = io.flags[0];
        s_out[7] = __double_as_longlong(d2);
        s_out[8] = __double_as_longlong(v2);
        s_out[9] = io.err[4];     // large-displacement check: member count
        s_out[10] = io.err[5];    // large-displacement check: violation flag
        s_out[11] = m;            // tiled list: largest staged neighbourhood of a tile
        s_out[12] = ran;
        s_out[13] = stop;
        if (step) g.run.gate[0] = stop;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < kFlagWords) io.out[lane] = s_out[lane];
    publish_flags(s_out, io);
}

__global__ __launch_bounds__(64) void k_gather_flags(const int64_t* __restrict__ status, GatherIo io, FlagGate g)
{
    const int64_t st[4] = {status[0], status[1], status[2], status[3]};
    gather_flags(st, io, g);
}

hipError_t launch_gather_flags(const int64_t* status, const GatherIo& io, hipStream_t s, const FlagGate& gate)
{
    hipLaunchKernelGGL(k_gather_flags, dim3(1), dim3(64), 0, s, status, io, gate);
    return hipGetLastError();
}

// List statistics: per-block (sum, stride needed) partials, then one block
// combines them in order (and gathers the flags that the host reads next); small
// grids in the last block alone.
constexpr int kStatsBlocks = 1024;
constexpr int64_t kStatsOneCells = 8192;

__device__ __forceinline__ void stats_of(const ListStats& l, int64_t i0, int64_t stride, long long& sum, long long& mx)
{
#pragma unroll 4
    for (int64_t c = i0; c < l.ncell; c += stride) {
        const long long r = l.cell_rows[c];
        sum += r;
        if (l.ntile == 0) mx = r > mx ? r : mx;
    }
    for (int64_t t = i0; t < l.ntile; t += stride) {
        const int cells = (int)t % l.nt == l.nt - 1 ? l.last_cells : l.tc;
        const long long r = (l.tile_used[t] + cells - 1) / cells;
        mx = r > mx ? r : mx;
    }
}

// (sum, max) of the block in thread 0 .. 63 of it
template <int BLOCK>
__device__ __forceinline__ void block_stats(long long& sum, long long& mx)
{
    __shared__ long long s_sum[BLOCK / 64], s_max[BLOCK / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o, 64);
        const long long y = __shfl_xor(mx, o, 64);
        mx = y > mx ? y : mx;
    }
    if ((threadIdx.x & 63) == 0) {
        s_sum[threadIdx.x >> 6] = sum;
        s_max[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    sum = mx = 0;
    for (int w = 0; w < BLOCK / 64; ++w) {
        sum += s_sum[w];
        mx = s_max[w] > mx ? s_max[w] : mx;
    }
}

__global__ __launch_bounds__(kStreamBlock) void k_stats_partial(ListStats l)
{
    long long sum = 0, mx = 0;
    stats_of(l, (int64_t)blockIdx.x * kStreamBlock + threadIdx.x, (int64_t)gridDim.x * kStreamBlock, sum, mx);
    block_stats<kStreamBlock>(sum, mx);
    if (threadIdx.x == 0) {
        l.part[2 * blockIdx.x] = sum;
        l.part[2 * blockIdx.x + 1] = mx;
    }
}

__global__ __launch_bounds__(kStatsBlocks) void k_stats_final(ListStats l, int nb, int gather, GatherIo io)
{
    long long sum = 0, mx = 0;
    if (nb == 0) {
        stats_of(l, threadIdx.x, kStatsBlocks, sum, mx);
    } else if ((int)threadIdx.x < nb) {
        sum = l.part[2 * threadIdx.x];
        mx = l.part[2 * threadIdx.x + 1];
    }
    block_stats<kStatsBlocks>(sum, mx);
    if (threadIdx.x >= 64) return;
    if (threadIdx.x == 0) {
        l.status[0] = sum;
        l.status[1] = mx;
    }
    if (gather) {
        const int64_t st[4] = {sum, mx, l.status[2], l.status[3]};
        gather_flags(st, io, FlagGate());
    }
}

hipError_t launch_list_stats(const ListStats& l, const GatherIo* gather, hipStream_t s)
{
    int nb = 0;
    if (l.ncell > kStatsOneCells) {
        nb = (int)std::min<int64_t>(ceil_div(l.ncell, kStreamBlock), kStatsBlocks);
        hipLaunchKernelGGL(k_stats_partial, dim3(nb), dim3(kStreamBlock), 0, s, l);
    }
    hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(kStatsBlocks), 0, s, l, nb, gather ? 1 : 0,
                       gather ? *gather : GatherIo());
    return hipGetLastError();
}

}  // namespace md
