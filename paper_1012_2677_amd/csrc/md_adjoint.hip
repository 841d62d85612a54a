// Adjoint kernels of the LJ force field (FP64), same row layout and lane
// grouping as the force kernel.
//
// Hessian-vector product.  With s = r^2, d = q_j - q_i, du = u_j - u_i and
// g(s) = -V'(r)/r, the force on i is F_i = -sum_j g d, so
//   (H u)_i = -dF_i[u] = sum_j [ 2 g'(s) (d . du) d + g du ],
// summed over listed partners with r < rc.  Each lane keeps its partial
// (H u)_i in registers; the group reduces it with shuffles.  The parameter
// derivative u . dF/dtheta = sum_pairs (dg/dtheta) d . du is accumulated over
// the full list and halved (each pair appears twice).
//
// Parameter gradient of U: dU/deps = U/eps and dU/dsigma = sum_pairs dV/dsigma
// with V = 4 eps [sigma^12 a(r) - sigma^6 b(r)],
//   a = r^-12 + 6 r^2 rc^-14 - 7 rc^-12,  b = r^-6 + 3 r^2 rc^-8 - 4 rc^-6,
// dV/dsigma = (48 eps sigma^12 a - 24 eps sigma^6 b) / sigma.

#include "md_internal.h"

namespace md {

struct AdjArgs {
    const double4* pos;
    const double2* rec;          // (x, y), (z, ux), (uy, uz) per slot, or nullptr
    const int32_t* cell_xyz;
    const int32_t* order;        // slots in cell order (nullptr: they are in it)
    const int64_t* offsets;
    const int32_t* counts;
    const uint32_t* nbr;
    const double* u;
    double* out;
    double* u_out;
    double* part;
    double alpha, beta, gamma, cu, cU, dt;
    double inv_eps, inv_sigma;   // 1/eps and 1/sigma, computed on the host
    int64_t n;
    double L[3], invL[3];
    int32_t nc[3];
    int32_t exact_all;
    LJ lj;
};

__device__ __forceinline__ bool boundary_cell_a(int32_t c, const int32_t* nc)
{
    const int x = c & 1023, y = (c >> 10) & 1023, z = (c >> 20) & 1023;
    return (x == 0) | (x == nc[0] - 1) | (y == 0) | (y == nc[1] - 1) | (z == 0) | (z == nc[2] - 1);
}

// Sum over each group of 8 lanes by DPP lane moves (every lane of the group gets
// it): mirror inside the group, then swap pairs of pairs, then neighbours.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xFFFFFFFFll), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return v + __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ double sum8(double v)
{
    v = dpp_add<0x141>(v);          // row_half_mirror
    v = dpp_add<0x4E>(v);           // quad_perm [2, 3, 0, 1]
    return dpp_add<0xB1>(v);        // quad_perm [1, 0, 3, 2]
}

template <int BLOCK>
__device__ __forceinline__ void block_partial2_a(double a, double b, double* part, int64_t blk)
{
    __shared__ double s_a[BLOCK / 64], s_b[BLOCK / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_a[wave] = a;
        s_b[wave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int w = 0; w < BLOCK / 64; ++w) {
            sa += s_a[w];
            sb += s_b[w];
        }
        part[2 * blk] = sa;
        part[2 * blk + 1] = sb;
    }
}

// One pass over the list for the key's partners with r < rc, in cell order,
// partners read from the records (REC) or the arrays, accumulating
//   Hu_i  = sum_j [2 g'(s) (d . du) d + g du]        (if HAS_U; du = u_j - u_i)
//   F_i   = -sum_j g d
//   t_e   = sum (dg/deps) d . du,   t_s = sum (dg/dsigma) d . du   (if HAS_U)
//   v_e   = sum V / eps,            v_s = sum dV/dsigma   (from the sums of r^-12, r^-6, r^2 and 1)
// then out_i = alpha out_i + beta Hu_i + gamma F_i (when out != nullptr),
// u_out_i = u_i + dt out_i (when u_out != nullptr), and the block partials
// (cu t_e + cU v_e, cu t_s + cU v_s) / 2 (each pair is visited twice).
template <int G, int U, bool HAS_U, bool REC>
__global__ __launch_bounds__(kForceBlock) void k_adjoint(AdjArgs a)
{
    const int64_t blk = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t place = blk * (kForceBlock / G) + threadIdx.x / G;
    const int sub = threadIdx.x % G;
    const bool valid = place < a.n;
    // keys in cell order, so that those walked together share their partners
    // in the caches
    const int64_t key = valid && a.order ? a.order[place] : place;
    const int64_t n = a.n;
    int64_t off = 0;
    int cnt = 0;
    double xi = 0.0, yi = 0.0, zi = 0.0, uxi = 0.0, uyi = 0.0, uzi = 0.0;
    bool minimg = false;
    if (valid) {
        off = a.offsets[key];
        cnt = a.counts[key];
        const double4 p = a.pos[key];
        xi = p.x;
        yi = p.y;
        zi = p.z;
        if (HAS_U) {
            uxi = a.u[key];
            uyi = a.u[n + key];
            uzi = a.u[2 * n + key];
        }
        minimg = (a.exact_all != 0) | boundary_cell_a(a.cell_xyz[key], a.nc);
    }
    const LJ& lj = a.lj;
    const double A12 = 12.0 * lj.A, B6 = -6.0 * lj.B, A14 = -14.0 * lj.A, B8 = 8.0 * lj.B;
    double hx = 0.0, hy = 0.0, hz = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
    double te = 0.0, ts = 0.0, s12 = 0.0, s6 = 0.0, s2 = 0.0;
    int pairs = 0;
    // U row entries per lane at a time: their loads, then the partners'
    // positions and u, then the pair terms, so that several gathers are in
    // flight per lane (slots past the row's end read the key itself and are
    // skipped).  32-bit byte offsets (slots are below 2^27) from uniform bases.
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    const uint32_t* row = a.nbr + off;
    const double *u0 = a.u, *u1 = a.u + n, *u2 = a.u + 2 * n;
    for (int t0 = sub; t0 < cnt; t0 += G * U) {
        uint32_t e[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int t = t0 + q * G;
            e[q] = t < cnt ? row[t] : kNone;
        }
        double4 pj[U];
        double ujx[U], ujy[U], ujz[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint32_t j = e[q] != kNone ? (e[q] & kSlotMask) : (uint32_t)key;
            if constexpr (REC) {
                const double2* rj = (const double2*)((const char*)a.rec + (uint64_t)j * 48u);
                const double2 r0 = rj[0], r1 = rj[1], r2 = rj[2];
                pj[q] = make_double4(r0.x, r0.y, r1.x, 0.0);
                ujx[q] = r1.y;
                ujy[q] = r2.x;
                ujz[q] = r2.y;
            } else {
                pj[q] = *(const double4*)((const char*)a.pos + (j << 5));
                if (HAS_U) {
                    ujx[q] = *(const double*)((const char*)u0 + (j << 3));
                    ujy[q] = *(const double*)((const char*)u1 + (j << 3));
                    ujz[q] = *(const double*)((const char*)u2 + (j << 3));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            double dx = pj[q].x - xi, dy = pj[q].y - yi, dz = pj[q].z - zi;
            if (minimg) {
                dx -= a.L[0] * rint(dx * a.invL[0]);
                dy -= a.L[1] * rint(dy * a.invL[1]);
                dz -= a.L[2] * rint(dz * a.invL[2]);
            }
            const double r2 = dx * dx + dy * dy + dz * dz;
            if (e[q] == kNone || !(r2 < lj.rc2)) continue;
            const double r2i = rcp64(r2);
            const double r6i = r2i * r2i * r2i;
            const double r8i = r2i * r6i;
            const double g = r8i * (lj.A * r6i - lj.B) - lj.C8;
            fx -= g * dx;
            fy -= g * dy;
            fz -= g * dz;
            if (HAS_U) {
                const double dux = ujx[q] - uxi, duy = ujy[q] - uyi, duz = ujz[q] - uzi;
                const double ddu = dx * dux + dy * duy + dz * duz;
                const double c = r2i * r8i * (A14 * r6i + B8) * ddu;   // 2 g' d . du
                hx += c * dx + g * dux;
                hy += c * dy + g * duy;
                hz += c * dz + g * duz;
                // eps dg/deps = g;  sigma dg/dsigma = 12 A s^-7 - 6 B s^-4 - Cs
                te += g * ddu;
                ts += (r8i * (A12 * r6i + B6) - lj.Cs) * ddu;
            }
            // V and dV/dsigma are sums of these with constant factors
            s12 += r6i * r6i;
            s6 += r6i;
            s2 += r2;
            ++pairs;
        }
    }
    fx = sum8(fx);
    fy = sum8(fy);
    fz = sum8(fz);
    if (HAS_U) {
        hx = sum8(hx);
        hy = sum8(hy);
        hz = sum8(hz);
    }
    if (valid && sub == 0 && a.out) {
        double ox = a.beta * hx + a.gamma * fx;
        double oy = a.beta * hy + a.gamma * fy;
        double oz = a.beta * hz + a.gamma * fz;
        if (a.alpha != 0.0) {
            ox += a.alpha * a.out[key];
            oy += a.alpha * a.out[n + key];
            oz += a.alpha * a.out[2 * n + key];
        }
        a.out[key] = ox;
        a.out[n + key] = oy;
        a.out[2 * n + key] = oz;
        if (a.u_out) {
            a.u_out[key] = uxi + a.dt * ox;
            a.u_out[n + key] = uyi + a.dt * oy;
            a.u_out[2 * n + key] = uzi + a.dt * oz;
        }
    }
    if (a.part) {
        const double np = (double)pairs;
        const double V = lj.A4 * s12 - lj.B4 * s6 + lj.C2 * s2 + lj.C0 * np;
        const double sa = s12 + 6.0 * lj.rc14i * s2 - 7.0 * lj.rc12i * np;
        const double sb = s6 + 3.0 * lj.rc8i * s2 - 4.0 * lj.rc6i * np;
        const double vs = 12.0 * lj.A4 * sa - 6.0 * lj.B4 * sb;
        block_partial2_a<kForceBlock>(0.5 * a.inv_eps * (a.cu * te + a.cU * V),
                                      0.5 * a.inv_sigma * (a.cu * ts + a.cU * vs), a.part, blk);
    }
}

// Records of the pass below: a partner's position and u in 48 consecutive bytes
// instead of four arrays.  The pass is bound by its gathers: a lane's 32-byte
// position and three 8-byte components of u cost five look-ups in the vector
// cache per pair, a record three.  Packing included, the fused kick takes
// 67 instead of 80 us at 256,000 particles and 264 instead of 344 us at 1.05
// million (with the pair sums of powers below, and without records 77 and 323);
// three entries in flight instead of two, 72 and 287 us; a record read by four
// lanes together and handed over in LDS (90 instead of 152 million look-ups at
// 1.05 million particles), 79 and 329 us.
__global__ __launch_bounds__(kStreamBlock) void k_pack_records(int64_t n, const double4* __restrict__ pos,
                                                               const double* __restrict__ u,
                                                               double2* __restrict__ rec)
{
    const int64_t i = (int64_t)blockIdx.x * kStreamBlock + threadIdx.x;
    if (i >= n) return;
    const double4 p = pos[i];
    const double ux = u[i], uy = u[n + i], uz = u[2 * n + i];
    rec[3 * i] = make_double2(p.x, p.y);
    rec[3 * i + 1] = make_double2(p.z, ux);
    rec[3 * i + 2] = make_double2(uy, uz);
}

#ifndef MD_ADJ_UNROLL
#define MD_ADJ_UNROLL 2
#endif
constexpr int kAdjUnroll = MD_ADJ_UNROLL;   // row entries in flight per lane

static AdjArgs make_args(const Geo& g, const LJ& lj, const double* pos, const md_cells& cells,
                         const md_pairlist& list)
{
    AdjArgs a;
    a.pos = (const double4*)pos;
    a.rec = nullptr;
    a.cell_xyz = cells.cell_xyz;
    a.order = cells.sorted ? nullptr : cells.order;
    a.offsets = list.offsets;
    a.counts = list.counts;
    a.nbr = list.nbr;
    a.u = nullptr;
    a.out = nullptr;
    a.u_out = nullptr;
    a.part = nullptr;
    a.alpha = a.beta = a.gamma = a.cu = a.cU = a.dt = 0.0;
    a.n = g.n;
    for (int k = 0; k < 3; ++k) {
        a.L[k] = g.L[k];
        a.invL[k] = g.invL[k];
        a.nc[k] = g.nc[k];
    }
    a.exact_all = g.exact_all;
    a.lj = lj;
    a.inv_eps = 1.0 / lj.eps;
    a.inv_sigma = 1.0 / lj.sigma;
    return a;
}

static void launch_adj(const Geo& g, const AdjArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)ceil_div(g.n, kKeysPerBlock)), block(kForceBlock);
    if (a.u && a.rec) {
        hipLaunchKernelGGL(k_pack_records, dim3((unsigned)ceil_div(g.n, kStreamBlock)), dim3(kStreamBlock), 0, s, g.n,
                           a.pos, a.u, (double2*)a.rec);
        hipLaunchKernelGGL((k_adjoint<kLanesPerKey, kAdjUnroll, true, true>), grid, block, 0, s, a);
    } else if (a.u) {
        hipLaunchKernelGGL((k_adjoint<kLanesPerKey, kAdjUnroll, true, false>), grid, block, 0, s, a);
    } else {
        hipLaunchKernelGGL((k_adjoint<kLanesPerKey, kAdjUnroll, false, false>), grid, block, 0, s, a);
    }
}

hipError_t launch_hvp(const Geo& g, const LJ& lj, const double* pos, const md_cells& cells,
                      const md_pairlist& list, const double* u, double* Hu, double* part, double* rec, hipStream_t s)
{
    AdjArgs a = make_args(g, lj, pos, cells, list);
    a.rec = (const double2*)rec;
    a.u = u;
    a.out = Hu;
    a.beta = 1.0;
    a.part = part;
    a.cu = 1.0;
    launch_adj(g, a, s);
    return hipGetLastError();
}

hipError_t launch_param_grad(const Geo& g, const LJ& lj, const double* pos, const md_cells& cells,
                             const md_pairlist& list, double* part, hipStream_t s)
{
    AdjArgs a = make_args(g, lj, pos, cells, list);
    a.part = part;
    a.cU = 1.0;
    launch_adj(g, a, s);
    return hipGetLastError();
}

hipError_t launch_adjoint_kick(const Geo& g, const LJ& lj, const double* pos, const md_cells& cells,
                               const md_pairlist& list, const double* u, double* out, double* u_out,
                               const AdjCoef& k, double* part, double* rec, hipStream_t s)
{
    AdjArgs a = make_args(g, lj, pos, cells, list);
    a.rec = (const double2*)rec;
    a.u = u;
    a.out = out;
    a.u_out = u_out;
    a.alpha = k.alpha;
    a.beta = k.beta;
    a.gamma = k.gamma;
    a.cu = k.cu;
    a.cU = k.cU;
    a.dt = k.dt;
    a.part = part;
    launch_adj(g, a, s);
    return hipGetLastError();
}

}  // namespace md
