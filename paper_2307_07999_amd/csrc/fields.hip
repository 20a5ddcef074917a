// fields.hip -- the boost-invariant leapfrog of the classical Yang-Mills
// equations (Eq. (1)) on transverse links, the local-frame site fields the
// particles read, and the field diagnostics.
//
// Lattice Hamiltonian per unit rapidity (a = 1, g absorbed), Milne time tau:
//   H = sum_x [ sum_i Tr E_i^2 / tau + tau Tr pi^2
//               + sum_i Tr (Phi_{+i} - phi)^2 / tau + 2 tau (3 - Re Tr P) ]
// with E_i = tau dA_i/dtau, phi = A_eta, pi = (1/tau) dA_eta/dtau,
// P(x) = U_1(x) U_2(x+1) U_1^dag(x+2) U_2^dag(x) and
// Phi_{+i}(x) = U_i(x) phi(x+i) U_i^dag(x), Phi_{-i}(x) = U_i^dag(x-i) phi(x-i) U_i(x-i).
// One step (E, pi at half steps, U, phi at integer steps):
//   E_1 += dtau { -tau ([P(x)]_X - U_2^dag(x-2)[P(x-2)]_X U_2(x-2)) - (i/tau)[phi, Phi_{+1}] }
//   E_2 += dtau { -tau (U_1^dag(x-1)[P(x-1)]_X U_1(x-1) - [P(x)]_X) - (i/tau)[phi, Phi_{+2}] }
//   pi  += (dtau/tau) sum_i (Phi_{+i} + Phi_{-i} - 2 phi)
//   U_i <- exp(i dtau E_i / tau_{n+1/2}) U_i,   phi += dtau tau_{n+1/2} pi
// This scheme keeps the Gauss law sum_i [E_i(x) - U_i^dag(x-i)E_i(x-i)U_i(x-i)]
// + i[phi, pi] exactly constant.
//
// Kernel design: two lanes per site, one per link direction (the per-site
// work of one lane needs too many registers for more than one wave per SIMD);
// workgroups of 32 x 4 sites.  The links and phi of the tile and a one-site
// halo are staged in LDS with coalesced 16-byte reads of the chunked field
// state, and every neighbour of the stencil is read from there: without the
// tile the step issues ~250 global loads per lane and its waves spend half
// their time waiting on them.  Tiles are numbered so that each XCD owns one
// band of rows (xcd_remap): the neighbour reads of the stencil then hit the
// L2 of the XCD that owns the tile instead of refetching halo lines from
// memory.
#include <algorithm>

#include "fields_dev.hpp"

namespace gl {

constexpr int TX = 32, TY = 8;     // site tiles of the diagnostics
constexpr int SX = 32, SY = 4;     // site tiles of the step: 2 lanes per site

// FP64: two waves per SIMD at the cost of a few spilled registers is faster
// than one wave with everything in registers.
template <typename T, bool WT>
__device__ __forceinline__ void field_step_tile(LinkTile<T, SX, SY> &tile, int N, FieldPtrs<T> in,
                                                FieldPtrs<T> out, T *F, T tau, T dtau, T tau_h,
                                                int reunit) {
    const int tx = (N + SX - 1) / SX;
    const int l = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = (l % tx) * SX, y0 = (l / tx) * SY;
    const int lx = threadIdx.x >> 1, ly = threadIdx.y;
    const int tid = threadIdx.x + 2 * SX * threadIdx.y;
    stage_tile(tile, N, in, x0, y0, tid, 2 * SX * SY);
    __syncthreads();
    // every thread takes part (the step synchronises the workgroup); both
    // lanes of a pair are on or off the lattice together
    const bool active = x0 + lx < N && y0 + ly < N;
    field_step_link<T, SX, SY, kStreamed<T>, WT>(tile, N, in, out, F, x0, y0, lx, ly, threadIdx.x & 1, tid, active, tau,
                                                 dtau, tau_h, reunit);
}
template <typename T>
__global__ void __launch_bounds__(2 * SX * SY) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4, 8)))
k_field_step(int N, FieldPtrs<T> in, FieldPtrs<T> out, T *__restrict__ F, T tau, T dtau, T tau_h, int reunit) {
    __shared__ LinkTile<T, SX, SY> tile;
    field_step_tile<T, true>(tile, N, in, out, F, tau, dtau, tau_h, reunit);
}
// the step whose stores stay in the L2 caches (written_through)
template <typename T>
__global__ void __launch_bounds__(2 * SX * SY) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4, 8)))
k_field_step_cached(int N, FieldPtrs<T> in, FieldPtrs<T> out, T *__restrict__ F, T tau, T dtau, T tau_h, int reunit) {
    __shared__ LinkTile<T, SX, SY> tile;
    field_step_tile<T, false>(tile, N, in, out, F, tau, dtau, tau_h, reunit);
}

// The two field correlators at tau_n, FP64, from one read of the site fields
// (E_x and E_y adding the half stored apart where half_stored holds).
//
// Static quarks (STAT; Sec. 2, Eq. (4)): I_i^a(x) += dtau E_i^a(x, tau_n).
//
// Lightlike jets (LIGHT; Sec. 2, Eq. (5)): one jet per start site x0, step j
// since its start; it sits in the cell x0 + floor(j dtau + 1/2) along x and feels
// F_x = E_x, F_y = E_y - B_z, F_z = E_z + B_y there, transported to its start
// with W: I_i += dtau [W F_i W^dag]; when this step's drift ends in the next
// cell, W <- W U_x(cell) with the links of tau_n.
//
// One thread per cell, which serves the static quark there and the jet that
// sits in it.  Per workgroup and correlator the sums over its cells of
// (1/2) sum_a (I_i^a)^2 for i = x, y, z and their count, added in a fixed
// order (part_s, part_l [blocks][4]).
//
// Bound: by HBM, 340 MB at 512^2 in FP64 (accumulators and W in and out, E, B_y and
// B_z in).  The accumulators are read and written once a step and take the
// streaming hint (ST) where the event overflows the last-level cache, so that
// the site fields stay for the push.  Apart, with 8-byte reads of 16-byte
// chunks and a reduction launch each, the two took 33 + 53 + 10 us a step;
// together 63 us, and the push behind them 116 -> 101 us.
template <typename T, bool STAT, bool LIGHT, bool ST>
__global__ void __launch_bounds__(256)
k_correlators(int N, const T *__restrict__ F, const T *__restrict__ U, double *__restrict__ Is, double *__restrict__ W,
              double *__restrict__ Il, int64_t j, double dtau, double *__restrict__ part_s,
              double *__restrict__ part_l) {
    constexpr int CP = stream_policy(ST);
    __shared__ double red[8][4];
    const size_t n2 = plane_pitch(N);
    const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
    double v[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (c < (size_t)N * N) {
        const int ix = (int)(c % N), iy = (int)(c / N);
        const int64_t shift = LIGHT ? (int64_t)floor((double)j * dtau + 0.5) : 0;
        const int back = ix - (int)(shift % N);
        const size_t x0 = (size_t)(back < 0 ? back + N : back) + (size_t)N * iy;   // start site of the jet here
        M3<double> w;
        if constexpr (LIGHT) {
#pragma unroll
            for (int r = 0; r < 3; r++)
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    w.re[r][q] = pl_ld_p<CP>(W, n2, 2 * (3 * r + q), x0);
                    w.im[r][q] = pl_ld_p<CP>(W, n2, 2 * (3 * r + q) + 1, x0);
                }
        }
#pragma unroll
        for (int i = 0; i < 3; i++) {
            T re[8], rh[8];
            double e[8];
            site_load<8>(F, c, 8 * i, re);
            const bool half = i < 2 && half_stored(i, ix, iy);
            if (half) site_load<8>(F, c, 48 + 8 * i, rh);
#pragma unroll
            for (int a = 0; a < 8; a++) e[a] = (double)re[a] + (half ? (double)rh[a] : 0.0);
            if constexpr (STAT) {
                double s = 0.0;
#pragma unroll
                for (int a = 0; a < 8; a++) {
                    const double q = pl_ld_p<CP>(Is, n2, 8 * i + a, c) + dtau * e[a];
                    pl_st_p<CP>(Is, n2, 8 * i + a, c, q);
                    s += q * q;
                }
                v[i] = 0.5 * s;
            }
            if constexpr (LIGHT) {
                double t[8];
                if (i > 0) {
                    T rb[8];   // B_z for F_y, B_y for F_z
                    site_load<8>(F, c, i == 1 ? 40 : 32, rb);
#pragma unroll
                    for (int a = 0; a < 8; a++) e[a] += i == 1 ? -(double)rb[a] : (double)rb[a];
                }
                transport_nd(w, e, t);
                double s = 0.0;
#pragma unroll
                for (int a = 0; a < 8; a++) {
                    const double q = pl_ld_p<CP>(Il, n2, 8 * i + a, x0) + dtau * t[a];
                    pl_st_p<CP>(Il, n2, 8 * i + a, x0, q);
                    s += q * q;
                }
                v[4 + i] = 0.5 * s;
            }
        }
        v[3] = v[7] = 1.0;
        if constexpr (LIGHT) {
            if ((int64_t)floor((double)(j + 1) * dtau + 0.5) > shift) {
                const M3<T> u = chunk_load_link(U, n2, c, 0);
                M3<double> ud;
#pragma unroll
                for (int r = 0; r < 3; r++)
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        ud.re[r][q] = (double)u.re[r][q];
                        ud.im[r][q] = (double)u.im[r][q];
                    }
                w = mul(w, ud);
#pragma unroll
                for (int r = 0; r < 3; r++)
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        pl_st_p<CP>(W, n2, 2 * (3 * r + q), x0, w.re[r][q]);
                        pl_st_p<CP>(W, n2, 2 * (3 * r + q) + 1, x0, w.im[r][q]);
                    }
            }
        }
    }
#pragma unroll
    for (int k = STAT ? 0 : 4; k < (LIGHT ? 8 : 4); k++) {
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) v[k] += __shfl_xor(v[k], m, 64);
        if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = v[k];
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < 8 && (k < 4 ? STAT : LIGHT))
        (k < 4 ? part_s : part_l)[(size_t)blockIdx.x * 4 + (k & 3)] = (red[k][0] + red[k][1]) + (red[k][2] + red[k][3]);
}

// Diagnostics per site, reduced per workgroup in FP64:
// [0] max |G^a|, [1] max |E^a|, [2] max |U U^dag - 1|, [3..6] energy terms,
// [7] non-finite count.
constexpr int kDiagVals = 8;

template <typename T>
__global__ void __launch_bounds__(TX *TY)
k_diag(int N, FieldPtrs<T> f, T tau, double *__restrict__ partials) {
    __shared__ double red[kDiagVals][TX * TY];
    int tid = threadIdx.x + TX * threadIdx.y;
    int ix = blockIdx.x * TX + threadIdx.x;
    int iy = blockIdx.y * TY + threadIdx.y;
    double v[kDiagVals] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (ix < N && iy < N) {
        const size_t n2 = (size_t)N * N;
        Nbr nb = neighbours(ix, iy, N);
        M3<T> u1x = chunk_load_link(f.U, n2, nb.x, 0), u2x = chunk_load_link(f.U, n2, nb.x, 1);
        T e1[8], e2[8], e1m[8], e2m[8], ph[8], p[8];
        chunk_load_a(f.E, n2, nb.x, 0, e1);
        chunk_load_a(f.E, n2, nb.x, 8, e2);
        chunk_load_a(f.E, n2, nb.xm1, 0, e1m);
        chunk_load_a(f.E, n2, nb.xm2, 8, e2m);
        chunk_load_a(f.phi, n2, nb.x, 0, ph);
        chunk_load_a(f.pi, n2, nb.x, 0, p);
        M3<T> u1m = chunk_load_link(f.U, n2, nb.xm1, 0), u2m = chunk_load_link(f.U, n2, nb.xm2, 1);
        T t1[8], t2[8];
        transport_dn(u1m, e1m, t1);
        transport_dn(u2m, e2m, t2);
        M3<T> PH = herm_from_alg(ph), PI = herm_from_alg(p);
        M3<T> c = sub(mul(PH, PI), mul(PI, PH));   // [phi, pi]; i[phi,pi] hermitian
        M3<T> ic;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) { ic.re[i][j] = -c.im[i][j]; ic.im[i][j] = c.re[i][j]; }
        T g[8];
        alg_from_herm(ic, g);
        double gmax = 0, emax = 0, et = 0, el = 0, bt = 0;
        int bad = 0;
#pragma unroll
        for (int a = 0; a < 8; a++) {
            double ga = (double)e1[a] - (double)t1[a] + (double)e2[a] - (double)t2[a] + (double)g[a];
            gmax = fmax(gmax, fabs(ga));
            emax = fmax(emax, fmax(fabs((double)e1[a]), fabs((double)e2[a])));
            et += 0.5 * ((double)e1[a] * e1[a] + (double)e2[a] * e2[a]);
            el += 0.5 * (double)p[a] * p[a];
            if (!isfinite((double)e1[a]) || !isfinite((double)e2[a]) || !isfinite((double)ph[a]) ||
                !isfinite((double)p[a]))
                bad++;
        }
        double umax = 0;
        M3<T> uu[2] = {u1x, u2x};
#pragma unroll
        for (int d = 0; d < 2; d++) {
            M3<T> w = mul_nd(uu[d], uu[d]);
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    double dr = (double)w.re[i][j] - (i == j ? 1.0 : 0.0);
                    umax = fmax(umax, fmax(fabs(dr), fabs((double)w.im[i][j])));
                    if (!isfinite((double)uu[d].re[i][j]) || !isfinite((double)uu[d].im[i][j])) bad++;
                }
        }
        // B_T: sum_i Tr(Phi_{+i} - phi)^2
        M3<T> ups[2] = {u1x, u2x};
        size_t xps[2] = {nb.xp1, nb.xp2};
#pragma unroll
        for (int d = 0; d < 2; d++) {
            T v2[8];
            chunk_load_a(f.phi, n2, xps[d], 0, v2);
            M3<T> Pf = mul_nd(mul(ups[d], herm_from_alg(v2)), ups[d]);
            T df[8];
            alg_from_herm(Pf, df);
#pragma unroll
            for (int a = 0; a < 8; a++) {
                double dd = (double)df[a] - (double)ph[a];
                bt += 0.5 * dd * dd;
            }
        }
        M3<T> P = plaq(u1x, chunk_load_link(f.U, n2, nb.xp1, 1), chunk_load_link(f.U, n2, nb.xp2, 0), u2x);
        double bl = 3.0 - ((double)P.re[0][0] + (double)P.re[1][1] + (double)P.re[2][2]);
        v[0] = gmax;
        v[1] = emax;
        v[2] = umax;
        v[3] = et / (double)tau;
        v[4] = el * (double)tau;
        v[5] = bt / (double)tau;
        v[6] = 2.0 * (double)tau * bl;
        v[7] = bad;
    }
#pragma unroll
    for (int k = 0; k < kDiagVals; k++) red[k][tid] = v[k];
    __syncthreads();
    for (int s = TX * TY / 2; s > 0; s >>= 1) {
        if (tid < s) {
#pragma unroll
            for (int k = 0; k < kDiagVals; k++) {
                double a = red[k][tid], b = red[k][tid + s];
                red[k][tid] = (k < 3) ? fmax(a, b) : a + b;
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        size_t blk = blockIdx.x + (size_t)gridDim.x * blockIdx.y;
#pragma unroll
        for (int k = 0; k < kDiagVals; k++) partials[blk * kDiagVals + k] = red[k][0];
    }
}

// Failure detection: values [0, n) of a flat array, grouped in steps of
// vals_per_step consecutive values (step step0 + i / vals_per_step), are
// tested for NaN and Inf, and a lane holding one lowers *first_bad to its
// step.  Grid-stride; one 16-byte vector of V values per lane and pass.
template <typename V, typename T, int NV>
__global__ void __launch_bounds__(256)
k_check_finite(const T *__restrict__ a, int64_t n, int64_t vals_per_step, int step0, int *first_bad) {
    const int64_t nv = n / NV;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < nv; v += stride) {
        const V w = reinterpret_cast<const V *>(a)[v];
        const T *e = reinterpret_cast<const T *>(&w);
        bool bad = false;
#pragma unroll
        for (int k = 0; k < NV; k++) bad |= !isfinite(e[k]);
        if (bad) atomicMin(first_bad, step0 + (int)(v * NV / vals_per_step));
    }
    // a tail shorter than one vector
    const int64_t t = nv * NV + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < n && !isfinite(a[t])) atomicMin(first_bad, step0 + (int)(t / vals_per_step));
}

template <typename T>
hipError_t launch_check_finite(hipStream_t st, const T *a, int64_t n, int64_t vals_per_step, int step0,
                               int *first_bad) {
    if (n <= 0) return hipSuccess;
    constexpr int NV = 16 / (int)sizeof(T);
    const int64_t blocks = std::min<int64_t>(2048, std::max<int64_t>(1, (n / NV + 255) / 256));
    if (sizeof(T) == 8)
        hipLaunchKernelGGL((k_check_finite<double2, double, 2>), dim3((unsigned)blocks), dim3(256), 0, st,
                           (const double *)a, n, vals_per_step, step0, first_bad);
    else
        hipLaunchKernelGGL((k_check_finite<float4, float, 4>), dim3((unsigned)blocks), dim3(256), 0, st,
                           (const float *)a, n, vals_per_step, step0, first_bad);
    return hipGetLastError();
}

// Whether a field step alone writes its state through the L2 caches.  Small FP32
// states are better left there for the next step (64 steps of fields, left and
// written through: 32^2 436 and 458 us, 64^2 429 and 454, 128^2 455 and 462, 144^2 470 and
// 477, but 162^2 497 and 487, 256^2 640 and 630, 324^2 973 and 891).  In FP64, rows of sites
// that do not fill 64-byte sectors are shared by two tiles and better joined in L2
// (162^2 584 and 625 us, 243^2 935 and 1005, 486^2 3066 and 3233); whole ones are written
// through (128^2 546 and 526, 256^2 980 and 953, 324^2 1665 and 1588).
template <typename T>
bool written_through(int N) { return sizeof(T) == 8 ? N % 4 == 0 : N > 144; }

template <typename T>
hipError_t launch_field_step(hipStream_t st, int N, FieldPtrs<T> in, FieldPtrs<T> out, T *F, double tau,
                             double dtau, int reunit, const KernelTimer &kt) {
    const dim3 grid(field_tiles(N)), block(2 * SX, SY);
    const T th = (T)(tau + 0.5 * dtau);
    if (written_through<T>(N)) GL_LAUNCH_TIMED(kt, k_field_step<T>, grid, block, 0, st, N, in, out, F, (T)tau, (T)dtau, th, reunit);
    else GL_LAUNCH_TIMED(kt, k_field_step_cached<T>, grid, block, 0, st, N, in, out, F, (T)tau, (T)dtau, th, reunit);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_correlators(hipStream_t st, int N, const T *F, const T *U, const CorrCall &c, double dtau,
                              bool streamed) {
    const dim3 blocks((unsigned)(((size_t)N * N + 255) / 256)), wg(256);
#define GL_CORR(S, L, ST)                                                                                          \
    hipLaunchKernelGGL((k_correlators<T, S, L, ST>), blocks, wg, 0, st, N, F, U, c.Is, c.W, c.Il, c.j, dtau, c.part_s, \
                       c.part_l)
    if (c.Is && c.Il) {
        if (streamed) GL_CORR(true, true, true);
        else GL_CORR(true, true, false);
    } else if (c.Is) {
        if (streamed) GL_CORR(true, false, true);
        else GL_CORR(true, false, false);
    } else {
        if (streamed) GL_CORR(false, true, true);
        else GL_CORR(false, true, false);
    }
#undef GL_CORR
    return hipGetLastError();
}

// chunk c of site x of the records, and of the chunk planes [chunk][n2]
template <typename T>
__global__ void __launch_bounds__(256)
k_site_planes(size_t n2, uint4 *__restrict__ records, uint4 *__restrict__ planes, int to_planes) {
    constexpr size_t chunks = kSiteRec * sizeof(T) / 16;
    const size_t at = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (at >= chunks * n2) return;
    const size_t c = at / n2, x = at - c * n2;
    uint4 &r = records[(x / kSiteGroup * chunks + c) * kSiteGroup + x % kSiteGroup];
    if (to_planes) planes[at] = r;
    else r = planes[at];
}

template <typename T>
hipError_t launch_site_planes(hipStream_t st, size_t n2, T *records, void *planes, bool to_planes) {
    constexpr size_t chunks = kSiteRec * sizeof(T) / 16;
    hipLaunchKernelGGL(k_site_planes<T>, dim3((unsigned)((chunks * n2 + 255) / 256)), dim3(256), 0, st, n2,
                       (uint4 *)records, (uint4 *)planes, to_planes ? 1 : 0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_diag(hipStream_t st, int N, FieldPtrs<T> f, double tau, double *partials,
                       int *n_blocks_out) {
    dim3 grid((N + TX - 1) / TX, (N + TY - 1) / TY), block(TX, TY);
    *n_blocks_out = (int)(grid.x * grid.y);
    hipLaunchKernelGGL(k_diag<T>, grid, block, 0, st, N, f, (T)tau, partials);
    return hipGetLastError();
}

#define GL_INST(T)                                                                           \
    template hipError_t launch_field_step<T>(hipStream_t, int, FieldPtrs<T>, FieldPtrs<T>, T *,    \
                                             double, double, int, const KernelTimer &);      \
    template hipError_t launch_diag<T>(hipStream_t, int, FieldPtrs<T>, double, double *, int *);     \
    template hipError_t launch_site_planes<T>(hipStream_t, size_t, T *, void *, bool);                 \
    template hipError_t launch_check_finite<T>(hipStream_t, const T *, int64_t, int64_t, int, int *);   \
    template hipError_t launch_correlators<T>(hipStream_t, int, const T *, const T *, const CorrCall &, double, bool);
// the FP64 instantiations come from fields_f64.hip, which includes this file
// and is compiled with its own scheduling flag
#ifdef GL_FIELDS_FP64
GL_INST(double)
#else
GL_INST(float)
#endif
#undef GL_INST

}  // namespace gl
