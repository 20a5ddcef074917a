// init.hip -- MV-model initial conditions of the Glasma (Sec. 1, "Glasma"),
// computed in FP64 on the device:
//   1. Gaussian color charges rho^a per (nucleus, sheet, site) from Philox,
//      packed two colors per complex plane (rho^{2j} + i rho^{2j+1}).
//   2. Poisson solve (-Lap + m^2) Lambda = rho with the 5-point Laplacian,
//      exact in Fourier space: 2-D FFT by LDS-resident mixed-radix (8, 4, 2, 9, 3)
//      Stockham line transforms, several adjacent lines per workgroup; the
//      kernel multiplication sits between the forward and inverse column
//      transforms of one pass.  The kernel is real and even, so the packed
//      pair separates again after the inverse.  Sheets are processed in
//      chunks (charges, transforms and the Wilson-line products of a chunk
//      in one launch each).
//   3. Wilson lines V = prod_s exp(-i Lambda_s), sheet 1 leftmost.
//   4. Matching of the nuclei's pure-gauge links U^n_i(x) = V_n(x) V_n^dag(x+i)
//      to the forward light cone: [(U^A + U^B)(1 + U^dag)]_X = 0 per link by
//      damped Newton with the analytic Jacobian J_ab = -2 Re Tr(T^a W U^dag T^b),
//      started from the SU(3) projection of W (W^dag)^{-1}, W = U^A + U^B.
//   5. pi0(x) = 1/2 sum_i { [(U_i(x) - 1)(U^B_i(x)^dag - U^A_i(x)^dag)]_X
//                         + [(U_i(x-i)^dag - 1)(U^B_i(x-i) - U^A_i(x-i))]_X },
//      and the first half step E^{1/2} = 0, pi^{1/2} = pi0, U^1 = U^0,
//      phi^1 = dtau * tau_{1/2} * pi0.
#include "internal.hpp"
#include "philox.hpp"
#include "su3.hpp"

#include <algorithm>

namespace gl {

// ---- 1. charges ---------------------------------------------------------------
// colours 2j, 2j + 1 of the charge of one sheet at site x: one counter-based
// draw, two normal deviates, scaled by sigma
__device__ __forceinline__ double2 mv_charge_pair(const MvDraw &mv, int nucleus, int sheet, int j, size_t x) {
#pragma clang fp contract(off)   // the charge itself, also where the transform's sums follow
    U4 w = draw(mv.seed, (uint32_t)x, (uint32_t)(4 * sheet + j), (uint32_t)nucleus);
    double g0, g1;
    box_muller(w, g0, g1);
    return make_double2(mv.sigma * g0, mv.sigma * g1);
}

// sheets sheet0 + blockIdx.y of one nucleus into planes [sheet][4][n2]
__global__ void __launch_bounds__(256)
k_mv_charges(int N, MvDraw mv, double2 *planes) {
    size_t n2 = (size_t)N * N;
    size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n2) return;
    const int sheet = mv.sheet0 + (int)blockIdx.y;
    double2 *pl = planes + (size_t)blockIdx.y * 4 * n2;
#pragma unroll
    for (int j = 0; j < 4; j++) pl[(size_t)j * n2 + x] = mv_charge_pair(mv, mv.nucleus, sheet, j, x);
}

// the caller's charges of consecutive sheets (blockIdx.y), rho [sheet][8][n2]
__global__ void __launch_bounds__(256)
k_pack(int N, const double *rho, double2 *planes) {
    size_t n2 = (size_t)N * N;
    size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n2) return;
    rho += (size_t)blockIdx.y * 8 * n2;
    planes += (size_t)blockIdx.y * 4 * n2;
#pragma unroll
    for (int j = 0; j < 4; j++)
        planes[(size_t)j * n2 + x] = make_double2(rho[(size_t)(2 * j) * n2 + x], rho[(size_t)(2 * j + 1) * n2 + x]);
}

__global__ void __launch_bounds__(256)
k_unpack(int N, const double2 *planes, double *rho) {
    size_t n2 = (size_t)N * N;
    size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n2) return;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        double2 v = planes[(size_t)j * n2 + x];
        rho[(size_t)(2 * j) * n2 + x] = v.x;
        rho[(size_t)(2 * j + 1) * n2 + x] = v.y;
    }
}

// ---- 2. FFT ------------------------------------------------------------------
constexpr int kFftThreads = 256;
constexpr int kFftMaxN = 1024;
constexpr int kFftStaged = kFftMaxN + kFftMaxN / 2;   // stages' twiddles, after tw and s2 in the table
constexpr int kFftElems = 2048;   // complex values per workgroup: C lines of N

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
#pragma clang fp contract(off)   // this order whatever the compiler knows of b's sign
    return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.y, b.x, a.x * b.y));
}

// One stage of the transform of N: radix, butterflies per line, values per
// transform before it and where its twiddles start in the table, with what
// divides an index below kFftElems by nb and Ns: a shift (N a power of two), or
// the multiplier m of t / d = t m >> 21, m = ceil(2^21 / d), exact for t < 2048
// and d <= 1024.
struct FftStage {
    int R, nb, Ns, tw;
    uint32_t nb_m, Ns_m;
};
constexpr int kFftMaxStages = 8;

// The transform of N = 2^a 3^b: radix-8 stages, then at most one radix-4 or
// radix-2, then radix-9 (two radix-3 stages in registers) and at most one
// radix-3.  2^log_c lines a workgroup, ls LDS elements apart.
struct FftPlan {
    int stages, log_c, ls;
    int n_tw;                     // twiddles of all stages, < N
    uint32_t n_m;                 // divides by N
    bool p2;                      // N is a power of two
    FftStage st[kFftMaxStages];
};

// LDS place of value i of a line: one element of padding every eight, so that
// the first stage's results, written eight apart, meet distinct banks
__host__ __device__ inline int fft_pad(int i) { return i + (i >> 3); }

static bool fft_plan(int N, FftPlan &p) {
    p.p2 = (N & (N - 1)) == 0;
    auto divider = [&](int d) -> uint32_t {
        if (!p.p2) return ((1u << 21) + (uint32_t)d - 1) / (uint32_t)d;
        uint32_t s = 0;
        while ((1 << s) < d) s++;
        return s;
    };
    p.stages = 0;
    p.n_tw = 0;
    int m = N, Ns = 1;
    for (int R : {8, 4, 2, 9, 3})
        while (m % R == 0) {
            if (p.stages == kFftMaxStages) return false;
            p.st[p.stages++] = FftStage{R, N / R, Ns, p.n_tw, divider(N / R), divider(Ns)};
            // none in the first stage; radix 9: those of both radix-3 stages
            p.n_tw += R == 9 ? (Ns > 1 ? 8 * Ns : 6 * Ns) : Ns > 1 ? (R - 1) * Ns : 0;
            m /= R;
            Ns *= R;
        }
    if (m != 1) return false;
    // lines per workgroup: the largest power of two that keeps C N within
    // kFftElems, at most 64 (the last group of a plane may hold fewer)
    p.log_c = 0;
    while (p.log_c < 6 && (2 << p.log_c) * N <= kFftElems) p.log_c++;
    // lines are skewed so that a column pass, which fills all C lines of one
    // row together, spreads over the banks too
    p.ls = fft_pad(N - 1) + 1 + std::max(1, 16 >> p.log_c);
    p.n_m = divider(N);
    return true;
}

template <bool P2>
__device__ __forceinline__ int fft_div(int t, uint32_t m) {
    return P2 ? t >> m : (int)(((uint32_t)t * m) >> 21);
}

// radix-R butterfly of v (twiddled inputs), sign = -1 forward, +1 inverse
template <int R>
__device__ __forceinline__ void butterfly(const double2 *v, double2 *o, int sign) {
    if constexpr (R == 2) {
        o[0] = make_double2(v[0].x + v[1].x, v[0].y + v[1].y);
        o[1] = make_double2(v[0].x - v[1].x, v[0].y - v[1].y);
    } else if constexpr (R == 4) {
        double2 a = make_double2(v[0].x + v[2].x, v[0].y + v[2].y);
        double2 b = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
        double2 c = make_double2(v[1].x + v[3].x, v[1].y + v[3].y);
        double2 d = make_double2(v[1].x - v[3].x, v[1].y - v[3].y);
        double2 di = make_double2(-sign * d.y, sign * d.x);   // sign * i * d
        o[0] = make_double2(a.x + c.x, a.y + c.y);
        o[2] = make_double2(a.x - c.x, a.y - c.y);
        o[1] = make_double2(b.x + di.x, b.y + di.y);
        o[3] = make_double2(b.x - di.x, b.y - di.y);
    } else if constexpr (R == 8) {
        // even and odd halves as radix-4 transforms, joined by
        // t_k = exp(sign i pi k / 4): o[k] = E[k] + t_k O[k], o[k+4] = E[k] - t_k O[k]
        const double h = 0.70710678118654752440;
        const double2 ve[4] = {v[0], v[2], v[4], v[6]}, vo[4] = {v[1], v[3], v[5], v[7]};
        double2 E[4], O[4];
        butterfly<4>(ve, E, sign);
        butterfly<4>(vo, O, sign);
        const double2 t1 = make_double2(h * (O[1].x - sign * O[1].y), h * (O[1].y + sign * O[1].x));
        const double2 t2 = make_double2(-sign * O[2].y, sign * O[2].x);
        const double2 t3 = make_double2(-h * (O[3].x + sign * O[3].y), h * (sign * O[3].x - O[3].y));
        o[0] = make_double2(E[0].x + O[0].x, E[0].y + O[0].y);
        o[4] = make_double2(E[0].x - O[0].x, E[0].y - O[0].y);
        o[1] = make_double2(E[1].x + t1.x, E[1].y + t1.y);
        o[5] = make_double2(E[1].x - t1.x, E[1].y - t1.y);
        o[2] = make_double2(E[2].x + t2.x, E[2].y + t2.y);
        o[6] = make_double2(E[2].x - t2.x, E[2].y - t2.y);
        o[3] = make_double2(E[3].x + t3.x, E[3].y + t3.y);
        o[7] = make_double2(E[3].x - t3.x, E[3].y - t3.y);
    } else {   // R == 3
        const double c3 = -0.5, s3 = 0.86602540378443864676 * sign;
        double2 t = make_double2(v[1].x + v[2].x, v[1].y + v[2].y);
        double2 u = make_double2(v[1].x - v[2].x, v[1].y - v[2].y);
        o[0] = make_double2(v[0].x + t.x, v[0].y + t.y);
        // fused by hand: which product joins a sum is otherwise the compiler's
        // choice, and differs between the stages this is inlined in
        const double2 m = make_double2(__builtin_fma(c3, t.x, v[0].x), __builtin_fma(c3, t.y, v[0].y));
        o[1] = make_double2(__builtin_fma(-s3, u.y, m.x), __builtin_fma(s3, u.x, m.y));
        o[2] = make_double2(__builtin_fma(s3, u.y, m.x), __builtin_fma(-s3, u.x, m.y));
    }
}

// Radix-R butterfly of a stage with its twiddles, tw[(r - 1) Ns + k] that of
// (r, k): consecutive lanes read consecutive values, where the table
// exp(-2 pi i j / N) itself was read at strides that met the same banks.  The
// first stage's (Ns = 1) are all 1.  tw holds the forward transform's; the
// inverse uses their conjugates.  Radix 9 is a radix-3 stage and the next one,
// the second's inputs taken from registers: the same operations as the two.
template <int R, bool FIRST>
__device__ __forceinline__ void twiddled(double2 *v, double2 *o, const double2 *tw, int Ns, int k, int sign) {
    auto turn = [&](double2 &x, int at) {
        double2 w = tw[at];
        if (sign > 0) w.y = -w.y;
        x = cmul(x, w);
    };
    if constexpr (R == 9) {
        double2 z[3][3];
#pragma unroll
        for (int m = 0; m < 3; m++) {
            double2 a[3] = {v[m], v[m + 3], v[m + 6]}, b[3];
            if constexpr (!FIRST) {
                turn(a[1], k);
                turn(a[2], Ns + k);
            }
            butterfly<3>(a, b, sign);
#pragma unroll
            for (int r = 0; r < 3; r++) z[r][m] = b[r];
        }
        const double2 *tw2 = FIRST ? tw : tw + 2 * Ns;
        auto turn2 = [&](double2 &x, int at) {
            double2 w = tw2[at];
            if (sign > 0) w.y = -w.y;
            x = cmul(x, w);
        };
#pragma unroll
        for (int r = 0; r < 3; r++) {
            double2 b[3];
            turn2(z[r][1], k + r * Ns);
            turn2(z[r][2], 3 * Ns + k + r * Ns);
            butterfly<3>(z[r], b, sign);
#pragma unroll
            for (int q = 0; q < 3; q++) o[r + 3 * q] = b[q];
        }
    } else {
        if constexpr (!FIRST)
#pragma unroll
            for (int r = 1; r < R; r++) turn(v[r], (r - 1) * Ns + k);
        butterfly<R>(v, o, sign);
    }
}

// What a stage's values come from and go to: in(line, i) and out(line, i, v).
// SYNC: both are the LDS lines, so the workgroup synchronises between.  FAST:
// lanes run over the lines first (global columns) instead of along a line.
template <int R, bool FIRST, bool FAST, bool SYNC, bool P2, class In, class Out>
__device__ __forceinline__ void fft_stage(const double2 *tw, int C, const FftPlan &p, const FftStage &s, int sign,
                                          In in, Out out) {
    constexpr int B = (kFftElems / R + kFftThreads - 1) / kFftThreads;   // butterflies per thread
    double2 v[B][R];
    int line[B], j[B];
#pragma unroll
    for (int b = 0; b < B; b++) {
        const int t = threadIdx.x + b * kFftThreads;
        if constexpr (FAST) {
            line[b] = t & ((1 << p.log_c) - 1);
            j[b] = t >> p.log_c;
            if (line[b] >= C || j[b] >= s.nb) line[b] = -1;
        } else {
            line[b] = fft_div<P2>(t, s.nb_m);
            j[b] = t - line[b] * s.nb;
            if (line[b] >= C) line[b] = -1;
        }
        if (line[b] >= 0)
#pragma unroll
            for (int r = 0; r < R; r++) v[b][r] = in(line[b], j[b] + r * s.nb);
    }
    // radix 9 has twiddles in the first stage too: the table must have arrived
    if constexpr (SYNC || (FIRST && R == 9)) __syncthreads();
#pragma unroll
    for (int b = 0; b < B; b++)
        if (line[b] >= 0) {
            const int q = FIRST ? j[b] : fft_div<P2>(j[b], s.Ns_m), k = FIRST ? 0 : j[b] - q * s.Ns;
            double2 o[R];
            twiddled<R, FIRST>(v[b], o, tw + s.tw, s.Ns, k, sign);
#pragma unroll
            for (int r = 0; r < R; r++) out(line[b], q * s.Ns * R + k + r * s.Ns, o[r]);
        }
}

template <bool FIRST, bool FAST, bool SYNC, bool P2, class In, class Out>
__device__ __forceinline__ void fft_stage_any(const double2 *tw, int C, const FftPlan &p, int s, int sign, In in,
                                              Out out) {
    const FftStage &st = p.st[s];
    if (st.R == 8) fft_stage<8, FIRST, FAST, SYNC, P2>(tw, C, p, st, sign, in, out);
    else if (st.R == 4) fft_stage<4, FIRST, FAST, SYNC, P2>(tw, C, p, st, sign, in, out);
    else if (P2 || st.R == 2) fft_stage<2, FIRST, FAST, SYNC, P2>(tw, C, p, st, sign, in, out);
    else if constexpr (!P2) {
        if (st.R == 9) fft_stage<9, FIRST, FAST, SYNC, P2>(tw, C, p, st, sign, in, out);
        else fft_stage<3, FIRST, FAST, SYNC, P2>(tw, C, p, st, sign, in, out);
    }
}

// The last stage of the forward transform, f(line, i, v) on its results and the
// first stage of the inverse, for a plan whose first and last radix are the
// same: a butterfly's results are then the inputs of the inverse's butterfly
// of the same index, and stay in registers.
template <int R, bool P2, class F>
__device__ __forceinline__ void fft_turn(double2 *buf, const double2 *tw, int C, const FftPlan &p, F f) {
    constexpr int B = (kFftElems / R + kFftThreads - 1) / kFftThreads;
    const FftStage &s = p.st[p.stages - 1];              // Ns = nb: q = 0, k = j
    double2 o[B][R];
    int line[B], j[B];
#pragma unroll
    for (int b = 0; b < B; b++) {
        const int t = threadIdx.x + b * kFftThreads;
        line[b] = fft_div<P2>(t, s.nb_m);
        j[b] = t - line[b] * s.nb;
        if (line[b] >= C) line[b] = -1;
        if (line[b] >= 0) {
            double2 v[R], u[R];
#pragma unroll
            for (int r = 0; r < R; r++) v[r] = buf[line[b] * p.ls + fft_pad(j[b] + r * s.nb)];
            twiddled<R, false>(v, u, tw + s.tw, s.Ns, j[b], -1);
#pragma unroll
            for (int r = 0; r < R; r++) u[r] = f(line[b], j[b] + r * s.nb, u[r]);
            twiddled<R, true>(u, o[b], tw + p.st[0].tw, 1, 0, +1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < B; b++)
        if (line[b] >= 0)
#pragma unroll
            for (int r = 0; r < R; r++) buf[line[b] * p.ls + fft_pad(j[b] * R + r)] = o[b][r];
    __syncthreads();
}

// stages first .. end - 1 (not the first of the transform) on the LDS lines
template <bool P2>
__device__ __forceinline__ void fft_stages(double2 *buf, const double2 *tw, int C, int sign, const FftPlan &p,
                                           int first, int end) {
    auto in = [&](int line, int i) { return buf[line * p.ls + fft_pad(i)]; };
    auto out = [&](int line, int i, double2 v) { buf[line * p.ls + fft_pad(i)] = v; };
    for (int s = first; s < end; s++) {
        fft_stage_any<false, false, true, P2>(tw, C, p, s, sign, in, out);
        __syncthreads();
    }
}

// Tables of one solve, filled once: tw[j] = exp(-2 pi i j / N) and
// s2[j] = 4 sin^2(pi j / N), j < N, and the stages' twiddles in their own order.
__device__ __forceinline__ double2 unit_root(int j, int N) {
    double sn, cs;
    sincospi(2.0 * (double)j / (double)N, &sn, &cs);
    return make_double2(cs, -sn);
}
__global__ void __launch_bounds__(256)
k_fft_tables(int N, FftPlan p, double2 *__restrict__ tw, double *__restrict__ s2, double2 *__restrict__ staged) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    tw[j] = unit_root(j, N);
    const double h = sinpi((double)j / (double)N);
    s2[j] = 4.0 * h * h;
    if (j >= p.n_tw) return;
    int s = p.stages - 1;
    while (p.st[s].tw > j) s--;
    int R = p.st[s].R, Ns = p.st[s].Ns, e = j - p.st[s].tw;
    if (R == 9) {
        const int n1 = Ns > 1 ? 2 * Ns : 0;              // the first of its radix-3 stages, then the second
        R = 3;
        if (e >= n1) {
            e -= n1;
            Ns *= 3;
        }
    }
    staged[j] = unit_root((e / Ns + 1) * (e % Ns) * (N / (Ns * R)), N);
}

// In-place transforms of the N x N planes: each workgroup transforms C
// adjacent lines of one plane (rows, or columns in MODE kFftPoisson), the
// twiddles copied from the solve's table into LDS.  The first stage takes its
// values from global memory (rows along the lines; columns C consecutive values
// of each row) and the last writes its results there, so LDS holds them only
// between stages.  sign = -1 forward, +1 inverse (unnormalised).  MODE
// kFftPoisson (after the forward row pass): the forward column transform, the
// multiplication of mode (kx, ky) by 1 / (N^2 (4 sin^2(pi kx/N) + 4 sin^2(pi
// ky/N) + m2)) (zero above uv2 > 0) and the inverse column transform, in one
// pass.  MODE kFftDraw (forward rows): the input lines are the MV charges, drawn
// here instead of being written to the planes by a pass of their own and read
// back.  Planes are [nucleus][sheet][4], mv.sheets sheets of each nucleus.
//
// Bound: by LDS and its latency (values in and out at every stage, and their
// twiddles); the inverse row pass is at 7 TB/s with what it reads and writes.
// Of 16 LDS passes of a column of 512 values (in, three stages forward, product,
// three back, out) the direct ends, and the last stage forward, the product and
// the first back in registers, leave 8; and the staged twiddles meet no bank
// twice.  Eight sheets of 512^2, 134 MB of planes: columns 84 -> 57 us, inverse
// rows 48 -> 38, forward rows with the draw 85 -> 76 (bound by the draw's
// arithmetic: 172 FP64 instructions a pair, most of them the logarithm's and the
// sine's).  3^5, both nuclei and 17 sheets: columns 136 -> 83.
constexpr int kFftLines = 0, kFftPoisson = 1, kFftDraw = 2;
template <int MODE, bool P2>
__global__ void __launch_bounds__(kFftThreads)
k_fft_lines(double2 *data, int N, int groups_per_plane, int sign, FftPlan fp, double m2, double uv2,
            const double2 *__restrict__ tw_tab, const double *__restrict__ s2_tab, MvDraw mv) {
    constexpr bool POISSON = MODE == kFftPoisson;
    // dynamic LDS sized for this N: the lines, then tw, then (POISSON) s2[N]
    extern __shared__ double2 lds[];
    double2 *buf = lds, *tw = lds + (fp.ls << fp.log_c);
    double *s2 = (double *)(tw + fp.n_tw);
    // contiguous runs of groups per XCD: the C-wide column segments of
    // neighbouring groups share cache lines, which then meet in one L2
    const int bid = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int plane = bid / groups_per_plane, l0 = (bid - plane * groups_per_plane) << fp.log_c;
    const int C = min(1 << fp.log_c, N - l0), last = fp.stages - 1;
    double2 *base = data + (size_t)plane * N * N;
    for (int j = threadIdx.x; j < fp.n_tw; j += kFftThreads) tw[j] = tw_tab[j];
    if constexpr (POISSON)
        for (int j = threadIdx.x; j < N; j += kFftThreads) s2[j] = s2_tab[j];
    auto from_lds = [&](int line, int i) { return buf[line * fp.ls + fft_pad(i)]; };
    auto to_lds = [&](int line, int i, double2 v) { buf[line * fp.ls + fft_pad(i)] = v; };
    auto place = [&](int line, int i) {
        return POISSON ? (uint32_t)(i * N + (l0 + line)) : (uint32_t)((l0 + line) * N + i);
    };
    const int sheet = plane / 4;
    auto input = [&](int line, int i) {
        if constexpr (MODE == kFftDraw)
            return mv_charge_pair(mv, mv.nucleus + sheet / mv.sheets, mv.sheet0 + sheet % mv.sheets, plane % 4,
                                  place(line, i));
        else return base[place(line, i)];
    };
    // the charges' rows are written through the L2 caches, beside the arithmetic
    // they are drawn with (76.2 -> 74.2 us at 512^2, 61.1 -> 58.5 at 256^2); a pass
    // bound by memory is slower for it (inverse rows 38.9 -> 42.1)
    auto output = [&](int line, int i, double2 v) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), gl::buf(base), place(line, i) * 16u, 0u,
                                               MODE == kFftDraw ? kWriteThrough : 0);
    };
    if constexpr (POISSON) {
        const double nn = (double)N * (double)N;
        auto poisson = [&](int line, int i, double2 v) {                 // kx = l0 + line, ky = i
#pragma clang fp contract(off)                                           // a product of its own, also before a sum
            const double k2 = s2[l0 + line] + s2[i];
            const double gk = (uv2 > 0.0 && k2 > uv2) ? 0.0 : 1.0 / (nn * (k2 + m2));
            return make_double2(v.x * gk, v.y * gk);
        };
        auto scaled = [&](int line, int i, double2 v) { to_lds(line, i, poisson(line, i, v)); };
        fft_stage_any<true, true, false, P2>(tw, C, fp, 0, -1, input, to_lds);
        __syncthreads();
        fft_stages<P2>(buf, tw, C, -1, fp, 1, last);
        const bool same = last > 0 && fp.st[last].R == fp.st[0].R;
        if (same && fp.st[0].R == 8) fft_turn<8, P2>(buf, tw, C, fp, poisson);
        else if (!P2 && same && fp.st[0].R == 9) fft_turn<9, P2>(buf, tw, C, fp, poisson);
        else {
            // the results to LDS, scaled, and back for the inverse's first stage
            if (last > 0) fft_stage_any<false, false, true, P2>(tw, C, fp, last, -1, from_lds, scaled);
            else
                for (int t = threadIdx.x; t < C * N; t += kFftThreads) {
                    const int line = fft_div<P2>(t, fp.n_m), i = t - line * N;
                    scaled(line, i, from_lds(line, i));
                }
            __syncthreads();
            if (last > 0) fft_stage_any<true, false, true, P2>(tw, C, fp, 0, +1, from_lds, to_lds);
            else fft_stage_any<true, true, false, P2>(tw, C, fp, 0, +1, from_lds, output);
            __syncthreads();
        }
        fft_stages<P2>(buf, tw, C, +1, fp, 1, last);
        if (last > 0) fft_stage_any<false, true, false, P2>(tw, C, fp, last, +1, from_lds, output);
    } else if (last == 0) {
        fft_stage_any<true, false, false, P2>(tw, C, fp, 0, sign, input, output);
    } else {
        fft_stage_any<true, false, false, P2>(tw, C, fp, 0, sign, input, to_lds);
        __syncthreads();
        fft_stages<P2>(buf, tw, C, sign, fp, 1, last);
        fft_stage_any<false, false, false, P2>(tw, C, fp, last, sign, from_lds, output);
    }
}

// ---- 3. Wilson lines --------------------------------------------------------
__global__ void __launch_bounds__(256)
k_wilson_init(int N, double *V) {
    size_t n2 = (size_t)N * N;
    size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n2) return;
    store_m(V, n2, x, m_ident<double>());
}

// V <- V exp(-i Lambda_s) for the n_sheets sheets of planes [sheet][4][n2], in
// sheet order (earlier sheets to the left), starting from V = 1 when first;
// nucleus blockIdx.y of planes [nucleus][sheet][4][n2] into V0 or V1.  Each
// sheet's values are loaded while the one before is exponentiated: the chain
// of a site is serial, and with two waves a SIMD the loads were its latency.
__global__ void __launch_bounds__(256)
k_wilson_accum(int N, const double2 *__restrict__ planes, int n_sheets, int first, double *__restrict__ V0,
               double *__restrict__ V1) {
    size_t n2 = (size_t)N * N;
    size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n2) return;
    planes += (size_t)blockIdx.y * n_sheets * 4 * n2;
    double *V = blockIdx.y == 0 ? V0 : V1;
    double2 next[4];
#pragma unroll
    for (int j = 0; j < 4; j++) next[j] = planes[(size_t)j * n2 + x];
    M3<double> v = first ? m_ident<double>() : load_m(V, n2, x);
#pragma unroll 1
    for (int s = 0; s < n_sheets; s++) {
        double lam[8];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            lam[2 * j] = next[j].x;
            lam[2 * j + 1] = next[j].y;
        }
        const size_t s1 = (size_t)min(s + 1, n_sheets - 1);
#pragma unroll
        for (int j = 0; j < 4; j++) next[j] = planes[(s1 * 4 + j) * n2 + x];
        v = mul(v, expi_alg(lam, -1.0));
    }
    store_m(V, n2, x, v);
}

// ---- dipole correlator (calibration of Q_s) -----------------------------------
// D(r) sums Re Tr V(x) V^dag(x + r e_d) over the sites and both directions, which
// is the autocorrelation of the nine complex entries along the lines of each
// direction: sum_x z(x) z*(x + r) = 1/N sum_k |Z_k|^2 cos(2 pi k r / N) with Z the
// transform of the line.  One pass over V per direction instead of one over V
// and its neighbours per separation (256^2, r <= 128: 206 -> 24 us).  Lattices the
// line transforms do not take and calls for a few separations (dipole_by_spectra) sum
// the sites of each separation.

// Workgroup (b, r): the sum over its 256 sites of Re Tr V(x) V^dag(x + r e_d),
// d = x, y; part[r][b]
__global__ void __launch_bounds__(256)
k_dipole_sites(int N, const double *__restrict__ V, double *__restrict__ part) {
    __shared__ double red[256];
    const size_t n2 = (size_t)N * N;
    const size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    double v = 0.0;
    if (x < n2) {
        const int ix = (int)(x % N), iy = (int)(x / N);
        const M3<double> a = load_m(V, n2, x);
        const size_t nb[2] = {(size_t)((ix + r) % N) + (size_t)N * iy, (size_t)ix + (size_t)N * ((iy + r) % N)};
#pragma unroll
        for (int d = 0; d < 2; d++) {
            const M3<double> b = load_m(V, n2, nb[d]);
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) v += a.re[i][j] * b.re[i][j] + a.im[i][j] * b.im[i][j];
        }
    }
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)r * gridDim.x + blockIdx.x] = red[0];
}

// D[r] = (sum of the nb partials of r in a fixed order) / (6 N^2)
__global__ void __launch_bounds__(256)
k_dipole_mean(int N, const double *__restrict__ part, int nb, double *__restrict__ D) {
    __shared__ double red[256];
    const int r = blockIdx.x;
    double v = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) v += part[(size_t)r * nb + b];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) D[r] = red[0] / (6.0 * (double)N * (double)N);
}

// Power spectra of C lines of entry blockIdx.y % 9 (rows for blockIdx.y < 9, else
// columns), summed over the lines: part[y][group][N]
template <bool P2>
__global__ void __launch_bounds__(kFftThreads)
k_dipole_lines(const double *__restrict__ V, int N, FftPlan fp, const double2 *__restrict__ tw_tab,
               double *__restrict__ part) {
    extern __shared__ double2 lds[];
    double2 *buf = lds, *tw = lds + (fp.ls << fp.log_c);
    const size_t n2 = (size_t)N * N;
    const int entry = blockIdx.y % 9, l0 = blockIdx.x << fp.log_c, C = min(1 << fp.log_c, N - l0);
    const bool cols = blockIdx.y >= 9;
    const double *re = V + (size_t)(2 * entry) * n2, *im = re + n2;
    for (int j = threadIdx.x; j < fp.n_tw; j += kFftThreads) tw[j] = tw_tab[j];
    auto to_lds = [&](int line, int i, double2 v) { buf[line * fp.ls + fft_pad(i)] = v; };
    auto entry_at = [&](size_t at) { return make_double2(re[at], im[at]); };
    if (cols)
        fft_stage_any<true, true, false, P2>(
            tw, C, fp, 0, -1, [&](int line, int i) { return entry_at((size_t)i * N + (l0 + line)); }, to_lds);
    else
        fft_stage_any<true, false, false, P2>(
            tw, C, fp, 0, -1, [&](int line, int i) { return entry_at((size_t)(l0 + line) * N + i); }, to_lds);
    __syncthreads();
    fft_stages<P2>(buf, tw, C, -1, fp, 1, fp.stages);
    double *out = part + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * N;
    for (int k = threadIdx.x; k < N; k += kFftThreads) {
        double s = 0.0;
        for (int line = 0; line < C; line++) {
            const double2 z = buf[line * fp.ls + fft_pad(k)];
            s += z.x * z.x + z.y * z.y;
        }
        out[k] = s;
    }
}

// S[k] = sum of the n partial spectra, 16 values of k a workgroup
__global__ void __launch_bounds__(256)
k_dipole_sum(int N, const double *__restrict__ part, int n, double *__restrict__ S) {
    __shared__ double red[256];
    const int t = threadIdx.x, k = blockIdx.x * 16 + (t & 15);
    double v = 0.0;
    if (k < N)
#pragma unroll 4
        for (int b = t >> 4; b < n; b += 16) v += part[(size_t)b * N + k];
    red[t] = v;
    __syncthreads();
    for (int w = 128; w >= 16; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    if (t < 16 && k < N) S[k] = red[t];
}

// D[r] = 1 / (6 N^3) sum_k S[k] cos(2 pi k r / N)
__global__ void __launch_bounds__(256)
k_dipole_curve(int N, const double *__restrict__ S, const double2 *__restrict__ tw, double *__restrict__ D) {
    __shared__ double red[256];
    const int r = blockIdx.x;
    double v = 0.0;
    for (int k = threadIdx.x; k < N; k += 256) v += S[k] * tw[(int)(((int64_t)k * r) % N)].x;
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) D[r] = red[0] / (6.0 * (double)N * (double)N * (double)N);
}

// ---- 4. matching ------------------------------------------------------------
__device__ inline void cdiv(double ar, double ai, double br, double bi, double &cr, double &ci) {
    double d = br * br + bi * bi;
    cr = (ar * br + ai * bi) / d;
    ci = (ai * br - ar * bi) / d;
}

__device__ inline void det3(const M3<double> &a, double &dr, double &di) {
    auto cm = [](double xr, double xi, double yr, double yi, double &zr, double &zi) {
        zr = xr * yr - xi * yi;
        zi = xr * yi + xi * yr;
    };
    double r = 0, i = 0;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        double m1r, m1i, m2r, m2i;
        cm(a.re[1][c1], a.im[1][c1], a.re[2][c2], a.im[2][c2], m1r, m1i);
        cm(a.re[1][c2], a.im[1][c2], a.re[2][c1], a.im[2][c1], m2r, m2i);
        double cofr = m1r - m2r, cofi = m1i - m2i;
        double tr, ti;
        cm(a.re[0][c], a.im[0][c], cofr, cofi, tr, ti);
        r += tr;
        i += ti;
    }
    dr = r;
    di = i;
}

// inverse by cofactors
__device__ inline M3<double> inv3(const M3<double> &a) {
    double dr, di;
    det3(a, dr, di);
    M3<double> r;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            int i1 = (i + 1) % 3, i2 = (i + 2) % 3, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
            double pr = a.re[i1][j1] * a.re[i2][j2] - a.im[i1][j1] * a.im[i2][j2];
            double pi = a.re[i1][j1] * a.im[i2][j2] + a.im[i1][j1] * a.re[i2][j2];
            double qr = a.re[i1][j2] * a.re[i2][j1] - a.im[i1][j2] * a.im[i2][j1];
            double qi = a.re[i1][j2] * a.im[i2][j1] + a.im[i1][j2] * a.re[i2][j1];
            double cr, ci;
            cdiv(pr - qr, pi - qi, dr, di, cr, ci);
            r.re[j][i] = cr;
            r.im[j][i] = ci;
        }
    return r;
}

__device__ inline M3<double> dagger(const M3<double> &a) {
    M3<double> r;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) { r.re[i][j] = a.re[j][i]; r.im[i][j] = -a.im[j][i]; }
    return r;
}

// unitary polar factor by X <- (X + X^{-dag})/2, then principal cube root of det removed
__device__ inline M3<double> su3_project(M3<double> X) {
    for (int it = 0; it < 100; it++) {
        M3<double> Y = add(X, dagger(inv3(X)));
        double ch = 0;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                Y.re[i][j] *= 0.5;
                Y.im[i][j] *= 0.5;
                double a = Y.re[i][j] - X.re[i][j], b = Y.im[i][j] - X.im[i][j];
                ch += a * a + b * b;
            }
        X = Y;
        if (sqrt(ch) < 1e-15) break;
    }
    double dr, di;
    det3(X, dr, di);
    double th = atan2(di, dr) / 3.0;
    double s, c;
    sincos(-th, &s, &c);
    M3<double> r;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            r.re[i][j] = X.re[i][j] * c - X.im[i][j] * s;
            r.im[i][j] = X.re[i][j] * s + X.im[i][j] * c;
        }
    return r;
}

__device__ inline double match_residual(const M3<double> &W, const M3<double> &U, double *R) {
    M3<double> M = add(W, mul_nd(W, U));   // W (1 + U^dag)
    alg_proj(M, R);
    double m = 0;
#pragma unroll
    for (int a = 0; a < 8; a++) m = fmax(m, fabs(R[a]));
    return m;
}

// Gaussian elimination with partial pivoting, unrolled so that J and b stay
// in registers: each column's largest remaining entry is moved to the pivot
// row by conditional swaps with the rows below it.
__device__ inline bool solve8(double J[8][8], double *b) {
#pragma unroll
    for (int c = 0; c < 8; c++) {
#pragma unroll
        for (int r = c + 1; r < 8; r++) {
            const bool sw = fabs(J[r][c]) > fabs(J[c][c]);
#pragma unroll
            for (int k = c; k < 8; k++) {
                const double t = J[c][k];
                J[c][k] = sw ? J[r][k] : t;
                J[r][k] = sw ? t : J[r][k];
            }
            const double t = b[c];
            b[c] = sw ? b[r] : t;
            b[r] = sw ? t : b[r];
        }
        if (J[c][c] == 0.0) return false;
#pragma unroll
        for (int r = c + 1; r < 8; r++) {
            const double f = J[r][c] / J[c][c];
#pragma unroll
            for (int k = c; k < 8; k++) J[r][k] -= f * J[c][k];
            b[r] -= f * b[c];
        }
    }
#pragma unroll
    for (int i = 7; i >= 0; i--) {
        double s = b[i];
#pragma unroll
        for (int k = i + 1; k < 8; k++) s -= J[i][k] * b[k];
        b[i] = s / J[i][i];
    }
    return true;
}

__device__ inline M3<double> nucleus_link(const double *V, size_t n2, size_t x, size_t xp) {
    return mul_nd(load_m(V, n2, x), load_m(V, n2, xp));
}

// one thread per link (d, x)
__global__ void __launch_bounds__(128)
k_match(int N, const double *VA, const double *VB, double *U0, int *status, int max_iter,
        double tol) {
    size_t n2 = (size_t)N * N;
    size_t t = (size_t)blockIdx.x * 128 + threadIdx.x;
    if (t >= 2 * n2) return;
    int d = (int)(t / n2);
    size_t x = t % n2;
    int ix = (int)(x % N), iy = (int)(x / N);
    size_t xp = d == 0 ? (size_t)(ix + 1 == N ? 0 : ix + 1) + (size_t)N * iy
                       : (size_t)ix + (size_t)N * (iy + 1 == N ? 0 : iy + 1);
    M3<double> W = add(nucleus_link(VA, n2, x, xp), nucleus_link(VB, n2, x, xp));
    M3<double> U = su3_project(mul(W, inv3(dagger(W))));
    double R[8];
    double rn = match_residual(W, U, R);
    int it = 0;
    while (rn >= tol && it < max_iter) {
        M3<double> M = mul_nd(W, U);
        double J[8][8];
        // unrolled: e is a constant unit vector, so M T^b folds to the few
        // non-zero entries of the generator
#pragma unroll
        for (int b = 0; b < 8; b++) {
            double e[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            e[b] = 1.0;
            double col[8];
            alg_from_herm(mul(M, herm_from_alg(e)), col);   // 2 Re Tr(T^a M T^b)
            for (int a = 0; a < 8; a++) J[a][b] = -col[a];
        }
        double dl[8];
        for (int a = 0; a < 8; a++) dl[a] = -R[a];
        if (!solve8(J, dl)) break;
        double step = 1.0, rnn = rn, Rn[8];
        M3<double> Un = U;
        for (int h = 0; h < 40; h++) {
            Un = mul(expi_alg(dl, step), U);
            rnn = match_residual(W, Un, Rn);
            if (rnn < rn) break;
            step *= 0.5;
        }
        U = Un;
        for (int a = 0; a < 8; a++) R[a] = Rn[a];
        rn = rnn;
        it++;
    }
    store_m(U0 + (size_t)d * 18 * n2, n2, x, U);
    if (!(rn < tol)) atomicOr(status, 1);
}

// ---- 5. pi0 -------------------------------------------------------------------
__global__ void __launch_bounds__(128)
k_pi0(int N, const double *VA, const double *VB, const double *U0, double *pi0) {
    size_t n2 = (size_t)N * N;
    size_t x = (size_t)blockIdx.x * 128 + threadIdx.x;
    if (x >= n2) return;
    int ix = (int)(x % N), iy = (int)(x / N);
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int d = 0; d < 2; d++) {
        int pxi = d == 0 ? (ix + 1 == N ? 0 : ix + 1) : ix, pyi = d == 0 ? iy : (iy + 1 == N ? 0 : iy + 1);
        int mxi = d == 0 ? (ix == 0 ? N - 1 : ix - 1) : ix, myi = d == 0 ? iy : (iy == 0 ? N - 1 : iy - 1);
        size_t xp = (size_t)pxi + (size_t)N * pyi, xm = (size_t)mxi + (size_t)N * myi;
        M3<double> one = m_ident<double>();
        {
            M3<double> u = load_m(U0 + (size_t)d * 18 * n2, n2, x);
            M3<double> ua = nucleus_link(VA, n2, x, xp), ub = nucleus_link(VB, n2, x, xp);
            M3<double> m = mul(sub(u, one), sub(dagger(ub), dagger(ua)));
            double v[8];
            alg_proj(m, v);
            for (int a = 0; a < 8; a++) acc[a] += v[a];
        }
        {
            M3<double> u = load_m(U0 + (size_t)d * 18 * n2, n2, xm);
            M3<double> ua = nucleus_link(VA, n2, xm, x), ub = nucleus_link(VB, n2, xm, x);
            M3<double> m = mul(sub(dagger(u), one), sub(ub, ua));
            double v[8];
            alg_proj(m, v);
            for (int a = 0; a < 8; a++) acc[a] += v[a];
        }
    }
    for (int a = 0; a < 8; a++) pi0[(size_t)a * n2 + x] = 0.5 * acc[a];
}

template <typename T>
__global__ void __launch_bounds__(256)
k_first_half_step(int N, const double *U0, const double *pi0, FieldPtrs<T> out, double dtau) {
    size_t n2 = (size_t)N * N;
    size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n2) return;
    // the field state is stored in chunked planes, written here in whole
    // chunks; it keeps the first two rows of each link
    constexpr int NV = 16 / (int)sizeof(T);
    for (int d = 0; d < 2; d++) {
        T v[kLinkVals];
        for (int c = 0; c < kLinkVals; c++) v[c] = (T)U0[(size_t)(18 * d + c) * n2 + x];
        for (int c = 0; c < kLinkVals; c += NV) chunk_st16(out.U, n2, x, kLinkVals * d + c, v + c);
    }
    const T zero[NV] = {};
    for (int c = 0; c < 16; c += NV) chunk_st16(out.E, n2, x, c, zero);
    const double th = 0.5 * dtau;
    T pv[8], fv[8];
    for (int a = 0; a < 8; a++) {
        double p = pi0[(size_t)a * n2 + x];
        pv[a] = (T)p;
        fv[a] = (T)(dtau * th * p);
    }
    for (int a = 0; a < 8; a += NV) {
        chunk_st16(out.pi, n2, x, a, pv + a);
        chunk_st16(out.phi, n2, x, a, fv + a);
    }
}

// ---- launchers ----------------------------------------------------------------
static inline unsigned blocks_for(size_t n, unsigned b) { return (unsigned)((n + b - 1) / b); }

hipError_t launch_mv_charges(hipStream_t st, int N, double sigma, uint64_t seed, int nucleus,
                             int sheet0, int n_sheets, double2 *planes) {
    const MvDraw mv{sigma, seed, nucleus, sheet0, n_sheets};
    hipLaunchKernelGGL(k_mv_charges, dim3(blocks_for((size_t)N * N, 256), n_sheets), dim3(256), 0, st, N, mv,
                       planes);
    return hipGetLastError();
}

hipError_t launch_charges_to_planes(hipStream_t st, int N, const double *rho, int n_sheets, double2 *planes) {
    hipLaunchKernelGGL(k_pack, dim3(blocks_for((size_t)N * N, 256), n_sheets), dim3(256), 0, st, N, rho, planes);
    return hipGetLastError();
}

hipError_t launch_planes_to_charges(hipStream_t st, int N, const double2 *planes, double *rho) {
    hipLaunchKernelGGL(k_unpack, dim3(blocks_for((size_t)N * N, 256)), dim3(256), 0, st, N, planes, rho);
    return hipGetLastError();
}

hipError_t launch_fft_tables(hipStream_t st, int N, double2 *tab) {
    FftPlan fp;
    if (N > kFftMaxN || !fft_plan(N, fp)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fft_tables, dim3((N + 255) / 256), dim3(256), 0, st, N, fp, tab, (double *)(tab + kFftMaxN),
                       tab + kFftStaged);
    return hipGetLastError();
}

// Poisson solve of n_planes planes: forward row transforms, the fused
// column pass (forward, kernel, inverse) and inverse row transforms; tab
// holds the tables of launch_fft_tables for this N.  With draw, the forward
// row pass draws the MV charges itself (the planes' input is not read).
template <bool P2>
static void poisson_passes(hipStream_t st, int N, double m2, double uv2, double2 *planes, int n_planes,
                           const double2 *tab, const MvDraw *draw, const FftPlan &fp) {
    const int groups = (N + (1 << fp.log_c) - 1) >> fp.log_c;
    const double *s2 = (const double *)(tab + kFftMaxN);
    const double2 *tw = tab + kFftStaged;
    const size_t lds_lines = ((size_t)(fp.ls << fp.log_c) + fp.n_tw) * sizeof(double2);
    const size_t lds_poisson = lds_lines + N * sizeof(double);
    const MvDraw mv = draw ? *draw : MvDraw{0.0, 0, 0, 0, 1};
    const dim3 grid(n_planes * groups), wg(kFftThreads);
    if (draw)
        hipLaunchKernelGGL((k_fft_lines<kFftDraw, P2>), grid, wg, lds_lines, st, planes, N, groups, -1, fp, m2,
                           uv2, tw, s2, mv);
    else
        hipLaunchKernelGGL((k_fft_lines<kFftLines, P2>), grid, wg, lds_lines, st, planes, N, groups, -1, fp, m2,
                           uv2, tw, s2, mv);
    hipLaunchKernelGGL((k_fft_lines<kFftPoisson, P2>), grid, wg, lds_poisson, st, planes, N, groups, -1, fp, m2,
                       uv2, tw, s2, mv);
    hipLaunchKernelGGL((k_fft_lines<kFftLines, P2>), grid, wg, lds_lines, st, planes, N, groups, +1, fp, m2, uv2,
                       tw, s2, mv);
}

hipError_t launch_poisson(hipStream_t st, int N, double m2, double uv2, double2 *planes, int n_planes,
                          const double2 *tab, const MvDraw *draw) {
    FftPlan fp;
    if (N > kFftMaxN || !fft_plan(N, fp)) return hipErrorInvalidValue;
    if (fp.p2) poisson_passes<true>(st, N, m2, uv2, planes, n_planes, tab, draw, fp);
    else poisson_passes<false>(st, N, m2, uv2, planes, n_planes, tab, draw, fp);
    return hipGetLastError();
}

// The spectra cost the same for any rmax, the sums over sites two reads of V a
// separation, and one launch less: a call for rmax = 1, 2, 4 by sums and by spectra,
// 256^2 29.6, 32.0, 37 and 37.5 us, 512^2 44, 55, 71 and 75, 1024^2 118, 155, 232 and 291;
// 64^2 28.8 to 31.5 up to rmax = 32 and 31.6 to 33.5.
bool dipole_by_spectra(int N, int rmax) {
    FftPlan fp;
    return N > 64 && rmax > 4 && N <= kFftMaxN && fft_plan(N, fp);
}

size_t dipole_scratch(int N, int rmax) {
    FftPlan fp;
    if (!dipole_by_spectra(N, rmax) || !fft_plan(N, fp)) return (size_t)(rmax + 1) * blocks_for((size_t)N * N, 256);
    const size_t groups = (N + (1 << fp.log_c) - 1) >> fp.log_c;
    return 18 * groups * N + N;
}

hipError_t launch_dipole(hipStream_t st, int N, const double *V, int rmax, const double2 *tab, double *scratch,
                         double *D) {
    FftPlan fp;
    if (!dipole_by_spectra(N, rmax) || !fft_plan(N, fp)) {
        const int nb = (int)blocks_for((size_t)N * N, 256);
        hipLaunchKernelGGL(k_dipole_sites, dim3(nb, rmax + 1), dim3(256), 0, st, N, V, scratch);
        hipLaunchKernelGGL(k_dipole_mean, dim3(rmax + 1), dim3(256), 0, st, N, (const double *)scratch, nb, D);
        return hipGetLastError();
    }
    const int groups = (N + (1 << fp.log_c) - 1) >> fp.log_c;
    double *S = scratch, *part = scratch + N;
    const size_t lds = ((size_t)(fp.ls << fp.log_c) + fp.n_tw) * sizeof(double2);
    if (fp.p2)
        hipLaunchKernelGGL(k_dipole_lines<true>, dim3(groups, 18), dim3(kFftThreads), lds, st, V, N, fp, tab + kFftStaged,
                           part);
    else
        hipLaunchKernelGGL(k_dipole_lines<false>, dim3(groups, 18), dim3(kFftThreads), lds, st, V, N, fp, tab + kFftStaged,
                           part);
    hipLaunchKernelGGL(k_dipole_sum, dim3((N + 15) / 16), dim3(256), 0, st, N, (const double *)part, 18 * groups, S);
    hipLaunchKernelGGL(k_dipole_curve, dim3(rmax + 1), dim3(256), 0, st, N, (const double *)S, tab, D);
    return hipGetLastError();
}

hipError_t launch_wilson_init(hipStream_t st, int N, double *V) {
    hipLaunchKernelGGL(k_wilson_init, dim3(blocks_for((size_t)N * N, 256)), dim3(256), 0, st, N, V);
    return hipGetLastError();
}

hipError_t launch_wilson_accum(hipStream_t st, int N, const double2 *planes, int n_sheets, bool first, int n_nuclei,
                               double *V0, double *V1) {
    hipLaunchKernelGGL(k_wilson_accum, dim3(blocks_for((size_t)N * N, 256), n_nuclei), dim3(256), 0, st, N, planes,
                       n_sheets, first ? 1 : 0, V0, V1);
    return hipGetLastError();
}

hipError_t launch_match_pi0(hipStream_t st, int N, const double *VA, const double *VB, double *U0,
                           double *pi0, int *status, int max_iter, double tol) {
    size_t n2 = (size_t)N * N;
    hipLaunchKernelGGL(k_match, dim3(blocks_for(2 * n2, 128)), dim3(128), 0, st, N, VA, VB, U0, status,
                       max_iter, tol);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pi0, dim3(blocks_for(n2, 128)), dim3(128), 0, st, N, VA, VB, U0, pi0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_first_half_step(hipStream_t st, int N, const double *U0, const double *pi0,
                                  FieldPtrs<T> out, double dtau) {
    hipLaunchKernelGGL(k_first_half_step<T>, dim3(blocks_for((size_t)N * N, 256)), dim3(256), 0, st, N,
                       U0, pi0, out, dtau);
    return hipGetLastError();
}

template hipError_t launch_first_half_step<double>(hipStream_t, int, const double *, const double *,
                                                   FieldPtrs<double>, double);
template hipError_t launch_first_half_step<float>(hipStream_t, int, const double *, const double *,
                                                  FieldPtrs<float>, double);

}  // namespace gl
