// batch_kernels.hip -- many events of uneven lattice and ensemble size in one
// launch per phase.  Work is flattened over events: the field phases walk a
// table of (event, tile) entries, the push a table of (event, particle block)
// entries.  Kernels are persistent: a grid sized to the chip walks its table
// with a stride, and the table is split into eight contiguous chunks, one per
// XCD (workgroup b runs on XCD b mod 8), so that neighbouring tiles of one
// lattice share an XCD's L2.  The step index lives in device memory (the
// batch control block), so one captured hipGraph of the step loop can be
// replayed without changing kernel arguments.
#include "batch_internal.hpp"
#include "fields_dev.hpp"
#include "push_dev.hpp"

namespace gl {

// First entry, stride and end of workgroup b's walk: the table is cut into
// nx = 8 contiguous chunks; chunk x is shared by the workgroups b = x mod 8
// (there are per = ceil((g - x) / 8) of them, j = b / 8 numbers them), so
// every entry is visited by exactly one workgroup for any grid size g.
__device__ __forceinline__ int64_t xcd_first(int64_t total, int64_t &stride, int64_t &end) {
    const int64_t g = gridDim.x, b = blockIdx.x;
    const int64_t nx = g >= 8 ? 8 : 1;
    const int64_t x = b % nx, j = b / nx, per = (g - x + nx - 1) / nx;
    const int64_t chunk = (total + nx - 1) / nx;
    const int64_t lo = x * chunk;
    end = lo + chunk < total ? lo + chunk : total;
    stride = per;
    return lo + j;
}

// one tile of an event: stage its links and phi, then the step of its sites
template <typename T, int TX, int TY, bool WT = true>
__device__ __forceinline__ void batch_field_tile(LinkTile<T, TX, TY> &tile, const BatchEv<T> &e, int2 w,
                                                 const BatchAt &at, int tid, int64_t n, T tau, T dtau, T tau_h) {
    const int lx = (tid % (2 * TX)) >> 1, ly = tid / (2 * TX);
    const int tx = (e.N + TX - 1) / TX;
    const int x0 = (w.y % tx) * TX, y0 = (w.y / tx) * TY;
    stage_tile(tile, e.N, e.f[at.in], x0, y0, tid, 2 * TX * TY);
    __syncthreads();
    // every thread takes part (the step synchronises the workgroup)
    const bool active = x0 + lx < e.N && y0 + ly < e.N;
    const int reunit = e.reunit_every > 0 && (n % e.reunit_every) == e.reunit_every - 1;
    // a large batch's working set overflows the last-level cache in either
    // precision: its streamed arrays take the non-temporal hint (a paired batch's
    // does not, and takes the hint all the same)
    field_step_link<T, TX, TY, true, WT>(tile, e.N, e.f[at.in], e.f[at.out], e.n_species > 0 ? e.F[at.F] : nullptr, x0,
                                         y0, lx, ly, tid & 1, tid, active, tau, dtau, tau_h, reunit);
}

template <typename T, int TX, int TY, bool WT>
__global__ void __launch_bounds__(2 * TX *TY)
k_batch_field(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ tiles, int64_t total, BatchAt at,
              const BatchCtl *__restrict__ ctl, T dtau) {
    __shared__ LinkTile<T, TX, TY> tile;
    const int tid = threadIdx.x + 2 * TX * threadIdx.y;
    const int64_t n = ctl->n + at.off;
    const T tau = dtau * (T)n, tau_h = dtau * ((T)n + T(0.5));
    int64_t stride, end;
    for (int64_t t = xcd_first(total, stride, end); t < end; t += stride) {
        const int2 w = tiles[t];
        if (*evs[w.x].fail != kNotFailed) continue;   // a failed event is masked (uniform per workgroup)
        __syncthreads();   // the previous tile's reads are done
        batch_field_tile<T, TX, TY, WT>(tile, evs[w.x], w, at, tid, n, tau, dtau, tau_h);
    }
}

// One workgroup per table entry (grid = entries), numbered so that each XCD
// takes one contiguous run of the table: the walk of the persistent kernel
// without its loop, which holds registers the step can use.
template <typename T, int TX, int TY, bool WT>
__global__ void __launch_bounds__(2 * TX *TY) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4, 8)))
k_batch_field_flat(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ tiles, int64_t total, BatchAt at,
                   const BatchCtl *__restrict__ ctl, T dtau) {
    __shared__ LinkTile<T, TX, TY> tile;
    const int tid = threadIdx.x + 2 * TX * threadIdx.y;
    const int64_t n = ctl->n + at.off;
    const T tau = dtau * (T)n, tau_h = dtau * ((T)n + T(0.5));
    const int2 w = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    if (*evs[w.x].fail != kNotFailed) return;   // a failed event is masked (uniform per workgroup)
    batch_field_tile<T, TX, TY, WT>(tile, evs[w.x], w, at, tid, n, tau, dtau, tau_h);
}

// one block of an event's particles; with PERM, position i takes the particle
// in slot perm[i] of buffer parity ppar (the pending sort) and the pushed
// particle goes, with its species, momenta at formation and id, to slot i of
// parity ppar ^ 1, as the single-event push that applies a sort does
template <typename T, bool PERM>
__device__ __forceinline__ void batch_push_block(SpeciesReduce &red, const BatchEv<T> &e, int2 w, const BatchAt &at,
                                                 int ppar, int n, T dtau) {
    const int64_t i = (int64_t)w.y * kPushBlock + threadIdx.x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int s = -1;
    if (i < e.n_slots) {
        if constexpr (PERM) {
            const PartPtrs<T> &P = e.P[ppar], &W = e.P[ppar ^ 1];
            const int64_t src = e.sort.vals[1][i];
            // the arrays that only move go first, so that nothing of them
            // stays live through the push
            W.species[i] = P.species[src];
            W.px0[i] = P.px0[src];
            W.py0[i] = P.py0[src];
            W.pz0[i] = P.pz0[src];
            e.ids[ppar ^ 1][i] = e.ids[ppar][src];
            __builtin_amdgcn_sched_barrier(0);
            s = push_particle<T, true, true>(e.N, P, src, W, i, e.f[at.in], e.F[at.F], e.tab, n, dtau, acc);
        } else {
            s = push_particle<T, false, true>(e.N, e.P[ppar], i, e.P[ppar], i, e.f[at.in], e.F[at.F], e.tab, n, dtau,
                                              acc);
        }
    }
    block_species_reduce(red, s, acc, e.n_species, e.partials + (size_t)w.y * e.n_species * 4);
}

// a masked (failed) event is not pushed, but a pending sort still moves its
// particles, so that its buffers follow the batch's parity
template <typename T, bool PERM>
__device__ __forceinline__ void batch_masked_block(const BatchEv<T> &e, int2 w, int ppar) {
    if constexpr (PERM) {
        const int64_t j = (int64_t)w.y * kPushBlock + threadIdx.x;
        if (j < e.n_slots) permute_one(e.P[ppar], e.P[ppar ^ 1], e.sort.vals[1], j, e.ids[ppar], e.ids[ppar ^ 1]);
    }
}

template <typename T, bool PERM>
__global__ void __launch_bounds__(kPushBlock)
k_batch_push(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ blocks, int64_t total, BatchAt at,
             int ppar, const BatchCtl *__restrict__ ctl, T dtau) {
    __shared__ SpeciesReduce red;
    const int n = (int)(ctl->n + at.off);
    int64_t stride, end;
    for (int64_t t = xcd_first(total, stride, end); t < end; t += stride) {
        const int2 w = blocks[t];
        if (*evs[w.x].fail != kNotFailed) {
            batch_masked_block<T, PERM>(evs[w.x], w, ppar);
            continue;
        }
        batch_push_block<T, PERM>(red, evs[w.x], w, at, ppar, n, dtau);
    }
}

template <typename T, bool PERM>
__global__ void __launch_bounds__(kPushBlock)
k_batch_push_flat(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ blocks, int64_t total, BatchAt at,
                  int ppar, const BatchCtl *__restrict__ ctl, T dtau) {
    __shared__ SpeciesReduce red;
    const int2 w = blocks[xcd_remap(blockIdx.x, gridDim.x)];
    if (*evs[w.x].fail != kNotFailed) {
        batch_masked_block<T, PERM>(evs[w.x], w, ppar);
        return;
    }
    batch_push_block<T, PERM>(red, evs[w.x], w, at, ppar, (int)(ctl->n + at.off), dtau);
}

// The field step of one time and the push of the time before it, which with a
// third field state and a second record do not wait for each other: for batches
// that fill the chip no more than a round or two (the rule of one event,
// pairs in event.hip), where each launch is bound by its own chain of
// dependent instructions.  Rows of FP32 runs, ms: 4 of 64^2 with 1000 particles
// 14.2 -> 9.4, 5 of 128^2 with 3000 20.0 -> 14.7, 10 of 128^2 with 10^4 28.3 ->
// 24.0, 2 of 256^2 with 10^4 12.1 -> 10.9.  Larger batches gain nothing: the
// field step then fills all waves of a SIMD and is near its issue rate, and a
// push workgroup beside it only holds the registers of another (24 of 256^2 296
// -> 288 us a step, ten of 128^2 to 512^2 424 -> 447).
template <typename T, int TX, int TY, bool PERM>
__global__ void __launch_bounds__(kPushBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4, 8)))
k_batch_field_push(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ tiles, int64_t n_tiles,
                   const int2 *__restrict__ blocks, int64_t n_blocks, BatchAt at, BatchAt push, int ppar,
                   const BatchCtl *__restrict__ ctl, T dtau) {
    static_assert(2 * TX * TY == kPushBlock, "a field tile and a push block share the workgroup size");
    union Lds {
        LinkTile<T, TX, TY> tile;
        SpeciesReduce red;
    };
    __shared__ __align__(16) unsigned char lds[sizeof(Lds)];
    // XCD x owns one run of the tiles and one of the push blocks; its
    // workgroups j take them in turn, the push blocks spread evenly
    const int64_t x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int64_t tq = n_tiles >> 3, tr = n_tiles & 7, pq = n_blocks >> 3, pr = n_blocks & 7;
    const int64_t mine_t = tq + (x < tr), mine_p = pq + (x < pr), all = mine_t + mine_p;
    if (j >= all) return;
    const int64_t p = j * mine_p / all;
    if ((j + 1) * mine_p / all > p) {
        const int2 w = blocks[x * pq + (x < pr ? x : pr) + p];
        if (*evs[w.x].fail != kNotFailed) {
            batch_masked_block<T, PERM>(evs[w.x], w, ppar);
            return;
        }
        batch_push_block<T, PERM>(*reinterpret_cast<SpeciesReduce *>(lds), evs[w.x], w, push, ppar,
                                  (int)(ctl->n + push.off), dtau);
        return;
    }
    const int2 w = tiles[x * tq + (x < tr ? x : tr) + (j - p)];
    if (*evs[w.x].fail != kNotFailed) return;
    const int64_t n = ctl->n + at.off;
    batch_field_tile(*reinterpret_cast<LinkTile<T, TX, TY> *>(lds), evs[w.x], w, at, (int)threadIdx.x, n, dtau * (T)n,
                     dtau, dtau * ((T)n + T(0.5)));
}

// one workgroup per (event, species): fixed-order sum of the event's partial
// rows into its series row n - 1, n taken from the control block
template <typename T>
__global__ void __launch_bounds__(256)
k_batch_reduce(const BatchEv<T> *__restrict__ evs, int off, const BatchCtl *__restrict__ ctl) {
    const BatchEv<T> &e = evs[blockIdx.x];
    const int s = blockIdx.y;
    if (s >= e.n_species) return;
    const int64_t n = ctl->n + off, row = n - 1;
    if (row < 0 || row >= e.max_steps) return;
    // masked since an earlier step: that push skipped the event, its partial
    // rows are stale.  Blocks of this launch lower fail to n + 1 at most, so
    // the test reads the same for every thread of the workgroup.
    if (*e.fail <= n) return;
    const int nb = (int)(e.n_slots / kPushBlock);
    __shared__ double red[256][4];
    double acc[4] = {0, 0, 0, 0};
    for (int b = threadIdx.x; b < nb; b += 256)
#pragma unroll
        for (int k = 0; k < 4; k++) acc[k] += e.partials[((size_t)b * e.n_species + s) * 4 + k];
#pragma unroll
    for (int k = 0; k < 4; k++) red[threadIdx.x][k] = acc[k];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w)
#pragma unroll
            for (int k = 0; k < 4; k++) red[threadIdx.x][k] += red[threadIdx.x + w][k];
        __syncthreads();
    }
    if (threadIdx.x < 4) {
        double v = red[0][threadIdx.x];
        if (threadIdx.x < 3 && red[0][3] > 0.0) v -= e.p0sum[s * 4 + threadIdx.x];
        e.series[((size_t)row * kMaxSpecies + s) * 4 + threadIdx.x] = v;
        // a non-finite sum fails the event at the step this push reached (n + 1)
        if (!isfinite(v)) atomicMin(e.fail, (int32_t)(n + 1 < kNotFailed ? n + 1 : kNotFailed - 1));
    }
}

// the batch's finite-value check: entry (event, chunk) tests values
// [chunk * kCheckChunk, ...) of the event's whole field state at parity fpar.
//
// Bound: by latency on small lattices, whose states are a chunk or two: the field
// step writes through L2, so every load comes from beyond it.  Hence 16 bytes a
// lane and kCheckAhead loads in flight (a value a lane and one load in flight took
// 77 us for eight events of 32^2, and 28 with their states in L2; now 8.6).
constexpr int kCheckAhead = 8;
template <typename T>
__global__ void __launch_bounds__(256)
k_batch_check(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ entries, int fpar,
              const BatchCtl *__restrict__ ctl) {
    const int2 w = entries[blockIdx.x];
    const BatchEv<T> &e = evs[w.x];
    const int64_t nvals = (int64_t)kStateVals * e.N * e.N;
    const int64_t lo = (int64_t)w.y * kCheckChunk, hi = lo + kCheckChunk < nvals ? lo + kCheckChunk : nvals;
    const T *a = e.f[fpar].U;   // the state's arrays lie contiguous from U on
    struct __align__(16) V { T v[16 / sizeof(T)]; };
    constexpr int NV = 16 / (int)sizeof(T);
    static_assert(kStateVals % NV == 0 && kCheckChunk % NV == 0, "whole vectors");
    const V *p = reinterpret_cast<const V *>(a + lo);
    const int64_t nv = (hi - lo) / NV;
    bool bad = false;
    for (int64_t i0 = threadIdx.x; i0 < nv; i0 += 256 * kCheckAhead) {
        V x[kCheckAhead];
#pragma unroll
        for (int u = 0; u < kCheckAhead; u++) x[u] = p[i0 + 256 * u < nv ? i0 + 256 * u : nv - 1];
#pragma unroll
        for (int u = 0; u < kCheckAhead; u++)
#pragma unroll
            for (int k = 0; k < NV; k++) bad |= !isfinite(x[u].v[k]);
    }
    if (bad) atomicMin(e.fail, (int32_t)(ctl->n < kNotFailed ? ctl->n : kNotFailed - 1));
}

__global__ void k_batch_advance(BatchCtl *ctl, int steps) {
    if (threadIdx.x == 0 && blockIdx.x == 0) ctl->n = ctl->n + steps;
}

template <typename T>
hipError_t launch_batch_fields(hipStream_t st, int shape, const BatchEv<T> *evs, const int2 *tiles, int64_t total,
                               const BatchAt &at, const BatchCtl *ctl, double dtau, int grid, bool whole_rows) {
    if (total <= 0) return hipSuccess;
    unsigned g = (unsigned)(grid > 0 && grid < total ? grid : total);
    // Written through the L2 caches where every lattice's rows fill whole 64-byte
    // sectors (whole_rows: N a multiple of four), else left there for the tiles that
    // share a sector to be joined, as in one event's step; 64 steps, left and
    // written through: FP64 8 of 162^2 5.90 and 6.13 ms, 6 of 243^2 12.75 and 13.50, 2 of
    // 486^2 11.85 and 12.73, and on the persistent walk 14.14 and 15.93, FP32 there 6.98 and
    // 7.23.  The FP32 step without the walk is at most 1 % longer written through,
    // and shorter in small batches (20 of 81^2 2.70 and 2.66).
#define GL_FIELD(K, TXv, TYv, WT)                                                                             \
    hipLaunchKernelGGL((K<T, TXv, TYv, WT>), dim3(g), dim3(2 * TXv, TYv), 0, st, evs, tiles, total, at, ctl,  \
                       (T)dtau)
#define GL_SHAPE(TXv, TYv)                                                                                    \
    {                                                                                                         \
        if (g == total) {                                                                                     \
            if (sizeof(T) == 4 || whole_rows) GL_FIELD(k_batch_field_flat, TXv, TYv, true);                   \
            else GL_FIELD(k_batch_field_flat, TXv, TYv, sizeof(T) == 4);                                      \
        } else {                                                                                              \
            if (whole_rows) GL_FIELD(k_batch_field, TXv, TYv, true);                                          \
            else GL_FIELD(k_batch_field, TXv, TYv, false);                                                    \
        }                                                                                                     \
    }
    switch (shape) {
        case 0: GL_SHAPE(32, 4) break;
        case 1: GL_SHAPE(64, 2) break;
        case 2: GL_SHAPE(16, 8) break;
        default: return hipErrorInvalidValue;
    }
#undef GL_SHAPE
#undef GL_FIELD
    return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_push(hipStream_t st, const BatchEv<T> *evs, const int2 *blocks, int64_t total,
                             const BatchAt &at, int ppar, const BatchCtl *ctl, double dtau, int grid, bool permuted) {
    if (total > 0) {
        unsigned g = (unsigned)(grid > 0 && grid < total ? grid : total);
#define GL_PUSH(PERM)                                                                                          \
    {                                                                                                          \
        if (g == total)                                                                                        \
            hipLaunchKernelGGL((k_batch_push_flat<T, PERM>), dim3(g), dim3(kPushBlock), 0, st, evs, blocks, total, \
                               at, ppar, ctl, (T)dtau);                                                        \
        else                                                                                                   \
            hipLaunchKernelGGL((k_batch_push<T, PERM>), dim3(g), dim3(kPushBlock), 0, st, evs, blocks, total,   \
                               at, ppar, ctl, (T)dtau);                                                        \
    }
        if (permuted)
            GL_PUSH(true)
        else
            GL_PUSH(false)
#undef GL_PUSH
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_pair(hipStream_t st, int shape, const BatchEv<T> *evs, const int2 *tiles, int64_t n_tiles,
                             const BatchAt &at, const int2 *blocks, int64_t n_blocks, const BatchAt &push, int ppar,
                             const BatchCtl *ctl, double dtau, bool permuted) {
    if (n_tiles <= 0 || n_blocks <= 0) return hipErrorInvalidValue;
    // as many workgroups an XCD as the fullest one has work for
    const unsigned g = (unsigned)(8 * ((n_tiles + 7) / 8 + (n_blocks + 7) / 8));
#define GL_SHAPE(TXv, TYv)                                                                                     \
    {                                                                                                          \
        if (permuted)                                                                                          \
            hipLaunchKernelGGL((k_batch_field_push<T, TXv, TYv, true>), dim3(g), dim3(kPushBlock), 0, st, evs, \
                               tiles, n_tiles, blocks, n_blocks, at, push, ppar, ctl, (T)dtau);                \
        else                                                                                                   \
            hipLaunchKernelGGL((k_batch_field_push<T, TXv, TYv, false>), dim3(g), dim3(kPushBlock), 0, st, evs, \
                               tiles, n_tiles, blocks, n_blocks, at, push, ppar, ctl, (T)dtau);                \
    }
    switch (shape) {
        case 0: GL_SHAPE(32, 4) break;
        case 1: GL_SHAPE(64, 2) break;
        case 2: GL_SHAPE(16, 8) break;
        default: return hipErrorInvalidValue;
    }
#undef GL_SHAPE
    return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_reduce(hipStream_t st, const BatchEv<T> *evs, int n_events, int off, const BatchCtl *ctl) {
    hipLaunchKernelGGL(k_batch_reduce<T>, dim3(n_events, kMaxSpecies), dim3(256), 0, st, evs, off, ctl);
    return hipGetLastError();
}

hipError_t launch_batch_advance(hipStream_t st, BatchCtl *ctl, int steps) {
    hipLaunchKernelGGL(k_batch_advance, dim3(1), dim3(64), 0, st, ctl, steps);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_check(hipStream_t st, const BatchEv<T> *evs, const int2 *entries, int64_t total, int fpar,
                              const BatchCtl *ctl) {
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_check<T>, dim3((unsigned)total), dim3(256), 0, st, evs, entries, fpar, ctl);
    return hipGetLastError();
}

#define GL_INST(T)                                                                                          \
    template hipError_t launch_batch_check<T>(hipStream_t, const BatchEv<T> *, const int2 *, int64_t, int,      \
                                              const BatchCtl *);                                             \
    template hipError_t launch_batch_fields<T>(hipStream_t, int, const BatchEv<T> *, const int2 *, int64_t,      \
                                               const BatchAt &, const BatchCtl *, double, int, bool);        \
    template hipError_t launch_batch_push<T>(hipStream_t, const BatchEv<T> *, const int2 *, int64_t,            \
                                             const BatchAt &, int, const BatchCtl *, double, int, bool);     \
    template hipError_t launch_batch_pair<T>(hipStream_t, int, const BatchEv<T> *, const int2 *, int64_t,       \
                                             const BatchAt &, const int2 *, int64_t, const BatchAt &, int,   \
                                             const BatchCtl *, double, bool);                                \
    template hipError_t launch_batch_reduce<T>(hipStream_t, const BatchEv<T> *, int, int, const BatchCtl *);
GL_INST(double)
GL_INST(float)
#undef GL_INST

}  // namespace gl
