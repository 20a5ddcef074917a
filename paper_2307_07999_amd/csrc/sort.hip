// sort.hip -- keeps the particle arrays ordered by cell so that the particles
// of one workgroup gather site fields of neighbouring cells (a few cache
// lines per plane per wave, L2 reuse).  Stable LSD radix sort of the valid
// slots [0, n) on their cell index (the padding slots behind them stay), in as few
// digits of at most 9 bits as the lattice's cells take (512^2: two of 9 bits),
// deterministic: counts per (digit, workgroup), a per-digit scan over
// workgroups, and a stable scatter whose ranks come from wave64 ballots.
// Particle sets of at most kSortSmall are sorted in one workgroup.
//
// Bound by the launches: a pass moves a few MB, and each of its three kernels
// takes 4-6 us of mostly fixed latency.  Hence two wide digits instead of
// three of 8 bits, the first pass taking its keys from the cells themselves,
// and a scatter that ranks a wave's keys without workgroup barriers.  512^2,
// 7e5 particles: 70 -> 52 us per sort; 1000 particles 34 -> 9.
#include "batch_internal.hpp"
#include "su3.hpp"

namespace gl {

constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortItems = 4;                              // keys per thread
constexpr int kSortTile = kSortThreads * kSortItems;       // keys per workgroup
constexpr int kSmallWaves = 16;
constexpr int kSortSmall = kSmallWaves * 64 * kSortItems;  // keys of the one-workgroup sort

int64_t sort_tiles(int64_t n) { return (n + kSortTile - 1) / kSortTile; }

// digits of the cells of an N x N lattice
__host__ __device__ inline int sort_bits(int N) {
    int b = 1;
    while (((int64_t)1 << b) < (int64_t)N * N) b++;
    return b;
}
int sort_passes(int N) { return (sort_bits(N) + kDigitBits - 1) / kDigitBits; }

// pass `pass` of `passes` on the cells of an N x N lattice: the digit, and the
// key and value buffers read and written (the last pass leaves the order in
// vals[1]; the first reads the cells)
struct SortPass {
    int shift, bits, in, out;
    bool first, last;
};
__host__ __device__ inline SortPass sort_pass(int N, int pass, int passes) {
    SortPass p;
    p.bits = (sort_bits(N) + passes - 1) / passes;
    p.shift = pass * p.bits;
    p.out = (passes - 1 - pass) & 1 ? 0 : 1;
    p.in = p.out ^ 1;
    p.first = pass == 0;
    p.last = pass == passes - 1;
    return p;
}

// ---- the phases, for one tile (workgroup) of one sort ---------------------

// cells and sort buffers of one particle set
struct SortView {
    const int32_t *cx, *cy;
    int N;
    int64_t n, n_slots, tiles;   // valid slots, all slots, sort tiles over n
    SortScratch s;
};

// selected, not indexed: an index would put the pointers in scratch memory
__device__ __forceinline__ uint32_t *key_buf(const SortView &v, int b) { return b ? v.s.keys[1] : v.s.keys[0]; }
__device__ __forceinline__ int32_t *val_buf(const SortView &v, int b) { return b ? v.s.vals[1] : v.s.vals[0]; }

__device__ __forceinline__ uint32_t sort_key(const SortView &v, const SortPass &p, int64_t i) {
    return p.first ? (uint32_t)(v.cx[i] + v.N * v.cy[i]) : key_buf(v, p.in)[i];
}

// per-digit counts of tile `tile`, stored digit-major: counts[d * tiles + tile]
__device__ __forceinline__ void radix_count_tile(const SortView &v, const SortPass &p, int64_t tile) {
    __shared__ uint32_t h[kDigits];
    for (int d = threadIdx.x; d < kDigits; d += kSortThreads) h[d] = 0;
    __syncthreads();
    const uint32_t mask = (1u << p.bits) - 1;
#pragma unroll
    for (int k = 0; k < kSortItems; k++) {
        const int64_t i = tile * kSortTile + k * kSortThreads + threadIdx.x;
        if (i < v.n) atomicAdd(&h[(sort_key(v, p, i) >> p.shift) & mask], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < 1 << p.bits; d += kSortThreads) v.s.counts[(size_t)d * v.tiles + tile] = h[d];
}

// exclusive scan of one digit's row of per-tile counts in place (256
// threads), and the digit's total
__device__ __forceinline__ void scan_row(uint32_t *__restrict__ row, int64_t tiles, uint32_t *__restrict__ total) {
    __shared__ uint32_t wsum[4];
    const int t = threadIdx.x, lane = t & 63;
    int64_t chunk = (tiles + 255) / 256;
    int64_t lo = t * chunk, hi = lo + chunk < tiles ? lo + chunk : tiles;
    uint32_t s = 0;
    for (int64_t i = lo; i < hi; i++) s += row[i];
    uint32_t inc = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(inc, off, 64);
        if (lane >= off) inc += u;
    }
    if (lane == 63) wsum[t >> 6] = inc;
    __syncthreads();
    uint32_t run = inc - s;
    for (int w = 0; w < t >> 6; w++) run += wsum[w];
    if (t == 255) *total = run + s;
    for (int64_t i = lo; i < hi; i++) {
        uint32_t u = row[i];
        row[i] = run;
        run += u;
    }
}

// Ranks of a wave's keys (kSortItems rounds of 64 consecutive ones) among
// those of the wave with the same digit, in order; count[digit] then holds the
// wave's number of each.  No barrier: a wave's LDS accesses keep their order.
__device__ __forceinline__ void rank_wave(const uint32_t (&digit)[kSortItems], const bool (&valid)[kSortItems], int bits,
                                          volatile uint32_t *count, uint32_t (&rank)[kSortItems]) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        // lanes of this wave holding the same digit
        uint64_t peers = __ballot(valid[r]);
        for (int b = 0; b < bits; b++) {
            const uint64_t m = __ballot(valid[r] && ((digit[r] >> b) & 1u));
            peers &= ((digit[r] >> b) & 1u) ? m : ~m;
        }
        const uint32_t before = valid[r] ? count[digit[r]] : 0u, in_round = (uint32_t)__popcll(peers & below);
        rank[r] = before + in_round;
        __builtin_amdgcn_wave_barrier();
        if (valid[r] && in_round == 0) count[digit[r]] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
}

// exclusive scan over kDigits of LDS values total[] in place, by the first
// kDigits / 2 threads (two digits each)
__device__ __forceinline__ void scan_digits(uint32_t *total, uint32_t *wsum) {
    const int t = threadIdx.x, lane = t & 63;
    uint32_t a = 0, b = 0, inc = 0;
    if (t < kDigits / 2) {
        a = total[2 * t];
        b = total[2 * t + 1];
        inc = a + b;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t u = __shfl_up(inc, off, 64);
            if (lane >= off) inc += u;
        }
        if (lane == 63) wsum[t >> 6] = inc;
    }
    __syncthreads();
    if (t < kDigits / 2) {
        uint32_t run = inc - a - b;
        for (int w = 0; w < t >> 6; w++) run += wsum[w];
        total[2 * t] = run;
        total[2 * t + 1] = run + a;
    }
    __syncthreads();
}

// stable scatter of tile `tile` by the digit of pass p
__device__ __forceinline__ void radix_scatter_tile(const SortView &v, const SortPass &p, int64_t tile) {
    __shared__ uint32_t wcount[kSortWaves][kDigits];
    __shared__ uint32_t base[kDigits], wsum[kSortWaves];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, nd = 1 << p.bits;
    for (int d = t; d < kDigits; d += kSortThreads) {
        base[d] = d < nd ? v.s.totals[d] : 0u;
#pragma unroll
        for (int w = 0; w < kSortWaves; w++) wcount[w][d] = 0;
    }
    uint32_t key[kSortItems], digit[kSortItems], rank[kSortItems];
    bool valid[kSortItems];
    const int64_t i0 = tile * kSortTile + (int64_t)wave * (64 * kSortItems) + lane;
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        valid[r] = i0 + 64 * r < v.n;
        key[r] = valid[r] ? sort_key(v, p, i0 + 64 * r) : 0u;
        digit[r] = (key[r] >> p.shift) & (uint32_t)(nd - 1);
    }
    __syncthreads();
    scan_digits(base, wsum);   // each digit's first position
    rank_wave(digit, valid, p.bits, wcount[wave], rank);
    __syncthreads();
    for (int d = t; d < nd; d += kSortThreads) {
        uint32_t run = base[d] + v.s.counts[(size_t)d * v.tiles + tile];
#pragma unroll
        for (int w = 0; w < kSortWaves; w++) {
            const uint32_t c = wcount[w][d];
            wcount[w][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; r++)
        if (valid[r]) {
            const uint32_t pos = wcount[wave][digit[r]] + rank[r];
            if (!p.last) key_buf(v, p.out)[pos] = key[r];
            val_buf(v, p.out)[pos] = p.first ? (int32_t)(i0 + 64 * r) : val_buf(v, p.in)[i0 + 64 * r];
        }
    // the padding keeps its place
    if (p.last && tile == v.tiles - 1)
        for (int64_t i = v.n + t; i < v.n_slots; i += kSortThreads) val_buf(v, p.out)[i] = (int32_t)i;
}

// the whole sort of at most kSortSmall particles in one workgroup: the
// keys stay in LDS between the passes
__device__ __forceinline__ void sort_small(const SortView &v, int passes) {
    __shared__ uint32_t keys[kSortSmall];
    __shared__ int32_t vals[kSortSmall];
    __shared__ uint32_t wcount[kSmallWaves][kDigits];
    __shared__ uint32_t base[kDigits], wsum[kSmallWaves];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, i0 = wave * (64 * kSortItems) + lane;
    uint32_t key[kSortItems], digit[kSortItems], rank[kSortItems];
    int32_t val[kSortItems];
    bool valid[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        val[r] = i0 + 64 * r;
        valid[r] = val[r] < v.n;
        key[r] = valid[r] ? (uint32_t)(v.cx[val[r]] + v.N * v.cy[val[r]]) : 0u;
    }
    for (int pass = 0; pass < passes; pass++) {
        const SortPass p = sort_pass(v.N, pass, passes);
        for (int d = lane; d < kDigits; d += 64) wcount[wave][d] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < kSortItems; r++) digit[r] = (key[r] >> p.shift) & ((1u << p.bits) - 1);
        rank_wave(digit, valid, p.bits, wcount[wave], rank);
        __syncthreads();
        if (t < kDigits) {
            uint32_t run = 0;
#pragma unroll
            for (int w = 0; w < kSmallWaves; w++) {
                const uint32_t c = wcount[w][t];
                wcount[w][t] = run;
                run += c;
            }
            base[t] = run;
        }
        __syncthreads();
        scan_digits(base, wsum);
#pragma unroll
        for (int r = 0; r < kSortItems; r++)
            if (valid[r]) {
                const uint32_t pos = base[digit[r]] + wcount[wave][digit[r]] + rank[r];
                keys[pos] = key[r];
                vals[pos] = val[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortItems; r++)
            if (valid[r]) {
                key[r] = keys[i0 + 64 * r];
                val[r] = vals[i0 + 64 * r];
            }
        // the next pass writes keys and vals only after its own barriers
    }
#pragma unroll
    for (int r = 0; r < kSortItems; r++)
        if (valid[r]) v.s.vals[1][i0 + 64 * r] = val[r];
    for (int64_t i = v.n + t; i < v.n_slots; i += 64 * kSmallWaves) v.s.vals[1][i] = (int32_t)i;
}

// ---- single-sort kernels ----------------------------------------------------

__global__ void __launch_bounds__(kSortThreads) k_radix_count(SortView v, SortPass p) {
    radix_count_tile(v, p, blockIdx.x);
}
// per digit d (one workgroup each): exclusive scan of counts[d][0..tiles) in
// place, and the digit's total
__global__ void __launch_bounds__(256) k_scan_rows(SortView v) {
    scan_row(v.s.counts + (size_t)blockIdx.x * v.tiles, v.tiles, v.s.totals + blockIdx.x);
}
__global__ void __launch_bounds__(kSortThreads) k_radix_scatter(SortView v, SortPass p) {
    radix_scatter_tile(v, p, blockIdx.x);
}
__global__ void __launch_bounds__(64 * kSmallWaves) k_sort_small(SortView v, int passes) { sort_small(v, passes); }

template <typename T>
__global__ void __launch_bounds__(256)
k_permute(PartPtrs<T> src, PartPtrs<T> dst, const int32_t *__restrict__ perm, int64_t n,
          int32_t *__restrict__ id_src, int32_t *__restrict__ id_dst) {
    int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < n) permute_one(src, dst, perm, j, id_src, id_dst);
}

// ---- batched kernels: one launch per phase for all events of a batch -------
// Work tables: pblocks (event, block of kPushBlock slots) over each event's
// used slots, stiles (event, sort tile) over its particles; an event's
// particles move from buffer parity ppar to ppar ^ 1.  Every event takes the same
// number of passes (that of the largest lattice), each with its own digits.

template <typename T>
__device__ __forceinline__ SortView batch_view(const BatchEv<T> &e, int ppar) {
    const PartPtrs<T> &P = ppar ? e.P[1] : e.P[0];
    return SortView{P.cx, P.cy, e.N, e.n_particles, e.n_slots, e.sort_tiles, e.sort};
}

template <typename T>
__global__ void __launch_bounds__(kSortThreads)
k_batch_radix_count(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ stiles, int ppar, int pass, int passes) {
    const int2 w = stiles[blockIdx.x];
    const BatchEv<T> &e = evs[w.x];
    radix_count_tile(batch_view(e, ppar), sort_pass(e.N, pass, passes), w.y);
}

// workgroup e * kDigits + d scans digit d of event e
template <typename T>
__global__ void __launch_bounds__(256) k_batch_scan_rows(const BatchEv<T> *__restrict__ evs, int pass, int passes) {
    const BatchEv<T> &e = evs[blockIdx.x / kDigits];
    const int d = blockIdx.x % kDigits;
    if (e.n_slots <= 0 || d >> sort_pass(e.N, pass, passes).bits) return;
    scan_row(e.sort.counts + (size_t)d * e.sort_tiles, e.sort_tiles, e.sort.totals + d);
}

template <typename T>
__global__ void __launch_bounds__(kSortThreads)
k_batch_radix_scatter(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ stiles, int ppar, int pass,
                      int passes) {
    const int2 w = stiles[blockIdx.x];
    const BatchEv<T> &e = evs[w.x];
    radix_scatter_tile(batch_view(e, ppar), sort_pass(e.N, pass, passes), w.y);
}

template <typename T>
__global__ void __launch_bounds__(256)
k_batch_permute(const BatchEv<T> *__restrict__ evs, const int2 *__restrict__ pblocks, int ppar) {
    const int2 w = pblocks[blockIdx.x];
    const BatchEv<T> &e = evs[w.x];
    const int64_t j = (int64_t)w.y * kPushBlock + threadIdx.x;
    if (j < e.n_slots) permute_one(e.P[ppar], e.P[ppar ^ 1], e.sort.vals[1], j, e.ids[ppar], e.ids[ppar ^ 1]);
}

// The sorted order of the slots of src by cell (n valid ones first, n_slots
// in all): perm[j] is the slot that goes to position j (in the sort
// scratch, see sort_perm).
template <typename T>
hipError_t launch_sort_order(hipStream_t st, int N, PartPtrs<T> src, int64_t n, int64_t n_slots, SortScratch s) {
    if (n <= 0) return hipSuccess;
    const SortView v{src.cx, src.cy, N, n, n_slots, sort_tiles(n), s};
    const int passes = sort_passes(N);
    if (n <= kSortSmall) {
        hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(64 * kSmallWaves), 0, st, v, passes);
        return hipGetLastError();
    }
    for (int pass = 0; pass < passes; pass++) {
        const SortPass p = sort_pass(N, pass, passes);
        hipLaunchKernelGGL(k_radix_count, dim3((unsigned)v.tiles), dim3(kSortThreads), 0, st, v, p);
        hipLaunchKernelGGL(k_scan_rows, dim3(1 << p.bits), dim3(256), 0, st, v);
        hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)v.tiles), dim3(kSortThreads), 0, st, v, p);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// the last pass leaves the permutation in the second value buffer
const int32_t *sort_perm(SortScratch s) { return s.vals[1]; }

template <typename T>
hipError_t launch_permute(hipStream_t st, PartPtrs<T> src, PartPtrs<T> dst, const int32_t *perm, int64_t n,
                          int32_t *id_src, int32_t *id_dst) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_permute<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, perm, n, id_src,
                       id_dst);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_sort_particles(hipStream_t st, int N, PartPtrs<T> src, PartPtrs<T> dst, int64_t n, int64_t n_slots,
                                 SortScratch s, int32_t *id_src, int32_t *id_dst) {
    hipError_t e = launch_sort_order<T>(st, N, src, n, n_slots, s);
    if (e != hipSuccess) return e;
    return launch_permute<T>(st, src, dst, sort_perm(s), n_slots, id_src, id_dst);
}

// the sorted order of every event of a batch by cell, of buffer parity ppar:
// `passes` digit passes (count, scan, scatter), one launch each for all
// events, leaving each event's permutation in its sort scratch (vals[1]);
// with permute, then the permutation itself (ppar to ppar ^ 1), else the next
// push applies it (launch_batch_push with permuted)
template <typename T>
hipError_t launch_batch_sort(hipStream_t st, const BatchEv<T> *evs, int n_events, int passes, const int2 *pblocks,
                             int64_t n_pblocks, const int2 *stiles, int64_t n_stiles, int ppar, bool permute) {
    if (n_pblocks <= 0 || n_stiles <= 0) return hipSuccess;
    for (int pass = 0; pass < passes; pass++) {
        hipLaunchKernelGGL(k_batch_radix_count<T>, dim3((unsigned)n_stiles), dim3(kSortThreads), 0, st, evs, stiles,
                           ppar, pass, passes);
        hipLaunchKernelGGL(k_batch_scan_rows<T>, dim3((unsigned)n_events * kDigits), dim3(256), 0, st, evs, pass,
                           passes);
        hipLaunchKernelGGL(k_batch_radix_scatter<T>, dim3((unsigned)n_stiles), dim3(kSortThreads), 0, st, evs,
                           stiles, ppar, pass, passes);
    }
    if (permute) return launch_batch_permute<T>(st, evs, pblocks, n_pblocks, ppar);
    return hipGetLastError();
}

// every event's pending permutation (left by launch_batch_sort) applied alone,
// buffer parity ppar to ppar ^ 1
template <typename T>
hipError_t launch_batch_permute(hipStream_t st, const BatchEv<T> *evs, const int2 *pblocks, int64_t n_pblocks,
                                int ppar) {
    if (n_pblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_permute<T>, dim3((unsigned)n_pblocks), dim3(256), 0, st, evs, pblocks, ppar);
    return hipGetLastError();
}

#define GL_INST(T)                                                                                            \
    template hipError_t launch_sort_particles<T>(hipStream_t, int, PartPtrs<T>, PartPtrs<T>, int64_t, int64_t,       \
                                                 SortScratch, int32_t *, int32_t *);                             \
    template hipError_t launch_sort_order<T>(hipStream_t, int, PartPtrs<T>, int64_t, int64_t, SortScratch);       \
    template hipError_t launch_permute<T>(hipStream_t, PartPtrs<T>, PartPtrs<T>, const int32_t *, int64_t,        \
                                          int32_t *, int32_t *);                                                  \
    template hipError_t launch_batch_sort<T>(hipStream_t, const BatchEv<T> *, int, int, const int2 *, int64_t,    \
                                             const int2 *, int64_t, int, bool);                                   \
    template hipError_t launch_batch_permute<T>(hipStream_t, const BatchEv<T> *, const int2 *, int64_t, int);
GL_INST(double)
GL_INST(float)
#undef GL_INST

}  // namespace gl
