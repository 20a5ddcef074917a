// batch_internal.hpp -- device descriptors of a batch of events stepped in
// lock-step by the flattened multi-event kernels (batch_kernels.hip).
#pragma once
#include "internal.hpp"
#include "su3.hpp"

namespace gl {

template <typename T>
struct BatchEv {
    int N;
    int reunit_every;
    int n_species;
    int max_steps;
    int64_t n_slots, n_particles;   // used slots, the valid ones first
    FieldPtrs<T> f[3];     // the event's two field states, and the spare one of a batch that pairs its launches
    PartPtrs<T> P[2];      // particle buffers; the current one alternates at each sort
    T *F[2];               // site-field records, written by the field phase when n_species > 0; the second as f[2]
    double *partials;      // [n_slots / kPushBlock][n_species][4]
    const double *p0sum;   // [kMaxSpecies][4]: sums of the squared momenta at formation
    double *series;        // [max_steps][kMaxSpecies][4]
    SpeciesTab<T> tab;
    SortScratch sort;      // the event's radix-sort scratch
    int64_t sort_tiles;    // sort tiles over n_particles
    int32_t *ids[2];       // particle ids, alternating with P
    int32_t *fail;         // first step at which the event failed (kNotFailed: none); failed events are skipped
};

constexpr int32_t kNotFailed = 0x7F7F7F7F;   // the value of bytes 0x7F, as hipMemsetAsync writes it
constexpr int64_t kCheckChunk = 65536;       // state values per entry of the batch's finite-value check

struct BatchCtl {
    int64_t n;             // common step index of all events
};

// A step of a launch: its place after the control block's step, the field
// states it reads and writes (a push: the state of its own time in `in`) and
// its site-field record.
struct BatchAt {
    int off, in, out, F;
};

constexpr int kBatchShapes = 3;   // field-kernel site tiles 32x4, 64x2, 16x8 (two lanes per site)

// position j of dst takes every array of slot perm[j] of src
template <typename T>
__device__ __forceinline__ void permute_one(const PartPtrs<T> &src, const PartPtrs<T> &dst,
                                            const int32_t *__restrict__ perm, int64_t j,
                                            const int32_t *__restrict__ id_src, int32_t *__restrict__ id_dst) {
    int64_t i = perm[j];
    dst.cx[j] = src.cx[i];
    dst.cy[j] = src.cy[i];
    dst.species[j] = src.species[i];
#pragma unroll
    for (int k = 0; k < kPartRec<T>; k += 16 / (int)sizeof(T)) {
        T v[16 / sizeof(T)];
        chunk_ld16(src.st, (size_t)src.cap, (size_t)i, k, v);
        chunk_st16(dst.st, (size_t)dst.cap, (size_t)j, k, v);
    }
    dst.px0[j] = src.px0[i];
    dst.py0[j] = src.py0[i];
    dst.pz0[j] = src.pz0[i];
    id_dst[j] = id_src[i];
}

template <typename T>
hipError_t launch_batch_fields(hipStream_t st, int shape, const BatchEv<T> *evs, const int2 *tiles, int64_t total,
                               const BatchAt &at, const BatchCtl *ctl, double dtau, int grid, bool whole_rows);
// the particle sort of every event, one launch per phase; pblocks (event,
// particle block) and stiles (event, sort tile) cover each event's used
// slots.  The sorted order of buffer parity ppar goes to each event's sort
// scratch; with permute the particles then move to parity ppar ^ 1, else the
// next push moves them (launch_batch_push with permuted) or
// launch_batch_permute does.
template <typename T>
hipError_t launch_batch_sort(hipStream_t st, const BatchEv<T> *evs, int n_events, int passes, const int2 *pblocks,
                             int64_t n_pblocks, const int2 *stiles, int64_t n_stiles, int ppar, bool permute);
template <typename T>
hipError_t launch_batch_permute(hipStream_t st, const BatchEv<T> *evs, const int2 *pblocks, int64_t n_pblocks,
                                int ppar);
// the push of every event from buffer parity ppar; with permuted, position j
// takes the particle in slot perm[j] of ppar (the pending sort) and the pushed
// particles go to parity ppar ^ 1 (a masked event's particles are moved
// without a push)
template <typename T>
hipError_t launch_batch_push(hipStream_t st, const BatchEv<T> *evs, const int2 *blocks, int64_t total,
                             const BatchAt &at, int ppar, const BatchCtl *ctl, double dtau, int grid, bool permuted);
// the field step `at` and the push of the step before it in one launch
template <typename T>
hipError_t launch_batch_pair(hipStream_t st, int shape, const BatchEv<T> *evs, const int2 *tiles, int64_t n_tiles,
                             const BatchAt &at, const int2 *blocks, int64_t n_blocks, const BatchAt &push, int ppar,
                             const BatchCtl *ctl, double dtau, bool permuted);
// the series rows of the push at step off
template <typename T>
hipError_t launch_batch_reduce(hipStream_t st, const BatchEv<T> *evs, int n_events, int off, const BatchCtl *ctl);
// the control block moves on by `steps`
hipError_t launch_batch_advance(hipStream_t st, BatchCtl *ctl, int steps);
// every event's field state at parity fpar checked for NaN/Inf in chunks of
// kCheckChunk values ((event, chunk) entries); a failing event's fail slot
// is lowered to the current step
template <typename T>
hipError_t launch_batch_check(hipStream_t st, const BatchEv<T> *evs, const int2 *entries, int64_t total, int fpar,
                              const BatchCtl *ctl);

}  // namespace gl
