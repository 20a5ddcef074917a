// pair.hip -- the field step n -> n+1 and the particle push n-1 -> n in one
// launch, for lattices whose step does not fill the chip.
//
// The push of a step reads the fields of its own time (links, phi and site
// fields at tau_{n-1}) and the field step those of tau_n, so neither waits for the
// other once there are three field states and two site-field records.
// On a small lattice each launch is one round of workgroups bound by its own
// chain of dependent instructions (about 9 us each for the FP64 field
// step and push at 32^2), so running them side by side nearly halves a step.
// The workgroups are those of the separate kernels, and the results the same
// bit for bit.  FP64 events to 0.5 fm: 32^2 5.7 -> 3.9 ms, 64^2 5.8 -> 3.7,
// 128^2 5.8 -> 5.0, 256^2 10.3 -> 9.6; FP32 256^2 7.5 -> 6.3.
#include <algorithm>

#include "fields_dev.hpp"
#include "push_dev.hpp"

namespace gl {

constexpr int SX = 32, SY = 4;     // site tile of the field step (fields.hip)
static_assert(2 * SX * SY == kPushBlock, "a field tile and a push block share the workgroup size");

template <typename T, bool PERM>
__global__ void __launch_bounds__(kPushBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4, 8)))
k_field_push(int N, int n_tiles, FieldPtrs<T> in, FieldPtrs<T> out, T *__restrict__ F, T tau, T dtau, T tau_h,
             int reunit, PushCall<T> p) {
    union Lds {
        LinkTile<T, SX, SY> tile;
        SpeciesReduce red;
    };
    __shared__ __align__(16) unsigned char lds[sizeof(Lds)];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < n_tiles) {
        LinkTile<T, SX, SY> &tile = *reinterpret_cast<LinkTile<T, SX, SY> *>(lds);
        const int tx = (N + SX - 1) / SX;
        const int l = (int)xcd_remap(blockIdx.x, n_tiles);
        const int x0 = (l % tx) * SX, y0 = (l / tx) * SY;
        const int lx = (tid % (2 * SX)) >> 1, ly = tid / (2 * SX);
        stage_tile(tile, N, in, x0, y0, tid, 2 * SX * SY);
        __syncthreads();
        const bool active = x0 + lx < N && y0 + ly < N;
        // these lattices fit the last-level cache: nothing is streamed past it
        field_step_link<T, SX, SY, false>(tile, N, in, out, F, x0, y0, lx, ly, tid & 1, tid, active, tau, dtau, tau_h,
                                          reunit);
        return;
    }
    push_block<T, PERM, false>(*reinterpret_cast<SpeciesReduce *>(lds), N,
                               xcd_remap((int)blockIdx.x - n_tiles, (int)gridDim.x - n_tiles), p);
}

template <typename T>
hipError_t launch_field_push(hipStream_t st, int N, FieldPtrs<T> in, FieldPtrs<T> out, T *F, double tau, double dtau,
                             int reunit, const PushCall<T> &p) {
    const int n_tiles = field_tiles(N), blocks = n_tiles + (int)(p.n_slots / kPushBlock);
    if (p.perm)
        hipLaunchKernelGGL((k_field_push<T, true>), dim3(blocks), dim3(kPushBlock), 0, st, N, n_tiles, in, out, F,
                           (T)tau, (T)dtau, (T)(tau + 0.5 * dtau), reunit, p);
    else
        hipLaunchKernelGGL((k_field_push<T, false>), dim3(blocks), dim3(kPushBlock), 0, st, N, n_tiles, in, out, F,
                           (T)tau, (T)dtau, (T)(tau + 0.5 * dtau), reunit, p);
    return hipGetLastError();
}

#define GL_INST(T)                                                                                          \
    template hipError_t launch_field_push<T>(hipStream_t, int, FieldPtrs<T>, FieldPtrs<T>, T *, double, double, int, \
                                             const PushCall<T> &);
GL_INST(double)
GL_INST(float)
#undef GL_INST

}  // namespace gl
