// mlp_rows.hpp -- the surrogate network as whole-network kernels: a workgroup
// takes a few tiles of 16 rows through every layer, so that one launch is an
// inference (k_rows_infer) or the forward and backward pass of a training
// step (k_rows_train), which leaves the gradients' operands for k_update.
//
// Layout.  All products run as W x^T: the MFMA's A operand is a 16 x 16 block
// of weights (row o), its B operand 16 rows of activations (column b).  The
// result lane l then holds row b = l % 16 and outputs o = 4 (l / 16) .. + 3 of
// its block, which is exactly the B operand of the next layer's step over
// k = o: an activation goes back to LDS as one 8-byte write and is read as it
// is.  Weights are kept in the same fragment order in global memory (16 bytes
// a lane, two steps over k), so that a wave's load is one contiguous KiB.
//
// Each of the 8 waves owns two blocks of 16 outputs (a hidden layer is padded
// to 256 outputs; narrow networks infer in groups of fewer waves, see
// k_rows_infer), holds their weights of the whole layer in registers (64
// VGPRs, loaded while the previous layer finishes) and reads every row's
// activations from LDS.
//
// The products accumulate in FP32 over k in steps of 16, in ascending order,
// and the scaling, bias, SiLU and BF16 rounding are those of the general
// kernels in mlp.hip: inference is bitwise the same on either path.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t bf16;

// round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16 f2bf(float f) { return __builtin_bit_cast(bf16, (__bf16)f); }

// input column c of a row, scaled to [-1, 1]
__device__ __forceinline__ bf16 scaled_input(float x, const float *__restrict__ sc, int nin, int c) {
    const float lo = sc[c], hi = sc[nin + c];
    return f2bf(2.f * (x - lo) / (hi - lo) - 1.f);
}

constexpr int kRowWidth = 256;                 // padded width of a hidden layer
constexpr int kRowTiles = kRowWidth / 16;      // its blocks of 16 outputs
constexpr int kRowPairs = kRowWidth / 32;      // steps over k, two MFMAs each
constexpr int kRowThreads = 512;
constexpr int kRowMaxDepth = 4;                // hidden layers of the training kernel

// a network that the whole-network kernels take (mlp_fused), with its
// parameters and fragment-ordered weights
struct NetView {
    int n_in, width, depth, n_out;
    int kp_in, ot_out, kp_out;                 // 32-wide k steps of the inputs, 16-blocks and 32-steps of the outputs
    int hb;                                    // 16-blocks of a hidden layer
    int pcol;
    int64_t n_w;                               // weights; the biases follow in P
    const float *P, *sc;
    bf16 *Wf, *Wt;                             // fragments of W (row o, k = input) and of W^T (row i, k = output)
};

constexpr int kFragBlock = 512;                // elements of one (16-block, 32-step) fragment pair

// fragments of layer l (0 .. depth) in Wf, and of layer l (1 .. depth) in Wt
__host__ __device__ inline size_t frag_off(const NetView &v, int l) {
    return l == 0 ? 0 : (size_t)kFragBlock * kRowTiles * (v.kp_in + (size_t)(l - 1) * kRowPairs);
}
__host__ __device__ inline size_t frag_off_t(const NetView &, int l) {
    return (size_t)kFragBlock * kRowTiles * kRowPairs * (size_t)(l - 1);
}
__host__ __device__ inline size_t frag_elems(const NetView &v) {
    return frag_off(v, v.depth) + (size_t)kFragBlock * v.ot_out * kRowPairs;
}
__host__ __device__ inline size_t frag_elems_t(const NetView &v) {
    return frag_off_t(v, v.depth) + (size_t)kFragBlock * kRowTiles * v.kp_out;
}
__host__ __device__ inline int layer_in(const NetView &v, int l) { return l == 0 ? v.n_in : v.width; }
__host__ __device__ inline int layer_out(const NetView &v, int l) { return l == v.depth ? v.n_out : v.width; }
__host__ __device__ inline int layer_pairs(const NetView &v, int l) { return l == 0 ? v.kp_in : kRowPairs; }
__host__ __device__ inline int64_t weight_off(const NetView &v, int l) {
    return l == 0 ? 0 : (int64_t)v.width * v.n_in + (int64_t)(l - 1) * v.width * v.width;
}

// element (row m, step index k) inside the fragments of a matrix of kp steps
__host__ __device__ inline size_t frag_at(int m, int k, int kp) {
    const int lane = m % 16 + 16 * ((k % 16) / 4);
    return (((size_t)(m / 16) * kp + k / 32) * 64 + lane) * 8 + (k / 16 % 2) * 4 + k % 4;
}

// the weight w of layer l, output o, input i, rounded into both orders
__device__ __forceinline__ void put_weight(const NetView &v, int l, int o, int i, float w) {
    const bf16 h = f2bf(w);
    v.Wf[frag_off(v, l) + frag_at(o, i, layer_pairs(v, l))] = h;
    if (l > 0) v.Wt[frag_off_t(v, l) + frag_at(i, o, l == v.depth ? v.kp_out : kRowPairs)] = h;
}

// layer, output and input of weight p
__device__ __forceinline__ void weight_place(const NetView &v, int64_t p, int &l, int &o, int &i) {
    l = 0;
    while (l < v.depth && p >= weight_off(v, l + 1)) l++;
    const int q = (int)(p - weight_off(v, l)), di = layer_in(v, l);
    o = q / di;
    i = q - o * di;
}

// the fragments of the weights in P (their padding stays zero from creation)
__global__ void __launch_bounds__(256) k_put_weights(NetView v) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= v.n_w) return;
    int l, o, i;
    weight_place(v, p, l, o, i);
    put_weight(v, l, o, i, v.P[p]);
}

// the wave of thread t, known to the compiler as uniform and below 8: the tests
// for a hidden layer's blocks then fold away, and with them the waits for loads
// that another path might have left pending
__device__ __forceinline__ int wave_of(int t) {
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    __builtin_assume(w >= 0 && w < kRowThreads / 64);
    return w;
}

// two steps of 16 over k, ascending
__device__ __forceinline__ floatx4 mma_pair(bf16x8 a, bf16x8 b, floatx4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_shufflevector(a, a, 0, 1, 2, 3),
                                                  __builtin_shufflevector(b, b, 0, 1, 2, 3), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_shufflevector(a, a, 4, 5, 6, 7),
                                                     __builtin_shufflevector(b, b, 4, 5, 6, 7), c, 0, 0, 0);
}

// a wave's fragments: blocks 2 wave, 2 wave + 1 of n_blocks, the first KP of kp steps
template <int KP = kRowPairs>
struct WaveWeights {
    bf16x8 w[2][KP];
};
template <int KP>
__device__ __forceinline__ void load_weights(WaveWeights<KP> &r, const bf16 *__restrict__ frags, int wave, int lane,
                                             int n_blocks, int kp) {
#pragma unroll
    for (int t = 0; t < 2; t++) {
        const int ot = 2 * wave + t;
        const bf16x8 *f = (const bf16x8 *)frags + (size_t)ot * kp * 64 + lane;
#pragma unroll
        for (int k = 0; k < KP; k++)
            if (ot < n_blocks && k < kp) r.w[t][k] = f[(size_t)k * 64];
    }
}

// acc[rt][t] = sum over k of the wave's blocks times row tile rt (LDS fragments [rt][kp][lane])
template <int RT, int KP>
__device__ __forceinline__ void layer_product(const WaveWeights<KP> &r, const bf16x8 *act, int act_stride, int wave,
                                              int lane, int n_blocks, int kp, floatx4 (&acc)[RT][2]) {
#pragma unroll
    for (int rt = 0; rt < RT; rt++)
#pragma unroll
        for (int t = 0; t < 2; t++) acc[rt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (2 * wave >= n_blocks) return;
#pragma unroll
    for (int k = 0; k < KP; k++)
        if (k < kp) {
#pragma unroll
            for (int rt = 0; rt < RT; rt++) {
                const bf16x8 b = act[rt * act_stride + k * 64 + lane];
#pragma unroll
                for (int t = 0; t < 2; t++)
                    if (2 * wave + t < n_blocks) acc[rt][t] = mma_pair(r.w[t][k], b, acc[rt][t]);
            }
        }
}

// all biases into LDS, kRowWidth a layer (zero beyond a layer's outputs)
__device__ __forceinline__ void stage_biases(const NetView &v, float *bias) {
    for (int u = threadIdx.x; u < (v.depth + 1) * kRowWidth; u += kRowThreads) {
        const int l = u / kRowWidth, o = u - l * kRowWidth;
        bias[u] = o < layer_out(v, l) ? v.P[v.n_w + (int64_t)l * v.width + o] : 0.f;
    }
}

__device__ __forceinline__ float silu(float v) { return v / (1.f + __expf(-v)); }

// silu of four values.  For |v| <= 80 numerator and denominator (1 to 2^116)
// need no scaling, and the division is one Newton-Raphson step on the hardware's
// reciprocal and two residual corrections of the quotient, which is what a
// division does between its three scaling instructions, and rounds the same
// while the quotient is a normal number (a fifth of the vector time of an
// activation); a wave with a larger value takes the division itself.
__device__ __forceinline__ floatx4 silu4(floatx4 v) {
    floatx4 h;
    const float big = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
    if (__any(!(big <= 80.f))) {
#pragma unroll
        for (int j = 0; j < 4; j++) h[j] = silu(v[j]);
        return h;
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const float d = 1.f + __expf(-v[j]);
        float r = __builtin_amdgcn_rcpf(d);
        r = fmaf(fmaf(-d, r, 1.f), r, r);
        float q = v[j] * r;
        q = fmaf(fmaf(-d, q, v[j]), r, q);
        h[j] = fmaf(fmaf(-d, q, v[j]), r, q);
    }
    return h;
}

// four outputs of a lane as BF16 activations, zero beyond dout (whatever the
// row holds: a non-finite activation must not reach a padded weight)
__device__ __forceinline__ bf16x4 pack_act(floatx4 h, int o0, int dout) {
    bf16x4 r;
#pragma unroll
    for (int j = 0; j < 4; j++) r[j] = o0 + j < dout ? (short)f2bf(h[j]) : (short)0;
    return r;
}

// LDS place of a lane's four outputs of block ot in the next layer's fragments
__device__ __forceinline__ bf16x4 *act_slot(bf16x8 *act, int ot, int lane) {
    return (bf16x4 *)(act + (ot >> 1) * 64 + lane) + (ot & 1);
}

// ---- inference -----------------------------------------------------------------
// 16 RT rows a group of KP waves, all layers, outputs in physical units.  A group
// holds layers (inputs and outputs too) of up to 32 KP, its waves 32 outputs each:
// networks up to 32, 64 and 128 wide run as 8, 4 and 2 groups a workgroup, each with
// rows of its own.
//
// RT = 4, many rows: bound by the SiLU (exponential and IEEE division, about 20
// vector instructions per activation) beside the MFMAs; each weight load
// serves four row tiles, and two workgroups share a compute unit (128 VGPRs),
// one loading or waiting at a barrier while the other computes.
// RT = 1, few rows: bound by latency, a chain of layers that each wait for their
// weights; with the registers of one workgroup a compute unit, the next
// layer's weights are loaded a whole layer ahead (AHEAD).
// 5 -> 256 x 3 -> 2, against six launches per 4096 rows: 10^6 rows 20.5 -> 0.67 ms,
// 410 rows 83 -> 11 us on the device.  Narrow networks, 2^20 rows through 5 -> 8 x 3 -> 2
// and 5 -> 32 x 4 -> 2: 676 and 901 us padded to 256, 83 and 97 in groups (161 and 438
// layer by layer in one pass of all rows).
template <int RT, bool AHEAD, int KP>
__global__ void __launch_bounds__(kRowThreads, AHEAD ? 2 : 4)
k_rows_infer(NetView v, const float *__restrict__ X, int64_t n, float *__restrict__ Y) {
    constexpr int kGroups = kRowPairs / KP, kStride = KP * 64;
    __shared__ bf16x8 act[2][kGroups * RT * kStride];
    extern __shared__ float bias[];            // [depth + 1][kRowWidth]
    const int t = threadIdx.x, group = kGroups > 1 ? (t >> 6) / KP : 0, wave = (t >> 6) - group * KP, lane = t & 63;
    const int64_t r0 = (int64_t)blockIdx.x * (16 * RT * kGroups);
    const int mine = group * RT * kStride;     // the group's part of act
    WaveWeights<KP> w[AHEAD ? 2 : 1];
    auto fetch = [&](WaveWeights<KP> &r, int l) {
        load_weights(r, v.Wf + frag_off(v, l), wave, lane, l == v.depth ? v.ot_out : kRowTiles, layer_pairs(v, l));
    };
    fetch(w[0], 0);
    if constexpr (AHEAD) fetch(w[1], 1);
    stage_biases(v, bias);
    for (int u = t; u < kGroups * RT * v.kp_in * 64; u += kRowThreads) {
        const int ln = u & 63, kp = (u >> 6) % v.kp_in, rt = (u >> 6) / v.kp_in;
        const int64_t row = r0 + 16 * rt + (ln & 15);
        bf16x8 x = {0, 0, 0, 0, 0, 0, 0, 0};
        if (row < n)
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const int c = 32 * kp + 16 * (e >> 2) + 4 * (ln >> 4) + (e & 3);
                if (c < v.n_in) x[e] = (short)scaled_input(X[row * v.n_in + c], v.sc, v.n_in, c);
            }
        act[0][rt * kStride + kp * 64 + ln] = x;
    }
    __syncthreads();
    floatx4 acc[RT][2];
    int cur = 0;
    auto hidden = [&](WaveWeights<KP> &r, int l) {
        layer_product<RT>(r, act[cur] + mine, kStride, wave, lane, kRowTiles, layer_pairs(v, l), acc);
        if (l + (AHEAD ? 2 : 1) <= v.depth) fetch(r, l + (AHEAD ? 2 : 1));
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int o = 16 * (2 * wave + k) + 4 * (lane >> 4);
            const floatx4 b = *(const floatx4 *)(bias + l * kRowWidth + o);
#pragma unroll
            for (int rt = 0; rt < RT; rt++) {
                const floatx4 h = silu4(acc[rt][k] + b);
                *act_slot(act[cur ^ 1] + mine + rt * kStride, 2 * wave + k, lane) = pack_act(h, o, v.width);
            }
        }
        cur ^= 1;
        __syncthreads();
    };
    auto outputs = [&](const WaveWeights<KP> &r) {
        layer_product<RT>(r, act[cur] + mine, kStride, wave, lane, v.ot_out, kRowPairs, acc);
    };
    if constexpr (AHEAD) {
        int l = 0;
        for (; l + 1 < v.depth; l += 2) {
            hidden(w[0], l);
            hidden(w[1], l + 1);
        }
        if (l < v.depth) {
            hidden(w[0], l);
            outputs(w[1]);
        } else {
            outputs(w[0]);
        }
    } else {
        for (int l = 0; l < v.depth; l++) hidden(w[0], l);
        outputs(w[0]);
    }
    // a wave turns its blocks into rows through its share of the other buffer,
    // so that all its lanes work on the few real outputs
    const float *sc_out = v.sc + 2 * v.n_in;
    float *zb = (float *)act[cur ^ 1] + (t >> 6) * (16 * 16 * RT);
    const int64_t g0 = r0 + group * (16 * RT);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int ot = 2 * wave + k;
        if (ot >= v.ot_out) break;
        const floatx4 b = *(const floatx4 *)(bias + v.depth * kRowWidth + 16 * ot + 4 * (lane >> 4));
#pragma unroll
        for (int rt = 0; rt < RT; rt++)
            *(floatx4 *)(zb + (16 * rt + (lane & 15)) * 16 + 4 * (lane >> 4)) = acc[rt][k] + b;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int cols = min(16, v.n_out - 16 * ot);
#pragma unroll 1
        for (int e = lane; e < 16 * RT * cols; e += 64) {
            const int r = e / cols, c = e - r * cols;
            const int64_t row = g0 + r;
            if (row >= n) break;
            float y = zb[r * 16 + c] * sc_out[v.n_out + 16 * ot + c] + sc_out[16 * ot + c];
            if (v.pcol >= 0) y *= powf(X[row * v.n_in + v.pcol], sc_out[2 * v.n_out + 16 * ot + c]);
            Y[row * v.n_out + 16 * ot + c] = y;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- a training step -----------------------------------------------------------
// Two launches: the rows through the network and back (k_rows_train), then the
// gradients from the operands that leaves, straight into Adam and the new
// BF16 weights (k_update).  Every sum runs in the order of the general
// kernels (weight gradients over the rows in steps of 16, biases and loss
// over 256 strided shares and a tree), so training is bitwise the same too.
// A step of 4096 rows of 5 -> 256 x 3 -> 2: 1350 us in 20 launches, 37 us in two.
struct TrainView {
    const float *X, *Y;
    const int32_t *idx;                        // sample of each row, or null: off + row
    int64_t off;
    int B;                                     // rows of this batch
    float scale;                               // 1 / (B n_out)
    int max_tiles;                             // row tiles of 16 the buffers hold
    // operands of the weight gradients, fragments over the rows: per layer
    // [tile][block of 16][lane][4], lane l the column l % 16 of the block
    // and rows 4 (l / 16) .. + 3 of the tile
    bf16 *Hf, *Df;
    // dZ in FP32 per layer, [tile][block of 16][lane][4]: lane l row l % 16 and
    // outputs 4 (l / 16) .. + 3 of the block
    float *Dz;
    float *dev;                                // deviations z - y [B][n_out]
};

constexpr int kGradBlock = 256;                // elements of one 16 x 16 block

__host__ __device__ inline int in_blocks(const NetView &v, int l) { return l == 0 ? (v.n_in + 15) / 16 : v.hb; }
__host__ __device__ inline int out_blocks(const NetView &v, int l) { return l == v.depth ? v.ot_out : v.hb; }
__host__ __device__ inline size_t h_off(const NetView &v, int l, int max_tiles) {
    return l == 0 ? 0 : (size_t)max_tiles * kGradBlock * (in_blocks(v, 0) + (size_t)(l - 1) * v.hb);
}
__host__ __device__ inline size_t d_off(const NetView &v, int l, int max_tiles) {
    return (size_t)max_tiles * kGradBlock * v.hb * (size_t)l;
}

// 16 bytes at byte `at` of an array of the training step's operands (whole offset
// in the vector offset).  They are written through (sc1): left dirty in the L2
// caches, the 26 MB of a step of 4096 rows are written back when the kernel ends,
// behind its work instead of beside it.  Without any of the stores the kernel
// takes 15.1 us, with ordinary ones 21.7, written through 19.7 (the non-temporal hint
// 19.1, but k_update then reads them from memory: 17.3 -> 20.0).
constexpr int kOperandStore = 16;
template <typename V>
__device__ __forceinline__ void store_operand(void *base, uint32_t at, V v) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v),
                                           __builtin_amdgcn_make_buffer_rsrc(base, (short)0, 0x7FFFFFFF, 0x00020000),
                                           at, 0u, kOperandStore);
}

// blocks of one row tile from their LDS fragments (k along the outputs) to
// fragments along the rows
__device__ __forceinline__ void store_rows(const bf16x8 *act, int blocks, bf16 *__restrict__ dst) {
    const bf16 *a = (const bf16 *)act;
    for (int u = threadIdx.x; u < blocks * 32; u += kRowThreads) {
        const int ob = u >> 5;
        bf16x8 x;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int ln = 2 * (u & 31) + (e >> 2), c = ln & 15, b = 4 * (ln >> 4) + (e & 3);
            x[e] = (short)a[((ob >> 1) * 64 + b + 16 * (c >> 2)) * 8 + (ob & 1) * 4 + (c & 3)];
        }
        store_operand(dst, (uint32_t)(ob * kGradBlock + (u & 31) * 8) * 2, x);
    }
}

// One workgroup per tile of 16 rows: gather and scale the rows, forward with
// every layer's pre-activations kept in registers, deviations, and dZ back to
// the first layer.
//
// Bound: by latency, since at a batch of 4096 each compute unit holds one
// tile: a chain of layer products (16 dependent MFMAs each) with a barrier
// between.  Hence the weights of a layer are loaded a whole layer ahead, the
// biases and targets at the start, and 16 rows a workgroup spread such a batch
// over the whole chip.
//
// FULL: hidden layers of all 16 blocks.  Narrower ones compute on the padding
// (their batches are bound by the same chain) but store their own blocks only.
template <int DEPTH, bool FULL>
__global__ void __launch_bounds__(kRowThreads, 2)
k_rows_train(NetView v, TrainView a) {
    __shared__ bf16x8 act[2][kRowPairs * 64];
    __shared__ float bias[(DEPTH + 1) * kRowWidth];
    __shared__ float target[16 * kRowWidth];
    const int t = threadIdx.x, lane = t & 63, wave = wave_of(t);
    const int tile = blockIdx.x, row = 16 * tile + (lane & 15);
    const bool valid = row < a.B;
    if (FULL) v.hb = kRowTiles;                          // known to the compiler
    const int hb = v.hb;
    const int o0 = 32 * wave + 4 * (lane >> 4);          // first output of the lane's two blocks: o0, o0 + 16
    // the chain of products: layers 0 .. DEPTH forward, then DEPTH .. 1 back
    WaveWeights<> w[2];
    auto fetch = [&](int s) {
        if (s <= DEPTH) {
            load_weights(w[s & 1], v.Wf + frag_off(v, s), wave, lane, s == DEPTH ? v.ot_out : kRowTiles,
                         layer_pairs(v, s));
        } else if (s <= 2 * DEPTH) {
            const int l = 2 * DEPTH + 1 - s;
            load_weights(w[s & 1], v.Wt + frag_off_t(v, l), wave, lane, kRowTiles, l == DEPTH ? v.kp_out : kRowPairs);
        }
    };
    fetch(0);
    fetch(1);
    stage_biases(v, bias);
    for (int u = t; u < v.kp_in * 64; u += kRowThreads) {
        const int ln = u & 63, kp = u >> 6, r = 16 * tile + (ln & 15);
        bf16x8 x = {0, 0, 0, 0, 0, 0, 0, 0};
        if (r < a.B) {
            const int64_t s = a.idx ? (int64_t)a.idx[a.off + r] : a.off + r;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const int c = 32 * kp + 16 * (e >> 2) + 4 * (ln >> 4) + (e & 3);
                if (c < v.n_in) x[e] = (short)scaled_input(a.X[s * v.n_in + c], v.sc, v.n_in, c);
            }
        }
        act[0][u] = x;
    }
    // the standardised targets, by the last waves while the first one gathers
    // the inputs
    for (int u = kRowThreads - 1 - t; u < 16 * v.n_out; u += kRowThreads) {
        const int r = u / v.n_out, c = u - r * v.n_out;
        if (16 * tile + r >= a.B) continue;
        const int64_t s = a.idx ? (int64_t)a.idx[a.off + 16 * tile + r] : a.off + 16 * tile + r;
        const float *sc_out = v.sc + 2 * v.n_in;
        float q = a.Y[s * v.n_out + c];
        if (v.pcol >= 0) q /= powf(a.X[s * v.n_in + v.pcol], sc_out[2 * v.n_out + c]);
        target[r * kRowWidth + c] = (q - sc_out[c]) / sc_out[v.n_out + c];
    }
    __syncthreads();
    store_rows(act[0], in_blocks(v, 0), a.Hf + (size_t)tile * in_blocks(v, 0) * kGradBlock);
    floatx4 acc[1][2], z[DEPTH][2];
    int cur = 0;
#pragma unroll
    for (int l = 0; l < DEPTH; l++) {
        layer_product<1>(w[l & 1], act[cur], 0, wave, lane, kRowTiles, layer_pairs(v, l), acc);
        fetch(l + 2);
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const floatx4 b = *(const floatx4 *)(bias + l * kRowWidth + o0 + 16 * k);
            z[l][k] = acc[0][k] + b;
            const floatx4 h = silu4(z[l][k]);
            *act_slot(act[cur ^ 1], 2 * wave + k, lane) = pack_act(h, o0 + 16 * k, valid ? v.width : 0);
        }
        cur ^= 1;
        __syncthreads();
        store_rows(act[cur], hb, a.Hf + h_off(v, l + 1, a.max_tiles) + (size_t)tile * hb * kGradBlock);
    }
    // outputs: deviation from the target and dZ = 2 (z - y) scale
    layer_product<1>(w[DEPTH & 1], act[cur], 0, wave, lane, v.ot_out, kRowPairs, acc);
    fetch(DEPTH + 2);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int ot = 2 * wave + k;
        if (ot >= 2 * v.kp_out) break;
        const floatx4 b = *(const floatx4 *)(bias + DEPTH * kRowWidth + o0 + 16 * k);
        floatx4 g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int c = o0 + 16 * k + j;
            if (valid && c < v.n_out) {
                const float zz = acc[0][k][j] + b[j], d = zz - target[(lane & 15) * kRowWidth + c];
                a.dev[(size_t)row * v.n_out + c] = d;
                g[j] = 2.f * d * a.scale;
            }
        }
        *act_slot(act[cur ^ 1], ot, lane) = pack_act(g, o0 + 16 * k, v.n_out);
        if (ot < v.ot_out)
            store_operand(a.Dz + d_off(v, DEPTH, a.max_tiles) + (size_t)tile * v.ot_out * kGradBlock,
                          (uint32_t)(ot * kGradBlock + 4 * lane) * 4, g);
    }
    cur ^= 1;
    __syncthreads();
    store_rows(act[cur], v.ot_out, a.Df + d_off(v, DEPTH, a.max_tiles) + (size_t)tile * v.ot_out * kGradBlock);
#pragma unroll
    for (int l = DEPTH; l >= 1; l--) {
        const int s = 2 * DEPTH + 1 - l;
        layer_product<1>(w[s & 1], act[cur], 0, wave, lane, kRowTiles, l == DEPTH ? v.kp_out : kRowPairs, acc);
        fetch(s + 2);
#pragma unroll
        for (int k = 0; k < 2; k++) {
            floatx4 g;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float zz = z[l - 1][k][j], sg = 1.f / (1.f + __expf(-zz));
                const float d = acc[0][k][j] * sg * (1.f + zz * (1.f - sg));
                g[j] = valid && o0 + 16 * k + j < v.width ? d : 0.f;
            }
            *act_slot(act[cur ^ 1], 2 * wave + k, lane) = pack_act(g, o0 + 16 * k, v.width);
            if (FULL || 2 * wave + k < hb)
                store_operand(a.Dz + d_off(v, l - 1, a.max_tiles) + (size_t)tile * hb * kGradBlock,
                              (uint32_t)((2 * wave + k) * kGradBlock + 4 * lane) * 4, g);
        }
        cur ^= 1;
        __syncthreads();
        store_rows(act[cur], hb, a.Df + d_off(v, l - 1, a.max_tiles) + (size_t)tile * hb * kGradBlock);
    }
}

struct AdamArgs {
    float lr, b1, b2, c1, c2, eps;
};

__device__ __forceinline__ float adam(float w, float g, float *__restrict__ m, float *__restrict__ v, int64_t i,
                                      const AdamArgs &a) {
    const float mi = a.b1 * m[i] + (1.f - a.b1) * g;
    const float vi = a.b2 * v[i] + (1.f - a.b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    return w - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

// workgroups (of one wave) of k_update: one per 16 x 16 block of a layer's
// weights; then one per four biases; then one for the loss
__host__ __device__ inline int weight_groups(const NetView &v, int l) { return out_blocks(v, l) * in_blocks(v, l); }
__host__ __device__ inline int bias_groups(const NetView &v) { return v.depth * ((v.width + 3) / 4) + (v.n_out + 3) / 4; }

// Gradients of one batch: dW[o][i] = sum over the rows of dZ[o] H[i], one chain
// of MFMAs over the row tiles per 16 x 16 block; db[o] = sum over the rows of
// dZ[o]; the loss.  Then Adam and the new weights in both fragment orders (G
// null), or the gradients to G.
//
// Bound: by the way of the operands (dZ and H of all layers, 12.8 MB at 4096
// rows, and 12.8 MB of FP32 dZ for the biases) from the other XCDs' L2 and by their
// latency; the MFMA chain itself is under 2 us.  So every block is a workgroup of
// one wave, which spreads the loads over all compute units, with kUpdateAhead row
// tiles in flight, and the biases' shares are fetched 16 at a time: a step of 4096
// rows of 5 -> 256 x 3 -> 2 took 22.7 us with four blocks and 16 tiles a workgroup,
// 36 with single shares, 19.1 / 18.2 / 17.3 us with 16 / 24 / 32 tiles.  Blocks are
// numbered so that each XCD takes one contiguous run of them, a layer's rows of
// blocks one after another: its L2 then holds the layer's H once and its own share
// of dZ, instead of all operands passing through every L2.
constexpr int kUpdateAhead = 32;
template <bool FULL>
__global__ void __launch_bounds__(64)
k_update(NetView v, TrainView a, float *__restrict__ P, float *__restrict__ Mo, float *__restrict__ Vo,
         float *__restrict__ G, float *__restrict__ loss, int tiles, AdamArgs aa) {
    if (FULL) v.hb = kRowTiles;
    const int lane = threadIdx.x;
    int l = 0, q = 0, n_groups = 0;
    for (int k = 0; k <= v.depth; k++) n_groups += weight_groups(v, k);
    if ((int)blockIdx.x < n_groups) {
        // contiguous runs per XCD (workgroups go round robin over 8)
        const int per = n_groups / 8, rem = n_groups % 8, x = blockIdx.x % 8, k = blockIdx.x / 8;
        q = x * per + min(x, rem) + k;
        while (q >= weight_groups(v, l)) q -= weight_groups(v, l++);
        const int ni = in_blocks(v, l), no = out_blocks(v, l);
        const int ob = q / ni, ib = q % ni;
        // tile b of the block's operands is `step` bytes after tile b - 1: a
        // scalar base per group of tiles and a scalar offset per tile, since one
        // wave a SIMD issues every address instruction itself
        const uint32_t d_step = no * kGradBlock * sizeof(bf16), h_step = ni * kGradBlock * sizeof(bf16);
        const char *D = (const char *)(a.Df + d_off(v, l, a.max_tiles)) + (size_t)ob * kGradBlock * sizeof(bf16);
        const char *H = (const char *)(a.Hf + h_off(v, l, a.max_tiles)) + (size_t)ib * kGradBlock * sizeof(bf16);
        // the loads of the next kUpdateAhead row tiles fly while these are multiplied
        bf16x4 d[kUpdateAhead], h[kUpdateAhead];
        auto base = [](const char *p) {
            return __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, 0x7FFFFFFF, 0x00020000);
        };
        auto load = [&](int u, int left, __amdgpu_buffer_rsrc_t rd, __amdgpu_buffer_rsrc_t rh) {
            const uint32_t w = min(u, left - 1);   // past the last tile: the last one again, not multiplied
            d[u] = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(rd, 8 * lane, w * d_step, 0));
            h[u] = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(rh, 8 * lane, w * h_step, 0));
        };
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        {
            const auto rd = base(D), rh = base(H);
#pragma unroll
            for (int u = 0; u < kUpdateAhead; u++) load(u, tiles, rd, rh);
        }
        int left = tiles - kUpdateAhead;   // tiles not loaded yet
        for (; left > 0; left -= kUpdateAhead) {
            D += (size_t)kUpdateAhead * d_step;
            H += (size_t)kUpdateAhead * h_step;
            const auto rd = base(D), rh = base(H);
#pragma unroll
            for (int u = 0; u < kUpdateAhead; u++) {
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(d[u], h[u], acc, 0, 0, 0);
                load(u, left, rd, rh);
            }
        }
        left += kUpdateAhead;              // tiles of the last group
#pragma unroll
        for (int u = 0; u < kUpdateAhead; u++)
            if (u < left) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(d[u], h[u], acc, 0, 0, 0);
        const int di = layer_in(v, l), dd = layer_out(v, l), i = 16 * ib + (lane & 15);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int o = 16 * ob + 4 * (lane >> 4) + j;
            if (o >= dd || i >= di) continue;
            const int64_t p = weight_off(v, l) + (int64_t)o * di + i;
            if (G) {
                G[p] = acc[j];
            } else {
                const float w = adam(P[p], acc[j], Mo, Vo, p, aa);
                P[p] = w;
                put_weight(v, l, o, i, w);
            }
        }
        return;
    }
    // the sums of biases and loss: 256 strided shares and a tree over them, four
    // shares a lane
    q = (int)blockIdx.x - n_groups;
    const int per_layer = (v.width + 3) / 4;
    const bool is_loss = q >= bias_groups(v);
    floatx4 s[4];
#pragma unroll
    for (int k = 0; k < 4; k++) s[k] = floatx4{0.f, 0.f, 0.f, 0.f};
    l = min(q / per_layer, v.depth);
    const int o = 4 * (q - l * per_layer), no = out_blocks(v, l);
    if (!is_loss) {
        // share m: rows m, m + 256, ...
        const float *dz = a.Dz + d_off(v, l, a.max_tiles) + (size_t)(o / 16) * kGradBlock +
                          4 * ((lane & 15) + 16 * (o % 16 / 4));
        for (int b0 = 0; b0 < tiles; b0 += 64) {
            floatx4 x[16];
#pragma unroll
            for (int k = 0; k < 16; k++) {
                const int b = min(b0 + 4 * k + (lane >> 4), tiles - 1);
                x[k] = *(const floatx4 *)(dz + (size_t)b * no * kGradBlock);
            }
#pragma unroll
            for (int k = 0; k < 16; k++)
                if (b0 + 4 * k + (lane >> 4) < tiles) s[k & 3] += x[k];
        }
    } else {
        const int count = a.B * v.n_out;
        for (int i0 = 0; i0 < count; i0 += 2048) {
            float x[32];
#pragma unroll
            for (int k = 0; k < 32; k++) x[k] = a.dev[min(i0 + 64 * k + lane, count - 1)];
#pragma unroll
            for (int k = 0; k < 32; k++)
                if (i0 + 64 * k + lane < count) s[k & 3][0] += x[k] * x[k];
        }
    }
    floatx4 r = (s[0] + s[2]) + (s[1] + s[3]);
#pragma unroll
    for (int m = 32; m > 0; m >>= 1)
#pragma unroll
        for (int j = 0; j < 4; j++) r[j] += __shfl_down(r[j], m, 64);
    if (is_loss) {
        if (lane == 0) *loss += r[0] * a.scale;
        return;
    }
#pragma unroll
    for (int j = 0; j < 4; j++)
        if (lane == 0 && o + j < layer_out(v, l)) {
            const int64_t p = v.n_w + (int64_t)l * v.width + o + j;
            if (G) G[p] = r[j];
            else P[p] = adam(P[p], r[j], Mo, Vo, p, aa);
        }
}

}  // namespace
