// Learned block refiner: a 4-layer 3D convolutional network on bf16 MFMA.
//
// Every layer is the same operation: a 3^3 convolution from a 10^3 grid (the
// block with a one-voxel halo, or the 8^3 block zero-padded) to the 8^3 block,
// 16 input and 16 output channels (layer 1 uses 2 real input channels, layer 4
// one real output channel; the others hold zeros).  As an implicit GEMM per
// block: M = 16 output channels, N = 512 voxels, K = 27 taps x 16 channels, two
// taps per K step of gfx950's v_mfma_f32_16x16x32_bf16 (layer 1, with its 2 real
// input channels stored as 4, takes 8 taps per K step).
//
// What bounds it is LDS: a K step of 16 voxels is a 1 KB fragment, 8 cycles of the
// CU's 128 bytes a cycle, for 16 cycles of one of its four matrix cores.  So
//   * activations lie in LDS with their halo of zeros, [8-channel half][10^3][8]:
//     a fragment is one conflict-free 16-byte read per lane at a constant offset
//     from one of three lane addresses, with no bounds test;
//   * a wave takes a column of planes of one pair of y rows, marching in z: the
//     fragments of a plane serve the taps below and above it (82 reads for the
//     112 K steps of 8 planes);
//   * a layer's weights are loaded once per wave into 56 registers;
//   * the voxels are MFMA columns, so a lane ends with 4 consecutive channels of
//     one voxel and stores them in one write.
// Inference runs a layer in place in one 33 KB buffer, 4 waves of 8 planes per
// workgroup, 3 workgroups per CU.  Measured (a forward pass of 4001 blocks): 214 us
// when every wave read each tap's voxels, under a bounds test, and its weights for
// 2 tiles of 16 voxels; 90 us (688 TFLOP/s) so, of which 60 are the LDS reads.
//
// Back-propagation reuses the same operation: the data gradient is the
// convolution of the output gradient with the tap-flipped, channel-transposed
// kernel; the weight gradient is, per tap, a 16 x 16 GEMM over the 512 voxels.
// Each block writes its gradient to its own row of a partial buffer; a second
// kernel sums the rows in a fixed order (deterministic) and, in a training step,
// applies Adam to the float32 master weights and re-rounds the bf16 copies.
#include <algorithm>

#include "itm_internal.hpp"

namespace itm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kC = 16, kTaps = 27, kLayers = 4;
constexpr int kNW = kRefineWeights;
constexpr int kNP = kRefineParams;

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);   // round to nearest even
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// 16 x 16 x 32: a lane holds 8 consecutive K values of its row (A) / column (B)
__device__ __forceinline__ f32x4 mfma32(i32x4 a, i32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

// A block's 16-channel grid in LDS, its halo of zeros included: channels 8 h .. 8 h
// + 7 of voxel (x, y, z) at kHalf h + 8 (x + 1 + 10 (y + 1) + 100 (z + 1)).  The pad
// takes the reads of a plane past the last (their lanes' values are dropped).
constexpr int kPlane = 100 * 8, kHalf = 10 * kPlane;
constexpr int kGrid = 2 * kHalf + kPlane;

// K steps 0 .. 13 of a layer with 16 input channels, as a lane holds them: K step p
// is taps 2 p (lanes 0-31) and 2 p + 1 (lanes 32-63), channels 8 h .. 8 h + 7 with h =
// (lane >> 4) & 1; tap 27 is zero.  W: bf16 [tap][row][channel].
template <int P0 = 0, int P1 = 14>
__device__ __forceinline__ void load_weights(const uint16_t *W, bool flip, int lane, i32x4 (&w)[14])
{
    const int n = lane & 15, h = (lane >> 4) & 1, s = lane >> 5;
    int at = (flip ? (kTaps - 1) * kC * kC : 0) + n * kC + 8 * h;
    // opaque: the 14 addresses would otherwise be kept over the whole kernel
    asm volatile("" : "+v"(at));
    const int step = flip ? -kC * kC : kC * kC;
#pragma unroll
    for (int p = P0; p < P1; p++)
        w[p] = *reinterpret_cast<const i32x4 *>(&W[at + (p < 13 ? 2 * p + s : 26) * step]);
    if (P1 == 14 && s) w[13] = i32x4{0, 0, 0, 0};
}

// the next convolution's weights, into the registers that the products of plane r of
// this one read last
template <int NZ>
__device__ __forceinline__ void next_weights(int r, const uint16_t *W, bool flip, int lane, i32x4 (&w)[14])
{
    if (r == NZ - 1) load_weights<0, 4>(W, flip, lane, w);
    if (r == NZ) load_weights<4, 9>(W, flip, lane, w);
    if (r == NZ + 1) load_weights<9, 14>(W, flip, lane, w);
}

// acc[j] (lane: voxel column lane & 15, channels 4 (lane >> 4) + r) = the
// convolution at the 16 voxels of rows 2 yp, 2 yp + 1 of plane z0 + j: for every
// output plane the K steps in order, taps 0 .. 26 in pairs.  Planes are visited
// once, r = 0 .. NZ + 1 (input plane z0 - 1 + r), tap = 9 dz + in-plane tap:
//   E  in-plane pairs (0,1) (2,3) (4,5) (6,7): taps of dz = 0 for plane r, of dz = 2
//      for plane r - 2;
//   S  in-plane tap 8 of the plane before with tap 0 of this one: taps 8, 9 of
//      plane r - 1; its first half, alone, is tap 26 of plane r - 3;
//   O  in-plane pairs (1,2) (3,4) (5,6) (7,8): dz = 1 of plane r - 1.
//
// In training (NZ = 4, two waves per SIMD) the reads run a plane ahead of the
// products: issued as they were used, two at a time, each convolution took twice
// what its reads take, and 8 training steps of 256 blocks 458 us (with this 424, with
// the weight gradients' reads ahead too 413).  Inference (NZ = 8, three waves per
// SIMD) has neither the registers for it (68 spilled) nor the need.  after(r) runs
// behind the products of plane r.
template <int NZ, typename After>
__device__ __forceinline__ void conv16(const uint16_t *grid, i32x4 (&w)[14], int yp, int z0, int lane,
                                       f32x4 (&acc)[NZ], After after)
{
    const int n = lane & 15, h = (lane >> 4) & 1, s = lane >> 5;
    // in-plane tap 0 of input plane r = 0; the second half of the lanes reads the
    // pair's other tap, 1, 8 or (the next plane) 78 voxels on
    const uint16_t *base = grid + h * kHalf + (z0 * 100 + (2 * yp + (n >> 3)) * 10 + (n & 7)) * 8;
    const uint16_t *b1 = base + s * 8, *b8 = base + s * 64, *b78 = base + s * 624;
    const i32x4 zero = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < NZ; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // f[a]: the pair from in-plane tap a of plane r (even: E, odd: O, 8: S)
    auto load = [&](int r, i32x4 (&f)[9]) {
        const bool edge = NZ == 8 && (r == 0 || r == NZ + 1);   // the halo plane: zeros
#pragma unroll
        for (int q = 0; q < 9; q++) {
            if (q < 8 && (q & 1) && !(r >= 1 && r <= NZ)) continue;
            if (q < 8 && !(q & 1) && edge) {
                f[q] = zero;
                continue;
            }
            const uint16_t *b = q == 8 ? b78 : q == 2 || q == 5 ? b8 : b1;
            f[q] = *reinterpret_cast<const i32x4 *>(b + (r * 100 + q % 3 + 10 * (q / 3)) * 8);
        }
    };
    constexpr bool kAhead = NZ == 4;
    i32x4 f[2][9], S = zero;
    if (kAhead) load(0, f[0]);
#pragma unroll
    for (int r = 0; r < NZ + 2; r++) {
        if (!kAhead) load(r, f[r & 1]);
        else if (r < NZ + 1) load(r + 1, f[(r + 1) & 1]);
        if (kAhead) __builtin_amdgcn_sched_barrier(0);
        const i32x4 (&c)[9] = f[r & 1];
        if (r >= 1 && r <= NZ) {
            acc[r - 1] = mfma32(w[4], S, acc[r - 1]);
#pragma unroll
            for (int q = 0; q < 4; q++) acc[r - 1] = mfma32(w[5 + q], c[2 * q + 1], acc[r - 1]);
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
            if (r < NZ) acc[r] = mfma32(w[q], c[2 * q], acc[r]);
            if (r >= 2) acc[r - 2] = mfma32(w[9 + q], c[2 * q], acc[r - 2]);
        }
        S = c[8];
        if (r >= 2) acc[r - 2] = mfma32(w[13], s ? zero : S, acc[r - 2]);
        after(r);
    }
}

// Layer 1: K step g holds taps 8 g + 2 kq and 8 g + 2 kq + 1, 4 stored channels each
// (lane group kq = lane >> 4); taps past 26 are zero.
__device__ __forceinline__ void load_weights0(const uint16_t *W, int lane, i32x4 (&w)[4])
{
    const int kq = lane >> 4, n = lane & 15;
#pragma unroll
    for (int g = 0; g < 4; g++) {
        const int ta = 8 * g + 2 * kq, tb = ta + 1;
        uint2 wa = *reinterpret_cast<const uint2 *>(&W[(min(ta, kTaps - 1) * kC + n) * kC]);
        uint2 wb = *reinterpret_cast<const uint2 *>(&W[(min(tb, kTaps - 1) * kC + n) * kC]);
        if (ta >= kTaps) wa = make_uint2(0, 0);
        if (tb >= kTaps) wb = make_uint2(0, 0);
        w[g] = i32x4{(int)wa.x, (int)wa.y, (int)wb.x, (int)wb.y};
    }
}

template <int NZ>
__device__ __forceinline__ void conv0(const uint16_t *x0, const i32x4 (&w)[4], int yp, int z0, int lane,
                                      f32x4 (&acc)[NZ])
{
    const int kq = lane >> 4, n = lane & 15;
    const uint16_t *base = x0 + (z0 * 100 + (2 * yp + (n >> 3)) * 10 + (n & 7)) * 4;
#pragma unroll
    for (int j = 0; j < NZ; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < 4; g++) {
        const int ta = 8 * g + 2 * kq, tb = ta + 1;
        const int ca = min(ta, kTaps - 1), cb = min(tb, kTaps - 1);
        const uint16_t *pa = base + (ca % 3 + 10 * (ca / 3 % 3) + 100 * (ca / 9)) * 4;
        const uint16_t *pb = base + (cb % 3 + 10 * (cb / 3 % 3) + 100 * (cb / 9)) * 4;
#pragma unroll
        for (int j = 0; j < NZ; j++) {
            uint2 xa = *reinterpret_cast<const uint2 *>(pa + j * 400);
            uint2 xb = *reinterpret_cast<const uint2 *>(pb + j * 400);
            if (g == 3) {   // taps 27 and on
                if (ta >= kTaps) xa = make_uint2(0, 0);
                if (tb >= kTaps) xb = make_uint2(0, 0);
            }
            acc[j] = mfma32(w[g], i32x4{(int)xa.x, (int)xa.y, (int)xb.x, (int)xb.y}, acc[j]);
        }
    }
}

// 4 channels of a lane's voxel, rounded to bf16
__device__ __forceinline__ uint2 pack4(f32x4 v) { return __builtin_bit_cast(uint2, __builtin_convertvector(v, bf16x4)); }

// where a lane's 4 channels of plane z0 lie in the grid (a plane on: + kPlane)
__device__ __forceinline__ int grid_out(int yp, int z0, int lane)
{
    const int n = lane & 15, kq = lane >> 4;
    return (kq >> 1) * kHalf + ((z0 + 1) * 100 + (2 * yp + (n >> 3) + 1) * 10 + (n & 7) + 1) * 8 + (kq & 1) * 4;
}

__device__ __forceinline__ f32x4 load_bias(const RefineParams &P, int l, int lane)
{
    return *reinterpret_cast<const f32x4 *>(&P.bias[l * kC + 4 * (lane >> 4)]);
}

__device__ __forceinline__ f32x4 relu(f32x4 v, f32x4 b)
{
    f32x4 o;
#pragma unroll
    for (int r = 0; r < 4; r++) o[r] = fmaxf(v[r] + b[r], 0.0f);
    return o;
}

// The inference kernels' workgroups: 4 waves, wave w the rows 2 w, 2 w + 1 of all
// 8 planes
constexpr int kInferThreads = 256;
struct alignas(16) InferLds {
    uint16_t grid[kGrid];
    uint16_t x0[1000 * 4];          // network input, 10^3 grid, channels F, W/max_w, 0, 0
};

// the grid's halo (and all else) zero: once per workgroup, the layers write the inside
__device__ __forceinline__ void clear_grid(uint16_t *grid)
{
    for (int i = threadIdx.x; i < kGrid / 8; i += blockDim.x)
        reinterpret_cast<i32x4 *>(grid)[i] = i32x4{0, 0, 0, 0};
}

__device__ __forceinline__ void store_x0(uint16_t *x0, int u, float F, float W)
{
    *reinterpret_cast<uint2 *>(&x0[u * 4]) = make_uint2((uint32_t)to_bf16(F) | (uint32_t)to_bf16(W) << 16, 0u);
}

// The 4 layers on L.x0 (every thread has stored its part).  delta[j]: the
// residual of voxel column lane & 15 of plane j, on lanes 0-15.
__device__ __forceinline__ void infer_layers(InferLds &L, const RefineParams &P, int wave, int lane, float (&delta)[8])
{
    f32x4 acc[8];
    i32x4 w[14];
    const int out = grid_out(wave, 0, lane);
    {
        i32x4 w0[4];
        load_weights0(P.Wf, lane, w0);
        __syncthreads();
        conv0<8>(L.x0, w0, wave, 0, lane, acc);
    }
#pragma unroll 1
    for (int l = 0; l < kLayers - 1; l++) {
        const f32x4 b = load_bias(P, l, lane);
        load_weights(P.Wf + (size_t)(l + 1) * kTaps * kC * kC, false, lane, w);
        if (l > 0) __syncthreads();   // every wave has read the layer's input
#pragma unroll
        for (int j = 0; j < 8; j++)
            *reinterpret_cast<uint2 *>(&L.grid[out + j * kPlane]) = pack4(relu(acc[j], b));
        __syncthreads();
        conv16<8>(L.grid, w, wave, 0, lane, acc, [](int) {});
    }
    const float b = P.bias[3 * kC];
#pragma unroll
    for (int j = 0; j < 8; j++) delta[j] = acc[j][0] + b;
}

// inference only: the refined F of each block
__global__ __launch_bounds__(kInferThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_refine_infer(RefineArgs a)
{
    __shared__ InferLds L;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    clear_grid(L.grid);
    for (int64_t blk = blockIdx.x; blk < a.n; blk += gridDim.x) {
        const float *in = a.in + blk * 2000;
        for (int u = threadIdx.x; u < 1000; u += kInferThreads) store_x0(L.x0, u, in[u], in[1000 + u]);
        float delta[8];
        infer_layers(L, a.P, wave, lane, delta);
        if (lane < 16) {
            const int x = lane & 7, y = 2 * wave + (lane >> 3);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const float z = in[(x + 1) + 10 * (y + 1) + 100 * (j + 1)] + delta[j];
                a.out[blk * 512 + x + 8 * y + 64 * j] = fminf(fmaxf(z, -1.0f), 1.0f);
            }
        }
        __syncthreads();   // the next block's layer 1 overwrites the grid
    }
}

// Training: 8 waves, wave w rows 2 (w & 3), + 1 of planes 4 (w >> 2) .. + 3.  The
// hidden activations are kept for the weight gradients as x-rows per channel,
// [channel][z + 1][y + 1][x] with a halo of zero rows, the output gradient as
// [channel][voxel] (both padded by 8 elements per channel, so the 16-byte reads of
// lanes with consecutive channels fall in different LDS banks), beside the grid the
// convolutions read, which holds the back-propagated gradient afterwards (142 KB:
// one workgroup per CU).  A batch of 256 blocks is one block per CU, so the time is
// one block's chain of layers, bound by its LDS reads (14 us at their rate) and the
// waits between them: 37.7 us in a run of steps, 40.3 where other work lies between
// (in a run of steps 68 with 16 waves of 2 tiles and activations copied to channel rows
// layer by layer, 43 with nothing read ahead).
constexpr int kTrainWaves = 8, kTrainNZ = 4;
constexpr int kRowT = 512 + 8;
constexpr int kRowA = 100 * 8 + 8;
struct alignas(16) TrainLds {
    uint16_t grid[kGrid];
    uint16_t x0[1000 * 4];
    uint16_t x0T[2 * 100 * 16];       // the input's two real channels, [channel][z][y][x, padded to 16]
    uint16_t aT[3][kC * kRowA];       // hidden activations
    uint16_t gT[kC * kRowT];          // the current layer's output gradient
    float red[2][kTrainWaves];
};

// 8 bf16 of an x-row (x = 0..7) moved by s = -1, 0, +1 elements: element j of the
// result is element j + s of the row, zero outside it
__device__ __forceinline__ i32x4 shift_row(i32x4 r, int s)
{
    if (s == 0) return r;
    i32x4 o;
    if (s > 0) {
        o[0] = (int)__builtin_amdgcn_alignbit((uint32_t)r[1], (uint32_t)r[0], 16);
        o[1] = (int)__builtin_amdgcn_alignbit((uint32_t)r[2], (uint32_t)r[1], 16);
        o[2] = (int)__builtin_amdgcn_alignbit((uint32_t)r[3], (uint32_t)r[2], 16);
        o[3] = (int)__builtin_amdgcn_alignbit(0u, (uint32_t)r[3], 16);
    } else {
        o[0] = (int)__builtin_amdgcn_alignbit((uint32_t)r[0], 0u, 16);
        o[1] = (int)__builtin_amdgcn_alignbit((uint32_t)r[1], (uint32_t)r[0], 16);
        o[2] = (int)__builtin_amdgcn_alignbit((uint32_t)r[2], (uint32_t)r[1], 16);
        o[3] = (int)__builtin_amdgcn_alignbit((uint32_t)r[3], (uint32_t)r[2], 16);
    }
    return o;
}

// elements d .. d + 7 (d = 0, 1, 2) of the 16 bf16 in (r0, r1)
__device__ __forceinline__ i32x4 window8(i32x4 r0, i32x4 r1, int d)
{
    if (d == 0) return r0;
    if (d == 2) return i32x4{r0[1], r0[2], r0[3], r1[0]};
    i32x4 o;
    o[0] = (int)__builtin_amdgcn_alignbit((uint32_t)r0[1], (uint32_t)r0[0], 16);
    o[1] = (int)__builtin_amdgcn_alignbit((uint32_t)r0[2], (uint32_t)r0[1], 16);
    o[2] = (int)__builtin_amdgcn_alignbit((uint32_t)r0[3], (uint32_t)r0[2], 16);
    o[3] = (int)__builtin_amdgcn_alignbit((uint32_t)r1[0], (uint32_t)r0[3], 16);
    return o;
}

// Weight gradient of the taps (dx, dy, dz), D0 <= dx < D1, of a layer: per tap a 16 x
// 16 GEMM (M = output channel, N = input channel) over the 512 voxels, K = 32 voxels
// (4 x-rows) a step, lane group kq taking row 4 ks + kq.  A = 8 voxels of the
// gradient's channel row; B = the input row at the tap's (y, z) offset, read once
// for its three x offsets.  Both are read four K steps ahead of the products: with the
// gradient's rows held in registers for all taps instead, there was no room for that
// (54 registers spilled, 465 us per 8 steps against 413, and 424 without reading ahead).
template <int D0, int D1, bool FIRST>
__device__ __forceinline__ void weight_grad(const uint16_t *xT, const uint16_t *gT, int c, int lane, float *gp)
{
    const int kq = lane >> 4, n = lane & 15, dz = c / 3, dy = c % 3;
    // row 4 ks + kq is y = 4 (ks & 1) + kq, z = ks >> 1
    const uint16_t *base = FIRST ? xT + ((min(n, 1) * 10 + dz) * 10 + kq + dy) * 16
                                 : xT + n * kRowA + (dz * 10 + kq + dy) * 8;
    f32x4 acc[3];
#pragma unroll
    for (int d = D0; d < D1; d++) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    // four rows ahead of the four in use
    const uint16_t *gr = &gT[n * kRowT + 8 * kq];
    i32x4 x[2][4][FIRST ? 2 : 1], g[2][4];
    auto load = [&](int b) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int ks = 4 * b + q;
            const uint16_t *p = base + ((ks >> 1) * 10 + 4 * (ks & 1)) * (FIRST ? 16 : 8);
            i32x4 (&r)[FIRST ? 2 : 1] = x[b & 1][q];
            r[0] = *reinterpret_cast<const i32x4 *>(p);
            g[b & 1][q] = *reinterpret_cast<const i32x4 *>(gr + 32 * ks);
            if constexpr (FIRST) {   // layer 1's input is the 10^3 grid: elements dx .. dx + 7 of its row
                r[1] = *reinterpret_cast<const i32x4 *>(p + 8);
                if (n > 1) r[0] = r[1] = i32x4{0, 0, 0, 0};
            }
        }
    };
    load(0);
#pragma unroll
    for (int b = 0; b < 4; b++) {
        if (b < 3) load(b + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int d = D0; d < D1; d++) {
                const i32x4 (&r)[FIRST ? 2 : 1] = x[b & 1][q];
                acc[d] = mfma32(g[b & 1][q], FIRST ? window8(r[0], r[FIRST ? 1 : 0], d) : shift_row(r[0], d - 1), acc[d]);
            }
    }
#pragma unroll
    for (int d = D0; d < D1; d++)
#pragma unroll
        for (int r = 0; r < 4; r++) gp[((3 * c + d) * kC + 4 * kq + r) * kC + n] = acc[d][r];
}

// a layer's 27 taps over the 8 waves: wave w the taps of (dy, dz) pair w, and one
// of the last pair's three on waves 1 to 3
template <bool FIRST>
__device__ __forceinline__ void weight_grads(const uint16_t *xT, const uint16_t *gT, int wave, int lane, float *gp)
{
    weight_grad<0, 3, FIRST>(xT, gT, wave, lane, gp);
    if (wave == 1) weight_grad<0, 1, FIRST>(xT, gT, 8, lane, gp);
    else if (wave == 2) weight_grad<1, 2, FIRST>(xT, gT, 8, lane, gp);
    else if (wave == 3) weight_grad<2, 3, FIRST>(xT, gT, 8, lane, gp);
}

__global__ __launch_bounds__(kTrainWaves * 64) void k_refine_train(RefineArgs a)
{
    constexpr int NZ = kTrainNZ;
    __shared__ TrainLds L;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // in a scalar register
    const int yp = wave & 3, z0 = NZ * (wave >> 2);
    for (int64_t blk = blockIdx.x; blk < a.n; blk += gridDim.x) {
        // opaque: what follows from the lane is formed again for each block, not kept
        // in registers over all of them
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int kq = lane >> 4, n = lane & 15;
        const int out = grid_out(yp, z0, lane);
        const int vox = (n & 7) + 8 * (2 * yp + (n >> 3)) + 64 * z0;   // the lane's voxel of plane z0
        const int voxA = (n & 7) + ((2 * yp + (n >> 3) + 1) + 10 * (z0 + 1)) * 8;
        // everything the block reads from memory, requested together
        const float *in = a.in + blk * 2000;
        float Fi[2], Wi[2], ctr[NZ], tgt[NZ];
        uint8_t msk[NZ];
        const int u1 = min((int)threadIdx.x + 512, 999);
        Fi[0] = in[threadIdx.x];
        Wi[0] = in[1000 + threadIdx.x];
        Fi[1] = in[u1];
        Wi[1] = in[1000 + u1];
        i32x4 w0[4], w[14];
        load_weights0(a.P.Wf, lane, w0);
#pragma unroll
        for (int j = 0; j < NZ; j++) {
            const int v = vox + 64 * j;
            ctr[j] = in[((v & 7) + 1) + 10 * (((v >> 3) & 7) + 1) + 100 * ((v >> 6) + 1)];
            tgt[j] = a.target[blk * 512 + v];
            msk[j] = a.mask[blk * 512 + v];
        }
        if (blk == (int64_t)blockIdx.x) {   // the halos of zeros: once, the layers write the inside
            clear_grid(L.grid);
            i32x4 *z = reinterpret_cast<i32x4 *>(L.aT[0]);
            for (int i = threadIdx.x; i < (int)(sizeof L.aT / 16); i += kTrainWaves * 64) z[i] = i32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int u = k ? u1 : (int)threadIdx.x;   // threads past the end store voxel 999 again
            store_x0(L.x0, u, Fi[k], Wi[k]);
            const int o = (u / 10) * 16 + u % 10;
            L.x0T[o] = to_bf16(Fi[k]);
            L.x0T[1600 + o] = to_bf16(Wi[k]);
        }
        f32x4 acc[NZ];
        uint64_t on = 0;   // bit 16 l + 4 j + r: hidden layer l, channel 4 kq + r of plane j is positive
        load_weights(a.P.Wf + kTaps * kC * kC, false, lane, w);
        __syncthreads();
        conv0<NZ>(L.x0, w0, yp, z0, lane, acc);
        // (not unrolled, nor the backward loop: a block runs the code once, and
        // fetching it takes as long as running it)
#pragma unroll 1
        for (int l = 0; l < kLayers - 1; l++) {
            const f32x4 b = load_bias(a.P, l, lane);
            if (l > 0) __syncthreads();   // every wave has read the layer's input
            uint32_t bits = 0u;
#pragma unroll
            for (int j = 0; j < NZ; j++) {
                const uint2 v = pack4(relu(acc[j], b));
                *reinterpret_cast<uint2 *>(&L.grid[out + j * kPlane]) = v;
                const uint16_t e[4] = {(uint16_t)v.x, (uint16_t)(v.x >> 16), (uint16_t)v.y, (uint16_t)(v.y >> 16)};
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    L.aT[l][(4 * kq + r) * kRowA + voxA + 80 * j] = e[r];
                    bits |= (from_bf16(e[r]) > 0.0f ? 1u : 0u) << (4 * j + r);
                }
            }
            on |= (uint64_t)bits << (16 * l);
            const uint16_t *wn =
                l < 2 ? a.P.Wf + (size_t)(l + 2) * kTaps * kC * kC : a.P.Wt + (size_t)3 * kTaps * kC * kC;
            __syncthreads();
            conv16<NZ>(L.grid, w, yp, z0, lane, acc, [&](int r) { next_weights<NZ>(r, wn, l == 2, lane, w); });
        }
        // residual, clamp, loss and its gradient (lanes 0-15 hold the output channel);
        // the gradient of the 15 unused channels is zero
        float sq = 0.0f, cnt = 0.0f;
        f32x4 G[NZ];
#pragma unroll
        for (int j = 0; j < NZ; j++) G[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (kq == 0) {
            const float b = a.P.bias[3 * kC];
#pragma unroll
            for (int j = 0; j < NZ; j++) {
                const int v = vox + 64 * j;
                const float z = ctr[j] + (acc[j][0] + b);
                const float Fo = fminf(fmaxf(z, -1.0f), 1.0f);
                const bool m = msk[j] != 0;
                const float e = Fo - tgt[j];
                if (m) { sq += e * e; cnt += 1.0f; }
                G[j][0] = (m && z > -1.0f && z < 1.0f) ? 2.0f * e : 0.0f;
                if (a.out) a.out[blk * 512 + v] = Fo;
            }
        }
        // loss partial: reduce over the wave, then over the waves in wave order
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            sq += __shfl_xor(sq, o, 64);
            cnt += __shfl_xor(cnt, o, 64);
        }
        if (lane == 0) { L.red[0][wave] = sq; L.red[1][wave] = cnt; }
        float *gp = a.grad_part + blk * kNP;
#pragma unroll 1
        for (int l = kLayers - 1; l >= 0; l--) {
            __syncthreads();   // the grid and the gradient rows are read
            if (l == kLayers - 1 && threadIdx.x == 0) {
                float s0 = 0.0f, s1 = 0.0f;
                for (int i = 0; i < kTrainWaves; i++) {
                    s0 += L.red[0][i];
                    s1 += L.red[1][i];
                }
                a.loss_part[blk * 2] = s0;
                a.loss_part[blk * 2 + 1] = s1;
            }
            // the layer's output gradient: for the data gradient's convolution and as
            // channel rows for the weight gradient
#pragma unroll
            for (int j = 0; j < NZ; j++) {
                const uint2 v = pack4(G[j]);
                *reinterpret_cast<uint2 *>(&L.grid[out + j * kPlane]) = v;
                const uint16_t e[4] = {(uint16_t)v.x, (uint16_t)(v.x >> 16), (uint16_t)v.y, (uint16_t)(v.y >> 16)};
#pragma unroll
                for (int r = 0; r < 4; r++) L.gT[(4 * kq + r) * kRowT + vox + 64 * j] = e[r];
            }
            __syncthreads();
            if (l > 0) {
                // data gradient into the layer before, masked by its ReLU
                const uint16_t *wn = a.P.Wt + (size_t)(l - 1) * kTaps * kC * kC;   // (at l = 1 not used)
                conv16<NZ>(L.grid, w, yp, z0, lane, acc, [&](int r) { next_weights<NZ>(r, wn, true, lane, w); });
                const uint32_t m = (uint32_t)(on >> (16 * (l - 1)));
#pragma unroll
                for (int j = 0; j < NZ; j++)
#pragma unroll
                    for (int r = 0; r < 4; r++) G[j][r] = (m >> (4 * j + r)) & 1u ? acc[j][r] : 0.0f;
                weight_grads<false>(L.aT[l - 1], L.gT, wave, lane, gp + l * kTaps * kC * kC);
            } else {
                weight_grads<true>(L.x0T, L.gT, wave, lane, gp);
            }
            // bias gradient: sum of the (bf16) output gradient over the voxels, by the
            // last wave: lane = channel + 16 quarter, each quarter's 128 voxels in
            // order, the quarters combined by a fixed butterfly
            if (wave == kTrainWaves - 1) {
                float s = 0.0f;
                const i32x4 *row = reinterpret_cast<const i32x4 *>(&L.gT[n * kRowT + 128 * kq]);
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const i32x4 q = row[v];
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        s += from_bf16((uint16_t)q[e]);
                        s += from_bf16((uint16_t)((uint32_t)q[e] >> 16));
                    }
                }
                s += __shfl_xor(s, 16, 64);
                s += __shfl_xor(s, 32, 64);
                if (kq == 0) gp[kNW + l * kC + n] = s;
            }
        }
        __syncthreads();   // the next block overwrites the input and the grid
    }
}

// Sum the per-block partial gradients, divide by the batch's count of supervised
// voxels.  A workgroup takes 64 parameters; its 4 waves each add a contiguous
// quarter of the block rows (in row order), and the quarters are added in a fixed
// order, so the result does not depend on scheduling.
// Adam's constants for one step (bias corrections from the step count)
struct AdamConst {
    float lr, b1, b2, eps, c1, c2;
};

// Adam on float32 master weight p (value w0, moments m0 and v0) with gradient
// g, then its bf16 copies
__device__ __forceinline__ void adam_update(const AdamStep &ad, const AdamConst &k, int p, float g, float w0,
                                            float m0, float v0)
{
    const float mm = k.b1 * m0 + (1.0f - k.b1) * g;
    const float vv = k.b2 * v0 + (1.0f - k.b2) * g * g;
    ad.m[p] = mm;
    ad.v[p] = vv;
    const float w = w0 - k.lr * (mm / k.c1) / (sqrtf(vv / k.c2) + k.eps);
    ad.master[p] = w;
    if (p < kNW) {
        ad.Wf[p] = to_bf16(w);
        const int ci = p % kC, co = (p / kC) % kC, lt = p / (kC * kC);
        ad.Wt[(lt * kC + ci) * kC + co] = to_bf16(w);
    } else {
        ad.bias[p - kNW] = w;
    }
}

// The mean gradient (and with ADAM the step it drives): per parameter, the
// partial rows added in a fixed order, divided by the count of masked voxels
template <bool ADAM>
__global__ __launch_bounds__(256) void k_refine_reduce(const float *grad_part, const float *loss_part, int64_t n,
                                                       float *grad, float *loss, AdamStep ad, AdamConst k)
{
    __shared__ float part[4][64];
    __shared__ float s_inv;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    const int64_t r0 = n * q / 4, r1 = n * (q + 1) / 4;
    // the weight and its moments are read first, so that their round trip
    // overlaps the partial rows'
    float w0 = 0.0f, m0 = 0.0f, v0 = 0.0f;
    if (ADAM && q == 0 && p < kNP) {
        w0 = ad.master[p];
        m0 = ad.m[p];
        v0 = ad.v[p];
    }
    // the quarter's rows added in row order, sixteen loads in flight ahead of
    // the additions (the scheduling barrier keeps the compiler from moving the
    // first additions, and so their waits, between the loads)
    float acc = 0.0f;
    if (p < kNP) {
        int64_t b = r0;
        for (; b + 16 <= r1; b += 16) {
            float v[16];
#pragma unroll
            for (int j = 0; j < 16; j++) v[j] = grad_part[(b + j) * kNP + p];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 16; j++) acc += v[j];
        }
        for (; b < r1; b++) acc += grad_part[b * kNP + p];
    }
    part[q][lane] = acc;
    if (q == 0) {
        // the counted voxels (integers, exact in any order) and, for the loss,
        // the squared errors: the first wave, a fixed butterfly, lane 0's sums
        float cnt = 0.0f, sq = 0.0f;
        for (int64_t b = lane; b < n; b += 64) {
            cnt += loss_part[2 * b + 1];
            if (blockIdx.x == 0) sq += loss_part[2 * b];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            cnt += __shfl_xor(cnt, o, 64);
            sq += __shfl_xor(sq, o, 64);
        }
        if (lane == 0) {
            s_inv = 1.0f / fmaxf(cnt, 1.0f);
            if (blockIdx.x == 0) loss[0] = sq * s_inv;
        }
    }
    __syncthreads();
    if (q == 0 && p < kNP) {
        const float g = ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane])) * s_inv;
        grad[p] = g;
        if (ADAM) adam_update(ad, k, p, g, w0, m0, v0);
    }
}

// bf16 copies of a master vector (after a parameter upload)
__global__ void k_refine_cast(const float *master, uint16_t *Wf, uint16_t *Wt, float *bias)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kNP) return;
    const float w = master[p];
    if (p < kNW) {
        Wf[p] = to_bf16(w);
        const int ci = p % kC, co = (p / kC) % kC, lt = p / (kC * kC);
        Wt[(lt * kC + ci) * kC + co] = to_bf16(w);
    } else {
        bias[p - kNW] = w;
    }
}

// The voxel blocks of a block and its 26 neighbours (index (dx + 1) + 3 (dy + 1) +
// 9 (dz + 1); -1 where absent), one hash lookup each by the first 27 threads: the
// 10^3 voxels around a block lie in them.
__device__ __forceinline__ void neighbour_blocks(const HashView &h, int kx, int ky, int kz, int32_t *nb)
{
    if (threadIdx.x < 27) {
        const int t = threadIdx.x;
        nb[t] = block_of(h, find_block_direct(h, kx + t % 3 - 1, ky + t / 3 % 3 - 1, kz + t / 9 - 1));
    }
}

// F and W / max_w of voxel u of the 10^3 grid around a block; voxels of absent
// blocks read F = 1, W = 0
template <int FMT>
__device__ __forceinline__ void halo_voxel(const int32_t *nb, const typename Vox<FMT>::S *S,
                                           const typename Vox<FMT>::Wt *W, float inv_max_w, int u, float &F, float &Wf)
{
    const int x = u % 10 + 7, y = u / 10 % 10 + 7, z = u / 100 + 7;   // + 7: the block index is the quotient by 8
    const int32_t p = nb[(x >> 3) + 3 * (y >> 3) + 9 * (z >> 3)];
    F = 1.0f;
    Wf = 0.0f;
    if (p >= 0) {
        const int64_t i = (int64_t)p * kBlockVox + (x & 7) + 8 * (y & 7) + 64 * (z & 7);
        F = Vox<FMT>::to_f(S[i]);
        Wf = Vox<FMT>::w_to_f(W[i]) * inv_max_w;
    }
}

// network input of a block from the volume
template <int FMT>
__global__ __launch_bounds__(256) void k_refine_gather(HashView h, const void *sdf, const void *w,
                                                       const int32_t *coords, int64_t n, float inv_max_w, float *out)
{
    using V = Vox<FMT>;
    __shared__ int32_t nb[27];
    for (int64_t b = blockIdx.x; b < n; b += gridDim.x) {
        neighbour_blocks(h, coords[3 * b], coords[3 * b + 1], coords[3 * b + 2], nb);
        __syncthreads();
        for (int u = threadIdx.x; u < 1000; u += blockDim.x) {
            float F, Wf;
            halo_voxel<FMT>(nb, (const typename V::S *)sdf, (const typename V::Wt *)w, inv_max_w, u, F, Wf);
            out[b * 2000 + u] = F;
            out[b * 2000 + 1000 + u] = Wf;
        }
        __syncthreads();
    }
}

// Per-frame inference gate: every visible block whose largest weight is below
// the threshold is refined; its network input is gathered straight from the
// volume into LDS and the refined F goes to a side buffer (half precision,
// indexed like the voxel block array) stamped with the frame number.
template <int FMT>
__global__ __launch_bounds__(kInferThreads) __attribute__((amdgpu_waves_per_eu(3))) void
k_refine_gated(RefineGateArgs a)
{
    using V = Vox<FMT>;
    __shared__ InferLds L;
    __shared__ int32_t nb[27];
    const auto *S = (const typename V::S *)a.sdf;
    const auto *Wv = (const typename V::Wt *)a.w;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    clear_grid(L.grid);
    // the visible list (workgroup-uniform loop)
    const VisPrefix vp = vis_prefix(a.list, lane);
    for (int bi = blockIdx.x; bi < vp.total; bi += gridDim.x) {
        const VisRec rec = vis_item(a.list, vp, bi);
        const int32_t ptr = block_of(a.h, rec.e);
        int kx, ky, kz;
        unpack_key(rec.key, kx, ky, kz);
        neighbour_blocks(a.h, kx, ky, kz, nb);
        // gate on the block's largest weight
        bool heavy = false;
        if (ptr >= 0)
#pragma unroll
            for (int i = 0; i < kBlockVox; i += kInferThreads)
                heavy |= V::w_to_f(Wv[(int64_t)ptr * kBlockVox + i + threadIdx.x]) >= a.w_threshold;
        if (__syncthreads_or(heavy || ptr < 0)) continue;   // uniform over the workgroup
        for (int u = threadIdx.x; u < 1000; u += kInferThreads) {
            float F, Wf;
            halo_voxel<FMT>(nb, S, Wv, a.inv_max_w, u, F, Wf);
            store_x0(L.x0, u, F, Wf);
        }
        float delta[8];
        infer_layers(L, a.P, wave, lane, delta);
        if (lane < 16) {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int64_t i = (int64_t)ptr * kBlockVox + lane + 16 * wave + 64 * j;   // x + 8 y + 64 z
                const float z = V::to_f(S[i]) + delta[j];
                a.refined[i] = __float2half_rn(fminf(fmaxf(z, -1.0f), 1.0f));
            }
        }
        if (threadIdx.x == 0) a.stamp[ptr] = a.frame;
        __syncthreads();   // the next block overwrites nb, the input and the grid
    }
}

hipError_t launch_refine_gated(int fmt, const RefineGateArgs &a, int grid, hipStream_t st)
{
    switch (fmt) {
    case ITM_VOX_F32: launch_k(k_refine_gated<ITM_VOX_F32>, grid, kInferThreads, st, a); break;
    case ITM_VOX_F16: launch_k(k_refine_gated<ITM_VOX_F16>, grid, kInferThreads, st, a); break;
    default: launch_k(k_refine_gated<ITM_VOX_S16U8>, grid, kInferThreads, st, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_refine(const RefineArgs &a, bool train, int grid, hipStream_t st)
{
    if (train) k_refine_train<<<grid, kTrainWaves * 64, 0, st>>>(a);
    else k_refine_infer<<<grid, kInferThreads, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_refine_reduce(const float *grad_part, const float *loss_part, int64_t n, float *grad,
                                float *loss, const AdamStep *adam, hipStream_t st)
{
    const int grid = (kNP + 63) / 64;
    if (adam) {
        AdamConst k;
        k.lr = adam->lr;
        k.b1 = 0.9f;
        k.b2 = 0.999f;
        k.eps = 1e-8f;
        k.c1 = 1.0f - powf(k.b1, (float)adam->step);
        k.c2 = 1.0f - powf(k.b2, (float)adam->step);
        k_refine_reduce<true><<<grid, 256, 0, st>>>(grad_part, loss_part, n, grad, loss, *adam, k);
    } else {
        k_refine_reduce<false><<<grid, 256, 0, st>>>(grad_part, loss_part, n, grad, loss, AdamStep{}, AdamConst{});
    }
    return hipGetLastError();
}

hipError_t launch_refine_cast(const float *master, uint16_t *Wf, uint16_t *Wt, float *bias, hipStream_t st)
{
    k_refine_cast<<<(kNP + 255) / 256, 256, 0, st>>>(master, Wf, Wt, bias);
    return hipGetLastError();
}

hipError_t launch_refine_gather(int fmt, const HashView &h, const void *sdf, const void *w, const int32_t *coords,
                                int64_t n, float inv_max_w, float *out, hipStream_t st)
{
    const int grid = (int)std::min<int64_t>(n, 4096);
    if (grid <= 0) return hipSuccess;
    switch (fmt) {
    case ITM_VOX_F32: k_refine_gather<ITM_VOX_F32><<<grid, 256, 0, st>>>(h, sdf, w, coords, n, inv_max_w, out); break;
    case ITM_VOX_F16: k_refine_gather<ITM_VOX_F16><<<grid, 256, 0, st>>>(h, sdf, w, coords, n, inv_max_w, out); break;
    default: k_refine_gather<ITM_VOX_S16U8><<<grid, 256, 0, st>>>(h, sdf, w, coords, n, inv_max_w, out); break;
    }
    return hipGetLastError();
}

}  // namespace itm
