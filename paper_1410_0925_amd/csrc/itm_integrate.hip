// Integration (section "Integration", computeUpdatedVoxelDepthInfo) over the
// voxels of the frame's visible blocks.
//
// One wave per visible block (two with colour), taken from the visible list the
// allocation built (its counters are read on the device: no count goes to the
// host).  Lane l owns voxels 4l..4l+3 and 256+4l..256+4l+3 of the block (with
// colour, one of the two groups), so every voxel load or store instruction of a
// wave covers one contiguous range (16 B per lane in the float form).  A lane
// reads its voxels, decides for
// each whether it is updated -- that needs only the voxel's position and the
// depth image -- and writes back a group of 4 voxels only when one of them is.
//
// Decisions follow a fixed binary32 evaluation order (so that they can be
// reproduced exactly): the block origin's camera coordinates are formed in binary64
// once per block and split into a binary32 pair hi + lo; the in-block offset
// (lx g_x + ly g_y) + lz g_z is added to lo first.  The value eta = d - p_z is
// formed as (d - hi_z) - (lo_z + offset_z), accurate to ~1e-8 m at room scale.
#include <algorithm>

#include "itm_alloc.hpp"

namespace itm {

// 4 consecutive voxels of one storage form.  put() replaces voxel j where upd; the
// empty statements in it keep the new value's arithmetic out of a branch on upd,
// which the compiler would otherwise make of the selects.
template <int FMT>
struct Group4;

template <>
struct Group4<ITM_VOX_F32> {
    float4 s, w;
    __device__ void load(const void *sdf, const void *wt, int64_t i)
    {
        s = *reinterpret_cast<const float4 *>((const float *)sdf + i);
        w = *reinterpret_cast<const float4 *>((const float *)wt + i);
    }
    __device__ void store(void *sdf, void *wt, int64_t i) const
    {
        *reinterpret_cast<float4 *>((float *)sdf + i) = s;
        *reinterpret_cast<float4 *>((float *)wt + i) = w;
    }
    __device__ float F(int j) const { return j == 0 ? s.x : j == 1 ? s.y : j == 2 ? s.z : s.w; }
    __device__ float Wv(int j) const { return j == 0 ? w.x : j == 1 ? w.y : j == 2 ? w.z : w.w; }
    __device__ void put(int j, bool upd, float f, float wv)
    {
        float &sj = j == 0 ? s.x : j == 1 ? s.y : j == 2 ? s.z : s.w;
        float &wj = j == 0 ? w.x : j == 1 ? w.y : j == 2 ? w.z : w.w;
        asm volatile("" : "+v"(f), "+v"(wv));
        sj = upd ? f : sj;
        wj = upd ? wv : wj;
    }
};

template <>
struct Group4<ITM_VOX_F16> {
    __half s[4], w[4];
    __device__ void load(const void *sdf, const void *wt, int64_t i)
    {
        const uint2 a = *reinterpret_cast<const uint2 *>((const __half *)sdf + i);
        const uint2 b = *reinterpret_cast<const uint2 *>((const __half *)wt + i);
        __builtin_memcpy(s, &a, 8);
        __builtin_memcpy(w, &b, 8);
    }
    __device__ void store(void *sdf, void *wt, int64_t i) const
    {
        uint2 a, b;
        __builtin_memcpy(&a, s, 8);
        __builtin_memcpy(&b, w, 8);
        *reinterpret_cast<uint2 *>((__half *)sdf + i) = a;
        *reinterpret_cast<uint2 *>((__half *)wt + i) = b;
    }
    __device__ float F(int j) const { return __half2float(s[j]); }
    __device__ float Wv(int j) const { return __half2float(w[j]); }
    __device__ void put(int j, bool upd, float f, float wv)
    {
        uint32_t sn = __half_as_ushort(__float2half_rn(f)), wn = __half_as_ushort(__float2half_rn(wv));
        asm volatile("" : "+v"(sn), "+v"(wn));
        s[j] = upd ? __ushort_as_half((unsigned short)sn) : s[j];
        w[j] = upd ? __ushort_as_half((unsigned short)wn) : w[j];
    }
};

template <>
struct Group4<ITM_VOX_S16U8> {
    int16_t s[4];
    uint8_t w[4];
    __device__ void load(const void *sdf, const void *wt, int64_t i)
    {
        const uint2 a = *reinterpret_cast<const uint2 *>((const int16_t *)sdf + i);
        const uint32_t b = *reinterpret_cast<const uint32_t *>((const uint8_t *)wt + i);
        __builtin_memcpy(s, &a, 8);
        __builtin_memcpy(w, &b, 4);
    }
    __device__ void store(void *sdf, void *wt, int64_t i) const
    {
        uint2 a;
        uint32_t b;
        __builtin_memcpy(&a, s, 8);
        __builtin_memcpy(&b, w, 4);
        *reinterpret_cast<uint2 *>((int16_t *)sdf + i) = a;
        *reinterpret_cast<uint32_t *>((uint8_t *)wt + i) = b;
    }
    __device__ float F(int j) const { return Vox<ITM_VOX_S16U8>::to_f(s[j]); }
    __device__ float Wv(int j) const { return (float)w[j]; }
    __device__ void put(int j, bool upd, float f, float wv)
    {
        int32_t sn = Vox<ITM_VOX_S16U8>::from_f(f);
        uint32_t wn = (uint8_t)wv;
        asm volatile("" : "+v"(sn), "+v"(wn));
        s[j] = upd ? (int16_t)sn : s[j];
        w[j] = upd ? (uint8_t)wn : w[j];
    }
};

// Colour sample of a voxel (section "Framework Flexibility" gives the voxel's
// RGB and colour weight; the update is the library's reading): each channel keeps
// the running average of its samples rounded to the nearest integer, ties to
// even, in exact integer arithmetic; the weight counts samples up to cap.
//
// Every integer here is below 2^17, so exact in binary32, and the quotient
// floor((w c + s) / (w + 1)) needs no division: (num + 1/2) / den lies at least
// 1/512 from any integer, and the product with the reciprocal (1 ulp) within 2^-13
// of it.
__device__ __forceinline__ uint32_t colour_step(uint32_t c, uint32_t s, float cap)
{
    const float w = (float)(c >> 24), den = w + 1.0f;
    const float rden = __builtin_amdgcn_rcpf(den);
    uint32_t out = (uint32_t)fminf(den, cap) << 24;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const float num = w * (float)((c >> (8 * k)) & 0xffu) + (float)((s >> (8 * k)) & 0xffu);
        const float q = floorf((num + 0.5f) * rden);
        const float r2 = 2.0f * (num - q * den);
        // q + 1/4, 1/2 or 3/4 rounds to even as the exact quotient does
        const float m = q + (r2 < den ? 0.25f : r2 > den ? 0.75f : 0.5f);
        out |= (uint32_t)rintf(m) << (8 * k);
    }
    return out;
}

// Waves per block.  With colour each takes half a block: a whole one needs 105 to 112
// registers (held to 92 for 5 waves per SIMD), a half 73 to 79 and runs 6 (24.4 and
// 22.2 us at 640x480 in S16U8).  Without colour the halves only repeat the block's own
// arithmetic (16.9 and 16.7 us at 640x480 in F32, 38.2 and 39.0 at 1280x720 in F16).
template <bool CLR>
constexpr int kParts = CLR ? 2 : 1;

// One visible block (entry e), or half of one, by one wave; returns the number of
// updated voxels (uniform over the wave).
//
// Bound by instruction issue.  Nothing branches on a voxel: a read that is not
// wanted goes to pixel 0, a voxel that is not updated keeps its bits by selects,
// and only a group of 4 voxels with none updated skips its arithmetic and its
// store.  With a branch for each test (six per voxel, some 50 cycles each) the
// kernel took 44.2 us at 1280x720 in F16, 19.4 at 640x480 in F32 and, with the
// colour's depth and RGB reads waited for voxel by voxel and three integer
// divisions each, 29.2 at 640x480 in S16U8 with colour; now 38.2,
// 16.9 and 22.2.
template <int FMT, bool CLR>
__device__ __forceinline__ uint32_t integrate_block(const FuseArgs &a, unsigned long long key, int32_t e, int lane,
                                                    int part)
{
    constexpr int kGroups = 2 / kParts<CLR>;
    const FrameGeom &g = a.fg;
    const int32_t ptr = __builtin_amdgcn_readfirstlane(block_of(a.h, e));   // the entry's voxel block
    if (ptr < 0) return 0;                  // swapping: no device block this frame
    int kx, ky, kz;
    unpack_key(key, kx, ky, kz);
    // The voxels are loaded together with the depth reads instead of after
    // them (the update decision needs only the depth image): one dependent
    // memory round less, for about 6% more voxel bytes read (whole 128-byte
    // lines are touched anyway).
    const int64_t vbase = (int64_t)ptr * kBlockVox;
    Group4<FMT> vg[kGroups];
    uint4 cg[kGroups];
#pragma unroll
    for (int grp = 0; grp < kGroups; grp++) {
        vg[grp].load(a.sdf, a.w, vbase + 4 * lane + 256 * (part + grp));
        if (CLR) cg[grp] = *reinterpret_cast<const uint4 *>(a.clr + vbase + 4 * lane + 256 * (part + grp));
    }
    // block origin in camera coordinates, binary64 -> binary32 pair
    const double o0 = (double)(8 * kx) * g.s, o1 = (double)(8 * ky) * g.s, o2 = (double)(8 * kz) * g.s;
    float hi[3], lo[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        double w = g.Rcw[3 * c + 0] * o0;
        w = w + g.Rcw[3 * c + 1] * o1;
        w = w + g.Rcw[3 * c + 2] * o2;
        w = w + g.tcw[c];
        hi[c] = (float)w;
        lo[c] = (float)(w - (double)hi[c]);
    }
    const float mu = g.mu_f, inv_mu = 1.0f / mu;
    // Voxel (x, y, z) of the block, x = 4 (lane & 1) + j: the lane's voxels are
    // all projected and their reads issued together (one memory round).
    const float fy_ = (float)((lane >> 1) & 7);
    float gx[4][3], gy[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        gy[c] = fy_ * g.g[1][c];
#pragma unroll
        for (int j = 0; j < 4; j++) gx[j][c] = (float)(4 * (lane & 1) + j) * g.g[0][c];
    }
    float dep[kGroups][4], zlo[kGroups][4];   // depth; the voxel's camera z without hi
    uint32_t smp[kGroups][4];
    bool seen[kGroups][4];
#pragma unroll
    for (int grp = 0; grp < kGroups; grp++) {
        const float fz_ = (float)((lane >> 4) + 4 * (part + grp));
        float yz[3];   // the group's y and z steps, shared by its 4 voxels
#pragma unroll
        for (int c = 0; c < 3; c++) yz[c] = gy[c] + fz_ * g.g[2][c];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float p[3], l[3];
#pragma unroll
            for (int c = 0; c < 3; c++) {
                l[c] = lo[c] + (gx[j][c] + yz[c]);
                p[c] = hi[c] + l[c];
            }
            zlo[grp][j] = l[2];
            const float rz = __builtin_amdgcn_rcpf(p[2]);   // 1 ulp; one reciprocal for x and y
            const float x = g.fx * p[0] * rz + g.cx;
            const float y = g.fy * p[1] * rz + g.cy;
            seen[grp][j] = !(p[2] <= 0.0f) & !(x < 1.0f) & !(x > (float)(g.W - 2)) & !(y < 1.0f) &
                           !(y > (float)(g.H - 2));
            const int pix = (int)(x + 0.5f) + __mul24((int)(y + 0.5f), g.W);   // sizes are <= 2^15
            const uint32_t at = seen[grp][j] ? (uint32_t)pix << 2 : 0u;        // pixel 0 when unseen: not used
            dep[grp][j] = *reinterpret_cast<const float *>((const char *)a.depth + at);
            if (CLR) smp[grp][j] = *reinterpret_cast<const uint32_t *>((const char *)a.rgbx + at);
        }
    }
    uint32_t n_upd = 0;
    const float ccap = fminf(g.max_w_f, 255.0f);
#pragma unroll
    for (int grp = 0; grp < kGroups; grp++) {
        float eta[4];
        bool upd[4], any = false;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float d = dep[grp][j];
            eta[j] = (d - hi[2]) - zlo[grp][j];
            // a finite depth above 0 (class: positive normal or subnormal)
            upd[j] = seen[grp][j] & __builtin_amdgcn_classf(d, 0x180) & !(eta[j] < -mu);
            n_upd += (uint32_t)__popcll(__ballot(upd[j]));
            any |= upd[j];
        }
        if (!any) continue;
        Group4<FMT> &v = vg[grp];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float f = fminf(1.0f, eta[j] * inv_mu);
            const float F = v.F(j), W = v.Wv(j);
            const float Wn = W + 1.0f;
            // running average F <- (W F + f) / (W + 1), in incremental form (the
            // reciprocal of the integer W + 1 to 1 ulp)
            const float Fn = F + (f - F) * __builtin_amdgcn_rcpf(Wn);
            v.put(j, upd[j], Fn, fminf(Wn, g.max_w_f));
        }
        v.store(a.sdf, a.w, vbase + 4 * lane + 256 * (part + grp));
        if constexpr (CLR) {
            uint32_t c4[4] = {cg[grp].x, cg[grp].y, cg[grp].z, cg[grp].w};
            bool cany = false;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const bool in = upd[j] & (eta[j] <= mu);   // inside the band: a colour sample
                uint32_t c = colour_step(c4[j], smp[grp][j], ccap);
                asm volatile("" : "+v"(c));   // as in put()
                c4[j] = in ? c : c4[j];
                cany |= in;
            }
            if (cany)
                *reinterpret_cast<uint4 *>(a.clr + vbase + 4 * lane + 256 * (part + grp)) =
                    make_uint4(c4[0], c4[1], c4[2], c4[3]);
        }
    }
    return n_upd;
}

// Allocation and visible list (itm_alloc.hpp), one thread per pixel:
//   1. housekeeping, every workgroup its share: the previous frame's claim slots
//      and, with the search range on, the next frame's bin counts are cleared
//      (the stores go out after step 2, the one count they need is loaded with
//      the depth);
//   2. each thread walks its pixel's band segment and claims the blocks' keys in
//      the workgroup's LDS set; the lane that claims a key first finds or inserts
//      the block and records its entry there;
//   3. every block of the set is stamped with the frame number (by the lane that
//      found it, as soon as it has the entry); the workgroup that stamps a block
//      first lists it (one atomic per workgroup on one of 32 list stripes), so
//      each visible block is listed exactly once;
//   4. with the search range on, the listed blocks' expected-depth rectangles
//      are binned by image tile.
__global__ __launch_bounds__(256) void k_alloc(FuseArgs a)
{
    const FrameGeom &g = a.fg;
    __shared__ int32_t s_e[kSet];
    __shared__ unsigned long long s_k[kSet];
    __shared__ int s_wave[4], s_n, s_base, s_ovf;
    // the previous frame's claim count (for the housekeeping) and the pixel's
    // depth are loaded first, together: one memory round before the allocation
    const int su = *a.set_used_prev;
    int tx, ty;
    if (!xcd_tile((g.W + 15) / 16, (g.H + 15) / 16, tx, ty)) {   // whole workgroup
        frame_housekeeping(a, su);
        return;
    }
    const int u = tx * 16 + (threadIdx.x & 15);
    const int v = ty * 16 + (threadIdx.x >> 4);
    const bool in_image = u < g.W && v < g.H;
    float depth = 0.0f;
    if (in_image) depth = a.depth[(int64_t)v * g.W + u];
#pragma unroll
    for (int j = 0; j < kSet / 256; j++) {
        s_e[threadIdx.x + 256 * j] = -1;
        s_k[threadIdx.x + 256 * j] = 0ull;
    }
    __syncthreads();
    // 2. allocation
    if (in_image && depth > 0.0f && !isinf(depth)) alloc_pixel(a, u, v, depth, s_e, s_k);
    __syncthreads();
    // 1. housekeeping, its stores off the allocation's path
    frame_housekeeping(a, su);
    // 3. the visible list: thread t takes set slots 8t..8t+7 (those its workgroup
    //    stamped first hold their entry)
    uint32_t win = 0;
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int32_t e = s_e[8 * threadIdx.x + j];
        if (e >= 0) win |= 1u << j;   // stamped and won in step 2
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int c = __builtin_popcount(win);
    int incl = c;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    unsigned long long wkey[8];
    int32_t went[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        wkey[j] = s_k[8 * threadIdx.x + j];
        went[j] = s_e[8 * threadIdx.x + j];
    }
    __syncthreads();
    // thread 0 reserves the workgroup's list records; the reservation is consumed
    // only after the binning's projections, which hide its round trip (barriers
    // wait for LDS traffic, not for this atomic)
    const int stripe = blockIdx.x % 32;
    int base = 0;
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < 4; w++) {
            const int x = s_wave[w];
            s_wave[w] = t;
            t += x;
        }
        s_n = t;
        // mbcnt of an empty mask is 0 on every lane, but not uniform to the
        // compiler: the atomic stays a plain returning one, waited for where
        // base is used, instead of a wave-aggregated one broadcast at once
        if (t) base = atomicAdd(&a.list.cnt[32 * stripe + (int)__builtin_amdgcn_mbcnt_lo(0u, 0u)], t);
    }
    __syncthreads();
    const int n_won = s_n;
    const int k0 = s_wave[wave] + incl - c;   // workgroup index of this thread's first record
    {
        int k = k0;
#pragma unroll
        for (int j = 0; j < 8; j++)
            if (win & (1u << j)) s_k[k++] = wkey[j];   // the won keys, in list order, for the binning
    }
    auto publish = [&]() {
        if (threadIdx.x != 0) return;
        // records past the stripe's capacity go to the overflow segment
        const int spill = min(n_won, max(0, base + n_won - a.list.cap));
        s_ovf = spill ? atomicAdd(&a.list.cnt[32 * 32], spill) : 0;
        s_base = base;
    };
    // 4. expected-depth rectangles
    if (a.rb.cnt && n_won > 0) {   // uniform
        __syncthreads();
        bin_blocks(g, a.rb, s_k, n_won, s_e, publish);   // s_e is free again: its entries are in registers
    } else {
        publish();
    }
    __syncthreads();
    const int lbase = s_base, ovf = s_ovf;
    int k = k0;
#pragma unroll
    for (int j = 0; j < 8; j++) {
        if (!(win & (1u << j))) continue;
        VisRec r;
        r.key = s_k[k];   // the binning only read the keys
        r.e = went[j];
        r.pad = 0;
        const int pos = lbase + k;   // stripe position
        const int64_t slot = pos < a.list.cap ? (int64_t)stripe * a.list.cap + pos
                                              : (int64_t)32 * a.list.cap + ovf + (pos - max(lbase, a.list.cap));
        a.list.rec[slot] = r;
        k++;
    }
}

// The order of the raycast's tiles, fullest bins first, by the first kOrderWgs
// workgroups of the integration (the allocation has filled the bins; nothing here
// waits for it).  A raycast's launch ends with its longest marches, and those are in
// tiles that see many blocks: started first, they end with the rest.  Workgroup x
// sorts the tiles x, x + 8, ... into the places x, x + 8, ...: neighbours differ
// little, so the eight lists run down together.  The counts are sorted in 256 classes
// of two; tiles of a class come in any order.
//
// k_raycast: 1280x720 F16 at 4 mm (3600 tiles) 122 -> 100 us, 640x480 F32 at 5 mm
// (1200) 50.5 -> 46.6, 3840x2160 F16 at 8 mm (32400) 588 -> 518.  The order is used
// from 3 tiles per CU on: a frame of 592x432 (999 tiles) takes 76.3 us against 78.0
// without it, of 560x400 (875) and 480x360 (690) the same, of 400x300 (475) 75.2
// against 74.2 -- all of its workgroups are resident at once and the bands share
// their XCD's L2.  A raycast that finds nothing pays for reading its places (VGA 5.0
// -> 6.2 us).
//
// The sort is two rounds of reads and of LDS counting, and has to be over when the
// integration is, which for a frame that sees little takes 4 us.  By one workgroup it
// took 8.6 us at 3600 tiles, 27 at 14400 and 111 at 65536 (tiles that see nothing are
// one class and queue at its count); by eight 4.0, 6.0 and 18.
constexpr int kOrderWgs = 8;
__device__ __forceinline__ void order_tiles(const RangeBins &rb, int x)
{
    __shared__ int32_t s_at[256], s_wave[4];
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    const int n = (rb.tw * rb.th - x + kOrderWgs - 1) / kOrderWgs;   // tiles x, x + kOrderWgs, ...
    auto each = [&](auto use) {   // 8 counts in flight
        for (int i0 = t; i0 < n; i0 += 8 * 256) {
            int32_t c[8];
#pragma unroll
            for (int k = 0; k < 8; k++) c[k] = rb.cnt[x + kOrderWgs * min(i0 + 256 * k, n - 1)];
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (i0 + 256 * k < n) use(i0 + 256 * k, 255 - min(c[k] >> 1, 255));
        }
    };
    s_at[t] = 0;
    __syncthreads();
    each([&](int, int cls) { atomicAdd(&s_at[cls], 1); });
    __syncthreads();
    const int c = s_at[t];
    int incl = c;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; w++) incl += s_wave[w];
    s_at[t] = incl - c;
    __syncthreads();
    each([&](int i, int cls) { rb.order[x + kOrderWgs * atomicAdd(&s_at[cls], 1)] = x + kOrderWgs * i; });
}

// Integration.  Wave gw (pair of waves with colour) begins with place gw / 32 of
// stripe gw % 32 of the visible list, whose record is loaded together with the
// counts -- it lies inside the stripe's storage whatever they say -- so
// the two take one memory round instead of two.  All that is left over, of the
// stripes and of the overflow segment, is dealt out as one list, the next block's
// record in flight while one is integrated.
//
// The stripes hold what their image tiles saw and differ: with each stripe served
// by its own waves to the end, the fullest one ended 5 us after the rest at
// 1280x720 (42.9 us, now 38.2).
// (every wave of the grid is resident at once: 5 per SIMD, 6 with colour)
template <int FMT, bool CLR, bool ORD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CLR ? 6 : 5))) void k_integrate(FuseArgs a)
{
    __shared__ unsigned long long s_red[2][4];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t n_upd = 0, n_blk = 0;
    constexpr int kP = kParts<CLR>;
    constexpr int skip = ORD ? kOrderWgs : 0;   // workgroups that put the raycast's tiles in order
    if (ORD && blockIdx.x < skip) {
        order_tiles(a.rb, blockIdx.x);
        return;
    }
    const int gw = (((int)blockIdx.x - skip) * 4 + wave) / kP, nw = ((int)gridDim.x - skip) * 4 / kP;
    const int first = nw >> 5, part = wave % kP;
    VisRec r = a.list.rec[(int64_t)(gw & 31) * a.list.cap + min(gw >> 5, a.list.cap - 1)];
    int c = 0;
    if (lane < 33) c = a.list.cnt[32 * lane];
    if (lane < 32) c = min(c, a.list.cap);
    const bool has = (gw >> 5) < min(first, __builtin_amdgcn_readlane(c, gw & 31));
    // the others, past the first places of the stripes, as one list
    if (lane < 32) c = max(c - first, 0);
    int incl = c;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
    }
    const int excl = incl - c, n = __builtin_amdgcn_readlane(incl, kWave - 1);
    auto fetch = [&](int i) {
        const int seg = __popcll(__ballot(incl <= i));   // segments wholly before item i
        const int k = i - __builtin_amdgcn_readlane(excl, seg) + (seg < 32 ? first : 0);
        return a.list.rec[(int64_t)seg * a.list.cap + k];
    };
    int i = has ? gw : gw + nw;
    if (!has && gw < n) r = fetch(gw);
    if (has || gw < n)
        for (;;) {
            const VisRec now = r;
            const bool more = i < n;
            if (more) r = fetch(i);
            n_upd += integrate_block<FMT, CLR>(a, now.key, __builtin_amdgcn_readfirstlane(now.e), lane, part);
            n_blk += part == 0;
            if (!more) break;
            i += nw;
        }
    // one counter update per workgroup, on one of kStripes separate lines
    if (lane == 0) {
        s_red[0][wave] = n_upd;
        s_red[1][wave] = n_blk;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long u = s_red[0][0] + s_red[0][1] + s_red[0][2] + s_red[0][3];
        const unsigned long long v = s_red[1][0] + s_red[1][1] + s_red[1][2] + s_red[1][3];
        const int sI = blockIdx.x % kStripes;
        if (u) {
            atomicAdd(&a.cnt->upd[a.parity][sI][0], u);
            atomicAdd(&a.cnt->upd[2][sI][0], u);
        }
        if (v) {
            atomicAdd(&a.cnt->vis[a.parity][sI][0], v);
            atomicAdd(&a.cnt->vis[2][sI][0], v);
        }
    }
}

// Loading a volume (itm_import_blocks): a frame of its own whose visited blocks
// are the n given keys.  One thread per key: housekeeping as in k_alloc, then
// find or insert the block, stamp it, and list it when this thread stamped it
// first (the key list has no repeats, so that is every key that found an
// entry); entry[i] = the block's entry (= its voxel block), -1 when dropped.
__global__ __launch_bounds__(256) void k_import_keys(FuseArgs a, const int32_t *coords, int32_t n, int32_t *entry)
{
    frame_housekeeping(a, *a.set_used_prev);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int bx = coords[3 * i], by = coords[3 * i + 1], bz = coords[3 * i + 2];
    const int32_t e = find_or_insert(a, bx, by, bz);
    entry[i] = e;
    if (e < 0) return;
    if (atomicExch(&a.stamp[e], a.stamp_now) == a.stamp_now) return;
    const int stripe = i % 32, sI = i % kStripes;
    const int pos = atomicAdd(&a.list.cnt[32 * stripe], 1);
    VisRec r;
    r.key = pack_key(bx, by, bz);
    r.e = e;
    r.pad = 0;
    if (pos < a.list.cap) a.list.rec[(int64_t)stripe * a.list.cap + pos] = r;
    else a.list.rec[(int64_t)32 * a.list.cap + atomicAdd(&a.list.cnt[32 * 32], 1)] = r;
    atomicAdd(&a.cnt->vis[a.parity][sI][0], 1ull);
    atomicAdd(&a.cnt->vis[2][sI][0], 1ull);
}

hipError_t launch_import_keys(const FuseArgs &a, const int32_t *coords, int32_t n, int32_t *entry, hipStream_t st)
{
    k_import_keys<<<std::max(1, (n + 255) / 256), 256, 0, st>>>(a, coords, n, entry);
    return hipGetLastError();
}

hipError_t launch_alloc(const FuseArgs &a, hipStream_t st)
{
    launch_k(k_alloc, xcd_grid(((a.fg.W + 15) / 16) * ((a.fg.H + 15) / 16)), 256, st, a);
    return hipGetLastError();
}

template <int FMT>
void launch_integrate_fmt(const FuseArgs &a, int grid, hipStream_t st)
{
    const bool clr = a.clr && a.rgbx, ord = a.rb.order != nullptr;
    if (clr && ord) launch_k(k_integrate<FMT, true, true>, grid, 256, st, a);
    else if (clr) launch_k(k_integrate<FMT, true, false>, grid, 256, st, a);
    else if (ord) launch_k(k_integrate<FMT, false, true>, grid, 256, st, a);
    else launch_k(k_integrate<FMT, false, false>, grid, 256, st, a);
}

hipError_t launch_integrate(int fmt, const FuseArgs &a, int grid, hipStream_t st)
{
    switch (fmt) {
    case ITM_VOX_F32: launch_integrate_fmt<ITM_VOX_F32>(a, grid, st); break;
    case ITM_VOX_F16: launch_integrate_fmt<ITM_VOX_F16>(a, grid, st); break;
    default: launch_integrate_fmt<ITM_VOX_S16U8>(a, grid, st); break;
    }
    return hipGetLastError();
}

}  // namespace itm
