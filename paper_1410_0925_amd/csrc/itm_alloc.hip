// Scene initialisation (empty hash table, zero counters, fresh voxels) and the
// export gather.  The allocation itself is device code in itm_alloc.hpp, run by
// the fused per-frame kernel of itm_integrate.hip.
#include <algorithm>

#include "itm_internal.hpp"

namespace itm {

// ---------------------------------------------------------------------------
// initialisation: empty hash entries, zero flags and counters, fresh voxels
// (F = 1, W = 0 -- the paper's initial voxel value)
// ---------------------------------------------------------------------------
template <int FMT>
__global__ void k_init_vba(typename Vox<FMT>::S *sdf, typename Vox<FMT>::Wt *w, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const auto one = Vox<FMT>::from_f(1.0f);
    const auto zero = Vox<FMT>::w_from_f(0.0f);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        sdf[i] = one;
        w[i] = zero;
    }
}

__global__ void k_init_hash(Bucket *b, int32_t *head, int64_t nb, Excess *x, int64_t nx, uint32_t *stamp,
                            int64_t nstamp, unsigned long long *set, int64_t nset, uint32_t *occ, int64_t nocc,
                            Counters *cnt)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t0; i < nb; i += stride) {
        b[i].key[0] = b[i].key[1] = 0ull;
        head[i] = -1;
    }
    for (int64_t i = t0; i < nx; i += stride) {
        x[i].key = 0ull;
        x[i].next = -1;
        x[i].pad = 0;
    }
    for (int64_t i = t0; i < nstamp; i += stride) stamp[i] = 0u;
    for (int64_t i = t0; i < nset; i += stride) set[i] = 0ull;
    for (int64_t i = t0; i < nocc; i += stride) occ[i] = 0u;
    if (t0 == 0) {
        Counters z = {};
        *cnt = z;
    }
}

// export: the voxels of the listed blocks, packed in list order
template <int FMT>
__global__ __launch_bounds__(256) void k_export_gather(const typename Vox<FMT>::S *sdf,
                                                       const typename Vox<FMT>::Wt *w, const int32_t *blocks,
                                                       int64_t n, typename Vox<FMT>::S *out_sdf,
                                                       typename Vox<FMT>::Wt *out_w)
{
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int64_t src = (int64_t)blocks[i] * kBlockVox, dst = i * kBlockVox;
        for (int l = threadIdx.x; l < kBlockVox; l += blockDim.x) {
            if (out_sdf) out_sdf[dst + l] = sdf[src + l];
            if (out_w) out_w[dst + l] = w[src + l];
        }
    }
}

hipError_t launch_export_gather(int fmt, const void *sdf, const void *w, const int32_t *blocks, int64_t n,
                                void *out_sdf, void *out_w, hipStream_t st)
{
    const int grid = (int)std::min<int64_t>(std::max<int64_t>(n, 1), 4096);
    switch (fmt) {
    case ITM_VOX_F32:
        k_export_gather<ITM_VOX_F32><<<grid, 256, 0, st>>>((const float *)sdf, (const float *)w, blocks, n,
                                                            (float *)out_sdf, (float *)out_w);
        break;
    case ITM_VOX_F16:
        k_export_gather<ITM_VOX_F16><<<grid, 256, 0, st>>>((const __half *)sdf, (const __half *)w, blocks, n,
                                                            (__half *)out_sdf, (__half *)out_w);
        break;
    default:
        k_export_gather<ITM_VOX_S16U8><<<grid, 256, 0, st>>>((const int16_t *)sdf, (const uint8_t *)w, blocks,
                                                              n, (int16_t *)out_sdf, (uint8_t *)out_w);
        break;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// blocks in key order
// ---------------------------------------------------------------------------

// a block key as an integer whose order is that of (x, y, z)
__device__ __forceinline__ unsigned long long sort_key(unsigned long long k)
{
    return ((k & 0xffffull) ^ 0x8000ull) << 32 | ((k >> 16 & 0xffffull) ^ 0x8000ull) << 16 |
           ((k >> 32 & 0xffffull) ^ 0x8000ull);
}
__device__ __forceinline__ void sort_coords(unsigned long long k, int32_t *c)
{
    c[0] = (int32_t)(k >> 32 & 0xffffull) - 32768;
    c[1] = (int32_t)(k >> 16 & 0xffffull) - 32768;
    c[2] = (int32_t)(k & 0xffffull) - 32768;
}

// every key of the table with its entry, in any order: a thread takes 4 buckets
// (8 keys) or 4 excess entries, a wave reserves its keys' places with one atomic.
// Bound by reading the table (18 MiB at 2^20 buckets, 5 us at the copy rate).
__global__ __launch_bounds__(256) void k_collect(HashView h, int32_t n, unsigned long long *key, int32_t *ent,
                                                 int32_t *count)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nb = h.n_buckets, n_slots = nb + h.n_excess;   // buckets, then excess entries
    for (int64_t base = (int64_t)blockIdx.x * 1024; base < n_slots; base += (int64_t)gridDim.x * 1024) {   // uniform
        unsigned long long k[8];
        int32_t e[8];
        int c = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int64_t i = base + 256 * j + threadIdx.x;
            ulonglong2 k2 = make_ulonglong2(0ull, 0ull);
            if (i < nb) k2 = *reinterpret_cast<const ulonglong2 *>(h.buckets[i].key);
            else if (i < n_slots) k2.x = h.excess[i - nb].key;
            k[2 * j] = k2.x;
            k[2 * j + 1] = k2.y;
            e[2 * j] = (int32_t)(i < nb ? 2 * i : nb + i);   // excess x: 2 nb + x, i = nb + x
            e[2 * j + 1] = e[2 * j] + 1;
        }
#pragma unroll
        for (int j = 0; j < 8; j++) c += (k[j] & kKeyValid) ? 1 : 0;
        int incl = c;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += y;
        }
        const int total = __shfl(incl, kWave - 1, kWave);
        int at = 0;
        if (total && lane == 0) at = atomicAdd(count, total);
        at = __shfl(at, 0, kWave) + incl - c;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            if (!(k[j] & kKeyValid)) continue;
            if (at < n) {
                key[at] = sort_key(k[j]);
                ent[at] = e[j];
            }
            at++;
        }
    }
}

// keys of the given coordinates (all within 16 bits), their positions as entries
__global__ __launch_bounds__(256) void k_coord_keys(const int32_t *coords, int32_t n, unsigned long long *key,
                                                    int32_t *ent)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    key[i] = sort_key(pack_key(coords[3 * i], coords[3 * i + 1], coords[3 * i + 2]));
    ent[i] = i;
}

// sort each tile of kSortTile keys (with their entries) in LDS: a bitonic network,
// the last tile padded with keys above all to a power of two (a few keys take 3 us,
// all 4096 places 25)
__global__ __launch_bounds__(1024) void k_sort_tiles(unsigned long long *key, int32_t *ent, int32_t n)
{
    __shared__ unsigned long long s_k[kSortTile];
    __shared__ int32_t s_e[kSortTile];
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    const int m = (int)min(n - base, (int64_t)kSortTile), size = m < 2 ? 1 : 2 << (31 - __clz(m - 1));
    for (int i = threadIdx.x; i < size; i += 1024) {
        const bool in = base + i < n;
        s_k[i] = in ? key[base + i] : ~0ull;
        s_e[i] = in ? ent[base + i] : -1;
    }
    for (int k = 2; k <= size; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < size / 2; i += 1024) {
                const int a = ((i & ~(j - 1)) << 1) | (i & (j - 1)), b = a | j;
                const unsigned long long ka = s_k[a], kb = s_k[b];
                if ((ka > kb) == ((a & k) == 0)) {
                    const int32_t ea = s_e[a];
                    s_k[a] = kb;
                    s_k[b] = ka;
                    s_e[a] = s_e[b];
                    s_e[b] = ea;
                }
            }
        }
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += 1024) {
        key[base + i] = s_k[i];
        ent[base + i] = s_e[i];
    }
}

// Merge the sorted runs of `run` keys pairwise: a key's place in the merged run is
// its place in its own plus the sibling's keys before it, by binary search (equal
// keys: the left run's first, so every place is taken once).
__global__ __launch_bounds__(256) void k_merge_runs(const unsigned long long *key, const int32_t *ent, int32_t n,
                                                    int64_t run, unsigned long long *out_key, int32_t *out_ent)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const unsigned long long k = key[i];
    const int64_t r = i / run;
    const bool left = !(r & 1);
    const int64_t start = min((r ^ 1) * run, (int64_t)n), end = min(start + run, (int64_t)n);
    int64_t lo = start, hi = end;
    while (lo < hi) {
        const int64_t m = (lo + hi) >> 1;
        const unsigned long long v = key[m];
        const bool before = left ? v < k : v <= k;
        lo = before ? m + 1 : lo;
        hi = before ? hi : m;
    }
    const int64_t at = (r & ~int64_t(1)) * run + (i - r * run) + (lo - start);
    out_key[at] = k;
    out_ent[at] = ent[i];
}

// what a caller wants of the sorted keys: entries and coordinates, or whether two
// neighbours are equal
__global__ __launch_bounds__(256) void k_sorted_out(const unsigned long long *key, const int32_t *ent, int32_t n,
                                                    int32_t *out_ent, int32_t *coords, int32_t *dup)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const unsigned long long k = key[i];
    if (dup && i > 0 && key[i - 1] == k) *dup = 1;
    if (out_ent) {
        out_ent[i] = ent[i];
        sort_coords(k, coords + 3 * (int64_t)i);
    }
}

// Sort the n keys of (b.key, b.ent) and hand them out.  Tiles in LDS, then merges:
// log2(n / 4096) passes of about as many dependent reads as a run has halvings (32768
// blocks: 3 passes, under 10 us each; the host's sort of them took 2.5 ms, after
// copying and scanning the table for 6).
static hipError_t sort_and_output(int32_t n, const SortedBlocks &b, int32_t *out_ent, int32_t *coords, int32_t *dup,
                                  hipStream_t st)
{
    const int grid = (n + 255) / 256;
    k_sort_tiles<<<(n + kSortTile - 1) / kSortTile, 1024, 0, st>>>(b.key, b.ent, n);
    unsigned long long *k0 = b.key, *k1 = b.key2;
    int32_t *e0 = b.ent, *e1 = b.ent2;
    for (int64_t run = kSortTile; run < n; run *= 2) {
        k_merge_runs<<<grid, 256, 0, st>>>(k0, e0, n, run, k1, e1);
        std::swap(k0, k1);
        std::swap(e0, e1);
    }
    k_sorted_out<<<grid, 256, 0, st>>>(k0, e0, n, out_ent, coords, dup);
    return hipGetLastError();
}

hipError_t launch_sort_blocks(const HashView &h, int32_t n, const SortedBlocks &b, hipStream_t st)
{
    if (hipError_t e = launch_range_clear(b.count, 1, st); e != hipSuccess) return e;
    const int64_t slots = (int64_t)h.n_buckets + h.n_excess;
    k_collect<<<(int)std::min<int64_t>((slots + 1023) / 1024, 2048), 256, 0, st>>>(h, n, b.key, b.ent, b.count);
    return sort_and_output(n, b, b.out_ent, b.coords, nullptr, st);
}

hipError_t launch_find_repeats(const int32_t *coords, int32_t n, const SortedBlocks &b, int32_t *dup, hipStream_t st)
{
    if (hipError_t e = launch_range_clear(dup, 1, st); e != hipSuccess) return e;
    k_coord_keys<<<(n + 255) / 256, 256, 0, st>>>(coords, n, b.key, b.ent);
    return sort_and_output(n, b, nullptr, nullptr, dup, st);
}

// export: the voxels of the listed blocks as floats, in list order; one workgroup
// per block, its first half F, its second W, 4 voxels a thread (one 16-byte store)
template <int FMT>
__global__ __launch_bounds__(256) void k_export_floats(const typename Vox<FMT>::S *sdf,
                                                       const typename Vox<FMT>::Wt *w, const int32_t *blocks,
                                                       int64_t n, float *out_sdf, float *out_w)
{
    const int l = 4 * (threadIdx.x & 127);
    const bool W = threadIdx.x >= 128;   // uniform over a wave
    if (!(W ? out_w : out_sdf)) return;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int64_t src = (int64_t)blocks[i] * kBlockVox + l, dst = i * kBlockVox + l;
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = W ? Vox<FMT>::w_to_f(w[src + j]) : Vox<FMT>::export_f(sdf[src + j]);
        *reinterpret_cast<float4 *>((W ? out_w : out_sdf) + dst) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

hipError_t launch_export_floats(int fmt, const void *sdf, const void *w, const int32_t *blocks, int64_t n,
                                float *out_sdf, float *out_w, hipStream_t st)
{
    const int grid = (int)std::min<int64_t>(std::max<int64_t>(n, 1), 8192);
    switch (fmt) {
    case ITM_VOX_F32:
        k_export_floats<ITM_VOX_F32><<<grid, 256, 0, st>>>((const float *)sdf, (const float *)w, blocks, n, out_sdf,
                                                            out_w);
        break;
    case ITM_VOX_F16:
        k_export_floats<ITM_VOX_F16><<<grid, 256, 0, st>>>((const __half *)sdf, (const __half *)w, blocks, n,
                                                            out_sdf, out_w);
        break;
    default:
        k_export_floats<ITM_VOX_S16U8><<<grid, 256, 0, st>>>((const int16_t *)sdf, (const uint8_t *)w, blocks, n,
                                                              out_sdf, out_w);
        break;
    }
    return hipGetLastError();
}

// import: the first voxel that is no valid state (F in [-1, 1], W an integer in
// [0, max_w]; NaN is none)
__global__ __launch_bounds__(256) void k_import_check(const float4 *sdf, const float4 *w, int64_t n4, int64_t base,
                                                      float max_w, unsigned long long *first)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
        const float4 f = sdf[i], v = w[i];
        const float F[4] = {f.x, f.y, f.z, f.w}, W[4] = {v.x, v.y, v.z, v.w};
        int bad = -1;
#pragma unroll
        for (int j = 3; j >= 0; j--)
            if (!(F[j] >= -1.0f && F[j] <= 1.0f) || !(W[j] >= 0.0f && W[j] <= max_w) || W[j] != floorf(W[j])) bad = j;
        if (bad >= 0) atomicMin(first, (unsigned long long)(base + 4 * i + bad));
    }
}

hipError_t launch_import_check(const float *sdf, const float *w, int64_t n, int64_t base, float max_w,
                               unsigned long long *first, hipStream_t st)
{
    const int64_t n4 = n / 4;
    k_import_check<<<(int)std::min<int64_t>((n4 + 255) / 256, 4096), 256, 0, st>>>(
        (const float4 *)sdf, (const float4 *)w, n4, base, max_w, first);
    return hipGetLastError();
}

// import: the given blocks' voxels (float32 F and W, export layout) into their
// voxel blocks, converted to the storage form; one workgroup per block
template <int FMT>
__global__ __launch_bounds__(256) void k_import_voxels(const int32_t *entry, const float *in_sdf, const float *in_w,
                                                       int64_t n, typename Vox<FMT>::S *sdf,
                                                       typename Vox<FMT>::Wt *w, uchar4 *clr)
{
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int32_t e = entry[i];
        if (e < 0) continue;   // dropped
        const int64_t dst = (int64_t)e * kBlockVox, src = i * kBlockVox;
        for (int l = threadIdx.x; l < kBlockVox; l += blockDim.x) {
            sdf[dst + l] = Vox<FMT>::from_f(in_sdf[src + l]);
            w[dst + l] = Vox<FMT>::w_from_f(in_w[src + l]);
            if (clr) clr[dst + l] = make_uchar4(0, 0, 0, 0);
        }
    }
}

hipError_t launch_import_voxels(int fmt, const int32_t *entry, const float *in_sdf, const float *in_w, int64_t n,
                                void *sdf, void *w, uchar4 *clr, hipStream_t st)
{
    const int grid = (int)std::min<int64_t>(std::max<int64_t>(n, 1), 4096);
    switch (fmt) {
    case ITM_VOX_F32:
        k_import_voxels<ITM_VOX_F32><<<grid, 256, 0, st>>>(entry, in_sdf, in_w, n, (float *)sdf, (float *)w, clr);
        break;
    case ITM_VOX_F16:
        k_import_voxels<ITM_VOX_F16><<<grid, 256, 0, st>>>(entry, in_sdf, in_w, n, (__half *)sdf, (__half *)w, clr);
        break;
    default:
        k_import_voxels<ITM_VOX_S16U8><<<grid, 256, 0, st>>>(entry, in_sdf, in_w, n, (int16_t *)sdf, (uint8_t *)w,
                                                              clr);
        break;
    }
    return hipGetLastError();
}

// export of colour voxels: the listed blocks' 512 x 4 bytes, packed in list order
__global__ __launch_bounds__(256) void k_export_colour(const uchar4 *clr, const int32_t *blocks, int64_t n,
                                                       uchar4 *out)
{
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int64_t src = (int64_t)blocks[i] * kBlockVox, dst = i * kBlockVox;
        for (int l = threadIdx.x; l < kBlockVox; l += blockDim.x) out[dst + l] = clr[src + l];
    }
}

hipError_t launch_export_colour(const uchar4 *clr, const int32_t *blocks, int64_t n, uchar4 *out, hipStream_t st)
{
    const int grid = (int)std::min<int64_t>(std::max<int64_t>(n, 1), 4096);
    k_export_colour<<<grid, 256, 0, st>>>(clr, blocks, n, out);
    return hipGetLastError();
}

hipError_t launch_init(Bucket *b, int32_t *head, int64_t nb, Excess *x, int64_t nx, uint32_t *stamp,
                       int64_t nstamp, unsigned long long *set, int64_t nset, uint32_t *occ, int64_t nocc,
                       Counters *cnt, int fmt, void *sdf, void *w, int64_t n_vox, hipStream_t st)
{
    k_init_hash<<<2048, 256, 0, st>>>(b, head, nb, x, nx, stamp, nstamp, set, nset, occ, nocc, cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    switch (fmt) {
    case ITM_VOX_F32:
        k_init_vba<ITM_VOX_F32><<<8192, 256, 0, st>>>((float *)sdf, (float *)w, n_vox);
        break;
    case ITM_VOX_F16:
        k_init_vba<ITM_VOX_F16><<<8192, 256, 0, st>>>((__half *)sdf, (__half *)w, n_vox);
        break;
    default:
        k_init_vba<ITM_VOX_S16U8><<<8192, 256, 0, st>>>((int16_t *)sdf, (uint8_t *)w, n_vox);
        break;
    }
    return hipGetLastError();
}

}  // namespace itm
