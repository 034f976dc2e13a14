// Swapping (section "Swapping"): the device keeps a pool of voxel blocks
// smaller than the map; blocks that leave the view move to the host, and a host
// copy comes back into the device block a block takes when it is visible again,
// merged with what the device fused into it meanwhile (the secondary
// integration).  The blocks that move are chosen here (fixed transfer sizes, in
// key order); the host reads how many, sees to the memory of their host copies,
// and the voxels move between the pool and those copies directly.
#include <algorithm>

#include "itm_internal.hpp"

namespace itm {

constexpr int kSwapThreads = 1024;   // of the scan and of the choice
constexpr int kSwapDigit = 12;       // bits of a key that one pass of the choice settles

// the key as one number in the order (x, y, z)
__device__ __forceinline__ unsigned long long order_key(unsigned long long key)
{
    const uint32_t x = (uint32_t)key & 0xffffu, y = (uint32_t)(key >> 16) & 0xffffu,
                   z = (uint32_t)(key >> 32) & 0xffffu;
    return ((unsigned long long)(x ^ 0x8000u) << 32) | ((y ^ 0x8000u) << 16) | (z ^ 0x8000u);
}

// The candidates of this frame's transfers, four hash entries per thread.
//   swap in:  entries holding a device block and a host copy not yet merged;
//   swap out: entries holding a device block, not listed in this frame (stamp !=
//             stamp_now), with nothing to merge once the swap-ins are done: one with
//             a host copy is in both lists, marked, and leaves only if it merges now.
// Each list gets (order, entry) records.  Thread 0 also resets a pool top that
// the allocation ran below zero, and the grid clears the counts of the choice.
//
// Bound by one pass over 9 B per entry.  Both lists' places are drawn by one
// atomic per workgroup of 4096 entries: drawn per candidate (entries hash, so a
// wave rarely holds two) they queued at one address: 48.5 us, now 10.8, over the
// 1.2 M entries and about 15 k candidates of a VGA frame.
__global__ __launch_bounds__(kSwapThreads) void k_swap_scan(SwapScanArgs a)
{
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    if (blockIdx.x == 0 && t == 0 && *a.pool.top < 0) *a.pool.top = 0;
    for (int i = blockIdx.x * kSwapThreads + t; i < kSwapHistWords; i += gridDim.x * kSwapThreads) a.hist[i] = 0;
    const int64_t e0 = ((int64_t)blockIdx.x * kSwapThreads + t) * 4;
    int32_t b[4] = {-1, -1, -1, -1};
    uint32_t st[4] = {0, 0, 0, 0}, oh = 0;
    if (e0 + 3 < a.n_entries) {
        const int4 bv = *(const int4 *)(a.h.blk + e0);
        const uint4 sv = *(const uint4 *)(a.stamp + e0);
        oh = *(const uint32_t *)(a.onhost + e0);
        b[0] = bv.x, b[1] = bv.y, b[2] = bv.z, b[3] = bv.w;
        st[0] = sv.x, st[1] = sv.y, st[2] = sv.z, st[3] = sv.w;
    } else {
        for (int k = 0; k < 4 && e0 + k < a.n_entries; k++) {
            b[k] = a.h.blk[e0 + k];
            st[k] = a.stamp[e0 + k];
            oh |= (uint32_t)a.onhost[e0 + k] << (8 * k);
        }
    }
    // candidates of this thread: in the low half the swap-ins, in the high the swap-outs
    uint32_t n = 0, np = 0;
    bool in[4], out[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        in[k] = b[k] >= 0 && ((oh >> (8 * k)) & 0xffu);
        out[k] = b[k] >= 0 && st[k] != a.stamp_now;
        n += (uint32_t)in[k] + ((uint32_t)out[k] << 16);
        np += in[k] && out[k];
    }
    // places within the workgroup: at most 4096 of each, so the halves never carry
    uint32_t incl = n;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    __shared__ uint32_t s_wave[kSwapThreads / kWave];
    __shared__ unsigned long long s_base;
    __shared__ uint32_t s_pend;
    if (lane == kWave - 1) s_wave[wave] = incl;
    if (t == 0) s_pend = 0;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kSwapThreads / kWave; w++) {
        before += w < wave ? s_wave[w] : 0;
        all += s_wave[w];
    }
    if (all == 0) return;   // uniform
    if (np) atomicAdd(&s_pend, np);
    if (t == 0)
        s_base = atomicAdd(&a.cnt->cand, (unsigned long long)(all & 0xffffu) | ((unsigned long long)(all >> 16) << 32));
    __syncthreads();
    if (t == 0 && s_pend) atomicAdd(&a.cnt->pend, s_pend);
    const uint32_t place = before + incl - n;
    uint32_t pi = (uint32_t)s_base + (place & 0xffffu), po = (uint32_t)(s_base >> 32) + (place >> 16);
#pragma unroll
    for (int k = 0; k < 4; k++) {
        if (!in[k] && !out[k]) continue;
        SwapRec r;
        r.key = order_key(entry_key(a.h, (int32_t)(e0 + k)));
        r.e = (int32_t)(e0 + k);
        r.pend = in[k] && out[k];
        if (in[k]) a.in_list[pi++] = r;
        if (out[k]) a.out_list[po++] = r;
    }
}

hipError_t launch_swap_scan(const SwapScanArgs &a, hipStream_t st)
{
    const int grid = (int)((a.n_entries + 4 * kSwapThreads - 1) / (4 * kSwapThreads));
    k_swap_scan<<<std::max(grid, 1), kSwapThreads, 0, st>>>(a);
    return hipGetLastError();
}

// One step of the choice: the digit of the cap-th smallest key, given the number
// of smaller keys per digit among those that share its higher digits.
// s.rem: the place (from 1) of that key among them.  Every thread of the
// workgroup calls; the result is uniform.
__device__ __forceinline__ SwapSel next_digit(const uint32_t *hist, SwapSel s, int t)
{
    __shared__ uint32_t s_wave[kSwapThreads / kWave];
    __shared__ SwapSel s_sel;
    const int lane = t & (kWave - 1), wave = t / kWave;
    static_assert(1 << kSwapDigit == 4 * kSwapThreads, "four digits a thread");
    const uint4 c = *(const uint4 *)(hist + 4 * t);
    const uint32_t n = c.x + c.y + c.z + c.w;
    uint32_t incl = n;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t below = incl - n;
    for (int w = 0; w < wave; w++) below += s_wave[w];
    if (below < s.rem && s.rem <= below + n) {   // one thread
        uint32_t d = 0, cs[3] = {c.x, c.y, c.z};
        for (; d < 3 && s.rem > below + cs[d]; d++) below += cs[d];
        s_sel.prefix = (s.prefix << kSwapDigit) | (4 * t + d);
        s_sel.rem = s.rem - below;
    }
    __syncthreads();
    return s_sel;
}

// The choice of the first cap[q] candidates of list q in key order (keys are
// distinct): a radix selection of the cap-th smallest 48-bit key, 12 bits a pass,
// one launch per pass and one more (pass 4) that lists the entries up to that
// key.  A list that fits its transfer is taken whole and the passes return at
// once.  A pass counts the digits of its candidates in LDS and adds the non-empty
// counts to the pass's; every workgroup of the next pass works the digit out of
// them again, which is less than another launch.
// Launch bound: 4.5 us a pass at 15 k candidates, with 8 to 64 workgroups per list
// alike; 64 for long lists.
//
// A block that merges in this frame may leave in it.  Where every in is taken, the
// marked outs all merge.  Where not, those up to the last in's key do: if the outs
// fit their transfer, pass 4 lists them by that key, else they wait for it, and a
// second round of the passes (late) chooses them.  (In a VGA frame of a camera that
// turns, with 2048 + 2048 blocks, one frame in three has marked outs, one in eight a
// second round.)
__global__ __launch_bounds__(kSwapThreads) void k_swap_choose(SwapSelArgs a, int pass, bool late)
{
    const int t = threadIdx.x, q = late ? 1 : blockIdx.y;
    const uint32_t n_in = (uint32_t)a.cnt->cand, pend = a.cnt->pend, cap = (uint32_t)a.cap[q];
    const uint32_t len = q ? (uint32_t)(a.cnt->cand >> 32) : n_in;
    const uint32_t n = late ? len - pend + a.cnt->pend_in : len;   // that may qualify
    const bool some = q && pend > 0 && n_in > (uint32_t)a.cap[0];  // marked outs: not all of them do
    const bool wait = some && !late && n > cap;
    const bool last = pass == kSwapPasses;
    const bool drawn = q && pend > 0 && n > 0 && !wait;            // how many move is known when all are listed
    if (last && blockIdx.x == 0 && t == 0) {
        if (!drawn) {   // read by the host after the launch
            a.moves[q] = wait ? -1 : (int32_t)min(n, cap);
            if (q) a.moves[2] = 0;
        }
        if (!late) {    // the next frame's counts
            if (q) a.cnt_next->out = 0;
            else {
                a.cnt_next->cand = 0;
                a.cnt_next->pend = a.cnt_next->pend_in = a.cnt_next->in = 0;
            }
        }
    }
    if (n == 0 || wait || (!last && n <= cap)) return;
    SwapSel s;
    s.prefix = 0;
    s.rem = cap;
    if (n > cap && pass > 0) {
        if (pass > 1) s = a.sel[q * kSwapPasses + pass - 1];
        s = next_digit(a.hist + ((q * kSwapPasses + pass - 1) << kSwapDigit), s, t);
        // (place 0 of list 0 is free: it takes the finished key)
        if (blockIdx.x == 0 && t == 0 && (!last || q == 0)) a.sel[last ? 0 : q * kSwapPasses + pass] = s;
    }
    // the largest key that merges: marked outs above it do not qualify
    unsigned long long top_in = ~0ull;
    if (some)
        top_in = late ? a.sel[0].prefix
                      : next_digit(a.hist + ((kSwapPasses - 1) << kSwapDigit), a.sel[kSwapPasses - 1], t).prefix;
    const SwapRec *list = a.list[q];
    const uint32_t stride = gridDim.x * kSwapThreads;
    if (last) {
        const unsigned long long top = n > cap ? s.prefix : ~0ull;
        const int lane = t & (kWave - 1);
        const unsigned long long below = (1ull << lane) - 1;
        for (uint32_t i0 = blockIdx.x * kSwapThreads; i0 < len; i0 += stride) {
            const uint32_t i = i0 + t;
            SwapRec r;
            r.key = ~0ull;
            r.e = -1;
            r.pend = 0;
            if (i < len) r = list[i];
            const bool take = i < len && r.key <= top && !(r.pend && r.key > top_in);
            const unsigned long long m = __ballot(take), mp = __ballot(take && r.pend);
            if (m == 0) continue;
            // the wave's lanes draw their places together
            unsigned long long base = 0;
            if (q == 0) {
                if (lane == 0) {
                    base = atomicAdd(&a.cnt->in, (uint32_t)__popcll(m));
                    if (mp) atomicAdd(&a.cnt->pend_in, (uint32_t)__popcll(mp));
                }
                base = __builtin_amdgcn_readfirstlane((uint32_t)base);
                if (take) a.chosen[0][base + __popcll(m & below)] = r.e;
            } else {
                if (lane == 0)
                    base = atomicAdd(&a.cnt->out, (unsigned long long)__popcll(m & ~mp) |
                                                      (unsigned long long)__popcll(mp) << 24);
                base = __shfl(base, 0, kWave);
                if (take && r.pend) a.chosen[2][(base >> 24 & 0xffffff) + __popcll(mp & below)] = r.e;
                else if (take) a.chosen[1][(base & 0xffffff) + __popcll(m & ~mp & below)] = r.e;
            }
        }
        if (drawn) {   // the last workgroup tells the host (one word: no fence between the counts)
            __syncthreads();
            if (t == 0) {
                const unsigned long long o = atomicAdd(&a.cnt->out, 1ull << 48);
                if ((o >> 48) == gridDim.x - 1) {
                    a.moves[1] = (int32_t)(o & 0xffffff);
                    a.moves[2] = (int32_t)(o >> 24 & 0xffffff);
                }
            }
        }
        return;
    }
    __shared__ uint32_t s_cnt[1 << kSwapDigit];
    for (int i = t; i < 1 << kSwapDigit; i += kSwapThreads) s_cnt[i] = 0;
    __syncthreads();
    const int low = kSwapDigit * (kSwapPasses - 1 - pass);
    for (uint32_t i = blockIdx.x * kSwapThreads + t; i < len; i += stride) {
        const SwapRec r = list[i];
        const unsigned long long k = r.key >> low;
        if ((k >> kSwapDigit) == s.prefix && !(r.pend && r.key > top_in))
            atomicAdd(&s_cnt[k & ((1 << kSwapDigit) - 1)], 1u);
    }
    __syncthreads();
    uint32_t *hist = a.hist + ((q * kSwapPasses + pass) << kSwapDigit);
    for (int i = t; i < 1 << kSwapDigit; i += kSwapThreads)
        if (s_cnt[i]) atomicAdd(&hist[i], s_cnt[i]);
}

hipError_t launch_swap_choose(const SwapSelArgs &a, bool late, hipStream_t st)
{
    for (int pass = 0; pass <= kSwapPasses; pass++)
        k_swap_choose<<<dim3(kSwapChooseWgs, late ? 1 : 2), kSwapThreads, 0, st>>>(a, pass, late);
    return hipGetLastError();
}

// The moves, one wave per block, between the pool and the blocks' host copies
// (pinned memory that the device reads and writes directly; F then W), or, where some
// copies are not pinned, xfer.
//   in:  the host copy merges into the entry's device block,
//          W = W_d + W_h; F = (W_d F_d + W_h F_h) / W, W = min(W, max_w)
//        (unchanged when both weights are 0); the copy's slot is free afterwards;
//   out: the device block's voxels go to a host slot, the block is reset (F = 1,
//        W = 0) and returned to the pool, and the entry has its data on the host.
// Slots freed by a launch are used from the next one on, so no wave writes a slot
// that another reads.  Blocks that merge and leave in the same frame are among the
// ins of its first launch and the outs of a second.
//
// Bound by the link to the host.  Ins and outs alternate, so that it carries both
// directions at once; every access to a host copy is 16 B per lane, a wave's
// contiguous (8 B for 8-bit weights).  One workgroup for every other CU keeps it
// full: a copy of 8 + 8 MiB took 210 us with 128 workgroups, 231 with 512, 244 with
// 4096 (and 155 us in one direction alone), 2048 + 2048 blocks in F32 214 us.
// With the lists sorted on the host and the blocks copied through a buffer between
// the device and their slots, a VGA frame with these transfers took 2003 us, now 374.
template <int FMT>
__global__ __launch_bounds__(256) void k_swap_move(SwapMoveArgs a)
{
    using V = Vox<FMT>;
    using S = typename V::S;
    using Wt = typename V::Wt;
    constexpr int kVox = 16 / sizeof(S);            // voxels per lane and access
    constexpr int kAcc = kBlockVox / (kWave * kVox);   // accesses per lane and block
    struct alignas(sizeof(S) * kVox) SV { S v[kVox]; };
    struct alignas(sizeof(Wt) * kVox) WV { Wt v[kVox]; };
    auto *sdf = (S *)a.sdf;
    auto *w = (Wt *)a.w;
    const int lane = threadIdx.x & (kWave - 1);
    const int both = 2 * min(a.n_in, a.n_out), n = a.n_in + a.n_out;
    for (int j = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + threadIdx.x / kWave); j < n; j += gridDim.x * 4) {
        const bool out = j < both ? (j & 1) : a.n_out > a.n_in;
        const int i = j < both ? j >> 1 : j - both / 2;
        const int32_t e = a.chosen[out ? 1 : 0][i];
        const int32_t b = a.h.blk[e];
        int32_t slot;
        if (!out)
            slot = a.slot_of[e];
        else
            slot = i < a.n_free ? a.free_ring[(a.ring_head + i) % a.ring_size] : a.slot_next + (i - a.n_free);
        constexpr size_t kBytes = (sizeof(S) + sizeof(Wt)) * kBlockVox;
        uint8_t *host = a.xfer ? a.xfer + (size_t)i * kBytes
                               : a.chunks[slot / kSwapChunk] + (size_t)(slot % kSwapChunk) * kBytes;
        SV *hs = (SV *)host;
        WV *hw = (WV *)(host + sizeof(S) * kBlockVox);
        SV *ds = (SV *)(sdf + (int64_t)b * kBlockVox);
        WV *dw = (WV *)(w + (int64_t)b * kBlockVox);
        SV vs[kAcc];
        WV vw[kAcc];
#pragma unroll
        for (int k = 0; k < kAcc; k++) {
            vs[k] = ds[lane + kWave * k];
            vw[k] = dw[lane + kWave * k];
        }
        if (out) {
            SV one;
            WV zero;
#pragma unroll
            for (int v = 0; v < kVox; v++) {
                one.v[v] = V::from_f(1.0f);
                zero.v[v] = V::w_from_f(0.0f);
            }
#pragma unroll
            for (int k = 0; k < kAcc; k++) {
                hs[lane + kWave * k] = vs[k];
                hw[lane + kWave * k] = vw[k];
                ds[lane + kWave * k] = one;
                dw[lane + kWave * k] = zero;
            }
            if (lane == 0) {
                a.pool.stack[atomicAdd(a.pool.top, 1)] = b;
                a.h.blk[e] = -1;
                a.onhost[e] = 1;
                a.slot_of[e] = slot;
            }
            continue;
        }
        SV ts[kAcc];
        WV tw[kAcc];
#pragma unroll
        for (int k = 0; k < kAcc; k++) {
            ts[k] = hs[lane + kWave * k];
            tw[k] = hw[lane + kWave * k];
        }
#pragma unroll
        for (int k = 0; k < kAcc; k++) {
#pragma unroll
            for (int v = 0; v < kVox; v++) {
                const float Fd = V::to_f(vs[k].v[v]), Wd = V::w_to_f(vw[k].v[v]);
                const float Fh = V::to_f(ts[k].v[v]), Wh = V::w_to_f(tw[k].v[v]);
                const float Wn = Wd + Wh;
                if (Wn > 0.0f) {
                    vs[k].v[v] = V::from_f((Wd * Fd + Wh * Fh) / Wn);
                    vw[k].v[v] = V::w_from_f(fminf(Wn, a.max_w));
                }
            }
            ds[lane + kWave * k] = vs[k];
            dw[lane + kWave * k] = vw[k];
        }
        if (lane == 0) {
            a.onhost[e] = 0;
            a.free_ring[(a.ring_tail + i) % a.ring_size] = slot;
        }
    }
}

hipError_t launch_swap_move(int fmt, const SwapMoveArgs &a, hipStream_t st)
{
    const int n = a.n_in + a.n_out;
    if (n <= 0) return hipSuccess;
    const int grid = std::min((n + 3) / 4, kSwapMoveWgs);
    switch (fmt) {
    case ITM_VOX_F32: k_swap_move<ITM_VOX_F32><<<grid, 256, 0, st>>>(a); break;
    case ITM_VOX_F16: k_swap_move<ITM_VOX_F16><<<grid, 256, 0, st>>>(a); break;
    default: k_swap_move<ITM_VOX_S16U8><<<grid, 256, 0, st>>>(a); break;
    }
    return hipGetLastError();
}

// pool initialisation: every device block free, no entry holding one
__global__ void k_swap_init(int32_t *stack, int32_t n_blocks, int32_t *top, int32_t *blk, uint8_t *onhost,
                            int64_t n_entries)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t0; i < n_blocks; i += stride) stack[i] = (int32_t)i;
    for (int64_t i = t0; i < n_entries; i += stride) {
        blk[i] = -1;
        onhost[i] = 0;
    }
    if (t0 == 0) *top = n_blocks;
}

hipError_t launch_swap_init(int32_t *stack, int32_t n_blocks, int32_t *top, int32_t *blk, uint8_t *onhost,
                            int64_t n_entries, hipStream_t st)
{
    k_swap_init<<<2048, 256, 0, st>>>(stack, n_blocks, top, blk, onhost, n_entries);
    return hipGetLastError();
}

}  // namespace itm
