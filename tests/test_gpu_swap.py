"""Swapping (section "Swapping") on the GPU through the C ABI against the
oracle's schedule: a device pool smaller than the map, blocks that leave the
view moved to the host in key order up to the transfer size, host copies merged
back into the device blocks new frames fused into (the secondary integration).

Bars: the allocated block set bit-exact; per frame the same numbers of blocks
on the device, on the host only, pending a merge, swapped in and out; the
exported volume (every block wherever it is, merged where both copies exist)
with W bit-exact and |dF| <= 1e-5 against the oracle's states."""
import numpy as np
import pytest

import oracle
from synth import make_stream
from tests.gpu_util import K_of, compare_volumes, gpu

pytestmark = pytest.mark.gpu


def run_both(st, n, pool, swap_in, swap_out, fmt="f32", ray_frames=()):
    itm, torch = gpu()
    g = itm.Scene.from_params(st.params, fmt=fmt)
    g.enable_swapping(pool, swap_in, swap_out)
    o = oracle.Scene.from_params(st.params)
    o.enable_swapping(pool, swap_in, swap_out)
    depth = torch.from_numpy(np.ascontiguousarray(st.depth[:n])).cuda()
    K = K_of(st)
    rays = {}
    for f in range(n):
        g.integrate(depth[f], K, st.T_wc[f])
        o.integrate(st.depth[f], st.intrinsics, st.T_wc[f])
        gs, os_ = g.swap_stats(), o.swap_stats()
        assert gs == os_, (f, gs, os_)
        if f in ray_frames:
            p, q = g.raycast(K, st.T_wc[f])
            rays[f] = (p.cpu().numpy(), q.cpu().numpy(),
                       o.raycast(st.width, st.height, st.intrinsics, st.T_wc[f], alternatives=True))
    torch.cuda.synchronize()
    return g, o, rays


def test_vga_pool_smaller_than_the_map():
    st = make_stream("vga", n_frames=60)
    print("case: swapping vga 60 frames, pool 12000 blocks", flush=True)
    g, o, rays = run_both(st, 60, 12000, 2000, 4000, ray_frames=(59,))
    n_alloc = g.stats()["n_allocated"]
    s = g.swap_stats()
    print(f"allocated {n_alloc}, {s}", flush=True)
    assert n_alloc > 12000 and s["n_host_only"] > 0 and s["swapped_in_total"] > 0
    assert s["no_block_total"] == 0
    compare_volumes(g.export(), o.export(), cands=o.export_candidates())
    # the raycast sees the blocks on the device only, like the oracle's
    from tests.gpu_util import compare_raycast_exact
    P, N, orr = rays[59]
    # the two volumes' device copies may differ where a voxel took another correct
    # state, so the raycast is compared end to end (fractions)
    from tests.gpu_util import compare_raycast
    print(compare_raycast((P, N), orr[:5], st.T_wc[59]))
    g.close()


def test_small_transfers_in_every_form():
    st = make_stream("vga", n_frames=40)
    for fmt in ("f32", "s16u8"):
        print(f"case: swapping vga 40 frames, {fmt}, transfers of 64 blocks", flush=True)
        g, o, _ = run_both(st, 40, 40000, 64, 64, fmt=fmt)
        tol = 1e-5 if fmt == "f32" else (lambda W: (0.5 / 32767 + 4 * 2.0 ** -23) * (np.asarray(W, np.float64) + 1) + 1e-6)
        compare_volumes(g.export(), o.export(), tol=tol, cands=o.export_candidates())
        g.close()


def test_swapping_arguments():
    itm, torch = gpu()
    st = make_stream("tiny", n_frames=1)
    sc = itm.Scene.from_params(st.params)
    with pytest.raises(itm.ItmError):
        sc.enable_swapping(0, 8, 8)
    with pytest.raises(itm.ItmError):
        sc.enable_swapping(1000, 0, 8)
    sc.integrate(torch.from_numpy(st.depth[0]).cuda(), K_of(st), st.T_wc[0])
    with pytest.raises(itm.ItmError):     # after the first frame
        sc.enable_swapping(1000, 8, 8)
    with pytest.raises(itm.ItmError):
        sc.swap_stats()
    sc2 = itm.Scene.from_params(st.params)
    sc2.enable_swapping(4096, 64, 64)
    with pytest.raises(itm.ItmError):
        sc2.enable_colour()
    with pytest.raises(itm.ItmError):
        sc2.import_blocks(np.zeros((1, 3), np.int32), np.ones((1, 512), np.float32), np.zeros((1, 512), np.float32))


def test_device_pool_without_transfers():
    """Transfer sizes 0: the voxel block array is a pool of the given size
    instead of one block per hash entry; with room for the map the volume is the
    plain one."""
    itm, torch = gpu()
    st = make_stream("vga", n_frames=30)
    print("case: vga 30 frames, a pool of 20000 blocks, no transfers", flush=True)
    g = itm.Scene.from_params(st.params)
    g.enable_swapping(20000, 0, 0)
    depth = torch.from_numpy(np.ascontiguousarray(st.depth[:30])).cuda()
    for f in range(30):
        g.integrate(depth[f], K_of(st), st.T_wc[f])
    torch.cuda.synchronize()
    s = g.swap_stats()
    assert s["no_block_total"] == 0 and s["swapped_out_total"] == 0 and s["n_host_only"] == 0
    assert g.stats()["vba_capacity"] == 20000 < g.stats()["n_entries"]
    o = oracle.Scene.from_params(st.params)
    for f in range(30):
        o.integrate(st.depth[f], st.intrinsics, st.T_wc[f])
    compare_volumes(g.export(), o.export(), cands=o.export_candidates())
    g.close()


@pytest.mark.parametrize("fmt,swap_in,swap_out", [("f32", 1, 1), ("f16", 33, 1 << 20), ("f16", 500, 37),
                                                  ("s16u8", 500, 43)])
def test_the_choice_at_its_edges(fmt, swap_in, swap_out):
    """The blocks that move, over transfers of one block, of exactly as many
    blocks as there are candidates, of fewer and of more (so that either list is
    taken whole or chosen from), with a number of entries that is no multiple of
    a thread's four: the numbers moved are the oracle's in every frame, and the
    volume is its volume.  Bars as above; half precision rounds F at every fusion
    and merge, by 2^-11 relative at most."""
    itm, torch = gpu()
    st = make_stream("tiny", n_frames=40)
    st.params = dict(st.params, n_excess=st.params["n_excess"] + 1)
    print(f"case: tiny 40 frames, {fmt}, transfers of {swap_in} and {swap_out} blocks", flush=True)
    g, o, _ = run_both(st, 40, 4096, swap_in, swap_out, fmt=fmt)
    s = g.swap_stats()
    assert s["swapped_in_total"] > 0 and s["swapped_out_total"] > 0
    tol = {"f32": 1e-5, "f16": lambda W: 2.0 ** -11 * (np.asarray(W, np.float64) + 1) + 1e-5,
           "s16u8": lambda W: (0.5 / 32767 + 4 * 2.0 ** -23) * (np.asarray(W, np.float64) + 1) + 1e-6}[fmt]
    compare_volumes(g.export(), o.export(), tol=tol, cands=o.export_candidates())
    g.close()


@pytest.mark.parametrize("fmt,swap_in,swap_out,stride", [("s16u8", 2, 43, 1), ("f32", 5, 9, 1), ("f32", 2, 3, 13),
                                                         ("f16", 2, 43, 13), ("f32", 20, 30, 13), ("s16u8", 60, 70, 13)])
def test_blocks_that_merge_and_leave_in_one_frame(fmt, swap_in, swap_out, stride):
    """Transfers smaller than what is pending, over a camera that jumps about: a host copy
    that waited until its block was out of view merges and, with nothing left to merge,
    may leave in the same frame -- with every pending copy merged in it or only some,
    with room in the transfer or not.  Numbers moved per frame and volume as above."""
    itm, torch = gpu()
    st = make_stream("tiny", n_frames=40 if stride == 1 else 60)
    order = [(stride * k) % st.n_frames for k in range(40)]
    st.depth, st.T_wc = st.depth[order], st.T_wc[order]
    print(f"case: tiny, every {stride}th frame, {fmt}, transfers of {swap_in} and {swap_out} blocks", flush=True)
    g, o, _ = run_both(st, 40, 4096, swap_in, swap_out, fmt=fmt)
    tol = {"f32": 1e-5, "f16": lambda W: 2.0 ** -11 * (np.asarray(W, np.float64) + 1) + 1e-5,
           "s16u8": lambda W: (0.5 / 32767 + 4 * 2.0 ** -23) * (np.asarray(W, np.float64) + 1) + 1e-6}[fmt]
    compare_volumes(g.export(), o.export(), tol=tol, cands=o.export_candidates())
    g.close()


def test_slots_go_round():
    """More blocks swapped in than the table has entries, so that the ring of free host
    slots starts over: numbers moved per frame and volume as above."""
    itm, torch = gpu()
    st = make_stream("tiny", n_frames=60)
    order = [(13 * k) % 60 for k in range(60)]
    st.depth, st.T_wc = st.depth[order], st.T_wc[order]
    st.params = dict(voxel_size=0.025, mu=0.1, max_w=100, n_buckets=2 ** 8, n_excess=131)
    print("case: tiny, 643 entries, transfers of 40 and 60 blocks", flush=True)
    g, o, _ = run_both(st, 60, 500, 40, 60)
    s = g.stats()
    assert s["n_entries"] == 643 and g.swap_stats()["swapped_in_total"] > 643
    assert o.stats()["n_dropped_total"] == 0
    compare_volumes(g.export(), o.export(), cands=o.export_candidates())
    g.close()
