"""What the library does where memory or a transfer is refused, and which kernel a rule
picks.  The refusals are made, and the launches counted, on the host, by limited_hip.c
in front of the HIP runtime, in one process of their own (this file, run as a program);
every kernel runs to its normal end."""
import ctypes as C
import json
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.gpu


def _swapping(itm, torch, st, frames, each=None, fmt="f32", pool=40000, swap_in=500, swap_out=300, stride=1):
    """st's frames (every stride-th, around) fused with swapping; each(scene, f) before
    frame f.  The exported map, the numbers moved and the frames that failed."""
    K = tuple(st.intrinsics) + (st.width, st.height)
    sc = itm.Scene.from_params(st.params, fmt=fmt)
    sc.enable_swapping(pool, swap_in, swap_out)
    stats, failed = [], []
    for f in range(frames):
        if each:
            each(sc, f)
        try:
            k = stride * f % st.n_frames
            sc.integrate(torch.from_numpy(st.depth[k]).cuda(), K, st.T_wc[k])
        except itm.ItmError as e:
            failed.append((f, str(e)))
        stats.append(sc.swap_stats())
    out = sc.export()
    sc.close()
    return out, stats, failed


def _same(a, b):
    return all(np.array_equal(x.view(np.uint32), y.view(np.uint32)) for x, y in zip(a, b))


def pointers_not_sent(itm, torch, hip, st):
    """The host copies' second memory (from 2049 copies on) is there, but its pointer does
    not reach the device in one frame: that frame moves nothing and says so, and the
    next one sends the pointer before any block goes there."""
    at = [None]

    def each(sc, f):
        if at[0] is None and sc.swap_stats()["n_host_only"] + 300 > 2048:
            at[0] = f
            hip.fail_copies(8, 1)      # the pointer is the only copy of 8 bytes
    (_, _, _), stats, failed = got = _swapping(itm, torch, st, 20, each)
    assert at[0] is not None and hip.refusals() == 1
    assert len(failed) == 1 and failed[0][0] == at[0], failed
    f = failed[0][0]
    s = stats[f]
    assert s["swapped_in_last"] == s["swapped_out_last"] == 0
    assert s["swapped_out_total"] == stats[f - 1]["swapped_out_total"]
    assert stats[f + 1]["n_host_only"] > 2048
    # a frame without moves only delays them: the map holds the same blocks and, once
    # merged, every sample (the averages are joined in another order)
    c, F, W = _swapping(itm, torch, st, 20)[0]
    assert np.array_equal(got[0][0], c) and np.array_equal(got[0][2], W)
    assert np.abs(got[0][1] - F).max() < 1e-5


def _pageable(itm, torch, hip, st, pinned, fmt, swap_in, swap_out):
    args = dict(fmt=fmt, swap_in=swap_in, swap_out=swap_out, stride=13)
    want, stats, _ = _swapping(itm, torch, st, 30, **args)
    assert max(s["n_host_only"] for s in stats) > 4096 and stats[-1]["swapped_in_total"] > 2048
    hip.limit_host(1 << 20, pinned)
    got, same, failed = _swapping(itm, torch, st, 30, **args)
    assert hip.refusals() == 1 and not failed      # it does not ask again
    assert same == stats and _same(got, want)


def pageable_after_one(itm, torch, hip, st):
    """With pinned memory for 2048 host copies the others take pageable memory: the same
    blocks move, in batches of 2048 and the rest, and the map is the same bits."""
    _pageable(itm, torch, hip, st, 1, "f32", 4000, 5000)


def pageable_after_two(itm, torch, hip, st):
    """As above for 4096 copies, in the 3-byte form and with blocks that merge and leave
    in one frame."""
    _pageable(itm, torch, hip, st, 2, "s16u8", 250, 3000)


def no_copies_at_all(itm, torch, hip, st):
    """Without any pinned memory a frame that has blocks to move out fuses, moves
    nothing and says so; once there is memory the blocks move."""
    def each(sc, f):
        if f in (0, 10):
            hip.limit_host(1 << 20 if f == 0 else 2 ** 63, 0)
    (c, F, W), stats, failed = _swapping(itm, torch, st, 20, each)
    assert failed and failed[-1][0] == 9 and all("host copies" in e for _, e in failed)
    assert all(s["swapped_out_total"] == s["swapped_in_total"] == s["n_host_only"] == 0 for s in stats[:10])
    assert stats[10]["swapped_out_last"] == 300
    want = _swapping(itm, torch, st, 20)[0]
    assert np.array_equal(c, want[0]) and np.array_equal(W, want[2]) and np.abs(F - want[1]).max() < 1e-5


def _map(n):
    rng = np.random.default_rng(n)
    c = np.unique(rng.integers(-60, 60, (2 * n, 3)), axis=0)
    c = c[rng.permutation(len(c))[:n]].astype(np.int32)
    F = (rng.integers(-32767, 32768, (n, 512)) / 32767).astype(np.float32)
    return c, F, rng.integers(0, 101, (n, 512)).astype(np.float32)


def _in_and_out(itm, n, limits):
    """A map of n blocks imported and exported, each call under limits(): refused as ever
    where it has to be, and the same map."""
    c, F, W = _map(n)
    at = np.lexsort((c[:, 2], c[:, 1], c[:, 0]))
    sc = itm.Scene(0.005, 0.02, 100, 1 << 15, 1 << 13)
    sc.enable_colour()
    for change, match in (((c[n - 1], c[0]), "twice"), ((F, 7 * 512 + 3), f"voxel {7 * 512 + 3}: F"),
                          ((W, n * 512 - 1), f"voxel {n * 512 - 1}: W")):
        a, b = change
        if match == "twice":
            old = a.copy()
            a[:] = b
        else:
            old = a.reshape(-1)[b]
            a.reshape(-1)[b] = -1.5
        limits()
        try:
            sc.import_blocks(c, F, W)
            raise AssertionError(match)
        except itm.ItmError as e:
            assert match in str(e), e
        if match == "twice":
            a[:] = old
        else:
            a.reshape(-1)[b] = old
    assert sc.stats()["n_allocated"] == 0
    limits()
    sc.import_blocks(c, F, W)
    limits()
    got = sc.export()
    limits()
    only = sc.export(values=False)[0]
    limits()
    rgbw = sc.export_colour()
    sc.close()
    assert np.array_equal(got[0], c[at]) and np.array_equal(only, c[at])
    assert np.array_equal(got[1], F[at]) and np.array_equal(got[2], W[at])
    assert rgbw.shape == (n, 512, 4) and not rgbw.any()


def device_memory_for_one(itm, torch, hip, st):
    """Device memory for one list, or one larger allocation, a call: the lists, which a
    call cannot do without, come before what only makes it faster."""
    _in_and_out(itm, 16389, lambda: hip.limit_device(40 * 16389, 1))
    assert hip.refusals() > 0


def no_device_memory(itm, torch, hip, st):
    """No device memory at all beside the scene's: lists, voxels and staging are pinned."""
    _in_and_out(itm, 5000, lambda: hip.limit_device(0, 0))
    assert hip.refusals() > 0


def no_staging(itm, torch, hip, st):
    """No pinned memory: the runtime copies to and from the caller's arrays."""
    _in_and_out(itm, 16389, lambda: hip.limit_host(0, 0))
    assert hip.refusals() > 0


def tiles_in_order(itm, torch, hip, st):
    """A raycast at the frame's own pose takes its tiles in the integration's order from 3
    tiles per compute unit on, up to 65536, and in bands beside that range; at the same
    pose with a zero of the other sign always in bands.  The rays are the same bit for
    bit, and every tile is cast (the outputs are NaN before)."""
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert cu % 8 == 0
    ordered = b"k_raycastILi0ELb0ELb0ELb1EEE"
    sizes = [((cu // 8) * 16, 24 * 16 - 16, False), ((cu // 8) * 16, 24 * 16, True),
             ((cu // 8) * 16 + 1, 24 * 16 + 3, True), (4096, 4096, True), (4097, 4096, False)]
    T, other = np.eye(4), np.eye(4)
    other[3, 0] = -0.0
    for w, h, order in sizes:
        print(f"  {w}x{h}", flush=True)
        K = (0.8 * w, 0.8 * w, (w - 1) / 2, (h - 1) / 2, w, h)
        depth = torch.full((h, w), 1.5, device="cuda")
        depth += 0.3 * (torch.arange(w, device="cuda") / w > 0.6)
        depth[:, : w // 3] = 0.0                         # tiles that see nothing
        sc = itm.Scene(0.02, 0.08, 100, 1 << 15, 1 << 13)
        sc.set_search_range(True)
        sc.integrate(depth, K, T)
        rays = []
        for pose in (T, other):
            out = [torch.full((h, w, 4), float("nan"), device="cuda") for _ in range(2)]
            hip.launches_of(ordered)
            sc.raycast(K, pose, *out)
            n = hip.launches_of(b"")
            assert n == (1 if order and pose is T else 0), (w, h, n)
            rays.append(out)
        for a, b in zip(*rays):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
        P = rays[0][0]
        assert not P.isnan().any() and 0.3 < (P[..., 3] > 0).float().mean() < 0.9
        sc.close()


CASES = {f.__name__: f for f in (pointers_not_sent, pageable_after_one, pageable_after_two, no_copies_at_all,
                                 device_memory_for_one, no_device_memory, no_staging, tiles_in_order)}


@pytest.fixture(scope="module")
def outcomes(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("limits") / "limited_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "limited_hip.c"), "-ldl"],
                   check=True)
    p = subprocess.run([sys.executable, "-u", os.path.abspath(__file__), so], cwd=ROOT, capture_output=True, text=True,
                       timeout=110)
    print(p.stdout[-4000:], p.stderr[-4000:], flush=True)
    got = dict(json.loads(x[6:]) for x in p.stdout.splitlines() if x.startswith("CASE: "))
    assert p.returncode == 0, (p.returncode, got)
    return got


@pytest.mark.parametrize("name", list(CASES))
def test_refused(name, outcomes):
    assert outcomes.get(name) == "ok", outcomes.get(name)


if __name__ == "__main__":
    hip = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)     # before the runtime is loaded
    for name in ("limit_host", "limit_device", "fail_copies"):
        getattr(hip, name).argtypes = [C.c_size_t, C.c_long]
    hip.launches_of.argtypes = [C.c_char_p]
    hip.refusals.restype = hip.launches_of.restype = C.c_long
    sys.path.insert(0, ROOT)
    import traceback

    import torch

    import paper_1410_0925_amd as itm
    from synth import make_stream
    st = make_stream("vga", n_frames=40)
    for name, case in CASES.items():
        if len(sys.argv) > 2 and name not in sys.argv[2:]:
            continue
        print("begin", name, flush=True)
        hip.refusals()
        try:
            case(itm, torch, hip, st)
            res = "ok"
        except Exception:
            res = traceback.format_exc()
        hip.limit_host(2 ** 63, 0)
        hip.limit_device(2 ** 63, 0)
        hip.fail_copies(0, 0)
        print("CASE: " + json.dumps([name, res]), flush=True)
