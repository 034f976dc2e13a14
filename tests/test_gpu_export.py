"""Export and import on the GPU: key order, values in every storage form, repeated
keys and invalid voxels, at the edges of the sort's tiles (4096 keys), the export's
chunks (4096 blocks) and the import's staging (1 GiB)."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_util import gpu

pytestmark = pytest.mark.gpu


def _map(n, seed):
    """n distinct blocks in random order over the key range, F and W of the s16u8 form."""
    rng = np.random.default_rng(seed)
    c = rng.integers(-32767, 32768, (2 * n + 16, 3))
    c[::2] = rng.integers(-40, 40, c[::2].shape)       # half of them close together
    c = np.unique(c, axis=0)
    c = c[rng.permutation(len(c))[:n]].astype(np.int32)
    assert len(c) == n
    q = rng.integers(-32767, 32768, (n, 512)).astype(np.float32)
    return c, q / np.float32(32767), rng.integers(0, 101, (n, 512)).astype(np.float32)


def _scene(itm, n, fmt):
    log2 = max(4, int(np.ceil(np.log2(n + 1))))
    return itm.Scene(0.005, 0.02, 100, 2 ** log2, 2 ** log2, fmt=fmt)


@pytest.mark.parametrize("fmt", ["f32", "f16", "s16u8"])
@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 12289])
def test_round_trip_in_key_order(n, fmt):
    itm, torch = gpu()
    c, F, W = _map(n, n)
    want = F.astype(np.float16).astype(np.float32) if fmt == "f16" else F
    with _scene(itm, n, fmt) as sc:
        sc.import_blocks(c, F, W)
        gc, gF, gW = sc.export()
        only, none, _ = sc.export(values=False)
    at = np.lexsort((c[:, 2], c[:, 1], c[:, 0]))
    assert none is None and np.array_equal(only, c[at])
    assert np.array_equal(gc, c[at]) and np.array_equal(gW, W[at])
    assert np.array_equal(gF, want[at])


@pytest.mark.parametrize("n", [12287, 12288, 20481])
def test_imports_through_the_staging(n):
    # 12288 blocks are the first to go through the pinned slots (4096 blocks each)
    itm, torch = gpu()
    c, F, W = _map(n, n)
    at = np.lexsort((c[:, 2], c[:, 1], c[:, 0]))
    with _scene(itm, n, "f32") as sc:
        for k in range(2):     # the second import changes every block
            sc.import_blocks(c, F * np.float32(1 - k / 2), W)
        gc, gF, gW = sc.export()
    assert np.array_equal(gc, c[at]) and np.array_equal(gW, W[at])
    assert np.array_equal(gF, F[at] * np.float32(0.5))


def test_partial_outputs_and_colour():
    itm, torch = gpu()
    n = 5000
    c, F, W = _map(n, 3)
    at = np.lexsort((c[:, 2], c[:, 1], c[:, 0]))
    with _scene(itm, n, "f32") as sc:
        sc.enable_colour()
        sc.import_blocks(c, F, W)
        out = np.empty((n, 512), np.float32)
        m = C.c_int64(0)
        for args, want in (((out.ctypes.data, None), F), ((None, out.ctypes.data), W)):
            out[:] = np.nan
            itm._check(itm.lib().itm_export_blocks(sc.h, None, *args, n, C.byref(m)))
            assert m.value == n and np.array_equal(out, want[at])
        with pytest.raises(itm.ItmError):
            itm._check(itm.lib().itm_export_blocks(sc.h, None, out.ctypes.data, None, n - 1, C.byref(m)))
        rgbw = sc.export_colour()
        assert rgbw.shape == (n, 512, 4) and not rgbw.any()


def test_refused_imports_change_nothing():
    itm, torch = gpu()
    n = 9000
    c, F, W = _map(n, 5)
    with _scene(itm, n, "f32") as sc:
        for a, b in ((0, 1), (10, 8999), (4095, 4096)):
            d = c.copy()
            d[a] = d[b]
            with pytest.raises(itm.ItmError, match="twice"):
                sc.import_blocks(d, F, W)
        for v, name, x in ((8999 * 512 + 500, "F", np.nan), (512, "F", 1.0001), (77, "W", 2.5),
                           (5000 * 512, "W", 101.0), (3, "W", -1.0), (4, "F", np.inf), (5, "W", np.inf)):
            f, w = F.copy(), W.copy()
            (f if name == "F" else w).reshape(-1)[v] = x
            f[n - 1, 511] = 2.0    # the first bad voxel is the one named
            with pytest.raises(itm.ItmError, match=f"voxel {v}: {name}"):
                sc.import_blocks(c, f, w)
        assert sc.stats()["n_allocated"] == 0 and len(sc.export()[0]) == 0
        sc.import_blocks(c, F, W)
        assert sc.stats()["n_allocated"] == n


def test_map_larger_than_the_staging():
    itm, torch = gpu()
    n = 2 ** 18 + 5
    c, F, W = _map(n, 9)
    with itm.Scene(0.005, 0.02, 100, 2 ** 18, 2 ** 17, fmt="s16u8") as sc:
        good = W[n - 1, 0]
        W[n - 1, 0] = 0.5
        with pytest.raises(itm.ItmError, match=f"voxel {(n - 1) * 512}: W"):
            sc.import_blocks(c, F, W)
        W[n - 1, 0] = good
        sc.import_blocks(c, F, W)
        gc, gF, gW = sc.export()
    at = np.lexsort((c[:, 2], c[:, 1], c[:, 0]))
    assert np.array_equal(gc, c[at]) and np.array_equal(gF, F[at]) and np.array_equal(gW, W[at])


@pytest.mark.parametrize("n", [3, 1025, 4097, 12287, 24577])
def test_every_way_out_and_in(n):
    """A scene's first transfers and its later ones, whole and one array at a time: sizes
    on either side of those from which the staging is taken (4, 16, 48 and 96 MiB), odd
    so that the memory behind the lists needs its alignment."""
    itm, torch = gpu()
    c, F, W = _map(n, n)
    at = np.lexsort((c[:, 2], c[:, 1], c[:, 0]))
    print(f"case: {n} blocks", flush=True)
    with _scene(itm, n, "f32") as sc:
        sc.enable_colour()
        for k in range(3):
            f = F * np.float32(1 - k / 4)
            sc.import_blocks(c, f, W)
            gc, gF, gW = sc.export()
            assert np.array_equal(gc, c[at]) and np.array_equal(gF, f[at]) and np.array_equal(gW, W[at])
            out, m = np.full((n, 512), np.nan, np.float32), C.c_int64(0)
            itm._check(itm.lib().itm_export_blocks(sc.h, None, None, out.ctypes.data, n, C.byref(m)))
            assert np.array_equal(out, W[at])
            rgbw = sc.export_colour()
            assert rgbw.shape == (n, 512, 4) and not rgbw.any()


@pytest.mark.parametrize("n", [1, 2, 64, 65])
def test_small_imports(n):
    """Up to 64 blocks are checked on the host, more on the device: the same refusals, the
    first bad voxel named, and nothing changed by them."""
    itm, torch = gpu()
    c, F, W = _map(n, 40 + n)
    at = np.lexsort((c[:, 2], c[:, 1], c[:, 0]))
    print(f"case: {n} blocks", flush=True)
    with _scene(itm, n, "f32") as sc:
        sc.import_blocks(c[:0], F[:0], W[:0])
        if n > 1:
            d = c.copy()
            d[n - 1] = d[0]
            with pytest.raises(itm.ItmError, match="twice"):
                sc.import_blocks(d, F, W)
        last = n * 512 - 1
        for v, name, x in ((last, "F", np.nan), (0, "F", -1.0001), (last, "W", 2.5), (1, "W", 101.0), (2, "W", -1.0),
                           (3, "F", -np.inf), (last, "W", np.inf), (4, "W", np.nan)):
            f, w = F.copy(), W.copy()
            w[n - 1, 511] = 0.5    # a later one, unless it is the one
            (f if name == "F" else w).reshape(-1)[v] = x
            with pytest.raises(itm.ItmError, match=f"voxel {v}: {name}"):
                sc.import_blocks(c, f, w)
        assert sc.stats()["n_allocated"] == 0
        F[0, 0], F[n - 1, 511], W[0, 1], W[n - 1, 510] = -1.0, 1.0, 0.0, 100.0
        sc.import_blocks(c, F, W)
        gc, gF, gW = sc.export()
    assert np.array_equal(gc, c[at]) and np.array_equal(gF, F[at]) and np.array_equal(gW, W[at])
