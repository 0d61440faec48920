"""The library's host side at sizes and on paths that need no GPU: what it
launches, how it sizes LDS and what it waits for, seen by a HIP runtime that
runs nothing (stand_in_hip.c).  Each case runs in a process of its own, which
loads that runtime before the library.
"""
import ctypes as C
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(HERE))
from paper_1805_06019_amd import lfc  # noqa: E402

DEVICE = 1 << 44    # an address of the stand-in's device memory
CASES = {}


def case(f):
    CASES[f.__name__] = f
    return f


@pytest.fixture(scope="session")
def stand_in(tmp_path_factory):
    if not shutil.which("gcc") or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("needs gcc and the HIP headers")
    so = str(tmp_path_factory.mktemp("hip") / "stand_in_hip.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "stand_in_hip.c"), "-o", so], check=True, timeout=120)
    return so


class Watch:
    """The launches the stand-in saw (kernel, grid, threads, LDS bytes; of a batch's interpolation also its first
    record, pieces of a row and requests), and the order of its launches, copies and waits."""

    def __init__(self, so):
        self.launches, self.events, self.fail = [], [], None
        hip = C.CDLL(so, C.RTLD_GLOBAL)
        launch_t = C.CFUNCTYPE(C.c_int, C.c_char_p, C.POINTER(C.c_uint32), C.c_uint32, C.c_size_t, C.POINTER(C.c_void_p))
        event_t = C.CFUNCTYPE(None, C.c_char_p, C.c_void_p, C.c_size_t)
        self.keep = launch_t(self.on_launch), event_t(self.on_event)
        hip.stand_in_watch(*self.keep)

    def on_launch(self, name, grid, threads, lds, args):
        g = tuple(grid[i] for i in range(3))
        more = None
        if b"interp" in name:   # (records, grid)
            pieces_n = C.cast(args[1], C.POINTER(C.c_int32))
            more = (C.cast(args[0], C.POINTER(C.c_uint64))[0], pieces_n[0], pieces_n[1])
        self.launches.append((name.decode(), g, threads, lds, more))
        self.events.append(("launch", name.decode(), 0))
        return 1 if self.fail and self.fail in name.decode() else 0

    def on_event(self, what, src, n):
        self.events.append((what.decode(), src, n))


def opened(U, V, W, H, block, levels, tile=0, threshold=1 << 20, seed=1):
    """An opened light field; the default threshold leaves it no residuals."""
    rgb = np.random.default_rng(seed).integers(0, 256, (V, U, H, W, 3), dtype=np.uint8)
    p = lfc.Params(U, V, W, H, block, levels, (2,) * (levels - 1), blk_threshold=threshold)
    s = np.frombuffer(lfc.lfc_encode(rgb, p), np.uint8)
    h = C.c_void_p()
    lfc._check(lfc.load().lfc_open_ex(s.ctypes.data, s.size, C.byref(lfc.c_open_config(tile)), None, C.byref(h)))
    return h


# ---------------------------------------------------------------------------

@case
def batch_of_many_requests_and_one_large(w):
    """Every band of output rows, piece of a row and request of a batch has a
    workgroup, whose number the kernel forms in 32 bits."""
    lib, lf = lfc.load(), opened(3, 3, 24, 16, 4, 2)
    b = C.c_void_p()
    lfc._check(lib.lfc_batch_create(C.byref(b)))
    for n, big_w, big_h in ((20000, 16384, 16384), (65535, 16384, 16384), (65535, 4097, 16381), (16384, 16384, 16384),
                            (16383, 16384, 16384), (70, 300, 200)):
        reqs = lfc._requests([(0, big_w if i == 7 else 1 + i % 5, big_h if i == 7 else 1 + i % 3, (1.0, 1.0, 0.0, 0.0))
                              for i in range(n)])
        outs = (C.c_void_p * n)(*([DEVICE] * n))
        w.launches.clear()
        lfc._check(lib.lfc_batch_render(b, (C.c_void_p * 1)(lf), 1, reqs, n, outs, None))
        interp = [x for x in w.launches if "interp" in x[0]]
        assert interp
        pieces, bands, served = -(-big_w // 256), -(-big_h // 4), 0
        at, record = interp[0][4][0], 0
        if len(interp) > 1:
            record = (interp[1][4][0] - at) // interp[0][4][2]
        for _, g, threads, _, (first, gp, gn) in interp:
            blocks = g[0] * g[1] * g[2]
            assert threads == 256 and gp == pieces and g[0] * threads < 1 << 32 and g[1] <= 65535 and g[2] == 1
            assert blocks <= 1 << 32, (n, big_w, big_h, g)   # the numbers 0 .. blocks - 1 fit
            assert blocks >= 8 * -(-bands // 8) * pieces * gn
            assert first == at + served * record
            served += gn
        assert served == n
    print("done")


@case
def gpu_encoder_fails_while_its_tables_are_copied(w):
    """A failed launch returns only after the copy of the host's tables, which the call frees, has been waited for."""
    p = lfc.Params(5, 4, 40, 24, 4, 3, (2, 2)).to_c()
    for kernel in ("k_enc_level0", "k_enc_filter", "k_enc_residual", "k_enc_group_words", "k_enc_offsets"):
        w.fail = kernel
        w.events.clear()
        out, n = C.c_void_p(), C.c_size_t()
        assert lfc.load().lfc_encode_gpu(DEVICE, C.byref(p), C.byref(out), C.byref(n), None, None) == -4
        what = [e[0] for e in w.events]
        assert any(e[0] == "launch" and kernel in e[1] for e in w.events)
        assert "wait" in what[what.index("copy in"):], (kernel, what)
    print("done")


@case
def gpu_encoder_of_large_views(w):
    """A dimension of a launch holds fewer than 2^32 threads, whatever size of view the encoder takes; every
    group, and the wave after the last one, has a wave of the packing kernel."""
    for W, H, block in ((65536, 1364, 2), (65536, 1366, 2), (65534, 21842, 2), (65536, 5464, 4), (640, 480, 4)):
        p = lfc.Params(2, 2, W, H, block, 2, (2,)).to_c()
        out, n = C.c_void_p(), C.c_size_t()
        w.launches.clear()
        lfc._check(lfc.load().lfc_encode_gpu(DEVICE, C.byref(p), C.byref(out), C.byref(n), None, None))
        lfc.load().lfc_free(out)
        groups = 3 * -(-W // block) * -(-H // block)
        for name, g, threads, _, _ in w.launches:
            assert g[0] * threads < 1 << 32 and g[1] <= 65535 and g[2] <= 65535, (W, H, block, name, g)
            if "k_enc_pack" in name:
                assert groups + 1 <= g[0] * g[1] * threads // 64 < 1 << 31
    print("done")


@case
def whole_field_decode_with_the_largest_tiles(w):
    """A tile that leaves room for 1,024 words of gather tables beside it, the LUT and extents and the key-view
    rows is decoded; a larger one is refused."""
    # sparse fields of large trees, as many runs in a chunk as its tables allow: 25 key views (not staged), one
    # and 16 (the most that are staged: 16 KB)
    for levels, grid, most in ((3, 17, 1232), (6, 17, 1224), (4, 32, 1104)):
        for block, tile in ((2, 2048), (4, 2048), (8, 512), (8, 520), (8, 1024), (8, 1032), (8, 1072), (8, 1080),
                            (8, 1104), (8, 1168), (8, most), (8, most + 8)):
            h = opened(grid, grid, 16, 8, block, levels, tile)
            w.launches.clear()
            st = lfc.load().lfc_decode_blocks(h, None, grid * grid, 1, DEVICE, None)
            fits = block < 8 or tile <= most
            assert st == (0 if fits else -6), (block, tile, levels, st)
            if fits:
                assert w.launches[0][3] <= 160 * 1024
            lfc.load().lfc_close(h)
    print("done")


def auto_tile(h, n, wo, ho):
    """The tile that an automatic plan reports, or None if it takes the decoded path."""
    plan, cfg, graph = C.c_void_p(), lfc.c_render_config(), C.c_int32()
    lfc._check(lfc.load().lfc_render_plan_create(h, None, DEVICE, n, wo, ho, DEVICE, 0, C.byref(plan)))
    lfc._check(lfc.load().lfc_render_plan_info(plan, C.byref(cfg), C.byref(graph)))
    lfc.load().lfc_render_plan_destroy(plan)
    return None if cfg.path == lfc.RENDER_DECODED else (cfg.tile_w, cfg.tile_h)


@case
def render_tuner_tries_the_automatic_tile(w):
    """The tuner's candidates hold the tile of the automatic choice for its number and size of views, so its
    result is no slower than plain renders, also where every other shape's footprint is too large."""
    h = opened(5, 5, 640, 480, 4, 2)
    for n, wo, ho in ((1, 512, 384), (1, 256, 256), (1, 80, 60), (2, 200, 150), (3, 90, 70), (1, 160, 60), (1, 640, 61)):
        tile = auto_tile(h, n, wo, ho)
        assert tile is not None
        res = lfc.c_render_tuning()
        lfc._check(lfc.load().lfc_render_tune(h, DEVICE, n, wo, ho, DEVICE, 2, C.byref(res), None))
        tried = [(res.cfg[k].path, res.cfg[k].tile_w, res.cfg[k].tile_h) for k in range(res.n_tried)]
        assert (lfc.RENDER_TILES, *tile) in tried and (lfc.RENDER_DECODED, 0, 0) in tried, (n, wo, ho, tile, tried)
        assert len(set(tried)) == len(tried) <= 16
    print("done")


@case
def renders_without_allocation_take_the_automatic_tile(w):
    """Where the decoded views exceed the static scratch, the automatic choice of the entry point that allocates
    nothing falls back to the tile of lfc_render_views (as that takes it for a view fewer)."""
    h = opened(17, 17, 256, 256, 4, 2)
    assert 17 * 17 * 256 * 256 * 4 > lfc.NOALLOC_SCRATCH_BYTES
    n = 17 * 17 * 256 * 256 // (20 * 128 * 128)
    tile = auto_tile(h, n, 128, 128)
    assert tile is not None and auto_tile(h, n + 1, 128, 128) is None
    w.launches.clear()
    lfc._check(lfc.load().lfc_render_views_noalloc(h, DEVICE, n + 1, 128, 128, DEVICE, None, None))
    assert [x[1] for x in w.launches] == [(-(-128 // tile[0]), -(-128 // tile[1]), n + 1)], (tile, w.launches)
    print("done")


@case
def batch_tiles_follow_the_number_of_requests(w):
    """The tile requests of a batch, of one size, take the tile of as many views of that size rendered at once."""
    lib, h = lfc.load(), opened(5, 5, 640, 480, 4, 2)
    b = C.c_void_p()
    lfc._check(lib.lfc_batch_create(C.byref(b)))
    for n, wo, ho in ((1, 512, 384), (1, 160, 100), (2, 160, 100), (6, 160, 100), (3, 200, 150), (1, 320, 240)):
        tile = auto_tile(h, n, wo, ho)
        reqs = lfc._requests([(0, wo, ho, (1.5, 2.0, 0.0, 0.0))] * n)
        w.launches.clear()
        lfc._check(lib.lfc_batch_render(b, (C.c_void_p * 1)(h), 1, reqs, n, (C.c_void_p * n)(*([DEVICE] * n)), None))
        assert [x[1] for x in w.launches] == [(-(-wo // tile[0]) * -(-ho // tile[1]), n, 1)], (n, wo, ho, tile, w.launches)
    print("done")


# ---------------------------------------------------------------------------

@pytest.mark.parametrize("name", CASES)
def test_host_side(stand_in, name):
    r = subprocess.run([sys.executable, __file__, name, stand_in], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.endswith("done\n"), r.stdout[-4000:]


if __name__ == "__main__":
    CASES[sys.argv[1]](Watch(sys.argv[2]))
