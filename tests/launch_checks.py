"""Checks of the launches that the library's calls make, over the stand-in runtime of fake_hip.py.
Each check runs in a process of its own (test_launches.py)."""
import ctypes
import re

import fake_hip

IN, OUT = 1 << 43, 1 << 42     # addresses of an input and an output that nothing reads


class BmLds(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("pitch8", "pitch16", "rows", "plane8", "off_p8", "off_p16", "off_n8",
                                              "off_n16", "off_tab", "off_rs", "total")]


def windows_and_steps():
    """Every accepted (window, step)."""
    return [(W, s) for W in range(3, 32, 2) for s in range(1, (64 - W) // 3 + 1)]


def _match_lds(launch, layout, W, s, h, w, frames):
    """Every LDS access of a matching launch lies within the array it is meant for."""
    L = launch.arg(layout, BmLds)
    where = (launch.name, W, s, h, w, frames)
    npl = int(re.search(r"ILi(\d+)E", launch.name).group(1))
    one = "video" in launch.name and "Lb1E" in launch.name
    rows = launch.block[0] // 256
    assert launch.lds == L.total <= 160 * 1024, where
    tab_stride = 964 if npl == 16 else 64 * npl + 4
    n = min(W, h - 7) * min(W, w - 7) * (frames if one else 1)
    uh, uw = min((rows - 1) * s + W, h - 7), min((REF_TILE - 1) * s + W, w - 7)
    prow, pcol = uh + 7, uw + 7
    staged = (pcol + 3) // 4 * 4
    plane16 = L.rows * L.pitch16
    last4 = (uw + 3) // 4 * 4 - 4
    # staging: rows of the planes, the last row of the last copy
    assert staged <= L.pitch8 and staged <= L.pitch16 and prow <= L.rows, where
    assert L.off_p8 + 3 * L.plane8 + (prow - 1) * L.pitch8 + staged <= L.off_p16, where
    assert L.off_p16 + 2 * (plane16 + (prow - 1) * L.pitch16 + staged) <= L.off_n8, where
    # rows of the norm pass: 11 values from each fourth column, in whole words
    assert L.off_p8 + (prow - 1) * L.pitch8 + last4 + 12 <= L.off_p16, where
    assert L.off_p16 + 2 * ((prow - 1) * L.pitch16 + last4 + 12) <= L.off_n8, where
    # its columns: 11 row sums from each fourth row, of both planes
    sums = L.off_rs if one else L.off_tab
    end = L.total if one or "video" not in launch.name else L.total - 16 * 32 * 8
    for u in range(max(1, uh - 3), uh + 1):
        last = 4 * ((u + 3) // 4) - 4 + 10
        assert sums + 4 * ((u + 7) * uw + last * uw + uw) <= end, where
    assert L.off_n8 + 4 * uh * uw <= L.off_n16 and L.off_n16 + 4 * uh * uw <= L.off_tab, where
    # operands of the distances
    assert L.off_p8 + 3 * L.plane8 + (uh + 6) * L.pitch8 + (uw - 1) // 4 * 4 + 8 <= L.off_p16, where
    assert L.off_p16 + 2 * (plane16 + (uh + 6) * L.pitch16 + (uw - 1) // 2 * 2 + 8) <= L.off_n8, where
    # the table: a window to a row, whole register rows read
    assert n <= 64 * npl and n <= tab_stride, where
    assert L.off_tab + 4 * ((4 * rows - 1) * tab_stride + max(tab_stride, 64 * npl)) <= (L.off_rs if one else end), where


REF_TILE = 4


def match_lds():
    f = fake_hip.FakeHip()
    ctx = f.context(())
    # images and frames larger than any union of windows, and sides that cut it to its parts
    sizes = [(200, 200), (38, 200), (200, 39), (46, 47), (64, 70), (15, 200), (200, 9)]
    for W, s in windows_and_steps():
        for h, w in sizes:
            p = f.params(1, stride=s, window=W, K=4)
            ref = ctypes.byref(p)
            seen = []
            f.watch = lambda l: seen.append(l) or _match_lds(l, 4, W, s, h, w, 1)
            f.call("htsvd_block_match", ctx, IN, h, w, 1, w, ref, OUT, OUT, None)
            assert len(seen) == 1
            for T, radius in ((1, 0), (3, 1), (7, 2), (70, 31)):
                seen = []
                f.watch = lambda l: seen.append(l) or _match_lds(l, 5, W, s, h, w, min(2 * radius + 1, T))
                f.call("htsvd_block_match_video", ctx, IN, T, h, w, 1, w, radius, ref, OUT, OUT, None)
                assert len(seen) == 1


def match_lds_batched():
    f = fake_hip.FakeHip()
    ctx = f.context((1,))
    ht = f.ht
    opts = ht.htsvd_batch_opts(0, 1, 0.0, 0)
    for W, s in windows_and_steps():
        if ((W - 1) // 2 + 1) ** 2 < 4:
            continue
        p = f.params(1, stride=s, window=W, K=4)
        for (h, w), other in (((200, 200), (40, 40)), ((38, 200), (15, 70)), ((46, 47), (46, 47))):
            imgs = (ht.htsvd_image * 2)(*[ht.htsvd_image(IN, a, b, 1, b, 20.0, 4, OUT, b) for a, b in ((h, w), other)])

            def look(l):
                if "bm_kernel_batched" in l.name:   # an image's own tiles lie in the layout of the largest
                    _match_lds(l, 3, W, s, max(h, other[0]), max(w, other[1]), 1)

            f.watch = look
            f.call("htsvd_denoise_batch", ctx, 2, imgs, ctypes.byref(p), ctypes.byref(opts), None)


def failed_basis_keeps_the_installed_one():
    """A basis for another band count that runs out of memory or cannot launch leaves the installed
    one, and its maps, in use."""
    import numpy as np
    f = fake_hip.FakeHip()
    ctx = f.context(())
    ht = f.ht
    eye = np.zeros((64, 8, 8))
    eye[0] = np.eye(8)
    h = w = 40
    p = f.params(1, stride=4, window=15, K=4)

    def denoise(bands):
        maps = []

        def look(l):
            if "band_rows_kernel" in l.name:
                maps.extend(l.arg(i, ctypes.c_uint64) for i in (6, 7, 8, 9))

        f.watch = look
        f.call("htsvd_denoise_bands", ctx, IN, h, w, bands, w * bands, ctypes.c_float(20.0), ctypes.byref(p), OUT,
               w * bands, None)
        assert len(maps) == 4 and all(f.holds(a) for a in maps), (bands, maps)

    def learn(bands, expect=0):
        f.call("htsvd_learn_basis", ctx, IN, h, w, bands, w * bands, 8, 4, None, None, None, expect=expect)

    def install(bands, expect=0):
        U = np.ascontiguousarray(eye[:bands])
        f.call("htsvd_set_basis", ctx, 8, bands, U.ctypes.data, U.ctypes.data, expect=expect)

    small = 4
    for first in (install, learn):
        for second in (install, learn):
            for big in (20, 64):
                first(small)
                denoise(small)
                allocations = 0
                for fail in range(8):   # the first, second, ... allocation of the call fails
                    f.c.fake_fail_malloc(fail)
                    before = len(f.live)
                    done = getattr(f.L, "htsvd_set_basis" if second is install else "htsvd_learn_basis")
                    U = np.ascontiguousarray(eye[:big])
                    args = (ctx, 8, big, U.ctypes.data, U.ctypes.data) if second is install else \
                        (ctx, IN, h, w, big, w * big, 8, 4, None, None, None)
                    status = done(*args)
                    f.c.fake_fail_malloc(-1)
                    if status == 0:
                        denoise(big)
                        break
                    assert status == ht.HTSVD_ENOMEM, (status, before)
                    allocations += 1
                    denoise(small)
                f.c.fake_fail_launches(1)
                learn(big // 2, expect=ht.HTSVD_EDEVICE)
                f.c.fake_fail_launches(0)
                denoise(big)
                learn(big)
                denoise(big)
    ht.htsvd_destroy(ctx)
    # everything but the fixed scratch array was given back
    assert sorted(f.live.values()) == [64 << 20], f.live


def _install_unit_basis(f, ctx, bands):
    import numpy as np
    U = np.zeros((bands, 8, 8))
    U[0] = np.eye(8)
    f.call("htsvd_set_basis", ctx, 8, bands, U.ctypes.data, U.ctypes.data)


def _denoise_bands(f, ctx, h, w, bands, p):
    return f.call("htsvd_denoise_bands", ctx, IN, h, w, bands, w * bands, ctypes.c_float(20.0), ctypes.byref(p), OUT,
                  w * bands, None)


def band_passes():
    """Passes of the band filter: their patch matrix within the cap or a single group, every row in one of
    them, and the row test only in passes of many rows of at most 31 bands."""
    f = fake_hip.FakeHip()
    ctx = f.context(())
    for bands in (2, 5, 16, 30, 31, 32, 64):
        _install_unit_basis(f, ctx, bands)
        for cap in (1 << 20, 1 << 24, 4 << 30, 2 ** 63 - 1):
            f.call("htsvd_set_band_memory", ctx, ctypes.c_int64(cap))
            for h, w, s, K, W in ((15, 30, 4, 8, 15), (48, 48, 4, 16, 21), (64, 60, 2, 32, 15), (9, 300, 1, 4, 31)):
                p = f.params(1, stride=s, window=W, K=K)
                rows, tested = [], []

                def look(l):
                    if "band_test_kernel" in l.name:
                        tested.append(l.arg(3, ctypes.c_int64))
                        assert bands <= 31 and tested[-1] > 2048 + 64 * (31 - bands)
                    if "band_rows_kernel" in l.name:
                        rows.append(l.arg(3, ctypes.c_int64))
                        listed = bands <= 31 and rows[-1] > 2048 + 64 * (31 - bands)
                        assert bool(l.arg(4, ctypes.c_uint64)) == listed and (not listed or tested[-1] == rows[-1])

                f.watch = look
                launches = _denoise_bands(f, ctx, h, w, bands, p)
                n_ref = f.L.htsvd_ref_count(h, 8, s) * f.L.htsvd_ref_count(w, 8, s)
                assert sum(rows) == n_ref * K, (bands, cap, h, w)
                assert all(r * 64 * bands * 8 <= cap or r == K for r in rows)
                assert len(launches) <= 4 + 3 * len(rows) + 2 * len(tested)


def zeroed_memory():
    """Memory of more than 2^31 words is cleared by several launches, each of less than 2^32 threads."""
    f = fake_hip.FakeHip()
    ctx = f.context(())
    bands, h, w = 64, 4096, 4095
    _install_unit_basis(f, ctx, bands)
    words = []

    def look(l):
        assert l.grid[0] * l.block[0] < 1 << 32, (l.name, l.grid, l.block)
        if "zero_words" in l.name:
            words.append((l.arg(0, ctypes.c_uint64), l.arg(1, ctypes.c_int64)))

    f.watch = look
    _denoise_bands(f, ctx, h, w, bands, f.params(1, stride=16, window=15, K=4))
    assert sum(n for _, n in words) >= 2 * h * w * bands + h * w
    assert words[0][0] + 4 * words[0][1] == words[1][0]


def _within_limits(l):
    """Launch limits of the device: threads along each side, blocks along y and z, threads and LDS of a
    block."""
    for n, b, most in zip(l.grid, l.block, ((1 << 32) - 1, 65535, 65535)):
        assert 0 < n * b < 1 << 32 and (n <= most), (l.name, l.grid, l.block)
    assert l.block[0] * l.block[1] * l.block[2] <= 1024 and l.lds <= 160 * 1024, (l.name, l.block, l.lds)


def large_videos():
    """Videos of up to 2^30 pixels of any shape."""
    f = fake_hip.FakeHip()
    ctx = f.context((1,))
    f.watch = _within_limits
    for T, h, w, s, W in ((1, 1 << 27, 8, 19, 7), (1, 8, 1 << 27, 19, 7), (1 << 13, 256, 500, 4, 15), (4, 1 << 14, 16000, 4, 15)):
        p = f.params(1, stride=s, window=W, K=4)
        launches = f.call("htsvd_denoise_video", ctx, IN, T, h, w, 1, w, 1, ctypes.c_float(20.0), ctypes.byref(p), OUT,
                          w, None)
        assert any("gather" in l.name or "normalize" in l.name for l in launches)


class TileGeom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("TY", "TX", "tiles_y", "tiles_x", "RH", "RW", "RP", "FS", "R")]


def _padded_fits(planes, rows, cols):
    """Planes with rows padded to 8 modulo 16 words beside 65 KB of tables, in the LDS of a workgroup
    without the lists' 6,184 bytes and 80 to spare."""
    return planes * rows * (cols + (24 - cols % 16) % 16) * 4 + 65 * 1024 <= 160 * 1024 - 6184 - 80


def _shift(contributions, least):
    """Largest shift up to 12 at which so many contributions of 1024 stay below 2^31, and >= least."""
    return max([f for f in range(13) if contributions * 1024 * 2 ** f < 2 ** 31 - 1], default=0) >= least


def _video_least_shift(c, K, T, h, w, s, W, radius):
    """Shift of the largest tile of at most 8 x 8 references whose padded slots fit, 9 at least; of the
    sums in memory where none does."""
    nslot, reach = min(2 * radius + 1, T), W - 1 + 8
    for side in range(8, 0, -1):
        n = (side - 1) * s + reach
        if _shift(side * side * K, 9) and _padded_fits(c, nslot * min(n, h), min(n, w)):
            return max(f for f in range(13) if _shift(side * side * K, f))
    return 12


def video_sums():
    """The video filter's sums are never coarser than those of the largest tile that fits with padded
    rows, its regions fit in LDS, and without memory for them the sums go straight to memory."""
    import random
    f = fake_hip.FakeHip()
    ctx = f.context()
    ht = f.ht
    rng = random.Random(5)
    forms = set()
    for _ in range(4000):
        T, h, w = rng.randint(1, 40), int(8 * 2 ** rng.uniform(0, 7)), int(8 * 2 ** rng.uniform(0, 7))
        c, K, (W, s) = rng.choice((1, 3)), rng.choice((4, 8, 16, 32)), rng.choice(windows_and_steps())
        radius = rng.choice((0, 1, 1, 2, 2, 3, 5, 10, 31))
        if min(W // 2 + 1, h - 7) * min(W // 2 + 1, w - 7) < K:
            continue
        where = (T, h, w, c, K, W, s, radius)
        seen = []

        def look(l):
            if "filter_mfma_ga" in l.name:
                seen.append((re.search(r"ELi(\d)EEE", l.name).group(1), l.arg(1, TileGeom), l.lds))
                assert l.lds + 6184 <= 160 * 1024, where

        f.watch = look
        p = f.params(c, stride=s, window=W, K=K)
        args = (ctx, IN, T, h, w, c, w * c, radius, ctypes.c_float(20.0), ctypes.byref(p), OUT, w * c, None)
        f.call("htsvd_denoise_video", *args)
        (form, tg, _), = seen
        forms.add(form)
        assert tg.FS >= _video_least_shift(c, K, T, h, w, s, W, radius), where + (tg.FS, tg.TY)
        if form == "2":
            assert _shift(tg.TY * tg.TX * K, tg.FS), where + (tg.TY, tg.TX, tg.FS)
        if rng.random() < 0.02:   # the first allocation of a new context's workspace fails
            other = ht.htsvd_create(0)
            ht.htsvd_set_basis(other, 8, c, *ht.load_basis_slices(c))
            del seen[:]
            f.c.fake_fail_malloc(0)
            status = f.L.htsvd_denoise_video(other, *args[1:])
            f.c.fake_fail_malloc(-1)
            assert status == ht.HTSVD_ENOMEM and not seen
            f.c.fake_fail_next(1)
            f.call("htsvd_denoise_video", other, *args[1:])
            f.c.fake_fail_next(0)
            assert [x[0] for x in seen] == ["1"], where
            ht.htsvd_destroy(other)
    assert forms == {"1", "2"}


def _image_least_shift(c, K, h, w, s, W, max_side=16):
    """Shift of the largest tile whose padded region fits, 9 at least."""
    for side in range(max_side, 0, -1):
        n = (side - 1) * s + W - 1 + 8
        if side == 1 or (_shift(side * side * K, 9) and _padded_fits(c + 1, min(n, h), min(n, w))):
            return max(f for f in range(13) if _shift(side * side * K, f))


def image_sums():
    """The filter's sums are never coarser than those of the largest tile that fits with padded rows, for
    one image and for a sweep; the call with fixed scratch takes coarser ones only where nothing else
    fits.  Regions fit in LDS."""
    import random
    f = fake_hip.FakeHip()
    ctx = f.context()
    ht = f.ht
    rng = random.Random(6)
    coarse = refused = 0
    for _ in range(6000):
        h, w = int(8 * 2 ** rng.uniform(0, 9)), int(8 * 2 ** rng.uniform(0, 9))
        c, K, (W, s) = rng.choice((1, 3)), rng.choice((4, 8, 16, 32)), rng.choice(windows_and_steps())
        if min(W // 2 + 1, h - 7) * min(W // 2 + 1, w - 7) < K:
            continue
        p = f.params(c, stride=s, window=W, K=K)
        least = {k: _image_least_shift(c, k, h, w, s, W) for k in (4, 8, 16, 32)}
        seen = []

        def look(l):
            if "filter_mfma_kernel" in l.name and "batched" not in l.name:
                seen.append((l.arg(2, ctypes.c_int), l.arg(1, TileGeom)))
                assert l.lds + 6184 <= 160 * 1024

        f.watch = look
        image = (ctx, IN, h, w, c, w * c, ctypes.c_float(20.0), ctypes.byref(p), OUT, w * c, None)
        f.call("htsvd_denoise", *image)
        Ks = [k for k in (4, 8, 16, 32) if k <= K]
        items = (ht.htsvd_sweep_item * len(Ks))(*[ht.htsvd_sweep_item(20.0, k, OUT, w * c) for k in Ks])
        f.call("htsvd_denoise_sweep", ctx, IN, h, w, c, w * c, len(Ks), items, ctypes.byref(p), None)
        assert len(seen) == 1 + len(Ks)
        for k, tg in seen:
            assert tg.FS >= least[k] and _shift(tg.TY * tg.TX * k, tg.FS), (h, w, c, k, W, s, tg.FS, tg.TY)
        del seen[:]
        if f.call("htsvd_denoise_noalloc", *image, expect=None) is None:
            refused += 1
            continue
        (k, tg), = seen
        coarse += tg.FS < least[k]
        assert _shift(tg.TY * tg.TX * k, max(9, tg.FS))
    assert coarse < 20 and refused > 100, (coarse, refused)


def match_forms():
    """The matcher's 64-register form runs for more than 512 tiles of which two share a CU, for every window
    class up to 640 positions, and only there."""
    f = fake_hip.FakeHip()
    ctx = f.context(())
    forms = set()
    for W, s in windows_and_steps():
        for side in (8 + 80 * s, 8 + 120 * s, 600):
            p = f.params(1, stride=s, window=W, K=4)
            (l,) = f.call("htsvd_block_match", ctx, IN, side, side, 1, side, ctypes.byref(p), OUT, None, None)
            npl, rows, many = re.search(r"bm_kernelILi(\d+)ELi(\d)ELb(\d)E", l.name).groups()
            n_ref = f.L.htsvd_ref_count(side, 8, s)
            tiles = -(-n_ref // int(rows)) * -(-n_ref // 4)
            two = 2 * (l.lds + 452 + 64) <= 160 * 1024   # 452 bytes of tile geometry, and some to round up
            assert (many == "1") == (tiles > 512 and two and npl != "16"), (W, s, side, l.name, l.lds)
            forms.add((npl, many))
    assert {(n, m) for n in ("4", "7", "10") for m in "01"} <= forms


def large_cubes():
    """Gram sums of cubes of up to 2^30 pixels at every step: launches within the device's limits, which
    take every chunk of 64 vectors once, at most 1,024 of them per workgroup."""
    f = fake_hip.FakeHip()
    ctx = f.context(())
    for bands in (2, 9, 64):
        for h, w, s in ((1 << 15, 1 << 15, 1), (1 << 15, 1 << 15, 4), (1 << 27, 8, 1), (8, 1 << 20, 1), (9, 9, 1)):
            slices = []

            def look(l):
                _within_limits(l)
                if "gram_bands" in l.name:
                    slices.append((l.arg(9, ctypes.c_int), l.arg(10, ctypes.c_int), l.grid[2]))

            f.watch = look
            f.call("htsvd_basis_gram", ctx, IN, h, w, bands, ctypes.c_int64(w * bands), 8, s, OUT, None)
            total = slices[0][1]
            assert [z0 for z0, _, _ in slices] == list(range(0, total, 65535)) and sum(n for _, _, n in slices) == total
            chunks = -(-f.L.htsvd_ref_count(h, 8, s) * f.L.htsvd_ref_count(w, 8, s) // 8)
            assert -(-chunks // total) <= 1024


def without_memory_for_the_fastest_tiles():
    """A call whose workspace does not fit with the fastest tiles runs with smaller regions, and fails only
    without room for these."""
    import random
    f = fake_hip.FakeHip()
    ht = f.ht
    rng = random.Random(7)
    for _ in range(400):
        h, w = int(8 * 2 ** rng.uniform(0, 8)), int(8 * 2 ** rng.uniform(0, 8))
        c, K, (W, s) = rng.choice((1, 3)), rng.choice((4, 16, 32)), rng.choice(windows_and_steps())
        if min(W // 2 + 1, h - 7) * min(W // 2 + 1, w - 7) < K:
            continue
        p = f.params(c, stride=s, window=W, K=K)
        image = ht.htsvd_image(IN, h, w, c, w * c, 20.0, K, OUT, w * c)
        item = ht.htsvd_sweep_item(20.0, K, OUT, w * c)
        opts = ht.htsvd_batch_opts(0, 1, 0.0, 0)
        calls = [("htsvd_denoise", (IN, h, w, c, w * c, ctypes.c_float(20.0), ctypes.byref(p), OUT, w * c, None)),
                 ("htsvd_denoise_tau", (IN, h, w, c, w * c, IN, ctypes.byref(p), OUT, w * c, None)),
                 ("htsvd_denoise_sweep", (IN, h, w, c, w * c, 1, ctypes.byref(item), ctypes.byref(p), None)),
                 ("htsvd_denoise_batch", (1, ctypes.byref(image), ctypes.byref(p), ctypes.byref(opts), None))]
        for name, args in calls:
            sizes = []
            for fail in (0, 1, 2):
                ctx = ht.htsvd_create(0)
                ht.htsvd_set_basis(ctx, 8, c, *ht.load_basis_slices(c))
                held = sum(f.live.values())
                f.c.fake_fail_next(fail)
                f.call(name, ctx, *args, expect=0 if fail < 2 else ht.HTSVD_ENOMEM)
                f.c.fake_fail_next(0)
                sizes.append(sum(f.live.values()) - held)
                ht.htsvd_destroy(ctx)
            assert sizes[1] <= sizes[0], (name, h, w, c, K, W, s, sizes)
