"""What the host side enqueues, looked at on the CPU: the library's own objects linked against a recorder that takes
kernel launches in place of the HIP runtime (tests/launch_recorder.cpp).  Device pointers are made up; nothing runs."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_23079_amd import FLAG_AUTO_EVICT, FLAG_CACHED, FLAG_GLOBAL_TOPK, FLAG_INTERVAL_NEW, FLAG_STREAMING, BuzzConfig

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests")
WS, KP, VP, QP, SP, PP, OUT = (0x100000 * i for i in (1, 2, 3, 4, 5, 6, 7))     # made-up device addresses

# (query heads per kv head, head_dim, type, rows, splits): one row is left for the last split, the one that the step appends
NEW_ROW_ALONE = [(1, 64, "fp32", 25, 3), (1, 128, "bf16", 61, 6), (1, 256, "bf16", 25, 3), (1, 256, "fp32", 17, 5), (4, 128, "bf16", 33, 3), (8, 128, "fp16", 513, 9),
                 (2, 64, "bf16", 129, 9), (4, 64, "fp32", 33, 3), (8, 128, "fp32", 25, 3), (3, 256, "fp32", 61, 6), (5, 128, "fp32", 25, 3), (1, 64, "fp16", 57, 8)]

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    from paper_2410_23079_amd.build import CSRC, SOURCES, build
    objs = [os.path.join(CSRC, stem + ".o") for _, stem, _ in SOURCES]
    if not all(os.path.exists(o) for o in objs):             # objects are left by the in-tree build
        build()
    tmp = tmp_path_factory.mktemp("recorder")
    rec, so = str(tmp / "launch_recorder.o"), str(tmp / "libbuzz_recorded.so")
    subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, "-c", os.path.join(HERE, "launch_recorder.cpp"), "-o", rec], check=True, capture_output=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,--no-undefined", "-o", so, rec, *objs], check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    P, I64 = ctypes.c_void_p, ctypes.c_int64
    lib.buzz_prefill.argtypes = [P, P, P, I64, P, I64, P, P]
    lib.buzz_decode_step.argtypes = [P] * 6
    lib.buzz_cache_export.argtypes = [P] * 6
    lib.buzz_cache_import.argtypes = [P, P, P, P, P, I64, I64, I64, P]
    lib.buzz_evict.argtypes = [P, P]
    lib.buzz_cache_destroy.argtypes = [P]
    lib.rec_kernel.restype = ctypes.c_char_p
    lib.rec_value.restype = ctypes.c_longlong
    lib.rec_value.argtypes = [ctypes.c_int, ctypes.c_char_p]
    return lib


def config(**kw):
    base = dict(batch=2, n_q_heads=8, n_kv_heads=2, head_dim=128, kv_dtype="bf16", sink=4, window=64, segment=16,
                keep=2, evict_every=16, max_context=4096, old_stride=1, flags=FLAG_AUTO_EVICT)
    base.update(kw)
    return BuzzConfig(**base)


def create(lib, cfg):
    h, raw = ctypes.c_void_p(), cfg.to_c()
    assert lib.buzz_cache_create(ctypes.byref(raw), ctypes.c_void_p(WS), ctypes.c_size_t(1 << 60), ctypes.byref(h)) == 0
    return h


def recorded(lib):
    return [(lib.rec_kernel(i).decode(), i) for i in range(lib.rec_count())]


@pytest.mark.parametrize("dtype,n_obs", [("bf16", 300), ("fp32", 40)])
def test_a_prefill_that_fails_while_it_scores_leaves_no_cache_behind(lib, dtype, n_obs):
    """The scratch of the prompt scoring overlays the logits that a pending score update needs: whatever launch of a
    prefill with observed queries fails, no later call may read the old rows' update from it."""
    h = create(lib, config(kv_dtype=dtype))
    lib.rec_reset(-1)
    assert lib.buzz_prefill(h, KP, VP, 600, QP, n_obs, None, None) == 0
    lib.rec_reset(-1)
    assert lib.buzz_prefill(h, KP, VP, 600, QP, n_obs, None, None) == 0
    count = lib.rec_count()
    assert count >= 4                                        # two scoring steps, selection, placement
    for fail in range(count):
        for _ in range(3):                                   # leaves a score update pending
            assert lib.buzz_decode_step(h, QP, KP, VP, OUT, None) == 0
        lib.rec_reset(fail)
        assert lib.buzz_prefill(h, KP, VP, 600, QP, n_obs, None, None) == -4
        lib.rec_reset(-1)
        assert lib.buzz_decode_step(h, QP, KP, VP, OUT, None) == -3
        assert lib.buzz_evict(h, None) == -3 and lib.buzz_cache_export(h, KP, VP, SP, PP, None) == -3
        assert lib.rec_count() == 0
        assert lib.buzz_prefill(h, KP, VP, 600, QP, n_obs, None, None) == 0
    assert lib.buzz_cache_destroy(h) == 0


def scoring_passes(lib):
    """Per scoring pass: the launch's own split of both steps, as recorded with the first step's arguments."""
    names = ("t_begin", "t_count", "heads", "units", "key_parts", "key_part_len", "item_parts", "item_part_len", "stats_cap",
             "partial_cap")
    return [{n: lib.rec_value(i, n.encode()) for n in names} for k, i in recorded(lib)
            if "obs_mfma_kernel" in k and "Li1ELb" in k]


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("fp16", 256), ("fp32", 64), ("fp32", 256)])
@pytest.mark.parametrize("units,G,N,n_obs", [
    (16, 4, 8192, 8192), (16, 4, 16384, 16384), (8, 4, 32768, 32768), (16, 1, 131072, 131072), (1, 1, 131072, 131072),
    (8, 1, 9000, 5001), (3, 7, 20000, 12289), (32, 2, 4097, 4097), (2, 8, 4096, 4096), (1, 8, 50000, 300), (64, 1, 4095, 1), (1, 1, 300, 300),
    (64, 8, 4096, 128), (64, 8, 4096, 64), (64, 8, 1400, 128), (72, 8, 4096, 128), (64, 8, 4096, 192), (600, 1, 4096, 65),
    (200, 1, 1000, 1000), (300, 1, 5000, 4500)])
def test_the_cut_of_the_scoring_steps_is_never_bound_by_its_scratch(lib, dtype, D, units, G, N, n_obs):
    """Both steps of every pass are cut as the rule says -- where the longest block has more than half a compute unit's
    share, or waves without queries leave SIMDs idle; parts of a quarter of that share, at most 16 per block --
    whatever part of the prompt the pass sees, and the parts' results fit the arrays of the workspace."""
    h = create(lib, config(batch=1, n_q_heads=units * G, n_kv_heads=units, head_dim=D, kv_dtype=dtype, max_context=N,
                           window=64, evict_every=64, segment=64, keep=1))
    lib.rec_reset(-1)
    assert lib.buzz_prefill(h, KP, VP, N, QP, n_obs, None, None) == 0
    passes = scoring_passes(lib)
    assert len(passes) == -(-n_obs // 4096)
    row_bytes = D * (4 if dtype == "fp32" else 2)
    rows, cols, cus, shift = 64 if row_bytes <= 256 else 16384 // row_bytes, 128 if dtype == "fp32" else 256, 256, N - n_obs

    def check(lengths, blocks_per_length, parts, length, idle=False):
        longest, total = max(lengths), sum(lengths) * blocks_per_length
        cut = longest > -(-total // (2 * cus)) or idle and longest >= 24
        assert (parts > 1) == (cut and longest > max(-(-total // (4 * cus)), -(-longest // 16)))
        assert parts == -(-longest // length)
        if parts > 1:
            assert length == max(-(-total // (4 * cus)), -(-longest // 16))

    for p in passes:
        t0, end = p["t_begin"], p["t_begin"] + p["t_count"]
        keys = shift + end                                   # some query of the pass sees these
        waves = units * G * -(-p["t_count"] // (cols // 4))  # with queries: few of them leave SIMDs idle
        idle = dtype != "fp32" and waves < 1.5 * 4 * cus and (D == 64 or D == 128 and waves >= 4 * cus)
        check([(shift + min(t + cols, end) - 1) // rows + 1 for t in range(t0, end, cols)], units * G, p["key_parts"], p["key_part_len"],
              idle)
        first = [t0 + max(j - shift - t0, 0) // rows * rows for j in range(0, keys, cols)]
        check([-(-(end - t) // rows) * G for t in first], units, p["item_parts"], p["item_part_len"])
        assert p["key_parts"] == 1 or p["key_parts"] * p["heads"] * p["t_count"] <= p["stats_cap"]
        assert p["heads"] * p["t_count"] <= p["stats_cap"]
        assert p["item_parts"] == 1 or p["item_parts"] * units * keys <= p["partial_cap"]
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("segment,keep,one", [(4093, 3, True), (4092, 4, True), (4095, 1, True), (3001, 1095, True), (64, 8, True),
                                              (4093, 4, False), (4094, 3, False), (4096, 1, False)])
def test_the_one_launch_eviction_takes_every_segment_that_fits_the_lds(lib, segment, keep, one):
    """Scores and kept offsets of four waves in 64 KB: segment + keep up to 4096 floats per wave, whatever the segment is
    modulo four."""
    h = create(lib, config(segment=segment, keep=keep, evict_every=64, window=10, max_context=20000, flags=0))
    assert lib.buzz_cache_import(h, KP, VP, SP, PP, 4 + 10 + 50, 0, 64, None) == 0
    lib.rec_reset(-1)
    assert lib.buzz_evict(h, None) == 0
    kernels = [k for k, _ in recorded(lib)]
    assert ["evict_new_rows_kernel" in k for k in kernels] == ([True] if one else [False, False])
    assert all(lib.rec_value(i, b"lds") <= 65536 for _, i in recorded(lib))
    assert lib.buzz_cache_destroy(h) == 0


def prepared(lib, units, G, D, dtype, rows, flags=0):
    h = create(lib, config(batch=1, n_q_heads=units * G, n_kv_heads=units, head_dim=D, kv_dtype=dtype, window=rows - 5, segment=8,
                           evict_every=64, max_context=rows + 200, flags=flags))
    assert lib.buzz_cache_import(h, KP, VP, SP, PP, rows - 1, 0, rows - 1, None) == 0
    lib.rec_reset(-1)
    assert lib.buzz_decode_step(h, QP, KP, VP, OUT, None) == 0
    assert lib.rec_count() == 1
    return h, lib.rec_kernel(0).decode()


@pytest.mark.parametrize("units,G,D,dtype,rows,flags,anchored", [
    (512, 2, 128, "bf16", 2000, 0, True), (32, 4, 128, "fp16", 20000, 4, True), (128, 2, 256, "bf16", 4000, 4, True),
    (512, 2, 128, "bf16", 1000, 4, False), (512, 2, 128, "bf16", 2000, 8, False), (512, 2, 64, "bf16", 4000, 4, False)])
def test_streaming_steps_of_long_splits_anchor_their_tiles(lib, units, G, D, dtype, rows, flags, anchored):
    h, kernel = prepared(lib, units, G, D, dtype, rows, flags)
    streaming, anchor = re.search(r"attn_split_mfma_kernel.*Lb([01])ELi[48]ELb([01])E", kernel).groups()
    assert anchor == "01"[anchored] and (streaming == "1" or not anchored), kernel
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("units,D,dtype,rows,flags,waves,first", [
    (256, 128, "bf16", 1450, 0, 8, True), (250, 64, "fp32", 1500, 0, 8, True), (600, 64, "fp16", 900, 0, 4, True),   # a tile is two loads
    (144, 256, "bf16", 1711, 0, 8, False), (144, 128, "fp32", 1769, 0, 8, False), (160, 256, "fp16", 1399, 0, 8, False),
    (300, 256, "bf16", 840, 0, 4, False), (560, 256, "fp16", 375, 0, 4, True), (1100, 256, "bf16", 220, 0, 4, False),
    (200, 128, "bf16", 2700, 0, 8, False), (96, 256, "bf16", 4663, 0, 8, False), (8, 128, "fp16", 9000, FLAG_STREAMING, 8, False),
    (272, 128, "bf16", 2872, 0, 4, False), (300, 64, "bf16", 5000, 0, 4, False), (400, 128, "bf16", 1953, 0, 4, False),
    (100, 64, "bf16", 19548, 0, 4, False),                                                                          # 3 blocks per unit
    (430, 128, "bf16", 1775, 0, 4, True), (512, 128, "bf16", 3900, 0, 4, True), (1024, 128, "fp32", 800, 0, 4, True), (1100, 128, "bf16", 1000, 0, 4, False),
    (96, 256, "fp32", 1000, 0, 8, True), (272, 256, "fp32", 799, 0, 4, True), (272, 256, "fp32", 200, 0, 4, True), (560, 256, "fp32", 300, 0, 4, False),
    (64, 256, "fp32", 4200, 0, 8, False)])
def test_the_first_tile_goes_first_where_that_was_faster(lib, units, D, dtype, rows, flags, waves, first):
    """One head: in front of the side requests it thins the stream wherever a tile is more loads than are certain to follow it."""
    h, kernel = prepared(lib, units, 1, D, dtype, rows, flags)
    nw, short, tile_first = re.search(r"attn_split_kernelI.*ELi([48])ELi([0-3])ELb([01])ELb[01]E", kernel).groups()
    assert (int(nw), short, tile_first) == (waves, "0", "01"[first]), kernel
    assert lib.buzz_cache_destroy(h) == 0


def split_kernel(kernel):
    """(waves per block, tiles of a short split or 0) of a decode kernel's name."""
    m = re.search(r"attn_split_kernelI.*ELi([48])ELi([0-3])ELb[01]ELb[01]E", kernel) or re.search(r"attn_split_mfma_kernelI.*Lb[01]ELi([48])ELb[01]ELi([01])E", kernel)
    return tuple(map(int, m.groups()))


@pytest.mark.parametrize("units,D,dtype,rows,splits,tiles", [
    (64, 256, "bf16", 500, 4, 1), (64, 256, "bf16", 784, 4, 0), (192, 256, "bf16", 149, 1, 2), (240, 256, "fp16", 214, 1, 0), (8, 256, "bf16", 3000, 24, 1),
    (16, 256, "fp16", 2000, 8, 2), (16, 256, "fp16", 2300, 10, 0), (256, 256, "bf16", 131, 1, 2), (256, 256, "bf16", 133, 1, 0),   # 33 MB: 132 rows
    (256, 128, "fp32", 151, 1, 2), (256, 128, "fp32", 153, 1, 0),                                                                  # 38 MB: 152 rows
    (224, 128, "bf16", 250, 1, 2), (256, 128, "bf16", 380, 1, 3), (256, 64, "fp32", 380, 1, 3), (256, 256, "fp32", 120, 1, 2)])
def test_wide_rows_are_requested_at_once_while_the_dies_caches_hold_them(lib, units, D, dtype, rows, splits, tiles):
    """Two tiles per wave of one head's 512-byte rows: up to 33 MB (16 bit) and 38 MB (fp32) of K and V per step; other rows
    have no such line."""
    h = create(lib, config(batch=1, n_q_heads=units, n_kv_heads=units, head_dim=D, kv_dtype=dtype, window=rows - 5, segment=8, evict_every=64,
                           max_context=rows + 200, flags=0))
    assert lib.buzz_cache_set_splits(h, splits) == 0
    assert lib.buzz_cache_import(h, KP, VP, SP, PP, rows - 1, 0, rows - 1, None) == 0
    lib.rec_reset(-1)
    assert lib.buzz_decode_step(h, QP, KP, VP, OUT, None) == 0
    assert split_kernel(lib.rec_kernel(0).decode()) == (8, tiles), lib.rec_kernel(0)
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("units", [2, 8])
@pytest.mark.parametrize("G,D,dtype,n,splits", NEW_ROW_ALONE)
def test_the_new_row_can_be_alone_in_the_last_split(lib, G, D, dtype, n, splits, units):
    h = create(lib, config(batch=1, n_q_heads=units * G, n_kv_heads=units, head_dim=D, kv_dtype=dtype, window=n, flags=0))
    assert lib.buzz_cache_set_splits(h, splits) == 0
    assert lib.buzz_cache_import(h, KP, VP, SP, PP, n - 1, 0, n - 1, None) == 0
    lib.rec_reset(-1)
    assert lib.buzz_decode_step(h, QP, KP, VP, OUT, None) == 0
    assert split_kernel(lib.rec_kernel(0).decode())[1] >= 1
    assert [lib.rec_value(0, b"grid_" + x) for x in (b"x", b"y", b"z")] in ([splits, units, 1], [8, splits, units // 8])
    rows_per_split = lib.rec_value(0, b"lds") // (4 * G)     # the staged logits
    assert n - (splits - 1) * rows_per_split == 1
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("G,D,dtype,waves,rows", [
    (1, 64, "bf16", 8, (128, 256, 384)), (1, 128, "fp16", 8, (128, 256, 384)), (1, 64, "fp32", 8, (128, 256, 384)), (1, 128, "fp32", 8, (128, 256)),
    (1, 256, "bf16", 8, (128, 256)), (1, 256, "fp32", 8, (64, 128)), (2, 64, "bf16", 8, (128,)), (4, 128, "fp16", 8, (128,)), (8, 128, "bf16", 8, (128,)),
    (4, 64, "fp32", 8, (128,)), (3, 128, "fp32", 8, (128,)), (4, 256, "fp32", 8, (64,)), (5, 64, "fp32", 8, (64, 128)), (8, 128, "fp32", 8, (64, 128)),
    (5, 256, "fp32", 8, (64,)), (8, 256, "bf16", 4, (64,)), (8, 256, "fp32", 4, (32,)), (1, 128, "bf16", 4, (64,)), (1, 256, "fp32", 4, (32,)),
    (4, 128, "bf16", 4, (64,)), (6, 64, "fp32", 4, (32,))])
@pytest.mark.parametrize("flags", [0, FLAG_STREAMING])
def test_which_splits_are_requested_at_once(lib, G, D, dtype, waves, rows, flags):
    """Up to so many rows per split in one, two and three tiles per wave; one row more takes the next kernel."""
    units = 4 if G * D >= 1505 or waves == 8 else 300
    def kernel(n):
        h = create(lib, config(batch=1, n_q_heads=units * G, n_kv_heads=units, head_dim=D, kv_dtype=dtype, window=n, flags=flags))
        assert lib.buzz_cache_set_splits(h, 1) == 0
        assert lib.buzz_cache_import(h, KP, VP, SP, PP, n - 1, 0, n - 1, None) == 0
        lib.rec_reset(-1)
        assert lib.buzz_decode_step(h, QP, KP, VP, OUT, None) == 0
        assert lib.rec_value(0, b"grid_x") * lib.rec_value(0, b"grid_y") == units and lib.buzz_cache_destroy(h) == 0
        return split_kernel(lib.rec_kernel(0).decode())
    for tiles, n in enumerate(rows, 1):
        assert kernel(n) == (waves, 0 if flags else tiles)
        assert kernel(n + 1) == (waves, 0 if flags or tiles == len(rows) else tiles + 1)
    assert kernel(1) == (waves, 0 if flags else 1)


@pytest.mark.parametrize("units,G,D,rows,paced", [
    (520, 3, 256, 319, True), (640, 3, 256, 200, True), (560, 4, 128, 800, True), (280, 4, 128, 2500, True),   # the last: 2 splits per unit
    (512, 3, 256, 319, False), (512, 4, 128, 800, False), (641, 4, 128, 600, False), (300, 3, 256, 300, False),
    (560, 3, 256, 64, True), (560, 3, 256, 60, False), (560, 4, 128, 128, True), (560, 4, 128, 120, False),
    (560, 4, 256, 300, False), (560, 3, 128, 500, False), (560, 2, 256, 300, False), (560, 5, 128, 300, False), (560, 4, 64, 800, False)])
def test_uneven_blocks_are_paced_where_that_was_faster(lib, units, G, D, rows, paced):
    """2 to 2.5 blocks per compute unit, 3 heads of 256 or 4 of 128 in fp32, 64 KB of K per split: the sum over a row's lanes goes
    through LDS."""
    h, kernel = prepared(lib, units, G, D, "fp32", rows)
    nw, short, first, via_lds = re.search(r"attn_split_kernelI.*ELi([48])ELi([0-3])ELb([01])ELb([01])E", kernel).groups()
    assert (nw, short, first, via_lds) == ("4", "0", "0", "01"[paced]), kernel
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("units,rows,resident", [
    (1000, 1000, 2), (1024, 600, 2), (512, 5000, 2),         # 4 blocks per compute unit: 2 + 2, not 3 + 1
    (1300, 600, 3), (1280, 1000, 3),                         # 5 or 6 of them: 3 + 3 as well
    (768, 1000, 3), (512, 2000, 3), (2000, 700, 3), (1024, 300, 3)])   # one round, many rounds, short blocks: as they come
def test_two_rounds_of_blocks_come_out_even(lib, units, rows, resident):
    """The recorder's kernels have three waves per SIMD and 8000 bytes of LDS of their own: the LDS that a step asks for
    says how many of its 4-wave blocks a compute unit takes at a time."""
    h, kernel = prepared(lib, units, 2, 64, "bf16", rows, 8)
    assert lib.rec_value(0, b"block_x") == 256
    assert min(3, 160 * 1024 // (8000 + lib.rec_value(0, b"lds"))) == resident
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("dtype,G,D", [("fp32", 1, 64), ("fp32", 8, 256), ("bf16", 4, 128), ("bf16", 8, 64), ("fp16", 1, 128)])
@pytest.mark.parametrize("units", [1, 7, 8, 16, 32, 255, 256, 300])
@pytest.mark.parametrize("rows", [17, 90, 130, 400, 1000, 5000, 12000])
def test_the_automatic_split_count(lib, dtype, G, D, units, rows):
    """A few rows are not split, a step has at most one block per compute unit unless the logits of a split would not fit
    the LDS, and the entry point with the static scratch splits the same (its results are the same bits)."""
    def splits(n, static=False):
        h = create(lib, config(batch=1, n_q_heads=units * G, n_kv_heads=units, head_dim=D, kv_dtype=dtype, window=n - 5, segment=8,
                               evict_every=64, max_context=n + 200, flags=0))
        assert lib.buzz_cache_import(h, KP, VP, SP, PP, n - 1, 0, n - 1, None) == 0
        lib.rec_reset(-1)
        assert (lib.buzz_decode_step_static if static else lib.buzz_decode_step)(h, QP, KP, VP, OUT, None) == 0
        last = lib.rec_count() - 1
        grid = [lib.rec_value(last, b"grid_" + x) for x in (b"x", b"y", b"z")]
        s, rest = divmod(grid[0] * grid[1] * grid[2], units)
        assert rest == 0
        assert (lib.rec_count() == 2) == (static and s > 1)  # the counters' clearing
        assert lib.buzz_cache_destroy(h) == 0
        return s
    lib.buzz_decode_step_static.argtypes = [ctypes.c_void_p] * 6
    s = splits(rows)
    assert s <= max(1, 256 // units) or s <= -(-rows * G // (4096 - 260 * G)) + 1
    assert rows > 64 or s == 1
    if units * s * G * (D + 2) * 4 <= 8 << 20:
        assert splits(rows, True) == s


@pytest.mark.parametrize("segment,keep", [(64, 8), (255, 31), (1000, 100), (4096, 500), (5000, 600), (90000, 20000)])
@pytest.mark.parametrize("why", ["no scores", "interval"])
def test_a_selection_that_compares_nothing_ranks_nothing(lib, segment, keep, why):
    """Prompts without scores and interval sampling keep the first rows of every segment: no block-wide selection, whose
    lanes would all queue on one counter, at prefill and in evictions that thin the old rows, whatever the length."""
    h = create(lib, config(n_q_heads=2, segment=segment, keep=keep, evict_every=32, window=10, max_context=2 * segment + 200, old_stride=2,
                           flags=FLAG_INTERVAL_NEW if why == "interval" else 0))
    for rows in (segment + 40, 2 * segment + 40):
        lib.rec_reset(-1)
        assert lib.buzz_prefill(h, KP, VP, rows, None, 0, SP if why == "interval" else None, None) == 0
        names = [k for k, _ in recorded(lib)]
        assert names and not any("segment_topk_block" in k for k in names)
        assert all(lib.rec_value(i, b"lds") <= 65536 for _, i in recorded(lib))
    if why == "interval":
        for _ in range(32):
            assert lib.buzz_decode_step(h, QP, KP, VP, OUT, None) == 0
        lib.rec_reset(-1)
        assert lib.buzz_evict(h, None) == 0
        names = [k for k, _ in recorded(lib)]
        assert any("segment_topk_kernel" in k for k in names) and not any("segment_topk_block" in k for k in names)
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("segments,segment,block", [
    (1, 255, False), (16, 256, True), (16, 4097, True), (1024, 256, False), (1024, 320, True), (2048, 320, False), (2048, 400, True),
    (4096, 360, False), (4096, 450, True), (4096, 512, True), (8192, 360, False), (8192, 450, True), (16384, 360, False)])
@pytest.mark.parametrize("units", [1, 8])
def test_segments_are_ranked_by_what_was_faster(lib, segments, segment, block, units):
    """A wave per segment or a block per segment, at measured shapes on either side of the line."""
    n_seg = -(-segments // units)
    h = create(lib, config(batch=1, n_q_heads=units, n_kv_heads=units, head_dim=64, segment=segment, keep=4, evict_every=segment,
                           window=64, max_context=n_seg * segment + 68))
    lib.rec_reset(-1)
    assert lib.buzz_prefill(h, KP, VP, n_seg * segment + 68, None, 0, SP, None) == 0
    names = [k for k, _ in recorded(lib)]
    assert any("segment_topk_block" in k for k in names) == block, names
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("flags,rows,past", [(0, 200, True), (0, 1000, False), (0, 9000, True), (FLAG_CACHED, 200, True), (FLAG_STREAMING, 1000, True), (FLAG_STREAMING, 9000, True),
                                             (FLAG_CACHED, 1000, False), (FLAG_CACHED, 9000, True)])
@pytest.mark.parametrize("call", ["import", "prefill", "sampled"])
def test_rows_go_into_the_cache_past_the_last_level_cache_or_not(lib, flags, rows, past, call):
    """64 units of 512-byte rows: 7, 33 and 590 MB (the sampled prompt keeps all rows).  Fewer than 10 MB, more than 256 MB, or a
    caller who has said that nothing survives there."""
    sampled = call == "sampled"
    h = create(lib, config(batch=1, n_q_heads=64, n_kv_heads=64, window=rows // 2, segment=64, keep=64 if sampled else 8,
                           evict_every=64 if sampled else rows, max_context=rows, flags=flags))
    lib.rec_reset(-1)
    if call == "import":
        assert lib.buzz_cache_import(h, KP, VP, SP, PP, rows, 0, rows, None) == 0
    else:
        assert lib.buzz_prefill(h, KP, VP, rows, None, 0, SP, None) == 0
    into = re.findall(r"gather_rows_kernelILb([01])E|place_sampled_kernelILb([01])E", lib.rec_kernel(lib.rec_count() - 1).decode())
    assert "".join(into[0]) == "01"[past]
    lib.rec_reset(-1)
    assert lib.buzz_cache_export(h, KP, VP, SP, PP, None) == 0 and "gather_rows_kernelILb1E" in lib.rec_kernel(0).decode()
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("rows", [200, 2048, 4400])
@pytest.mark.parametrize("kind", ["thinned", "global"])
def test_rows_that_an_eviction_moves_do_not_stay_in_the_last_level_cache(lib, rows, kind):
    """Stored normally they are written back under the next steps, of this cache or of the others that take their turn."""
    moved = rows // 2
    h = create(lib, config(batch=1, n_q_heads=256, n_kv_heads=256, window=64, segment=32, keep=moved if kind == "global" else 4, evict_every=256,
                           max_context=40000, old_stride=2, flags=FLAG_GLOBAL_TOPK if kind == "global" else 0,
                           capacity=0 if kind == "global" else 4 + 64 + 256 + 2 * rows))
    n_old = moved if kind == "global" else rows
    assert lib.buzz_cache_import(h, KP, VP, SP, PP, 4 + 64 + n_old + 255, n_old, 30000, None) == 0
    lib.rec_reset(-1)
    assert lib.buzz_evict(h, None) == 0
    names = [k for k, _ in recorded(lib) if "gather_rows" in k]
    assert len(names) == (2 if kind == "global" else 3) and all("ILb1E" in k and "ILb0E" not in k and "ELb0E" not in k for k in names), names
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("dtype,D,units,G,N,n_obs,steps_place", [
    ("bf16", 256, 16, 1, 700, 16, False), ("bf16", 256, 32, 1, 700, 16, False), ("bf16", 256, 16, 1, 2000, 16, True), ("bf16", 256, 32, 1, 2000, 16, True),
    ("fp32", 256, 4, 1, 700, 16, False), ("fp32", 256, 16, 1, 2000, 16, True),
    ("bf16", 256, 4, 2, 3000, 500, True), ("bf16", 256, 1, 2, 12000, 256, False), ("bf16", 256, 1, 1, 2000, 2000, True),
    ("bf16", 128, 1, 1, 700, 16, False), ("bf16", 128, 8, 1, 200, 16, True), ("bf16", 128, 1, 1, 12000, 16, False), ("bf16", 128, 8, 1, 12000, 16, True),
    ("fp32", 128, 1, 1, 12000, 16, False), ("fp32", 128, 8, 2, 700, 256, True), ("fp16", 128, 256, 1, 4096, 256, True),
    ("bf16", 128, 16, 4, 4001, 4001, True), ("bf16", 128, 1, 1, 12000, 12000, True), ("fp16", 128, 4, 1, 10512, 2, True), ("bf16", 256, 4, 1, 12000, 16, True),
    ("fp16", 64, 1, 1, 200, 16, True), ("fp32", 64, 1, 1, 12000, 16, True), ("fp32", 64, 8, 1, 2048, 2048, True)])
def test_a_scored_prompt_that_is_kept_whole_is_placed_where_that_was_faster(lib, dtype, D, units, G, N, n_obs, steps_place):
    """By the scoring steps or by a copy of its own, at measured shapes on either side of the line."""
    h = create(lib, config(batch=1, n_q_heads=units * G, n_kv_heads=units, head_dim=D, kv_dtype=dtype, max_context=N, evict_every=N))
    lib.rec_reset(-1)
    assert lib.buzz_prefill(h, KP, VP, N, QP, n_obs, None, None) == 0
    names = [k for k, _ in recorded(lib)]
    assert "obs_" in names[0] and any("gather_rows" in k for k in names) == (not steps_place), names
    places = [lib.rec_value(i, b"places") for k, i in recorded(lib) if "obs_mfma" in k]
    assert places[-2:] == [steps_place] * 2 and not any(places[:-2])        # the last pass
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("units,rows,G,dtype,D,splits", [
    (8, 110, 1, "fp32", 64, 1), (100, 154, 8, "fp16", 64, 1), (72, 140, 2, "fp16", 128, 1), (256, 5000, 1, "bf16", 128, 1),      # whole
    (8, 300, 1, "fp32", 64, 3), (8, 1512, 4, "bf16", 128, 12), (8, 846, 4, "fp32", 64, 7),                                       # of 128 rows
    (3, 175, 4, "fp32", 256, 8), (12, 431, 4, "fp32", 256, 8),                                                                   # shorter
    (1, 12000, 4, "bf16", 128, 40), (1, 16000, 1, "bf16", 128, 56), (2, 20000, 4, "bf16", 64, 40), (3, 22272, 1, "fp16", 128, 85),  # longer
    (80, 320, 2, "fp16", 64, 3), (120, 220, 1, "fp32", 64, 2), (64, 286, 4, "fp16", 64, 1), (48, 262, 4, "bf16", 64, 1),           # many units
    # one head: as few splits as request their rows at once, where the merge saves more than the longer splits cost
    (8, 4200, 1, "bf16", 128, 17), (6, 5500, 1, "fp32", 128, 22), (10, 4000, 1, "fp16", 256, 16), (8, 4000, 1, "fp32", 64, 16),
    (2, 4053, 1, "fp32", 128, 32), (2, 4700, 1, "bf16", 256, 37), (1, 2000, 1, "fp32", 256, 32),                                   # wide rows, few units
    (1, 12000, 1, "bf16", 64, 40), (1, 9000, 1, "bf16", 64, 32), (3, 11000, 1, "fp32", 64, 40), (4, 12288, 1, "bf16", 128, 40),    # never more
    (8, 3072, 1, "bf16", 128, 24), (8, 3073, 1, "bf16", 128, 13),                                                                  # from 13 on
    (5, 12288, 1, "fp32", 128, 48), (5, 12289, 1, "fp32", 128, 51),                                                                # up to 48
    # whole: one head up to 55000 bytes of K per unit; up to 128 rows unless a split saves 1.6 us
    (8, 214, 1, "bf16", 128, 1), (8, 215, 1, "bf16", 128, 2), (8, 107, 1, "fp32", 128, 1), (8, 256, 1, "bf16", 64, 1),
    (8, 111, 8, "fp32", 64, 1), (8, 112, 8, "fp32", 64, 5), (8, 128, 4, "bf16", 128, 1), (8, 88, 6, "fp32", 128, 1), (8, 89, 6, "fp32", 128, 5)])
def test_the_automatic_split_count_at_measured_shapes(lib, units, rows, G, dtype, D, splits):
    h, _ = prepared(lib, units, G, D, dtype, rows)
    grid = [lib.rec_value(0, b"grid_" + x) for x in (b"x", b"y", b"z")]
    assert grid[0] * grid[1] * grid[2] == units * splits
    assert lib.buzz_cache_destroy(h) == 0


@pytest.mark.parametrize("units,rows,D,dtype,segment,keep,one", [
    (32, 32768, 128, "bf16", 64, 8, True), (128, 4096, 128, "bf16", 16, 2, True), (32, 32768, 64, "bf16", 32, 4, True), (8, 4096, 128, "bf16", 64, 8, True),
    (1, 1000, 64, "fp32", 16, 1, True), (4, 32768, 64, "bf16", 5, 1, False), (32, 8192, 64, "bf16", 100, 12, False), (8, 4096, 256, "bf16", 100, 12, False),
    (32, 32768, 128, "bf16", 5, 1, False), (8, 4096, 128, "bf16", 32, 4, False), (4, 4096, 128, "bf16", 1000, 8, False)])
@pytest.mark.parametrize("thinned", [False, True])
def test_a_sampled_prompt_is_placed_in_one_launch_or_two(lib, units, rows, D, dtype, segment, keep, one, thinned):
    """At measured shapes on either side of the line; two launches where the survivors are thinned before they are placed."""
    window = rows // 8
    h = create(lib, config(batch=1, n_q_heads=units, n_kv_heads=units, head_dim=D, kv_dtype=dtype, window=window, segment=segment, keep=keep,
                           evict_every=segment, max_context=rows, old_stride=2 if thinned else 1,
                           capacity=4 + window + segment + (rows - window) * keep // segment // 2 + keep + 8 if thinned else 0))
    lib.rec_reset(-1)
    assert lib.buzz_prefill(h, KP, VP, rows, None, 0, SP, None) == 0
    names = [k for k, _ in recorded(lib)]
    if one and not thinned:
        assert len(names) == 1 and "place_sampled" in names[0]
    else:
        assert len(names) == 2 and "segment_topk" in names[0] and "gather_rows" in names[1]
    assert lib.buzz_cache_destroy(h) == 0
