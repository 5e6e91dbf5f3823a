"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle in lock-step.

Bars (written out in tests/lockstep.py): retained positions, K rows and V rows bit-exact; attention
outputs within 2e-3 max relative error per head vector (and within 1e-4, what fp32 accumulation gives);
accumulated scores within 1e-4.
"""
import numpy as np
import pytest
import torch

from tests.test_launches_host import NEW_ROW_ALONE
from workloads import decode_inputs, get_workload, prompt_inputs

pytestmark = pytest.mark.gpu


def lockstep():
    from tests import lockstep as ls
    return ls


def small(name="tiny", **kw):
    return get_workload(name).scaled(**kw)


def run(wl, device="cuda", **kw):
    p = prompt_inputs(wl, device=device)
    d = decode_inputs(wl, device=device)
    print(f"[parity] {wl.name} B{wl.batch} Hq{wl.n_q_heads} Hkv{wl.n_kv_heads} D{wl.head_dim} {wl.dtype} "
          f"N{wl.prompt} steps{wl.decode_steps} k{wl.sink} w{wl.window} s{wl.segment} c{wl.keep} "
          f"T{wl.evict_every} sh{wl.old_stride} {kw}", flush=True)
    st = lockstep().run_lockstep(wl, p, d, **kw)
    print(f"[parity]   worst out {st['out']:.2e} score {st['score']:.2e} prefill-score {st['prefill_score']:.2e} "
          f"evictions {st['evictions']}", flush=True)
    return st


# ------------------------------------------------------------------ config 1 in full
def test_tiny_full():
    st = run(get_workload("tiny"))
    assert st["evictions"] == 256 // 16


def test_tiny_full_default_mode():
    """Without FLAG_DETERMINISTIC the waves claim tiles dynamically: same bars against the oracle."""
    st = run(get_workload("tiny"), deterministic=False)
    assert st["evictions"] == 256 // 16


def test_tiny_paper_old_stride():
    """The paper's default s^ = floor((s+1)/2): old survivors are interval-sampled at every eviction."""
    st = run(small(old_stride=0))
    assert st["evictions"] == 16


def test_tiny_paper_old_stride_with_capacity():
    """Remark 2: with an explicit capacity the prefill keeps sampling until the rows fit."""
    wl = small(old_stride=0, prompt=512, decode_steps=40)
    run(wl, capacity=wl.sink + wl.window + wl.evict_every + 6)


# ------------------------------------------------------------------ shapes, dtypes, group sizes, ragged everything
@pytest.mark.parametrize("dtype", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8])
def test_shapes(dtype, D, G):
    wl = small(batch=2, n_kv_heads=2, n_q_heads=2 * G, head_dim=D, dtype=dtype, prompt=300, decode_steps=45,
               sink=3, window=40, segment=7, keep=2, evict_every=10, n_obs=9)
    run(wl)


@pytest.mark.parametrize("deterministic", [True, False])
@pytest.mark.parametrize("G", [2, 8])
def test_group_sizes(G, deterministic):
    wl = small(batch=1, n_kv_heads=3, n_q_heads=3 * G, head_dim=128, dtype="bf16", prompt=700, decode_steps=40,
               sink=4, window=64, segment=16, keep=3, evict_every=16, n_obs=40)
    run(wl, deterministic=deterministic)


@pytest.mark.parametrize("dtype", ["fp32", "fp16"])
def test_single_block_units_default_mode(dtype):
    """One split per unit, many tiles per wave, tiles claimed dynamically."""
    wl = small(batch=1, n_kv_heads=4, n_q_heads=4, head_dim=128, dtype=dtype, prompt=3000, decode_steps=24,
               sink=4, window=1500, segment=16, keep=4, evict_every=8, n_obs=16)
    run(wl, splits=1, deterministic=False)


@pytest.mark.parametrize("kv_loads", ["streaming", "cached"])
@pytest.mark.parametrize("G,dtype", [(1, "fp16"), (4, "bf16"), (2, "fp32")])
def test_forced_kv_load_flavour(G, dtype, kv_loads):
    """Both load flavours of every kernel family, whatever the working-set size would have chosen."""
    wl = small(batch=1, n_kv_heads=3, n_q_heads=3 * G, head_dim=128, dtype=dtype, prompt=1300, decode_steps=24,
               sink=4, window=128, segment=16, keep=2, evict_every=16, n_obs=12)
    run(wl, kv_loads=kv_loads)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_widest_rows_and_groups(dtype):
    """head_dim 256 with 8 query heads per kv head: the largest per-block footprint the kernels support."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=16, head_dim=256, dtype=dtype, prompt=900, decode_steps=36,
               sink=4, window=128, segment=16, keep=2, evict_every=16, n_obs=12)
    run(wl)


@pytest.mark.parametrize("splits", [1, 2, 5, 16])
def test_split_counts(splits):
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2, head_dim=128, dtype="fp16", prompt=2000, decode_steps=20,
               sink=4, window=900, segment=16, keep=4, evict_every=8, n_obs=16)
    run(wl, splits=splits, check_auto=False)


@pytest.mark.parametrize("G,D,dtype,splits,prompt", [
    (1, 64, "bf16", 17, 900), (3, 64, "fp32", 9, 900), (8, 256, "bf16", 9, 700), (5, 128, "fp16", 33, 900),
    (4, 128, "bf16", 100, 1900), (1, 64, "fp16", 1, 5000), (2, 64, "bf16", 1, 3100)])
def test_split_merge_rounds_and_side_rounds(G, D, dtype, splits, prompt):
    """Merges of more splits than one round of loads covers (8 or 16), groups of 64 outputs that do not divide over
    the merging waves, and single splits with more rows than a thread requests ahead."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=D, dtype=dtype, prompt=prompt, decode_steps=9,
               sink=3, window=prompt - 77, segment=16, keep=3, evict_every=16, n_obs=8)
    run(wl, splits=splits)


@pytest.mark.parametrize("G,D,dtype,sink,T,steps", [(2, 128, "bf16", 3, 16, 40), (4, 128, "fp16", 17, 33, 70), (5, 128, "bf16", 0, 7, 20),
                                                    (3, 256, "fp16", 5, 50, 55)])
def test_anchored_tiles_of_long_streaming_splits(G, D, dtype, sink, T, steps):
    """One split of more than 1024 rows per unit, read with the streaming loads: tiles anchored at multiples of 16 physical
    rows, runs that start and end anywhere, the ring's wrap inside and between tiles."""
    n = 1200
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=D, dtype=dtype, prompt=n, decode_steps=steps, sink=sink,
               window=n - 70, segment=16, keep=3, evict_every=T, n_obs=8)
    run(wl, splits=1, kv_loads="streaming")


@pytest.mark.parametrize("G,D,dtype", [(1, 64, "fp32"), (1, 128, "bf16"), (1, 64, "fp16"), (1, 256, "fp32"), (4, 64, "fp32"), (3, 256, "fp32"),
                                       (4, 128, "bf16"), (8, 128, "fp16"), (2, 64, "bf16"), (8, 256, "bf16"), (1, 128, "fp32"), (1, 256, "bf16"),
                                       (5, 128, "fp32"), (8, 128, "fp32")])
@pytest.mark.parametrize("rows,splits", [(0, 1), (15, 1), (60, 1), (63, 2), (126, 1), (120, 3), (250, 1), (255, 2), (390, 4), (262, 1),
                                         (378, 1), (391, 1)])
def test_short_splits(G, D, dtype, rows, splits):
    """Splits whose rows are all requested at once: one row, tiles and blocks that are just full or just not, the ring's wrap and
    the linear region's end inside a tile, and the first size that is streamed instead."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=D, dtype=dtype, prompt=rows, decode_steps=14, sink=3,
               window=max(1, rows - 20), segment=4, keep=1, evict_every=7, n_obs=min(rows, 5))
    run(wl, splits=splits, check_auto=False)


@pytest.mark.parametrize("heads", [2, 8])
@pytest.mark.parametrize("G,D,dtype,n,splits", NEW_ROW_ALONE)
def test_the_new_row_alone_in_the_last_split(G, D, dtype, n, splits, heads):
    """The last block has no stored row: every lane takes the caller's, and there are no side rows.  Step 5 has n rows (that
    this leaves one for the last split is checked where the launch is looked at on the host); the cache grows through it."""
    wl = small(batch=1, n_kv_heads=heads, n_q_heads=heads * G, head_dim=D, dtype=dtype, prompt=n - 5, decode_steps=8, sink=3,
               window=n + 20, segment=4, keep=1, evict_every=16, n_obs=5)
    run(wl, splits=splits, check_auto=False)


@pytest.mark.parametrize("rows", [20, 40, 70])
@pytest.mark.parametrize("G,dtype", [(1, "fp32"), (1, "bf16"), (4, "bf16"), (6, "fp32"), (8, "fp16")])
def test_short_splits_of_more_units_than_compute_units(G, dtype, rows):
    """320 units: 4-wave blocks of one split each, requested at once up to 64 rows (32 with 6 fp32 heads), streamed beyond."""
    wl = small(batch=5, n_kv_heads=64, n_q_heads=64 * G, head_dim=64, dtype=dtype, prompt=rows, decode_steps=9, sink=3, window=rows - 10,
               segment=4, keep=1, evict_every=7, n_obs=5)
    run(wl, units=[(0, 0), (2, 17), (4, 63)])


@pytest.mark.parametrize("G,D,rows", [(3, 256, 90), (4, 128, 150)])
def test_blocks_paced_by_their_row_sums(G, D, rows):
    """520 units: two to three 4-wave blocks per compute unit, whose row sums exchange through LDS."""
    wl = small(batch=65, n_kv_heads=8, n_q_heads=8 * G, head_dim=D, dtype="fp32", prompt=rows, decode_steps=9, sink=3, window=rows - 10, segment=4,
               keep=1, evict_every=7, n_obs=3)
    run(wl, units=[(0, 0), (31, 3), (64, 7)])


@pytest.mark.parametrize("dtype", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8])
def test_shapes_of_cached_splits_that_are_streamed(dtype, D, G):
    """Whole caches of more rows than a block requests at once: runs up to the linear region's end, the ring's wrap and the new
    row, tiles that the waves claim, further rounds of side rows."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=D, dtype=dtype, prompt=600, decode_steps=12, sink=3, window=420, segment=7, keep=2,
               evict_every=10, n_obs=9)
    run(wl, splits=1, kv_loads="cached", check_auto=False)


@pytest.mark.parametrize("device_merge", [False, True])
@pytest.mark.parametrize("G,D,dtype,splits,rows", [(5, 256, "bf16", 9, 1500), (5, 128, "fp16", 9, 1500), (8, 256, "fp32", 9, 1500), (6, 128, "fp32", 10, 1600),
                                                   (3, 64, "fp32", 9, 1500), (1, 128, "bf16", 9, 3700), (1, 256, "fp32", 9, 1500)])
def test_merges_of_long_splits(G, D, dtype, splits, rows, device_merge):
    """More splits than a round of loads covers, each longer than a block requests at once: half of the block merges while the
    other half starts the side phase."""
    wl = small(batch=1, n_kv_heads=8, n_q_heads=8 * G, head_dim=D, dtype=dtype, prompt=rows, decode_steps=3, sink=3, window=rows - 120, segment=16,
               keep=3, evict_every=16, n_obs=8)
    run(wl, splits=splits, device_merge=device_merge, units=[(0, 0), (0, 5)])


@pytest.mark.parametrize("device_merge", [False, True])
@pytest.mark.parametrize("G,D,dtype,splits", [(1, 64, "fp16", 17), (1, 256, "bf16", 9), (2, 256, "fp32", 20), (3, 128, "bf16", 33),
                                              (4, 128, "fp16", 18), (5, 256, "bf16", 10), (6, 256, "fp16", 9), (7, 256, "bf16", 17),
                                              (8, 64, "bf16", 40), (8, 256, "fp32", 12)])
def test_merge_rounds_through_one_die_and_device_memory(G, D, dtype, splits, device_merge):
    """Merges of more splits than one round of loads covers, with every way the outputs of a unit are dealt to the
    merging waves (whole heads, parts of a head, more heads than waves), in both forms of the merge."""
    wl = small(batch=1, n_kv_heads=8, n_q_heads=8 * G, head_dim=D, dtype=dtype, prompt=900, decode_steps=5,
               sink=3, window=780, segment=16, keep=3, evict_every=16, n_obs=8)
    run(wl, splits=splits, device_merge=device_merge, units=[(0, 0), (0, 5)])


@pytest.mark.parametrize("device_merge", [False, True])
@pytest.mark.parametrize("G,dtype,heads", [(1, "fp16", 8), (4, "bf16", 8), (2, "fp32", 16), (8, "bf16", 8)])
def test_split_merge_through_one_die_or_device_memory(G, dtype, heads, device_merge):
    """Units that divide evenly over the 8 dies with several splits each: by default a unit's blocks share a
    die and merge through its L2 (eq. 3 / eq. 5 split softmax); with the flag they merge through device memory."""
    wl = small(batch=1, n_kv_heads=heads, n_q_heads=heads * G, head_dim=128, dtype=dtype, prompt=2600, decode_steps=36,
               sink=4, window=1100, segment=16, keep=3, evict_every=16, n_obs=24)
    run(wl, device_merge=device_merge, deterministic=False)


@pytest.mark.parametrize("G,dtype,old_stride", [(1, "fp32", 1), (4, "bf16", 1), (1, "fp16", 0)])
def test_export_then_import_resumes_the_cache(G, dtype, old_stride):
    """Checkpoint / resume: rows exported from a running cache and imported into a fresh one give the same
    attention outputs (same rows, other places in the ring: sums within rounding), the same evictions and the
    same final rows."""
    from paper_2410_23079_amd import FLAG_AUTO_EVICT, FLAG_DETERMINISTIC, BuzzCache
    ls = lockstep()
    wl = small(batch=2, n_kv_heads=2, n_q_heads=2 * G, head_dim=128, dtype=dtype, prompt=900, decode_steps=90,
               sink=4, window=100, segment=16, keep=2, evict_every=16, old_stride=old_stride, n_obs=24)
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    a, b = (BuzzCache(ls.buzz_config(wl, flags=FLAG_AUTO_EVICT | FLAG_DETERMINISTIC)) for _ in range(2))
    a.prefill(p["K"], p["V"], q_obs=p["q_obs"])
    out_a, out_b = (torch.empty(wl.batch, wl.n_q_heads, wl.head_dim, dtype=torch.float32, device="cuda") for _ in range(2))
    first = 37                                                  # mid-cycle: buffered rows, ring head moved twice
    for t in range(first):
        a.decode_step(d["q"][t], d["k"][t], d["v"][t], out_a)
    K, V, S, P = a.export()
    n, n_old, _ = a.lengths()
    b.import_rows(K, V, S, P, n_old=n_old, tokens_seen=wl.prompt + first)
    assert a.lengths() == b.lengths()
    for t in range(first, wl.decode_steps):
        a.decode_step(d["q"][t], d["k"][t], d["v"][t], out_a)
        b.decode_step(d["q"][t], d["k"][t], d["v"][t], out_b)
        e = ls.rel_err(out_b.double().cpu().numpy(), out_a.double().cpu().numpy())
        assert e <= ls.REPRO_TOL, f"step {t}: resumed cache differs by {e}"
        assert a.lengths() == b.lengths()
    for i, (x, y) in enumerate(zip(a.export(), b.export())):
        if i == 2:
            assert torch.allclose(x, y, rtol=ls.REPRO_TOL, atol=ls.REPRO_TOL)
        else:
            assert torch.equal(x, y)


@pytest.mark.parametrize("G,dtype,old_stride", [(1, "fp32", 1), (4, "bf16", 1), (1, "fp16", 0), (3, "fp32", 0)])
def test_export_does_not_disturb_the_cache(G, dtype, old_stride):
    """The score update a step leaves pending is applied to the exported copy only: a cache that is exported after
    every step gives bit for bit what one that is exported once does, and an export repeats itself."""
    from paper_2410_23079_amd import FLAG_AUTO_EVICT, FLAG_DETERMINISTIC, BuzzCache
    ls = lockstep()
    wl = small(batch=1, n_kv_heads=3, n_q_heads=3 * G, head_dim=64, dtype=dtype, prompt=300, decode_steps=41,
               sink=4, window=37, segment=16, keep=2, evict_every=16, old_stride=old_stride, n_obs=24)
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    a, b = (BuzzCache(ls.buzz_config(wl, flags=FLAG_AUTO_EVICT | FLAG_DETERMINISTIC)) for _ in range(2))
    out_a, out_b = (torch.empty(wl.batch, wl.n_q_heads, wl.head_dim, dtype=torch.float32, device="cuda") for _ in range(2))
    for c in (a, b):
        c.prefill(p["K"], p["V"], q_obs=p["q_obs"])
    for t in range(wl.decode_steps):
        a.decode_step(d["q"][t], d["k"][t], d["v"][t], out_a)
        b.decode_step(d["q"][t], d["k"][t], d["v"][t], out_b)
        assert torch.equal(out_a, out_b)
        first = b.export()
        for x, y in zip(first, b.export()):
            assert torch.equal(x, y)
    for x, y in zip(a.export(), b.export()):
        assert torch.equal(x, y)


def test_die_local_merge_refuses_blocks_on_an_unexpected_die():
    """The guard of the die-local merge, forced from the host: with a wrong record of which die serves which
    launch-order number every block reports a mismatch and the outputs of the step are NaN, not numbers; the
    kernels run to their end, and with the probe's record restored the cache goes on as if nothing had happened
    (the stored rows and scores never depended on the merge)."""
    from paper_2410_23079_amd import FLAG_AUTO_EVICT, FLAG_DETERMINISTIC, BuzzCache
    ls = lockstep()
    wl = small(batch=1, n_kv_heads=8, n_q_heads=32, head_dim=128, dtype="bf16", prompt=2600, decode_steps=12,
               sink=4, window=1100, segment=16, keep=3, evict_every=16, n_obs=24)
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    a, b = (BuzzCache(ls.buzz_config(wl, flags=FLAG_AUTO_EVICT | FLAG_DETERMINISTIC)) for _ in range(2))
    for c in (a, b):
        c.prefill(p["K"], p["V"], q_obs=p["q_obs"])
    out_a, out_b = (torch.empty(wl.batch, wl.n_q_heads, wl.head_dim, dtype=torch.float32, device="cuda") for _ in range(2))
    for t in range(wl.decode_steps):
        wrong = t in (3, 4)
        b.override_die_map(0x88888888 if wrong else -1)          # die 8 does not exist: no block can match
        a.decode_step(d["q"][t], d["k"][t], d["v"][t], out_a)
        b.decode_step(d["q"][t], d["k"][t], d["v"][t], out_b)
        if wrong:
            assert torch.isnan(out_b).all() and torch.isfinite(out_a).all()
        else:
            assert torch.equal(out_a, out_b)
    for x, y in zip(a.export(), b.export()):
        assert torch.equal(x, y)


@pytest.mark.parametrize("deterministic", [True, False])
@pytest.mark.parametrize("G,dtype", [(1, "bf16"), (4, "fp16"), (2, "fp32")])
def test_more_units_than_compute_units(deterministic, G, dtype):
    """360 units on 256 compute units: one 4-wave block per unit, several blocks per compute unit."""
    wl = small(batch=45, n_kv_heads=8, n_q_heads=8 * G, head_dim=64, dtype=dtype, prompt=300, decode_steps=40,
               sink=2, window=150, segment=8, keep=2, evict_every=8, n_obs=4)
    st = run(wl, units=[(0, 0), (17, 3), (31, 7), (44, 5), (44, 7)], deterministic=deterministic)
    assert st["evictions"] == 5


@pytest.mark.parametrize("dtype,G", [("bf16", 1), ("fp16", 2)])
def test_prefill_scores_from_every_prompt_query(dtype, G):
    """n_obs = N (H2O-style prompt scores) beyond one scoring pass of 4096 queries, ragged tiles everywhere."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=64, dtype=dtype, prompt=4500, decode_steps=8,
               sink=4, window=700, segment=32, keep=3, evict_every=8, n_obs=4500)
    run(wl, units=[(0, 1)])


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_prefill_scores_from_every_prompt_query_wide_rows(dtype):
    """head_dim 256 takes the matrix-core scoring with 32-row chunks; several chunks, blocks and a ragged end."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=4, head_dim=256, dtype=dtype, prompt=1130, decode_steps=4,
               sink=4, window=200, segment=16, keep=2, evict_every=8, n_obs=1130)
    run(wl, units=[(0, 1)])


@pytest.mark.parametrize("dtype,D,G,prompt,n_obs", [
    ("bf16", 128, 4, 1537, 1537), ("fp16", 64, 1, 1025, 1025), ("bf16", 64, 3, 2049, 1), ("fp16", 128, 2, 4097, 257),
    ("bf16", 256, 2, 511, 300), ("fp16", 128, 1, 65, 65),
    ("fp32", 64, 1, 1025, 1025), ("fp32", 64, 3, 2050, 1), ("fp32", 128, 2, 700, 129), ("fp32", 256, 2, 385, 385),
    ("fp32", 64, 1, 4300, 4200), ("fp32", 128, 1, 33, 33)])
def test_prompt_scoring_cut_into_parts(dtype, D, G, prompt, n_obs):
    """Few heads: both scoring steps are cut into several blocks per group of queries / block of keys, with ragged
    last parts, groups of fewer parts than others, one query, one chunk, a second pass; fp32 and 16-bit operands."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=D, dtype=dtype, prompt=prompt, decode_steps=1,
               sink=4, window=prompt // 4, segment=16, keep=2, evict_every=8, n_obs=n_obs)
    run(wl)


@pytest.mark.parametrize("dtype,D,units,G,N,n_obs", [("bf16", 64, 8, 1, 8200, 8200), ("fp16", 128, 12, 1, 9001, 5000),
                                                     ("fp32", 64, 8, 1, 8193, 4097), ("bf16", 256, 6, 2, 6000, 4400),
                                                     ("fp16", 64, 64, 8, 1537, 1), ("bf16", 128, 64, 8, 1600, 100)])
def test_prompt_scoring_cut_into_parts_of_a_pass_and_of_idle_waves(dtype, D, units, G, N, n_obs):
    """More observed queries than one pass takes, few enough heads that every pass is cut: early passes see a part of the
    keys only.  Many heads with a few queries each, whose blocks are cut because they leave waves idle.  The column sums are compared with 64-bit softmax rows; the keys' scores start from the caller's."""
    from paper_2410_23079_amd import BuzzCache, BuzzConfig
    dt = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[dtype]
    g = torch.Generator(device="cuda").manual_seed(N)
    k = torch.randn(1, units, N, D, generator=g, device="cuda").to(dt)
    q = torch.randn(1, units * G, n_obs, D, generator=g, device="cuda").to(dt)
    init = torch.rand(1, units, N, generator=g, device="cuda")
    print(f"[passes] {dtype} D{D} units {units} G{G} N{N} n_obs{n_obs}", flush=True)
    c = BuzzCache(BuzzConfig(1, units * G, units, D, dtype, 0, N, 16, 1, 16, N + 1, old_stride=1))
    c.prefill(k, k, q_obs=q, init_score=init)
    got = c.export()[2][0].double()
    c.prefill(k, k, q_obs=q, init_score=init)
    assert torch.equal(got, c.export()[2][0].double())         # the same bits every time
    at = torch.arange(N - n_obs, N, device="cuda")
    hidden = torch.arange(N, device="cuda")[None, :] > at[:, None]
    for h in range(units):
        want = init[0, h].double()
        for j in range(G):
            s = torch.matmul(q[0, h * G + j].double(), k[0, h].double().t().contiguous()) / D ** 0.5
            want = want + torch.softmax(s.masked_fill_(hidden, -float("inf")), 1).sum(0)
        err = ((got[h] - want).abs() / want.clamp(min=1.0)).max().item()
        assert err <= lockstep().SCORE_TOL, f"head {h}: scores off by {err}"


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("D,G,prompt,n_obs", [(64, 1, 200, 200), (128, 2, 700, 333), (256, 1, 90, 41)])
def test_a_query_that_is_not_a_number_stays_with_the_keys_it_sees(dtype, D, G, prompt, n_obs):
    """One observed query holds a NaN, another an infinity: the scores of every key they see are NaN, those of the keys
    behind them (in the same tiles, too) are what the other queries leave there."""
    from oracle.buzz_oracle import OracleCache
    ls = lockstep()
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=D, dtype=dtype, prompt=prompt, decode_steps=1, sink=4,
               window=prompt // 4, segment=16, keep=2, evict_every=8, n_obs=n_obs)
    p = prompt_inputs(wl, device="cuda")
    p["q_obs"][0, 0, n_obs // 2, 3] = float("nan")
    p["q_obs"][0, G, n_obs // 3, D - 1] = float("inf")
    print(f"[odd queries] {dtype} D{D} G{G} N{prompt} n_obs{n_obs}", flush=True)
    got = ls.gpu_prompt_scores(wl, p, n_obs).double().cpu().numpy()
    units = [(0, 0), (0, 1)]
    o = OracleCache(ls.oracle_config(wl, 2, sink=0, window=prompt + 1, old_stride=1))
    o.prefill(ls.unit_slices(p["K"], units, 1), ls.unit_slices(p["V"], units, 1), q_obs=ls.unit_slices(p["q_obs"], units, G))
    want = o.export()[2][:, 0]
    last = [prompt - n_obs + n_obs // 2, prompt - n_obs + n_obs // 3]         # positions of the two queries
    for h in range(2):
        assert np.isnan(want[h, :last[h] + 1]).all() and np.isfinite(want[h, last[h] + 1:]).all()
    assert ls.score_err(got[0], want) <= ls.SCORE_TOL


@pytest.mark.parametrize("G", [1, 2])
def test_prefill_scores_when_logits_jump(G):
    """Key rows of growing norm late in the prompt: the scaled logits of one query jump by ~20, then by far more
    than 2^7 in log2 units, so a softmax sum taken against an earlier reference overflows single precision and
    the matrix-core scoring has to move its reference (both when the sum grows large and when it is infinite)."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=128, dtype="fp16", prompt=900, decode_steps=6,
               sink=4, window=64, segment=16, keep=2, evict_every=8, n_obs=900)
    p = prompt_inputs(wl, device="cuda")
    d = decode_inputs(wl, device="cuda")
    K = p["K"].float()
    K[:, :, 300:304] *= 20.0
    K[:, :, 520:523] *= 60.0
    K[:, 1, 700:702] *= 200.0
    p["K"] = K.to(p["K"].dtype)
    st = lockstep().run_lockstep(wl, p, d)
    print(f"[parity]   jumping logits G{G}: prefill-score {st['prefill_score']:.2e} out {st['out']:.2e}", flush=True)


@pytest.mark.parametrize("seed", range(48))
def test_random_configurations(seed):
    """Seeded random shapes, cache parameters and variants through the whole lock-step protocol."""
    r = np.random.default_rng(9000 + seed)
    dtype = ["fp32", "fp16", "bf16"][seed % 3]
    D = int(r.choice([64, 128, 256]))
    G = int(r.choice([1, 1, 2, 3, 4, 8]))
    Hkv = int(r.choice([1, 2, 3, 8]))
    B = int(r.choice([1, 2]))
    k, w = int(r.integers(0, 6)), int(r.integers(0, 200))
    s = int(r.integers(1, 40))
    c = int(r.integers(0, 5))
    T = int(r.integers(1, 40))
    old_stride = int(r.choice([1, 1, 0, 2, 3]))
    N = int(r.integers(0, 1500))
    steps = int(r.integers(T + 1, 3 * T + 30))
    variant = seed % 4
    kw = {}
    if variant == 1:
        kw["log_n"] = True
    elif variant == 2 and c > 0:
        kw["global_topk"] = True
        c = int(r.integers(1, 60))
    elif variant == 3:
        kw["interval_new"] = True
    wl = small(batch=B, n_kv_heads=Hkv, n_q_heads=Hkv * G, head_dim=D, dtype=dtype, prompt=N, decode_steps=steps,
               sink=k, window=w, segment=s, keep=c, evict_every=T, old_stride=old_stride, n_obs=min(N, int(r.integers(0, 40))))
    run(wl, deterministic=bool(seed % 2), device_merge=bool((seed // 2) % 2), **kw)


@pytest.mark.parametrize("seed", range(10))
def test_random_long_configurations(seed):
    """The same with long prompts, windows and segments and large keep (several blocks per unit, long segments)."""
    r = np.random.default_rng(770000 + seed)
    dtype = ["fp32", "fp16", "bf16"][seed % 3]
    D = int(r.choice([64, 128, 128, 256]))
    G = int(r.choice([1, 1, 2, 4, 5, 8]))
    Hkv = int(r.choice([1, 2, 4, 8]))
    B = int(r.choice([1, 2, 4]))
    k, w = int(r.integers(0, 9)), int(r.integers(0, 5000))
    s = int(r.integers(1, 300))
    c = int(r.integers(0, 40))
    T = int(r.integers(1, 300))
    old_stride = int(r.choice([1, 1, 1, 0, 2, 5]))
    N = int(r.integers(0, 24000))
    steps = int(min(400, r.integers(T + 1, 2 * T + 40)))
    variant = seed % 5
    kw = {}
    if variant == 1:
        kw["log_n"] = True
    elif variant == 2 and c > 0:
        kw["global_topk"] = True
        c = int(r.integers(1, 600))
    elif variant == 3:
        kw["interval_new"] = True
    wl = small(batch=B, n_kv_heads=Hkv, n_q_heads=Hkv * G, head_dim=D, dtype=dtype, prompt=N, decode_steps=steps,
               sink=k, window=w, segment=s, keep=c, evict_every=T, old_stride=old_stride, n_obs=min(N, int(r.integers(0, 48))))
    run(wl, deterministic=bool(seed % 2), device_merge=bool((seed // 2) % 2), **kw)


@pytest.mark.parametrize("seed", range(10))
def test_random_prompt_scoring(seed):
    """Prompt scores from all or a random number of prompt queries, both scoring paths, random shapes."""
    r = np.random.default_rng(880000 + seed)
    dtype = ["fp16", "bf16", "fp16", "bf16", "fp32"][seed % 5]
    D = int(r.choice([64, 128, 128, 256]))
    G = int(r.choice([1, 2, 4, 8]))
    Hkv = int(r.choice([1, 2, 3]))
    B = int(r.choice([1, 2]))
    N = int(r.integers(1, 1200 if dtype == "fp32" else 5200))
    n_obs = N if seed % 2 == 0 else int(r.integers(0, N + 1))
    k, w = int(r.integers(0, 6)), int(r.integers(0, 600))
    s, c, T = int(r.integers(1, 80)), int(r.integers(0, 6)), int(r.integers(1, 100))
    kw = {"log_n": True} if seed % 3 == 0 else {}
    wl = small(batch=B, n_kv_heads=Hkv, n_q_heads=Hkv * G, head_dim=D, dtype=dtype, prompt=N, decode_steps=3,
               sink=k, window=w, segment=s, keep=c, evict_every=T, old_stride=1, n_obs=n_obs)
    run(wl, **kw)


# ------------------------------------------------------------------ degenerate cases of the method
def test_keep_zero_streaming():
    run(small(prompt=200, decode_steps=40, keep=0, n_obs=8))


def test_keep_covers_segment():
    run(small(prompt=200, decode_steps=40, segment=4, keep=4, evict_every=8, n_obs=8))


def test_no_sink_no_window():
    run(small(prompt=150, decode_steps=30, sink=0, window=0, segment=5, keep=1, evict_every=5, n_obs=8))


def test_prompt_shorter_than_sink_and_window_fill():
    """Remark 1: sink and window fill first; the first eviction happens only after T tokens left the window."""
    run(small(prompt=2, decode_steps=120, sink=4, window=32, segment=8, keep=1, evict_every=8, n_obs=2))


def test_empty_prompt():
    run(small(prompt=0, decode_steps=60, sink=2, window=16, segment=4, keep=1, evict_every=4, n_obs=0))


@pytest.mark.parametrize("keep", [5, 150])
def test_segment_longer_than_wave(keep):
    run(small(prompt=1500, decode_steps=10, sink=4, window=64, segment=200, keep=keep, evict_every=300, n_obs=16))


def test_longest_segment_one_wave_ranks():
    """segment = 4096 (the most one wave ranks): two full segments and a ragged one at prefill, ties broken by index."""
    run(small(prompt=9000, decode_steps=6, sink=4, window=64, segment=4096, keep=9, evict_every=5000, n_obs=16))


def test_keep_larger_than_segment_keeps_everything():
    """A segment cannot yield more rows than it has: keep = 9 on segments of 4 behaves like keep = 4."""
    st = run(small(prompt=200, decode_steps=40, segment=4, keep=9, evict_every=8, n_obs=8))
    assert st["evictions"] == 5


@pytest.mark.parametrize("between", [15, 16, 17])
def test_prompt_with_exactly_T_tokens_between_sink_and_window(between):
    """Alg. 1's first loops: a prompt is sampled as soon as T (= 16) tokens lie between sink and window, not one
    earlier, and a 17th starts a ragged second segment."""
    wl = small(prompt=4 + between + 64, decode_steps=20, n_obs=8)            # k 4, w 64, s 16, T 16
    from paper_2410_23079_amd import BuzzCache
    g = BuzzCache(lockstep().buzz_config(wl, flags=2))                       # dry run: sizes only
    g.prefill(None, None, n_prompt=wl.prompt)
    assert g.lengths() == {15: (83, 0, 15), 16: (69, 1, 0), 17: (70, 2, 0)}[between]
    run(wl)


def plant_odd_scores(ps):
    """NaN, +inf and -inf among the starting scores, several per segment, on every unit."""
    N = ps.shape[-1]
    for j in range(5, N, 7):
        ps[..., j] = float("nan")
    for j in range(9, N, 23):
        ps[..., j] = float("inf")
    for j in range(12, N, 11):
        ps[..., j] = float("-inf")
    ps[..., 40:56] = float("nan")                            # one whole segment of NaN: the lowest indices win


@pytest.mark.parametrize("keep,old_stride", [(1, 1), (3, 1), (2, 0)])
def test_nan_and_infinite_scores_rank_as_stated(keep, old_stride):
    """Alg. 2's argmax on scores that are not numbers: NaN ranks below everything (ties with -inf), +inf above,
    ties go to the lowest index -- at the prefill (separate selection kernel) and in decode evictions (one-launch
    eviction for persistent survivors, selection + gather where old rows are re-sampled)."""
    wl = small(prompt=600, decode_steps=50, sink=4, window=64, segment=16, keep=keep, evict_every=16,
               old_stride=old_stride, n_obs=12)
    st = run(wl, plant=plant_odd_scores)
    assert st["evictions"] == 3


@pytest.mark.parametrize("segment,keep,old_stride", [(1, 1, 1), (5, 2, 1), (63, 7, 1), (64, 64, 1), (65, 9, 0), (131, 70, 1),
                                                      (4093, 3, 1), (4093, 4, 1)])
def test_equal_scores_across_the_survivors_boundary(segment, keep, old_stride):
    """Starting scores of three values only: nearly every segment has equal scores on both sides of its boundary, which
    the lowest indices win; segments of one row to the longest, lengths that are no multiple of four, the LDS limit."""
    def plant(ps):
        ps.copy_(torch.floor(torch.rand(ps.shape, generator=torch.Generator().manual_seed(segment)) * 3.0).to(ps))
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2, head_dim=64, dtype="fp16", prompt=3 * segment + 200, decode_steps=6,
               sink=3, window=40, segment=segment, keep=keep, evict_every=4, old_stride=old_stride, n_obs=0)
    run(wl, plant=plant)


def eviction_time(segment, keep, new, scores, flags=0):
    """Shortest of several explicit evictions (device time, ms) of `new` buffered rows on 32 units."""
    from paper_2410_23079_amd import BuzzCache, BuzzConfig
    H, D, w, old = 32, 64, 64, 1
    n = 4 + old + new + w
    c = BuzzCache(BuzzConfig(1, H, H, D, "fp16", 4, w, segment, keep, max(new, segment) + 8, 4 * n + 4 * segment, old_stride=1, flags=flags))
    k = torch.zeros(1, H, n, D, dtype=torch.float16, device="cuda")
    sc = scores(H, n).to("cuda", torch.float32).contiguous()
    pos = torch.arange(n, dtype=torch.int32, device="cuda").expand(1, H, n).contiguous()
    times = []
    for _ in range(8):
        c.import_rows(k, k, sc, pos, old, n)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        c.evict()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def distinct(H, n):
    return torch.rand(1, H, n, generator=torch.Generator().manual_seed(7))


def test_equal_scores_rank_as_fast_as_distinct_ones():
    """Whatever the scores are, a segment costs one comparison per pair of rows: ranking by a second such pass where equal
    scores straddle the survivors' boundary took 2.8 times as long."""
    some, same = eviction_time(1000, 100, 1000, distinct), eviction_time(1000, 100, 1000, lambda H, n: torch.zeros(1, H, n))
    print(f"[rank] distinct {some * 1e3:.1f} us, equal {same * 1e3:.1f} us", flush=True)
    assert same <= 1.5 * some


def test_few_rows_rank_as_fast_in_a_long_segment_as_in_a_short_one():
    """An explicit eviction (or a ragged last segment) of 100 rows costs what 100 rows cost, whatever the configured
    segment is: ranked against a whole segment of 4000 it took ten times as long."""
    short, long = eviction_time(100, 3, 100, distinct), eviction_time(4000, 3, 100, distinct)
    print(f"[rank] 100 rows in a segment of 100: {short * 1e3:.1f} us, of 4000: {long * 1e3:.1f} us", flush=True)
    assert long <= 2 * short


def test_evictions_that_ignore_the_scores_do_not_rank_them():
    """Interval sampling of the new rows keeps the first rows of every segment: nothing is compared."""
    from paper_2410_23079_amd import FLAG_INTERVAL_NEW
    ranked, first = eviction_time(1000, 100, 1000, distinct), eviction_time(1000, 100, 1000, distinct, FLAG_INTERVAL_NEW)
    print(f"[rank] by score {ranked * 1e3:.1f} us, by index {first * 1e3:.1f} us", flush=True)
    assert first <= 0.5 * ranked


@pytest.mark.parametrize("segment,keep", [(5000, 7), (9000, 300)])
def test_segments_longer_than_one_wave_can_rank(segment, keep):
    """Segments beyond 4096 rows take the block-wide selection (radix select + prefix sum): two full segments and a
    ragged one at prefill, ties everywhere (prompt scores of a short observation window are mostly equal)."""
    run(small(prompt=2 * segment + 1500, decode_steps=4, sink=4, window=64, segment=segment, keep=keep,
              evict_every=segment + 1000, n_obs=16))


@pytest.mark.parametrize("segment,rows,keep,global_topk", [(255, 600, 31, False), (256, 773, 1, False), (256, 773, 255, False), (300, 2999, 40, False),
                                                           (1023, 1023, 100, False), (1025, 1025, 1024, False), (4000, 9000, 3, False),
                                                           (4096, 4096, 9, False), (4097, 4097, 9, False), (16384, 16384, 2000, False),
                                                           (16385, 16385, 2000, False), (32768, 32768, 40, False), (32769, 32769, 4000, False), (64, 40001, 5000, True),
                                                           (64, 257, 200, True)])
@pytest.mark.parametrize("values", ["distinct", "three", "equal", "odd"])
def test_selection_of_long_segments(segment, rows, keep, global_topk, values):
    """Whole segments, remainders and the lengths at which the selection changes its kernel or the place of its keys,
    against a stable sort on the CPU: score descending, ties to the lowest index, NaN lowest, -0 equal to +0."""
    from paper_2410_23079_amd import FLAG_GLOBAL_TOPK, BuzzCache, BuzzConfig
    print(f"[selection] segment {segment} rows {rows} keep {keep} global {global_topk} {values}", flush=True)
    sink, window, units, D, N = 3, 7, 2, 64, rows + 10
    g = torch.Generator().manual_seed(segment + rows)
    score = torch.exp(torch.randn(1, units, N, generator=g))
    if values == "three":
        score = torch.floor(torch.rand(1, units, N, generator=g) * 3.0)
    elif values == "equal":
        score = torch.full((1, units, N), -2.5)
    elif values == "odd":
        odd = torch.tensor([float("nan"), float("inf"), -float("inf"), 0.0, -0.0, -1.0, 1e-40, -1e-40])
        score = odd[torch.randint(0, 8, (1, units, N), generator=g)]
    k = torch.randn(1, units, N, D, generator=g).to("cuda", torch.bfloat16)
    c = BuzzCache(BuzzConfig(1, units, units, D, "bf16", sink, window, segment, keep, rows, N, old_stride=1,
                             flags=FLAG_GLOBAL_TOPK if global_topk else 0))
    c.prefill(k, k, init_score=score.cuda())
    K, _, _, pos = c.export()
    s = score.double()
    s = torch.where(s.isnan(), torch.full_like(s, -float("inf")), s)[0]
    step, want = rows if global_topk else segment, []
    for u in range(units):
        kept = list(range(sink))
        for lo in range(sink, sink + rows, step):
            hi = min(lo + step, sink + rows)
            kept += sorted((torch.sort(s[u, lo:hi], descending=True, stable=True).indices[:keep] + lo).tolist())
        want.append(kept + list(range(N - window, N)))
    want = torch.tensor(want, dtype=torch.int32)
    assert torch.equal(pos[0].cpu(), want)
    assert torch.equal(K[0], torch.gather(k[0], 1, want.long().cuda()[..., None].expand(-1, -1, D)))


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("fp16", 128), ("fp32", 256)])
@pytest.mark.parametrize("units,segment,keep,rows,window", [(1, 16, 1, 16, 0), (3, 16, 2, 331, 5), (2, 64, 8, 1000, 70), (1, 64, 16, 64, 1),
                                                            (5, 7, 7, 100, 16), (2, 250, 5, 777, 300), (40, 5, 1, 2003, 9), (2, 64, 33, 640, 33)])
@pytest.mark.parametrize("scored", [True, False])
def test_sampled_prompts_are_placed_in_one_launch_or_two(dtype, D, units, segment, keep, rows, window, scored):
    """Either way of the rule, at its edges: rows, scores and positions against a stable sort on the CPU, from a workspace
    that holds garbage; without scores the first rows of a segment survive."""
    from paper_2410_23079_amd import BuzzCache, BuzzConfig
    print(f"[sampled] {dtype} D{D} units{units} s{segment} c{keep} rows{rows} w{window} scored{scored}", flush=True)
    sink, N = 2, 2 + rows + window
    g = torch.Generator().manual_seed(segment * 1000 + rows + D)
    score = torch.floor(torch.randn(1, units, N, generator=g) * 8.0)
    dt = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[dtype]
    k, v = (torch.randn(1, units, N, D, generator=g).to("cuda", dt) for _ in range(2))
    c = BuzzCache(BuzzConfig(1, units, units, D, dtype, sink, window, segment, keep, rows, N + 4, old_stride=1))
    c.workspace.fill_(0xFF)
    c.prefill(k, v, init_score=score.cuda() if scored else None)
    K, V, S, pos = c.export()
    want = []
    for u in range(units):
        kept = list(range(sink))
        for lo in range(sink, sink + rows, segment):
            s = score[0, u, lo:min(lo + segment, sink + rows)] if scored else torch.zeros(min(segment, sink + rows - lo))
            kept += sorted((torch.sort(s, descending=True, stable=True).indices[:keep] + lo).tolist())
        want.append(kept + list(range(N - window, N)))
    want = torch.tensor(want)
    assert torch.equal(pos[0].cpu(), want.int())
    at = want.cuda()[..., None].expand(-1, -1, D)
    assert torch.equal(K[0], torch.gather(k[0], 1, at)) and torch.equal(V[0], torch.gather(v[0], 1, at))
    assert torch.equal(S[0].cpu(), torch.gather(score[0], 1, want) if scored else torch.zeros_like(want, dtype=torch.float32))
    out, q = torch.empty(1, units, D, device="cuda"), torch.randn(1, units, D, generator=g).to("cuda", dt)
    c.decode_step(q, q, q, out)                              # the arrival counters are clear
    Ka, Va = (torch.cat([x[0].double(), q[0, :, None].double()], 1) for x in (K, V))
    p = torch.softmax(torch.matmul(Ka, q[0, :, :, None].double())[..., 0] / D ** 0.5, -1)
    o = torch.matmul(p[:, None], Va)[:, 0]
    assert float((out[0] - o).abs().max() / o.abs().max()) < 1e-4


@pytest.mark.parametrize("segment,keep,rows", [(300, 40, 2999), (1000, 1000, 1500), (4097, 9, 9000), (5000, 600, 5003), (64, 5000, 40001)])
@pytest.mark.parametrize("why", ["no scores", "interval", "global"])
def test_long_segments_without_scores_keep_their_first_rows(segment, keep, rows, why):
    from paper_2410_23079_amd import FLAG_GLOBAL_TOPK, FLAG_INTERVAL_NEW, BuzzCache, BuzzConfig
    print(f"[first rows] segment {segment} keep {keep} rows {rows} {why}", flush=True)
    sink, window, units, D, N = 3, 7, 3, 64, rows + 10
    g = torch.Generator(device="cuda").manual_seed(rows)
    k = torch.randn(1, units, N, D, device="cuda", generator=g).to(torch.bfloat16)
    score = torch.randn(1, units, N, device="cuda", generator=g)
    c = BuzzCache(BuzzConfig(1, units, units, D, "bf16", sink, window, segment, keep, rows, N, old_stride=1,
                             flags={"global": FLAG_GLOBAL_TOPK, "interval": FLAG_INTERVAL_NEW}.get(why, 0)))
    c.workspace.fill_(0xFF)
    c.prefill(k, k, init_score=score if why == "interval" else None)
    K, _, S, pos = c.export()
    step = rows if why == "global" else segment
    kept = [r for lo in range(sink, sink + rows, step) for r in range(lo, min(lo + min(keep, step), sink + rows))]
    want = torch.tensor(list(range(sink)) + kept + list(range(N - window, N)), device="cuda")
    assert torch.equal(pos, want.int().expand(1, units, -1))
    assert torch.equal(K, k[:, :, want]) and torch.equal(S, score[:, :, want] if why == "interval" else torch.zeros_like(S))


def test_prompts_without_scores_are_not_ranked():
    """Such a prompt costs a fraction of one whose equal scores are compared: the same rows, 27 us against 66 when
    measured; a block-wide search of the keys that are all equal took 64."""
    from paper_2410_23079_amd import BuzzCache, BuzzConfig
    units, N, D = 32, 32768, 128
    k = torch.randn(1, units, N, D, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    c = BuzzCache(BuzzConfig(1, units, units, D, "bf16", 4, 64, 512, 64, 512, N, old_stride=1))
    best = {}
    for name, score in (("none", None), ("equal", torch.zeros(1, units, N, device="cuda"))) * 3:
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        c.prefill(k, k, init_score=score)
        a.record()
        for _ in range(20):
            c.prefill(k, k, init_score=score)
        b.record()
        b.synchronize()
        best[name] = min(best.get(name, 1e9), a.elapsed_time(b) / 20)
    print(f"[prefill] without scores {best['none'] * 1e3:.1f} us, equal scores {best['equal'] * 1e3:.1f} us", flush=True)
    assert best["none"] <= 0.7 * best["equal"]


def test_long_segments_with_nan_and_infinite_scores():
    st = run(small(prompt=11000, decode_steps=4, sink=4, window=64, segment=5000, keep=40, evict_every=6000, n_obs=12),
             plant=plant_odd_scores)
    assert st["evictions"] == 0                                  # everything happens in the prefill's selection


@pytest.mark.parametrize("prompt,keep,G,dtype", [(700, 40, 1, "fp32"), (9000, 500, 1, "fp16"), (9000, 5000, 4, "bf16")])
def test_global_topk_h2o_style(prompt, keep, G, dtype):
    """Sec. 4.1's H2O baseline as a variant: the top `keep` accumulated scores among all rows between sink and
    window survive every eviction (short middle: one wave ranks it; long middle: the block-wide selection)."""
    wl = small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=64, dtype=dtype, prompt=prompt, decode_steps=40,
               sink=4, window=64, segment=16, keep=keep, evict_every=16, n_obs=24)
    st = run(wl, global_topk=True)
    assert st["evictions"] == 2


def test_global_topk_with_odd_scores():
    wl = small(prompt=600, decode_steps=40, sink=4, window=64, segment=16, keep=30, evict_every=16, n_obs=12)
    run(wl, global_topk=True, plant=plant_odd_scores)


def test_unbuffered_eviction_every_step():
    run(small(prompt=100, decode_steps=50, sink=2, window=20, segment=3, keep=1, evict_every=1, n_obs=4))


def test_capacity_error_when_eviction_is_skipped():
    from paper_2410_23079_amd import BuzzCache, BuzzError
    ls = lockstep()
    wl = small(prompt=100, decode_steps=64, sink=2, window=20, segment=4, keep=1, evict_every=4)
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    c = BuzzCache(ls.buzz_config(wl, flags=0))
    c.prefill(p["K"], p["V"])
    out = torch.empty(wl.batch, wl.n_q_heads, wl.head_dim, dtype=torch.float32, device="cuda")
    for t in range(4):
        c.decode_step(d["q"][t], d["k"][t], d["v"][t], out)
    before = c.lengths()
    with pytest.raises(BuzzError) as e:
        c.decode_step(d["q"][4], d["k"][4], d["v"][4], out)
    assert e.value.code == -2 and c.lengths() == before        # failed call left the cache unchanged
    c.evict()
    c.decode_step(d["q"][4], d["k"][4], d["v"][4], out)
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype,D", [("fp32", 64), ("fp32", 256), ("bf16", 64), ("fp16", 128), ("bf16", 256)])
@pytest.mark.parametrize("units,G,N,n_obs,sink", [(1, 1, 1, 1, 4), (2, 3, 64, 1, 0), (3, 1, 65, 65, 4), (8, 2, 257, 257, 300), (2, 2, 1000, 130, 4),
                                                  (1, 1, 4200, 4200, 1)])
def test_a_scored_prompt_that_is_kept_whole_is_placed_by_the_scoring(dtype, D, units, G, N, n_obs, sink):
    """Rows and positions bit-exact, scores against 64-bit column sums, and a decode step on the cache: the workspace
    holds garbage before, so whatever the placement leaves out shows.  Bars: scores 1e-5 of their norm (32-bit sums), outputs 1e-4."""
    from paper_2410_23079_amd import BuzzCache, BuzzConfig
    print(f"[placement] {dtype} D{D} units{units} G{G} N{N} n_obs{n_obs} sink{sink}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N * 7 + D)
    dt = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[dtype]
    k, v, q, kn, vn, qn = (torch.randn(*shape, D, generator=g, device="cuda").to(dt) for shape in
                           ((1, units, N), (1, units, N), (1, units * G, n_obs), (1, units), (1, units), (1, units * G)))
    c = BuzzCache(BuzzConfig(1, units * G, units, D, dtype, sink, 16, 16, 1, N + 16, N + 8, old_stride=1))
    c.workspace.fill_(0xFF)
    c.prefill(k, v, q_obs=q)
    K, V, score, pos = c.export()
    assert torch.equal(K, k) and torch.equal(V, v)
    assert torch.equal(pos, torch.arange(N, device="cuda", dtype=torch.int32).expand(1, units, N))
    s = torch.matmul(q.double().view(units, G * n_obs, D), k[0].double().transpose(1, 2).contiguous()) / D ** 0.5
    at = torch.arange(N - n_obs, N, device="cuda").repeat(G)
    s.masked_fill_(torch.arange(N, device="cuda")[None] > at[:, None], -float("inf"))
    ref = torch.softmax(s, -1).sum(1)
    assert float((score[0] - ref).norm() / ref.norm()) < 1e-5
    out = torch.empty(1, units * G, D, device="cuda")
    for _ in range(2):                                       # the second step finds the counters as the first left them
        c.decode_step(qn, kn, vn, out)
    Ka, Va = (torch.cat([x[0].double(), y[0, :, None].double(), y[0, :, None].double()], 1) for x, y in ((k, kn), (v, vn)))
    p = torch.softmax(torch.matmul(qn.double().view(units, G, D), Ka.transpose(1, 2).contiguous()) / D ** 0.5, -1)
    want = torch.matmul(p, Va).view(1, units * G, D)
    assert float((out - want).abs().max() / want.abs().max()) < 1e-4


@pytest.mark.parametrize("dtype,D,units,G,N,n_obs,sink", [("bf16", 64, 2, 3, 771, 300, 4), ("fp32", 128, 3, 1, 1999, 1999, 0), ("fp16", 256, 5, 2, 515, 250, 4),
                                                          ("fp32", 256, 2, 5, 130, 129, 1), ("bf16", 128, 64, 1, 400, 3, 4), ("bf16", 256, 70, 1, 300, 2, 0),
                                                          ("fp32", 256, 66, 2, 257, 40, 4), ("fp32", 64, 130, 1, 129, 1, 4)])
def test_value_rows_of_a_scored_prompt_are_shared_by_the_parts(dtype, D, units, G, N, n_obs, sink):
    """Steps cut into few and into many parts, more parts than pieces per thread, and whole ones: every row arrives."""
    test_a_scored_prompt_that_is_kept_whole_is_placed_by_the_scoring(dtype, D, units, G, N, n_obs, sink)


@pytest.mark.parametrize("dtype,D,units,G,N,n_obs", [("bf16", 256, 4, 2, 3000, 500), ("bf16", 256, 4, 2, 2000, 256), ("fp32", 128, 8, 2, 700, 256),
                                                     ("bf16", 128, 32, 2, 700, 256)])
def test_placing_a_prompt_under_its_scoring_costs_less_than_copying_it(dtype, D, units, G, N, n_obs):
    """The same prompt, scored, all of its rows kept: placed by the scoring, or by a launch of its own (interval sampling
    that keeps whole segments).  The former saves two launches, 11 to 16% of the call when measured; with the value rows in the
    hands of few blocks it took 6% less to 12% more."""
    from paper_2410_23079_amd import FLAG_INTERVAL_NEW, BuzzCache, BuzzConfig
    dt = {"fp32": torch.float32, "bf16": torch.bfloat16}[dtype]
    k, v = (torch.randn(1, units, N, D, device="cuda").to(dt) for _ in range(2))
    q = torch.randn(1, units * G, n_obs, D, device="cuda").to(dt)
    caches = {name: BuzzCache(BuzzConfig(1, units * G, units, D, dtype, 4, 16, 64, 64, T, N + 8, old_stride=1, flags=FLAG_INTERVAL_NEW))
              for name, T in (("placed", N), ("copied", N - 64))}
    best = {}
    for name in ("placed", "copied") * 5:
        c, a, b = caches[name], torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        c.prefill(k, v, q_obs=q)
        assert c.lengths()[0] == N
        a.record()
        for _ in range(30):
            c.prefill(k, v, q_obs=q)
        b.record()
        b.synchronize()
        best[name] = min(best.get(name, 1e9), a.elapsed_time(b) / 30)
    print(f"[placement] {dtype} D{D} units{units} N{N}: {best['placed'] * 1e3:.1f} us, copied {best['copied'] * 1e3:.1f} us", flush=True)
    assert best["placed"] <= 0.93 * best["copied"]


def test_log_n_scale_argument():
    """Sec. 3.5: the log-n variant only changes the softmax scale, which is a configuration argument."""
    import math
    ls = lockstep()
    wl = small(prompt=300, decode_steps=20, n_obs=8)
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    scale = math.log(812) / math.log(512) / math.sqrt(wl.head_dim)
    from oracle.buzz_oracle import OracleCache
    from paper_2410_23079_amd import BuzzCache
    units = [(0, h) for h in range(wl.n_kv_heads)]
    g = BuzzCache(ls.buzz_config(wl, softmax_scale=scale))
    o = OracleCache(ls.oracle_config(wl, len(units), softmax_scale=scale, auto_evict=True))
    g.prefill(p["K"], p["V"])
    o.prefill(ls.unit_slices(p["K"], units, 1), ls.unit_slices(p["V"], units, 1))
    out = torch.empty(wl.batch, wl.n_q_heads, wl.head_dim, dtype=torch.float32, device="cuda")
    for t in range(3):                                           # no eviction yet: scores cannot reorder anything
        g.decode_step(d["q"][t], d["k"][t], d["v"][t], out)
        ref = o.decode_step(ls.unit_slices(d["q"][t], units, 1), ls.unit_slices(d["k"][t], units, 1),
                            ls.unit_slices(d["v"][t], units, 1))
        assert ls.rel_err(ls.unit_slices(out, units, 1), ref) <= ls.OUT_EXPECT


# ------------------------------------------------------------------ variants named by the paper
def test_log_n_scaled_attention_tracks_context_length():
    """Sec. 3.5: scale = log_512(n)/sqrt(d) with n = tokens the query sees, prompt scoring included."""
    run(small(prompt=480, decode_steps=64, n_obs=24), log_n=True)          # crosses n = 512


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_log_n_prompt_scores_from_the_first_query_on(dtype):
    """Sec. 3.5 at n = 1: log_512(1) = 0, the first prompt query attends uniformly (to its one visible key)."""
    run(small(batch=1, n_kv_heads=2, n_q_heads=4, head_dim=128, dtype=dtype, prompt=330, decode_steps=12,
              sink=4, window=64, segment=16, keep=2, evict_every=8, n_obs=330), log_n=True)


@pytest.mark.parametrize("G,dtype", [(1, "fp32"), (4, "bf16")])
def test_log_n_from_an_empty_cache(G, dtype):
    """Sec. 3.5 during decode at n = 1, 2, ...: the scale starts at 0 and grows with the tracked length."""
    run(small(batch=1, n_kv_heads=2, n_q_heads=2 * G, head_dim=128, dtype=dtype, prompt=0, decode_steps=70,
              sink=2, window=16, segment=4, keep=1, evict_every=4, n_obs=0), log_n=True)


def test_log_n_with_grouped_queries():
    run(small(batch=1, n_kv_heads=2, n_q_heads=8, head_dim=128, dtype="bf16", prompt=600, decode_steps=40,
              sink=4, window=64, segment=16, keep=2, evict_every=16, n_obs=20), log_n=True)


def test_threshold_bounds_old_plus_new_with_theorem_parameters():
    """The proof's reading of T, with T from the Parameter Estimation theorem (s = 5: T/w = 4.33)."""
    from paper_2410_23079_amd import suggest_threshold
    w, s = 24, 5
    T = suggest_threshold(s, w)
    assert T == round(w * 26 / 6)
    wl = small(prompt=400, decode_steps=260, sink=2, window=w, segment=s, keep=1, evict_every=T, old_stride=0, n_obs=16)
    st = run(wl, threshold_total=True, capacity=wl.sink + w + 2 * T)
    assert st["evictions"] >= 3
    st = run(wl, threshold_total=True)                   # Remark 2's own container: T + k + w rows, no capacity given
    assert st["evictions"] >= 3


def test_interval_sampling_of_new_tokens():
    """Ablation of Sec. 4.3 without the local-max function."""
    run(small(prompt=300, decode_steps=48, keep=2), interval_new=True)


def objective_table(wl, tag):
    """Mean |O^ - O| / |O| over the decode steps (the eviction objective of Sec. 3.1, O = full attention written
    out with torch in float64) for BUZZ, the two ablations of Sec. 4.3 and the baselines of Sec. 4.1 as variants of
    this library: H2O-style (global top-k of accumulated scores) and sink + window, the last two also with the
    budget BUZZ ends up with (H2O-style: keep = BUZZ's final survivor count; sink + window: the window widened by
    it).  Returns {variant: (deviation, retained rows at the end)}."""
    import math
    from paper_2410_23079_amd import FLAG_AUTO_EVICT, FLAG_GLOBAL_TOPK, FLAG_INTERVAL_NEW, BuzzCache
    ls = lockstep()
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    steps, N, G = wl.decode_steps, wl.prompt, wl.group
    Kall = torch.cat([p["K"], d["k"].permute(1, 2, 0, 3)], dim=2).double().repeat_interleave(G, dim=1)   # [B,Hq,N+steps,D]
    Vall = torch.cat([p["V"], d["v"].permute(1, 2, 0, 3)], dim=2).double().repeat_interleave(G, dim=1)
    full = []
    for t in range(steps):
        n = N + t + 1
        lg = torch.einsum("bhd,bhnd->bhn", d["q"][t].double(), Kall[:, :, :n]) / math.sqrt(wl.head_dim)
        full.append(torch.einsum("bhn,bhnd->bhd", torch.softmax(lg, dim=-1), Vall[:, :, :n]))

    def deviation(flags=0, **over):
        cfg = ls.buzz_config(wl, flags=FLAG_AUTO_EVICT | flags, **over)
        c = BuzzCache(cfg)
        c.prefill(p["K"], p["V"], q_obs=p["q_obs"])
        out = torch.empty(wl.batch, wl.n_q_heads, wl.head_dim, dtype=torch.float32, device="cuda")
        dev = 0.0
        for t in range(steps):
            c.decode_step(d["q"][t], d["k"][t], d["v"][t], out)
            dev += float(((out.double() - full[t]).norm(dim=-1) / full[t].norm(dim=-1)).mean())
        rows = c.lengths()[0]
        c.close()
        return dev / steps, rows

    res = {"BUZZ": deviation()}
    budget = res["BUZZ"][1] - wl.sink - wl.window             # survivors (and buffered rows) BUZZ ends with
    res["no local max"] = deviation(FLAG_INTERVAL_NEW)
    res["swapped strides"] = deviation(segment=(wl.segment + 1) // 2, old_stride=wl.segment)
    res["H2O-style, same budget"] = deviation(FLAG_GLOBAL_TOPK, keep=budget)
    res["sink + window, same budget"] = deviation(keep=0, window=wl.window + budget)
    res["sink + window"] = deviation(keep=0)
    print(f"[objective, {tag}] mean |O^ - O| / |O| (retained rows): "
          + "; ".join(f"{k} {v[0]:.4f} ({v[1]})" for k, v in res.items()), flush=True)
    return res


def test_objective_on_clustered_keys():
    """The objective on config 5's recipe (keys and queries around 50 topic means per head), scaled down.  Heavy
    hitters are query-dependent there, so only the weakest claims are asserted: segment winners beat keeping
    nothing but sink and window, at the small budget and at BUZZ's own."""
    wl = small("long131k", batch=1, n_kv_heads=4, n_q_heads=4, head_dim=128, dtype="bf16", prompt=4096, decode_steps=64,
               sink=4, window=256, segment=32, keep=4, evict_every=32, n_obs=256)
    res = objective_table(wl, "clustered keys")
    assert res["BUZZ"][0] < res["sink + window"][0]
    assert res["BUZZ"][1] == res["no local max"][1]
    assert abs(res["H2O-style, same budget"][1] - res["BUZZ"][1]) <= wl.evict_every
    assert abs(res["sink + window, same budget"][1] - res["BUZZ"][1]) <= wl.evict_every


def test_local_max_beats_the_ablations_on_the_papers_objective():
    """Sec. 3.1 states the goal as keeping the evicted cache's attention output close to the full one.
    On synthetic keys with planted heavy hitters, at one cache budget, BUZZ's output must be closer to full
    attention than the no-local-max ablation and than sink + window (Sec. 4.3 reports the same ordering in ROUGE,
    which needs the trained model and is not reproduced here).  The H2O-style baseline is reported at the same
    budget; no order between it and BUZZ is asserted (planted keys are heavy for every query, which is the case
    greedy global selection is made for; the paper's case against it rests on the structure of natural text)."""
    wl = small(batch=2, n_kv_heads=4, n_q_heads=4, head_dim=64, dtype="fp32", prompt=2048, decode_steps=128,
               sink=4, window=128, segment=16, keep=1, evict_every=16, n_obs=256, planted_frac=0.04)
    res = objective_table(wl, "planted heavy keys")
    assert res["BUZZ"][1] == res["no local max"][1]
    assert res["BUZZ"][0] < res["no local max"][0] < res["sink + window"][0]
    assert res["BUZZ"][0] < res["sink + window, same budget"][0]
    assert abs(res["H2O-style, same budget"][1] - res["BUZZ"][1]) <= wl.evict_every


@pytest.mark.parametrize("name,kw", [("tiny", {}), ("llama7b_layer", dict(batch=1, n_kv_heads=4, n_q_heads=4, decode_steps=256))])
def test_free_run_parts_only_at_near_ties(name, kw):
    """GPU (fp32 scores) and oracle (fp64 scores) evicting on their own scores keep the same rows, or part at a
    near-tie (relative score gap below 1e-5)."""
    wl = small(name, **kw)
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    res = lockstep().run_free(wl, p, d)
    print(f"[free run] {wl.name}: {res['agreed']} evictions agreed, parted at step {res['parted_at']}, "
          f"largest gap {res['gap']:.2e}", flush=True)
    # either every eviction of the run agreed (16 for config 1, 8 for the slice of config 2; what these seeds
    # give), or the runs parted at a near-tie, which run_free has verified row by row
    if res["parted_at"] is None:
        assert res["agreed"] == wl.decode_steps // wl.evict_every
    else:
        assert res["gap"] <= 1e-5


def test_default_and_deterministic_modes_agree_over_many_steps():
    """Config 4's shape (eight blocks per unit merge through device memory in every launch), 10 240 steps with
    evictions: a cache in the default mode and one in the deterministic mode stay within rounding of each other.
    (A merge that ran ahead of a partial showed up about once in 10^5 launches before the publishing waves
    waited for their own stores.)"""
    from paper_2410_23079_amd import FLAG_AUTO_EVICT, FLAG_DETERMINISTIC, FLAG_DEVICE_MERGE, BuzzCache
    ls = lockstep()
    wl = get_workload("gqa8b_layer")
    p, d = prompt_inputs(wl, device="cuda"), decode_inputs(wl, device="cuda")
    steps = wl.decode_steps
    # the first cache merges a unit's splits through one die's L2, the second through device memory
    caches = [BuzzCache(ls.buzz_config(wl, flags=FLAG_AUTO_EVICT | f, max_context=wl.prompt + steps + 1))
              for f in (0, FLAG_DETERMINISTIC | FLAG_DEVICE_MERGE)]
    outs = [torch.empty(wl.batch, wl.n_q_heads, wl.head_dim, dtype=torch.float32, device="cuda") for _ in caches]
    worst = torch.zeros((), device="cuda")
    for _ in range(10240 // steps):
        for c in caches:
            c.prefill(p["K"], p["V"], q_obs=p["q_obs"])
        for t in range(steps):
            for c, o in zip(caches, outs):
                c.decode_step(d["q"][t], d["k"][t], d["v"][t], o)
            worst = torch.maximum(worst, (outs[0] - outs[1]).abs().amax() / outs[1].abs().amax())
        assert caches[0].lengths() == caches[1].lengths()
    print(f"[parity]   default vs deterministic over 10240 steps: worst relative difference {float(worst):.2e}", flush=True)
    assert float(worst) < 1e-4


# ------------------------------------------------------------------ full-size configs, sampled units
def sampled_units(wl, count, seed):
    r = np.random.default_rng(seed)
    flat = r.choice(wl.batch * wl.n_kv_heads, size=min(count, wl.batch * wl.n_kv_heads), replace=False)
    return sorted((int(u) // wl.n_kv_heads, int(u) % wl.n_kv_heads) for u in flat)


def test_llama7b_layer_full_size():
    wl = get_workload("llama7b_layer")
    st = run(wl, units=sampled_units(wl, 6, 2), deterministic=False)
    assert st["evictions"] == 512 // 32


@pytest.mark.parametrize("device_merge", [False, True])
def test_gqa8b_layer_full_size(device_merge):
    """Config 4 at full size against the oracle: eight blocks per unit merge in every launch, through one die's
    L2 (default) or through device memory."""
    wl = get_workload("gqa8b_layer").scaled(decode_steps=130)
    st = run(wl, units=sampled_units(wl, 3, 4), check_auto=False, deterministic=False, device_merge=device_merge)
    assert st["evictions"] == 2


def test_long131k_full_size():
    wl = get_workload("long131k").scaled(decode_steps=130)
    st = run(wl, units=sampled_units(wl, 2, 5), check_auto=False, deterministic=False)
    assert st["evictions"] == 1


def test_llama7b_full_one_layer_full_size():
    wl = get_workload("llama7b_full").scaled(decode_steps=66)
    st = run(wl, units=sampled_units(wl, 3, 3), check_auto=False, deterministic=False)
    assert st["evictions"] == 1


def test_paper_parameters_full_size():
    """Config 2's shape with the paper's parameterisation (s = 5, s^ = 3, T from the theorem, bounding old + new)."""
    wl = get_workload("llama7b_layer_paper").scaled(decode_steps=360)
    st = run(wl, units=sampled_units(wl, 4, 6), check_auto=False, deterministic=False)
    assert st["evictions"] == 1
