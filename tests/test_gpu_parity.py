"""GPU parity: the HIP library (through its C ABI) against the CPU oracle, element by element.

Tolerances (max|y - ref| / max|ref| per layer): fp32 1e-5, fp16 2e-2, integer paths bit-exact."""
import numpy as np
import pytest

from paper_2112_15445_amd import binding as B
from paper_2112_15445_amd import workloads as wl

import gpu_util as G

pytestmark = pytest.mark.gpu

DT = ["f32", "f16", "i8", "cb4", "cb4h"]


def _both_variants(plan):
    """Yield a label for every kernel family that can run this plan (after installing it)."""
    for variant, extra in ((B.SC_VARIANT_GATHER, {}), (B.SC_VARIANT_SLAB, {"wsrc": 0}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1}), (B.SC_VARIANT_SLAB, {"wsrc": 2}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 3}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 3, "pipeline": 1, "wg_threads": 512}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 1, "wg_threads": 512, "chunk_c": 5,
                                                "tile_q": 128}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 1, "wg_threads": 256, "chunk_c": 8,
                                                "tile_d": 4, "tile_q": 64, "producers": 1}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 1, "wg_threads": 512, "producers": 1}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 2, "pipeline": 1, "wg_threads": 512, "producers": 4}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 2, "wg_threads": 256}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 3, "tile_d": 4, "wg_threads": 128, "tile_p": 2,
                                                "tile_q": 1000}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 3, "tile_d": 4, "wg_threads": 256, "tile_p": 3,
                                                "tile_q": 16, "sub_batch": 2}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 2, "wg_threads": 128, "tile_p": 4,
                                                "tile_q": 8, "sub_batch": 3}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 3, "chunk_c": 2, "wg_threads": 256}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 3, "chunk_c": 3, "tile_d": 4, "wg_threads": 128, "tile_p": 2,
                                                "tile_q": 1000}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 3, "chunk_c": 3, "tile_d": 4, "wg_threads": 256, "tile_p": 3,
                                                "tile_q": 16, "sub_batch": 2}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 2, "wg_threads": 256, "pack": 1}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 3, "tile_d": 4, "wg_threads": 128, "tile_p": 2,
                                                "tile_q": 1000, "pack": 1}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 64, "tile_d": 3, "wg_threads": 64, "tile_p": 5,
                                                "tile_q": 37, "pack": 1}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 1, "wg_threads": 512, "chunk_c": 5,
                                                "tile_q": 128, "pack": 1}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 2, "wg_threads": 192, "chunk_c": 7,
                                                "tile_q": 64, "tile_d": 5, "pack": 1}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 2, "wg_threads": 256, "pack": 2}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "chunk_c": 3, "tile_d": 4, "wg_threads": 128, "tile_p": 2,
                                                "tile_q": 1000, "pack": 2}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 1, "wg_threads": 512, "chunk_c": 5,
                                                "tile_q": 128, "pack": 2}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 2, "wg_threads": 192, "chunk_c": 7,
                                                "tile_q": 64, "tile_d": 5, "pack": 2}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 2, "wg_threads": 1024}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 2, "wg_threads": 192, "tile_q": 64}),
                           (B.SC_VARIANT_SLAB, {"wsrc": 1, "pipeline": 2, "wg_threads": 448, "tile_q": 96}),
                           (B.SC_VARIANT_DENSE, {}),
                           (B.SC_VARIANT_DENSE, {"tile_d": 32, "tile_p": 1, "wg_per_cu": 4, "waves_m": 1}),
                           (B.SC_VARIANT_DENSE, {"tile_d": 32, "tile_p": 2, "chunk_c": 64}),
                           (B.SC_VARIANT_DENSE, {"tile_d": 64, "tile_p": 1000, "sub_batch": 2}),
                           (B.SC_VARIANT_DENSE, {"tile_d": 128, "tile_p": 3, "wg_per_cu": 1})):
        try:
            plan.set_tuning(B.sc_tuning_t(), variant=variant, **extra)
        except B.SparseConvError as e:
            assert e.status == 4      # does not fit / not available for this dtype
            continue
        yield f"variant={variant} {extra}"


@pytest.mark.parametrize("dtype", DT)
def test_config1_layer(dtype):
    (l,) = wl.config1()
    l = l.replace(dtype=dtype)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    assert plan.info().n == 58
    for label in _both_variants(plan):
        print("case", l.name, dtype, label, flush=True)
        G.check(l, G.run_gpu(plan, data["x"]), ref, label)


def test_stretch_pass_offsets_match_oracle():
    import oracle
    for l in (wl.config1()[0], wl.Layer("t", 5, 7, 9, 11, 3, 2, 2, 1, 1, 2, N=1, sparsity=0.5)):
        data = wl.prepare(l, ragged=True)
        st = oracle.sparse_conv_steps(data["x"], data["rowptr"], data["colidx"], data["values"], l.R,
                                      l.S, (l.stride_h, l.stride_w), (l.pad_h, l.pad_w))
        plan = G.make_plan(l, data)
        lam = plan.debug_offsets()
        assert lam.shape == st["lam"].shape and np.array_equal(lam, st["lam"])


SHAPES = [
    # name, C, D, H, W, R, S, sh, sw, ph, pw, N, sparsity
    ("odd_3x3", 5, 7, 13, 11, 3, 3, 1, 1, 1, 1, 3, 0.6),
    ("stride2_3x3", 6, 5, 14, 15, 3, 3, 2, 2, 1, 1, 2, 0.7),
    ("stride2_nopad", 4, 6, 9, 10, 3, 3, 2, 2, 0, 0, 2, 0.5),
    ("pad2_5x5", 3, 4, 8, 9, 5, 5, 1, 1, 2, 2, 2, 0.8),
    ("rect_filter", 4, 5, 10, 12, 2, 3, 1, 2, 0, 1, 2, 0.5),
    ("pointwise", 24, 10, 7, 9, 1, 1, 1, 1, 0, 0, 3, 0.7),
    ("pointwise_vec", 16, 12, 8, 8, 1, 1, 1, 1, 0, 0, 2, 0.6),
    ("pointwise_s2", 8, 6, 9, 9, 1, 1, 2, 2, 0, 0, 2, 0.5),
    ("conv1d_like", 30, 8, 1, 64, 1, 3, 1, 1, 0, 0, 2, 0.8),
    ("stride3", 3, 4, 11, 13, 3, 3, 3, 3, 1, 1, 2, 0.5),
    ("wide_tiles", 2, 3, 6, 150, 3, 3, 1, 1, 1, 1, 1, 0.5),
]


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("shape", SHAPES, ids=[s[0] for s in SHAPES])
def test_shapes_both_variants(shape, dtype):
    name, C, D, H, W, R, S, sh, sw, ph, pw, N, sp = shape
    l = wl.Layer(name, C, D, H, W, R, S, sh, sw, ph, pw, N=N, sparsity=sp, dtype=dtype, seed=4242)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    ran = 0
    for label in _both_variants(plan):
        print("case", name, dtype, label, flush=True)
        G.check(l, G.run_gpu(plan, data["x"]), ref, f"{name} {label}")
        ran += 1
    assert ran >= 1


@pytest.mark.parametrize("dtype", DT)
def test_ragged_rows_empty_rows_and_extremes(dtype):
    base = wl.Layer("ragged", 6, 9, 10, 9, 3, 3, 1, 1, 1, 1, N=2, sparsity=0.6, dtype=dtype, seed=99)
    cases = {
        "ragged": wl.prepare(base, ragged=True),
        "n=1": wl.prepare(base, n=1),
        "n=K (0% sparsity)": wl.prepare(base, n=base.K),
    }
    # a table with empty rows
    d = wl.prepare(base, ragged=True)
    rp = d["rowptr"].copy()
    keep = np.ones(rp[-1], bool)
    for row in (0, 4):
        keep[rp[row]:rp[row + 1]] = False
    lens = np.diff(rp)
    lens[[0, 4]] = 0
    d["rowptr"] = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    d["colidx"], d["values"] = d["colidx"][keep], d["values"][keep]
    cases["empty rows"] = d
    for what, data in cases.items():
        ref = G.oracle_out(base, data)
        plan = G.make_plan(base, data)
        for label in _both_variants(plan):
            print("case", what, dtype, label, flush=True)
            G.check(base, G.run_gpu(plan, data["x"]), ref, f"{what} {label}")


@pytest.mark.parametrize("dtype", ["f32", "i8"])
def test_all_zero_table_gives_zero_output(dtype):
    l = wl.Layer("empty", 3, 4, 6, 6, 3, 3, 1, 1, 1, 1, N=2, dtype=dtype)
    data = wl.prepare(l, n=0)
    assert data["rowptr"][-1] == 0
    plan = G.make_plan(l, data)
    assert plan.info().n == 0
    for label in _both_variants(plan):
        y = G.run_gpu(plan, data["x"])
        assert y.shape == (2, 4, 6, 6) and not np.any(y), label


@pytest.mark.parametrize("dtype", ["f32", "cb4", "cb4h"])
def test_long_rows_are_chunked(dtype):
    """n larger than one LDS weight stage / one gather row chunk (dense 3x3 over 160 channels)."""
    l = wl.Layer("long", 160, 6, 6, 6, 3, 3, 1, 1, 1, 1, N=1, sparsity=0.0, dtype=dtype, seed=5)
    data = wl.prepare(l)
    assert l.n == 1440
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    for label in _both_variants(plan):
        print("case long", dtype, label, flush=True)
        G.check(l, G.run_gpu(plan, data["x"]), ref, label)


@pytest.mark.parametrize("dtype", DT)
def test_wavefront_split_reduction(dtype):
    """Few output positions (batch 1, 3x3 plane): the stored entries of one output are split over
    4 / 16 / 64 lanes and combined by the wavefront-level shuffle reduction."""
    l = wl.Layer("split", 40, 9, 5, 5, 3, 3, 1, 1, 0, 0, N=1, sparsity=0.5, dtype=dtype, seed=77)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    for ns in (1, 4, 16, 64):
        for sb in (1, 2, 8):
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_GATHER, split_n=ns, sub_batch=sb)
            t = plan.get_tuning()
            assert (t.split_n, t.sub_batch) == (ns, sb)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"split_n={ns} sub_batch={sb}")


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_channel_chunked_pipeline(dtype):
    """Pointwise layer through the channel-chunked persistent kernel: chunk sizes that do and do not
    divide C, output-channel blocks, many tiles per workgroup, ragged rows."""
    l = wl.Layer("chunked", 40, 24, 12, 12, 1, 1, 1, 1, 0, 0, N=50, sparsity=0.6, dtype=dtype, seed=5)
    data = wl.prepare(l, ragged=True)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    ran = 0
    for thr, tq, cc, td, npd in ((512, 64, 8, 0, 2), (1024, 128, 16, 16, 2), (1024, 144, 33, 0, 1),
                                 (512, 144, 7, 10, 4), (256, 64, 40, 0, 1)):
        try:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pipeline=1, wg_threads=thr,
                            tile_q=tq, chunk_c=cc, tile_d=td, producers=npd)
        except B.SparseConvError as e:
            assert e.status == 4
            continue
        t = plan.get_tuning()
        assert t.chunk_c == min(cc, 40) and t.pipeline == 1
        G.check(l, G.run_gpu(plan, data["x"]), ref, str(t.as_dict()))
        ran += 1
    assert ran >= 3


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
@pytest.mark.parametrize("D", [24, 10, 1])
def test_symmetric_pipeline(dtype, D):
    """Pointwise layer through the persistent kernel in which every wave copies and multiplies: more
    tiles than workgroups, row counts that do and do not divide the wave count (including waves
    without rows), ragged rows, odd and tiny row lengths, a tile tail."""
    l = wl.Layer("sym", 40, D, 16, 16, 1, 1, 1, 1, 0, 0, N=70, sparsity=0.6, dtype=dtype, seed=7)
    ran = 0
    for n, ragged in ((None, True), (1, False), (3, False)):
        data = wl.prepare(l, n=n, ragged=ragged)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for thr, tq, cc, td in ((64, 32, 0, 0), (320, 64, 0, 0), (1024, 48, 0, 0), (1024, 128, 0, 0),
                                (704, 256, 0, 0), (1024, 128, 16, 0), (256, 256, 7, 0), (128, 64, 20, 8),
                                (512, 192, 33, 0)):
            try:
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pipeline=2,
                                wg_threads=thr, tile_q=tq, chunk_c=cc, tile_d=td)
            except B.SparseConvError as e:
                assert e.status == 4
                continue
            t = plan.get_tuning()
            assert t.pipeline == 2 and t.producers == 0
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"n={n} {t.as_dict()}")
            ran += 1
    assert ran >= 15


@pytest.mark.parametrize("dtype", ["f16", "i8"])
def test_packed_positions_in_the_producer_consumer_kernel(dtype):
    """16- and 8-bit activations through the persistent kernel whose lanes own 2 / 4 adjacent
    positions per LDS dword: one to four dwords per lane, a ragged last tile, ragged rows."""
    l = wl.Layer("packed", 24, 20, 24, 24, 1, 1, 1, 1, 0, 0, N=40, sparsity=0.5, dtype=dtype, seed=13)
    data = wl.prepare(l, ragged=True)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    ran = 0
    for thr, tq, npd in ((1024, 128, 2), (512, 256, 1), (1024, 512, 4), (768, 192, 1), (1024, 64, 2)):
        try:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pipeline=1,
                            wg_threads=thr, tile_q=tq, producers=npd)
        except B.SparseConvError as e:
            assert e.status == 4
            continue
        G.check(l, G.run_gpu(plan, data["x"]), ref, str(plan.get_tuning().as_dict()))
        ran += 1
    assert ran >= 4


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_symmetric_pipeline_rows_not_16_byte_aligned(dtype):
    """7x7 planes (49 elements per channel row): fp32 rows are only 4-byte aligned, so the symmetric
    kernels copy 4 bytes per lane; fp16 / int8 rows of odd length cannot be copied that way and the
    tuning must be refused."""
    l = wl.Layer("sym7", 72, 40, 7, 7, 1, 1, 1, 1, 0, 0, N=9, sparsity=0.7, dtype=dtype, seed=11)
    data = wl.prepare(l, ragged=True)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    ran = 0
    for thr, tq, cc, td in ((1024, 64, 0, 0), (384, 49, 24, 0), (512, 32, 16, 16), (1024, 64, 36, 8)):
        try:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pipeline=2,
                            wg_threads=thr, tile_q=tq, chunk_c=cc, tile_d=td)
        except B.SparseConvError as e:
            assert e.status == 4
            continue
        G.check(l, G.run_gpu(plan, data["x"]), ref, str(plan.get_tuning().as_dict()))
        ran += 1
    assert ran == (4 if dtype == "f32" else 0)


def test_ell_entry_point_and_unsorted_duplicate_columns():
    rng = np.random.default_rng(3)
    l = wl.Layer("ell", 4, 5, 8, 8, 3, 3, 1, 1, 1, 1, N=2, dtype="i8")
    n = 7
    col = rng.integers(0, l.K, size=(l.D, n)).astype(np.int32)       # unsorted, duplicates likely
    col[:, 3] = col[:, 2]
    val = rng.integers(-127, 128, size=(l.D, n)).astype(np.int8)
    x = rng.integers(-127, 128, size=(2, 4, 8, 8)).astype(np.int8)
    import oracle
    rp = (np.arange(l.D + 1) * n).astype(np.int32)
    ref = oracle.sparse_conv(x, rp, col.ravel(), val.ravel(), 3, 3, (1, 1), (1, 1))
    plan = B.Plan.create_ell(G.layer_desc(l), B.SC_I8, n, col, val, scales=np.ones(l.D, np.float32))
    for label in _both_variants(plan):
        assert np.array_equal(G.run_gpu(plan, x), ref), label


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_every_autotune_candidate_on_mid_size_layers(dtype):
    """Layers large enough for the wide-tile, channel-chunked, packed and pipelined candidates to
    fit (planes of 1024 and 784 positions, 96 / 160 input channels, a stride-2 layer): every
    candidate the autotuner would time gives the oracle's result."""
    for l in (wl.Layer("mid1x1", 96, 80, 32, 32, 1, 1, 1, 1, 0, 0, N=3, sparsity=0.85, dtype=dtype, seed=18),
              wl.Layer("mid3x3", 160, 48, 28, 28, 3, 3, 1, 1, 1, 1, N=2, sparsity=0.9, dtype=dtype, seed=19),
              wl.Layer("mid3x3s2", 48, 40, 28, 28, 3, 3, 2, 2, 1, 1, N=2, sparsity=0.8, dtype=dtype, seed=20)):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        nc = plan.num_candidates()
        kinds = set()
        for i in range(nc):
            t = plan.candidate(i)
            plan.set_tuning(t)
            d = t.as_dict()
            kinds.add((d["variant"], d["pipeline"], d["chunk_c"] > 0, d["pack"], d["wsrc"], d["sub_batch"] > 1))
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} candidate {i} {d}")
        print("case", l.name, dtype, nc, "candidates,", len(kinds), "kinds", flush=True)
        assert nc >= 50 and len(kinds) >= 6


def test_every_autotune_candidate_gives_the_same_answer():
    for l in (wl.Layer("cand3x3", 16, 24, 20, 20, 3, 3, 1, 1, 1, 1, N=3, sparsity=0.8, seed=8),
              wl.Layer("cand1x1", 32, 40, 16, 16, 1, 1, 1, 1, 0, 0, N=3, sparsity=0.8, seed=9)):
        data = wl.prepare(l)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        nc = plan.num_candidates()
        assert nc >= 8
        for i in range(nc):
            t = plan.candidate(i)
            plan.set_tuning(t)
            print("candidate", l.name, i, t.as_dict(), flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} candidate {i} {t.as_dict()}")


def test_autotune_installs_a_valid_tuning():
    import torch
    l = wl.Layer("tune", 32, 32, 28, 28, 3, 3, 1, 1, 1, 1, N=4, sparsity=0.9, seed=10)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    x = G.to_device(data["x"])
    y = torch.empty((4, 32, 28, 28), device="cuda")
    ws = torch.empty(max(plan.workspace_size_max(4), 1), dtype=torch.uint8, device="cuda")
    plan.autotune(x.data_ptr(), y.data_ptr(), 4, ws.data_ptr(), ws.numel(),
                  torch.cuda.current_stream().cuda_stream)
    t = plan.get_tuning()
    assert t.variant in (B.SC_VARIANT_GATHER, B.SC_VARIANT_SLAB)
    G.check(l, G.run_gpu(plan, data["x"]), ref, str(t.as_dict()))
    assert plan.info().grid_size > 0


@pytest.mark.parametrize("cfg,dtype", [(2, "f32"), (5, "i8"), (5, "cb4"), (7, "cb4h")])
def test_vgg_stack_layers_at_reduced_batch(cfg, dtype):
    layers = [l for l in wl.CONFIGS[cfg]() if l.dtype == dtype]
    assert len(layers) == 13
    for l in layers:
        data = wl.prepare(l, N=2)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        print("case", l.name, plan.get_tuning().as_dict(), flush=True)
        G.check(l, G.run_gpu(plan, data["x"]), ref, l.name)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_resnet_layers_full_batch_sampled(dtype):
    """Full-size ResNet-50-shaped layers (batch 32, 90 %) in the default launch configuration;
    the oracle checks the first and last sample completely."""
    layers = [l for l in wl.config3() if l.name.endswith("sp90")]
    for l in layers:
        l = l.replace(dtype=dtype)
        data = wl.prepare(l)
        plan = G.make_plan(l, data)
        print("case", l.name, dtype, plan.get_tuning().as_dict(), flush=True)
        y = G.run_gpu(plan, data["x"])
        for b in (0, l.N - 1):
            ref = G.oracle_out(l, data, samples=[b])
            G.check(l, y[b:b + 1], ref, f"{l.name} sample {b}")


def test_headline_layer_full_size_as_benchmarked():
    """The benchmark's layer at full size in the launch shape the benchmark times: autotuned, then
    the oracle checks the first and the last sample completely; also the three persistent kernel
    families pinned explicitly."""
    import torch
    l = wl.headline_layer()
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    x = G.to_device(data["x"])
    y = torch.empty((l.N, l.D, l.P, l.Q), device="cuda")
    ws = torch.empty(max(plan.workspace_size_max(l.N), 1), dtype=torch.uint8, device="cuda")
    plan.autotune(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(),
                  torch.cuda.current_stream().cuda_stream)
    refs = {b: G.oracle_out(l, data, samples=[b]) for b in (0, l.N - 1)}
    tuned = plan.get_tuning().as_dict()
    print("autotuned", tuned, flush=True)
    assert tuned["variant"] == B.SC_VARIANT_SLAB and tuned["pipeline"] >= 1
    y = G.run_gpu(plan, data["x"])
    for b, ref in refs.items():
        G.check(l, y[b:b + 1], ref, f"autotuned {tuned} sample {b}")
    for extra in ({"pipeline": 1, "producers": 1, "tile_q": 64}, {"pipeline": 2, "tile_q": 64},
                  {"pipeline": 1, "producers": 2, "tile_q": 256, "chunk_c": 64},
                  {"pipeline": 2, "tile_q": 128, "chunk_c": 128}):
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=1024, **extra)
        y = G.run_gpu(plan, data["x"])
        for b, ref in refs.items():
            G.check(l, y[b:b + 1], ref, f"{extra} sample {b}")


@pytest.mark.parametrize("name,extra", [
    ("s28_conv3x3_s2_sp90", {"tile_p": 4, "chunk_c": 64, "wg_per_cu": 1}),
    ("s14_conv3x3_sp90", {"tile_p": 7, "chunk_c": 128, "tile_d": 128, "wg_per_cu": 2}),
    ("s7_conv3x3_sp90", {"tile_p": 7, "chunk_c": 64, "tile_d": 128, "sub_batch": 2}),
    ("s7_expand1x1_sp90", {"tile_p": 1, "tile_q": 49, "chunk_c": 128, "tile_d": 128, "sub_batch": 4, "wg_per_cu": 1}),
    ("s14_reduce1x1_sp90", {"tile_p": 1, "tile_q": 128, "chunk_c": 128, "tile_d": 128, "pipeline": 2}),
    ("s7_reduce1x1_sp90", {"tile_p": 1, "tile_q": 49, "chunk_c": 768, "tile_d": 64, "wg_per_cu": 1}),
    ("s7_conv3x3_sp80", {"tile_p": 7, "chunk_c": 192, "tile_d": 32, "sub_batch": 2, "wg_per_cu": 1}),
    ("s7_conv3x3_sp80", {"tile_p": 7, "chunk_c": 64, "tile_d": 16, "wg_per_cu": 1, "pack": 3}),
    ("s56_conv3x3_sp80", {"tile_p": 2, "chunk_c": 32, "tile_d": 64, "wg_per_cu": 1, "pack": 3}),
    ("s14_conv3x3_s2_sp90", {"tile_p": 4, "chunk_c": 32, "tile_d": 32, "wg_per_cu": 1, "pack": 3}),
])
def test_full_size_layers_through_the_chunked_kernels(name, extra):
    """Full-size ResNet-50-shaped layers (batch 32) through the channel-chunked kernels with
    output-channel blocks, several samples per workgroup and samples interleaved in the LDS word;
    first and last sample checked."""
    l = {x.name: x for x in wl.config3()}[name]
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=1024, **extra)
    t = plan.get_tuning().as_dict()
    assert t["chunk_c"] == extra["chunk_c"]
    y = G.run_gpu(plan, data["x"])
    for b in (0, l.N - 1):
        G.check(l, y[b:b + 1], G.oracle_out(l, data, samples=[b]), f"{name} {t} sample {b}")


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_one_dimensional_convolution_workload(dtype):
    """The 1-D convolution layers (300 channels, length 64, kernels 2 and 3, batch 128) at full
    size, autotuned; the oracle checks three samples completely."""
    import torch
    for l in [x for x in wl.config6() if x.dtype == dtype]:
        data = wl.prepare(l)
        plan = G.make_plan(l, data)
        x = G.to_device(data["x"])
        y = torch.empty((l.N, l.D, l.P, l.Q), device="cuda", dtype=B.torch_out_dtype(plan.dtype))
        ws = torch.empty(max(plan.workspace_size_max(l.N), 1), dtype=torch.uint8, device="cuda")
        plan.autotune(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(),
                      torch.cuda.current_stream().cuda_stream)
        t = plan.get_tuning().as_dict()
        print("case", l.name, t, flush=True)
        out = G.run_gpu(plan, data["x"])
        for b in (0, 77, l.N - 1):
            G.check(l, out[b:b + 1], G.oracle_out(l, data, samples=[b]), f"{l.name} {t} sample {b}")


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_ragged_table_option_matches_the_unified_result(dtype):
    """Rows of different lengths walked over their own entries only (tuning.ragged = 1, the filler
    entries left out of the per-chunk segments) through the three chunked kernels: the result is
    the oracle's, as for the unified table."""
    for l in (wl.Layer("rag3x3", 20, 36, 14, 14, 3, 3, 2, 2, 1, 1, N=5, sparsity=0.7, dtype=dtype, seed=21),
              wl.Layer("rag1x1", 48, 24, 16, 16, 1, 1, 1, 1, 0, 0, N=9, sparsity=0.6, dtype=dtype, seed=22)):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        ran = 0
        for extra in ({"chunk_c": 6, "tile_p": 4, "tile_d": 16}, {"chunk_c": 16, "tile_p": 2, "sub_batch": 2},
                      {"chunk_c": 16, "pipeline": 1, "tile_q": 128, "producers": 1},
                      {"chunk_c": 12, "pipeline": 2, "tile_q": 64, "tile_d": 8}):
            for ragged in (0, 1):
                try:
                    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=512,
                                    ragged=ragged, **extra)
                except B.SparseConvError as e:
                    assert e.status == 4
                    continue
                t = plan.get_tuning().as_dict()
                assert t["ragged"] == ragged
                G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
                ran += 1
        assert ran >= 4


@pytest.mark.parametrize("dtype", ["f16", "i8"])
def test_packed_positions_in_the_chunked_one_shot_kernel(dtype):
    """tuning.pack = 1: a lane owns the 2 (f16) or 4 (i8) adjacent positions of one 32-bit word of the
    staged tile.  Filter taps make the word start at any element (odd offsets), tiles end in the
    middle of a word, stride phases and padding are in play, and tiles of 1..4 words per lane."""
    for l, tunings in (
            (wl.Layer("pk3x3", 20, 24, 28, 28, 3, 3, 1, 1, 1, 1, N=3, sparsity=0.8, dtype=dtype, seed=31),
             [{"tile_p": 4, "chunk_c": 8}, {"tile_p": 7, "chunk_c": 20, "tile_d": 8}, {"tile_p": 16, "chunk_c": 4},
              {"tile_p": 2, "chunk_c": 16, "wg_per_cu": 3}]),
            (wl.Layer("pk3x3s2", 12, 10, 29, 27, 3, 3, 2, 2, 1, 1, N=2, sparsity=0.7, dtype=dtype, seed=32),
             [{"tile_p": 4, "chunk_c": 5}, {"tile_p": 14, "chunk_c": 12}]),
            (wl.Layer("pk1x1", 96, 40, 14, 14, 1, 1, 1, 1, 0, 0, N=5, sparsity=0.9, dtype=dtype, seed=33),
             [{"tile_q": 64, "chunk_c": 32}, {"tile_q": 200, "chunk_c": 16, "tile_d": 16}, {"tile_q": 512, "chunk_c": 64}]),
            (wl.Layer("pk5x1", 9, 6, 40, 7, 5, 1, 1, 1, 2, 0, N=2, sparsity=0.5, dtype=dtype, seed=34),
             [{"tile_p": 9, "chunk_c": 4}])):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in tunings:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=512, pack=1, **extra)
            t = plan.get_tuning().as_dict()
            assert t["pack"] == 1
            print("case", l.name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
    # the pipelined chunked kernels of the pointwise layers (rows and tiles are whole words there)
    l = wl.Layer("pk1x1p", 72, 50, 20, 28, 1, 1, 1, 1, 0, 0, N=4, sparsity=0.8, dtype=dtype, seed=36)
    data = wl.prepare(l, ragged=True)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    for extra in ({"pipeline": 1, "tile_q": 128, "chunk_c": 16, "producers": 1},
                  {"pipeline": 1, "tile_q": 512, "chunk_c": 24, "tile_d": 32, "producers": 2},
                  {"pipeline": 2, "tile_q": 256, "chunk_c": 32}, {"pipeline": 2, "tile_q": 64, "chunk_c": 9, "tile_d": 24},
                  {"pipeline": 2, "tile_q": 384, "chunk_c": 16, "ragged": 1}):
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=1024, pack=1, **extra)
        t = plan.get_tuning().as_dict()
        assert t["pack"] == 1 and t["pipeline"] == extra["pipeline"]
        print("case", l.name, dtype, t, flush=True)
        G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
    # not for 32-bit activations
    l = wl.Layer("pkf32", 8, 8, 8, 8, 1, 1, 1, 1, 0, 0, N=2, sparsity=0.5, dtype="f32", seed=35)
    plan = G.make_plan(l, wl.prepare(l))
    for extra in ({"chunk_c": 4}, ):
        with pytest.raises(B.SparseConvError):
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pack=1, **extra)


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_lane_distributed_weights_in_the_chunked_one_shot_kernel(dtype):
    """tuning.wsrc = 3 with chunk_c > 0: segments longer than one batch of 64 entries, empty segments,
    rows of uneven length (with and without the fillers), one and several samples per workgroup."""
    for l, tunings in (
            (wl.Layer("ln1x1", 320, 40, 7, 7, 1, 1, 1, 1, 0, 0, N=6, sparsity=0.3, dtype=dtype, seed=41),
             [{"chunk_c": 160, "tile_q": 49, "sub_batch": 4}, {"chunk_c": 100, "tile_q": 49, "tile_d": 16, "sub_batch": 2},
              {"chunk_c": 64, "tile_q": 49, "ragged": 1}]),
            (wl.Layer("ln3x3", 24, 20, 14, 14, 3, 3, 1, 1, 1, 1, N=3, sparsity=0.5, dtype=dtype, seed=42),
             [{"chunk_c": 24, "tile_p": 7}, {"chunk_c": 5, "tile_p": 4, "tile_d": 8}, {"chunk_c": 12, "tile_p": 14, "ragged": 1}])):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in tunings:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=3, wg_threads=512, wg_per_cu=1, **extra)
            t = plan.get_tuning().as_dict()
            assert t["wsrc"] == 3 and t["chunk_c"] > 0
            print("case", l.name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_pointwise_whole_plane_tiles_staged_as_a_plain_copy(dtype):
    """Pointwise layer, one tile per plane, chunk images that are 16-byte aligned blocks of the input:
    the chunked one-shot kernel copies them with 16-byte loads.  7x7 and 14x14 planes, a last chunk
    with fewer channels, one and several samples per workgroup, a batch that does not divide."""
    for l, tunings in (
            (wl.Layer("flat7", 72, 24, 7, 7, 1, 1, 1, 1, 0, 0, N=5, sparsity=0.8, dtype=dtype, seed=51),
             [{"chunk_c": 16, "tile_q": 49}, {"chunk_c": 32, "tile_q": 49, "sub_batch": 2},
              {"chunk_c": 16, "tile_q": 49, "sub_batch": 4, "tile_d": 8}]),
            (wl.Layer("flat14", 40, 20, 14, 14, 1, 1, 1, 1, 0, 0, N=3, sparsity=0.7, dtype=dtype, seed=52),
             [{"chunk_c": 8, "tile_q": 196}, {"chunk_c": 40, "tile_q": 256, "tile_d": 8}] +
             ([{"chunk_c": 8, "tile_q": 196, "pack": 2, "tile_d": 8}] if dtype == "f32" else []) +
             ([{"chunk_c": 16, "tile_q": 196, "pack": 1}] if dtype != "f32" else []))):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in tunings:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=512, wg_per_cu=1, **extra)
            t = plan.get_tuning().as_dict()
            assert t["tile_q"] == l.H * l.W and t["chunk_c"] == extra["chunk_c"]
            print("case", l.name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_full_width_tiles_staged_by_row_runs(dtype):
    """Unit strides and tiles as wide as the plane: the chunked one-shot kernel copies whole input rows
    with 4-, 8- or 16-byte loads and writes the zero padding once.  Widths that give each load size
    (and one that gives none), paddings 0..2, tiles that end below the plane, packed positions."""
    shapes = [("rr56", 12, 10, 13, 56, 3, 3, 1, 1, 1), ("rr24", 10, 12, 9, 24, 3, 3, 1, 1, 1), ("rr20", 9, 8, 11, 20, 5, 5, 2, 2, 1),
              ("rr12", 16, 6, 12, 12, 3, 3, 0, 0, 1), ("rr8", 20, 9, 8, 8, 1, 3, 0, 1, 1), ("rr14", 7, 5, 14, 14, 3, 3, 1, 1, 1),
              ("rr10", 6, 5, 10, 10, 3, 3, 2, 1, 1),
              # strides of two: rows and columns split by parity into the four phase images
              ("rs56", 10, 8, 30, 56, 3, 3, 1, 1, 2), ("rs24", 12, 10, 17, 24, 3, 3, 0, 0, 2), ("rs16", 8, 6, 16, 16, 2, 2, 0, 0, 2),
              ("rs20", 6, 7, 19, 20, 5, 5, 2, 2, 2), ("rs12", 9, 5, 12, 12, 3, 3, 1, 1, 2)]
    for name, C, D, H, W, R, S, ph, pw, st in shapes:
        l = wl.Layer(name, C, D, H, W, R, S, st, st, ph, pw, N=3, sparsity=0.6, dtype=dtype, seed=61)
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        ran = 0
        for extra in ({"tile_p": 4, "chunk_c": 3}, {"tile_p": 3, "chunk_c": 64, "tile_d": 4},
                      {"tile_p": 5, "chunk_c": 4, "pack": 1}, {"tile_p": 8, "chunk_c": 2, "pack": 1, "tile_d": 3}):
            try:
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=256, wg_per_cu=1,
                                tile_q=10000, **extra)
            except B.SparseConvError as e:
                assert e.status == 4 and extra.get("pack") and dtype == "f32"    # packing: 16- and 8-bit only
                continue
            t = plan.get_tuning().as_dict()
            print("case", name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{name} {t}")
            ran += 1
        assert ran >= 2


@pytest.mark.parametrize("name,extra", [
    ("s56_conv3x3_sp80", {"tile_p": 7, "chunk_c": 64, "wg_per_cu": 1, "pack": 1}),
    ("s28_conv3x3_sp80", {"tile_p": 7, "chunk_c": 128, "tile_d": 64, "wg_per_cu": 1, "pack": 1}),
    ("s14_conv3x3_s2_sp90", {"tile_p": 7, "chunk_c": 64, "tile_d": 64, "wg_per_cu": 1, "pack": 1}),
    ("s28_reduce1x1_sp80", {"pipeline": 1, "producers": 1, "tile_q": 256, "chunk_c": 128, "tile_d": 64, "pack": 1}),
    ("s14_reduce1x1_sp90", {"pipeline": 2, "tile_q": 128, "chunk_c": 256, "tile_d": 64, "pack": 1}),
    ("s7_reduce1x1_sp90", {"tile_q": 49, "chunk_c": 256, "tile_d": 32, "sub_batch": 2, "wg_per_cu": 1}),
    ("s7_expand1x1_sp90", {"tile_q": 49, "chunk_c": 256, "tile_d": 64, "sub_batch": 4, "wg_per_cu": 1, "wsrc": 3}),
    ("s7_reduce1x1_sp80", {"tile_q": 49, "chunk_c": 768, "tile_d": 32, "sub_batch": 2, "wg_per_cu": 1}),
    ("s7_expand1x1_sp80", {"tile_q": 49, "chunk_c": 256, "tile_d": 64, "sub_batch": 4, "wg_per_cu": 1, "pack": 1}),
])
def test_full_size_half_precision_layers_packed_and_small_plane_forms(name, extra):
    """Full-size ResNet-50-shaped fp16 layers (batch 32) in the launch shapes the per-layer report
    picks: packed positions (shifted images on the 3x3 layers, row-run staging where the tile spans
    the plane), whole-plane copies, lane-distributed weights, chunks of 768 channels and the planes
    of four samples end to end in one packed tile on the 7x7 layers.  First and last sample checked
    completely against the oracle."""
    l = {x.name: x for x in wl.config4()}[name]
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wg_threads=1024, **{"wsrc": 1, **extra})
    t = plan.get_tuning().as_dict()
    assert t["chunk_c"] == extra["chunk_c"] and t["pack"] == extra.get("pack", 0)
    y = G.run_gpu(plan, data["x"])
    for b in (0, l.N - 1):
        G.check(l, y[b:b + 1], G.oracle_out(l, data, samples=[b]), f"{name} {t} sample {b}")


def test_power_of_two_quantised_layer_is_bit_exact():
    """The paper's linear quantiser (per-tensor power-of-two step, activations saturated at 0.99)
    applied by the library's plan-time helper, then the int8 path: same codes as the oracle's
    quantiser, same int32 outputs as the oracle's convolution of those codes."""
    import oracle
    l = wl.Layer("pow2", 48, 40, 14, 14, 3, 3, 1, 1, 1, 1, N=4, sparsity=0.85, dtype="f32", seed=71)
    data = wl.prepare(l)
    wq, wf = B.quantize_pow2(data["values"], 8)
    xq, xf = B.quantize_pow2(data["x"], 8, 0.99)
    wo, wfo = oracle.quantise_pow2(data["values"], 8)
    xo, xfo = oracle.quantise_pow2(data["x"], 8, 0.99)
    assert (wf, xf) == (wfo, xfo) == (9, 7) and np.array_equal(wq, wo) and np.array_equal(xq, xo)
    li = l.replace(dtype="i8")
    qd = dict(data, values=wq, x=xq, scales=np.full(l.D, 2.0 ** -wf, np.float32), codebook=None)
    ref = G.oracle_out(li, qd)
    assert ref.dtype == np.int32 and np.any(ref)
    plan = G.make_plan(li, qd)
    for label in _both_variants(plan):
        G.check(li, G.run_gpu(plan, xq), ref, label)
    # dequantised, the result is the fp32 layer's up to the quantisation noise
    y = ref.astype(np.float64) * 2.0 ** -(wf + xf)
    yf = G.oracle_out(l, data).astype(np.float64)
    assert np.max(np.abs(y - yf)) / np.max(np.abs(yf)) < 0.05


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_autotune_and_forward_with_unaligned_device_pointers(dtype):
    """x and y that start one element into their allocations: the launch shapes that need 16-byte
    aligned rows are skipped by the autotuner (forward reports them as unsupported instead of
    launching), and the shape it installs gives the oracle's result."""
    import torch
    l = wl.Layer("unal", 32, 24, 16, 16, 1, 1, 1, 1, 0, 0, N=6, sparsity=0.7, dtype=dtype, seed=81)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    x0 = G.to_device(data["x"])
    xbuf = torch.empty(x0.numel() + 8, dtype=x0.dtype, device="cuda")
    x = xbuf[1:1 + x0.numel()].view(x0.shape)
    x.copy_(x0)
    ybuf = torch.full((l.N * l.D * l.P * l.Q + 8,), 7, dtype=B.torch_out_dtype(plan.dtype), device="cuda")
    y = ybuf[1:1 + l.N * l.D * l.P * l.Q].view(l.N, l.D, l.P, l.Q)
    assert x.data_ptr() % 16 != 0 and y.data_ptr() % 16 != 0
    ws = torch.empty(max(plan.workspace_size_max(l.N), 16), dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    plan.autotune(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), st)
    t = plan.get_tuning().as_dict()
    print("case unaligned", dtype, t, flush=True)
    plan.forward(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), st)
    torch.cuda.synchronize()
    G.check(l, G.to_host(y), ref, f"unaligned {t}")
    assert int(ybuf[0]) == 7 and int(ybuf[-1]) == 7          # nothing written outside y
    # a pipelined shape asked for explicitly installs, but forward refuses these pointers
    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=512, pipeline=2, tile_q=64, chunk_c=8)
    with pytest.raises(B.SparseConvError) as e:
        plan.forward(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), st)
    assert e.value.status == 4


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_positions_packed_in_128_bit_words(dtype):
    """tuning.pack = 2: a lane owns the 4 (f32) or 8 (f16) adjacent positions of one 128-bit word, read
    with one LDS instruction.  Pointwise layers through the one-shot and both pipelined chunked
    kernels (tiles of one and two words per lane, ragged last tile, output-channel blocks), other
    layers through the one-shot kernel with its shifted images (odd offsets, strides, padding)."""
    cases = (
        (wl.Layer("w1x1", 72, 50, 20, 28, 1, 1, 1, 1, 0, 0, N=4, sparsity=0.8, dtype=dtype, seed=91),
         [{"tile_q": 256}, {"tile_q": 512, "wg_threads": 256}, {"tile_q": 128, "wg_per_cu": 2},
          {"chunk_c": 16, "tile_q": 256}, {"chunk_c": 24, "tile_q": 512, "tile_d": 16}, {"chunk_c": 72, "tile_q": 128},
          {"pipeline": 1, "tile_q": 256, "producers": 1}, {"pipeline": 1, "tile_q": 512, "producers": 2},
          {"pipeline": 1, "tile_q": 256, "chunk_c": 16, "producers": 1},
          {"pipeline": 1, "tile_q": 512, "chunk_c": 24, "tile_d": 32, "producers": 2},
          {"pipeline": 2, "tile_q": 256, "chunk_c": 32}, {"pipeline": 2, "tile_q": 128, "chunk_c": 9, "tile_d": 24},
          {"pipeline": 2, "tile_q": 512, "chunk_c": 16, "ragged": 1}]),
        (wl.Layer("w3x3", 20, 24, 28, 28, 3, 3, 1, 1, 1, 1, N=3, sparsity=0.8, dtype=dtype, seed=92),
         [{"tile_p": 4, "chunk_c": 4}, {"tile_p": 8, "chunk_c": 5, "tile_d": 8}, {"tile_p": 2, "chunk_c": 8, "wg_per_cu": 2}]),
        (wl.Layer("w3x3s2", 12, 10, 29, 27, 3, 3, 2, 2, 1, 1, N=2, sparsity=0.7, dtype=dtype, seed=93),
         [{"tile_p": 4, "chunk_c": 3}, {"tile_p": 14, "chunk_c": 4}]),
        (wl.Layer("w1x1odd", 40, 12, 7, 7, 1, 1, 1, 1, 0, 0, N=5, sparsity=0.6, dtype=dtype, seed=94),
         [{"tile_q": 49, "chunk_c": 8}]))
    for l, tunings in cases:
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        ran = 0
        for extra in tunings:
            try:
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pack=2,
                                **{"wg_per_cu": 1, "wg_threads": 1024, **extra})
            except B.SparseConvError as e:
                assert e.status == 4
                print("does not fit", l.name, dtype, extra, flush=True)
                continue
            t = plan.get_tuning().as_dict()
            assert t["pack"] == 2 and t["pipeline"] == extra.get("pipeline", 0)
            print("case", l.name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
            ran += 1
        assert ran >= 1, l.name


def test_autotune_takes_the_ragged_table_when_rows_are_uneven():
    """Rows with uniform lengths in [0, n] (about half of the unified table is fillers): the
    autotuner's candidates include the chunked shapes with the fillers left out, it installs one of
    them, and the result is the oracle's.  A table with equal rows gets no such candidates."""
    import torch
    l = wl.Layer("ragtune", 128, 64, 28, 28, 3, 3, 1, 1, 1, 1, N=4, sparsity=0.8, seed=95)
    even = G.make_plan(l, wl.prepare(l))
    assert not any(even.candidate(i).ragged for i in range(even.num_candidates()))
    data = wl.prepare(l, ragged=True)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    assert any(plan.candidate(i).ragged for i in range(plan.num_candidates()))
    x = G.to_device(data["x"])
    y = torch.empty((l.N, l.D, l.P, l.Q), device="cuda")
    ws = torch.empty(max(plan.workspace_size_max(l.N), 1), dtype=torch.uint8, device="cuda")
    plan.autotune(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    t = plan.get_tuning().as_dict()
    print("case ragtune", t, flush=True)
    assert t["ragged"] == 1
    G.check(l, G.run_gpu(plan, data["x"]), ref, str(t))


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_samples_laid_end_to_end_in_one_packed_tile(dtype):
    """Pointwise layers with small planes: sub_batch samples end to end along the position axis of
    one packed tile.  7x7, 5x3 and 14x14 planes (channel pitches that need rounding up to a word),
    batches that leave a short last group, a last chunk with fewer channels, output-channel blocks,
    one and two slots per lane, 32- and 128-bit words."""
    packs = {"f32": [2], "f16": [1, 2], "i8": [1]}[dtype]
    for l, shapes in (
            (wl.Layer("e2e7", 72, 24, 7, 7, 1, 1, 1, 1, 0, 0, N=11, sparsity=0.8, dtype=dtype, seed=61),
             [{"sub_batch": 2, "chunk_c": 16}, {"sub_batch": 4, "chunk_c": 32, "tile_d": 8},
              {"sub_batch": 5, "chunk_c": 72}, {"sub_batch": 10, "chunk_c": 16, "tile_d": 16}]),
            (wl.Layer("e2e53", 33, 10, 5, 3, 1, 1, 1, 1, 0, 0, N=9, sparsity=0.6, dtype=dtype, seed=62),
             [{"sub_batch": 3, "chunk_c": 8}, {"sub_batch": 16, "chunk_c": 16}]),
            (wl.Layer("e2e14", 40, 20, 14, 14, 1, 1, 1, 1, 0, 0, N=3, sparsity=0.7, dtype=dtype, seed=63),
             [{"sub_batch": 2, "chunk_c": 8, "tile_d": 8}])):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in shapes:
            for pack in packs:
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=256, wg_per_cu=1,
                                tile_q=l.H * l.W, pack=pack, **extra)
                t = plan.get_tuning().as_dict()
                assert t["sub_batch"] == extra["sub_batch"] and t["pack"] == pack and t["chunk_c"] == extra["chunk_c"]
                print("case", l.name, dtype, t, flush=True)
                G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_samples_interleaved_in_the_lds_word(dtype):
    """tuning.pack = 3: an LDS word holds the same position of 4 (f32, i8) or 8 (f16) consecutive
    samples, so the wide reads work on any layer shape.  3x3 with padding, stride 2, a 1x3 filter, a
    pointwise layer; batches that leave a short last group (and one smaller than a word); a last
    chunk with fewer channels; one and two slots per lane; output-channel blocks."""
    for l, shapes in (
            (wl.Layer("si3x3", 40, 24, 7, 7, 3, 3, 1, 1, 1, 1, N=11, sparsity=0.8, dtype=dtype, seed=71),
             [{"tile_p": 7, "chunk_c": 16}, {"tile_p": 7, "chunk_c": 8, "tile_d": 8}, {"tile_p": 3, "chunk_c": 40}]),
            (wl.Layer("si14", 24, 12, 14, 14, 3, 3, 1, 1, 1, 1, N=5, sparsity=0.7, dtype=dtype, seed=72),
             [{"tile_p": 4, "chunk_c": 8}] + ([{"tile_p": 8, "chunk_c": 8, "tile_d": 4}] if dtype != "f16" else [])),
            (wl.Layer("sis2", 20, 16, 15, 13, 3, 3, 2, 2, 1, 1, N=3, sparsity=0.6, dtype=dtype, seed=73),
             [{"tile_p": 4, "chunk_c": 8}, {"tile_p": 8, "chunk_c": 4}]),
            (wl.Layer("si1x3", 30, 10, 1, 40, 1, 3, 1, 1, 0, 1, N=9, sparsity=0.5, dtype=dtype, seed=74),
             [{"tile_p": 1, "chunk_c": 16}]),
            (wl.Layer("sipw", 32, 16, 6, 5, 1, 1, 1, 1, 0, 0, N=6, sparsity=0.5, dtype=dtype, seed=75),
             [{"tile_p": 1, "tile_q": 30, "chunk_c": 8}])):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in shapes:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=256, wg_per_cu=1,
                            pack=3, **{"tile_q": l.Q if l.R * l.S > 1 else l.H * l.W, **extra})
            t = plan.get_tuning().as_dict()
            assert t["pack"] == 3 and t["chunk_c"] == extra["chunk_c"]
            print("case", l.name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")


@pytest.mark.parametrize("dtype", ["f16", "i8", "cb4", "cb4h"])
def test_dense_variant_on_the_matrix_cores(dtype):
    """The densified tile (MFMA) against the oracle: several channel blocks and LDS chunks, output
    channels that do not fill a 16-row block, batches that do not fill a sample group, strides,
    paddings, rectangular filters; integer dtypes bit-exact."""
    shapes = [("deep_3x3", 150, 70, 9, 11, 3, 3, 1, 1, 1, 1, 5, 0.8),
              ("deep_pointwise", 200, 37, 7, 7, 1, 1, 1, 1, 0, 0, 7, 0.7),
              ("stride2", 70, 20, 13, 12, 3, 3, 2, 2, 1, 1, 3, 0.5),
              ("rect_pad", 40, 130, 6, 17, 2, 3, 1, 2, 0, 2, 2, 0.6),
              ("tiny_plane", 96, 48, 2, 2, 3, 3, 1, 1, 1, 1, 19, 0.9),
              ("one_step", 24, 40, 9, 8, 1, 1, 1, 1, 0, 0, 3, 0.5)]      # one channel block, one tap: a single step
    for name, C, D, H, W, R, S, sh, sw, ph, pw, N, sp in shapes:
        l = wl.Layer(name, C, D, H, W, R, S, sh, sw, ph, pw, N=N, sparsity=sp, dtype=dtype, seed=777)
        data = wl.prepare(l)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        ran = piped = 0
        for extra in ({}, {"tile_d": 16}, {"tile_d": 32, "tile_p": 1}, {"tile_d": 64, "tile_p": 2, "chunk_c": 64},
                      {"tile_d": 128, "wg_per_cu": 1}, {"tile_d": 64, "tile_p": 1000, "sub_batch": 4},
                      {"tile_d": 128, "waves_m": 2, "tile_p": 2}, {"tile_d": 128, "waves_m": 4}, {"tile_d": 64, "waves_m": 1, "tile_p": 3},
                      {"tile_d": 64, "waves_m": 2, "chunk_c": 64},
                      {"tile_d": 32, "waves_m": 2, "tile_p": 1000, "sub_batch": 3},
                      {"tile_d": 32, "tile_p": 1000, "sub_batch": 16, "chunk_c": 128, "wg_per_cu": 1},
                      # several blocks of output channels per workgroup, one after the other on the resident tile
                      {"tile_d": 16, "split_n": 2}, {"tile_d": 32, "tile_p": 2, "split_n": 3}, {"tile_d": 16, "tile_p": 1, "split_n": 16},
                      {"tile_d": 64, "waves_m": 2, "split_n": 2, "tile_p": 1000, "sub_batch": 2}):
            # four waves, and eight (two groups that split the steps of the contraction and meet in LDS);
            # one-shot staging, and the pipelined form (staging waves of their own, two chunk buffers)
            cb = 64 if dtype in ("i8", "cb4") else 32
            for threads in (256, 512):
                for pipe in ({}, {"pipeline": 1}, {"pipeline": 1, "producers": 4, "chunk_c": cb}, {"pipeline": 1, "producers": 1, "chunk_c": 3 * cb}):
                    if pipe and "chunk_c" in extra and "chunk_c" in pipe:
                        continue
                    kw = {**extra, **pipe}
                    try:
                        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, wg_threads=threads, **kw)
                    except B.SparseConvError as e:
                        assert e.status == 4
                        continue
                    t = plan.get_tuning()
                    assert t.variant == B.SC_VARIANT_DENSE and t.wg_threads == threads and t.pipeline == pipe.get("pipeline", 0)
                    assert t.producers == (pipe.get("producers", 2) if pipe else 0)
                    print("case dense", name, dtype, t.as_dict(), flush=True)
                    G.check(l, G.run_gpu(plan, data["x"]), ref, f"{name} dense {kw} {threads}")
                    ran += 1
                    piped += 1 if pipe else 0
        assert ran >= 6 and piped >= 6, (name, ran, piped)
        plan.destroy()


def test_dense_variant_is_refused_where_it_does_not_apply():
    l = wl.Layer("refuse", 8, 4, 6, 6, N=1, sparsity=0.5, dtype="f32", seed=5)
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    with pytest.raises(B.SparseConvError) as e:
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE)       # 32-bit activations
    assert e.value.status == 4
    plan.destroy()
    # a column stored twice in one row adds up in the gather kernels; it has no exact dense image
    l = l.replace(dtype="i8")
    data = wl.prepare(l)
    rp, ci, va = data["rowptr"], data["colidx"].copy(), data["values"]
    ci[rp[1] + 1] = ci[rp[1]]
    plan = B.Plan.create_csr(G.layer_desc(l), B.DTYPES["i8"], rp, ci, va, data["scales"], None)
    before = plan.get_tuning().as_dict()
    with pytest.raises(B.SparseConvError) as e:
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE)
    assert e.value.status == 4 and plan.get_tuning().as_dict() == before
    plan.destroy()


@pytest.mark.parametrize("dtype,sparsity", [("f16", 0.5), ("f32", 0.9), ("i8", 0.8)])
def test_per_layer_dispatch_records_three_contenders_and_forward_honours_the_choice(dtype, sparsity):
    """sparse_conv_plan_dispatch: the gather kernels, the densified MFMA tile and the dense library timed
    on one layer; every contender that was available gives the oracle's result through
    sparse_conv_forward."""
    import torch
    l = wl.Layer("dispatch", 96, 80, 14, 14, 3, 3, 1, 1, 1, 1, N=8, sparsity=sparsity, dtype=dtype, seed=31)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    with pytest.raises(B.SparseConvError) as e:
        plan.set_path(B.SC_PATH_SPARSE)                      # nothing measured yet
    assert e.value.status == 4
    xd = G.to_device(data["x"])
    y = torch.empty((l.N, l.D, l.P, l.Q), dtype=B.torch_out_dtype(plan.dtype), device="cuda")
    ws = torch.empty(plan.autotune_workspace_size(l.N), dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    rec = plan.dispatch(xd.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), st)
    print("dispatch", dtype, rec.as_dict(), flush=True)
    assert rec.sparse_ms > 0 and rec.dense_ms > 0
    # (the two contenders are what their names say: for fp32 the densified tile is the split form)
    assert rec.sparse_tuning.variant != B.SC_VARIANT_DENSE and not _is_split(rec.sparse_tuning)
    assert rec.dense_tuning.variant == B.SC_VARIANT_DENSE or _is_split(rec.dense_tuning)
    assert _is_split(rec.dense_tuning) == (dtype == "f32")
    if dtype == "i8":
        assert rec.library_ms < 0                            # the dense library is used for floating point only
    times = {B.SC_PATH_SPARSE: rec.sparse_ms}
    if rec.dense_ms > 0:
        times[B.SC_PATH_DENSE] = rec.dense_ms
    best = min(times, key=times.get)
    assert rec.choice in (best, B.SC_PATH_LIBRARY)
    if rec.choice == B.SC_PATH_LIBRARY:
        assert 0 < rec.library_ms < 0.9 * times[best]

    def run():
        y.view(torch.uint8).fill_(0x7f)
        need = plan.workspace_size(l.N)
        w2 = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
        plan.forward(xd.data_ptr(), y.data_ptr(), l.N, w2.data_ptr(), w2.numel(), st)
        torch.cuda.synchronize()
        return G.to_host(y)

    if rec.choice != B.SC_PATH_LIBRARY:
        G.check(l, run(), ref, f"dispatch {dtype}: installed choice {rec.choice}")
    for path in (B.SC_PATH_SPARSE, B.SC_PATH_DENSE, B.SC_PATH_LIBRARY):
        try:
            plan.set_path(path)
        except B.SparseConvError as e:
            assert e.status == 4
            assert path != B.SC_PATH_SPARSE
            continue
        print("case dispatch path", dtype, path, flush=True)
        if path == B.SC_PATH_LIBRARY:
            # the dense library picks its own algorithm (possibly a transform-domain one): its
            # rounding is its own, so this leg is held to 1e-3 (fp32) / 2e-2 (fp16), not to the
            # library's own kernels' 1e-5
            got = run()
            assert G.rel_err(got, ref) <= (1e-3 if dtype == "f32" else 2e-2), G.rel_err(got, ref)
        else:
            G.check(l, run(), ref, f"dispatch {dtype}: path {path}")
    plan.destroy()


def _run_epi(plan, l, x, out_np_dtype):
    import torch
    inf = plan.info()
    xd = G.to_device(np.ascontiguousarray(x))
    tdt = {np.int8: torch.int8, np.int32: torch.int32, np.float16: torch.float16, np.float32: torch.float32}[out_np_dtype]
    y = torch.empty((x.shape[0], l.D, inf.out_P, inf.out_Q), dtype=tdt, device="cuda")
    y.view(torch.uint8).fill_(0x7f)
    assert inf.out_elem_bytes == y.element_size()
    need = plan.workspace_size(x.shape[0])
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    plan.forward(xd.data_ptr(), y.data_ptr(), x.shape[0], ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return G.to_host(y)


@pytest.mark.parametrize("dtype", DT)
def test_fused_epilogue_relu_pool_requantise(dtype):
    """ReLU / 2x2 max-pool / requantisation fused into the store of the GATHER and DENSE kernels,
    against the oracle's epilogue applied to the oracle's accumulators; requantised codes bit-exact."""
    import oracle
    shapes = [("even", 20, 24, 8, 12, 3, 3, 1, 1, 1, 1, 5, 0.6),
              ("odd_plane", 40, 36, 7, 9, 3, 3, 1, 1, 1, 1, 3, 0.7),
              ("pointwise", 70, 18, 6, 6, 1, 1, 1, 1, 0, 0, 4, 0.5),
              ("stride2", 12, 20, 13, 11, 3, 3, 2, 2, 1, 1, 2, 0.5),
              ("tiny", 96, 33, 2, 2, 3, 3, 1, 1, 1, 1, 9, 0.9)]
    integer = dtype in ("i8", "cb4")
    rng = np.random.default_rng(3)
    for name, C, D, H, W, R, S, sh, sw, ph, pw, N, sp in shapes:
        l = wl.Layer(name, C, D, H, W, R, S, sh, sw, ph, pw, N=N, sparsity=sp, dtype=dtype, seed=123)
        data = wl.prepare(l)
        acc = oracle.sparse_conv_steps(data["x"], data["rowptr"], data["colidx"], data["values"], R, S, (sh, sw), (ph, pw),
                                       codebook=data["codebook"])["y"]
        plan = G.make_plan(l, data)
        # multipliers that spread the codes over the int8 range
        rq = (100.0 / max(1.0, float(np.abs(acc).max())) * (0.5 + rng.random(D))).astype(np.float32)
        for relu, pool, requant in ((1, 0, 0), (0, 2, 0), (1, 2, 0), (1, 2, 1), (0, 0, 1), (1, 0, 1)):
            if requant and not integer:
                with pytest.raises(B.SparseConvError) as e:
                    plan.set_epilogue(relu=relu, pool=pool, requant_scale=rq)
                assert e.value.status == 4
                continue
            plan.set_epilogue(relu=relu, pool=pool, requant_scale=rq if requant else None)
            out_dt = np.int8 if requant else G.NP_OUT[dtype]
            ref = oracle.epilogue(acc, relu=bool(relu), pool=pool, requant_scale=rq if requant else None,
                                  out_dtype=None if requant else G.NP_OUT[dtype])
            with pytest.raises(B.SparseConvError) as e:
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=0)      # no epilogue in the slab kernels
            assert e.value.status == 4
            ran = 0
            for variant, extra in ((B.SC_VARIANT_GATHER, {}), (B.SC_VARIANT_GATHER, {"sub_batch": 2}),
                                   (B.SC_VARIANT_DENSE, {}), (B.SC_VARIANT_DENSE, {"tile_d": 32, "tile_p": 2}),
                                   (B.SC_VARIANT_DENSE, {"tile_d": 64, "tile_p": 1000, "sub_batch": 3, "waves_m": 2}),
                                   (B.SC_VARIANT_DENSE, {"tile_d": 128, "tile_p": 4, "waves_m": 4, "chunk_c": 64}),
                                   (B.SC_VARIANT_DENSE, {"wg_threads": 512}), (B.SC_VARIANT_DENSE, {"tile_d": 32, "tile_p": 2, "wg_threads": 512}),
                                   (B.SC_VARIANT_DENSE, {"tile_d": 64, "tile_p": 1000, "sub_batch": 3, "waves_m": 2, "wg_threads": 512}),
                                   # the pipelined form: its staging waves are gone when the epilogue's barriers are met
                                   (B.SC_VARIANT_DENSE, {"pipeline": 1}), (B.SC_VARIANT_DENSE, {"pipeline": 1, "tile_d": 32, "tile_p": 2, "producers": 1}),
                                   (B.SC_VARIANT_DENSE, {"pipeline": 1, "tile_d": 64, "tile_p": 1000, "sub_batch": 3, "waves_m": 2, "wg_threads": 512, "producers": 4}),
                                   (B.SC_VARIANT_DENSE, {"pipeline": 1, "wg_threads": 512, "tile_p": 2, "producers": 3})):
                try:
                    plan.set_tuning(B.sc_tuning_t(), variant=variant, **extra)
                except B.SparseConvError as e:
                    assert e.status == 4
                    continue
                print("case epilogue", name, dtype, (relu, pool, requant), variant, extra, flush=True)
                got = _run_epi(plan, l, data["x"], out_dt)
                assert got.shape == ref.shape, (got.shape, ref.shape)
                if requant or integer:
                    assert np.array_equal(got, ref), (name, relu, pool, requant, variant, extra, np.count_nonzero(got != ref))
                else:
                    G.check(l, got, ref, f"{name} epilogue {(relu, pool)} {variant} {extra}")
                ran += 1
            assert ran >= 2 if dtype != "f32" else ran >= 1
        plan.set_epilogue()                                      # and back to the plain convolution
        G.check(l, G.run_gpu(plan, data["x"]), G.oracle_out(l, data), f"{name} epilogue removed")
        plan.destroy()


@pytest.mark.parametrize("dtype", ["i8", "cb4"])
def test_quantised_vgg_stack_chains_through_the_fused_epilogue(dtype):
    """The VGG-16-shaped stack at batch 4 as ONE chain: every layer's int8 output (ReLU, max-pool at
    the end of a stage, requantisation) is the next layer's input, on the GPU through the DENSE
    kernel (first layer: GATHER) and in the oracle; the codes agree bit for bit after 13 layers."""
    import oracle
    import torch
    layers = [l.replace(N=4) for l in wl.config5() if (l.dtype == dtype)]
    assert len(layers) == 13
    x_ref = wl.prepare(layers[0])["x"]
    x_gpu = G.to_device(x_ref)
    for k, l in enumerate(layers):
        data = wl.prepare(l)
        pool = 2 if (k + 1 < len(layers) and layers[k + 1].H * 2 == l.H) else 0
        acc = oracle.sparse_conv_steps(x_ref, data["rowptr"], data["colidx"], data["values"], l.R, l.S,
                                       (l.stride_h, l.stride_w), (l.pad_h, l.pad_w), codebook=data["codebook"])["y"]
        post = oracle.epilogue(acc, relu=True, pool=pool)
        rq = np.full(l.D, 120.0 / max(1.0, float(post.max())), dtype=np.float32)
        x_next_ref = oracle.epilogue(acc, relu=True, pool=pool, requant_scale=rq)
        plan = G.make_plan(l, data)
        plan.set_epilogue(relu=True, pool=pool, requant_scale=rq)
        try:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE)
        except B.SparseConvError:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_GATHER)
        inf = plan.info()
        y = torch.empty((l.N, l.D, inf.out_P, inf.out_Q), dtype=torch.int8, device="cuda")
        ws = torch.empty(max(plan.workspace_size(l.N), 16), dtype=torch.uint8, device="cuda")
        plan.forward(x_gpu.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        print("case chain", dtype, k, l.name, "variant", plan.get_tuning().variant, "pool", pool, got.shape, flush=True)
        assert np.array_equal(got, x_next_ref), (k, l.name, np.count_nonzero(got != x_next_ref))
        assert np.count_nonzero(got) > 0
        x_ref, x_gpu = x_next_ref, y
        plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_chunk_buffer_ring_of_the_producer_consumer_kernel(dtype):
    """tuning.buffers = 3 .. 5: a producer wave per chunk in flight, one barrier per phase; with tile
    widths whose rows are copied as whole instructions plus a partly filled one (not a power of two,
    not a multiple of an instruction), ragged last tiles, a last chunk with fewer channels, more
    workgroup units than workgroups, uneven rows, and the packed forms."""
    for l in (wl.Layer("ring_a", 72, 50, 20, 28, 1, 1, 1, 1, 0, 0, N=5, sparsity=0.8, dtype=dtype, seed=71),
              wl.Layer("ring_b", 40, 24, 28, 28, 1, 1, 1, 1, 0, 0, N=3, sparsity=0.9, dtype=dtype, seed=72)):
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        words16 = 16 // {"f32": 4, "f16": 2, "i8": 1}[dtype]
        cases = [{"buffers": 3, "tile_q": 128, "chunk_c": 16}, {"buffers": 3, "tile_q": 392, "chunk_c": 24},
                 {"buffers": 4, "tile_q": 448, "chunk_c": 8, "tile_d": 16}, {"buffers": 5, "tile_q": 192, "chunk_c": 7},
                 {"buffers": 3, "producers": 2, "tile_q": 272, "chunk_c": 32, "wg_threads": 512, "tile_d": 24},
                 {"buffers": 0, "producers": 2, "tile_q": 448, "chunk_c": 16},      # the partial-row copies with two buffers
                 {"buffers": 0, "producers": 1, "tile_q": 400, "chunk_c": 24}]
        if dtype != "f32":
            cases += [{"buffers": 3, "tile_q": 384, "chunk_c": 16, "pack": 1}]
        if dtype != "i8":
            cases += [{"buffers": 3, "tile_q": 512, "chunk_c": 16, "pack": 2}, {"buffers": 4, "tile_q": 384 // words16 * words16, "chunk_c": 9, "pack": 2}]
        for extra in cases:
            kw = dict(variant=B.SC_VARIANT_SLAB, wsrc=1, pipeline=1, wg_threads=1024)
            kw.update(extra)
            kw["tile_q"] = -(-kw["tile_q"] // words16) * words16          # rows and tiles are whole 16-byte words
            plan.set_tuning(B.sc_tuning_t(), **kw)
            t = plan.get_tuning().as_dict()
            assert t["buffers"] == extra["buffers"] and (not t["buffers"] or t["producers"] == t["buffers"] - 1)
            print("case", l.name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
        # refused: without channel chunks, outside the producer/consumer form, producers that do not match
        for bad in ({"pipeline": 1, "buffers": 3}, {"pipeline": 2, "buffers": 3, "chunk_c": 16},
                    {"pipeline": 0, "buffers": 3, "chunk_c": 16}, {"pipeline": 1, "buffers": 3, "producers": 1, "chunk_c": 16},
                    {"pipeline": 1, "buffers": 6, "chunk_c": 16}, {"pipeline": 1, "buffers": 1, "chunk_c": 16}):
            with pytest.raises(B.SparseConvError):
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=1024, **bad)
        plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_sample_groups_along_the_lanes_with_interleaved_samples(dtype):
    """tuning.pack = 3 with tuning.sub_batch = 2 .. 8 on small planes: a workgroup takes that many groups
    of 4 (8 for f16) samples and numbers its lanes over (group, position).  Batches that end inside a
    word and inside a group, planes of 2 x 2 .. 5 x 3 with and without padding, stride 2, several
    chunks with a short last one, output-channel blocks that leave waves without rows; and the refusals."""
    cases = ((wl.Layer("sg2x2", 40, 24, 2, 2, 3, 3, 1, 1, 1, 1, N=37, sparsity=0.8, dtype=dtype, seed=81),
              [dict(tile_p=2, sub_batch=8, chunk_c=16, tile_d=8, wg_threads=256), dict(tile_p=2, sub_batch=4, chunk_c=40, wg_threads=512),
               dict(tile_p=1, sub_batch=2, chunk_c=7, tile_d=5, wg_threads=1024), dict(tile_p=2, sub_batch=3, chunk_c=24, tile_d=4, wg_threads=128)]),
             (wl.Layer("sg4x4", 24, 20, 4, 4, 3, 3, 1, 1, 1, 1, N=21, sparsity=0.7, dtype=dtype, seed=82),
              [dict(tile_p=4, sub_batch=2, chunk_c=8, tile_d=16, wg_threads=1024), dict(tile_p=2, sub_batch=5, chunk_c=24, wg_threads=256),
               dict(tile_p=1, sub_batch=8, chunk_c=5, tile_d=7, wg_threads=512)]),
             (wl.Layer("sg5x3s2", 16, 12, 9, 6, 3, 2, 2, 2, 1, 0, N=19, sparsity=0.6, dtype=dtype, seed=83),
              [dict(tile_p=5, sub_batch=2, chunk_c=6, wg_threads=256), dict(tile_p=2, sub_batch=4, chunk_c=16, tile_d=4, wg_threads=512)]),
             (wl.Layer("sg1x1", 32, 16, 3, 3, 1, 1, 1, 1, 0, 0, N=9, sparsity=0.5, dtype=dtype, seed=84),
              []))
    for l, tunings in cases:
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in tunings:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pack=3, **extra)
            t = plan.get_tuning().as_dict()
            assert t["pack"] == 3 and t["sub_batch"] == extra["sub_batch"]
            print("case", l.name, dtype, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
        # refused: groups that do not fit a wave, more than one slot per lane, too many groups
        for bad in (dict(tile_p=l.P, sub_batch=64 // max(l.P * (l.Q + (l.S - 1) // l.stride_w), 1) + 1, chunk_c=8),
                    dict(tile_p=1, sub_batch=9, chunk_c=8)):
            if bad["sub_batch"] > 1:
                with pytest.raises(B.SparseConvError):
                    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pack=3, **bad)
        plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "i8"])
def test_channel_chunks_dealt_to_several_workgroups(dtype):
    """tuning.split_n = 2 .. 16 on the chunked one-shot slab kernel: the chunks of a tile go to that many
    workgroups, which add their partial sums into y (cleared first) with atomic adds.  Splits that do
    not divide the number of chunks, a short last chunk, every staging form of that kernel (table, row
    runs, plain copy, interleaved samples with and without sample groups, several samples per
    workgroup, lane-distributed weights); y poisoned before every launch; int8 sums stay exact."""
    cases = ((wl.Layer("ks3x3", 40, 24, 9, 7, 3, 3, 1, 1, 1, 1, N=6, sparsity=0.7, dtype=dtype, seed=91),
              [dict(chunk_c=8, split_n=2, tile_p=3), dict(chunk_c=6, split_n=7, tile_p=9, tile_d=8),
               dict(chunk_c=4, split_n=10, tile_p=2, pack=3), dict(chunk_c=8, split_n=5, tile_p=1, pack=3, sub_batch=2, tile_d=16),
               dict(chunk_c=7, split_n=3, tile_p=4, sub_batch=2), dict(chunk_c=5, split_n=4, tile_p=3, wsrc=3)]),
             (wl.Layer("ks1x1", 96, 50, 7, 7, 1, 1, 1, 1, 0, 0, N=5, sparsity=0.8, dtype=dtype, seed=92),
              [dict(chunk_c=16, split_n=6, tile_q=49, wg_threads=1024), dict(chunk_c=32, split_n=3, tile_q=49, tile_d=16, sub_batch=2),
               dict(chunk_c=20, split_n=2, tile_q=32, wg_threads=512)]),
             (wl.Layer("ks3x3s2", 32, 20, 14, 14, 3, 3, 2, 2, 1, 1, N=5, sparsity=0.6, dtype=dtype, seed=93),
              [dict(chunk_c=8, split_n=4, tile_p=7), dict(chunk_c=4, split_n=8, tile_p=7, pack=3, tile_d=8)]))
    for l, tunings in cases:
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in tunings:
            kw = dict(variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=256)
            kw.update(extra)
            plan.set_tuning(B.sc_tuning_t(), **kw)
            t = plan.get_tuning().as_dict()
            assert t["split_n"] == extra["split_n"] and t["chunk_c"] == extra["chunk_c"]
            print("case", l.name, dtype, t, flush=True)
            for _ in range(2):                         # twice: the second launch finds y full of the first result
                G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
        # refused: more workgroups than chunks, outside the chunked one-shot form, more than 16
        for bad in (dict(chunk_c=l.C, split_n=2), dict(chunk_c=8, split_n=17), dict(chunk_c=0, split_n=2)):
            with pytest.raises(B.SparseConvError):
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, wg_threads=256, **bad)
        plan.destroy()
    # 16-bit outputs cannot be added atomically with one rounding: refused
    l = wl.Layer("ksf16", 32, 16, 6, 6, 3, 3, 1, 1, 1, 1, N=2, sparsity=0.5, dtype="f16", seed=94)
    plan = G.make_plan(l, wl.prepare(l))
    with pytest.raises(B.SparseConvError):
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, chunk_c=8, split_n=2)
    plan.destroy()


def test_forward_captured_in_a_hip_graph_replays_correctly():
    """The forward path records kernels only (no memset, no allocation), so a caller may capture it:
    a gather-kernel shape with its padding pre-pass, split-K shapes with their clear kernel, and the
    matrix-core tiles, each captured once and replayed three times with eager launches and
    synchronisations in between; every replay is checked against the oracle on poisoned outputs."""
    import torch
    cases = (("f32", dict(variant=B.SC_VARIANT_GATHER, sub_batch=2)),
             ("f32", dict(variant=B.SC_VARIANT_SLAB, wsrc=1, pack=3, chunk_c=8, split_n=3, tile_p=3, wg_threads=256)),
             ("i8", dict(variant=B.SC_VARIANT_SLAB, wsrc=1, chunk_c=8, split_n=2, tile_p=3, wg_threads=256)),
             ("f16", dict(variant=B.SC_VARIANT_DENSE, wg_threads=512)),
             ("i8", dict(variant=B.SC_VARIANT_DENSE, pipeline=1, producers=4, tile_p=3)),
             ("f32", dict(variant=B.SC_VARIANT_SLAB, pipeline=3)),
             ("f32", dict(variant=B.SC_VARIANT_SLAB, pipeline=3, chunk_c=32, split_n=2, tile_p=3)),
             ("f32", dict(variant=B.SC_VARIANT_SLAB, pipeline=3, producers=4, chunk_c=32, tile_p=3)))
    for dtype, tuning in cases:
        l = wl.Layer("graph", 40, 24, 9, 7, 3, 3, 1, 1, 1, 1, N=6, sparsity=0.7, dtype=dtype, seed=101)
        data = wl.prepare(l)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        plan.set_tuning(B.sc_tuning_t(), **tuning)
        x = G.to_device(np.ascontiguousarray(data["x"]))
        inf = plan.info()
        y = torch.empty((l.N, l.D, inf.P, inf.Q), dtype=B.torch_out_dtype(plan.dtype), device="cuda")
        ws = torch.empty(max(plan.workspace_size(l.N), 16), dtype=torch.uint8, device="cuda")
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            plan.forward(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), side.cuda_stream)   # warm-up outside capture
            side.synchronize()
            with torch.cuda.graph(g, stream=side):
                plan.forward(x.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), side.cuda_stream)
        torch.cuda.synchronize()
        for rep in range(3):
            y.view(torch.uint8).fill_(0x7f)                  # eager work between the replays
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            print("case graph", dtype, tuning, "replay", rep, flush=True)
            G.check(l, G.to_host(y), ref, f"graph replay {rep} {dtype} {tuning}")
        del g
        plan.destroy()


def test_interleaved_samples_staged_by_rows():
    """tuning.stage_rows = 1 (fp32, pack = 3): rows of 16- and 8-byte loads, strides of one and two, tiles
    at the top and bottom edge of the plane, several chunks with a short last one, sample groups,
    split-K, batches that end inside a word; refused where rows are no whole 8-byte loads, where the
    tile is narrower than the plane, for other types and without interleaved samples."""
    cases = ((wl.Layer("rows16", 40, 24, 9, 8, 3, 3, 1, 1, 1, 1, N=7, sparsity=0.7, dtype="f32", seed=111),
              [dict(tile_p=3, chunk_c=8), dict(tile_p=9, chunk_c=16, tile_d=8), dict(tile_p=1, chunk_c=7, wg_threads=768),
               dict(tile_p=2, chunk_c=8, split_n=3), dict(tile_p=4, chunk_c=12, sub_batch=1)]),
             (wl.Layer("rows8", 24, 20, 6, 6, 3, 3, 1, 1, 1, 1, N=21, sparsity=0.6, dtype="f32", seed=112),
              [dict(tile_p=2, chunk_c=8, sub_batch=3), dict(tile_p=6, chunk_c=24), dict(tile_p=3, chunk_c=5, split_n=4, tile_d=16)]),
             (wl.Layer("rows_s2", 32, 20, 14, 12, 3, 3, 2, 2, 1, 1, N=5, sparsity=0.6, dtype="f32", seed=113),
              [dict(tile_p=7, chunk_c=8), dict(tile_p=2, chunk_c=4, tile_d=8), dict(tile_p=3, chunk_c=16, split_n=2)]),
             (wl.Layer("rows_5x5", 16, 12, 10, 12, 5, 5, 1, 1, 2, 2, N=3, sparsity=0.8, dtype="f32", seed=114),
              [dict(tile_p=4, chunk_c=8)]))
    for l, tunings in cases:
        data = wl.prepare(l, ragged=True)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for extra in tunings:
            kw = dict(variant=B.SC_VARIANT_SLAB, wsrc=1, pack=3, stage_rows=1, wg_threads=256)
            kw.update(extra)
            plan.set_tuning(B.sc_tuning_t(), **kw)
            t = plan.get_tuning().as_dict()
            assert t["stage_rows"] == 1 and t["pack"] == 3
            print("case", l.name, t, flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} {t}")
        with pytest.raises(B.SparseConvError):          # without interleaved samples
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, stage_rows=1, chunk_c=8, tile_p=2)
        with pytest.raises(B.SparseConvError):          # GATHER
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_GATHER, stage_rows=1)
        plan.destroy()
    for l in (wl.Layer("rows_odd", 16, 12, 9, 7, 3, 3, 1, 1, 1, 1, N=3, sparsity=0.5, dtype="f32", seed=115),     # rows of 28 bytes
              wl.Layer("rows_f16", 16, 12, 8, 8, 3, 3, 1, 1, 1, 1, N=9, sparsity=0.5, dtype="f16", seed=116)):
        plan = G.make_plan(l, wl.prepare(l))
        with pytest.raises(B.SparseConvError):
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1, pack=3, stage_rows=1, chunk_c=8, tile_p=2)
        plan.destroy()


def test_random_candidates_on_seeded_random_layers():
    """Eighteen seeded layers of random geometry (filters 1x1 .. 5x5, strides, paddings, planes of 2 .. 20,
    3 .. 130 channels, batches 1 .. 9, every type, unified and ragged tables), and on each about forty
    of the autotuner's candidates drawn at random: each gives the oracle's result."""
    for seed in range(18):
        rng = np.random.default_rng(1000 + seed)
        dtype = ["f32", "f16", "i8", "cb4", "cb4h", "f32"][seed % 6]
        R, S = [(1, 1), (3, 3), (1, 3), (5, 5), (2, 2), (3, 1)][int(rng.integers(6))]
        sh, sw = (int(rng.integers(1, 3)), int(rng.integers(1, 3))) if R * S > 1 else (1, 1)
        ph, pw = int(rng.integers(0, R // 2 + 1)), int(rng.integers(0, S // 2 + 1))
        H, W = int(rng.integers(max(R, 2), 21)), int(rng.integers(max(S, 2), 21))
        C, D, N = int(rng.integers(3, 131)), int(rng.integers(3, 91)), int(rng.integers(1, 10))
        sp = float(rng.uniform(0.3, 0.95))
        l = wl.Layer(f"rand{seed}", C, D, H, W, R, S, sh, sw, ph, pw, N=N, sparsity=sp, dtype=dtype, seed=500 + seed)
        data = wl.prepare(l, ragged=bool(seed & 1))
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        nc = plan.num_candidates()
        pick = sorted(set(int(i) for i in rng.integers(0, nc, size=44)))
        print(f"case rand{seed}: {dtype} C{C} D{D} {H}x{W} {R}x{S} s{sh},{sw} p{ph},{pw} N{N} sp{sp:.2f}: {nc} candidates, {len(pick)} drawn", flush=True)
        for i in pick:
            t = plan.candidate(i)
            plan.set_tuning(t)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} candidate {i} { {k: v for k, v in t.as_dict().items() if v} }")
        plan.destroy()


@pytest.mark.parametrize("dtype", ["f16", "i8", "cb4", "cb4h"])
def test_dense_variant_on_pointwise_layers_in_their_natural_layout(dtype):
    """tuning.stage_rows = 1 on the matrix-core tile (pointwise layers): the tile is copied to LDS as
    [channel][position] and read with the transposing LDS reads.  Planes whose runs are whole 16-,
    8-, 4-, 2-byte loads and odd ones, several chunks with a last one that is not full, channels
    that do not fill a block, tiles of rows and whole planes of several samples, batches that do
    not fill the last group, four and eight waves; refused for filters with taps and with the
    pipelined form."""
    shapes = [("pw16", 150, 70, 8, 8, 7, 0.7), ("pw28", 64, 40, 28, 28, 3, 0.5), ("pw14", 200, 37, 14, 14, 5, 0.8),
              ("pw7", 96, 48, 7, 7, 19, 0.9), ("pw5x6", 40, 130, 5, 6, 9, 0.6), ("pw_one_block", 24, 40, 9, 8, 3, 0.5)]
    cb = 64 if dtype in ("i8", "cb4") else 32
    for name, C, D, H, W, N, sp in shapes:
        l = wl.Layer(name, C, D, H, W, 1, 1, 1, 1, 0, 0, N=N, sparsity=sp, dtype=dtype, seed=888)
        data = wl.prepare(l)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        ran = 0
        for extra in ({}, {"tile_d": 16}, {"tile_d": 32, "tile_p": 1}, {"tile_d": 64, "tile_p": 2, "chunk_c": cb},
                      {"tile_d": 128, "wg_per_cu": 1}, {"tile_d": 64, "tile_p": 1000, "sub_batch": 4, "chunk_c": 2 * cb},
                      {"tile_d": 128, "waves_m": 2, "tile_p": 2}, {"tile_d": 64, "waves_m": 1, "tile_p": 3},
                      {"tile_d": 32, "waves_m": 2, "tile_p": 1000, "sub_batch": 3},
                      {"tile_d": 32, "tile_p": 1000, "sub_batch": 16, "chunk_c": 128, "wg_per_cu": 1},
                      {"tile_d": 16, "split_n": 2}, {"tile_d": 32, "tile_p": 2, "split_n": 3}, {"tile_d": 16, "tile_p": 1, "split_n": 16}):
            for threads in (256, 512):
                try:
                    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, wg_threads=threads, stage_rows=1, **extra)
                except B.SparseConvError as e:
                    assert e.status == 4
                    continue
                t = plan.get_tuning()
                assert t.variant == B.SC_VARIANT_DENSE and t.stage_rows == 1 and t.wg_threads == threads
                print("case dense natural", name, dtype, t.as_dict(), flush=True)
                G.check(l, G.run_gpu(plan, data["x"]), ref, f"{name} dense natural {extra} {threads}")
                ran += 1
        assert ran >= 6, (name, ran)
        # pipelined: the chunks are copied by direct-to-LDS loads (runs and planes of whole 16-byte words, one
        # sample per workgroup); refused otherwise
        piped = 0
        for extra in ({}, {"tile_p": 1, "chunk_c": cb, "producers": 1}, {"tile_p": 2, "tile_d": 32, "producers": 4},
                      {"tile_p": 4, "tile_d": 64, "waves_m": 1, "chunk_c": 3 * cb}, {"tile_p": 1000, "tile_d": 128, "chunk_c": cb}):
            for threads in (256, 512):
                try:
                    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, wg_threads=threads, stage_rows=1, pipeline=1, **extra)
                except B.SparseConvError as e:
                    assert e.status == 4
                    continue
                t = plan.get_tuning()
                assert t.stage_rows == 1 and t.pipeline == 1 and t.sub_batch == 1
                print("case dense natural pipelined", name, dtype, t.as_dict(), flush=True)
                G.check(l, G.run_gpu(plan, data["x"]), ref, f"{name} dense natural pipelined {extra} {threads}")
                piped += 1
        whole_words = (H * W * (1 if dtype in ("i8", "cb4") else 2)) % 16 == 0
        assert (piped >= 2) == whole_words, (name, piped)
        plan.destroy()
    l = wl.Layer("taps", 32, 16, 8, 8, 3, 3, 1, 1, 1, 1, N=2, sparsity=0.5, dtype=dtype, seed=889)
    plan = G.make_plan(l, wl.prepare(l))
    with pytest.raises(B.SparseConvError):
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, stage_rows=1)
    plan.destroy()


def test_natural_layout_candidates_on_seeded_random_pointwise_layers():
    """Twelve seeded pointwise layers (planes of whole 16-byte words and odd ones, 3 .. 300 channels, batches
    1 .. 11, the four 16- and 8-bit types) and on each up to thirty of the autotuner's natural-layout
    candidates of the matrix-core tile (register copy and direct-to-LDS copy) drawn at random."""
    ran = 0
    for seed in range(12):
        rng = np.random.default_rng(7000 + seed)
        dtype = ["f16", "i8", "cb4h", "cb4"][seed % 4]
        H, W = int(rng.integers(1, 9)) * 4, int(rng.integers(1, 9)) * 4
        if seed % 3 == 0:
            H, W = int(rng.integers(2, 30)), int(rng.integers(2, 30))
        C, D, N = int(rng.integers(3, 300)), int(rng.integers(3, 200)), int(rng.integers(1, 12))
        sp = float(rng.uniform(0.3, 0.95))
        l = wl.Layer(f"rnat{seed}", C, D, H, W, 1, 1, 1, 1, 0, 0, N=N, sparsity=sp, dtype=dtype, seed=900 + seed)
        data = wl.prepare(l, ragged=bool(seed & 1))
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        nat = [i for i in range(plan.num_candidates())
               if plan.candidate(i).stage_rows and plan.candidate(i).variant == B.SC_VARIANT_DENSE]
        pick = [nat[int(i)] for i in sorted(set(rng.integers(0, len(nat), size=30)))] if nat else []
        print(f"case rnat{seed}: {dtype} C{C} D{D} {H}x{W} N{N} sp{sp:.2f}: {len(nat)} natural-layout candidates, {len(pick)} drawn", flush=True)
        for i in pick:
            t = plan.candidate(i)
            plan.set_tuning(t)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"{l.name} candidate {i} { {k: v for k, v in t.as_dict().items() if v} }")
            ran += 1
        plan.destroy()
    assert ran >= 150, ran


def _is_split(t):
    return t.variant == B.SC_VARIANT_SLAB and t.pipeline == 3


def _split(plan, **kw):
    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, pipeline=3, **kw)


@pytest.mark.parametrize("name,C,D,H,W,R,S,sh,sw,ph,pw,N,scale", [
    ("odd3x3", 37, 45, 13, 11, 3, 3, 1, 1, 1, 1, 5, 1.0),
    ("stride2", 64, 70, 14, 15, 3, 3, 2, 2, 1, 1, 3, 1.0),
    ("pointwise7", 200, 33, 7, 7, 1, 1, 1, 1, 0, 0, 9, 1.0),
    ("pointwise28", 96, 130, 28, 28, 1, 1, 1, 1, 0, 0, 2, 2.0 ** 60),
    ("conv1d", 70, 20, 1, 61, 1, 3, 1, 1, 0, 0, 6, 2.0 ** -60),
    ("wide_pad", 8, 17, 6, 9, 2, 3, 1, 2, 4, 3, 2, 1.0),
    ("one_channel", 1, 3, 4, 4, 1, 1, 1, 1, 0, 0, 1, 1.0),
])
def test_fp32_split_form_on_the_matrix_cores(name, C, D, H, W, R, S, sh, sw, ph, pw, N, scale):
    """SLAB tunings with pipeline = 3: tails of channels, rows, columns and output channels, several chunks,
    four and eight waves, several samples per workgroup, chunks dealt to several workgroups, large and
    small magnitudes.  The six kept products are within 2^-24 of the exact one and the sum is rounded
    2 K / 32 times, so a result is held to 4e-7 of the sum of the magnitudes' root mean square -- and to
    no more error than the gather kernel's on the same table, times 1.2 for the draw, or than half a unit, to which the
    oracle's own output is rounded (element by element against 64 bits: the test after this one)."""
    l = wl.Layer(name, C, D, H, W, R, S, sh, sw, ph, pw, N=N, sparsity=0.6, dtype="f32", seed=sum(map(ord, name)))
    data = wl.prepare(l, ragged=True)
    data["x"] = data["x"] * np.float32(scale)
    ref = G.oracle_out(l, data).astype(np.float64)
    nrm = np.sqrt(np.sum(ref * ref))
    plan = G.make_plan(l, data)
    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_GATHER, split_n=1)
    gather = np.sqrt(np.sum((G.run_gpu(plan, data["x"]) - ref) ** 2)) / nrm
    ran = 0
    for threads in (256, 512):
        for kw in ({}, {"tile_d": 16, "waves_m": 1}, {"tile_d": 32, "waves_m": 1, "tile_p": 1}, {"tile_d": 32, "waves_m": 2, "chunk_c": 32},
                   {"tile_d": 64, "waves_m": 4, "tile_p": 2}, {"tile_d": 128, "waves_m": 4, "tile_p": 1, "wg_per_cu": 2},
                   {"tile_d": 64, "waves_m": 2, "tile_p": 1000, "sub_batch": 2, "chunk_c": 32}, {"tile_d": 32, "waves_m": 2, "tile_p": 1000, "sub_batch": 3},
                   {"tile_d": 64, "waves_m": 4, "tile_p": 3, "chunk_c": 64}, {"tile_d": 32, "waves_m": 1, "tile_p": 4, "chunk_c": 32, "split_n": 2},
                   {"tile_d": 128, "waves_m": 4, "tile_p": 2, "chunk_c": 32, "split_n": 3},
                   # pipelined: staging waves of their own (with eight multiplying waves only)
                   {"producers": 4}, {"producers": 4, "tile_d": 32, "waves_m": 1, "tile_p": 1, "chunk_c": 32},
                   {"producers": 4, "tile_d": 64, "waves_m": 4, "tile_p": 3, "chunk_c": 64}, {"producers": 4, "tile_d": 64, "waves_m": 2, "tile_p": 1000, "sub_batch": 2, "chunk_c": 32},
                   {"producers": 4, "tile_d": 128, "waves_m": 4, "tile_p": 2, "chunk_c": 96, "ragged": 1},
                   # ... in four groups: wave tiles of one block and of a number that four does not divide among them
                   {"producers": 4, "buffers": 4}, {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 1, "chunk_c": 32},
                   {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 1000, "chunk_c": 32}, {"producers": 4, "buffers": 4, "tile_d": 64, "waves_m": 2, "tile_p": 2, "chunk_c": 64}):
            try:
                _split(plan, wg_threads=threads, **kw)
            except B.SparseConvError as e:
                assert e.status == 4
                continue
            t = plan.get_tuning().as_dict()
            print("case split", name, t, flush=True)
            got = G.run_gpu(plan, data["x"])
            G.check(l, got, ref.astype(np.float32), f"{name} {t}", tol=2e-6)
            err = np.sqrt(np.sum((got - ref) ** 2)) / nrm
            assert err <= (4e-7 if C * R * S > 64 else 1.2e-7) and err <= max(1.2 * gather, 2.0 ** -24), (name, t, err, gather)
            ran += 1
    assert ran >= 8, (name, ran)
    plan.destroy()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 15, 16, 40])
def test_fp32_split_form_element_by_element_on_short_rows(n):
    """Rows of few stored weights, where no averaging hides what a product lost: every output against
    64 bits, one-shot and pipelined, over random significands and the ones whose mid lo is largest.  Up to 15 weights a
    row only lo lo is dropped, at most 2^-34 of a product (mid is at most 2^-8 of the value and lo 2^-17), from
    16 on mid lo and lo mid, 2^-24 of it together.  The accumulators are rounded once each per matrix
    instruction, hi hi to 2^-24 of the sum so far, the small terms to 2^-24 of a 2^-7 part, and the two are added
    with one rounding: for one weight 1 + 1/8 roundings of half a unit (2^-24) in all, for n the n + 1/8 that a sum of n
    products may have, and no more than 4 of them where the products are summed inside the instruction."""
    C = n
    l = wl.Layer("short", C, 64, 24, 24, 1, 1, 1, 1, 0, 0, N=6, sparsity=0.0, dtype="f32", seed=n)
    rng = np.random.default_rng(n)
    worst = np.array([0x3f807fc0, 0x3f808040, 0x3f807ec0, 0x3f817fc0, 0x3f80feff], np.uint32).view(np.float32)

    def values(count):
        v = rng.uniform(1, 2, count).astype(np.float32)
        v[::3] = rng.choice(worst, v[::3].size)
        return v * rng.choice(np.float32([-1, 1]), count) * np.float32(2.0) ** rng.integers(-3, 4, count).astype(np.float32)

    w = values(l.D * n)
    x = values(l.N * C * l.H * l.W).reshape(l.N, C, l.H, l.W)
    plan = B.Plan.create_csr(G.layer_desc(l), B.DTYPES["f32"], np.arange(l.D + 1, dtype=np.int32) * n,
                             np.tile(np.arange(n, dtype=np.int32), l.D), w, None, None)
    w64, x64 = w.astype(np.float64).reshape(l.D, n), x.astype(np.float64)
    ref = np.einsum("dc,bchw->bdhw", w64, x64)
    mag = np.einsum("dc,bchw->bdhw", np.abs(w64), np.abs(x64))

    def error():
        return np.abs(G.run_gpu(plan, x).astype(np.float64) - ref) / mag

    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_GATHER, split_n=1)
    gather = error()
    # (the last one: wave tiles of seven blocks, 192 positions)
    for kw in ({}, {"wg_threads": 256, "tile_d": 64, "waves_m": 2}, {"producers": 4}, {"producers": 4, "buffers": 4},
               {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 1}, {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 8}):
        _split(plan, **kw)
        print("case split short rows", n, plan.get_tuning().as_dict(), flush=True)
        e = error()
        print("   largest", e.max(), "gather", gather.max(), flush=True)
        assert e.max() <= min(n + 0.125, 4.0) * 2.0 ** -24, (n, kw, e.max(), gather.max())
        rms, rms_g = np.sqrt((e * e).mean()), np.sqrt((gather * gather).mean())
        assert rms <= 1.02 * rms_g, (n, kw, rms, rms_g)          # (2 %: the small terms' own roundings)
    plan.destroy()


@pytest.mark.parametrize("C,D,H,W,k,stride,pad,N", [(70, 20, 9, 11, 3, 2, 1, 3), (64, 33, 7, 7, 1, 1, 0, 5), (40, 70, 12, 8, 3, 1, 1, 2)])
@pytest.mark.parametrize("xe,we", [(-112, 0), (-122, 0), (-140, 0), (-60, -64), (-90, -30), (-120, 60)])
def test_fp32_split_form_sums_outputs_that_the_terms_do_not_serve_entry_by_entry(C, D, H, W, k, stride, pad, N, xe, we):
    """Inputs so small that bfloat16 has no room for their last terms, or their products none in fp32: everywhere
    (the gather kernel's sums, bit for bit; zero from inputs of 2^-134 and less), in one value of one sample only, and
    in a few channels.  A sum of n products rounded n times is within n 2^-24 of the sum of the magnitudes, n
    2^-150 where it is denormal; the tile that holds the values rounds less often and is off by 2^-28 of the smallest
    output it keeps, n (2^-133 of the largest weight + 2^-147)."""
    l = wl.Layer("tiny", C, D, H, W, k, k, stride, stride, pad, pad, N=N, sparsity=0.6, dtype="f32", seed=C)
    data = wl.prepare(l)
    data["values"] = data["values"] * np.float32(2.0 ** we)
    plan = G.make_plan(l, data)
    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_GATHER, split_n=1)
    one = np.where(data["x"] == 0, np.float32(1), data["x"])
    everywhere = one * np.float32(2.0 ** xe)
    single, shared = one.copy(), one.copy()
    single[1, C // 2, H // 2, W // 2] = 2.0 ** xe
    shared[:, :4] *= np.float32(2.0 ** xe)
    gather = G.run_gpu(plan, everywhere)

    def dense64(x, values):
        w = np.zeros((D, C * k * k))
        w[np.repeat(np.arange(D), np.diff(data["rowptr"])), data["colidx"]] = values
        xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (pad, pad), (pad, pad)))
        cols = np.stack([xp[:, :, r:r + (l.P - 1) * stride + 1:stride, c:c + (l.Q - 1) * stride + 1:stride] for r in range(k) for c in range(k)], 2)
        return np.einsum("dk,bkpq->bdpq", w, cols.reshape(N, C * k * k, l.P, l.Q))

    v = data["values"].astype(np.float64)
    for kw in ({}, {"wg_threads": 256, "tile_d": 64, "waves_m": 4, "tile_p": 3}, {"tile_d": 32, "waves_m": 1, "tile_p": 2, "chunk_c": 32, "split_n": 2},
               {"producers": 4, "tile_d": 32, "waves_m": 2, "tile_p": 2, "chunk_c": 32}, {"tile_d": 64, "waves_m": 2, "tile_p": 1000, "sub_batch": 2, "chunk_c": 32},
               {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 1, "chunk_c": 32}, {"producers": 4, "buffers": 4, "tile_d": 32, "waves_m": 2, "tile_p": 2, "chunk_c": 32},
               {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 1000, "sub_batch": 3 if H == 7 else 1, "chunk_c": 32}):
        _split(plan, **kw)
        for what, x in (("everywhere", everywhere), ("single", single), ("shared", shared)):
            print("case split tiny", C, D, xe, we, kw, what, flush=True)
            got = G.run_gpu(plan, x)
            if what == "everywhere" and "split_n" not in kw:
                assert np.array_equal(got, gather) or xe < -134 and not np.any(got), (kw, what)
            mag = dense64(np.abs(x), np.abs(v))
            excess = np.abs(got.astype(np.float64) - dense64(x, v)) - l.n * (2.0 ** -24 * mag + 2.0 ** -133 * np.abs(v).max() + 2.0 ** -147)
            assert excess.max() <= 0, (kw, what, np.unravel_index(excess.argmax(), excess.shape))
    plan.destroy()


@pytest.mark.parametrize("bad", [3.4e38, -np.inf, np.nan])
def test_fp32_split_form_on_inputs_whose_first_term_is_infinite(bad):
    """Inputs that round to an infinite bfloat16, infinities and NaN in one place: the gather kernel's result
    where an output reads that place (the table has no fillers), the usual one elsewhere in the tile, and
    weights that round to an infinite bfloat16 beside zeros and ordinary inputs."""
    l = wl.Layer("huge", 48, 40, 9, 9, 3, 3, 1, 1, 1, 1, N=3, sparsity=0.7, dtype="f32", seed=3)
    data = wl.prepare(l)
    data["values"] = data["values"] * np.float32(1e-3)
    x = data["x"].copy()
    x[1, 7, 4, 5] = bad
    x[2] = 0
    huge = data["values"].copy()
    huge[::50] = np.float32(3.4e38)
    for values, inp in ((data["values"], x), (huge, np.nan_to_num(x, nan=0, neginf=0) * np.float32(1e-30))):
        plan = B.Plan.create_csr(G.layer_desc(l), B.DTYPES["f32"], data["rowptr"], data["colidx"], values, None, None)
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_GATHER, split_n=1)
        want = G.run_gpu(plan, inp)
        for kw in ({}, {"producers": 4, "tile_d": 32, "waves_m": 2, "tile_p": 2}, {"wg_threads": 256, "chunk_c": 32, "tile_p": 3},
                   {"producers": 4, "buffers": 4, "tile_d": 32, "waves_m": 2, "tile_p": 2}, {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 1, "chunk_c": 32},
                   {"producers": 4, "buffers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 1000, "sub_batch": 2, "chunk_c": 32}):
            _split(plan, **kw)
            print("case split huge", bad, kw, flush=True)
            got = G.run_gpu(plan, inp)
            fin = np.isfinite(want)
            assert np.array_equal(got[~fin], want[~fin], equal_nan=True), kw
            assert np.abs(got[fin].astype(np.float64) - want[fin]).max() <= 1e-5 * np.abs(want[fin]).max(), kw
            assert not np.any(got[2]) and np.array_equal(np.isfinite(got), fin), kw
        plan.destroy()


@pytest.mark.parametrize("W,shift", [(28, 0), (28, 1), (28, 2), (14, 0), (14, 1), (6, 2), (7, 0), (7, 3)])
@pytest.mark.parametrize("R", [1, 3])
def test_fp32_split_form_staging_loads_of_every_width(W, shift, R):
    """Rows of a multiple of 4, of 2 and odd ones, x at 4, 8 and 12 bytes past 16, one-shot and pipelined, tiles of rows and of whole
    planes, output channels that fill one block of 16 or less of it.  (The width of a load follows neither row length nor pointer
    but an estimate of the time; every width with and without a run's last block overlapping the one before: the next test.)"""
    import torch
    l = wl.Layer("widths", 45, 13, 8, W, R, R, 1, 1, R // 2, R // 2, N=3, sparsity=0.6, dtype="f32", seed=W)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    buf = torch.full((data["x"].size + 8,), float("nan"), device="cuda")
    x = buf[shift:shift + data["x"].size]
    x.copy_(torch.from_numpy(np.ascontiguousarray(data["x"])).cuda().flatten())
    plan = G.make_plan(l, data)
    for kw in ({}, {"tile_d": 16, "waves_m": 1, "tile_p": 3, "wg_threads": 256}, {"tile_d": 32, "waves_m": 2, "tile_p": 1, "chunk_c": 32},
               {"tile_p": 1000, "sub_batch": 2, "chunk_c": 32}, {"producers": 4, "tile_p": 2}, {"producers": 4, "tile_d": 16, "waves_m": 1, "tile_p": 3, "chunk_c": 32}):
        try:
            _split(plan, **kw)
        except B.SparseConvError as e:
            assert e.status == 4 and kw.get("tile_p") == 1000
            continue
        print("case split widths", W, shift, R, kw, flush=True)
        y = torch.full(ref.shape, float("nan"), device="cuda")
        plan.forward(x.data_ptr(), y.data_ptr(), l.N, 0, 0, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        G.check(l, G.to_host(y), ref, f"widths {W} {shift} {kw}", tol=2e-6)
    plan.destroy()


@pytest.mark.parametrize("form", ["one", "two", "pipe2", "pipe4"])
def test_fp32_split_form_staging_of_every_width_and_tail(form):
    """Every instantiation by the columns of a staging load in every form -- one-shot with one and two groups of waves, pipelined with
    two and four --, with runs that are whole loads and runs that end in a load overlapping the one before, with chunks of no
    more rounds than are loaded ahead and of more, x at each multiple of 4 bytes; and the one-shot wave tile of 2 x 7 blocks, which stages
    one block at a time, in each width.  What a shape stages is worked out by split_staging; none of it may be left out."""
    import torch
    kw = {"one": dict(wg_threads=256), "two": dict(wg_threads=512), "pipe2": dict(producers=4), "pipe4": dict(producers=4, buffers=4)}[form]
    everything = {(c, tail, more) for c in (1, 2, 4) for tail in (False, True) for more in (False, True) if c > 1 or not tail}
    seen, large = {}, set()
    for k, (C, H, W, R, sw, N) in enumerate([(130, 8, 31, 1, 1, 3), (100, 8, 31, 1, 1, 2), (45, 6, 28, 1, 1, 3), (100, 6, 28, 1, 1, 2), (45, 9, 14, 1, 1, 4), (130, 14, 14, 1, 1, 1),
                                             (128, 200, 2, 1, 2, 2), (45, 7, 7, 3, 1, 5), (70, 9, 31, 3, 1, 2), (64, 13, 28, 1, 1, 2)]):
        l = wl.Layer("stage", C, 29, H, W, R, R, 1, sw, R // 2, R // 2, N=N, sparsity=0.6, dtype="f32", seed=980 + k)
        data = wl.prepare(l)
        ref = None
        plan = G.make_plan(l, data)
        buf = torch.full((data["x"].size + 8,), float("nan"), device="cuda")
        for td, tp, ns, cc in ((td, tp, ns, cc) for td in (16, 32) for tp in (1, 2, 3, 5, 9, 13, 1000) for ns in (1, 2, 3, 4) for cc in (32, 64, 96, 128, 256)):
            if tp >= l.P and tp != 1000 or tp != 1000 and ns > 1 or ns > N:
                continue
            try:
                _split(plan, tile_d=td, waves_m=1, tile_p=tp, sub_batch=ns, chunk_c=cc, **kw)
            except B.SparseConvError as e:
                assert e.status == 4
                continue
            t = plan.get_tuning()
            key = G.split_staging(l, t)
            blocks = -(-t.sub_batch * t.tile_p * l.Q // 16)           # of 16 positions; four waves along them in the one-shot form
            by_one = td == 32 and 16 < blocks <= 28 and not kw.get("producers")
            if seen.get((key, k), 0) >= 2 and (not by_one or key[0] in large):
                continue
            if ref is None:
                ref = G.oracle_out(l, data)
            shift = sum(seen.values()) % 4
            seen[key, k] = seen.get((key, k), 0) + 1
            if by_one:
                large.add(key[0])
            x = buf[shift:shift + data["x"].size]
            x.copy_(torch.from_numpy(np.ascontiguousarray(data["x"])).cuda().flatten())
            y = torch.full(ref.shape, float("nan"), device="cuda")
            print("case stage", form, key, shift, (C, H, W, R), t.as_dict(), flush=True)
            plan.forward(x.data_ptr(), y.data_ptr(), l.N, 0, 0, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            G.check(l, G.to_host(y), ref, f"stage {form} {key} {t.as_dict()}", tol=2e-6)
        plan.destroy()
    assert {key for key, _ in seen} == everything, everything - {key for key, _ in seen}
    assert kw.get("producers") or large == {1, 2, 4}, large


def test_autotune_gives_the_dense_weights_back_when_a_gather_kernel_wins():
    """A very sparse fp32 layer: the search tries the split form, for which it makes 32 MB of dense weights, installs
    a gather kernel and leaves none of them behind; a shape on the dense weights works afterwards."""
    import torch
    l = wl.Layer("verysparse", 2304, 2304, 5, 5, 1, 1, 1, 1, 0, 0, N=1, sparsity=0.998, dtype="f32", seed=7)
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    xd = G.to_device(data["x"])
    y = torch.empty((l.N, l.D, l.P, l.Q), device="cuda")
    ws = torch.empty(plan.autotune_workspace_size(l.N), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plan.autotune(xd.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    after = torch.cuda.mem_get_info()[0]
    assert not _is_split(plan.get_tuning()), plan.get_tuning().as_dict()
    assert before - after < 16 << 20, (before, after)
    G.check(l, G.run_gpu(plan, data["x"]), G.oracle_out(l, data), "after the search")
    _split(plan)
    G.check(l, G.run_gpu(plan, data["x"]), G.oracle_out(l, data), "split form after the search")
    plan.destroy()


def test_fp32_split_form_is_refused_where_it_does_not_apply():
    l = wl.Layer("splitno", 96, 12, 6, 6, N=2, sparsity=0.7, dtype="f32", seed=6)
    data = wl.prepare(l)

    def refused(plan, **kw):
        before = plan.get_tuning().as_dict()
        with pytest.raises(B.SparseConvError) as e:
            _split(plan, **kw)
        assert e.value.status == 4 and plan.get_tuning().as_dict() == before

    plan = G.make_plan(l, data)
    # (96 channels in chunks of 32: four shares would leave a workgroup without a chunk)
    for kw in (dict(chunk_c=32, split_n=4), dict(chunk_c=33), dict(tile_d=48), dict(wg_threads=384), dict(wsrc=1), dict(pack=2),
               dict(producers=2), dict(stage_rows=1), dict(ragged=2), dict(tile_d=32, waves_m=4)):
        refused(plan, **kw)
    plan.set_epilogue(relu=True)
    refused(plan)
    plan.destroy()
    for bad in (np.inf, np.nan, 1e-35):                       # weights that three terms do not hold
        va = data["values"].copy()
        va[5] = bad
        plan = B.Plan.create_csr(G.layer_desc(l), B.DTYPES["f32"], data["rowptr"], data["colidx"], va, None, None)
        refused(plan)
        plan.destroy()
    ci = data["colidx"].copy()
    ci[1] = ci[0]                                             # a column stored twice in one row
    plan = B.Plan.create_csr(G.layer_desc(l), B.DTYPES["f32"], data["rowptr"], ci, data["values"], None, None)
    refused(plan)
    plan.destroy()
    l16 = l.replace(dtype="f16")
    plan = G.make_plan(l16, wl.prepare(l16))
    refused(plan)
    plan.destroy()


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("C,D,H,W,k,stride,pad,N,sparsity", [
    (40, 24, 9, 9, 3, 1, 1, 3, 0.6),          # few output channels
    (64, 130, 10, 10, 3, 1, 1, 2, 0.5),       # matrix-core tile for every type
    (64, 130, 10, 10, 3, 1, 1, 2, 0.92),      # one weight in 12.5: not for fp32 and fp16
    (64, 130, 10, 10, 3, 1, 1, 2, 0.96),      # one weight in 25
    (384, 520, 3, 4, 3, 1, 1, 2, 0.96),       # the same in a large table
    (100, 200, 7, 7, 1, 1, 0, 5, 0.5),        # 10000 entries: for the codebook types only
    (33, 70, 8, 5, 3, 2, 1, 5, 0.9),          # rows of 30
    (3, 16, 12, 12, 3, 1, 1, 1, 0.5),
    (64, 48, 260, 260, 3, 1, 1, 1, 0.8)])     # rows of 115; the slab of such a plane does not fit for every type
def test_default_launch_shape_of_a_new_plan(dtype, C, D, H, W, k, stride, pad, N, sparsity):
    """A plan nobody has tuned takes the matrix-core tile (fp32: the split form) where its table is large and dense
    enough for the type and each column is stored once, and a gather kernel otherwise; both give the oracle's
    result."""
    for dup in (False, True):
        l = wl.Layer("default", C, D, H, W, k, k, stride, stride, pad, pad, N=N, sparsity=sparsity, dtype=dtype, seed=C + D)
        data = wl.prepare(l, ragged=False)
        if dup:
            data["colidx"] = data["colidx"].copy()
            data["colidx"][1] = data["colidx"][0]
        plan = G.make_plan(l, data)
        t = plan.get_tuning()
        matrix = t.variant == B.SC_VARIANT_DENSE or (t.variant == B.SC_VARIANT_SLAB and t.pipeline == 3)
        entries, per = {"f32": (32768, 12), "f16": (16384, 12), "i8": (16384, 24)}.get(dtype, (8192, 24))
        block = 64 if dtype in ("i8", "cb4") else 32
        K = (C + block - 1) // block * block * k * k
        takes = D >= 32 and l.n >= 32 and D * l.n >= entries and l.n * 32 >= K and not dup
        large = l.n >= 128 and D * l.n >= 2 * entries
        takes = takes and (large or l.n * per >= K)
        got = G.run_gpu(plan, data["x"])
        try:
            plan.set_tuning(B.sc_tuning_t(), wg_threads=1024, wsrc=0 if dtype in ("cb4", "cb4h") else 1)
        except B.SparseConvError:
            plan.set_tuning(B.sc_tuning_t())
        if plan.get_tuning().variant == B.SC_VARIANT_GATHER:     # the slab does not fit
            takes = takes and (large or l.n >= 128 and l.n * 16 >= K)
        assert matrix == takes, (t.as_dict(), l.n, K)
        assert not matrix or (t.pipeline == 3) == (dtype == "f32")
        print("case default", dtype, C, D, sparsity, dup, t.as_dict(), flush=True)
        G.check(l, got, G.oracle_out(l, data), f"default {t.as_dict()}")
        plan.destroy()


@pytest.mark.parametrize("dtype,relu,pool,requant", [("f16", True, 2, False), ("i8", True, 2, True), ("cb4", False, 2, False), ("f16", True, 0, False), ("f32", True, 2, False)])
@pytest.mark.parametrize("P", [7, 21, 28])
def test_epilogue_on_a_plan_that_nobody_tuned(dtype, relu, pool, requant, P):
    """Large tables (the default is the matrix-core tile) under each epilogue: the plan keeps a matrix-core tile,
    another one where pooling rules its own out, and gives the oracle's result; fp32 goes to GATHER.  A shape that
    was set by hand and is ruled out goes to GATHER."""
    import oracle
    import torch
    l = wl.Layer("untuned", 96, 160, P, P, N=3, sparsity=0.75, dtype=dtype, seed=P)
    data = wl.prepare(l)
    acc = G.oracle_out(l, data)
    rq = (np.linspace(40.0, 160.0, l.D) / max(1.0, float(np.abs(acc).max()))).astype(np.float32) if requant else None
    want = oracle.epilogue(acc, relu=relu, pool=pool, requant_scale=rq)
    xd = G.to_device(data["x"])
    for by_hand in (False, True):
        plan = G.make_plan(l, data)
        matrix = plan.get_tuning().variant == B.SC_VARIANT_DENSE
        assert matrix == (dtype != "f32")
        if by_hand:
            if dtype == "f32":
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_SLAB, wsrc=1)
            else:
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, tile_p=3)
        plan.set_epilogue(relu=relu, pool=pool, requant_scale=rq)
        t = plan.get_tuning()
        print("case untuned epilogue", dtype, relu, pool, requant, P, by_hand, t.as_dict(), flush=True)
        assert t.variant == (B.SC_VARIANT_DENSE if matrix and not (by_hand and pool) else B.SC_VARIANT_GATHER)
        y = torch.empty(want.shape, dtype=torch.int8 if requant else B.torch_out_dtype(plan.dtype), device="cuda")
        ws = torch.empty(max(plan.workspace_size(l.N), 16), dtype=torch.uint8, device="cuda")
        plan.forward(xd.data_ptr(), y.data_ptr(), l.N, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = G.to_host(y)
        if requant:
            assert np.array_equal(got, want)
        else:
            G.check(l, got, want, f"untuned epilogue {t.as_dict()}")
        plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_matrix_core_tiles_run_a_batch_of_more_workgroups_than_one_launch_holds_in_slices(dtype):
    """A launch decodes at most 2^19 - 1 workgroups; 2^19 + 3 samples of one workgroup each take two."""
    n = 2 ** 19 + 3
    l = wl.Layer("slices", 4, 3, 1, 2, 1, 1, 1, 1, 0, 0, N=n, sparsity=0.4, dtype=dtype, seed=12)
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    if dtype == "f32":
        _split(plan, tile_p=1, sub_batch=1)
    else:
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, tile_p=1, sub_batch=1)
    print("case slices", dtype, plan.get_tuning().as_dict(), flush=True)
    got = G.run_gpu(plan, data["x"])
    pick = [0, 1, 2 ** 19 - 2, 2 ** 19 - 1, 2 ** 19, n - 1]
    G.check(l, got[pick], G.oracle_out(l, data, samples=pick), f"slices {dtype}")
    assert not np.any(got.view(np.uint8).reshape(n, -1).min(axis=1) == 0x7f)      # every sample was written
    plan.destroy()


@pytest.mark.parametrize("dtype", ["i8", "cb4"])
@pytest.mark.parametrize("C,D,H,W,k,N,relu", [(5, 37, 6, 8, 3, 3, True), (64, 18, 2, 2, 3, 7, False), (70, 64, 4, 3, 1, 5, True), (9, 16, 5, 5, 3, 2, True)])
def test_requantised_codes_stored_four_positions_at_a_time(dtype, C, D, H, W, k, N, relu):
    """Planes of whole groups of four positions (the last shape is not one: byte stores), output channels that are
    no multiple of 16 or 4, batches that end inside a workgroup, tiles of one row and of whole planes, and a y that
    is not aligned to four bytes: bit-exact codes, nothing written past the end."""
    import oracle
    import torch
    l = wl.Layer("quads", C, D, H, W, k, k, 1, 1, k // 2, k // 2, N=N, sparsity=0.5, dtype=dtype, seed=C + D)
    data = wl.prepare(l)
    acc = G.oracle_out(l, data)
    rq = (np.linspace(40.0, 160.0, D) / max(1.0, float(np.abs(acc).max()))).astype(np.float32)
    want = oracle.epilogue(acc, relu=relu, pool=0, requant_scale=rq)
    plan = G.make_plan(l, data)
    plan.set_epilogue(relu=relu, requant_scale=rq)
    xd = G.to_device(data["x"])
    ran = 0
    for kw in ({}, {"tile_d": 16, "tile_p": 1}, {"tile_d": 32, "waves_m": 2, "tile_p": 1000, "sub_batch": 4}, {"tile_d": 64, "waves_m": 4, "tile_p": 2},
               {"tile_d": 16, "tile_p": 1000, "split_n": 2}, {"wg_threads": 512, "tile_d": 32}, {"pipeline": 1, "tile_d": 32}):
        try:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, **kw)
        except B.SparseConvError as e:
            assert e.status == 4
            continue
        for shift in (0, 1):
            buf = torch.full((want.size + 16,), 0x55, dtype=torch.int8, device="cuda")
            print("case quads", dtype, C, D, kw, shift, flush=True)
            plan.forward(xd.data_ptr(), buf.data_ptr() + shift, N, 0, 0, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            got = buf.cpu().numpy()
            assert np.array_equal(got[shift:shift + want.size].reshape(want.shape), want), (dtype, kw, shift)
            assert np.all(got[:shift] == 0x55) and np.all(got[shift + want.size:] == 0x55)
            ran += 1
    assert ran >= 8
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f16", "i8", "cb4", "cb4h"])
@pytest.mark.parametrize("name,C,D,H,W,R,S,sh,sw,ph,pw,N", [
    ("odd_runs", 70, 37, 9, 13, 3, 3, 1, 1, 1, 1, 3),            # rows of 13: loads that end before a run's end
    ("short_runs", 130, 20, 5, 3, 3, 3, 1, 1, 1, 1, 7),          # runs shorter than the widest load; groups of four over samples
    ("flat", 147, 50, 1, 23, 1, 3, 1, 1, 0, 0, 5),               # rows without padding columns, 21 positions a sample
    ("flat7", 40, 130, 7, 7, 1, 1, 1, 1, 0, 0, 6),
    ("strided", 33, 16, 11, 10, 3, 3, 2, 2, 1, 1, 4),
    ("padding_tiles", 16, 33, 3, 4, 1, 1, 1, 1, 4, 4, 2),        # tiles that lie in the padding altogether
    ("one_step", 8, 64, 6, 6, 1, 1, 1, 1, 0, 0, 2)])             # fewer steps than groups that split them
def test_dense_contraction_split_among_the_waves(name, C, D, H, W, R, S, sh, sw, ph, pw, N, dtype):
    """tuning.buffers on the one-shot matrix-core tile: 1, 2, 4 or 8 groups of waves split the contraction and meet in
    LDS, with every layout of four and eight waves, tiles of rows and whole planes of several samples, one and
    several chunks, and inputs that start at any element; other values are refused."""
    import torch
    l = wl.Layer(name, C, D, H, W, R, S, sh, sw, ph, pw, N=N, sparsity=0.6, dtype=dtype, seed=901)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    ran = set()
    for threads in (256, 512):
        for kg in (1, 2, 4, 8):
            for wm, td in ((1, 16), (1, 64), (2, 32), (2, 128), (4, 64)):
                for extra in ({"tile_p": 2}, {"tile_p": 1000, "sub_batch": 3}, {"tile_p": 1, "chunk_c": 64}):
                    try:
                        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, wg_threads=threads, waves_m=wm, tile_d=td, buffers=kg, **extra)
                    except B.SparseConvError as e:
                        assert e.status == 4
                        continue
                    t = plan.get_tuning()
                    assert t.buffers == (0 if kg == threads // 256 else kg)
                    print("case split", name, dtype, t.as_dict(), flush=True)
                    G.check(l, G.run_gpu(plan, data["x"]), ref, f"{name} split {threads} {kg} {wm} {td} {extra}")
                    ran.add(kg)
    assert ran == {1, 2, 4, 8}, ran
    # x that is aligned to its elements only
    xd = G.to_device(np.ascontiguousarray(data["x"]))
    raw = torch.empty(xd.numel() + 1, dtype=xd.dtype, device="cuda")
    raw[1:].copy_(xd.reshape(-1))
    y = torch.empty((N, D, plan.info().P, plan.info().Q), dtype=B.torch_out_dtype(plan.dtype), device="cuda")
    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, wg_threads=512, waves_m=1, tile_d=32, tile_p=1)
    plan.forward(raw[1:].data_ptr(), y.data_ptr(), N, 0, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    G.check(l, G.to_host(y), ref, f"{name} shifted x")
    for bad in ({"buffers": 3}, {"buffers": 16}, {"buffers": 4, "waves_m": 4}, {"buffers": 2, "pipeline": 1}, {"buffers": 2, "split_n": 2, "tile_d": 16}):
        with pytest.raises(B.SparseConvError) as e:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, **{"wg_threads": 512, **bad})
        assert e.value.status == 4
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("C,D,H,W,N", [(70, 40, 8, 16, 3), (64, 24, 6, 8, 5), (40, 33, 4, 4, 7), (33, 18, 5, 7, 4)])
def test_dense_epilogue_with_the_contraction_split(C, D, H, W, N, dtype):
    """The fused epilogue behind 1, 2, 4 and 8 groups of waves: pooled rows of whole groups of four outputs and odd
    ones, tiles of rows and planes of several samples, requantised codes (bit-exact) and fp16."""
    import oracle
    l = wl.Layer("episplit", C, D, H, W, 3, 3, 1, 1, 1, 1, N=N, sparsity=0.6, dtype=dtype, seed=902)
    data = wl.prepare(l)
    acc = oracle.sparse_conv(data["x"], data["rowptr"], data["colidx"], data["values"], l.R, l.S, (1, 1), (1, 1),
                             codebook=data["codebook"], out_dtype=np.int32 if dtype == "i8" else np.float32)
    plan = G.make_plan(l, data)
    rq = (100.0 / max(1.0, float(np.abs(acc).max())) * (0.5 + np.random.default_rng(3).random(D))).astype(np.float32) if dtype == "i8" else None
    for relu, pool, requant in ((1, 2, 1), (1, 0, 1), (1, 2, 0), (0, 2, 0), (1, 0, 0)):
        if requant and dtype != "i8":
            continue
        plan.set_epilogue(relu=relu, pool=pool, requant_scale=rq if requant else None)
        out_dt = np.int8 if requant else G.NP_OUT[dtype]
        ref = oracle.epilogue(acc, relu=bool(relu), pool=pool, requant_scale=rq if requant else None, out_dtype=None if requant else G.NP_OUT[dtype])
        ran = set()
        for threads, kg, wm, td in ((256, 1, 2, 32), (256, 4, 1, 32), (512, 1, 2, 64), (512, 2, 2, 64), (512, 4, 1, 16), (512, 4, 2, 32), (512, 8, 1, 32)):
            for extra in ({"tile_p": 2}, {"tile_p": 4}, {"tile_p": 1000, "sub_batch": 2}):
                try:
                    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, wg_threads=threads, waves_m=wm, tile_d=td, buffers=kg, **extra)
                except B.SparseConvError as e:
                    assert e.status == 4
                    continue
                print("case episplit", dtype, (relu, pool, requant), plan.get_tuning().as_dict(), flush=True)
                got = _run_epi(plan, l, data["x"], out_dt)
                if dtype == "i8":
                    assert np.array_equal(got, ref), (relu, pool, requant, threads, kg, extra, np.count_nonzero(got != ref))
                else:
                    G.check(l, got, ref, f"episplit {(relu, pool)} {threads} {kg} {extra}")
                ran.add(kg)
        assert ran == {1, 2, 4, 8}, ran
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("W", [1, 2, 3, 7, 8, 9, 16, 17, 25, 33, 40])
def test_dense_staging_deals_blocks_by_fours(W, dtype):
    """The blocks of a channel group are dealt to the lanes four at a time: 1 .. 5 and more of them in a tile, whole and
    shared last blocks, one and several samples, rows that carry padding and rows staged as one run, a last channel group that is not whole."""
    for C, H, pad, N in ((40, 1, 0, 3), (150, 3, 1, 2), (64, 2, 1, 5)):
        l = wl.Layer("quads", C, 24, H, W, 1 if H == 1 else 3, 1 if W < 3 and not pad else 3, 1, 1, pad if H > 1 else 0, pad, N=N, sparsity=0.5, dtype=dtype, seed=910 + W)
        data = wl.prepare(l)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        ran = 0
        for threads in (256, 512):
            for extra in ({"tile_p": 1}, {"tile_p": 1000, "sub_batch": 2}, {"tile_p": 1000, "sub_batch": 4, "chunk_c": 64}):
                try:
                    plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, wg_threads=threads, waves_m=1, tile_d=32, **extra)
                except B.SparseConvError as e:
                    assert e.status == 4
                    continue
                print("case quads", dtype, C, H, W, plan.get_tuning().as_dict(), flush=True)
                G.check(l, G.run_gpu(plan, data["x"]), ref, f"quads {C} {H} {W} {threads} {extra}")
                ran += 1
        assert ran >= 2
        plan.destroy()


@pytest.mark.parametrize("dtype", ["f16", "i8"])
def test_dense_one_shot_kernel_in_every_instantiation(dtype):
    """Every wave tile with every width of a staging load, runs that are whole loads and runs that end in a load overlapping the one
    before, a last chunk that is not whole.  What a shape runs is worked out by tile_staging; none of it may be left out."""
    block = 64 if dtype == "i8" else 32
    seen = set()
    for k, (C, H, W, R) in enumerate([(2060, 1, 16, 1), (2060, 3, 5, 1), (1030, 2, 16, 1), (1030, 5, 6, 1), (1030, 4, 16, 1), (1030, 7, 9, 1), (1030, 7, 16, 1),
                                      (1030, 7, 15, 1), (1030, 8, 16, 1), (1030, 9, 13, 1), (200, 8, 15, 3), (70, 6, 9, 3)]):
        l = wl.Layer("inst", C, 70, H, W, R, R, 1, 1, R // 2, R // 2, N=2, sparsity=0.9, dtype=dtype, seed=990 + k)
        data = wl.prepare(l)
        ref = G.oracle_out(l, data)
        plan = G.make_plan(l, data)
        for td, threads, kg, cc in ((td, threads, kg, cc) for td in (16, 32, 64) for threads in (256, 512) for kg in (4, 8) for cc in (32, 64, 128, 256, 512, 1024, 2048)):
            if cc % block:
                continue
            try:
                plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, tile_d=td, waves_m=1, wg_threads=threads, buffers=kg, wg_per_cu=1, chunk_c=cc, tile_p=1000, sub_batch=1)
            except B.SparseConvError as e:
                assert e.status == 4
                continue
            key = G.tile_staging(l, plan.get_tuning())
            if key in seen:
                continue
            seen.add(key)
            print("case inst", dtype, key, plan.get_tuning().as_dict(), flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"inst {dtype} {key}")
        plan.destroy()
    assert seen == {((m, n, c), tail) for m in (1, 2, 4) for n in (1, 2, 4, 7, 8) for c in (1, 2, 4, 8) for tail in (False, True)
                    if (m < 4 or n <= 4) and (c > 1 or not tail)}


@pytest.mark.parametrize("pool", [0, 2])
@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("D,tile_d,threads,split_n", [(37, 64, 256, 2), (16, 16, 256, 16), (37, 64, 512, 2), (130, 128, 256, 16)])
def test_dense_blocks_per_workgroup_more_than_the_layer_has(D, tile_d, threads, split_n, dtype, pool):
    """tuning.split_n beyond the blocks of output channels of the layer is cut to them, and to the plain one-shot form where
    there is one: the tile that runs is the one that the plan reports, so that installing the report again changes nothing."""
    import oracle
    l = wl.Layer("dlclamp", 40, D, 8, 16, 3, 3, 1, 1, 1, 1, N=3, sparsity=0.6, dtype=dtype, seed=920)
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    plan.set_epilogue(relu=False, pool=pool)
    shape = dict(variant=B.SC_VARIANT_DENSE, tile_d=tile_d, waves_m=2 if tile_d == 128 else 1, wg_threads=threads, split_n=split_n, tile_p=2)
    if pool and D > tile_d:                                  # (several blocks on one tile do not pool)
        with pytest.raises(B.SparseConvError) as e:
            plan.set_tuning(B.sc_tuning_t(), **shape)
        assert e.value.status == 4
        plan.destroy()
        return
    ref = oracle.epilogue(oracle.sparse_conv(data["x"], data["rowptr"], data["colidx"], data["values"], l.R, l.S, (1, 1), (1, 1),
                                             out_dtype=np.int32 if dtype == "i8" else np.float32), relu=False, pool=pool, out_dtype=G.NP_OUT[dtype])
    plan.set_tuning(B.sc_tuning_t(), **shape)
    first, lds = plan.get_tuning(), plan.info().lds_bytes
    blocks = -(-D // tile_d)
    assert first.split_n == (min(split_n, blocks) if blocks > 1 else 0)
    plan.set_tuning(first)
    assert plan.get_tuning().as_dict() == first.as_dict() and plan.info().lds_bytes == lds
    for k in range(2):
        if k:
            plan.set_tuning(B.sc_tuning_t(), **shape)
        print("case dlclamp", D, dtype, pool, plan.get_tuning().as_dict(), plan.info().lds_bytes, flush=True)
        G.check(l, _run_epi(plan, l, data["x"], G.NP_OUT[dtype]), ref, f"dlclamp {D} {pool} {k}")
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("D,W", [(20, 9), (37, 9), (100, 9), (300, 9), (37, 80), (100, 80), (100, 128)])
def test_dense_defaults_beside_the_contraction_split(D, W, dtype):
    """tuning.buffers with every other field left to the heuristics: waves_m, tile_d and wg_threads follow the waves that the groups
    leave, and only more groups than waves are refused."""
    l = wl.Layer("splitdef", 70, D, 5, W, 3, 3, 1, 1, 1, 1, N=2, sparsity=0.6, dtype=dtype, seed=930)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    for threads in (0, 256, 512):
        for kg in (0, 1, 2, 4, 8):
            shape = dict(variant=B.SC_VARIANT_DENSE, wg_threads=threads, buffers=kg)
            if (threads, kg) == (256, 8):
                with pytest.raises(B.SparseConvError) as e:
                    plan.set_tuning(B.sc_tuning_t(), **shape)
                assert e.value.status == 4
                continue
            plan.set_tuning(B.sc_tuning_t(), **shape)
            t = plan.get_tuning()
            waves = 8 if threads == 512 or kg == 8 else 4
            assert t.wg_threads == 64 * waves and t.buffers == (0 if kg == waves // 4 else kg)
            print("case splitdef", D, W, dtype, t.as_dict(), flush=True)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"splitdef {D} {W} {threads} {kg}")
    plan.destroy()


@pytest.mark.parametrize("name,C,D,H,W,stride,dtype,sparsity,split", [
    ("halo", 283, 68, 20, 17, 2, "i8", 0.7, False),           # tiles of two rows: five staged rows for two of outputs
    ("halo", 80, 383, 6, 6, 1, "cb4h", 0.6, False),
    ("deep", 256, 256, 14, 14, 1, "f16", 0.8, True),
    ("deep", 512, 512, 4, 4, 1, "cb4h", 0.9, True)])
def test_default_tile_splits_the_contraction_only_where_large_batches_agree(name, C, D, H, W, stride, dtype, sparsity, split):
    """The tile of a plan that nobody has tuned: four and eight groups of waves (small tiles that stage their halo again
    and again) only where they are no slower at a batch of 128 than the best tile without."""
    l = wl.Layer(name, C, D, H, W, 3, 3, stride, stride, 1, 1, N=2, sparsity=sparsity, dtype=dtype, seed=940)
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    t = plan.get_tuning()
    print("case default split", t.as_dict(), flush=True)
    assert t.variant == B.SC_VARIANT_DENSE and (t.buffers >= 4) == split
    G.check(l, G.run_gpu(plan, data["x"]), G.oracle_out(l, data), f"{name} default")
    plan.destroy()


@pytest.mark.parametrize("name,C,D,HW,N,sparsity,dtype", [
    ("s56_conv3x3", 64, 64, 56, 32, 0.8, "f16"), ("s14_conv3x3", 256, 256, 14, 32, 0.8, "f16"), ("s7_conv3x3", 512, 512, 7, 32, 0.9, "f16"),
    ("vgg_4", 512, 512, 4, 64, 0.9, "cb4h"), ("vgg_4", 512, 512, 4, 64, 0.9, "i8"), ("vgg_16", 128, 128, 16, 64, 0.9, "i8")])
def test_contraction_split_on_whole_layers(name, C, D, HW, N, sparsity, dtype):
    """Four and eight groups of waves on layers of the workloads at full batch: hundreds of steps a wave, tables of more than
    one register, several chunks, the order of the workgroups by output channels (512 x 512)."""
    l = wl.Layer(name, C, D, HW, HW, 3, 3, 1, 1, 1, 1, N=N, sparsity=sparsity, dtype=dtype, seed=950)
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    x_dev = G.to_device(np.ascontiguousarray(data["x"]))
    ran = []
    for shape in (dict(), dict(wg_threads=512, tile_d=128, waves_m=2, tile_p=4, buffers=4), dict(wg_threads=512, tile_d=64, waves_m=1, tile_p=2, buffers=8),
                  dict(wg_threads=512, tile_d=64, waves_m=1, tile_p=1, chunk_c=128, buffers=8), dict(wg_threads=256, tile_d=32, waves_m=1, tile_p=2, buffers=4),
                  dict(wg_threads=512, tile_d=32, waves_m=1, tile_p=1000, sub_batch=2, chunk_c=256, buffers=4)):
        try:
            plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, **shape)
        except B.SparseConvError as e:
            assert e.status == 4                             # (whole planes of more positions than the waves hold)
            continue
        t = plan.get_tuning()
        print("case whole layer", name, dtype, t.as_dict(), flush=True)
        res = G.full_batch_parity(l, data, plan, x_dev=x_dev)
        assert res["ok"], (shape, res)
        ran.append(t.buffers)
    assert 8 in ran and 4 in ran
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("name,C,D,H,W,R,S,stride,ph,pw,N,shapes", [
    ("more positions than threads", 40, 20, 9, 70, 3, 3, 1, 1, 1, 2, [dict(tile_p=6, tile_d=32), dict(tile_p=2, tile_d=16, wg_threads=512)]),
    ("several samples, the last group short", 70, 20, 3, 3, 3, 3, 1, 2, 2, 5, [dict(tile_p=5, sub_batch=3), dict(tile_p=5, sub_batch=2, wg_threads=512)]),
    ("columns only", 150, 37, 1, 30, 1, 5, 1, 0, 2, 3, [dict(tile_p=1), dict(tile_p=1, sub_batch=2, chunk_c=64)]),
    ("rows only", 33, 16, 7, 9, 3, 1, 1, 1, 0, 2, [dict(tile_p=3), dict(tile_p=7, sub_batch=2)]),
    ("strided", 70, 20, 11, 13, 3, 3, 2, 1, 1, 3, [dict(tile_p=2, chunk_c=64), dict(tile_p=6, wg_threads=512)]),
    ("one column of input", 64, 16, 5, 1, 3, 3, 1, 1, 1, 2, [dict(tile_p=2), dict(tile_p=5)]),
])
def test_dense_padding_is_cleared_and_nothing_else(name, C, D, H, W, R, S, stride, ph, pw, N, shapes, dtype):
    """The padding of a staged tile is cleared position by position, next to the staging: right whatever the LDS holds when the
    workgroup starts.  A launch on NaN (on codes of 127) runs ahead, so that a position left out shows."""
    import torch
    l = wl.Layer("pad", C, D, H, W, R, S, stride, stride if S > 1 else 1, ph, pw, N=N, sparsity=0.6, dtype=dtype, seed=940)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    dirty = wl.Layer("dirty", 64, 64, 32, 32, 3, 3, 1, 1, 1, 1, N=32, sparsity=0.6, dtype=dtype, seed=941)
    ddata = wl.prepare(dirty)
    dplan = G.make_plan(dirty, ddata)
    dplan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, tile_p=8, tile_d=32, wg_threads=256)
    dx = torch.full((32, 64, 32, 32), float("nan") if dtype == "f16" else 127, device="cuda", dtype=torch.float16 if dtype == "f16" else torch.int8)
    dy = torch.empty((32, 64, 32, 32), device="cuda", dtype=B.torch_out_dtype(dplan.dtype))
    plan = G.make_plan(l, data)
    for shape in shapes:
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, **shape)
        print("case pad", name, dtype, plan.get_tuning().as_dict(), flush=True)
        for k in range(2):
            B.forward_torch(dplan, dx, dy)
            G.check(l, G.run_gpu(plan, data["x"]), ref, f"pad {name} {shape} {k}")
    plan.destroy()
    dplan.destroy()


@pytest.mark.parametrize("name,C,D,H,W,R,S,stride,ph,pw,N,sparsity", [
    ("a step for some groups only", 32, 20, 6, 9, 1, 1, 1, 0, 0, 3, 0.5),
    ("steps no multiple of the groups, a last chunk of one block", 100, 37, 9, 8, 3, 3, 1, 1, 1, 2, 0.6),
    ("more steps than a table holds", 300, 40, 5, 6, 3, 3, 1, 1, 1, 2, 0.8),
    ("more steps than two tables hold", 1100, 24, 4, 7, 3, 3, 2, 1, 1, 2, 0.9),
    ("one dimension", 70, 33, 1, 40, 1, 5, 1, 0, 2, 3, 0.5),
    ("rows of two weights", 64, 18, 7, 7, 3, 3, 1, 1, 1, 2, 0.997),
])
def test_fp32_split_form_steps_from_tables(name, C, D, H, W, R, S, stride, ph, pw, N, sparsity):
    """The steps of a wave come from tables of 64: one-shot and pipelined, two and four groups of waves (tuning.buffers = 4), every
    wave tile that fits, chunks of one to all channel blocks; no further from 64 bits than 2e-6 of the largest output (the sums
    are of at most 1000 products of 24-bit factors, rounded once for each 32 channels of a tap)."""
    l = wl.Layer("tables", C, D, H, W, R, S, stride, stride if S > 1 else 1, ph, pw, N=N, sparsity=sparsity, dtype="f32", seed=950)
    data = wl.prepare(l)
    ref = G.oracle_out(l, data)
    plan = G.make_plan(l, data)
    P = plan.info().P
    ran = 0
    for td, wm in ((16, 1), (32, 1), (32, 2), (64, 2), (64, 4)):
        for kw in (dict(buffers=4, producers=4), dict(producers=4), dict(wg_threads=256), dict(wg_threads=512)):
            for cc, tp in ((32, 1), (64, P), (0, 2)):
                try:
                    _split(plan, tile_d=td, waves_m=wm, chunk_c=cc, tile_p=tp, **kw)
                except B.SparseConvError as e:
                    assert e.status == 4
                    continue
                t = plan.get_tuning()
                assert t.buffers == kw.get("buffers", 0) and t.producers == kw.get("producers", 0)
                print("case tables", name, t.as_dict(), flush=True)
                G.check(l, G.run_gpu(plan, data["x"]), ref, f"tables {name} {td} {wm} {kw} {cc} {tp}", tol=2e-6)
                shape, lds = t.as_dict(), plan.info().lds_bytes
                plan.set_tuning(t)                            # the report installs the same shape again
                assert plan.get_tuning().as_dict() == shape and plan.info().lds_bytes == lds
                ran += 1
    assert ran >= 20
    for bad in (dict(buffers=4), dict(buffers=8, producers=4), dict(buffers=2, producers=4), dict(buffers=4, producers=4, waves_m=4, tile_d=64),
                dict(buffers=4, producers=4, wg_threads=256)):
        before = plan.get_tuning().as_dict()
        with pytest.raises(B.SparseConvError) as e:
            _split(plan, **bad)
        assert e.value.status == 4 and plan.get_tuning().as_dict() == before
    plan.destroy()


def test_a_forward_call_takes_no_time_per_tile_on_the_host():
    """A tall layer without padding columns in tiles of one row: 200000 tiles, and a call that only launches them.  (Their count
    must not be walked over in front of every launch, which took 140 us here.)"""
    import time
    import torch
    l = wl.Layer("tall", 32, 16, 200000, 1, 1, 1, 1, 1, 0, 0, N=1, sparsity=0.5, dtype="f32", seed=960)
    data = wl.prepare(l)
    plan = G.make_plan(l, data)
    x = G.to_device(data["x"])
    y = torch.empty((1, l.D, l.P, l.Q), device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    seconds = {}
    for tp in (64, 1):
        _split(plan, tile_p=tp, tile_d=16, waves_m=1)
        print("case tall", plan.get_tuning().as_dict(), flush=True)
        times = []
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            plan.forward(x.data_ptr(), y.data_ptr(), 1, 0, 0, stream)
            times.append(time.perf_counter() - t0)
        torch.cuda.synchronize()
        seconds[tp] = min(times)
        G.check(l, G.to_host(y), G.oracle_out(l, data), f"tall {tp}")
    print("   seconds of a call", seconds, flush=True)
    assert seconds[1] <= 3 * seconds[64] + 30e-6, seconds
    plan.destroy()


@pytest.mark.parametrize("dtype,C", [("f16", 16_000_000), ("i8", 32_000_000)])
def test_dense_tile_on_weights_of_more_than_4_gb_a_row_block(dtype, C):
    """The one-shot matrix-core kernel where 16 output channels have more than 4 GB of dense weights (9 taps x 500000 channel blocks of
    1 KB, 36.9 GB in all): a few weights anywhere, and in the last channels, whose last tap lies past 4 GB.  Every output against
    the sum of its products; fp16 to its rounding (2^-11) and that of 60 fp32 sums."""
    import torch
    D, H, W, N = 40, 2, 2, 2
    rng = np.random.default_rng(970)
    K = 9 * C
    rowptr = np.zeros(D + 1, np.int32)
    cols = []
    for d in range(D):
        c = np.concatenate([rng.integers(0, K, 40), K - 1 - rng.integers(0, 9 * 500, 20)])
        cols.append(np.unique(c))
        rowptr[d + 1] = rowptr[d] + cols[-1].size
    colidx = np.concatenate(cols).astype(np.int32)
    if dtype == "f16":
        values, scales = rng.normal(0, 0.05, colidx.size).astype(np.float16), None
        x = rng.integers(-100, 100, (N, C, H, W), dtype=np.int8).astype(np.float16)
    else:
        values, scales = rng.integers(-127, 128, colidx.size).astype(np.int8), np.full(D, 0.01, np.float32)
        x = rng.integers(-127, 128, (N, C, H, W), dtype=np.int8)
    ref = np.zeros((N, D, H, W))
    mag = np.zeros((N, D, H, W))
    for d in range(D):
        for j in range(rowptr[d], rowptr[d + 1]):
            c, tap = divmod(int(colidx[j]), 9)
            xp = np.pad(x[:, c].astype(np.float64), ((0, 0), (1, 1), (1, 1)))[:, tap // 3:tap // 3 + H, tap % 3:tap % 3 + W]
            ref[:, d] += float(values[j]) * xp
            mag[:, d] += abs(float(values[j])) * np.abs(xp)
    plan = B.Plan.create_csr(B.make_layer(C, D, H, W, 3, 3, (1, 1), (1, 1)), B.DTYPES[dtype], rowptr, colidx, values, scales)
    xd = G.to_device(x)
    y = torch.empty((N, D, H, W), device="cuda", dtype=B.torch_out_dtype(plan.dtype))
    for shape in (dict(tile_d=16, waves_m=1, wg_threads=512, buffers=8, chunk_c=2048), dict(tile_d=64, waves_m=2, sub_batch=2, chunk_c=1024)):
        plan.set_tuning(B.sc_tuning_t(), variant=B.SC_VARIANT_DENSE, tile_p=H, **shape)
        print("case wide", dtype, plan.get_tuning().as_dict(), flush=True)
        y.view(torch.uint8).fill_(0x7f)
        plan.forward(xd.data_ptr(), y.data_ptr(), N, 0, 0, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = G.to_host(y).astype(np.float64)
        if dtype == "i8":
            assert np.array_equal(got, ref)
        else:
            assert np.all(np.abs(got - ref) <= 2.0 ** -11 * np.abs(ref) + 60 * 2.0 ** -24 * mag)
    plan.destroy()
