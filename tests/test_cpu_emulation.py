"""The library's kernels compiled for host threads (tests/cpu_emul) against the oracle, on the CPU.

Not a product path: the stand-in runs one OS thread per GPU thread so that the control flow, indexing and
synchronisation of the kernels can be exercised (and debugged with host tools) where there is no GPU."""
import ctypes
import math
import shutil

import numpy as np
import pytest

from paper_2507_07990_amd import workloads as wl
from tests import parity as P

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


class _EmulLib:
    STTM_BF16, STTM_F32, STTM_F16 = 1, 0, 2

    def __init__(self, rc):
        self._lib = rc.load()
        self._lib.sttm_node_index.restype = int

    def sttm_node_index(self, H, W, R, lvl, by, bx):
        return self._lib.sttm_node_index(H, W, R, lvl, by, bx)


@pytest.fixture(scope="module")
def emul():
    from tests.cpu_emul import build_cpu, run_cpu
    build_cpu.build()
    return run_cpu, _EmulLib(run_cpu)


def _variant(seed, B, T, H, W, D, dtype):
    depth = int(math.log2(wl.pow2_ceil(max(H, W))))
    return wl.Workload("v", seed, B, T, H, W, D, dtype, depth, 0.1, 0.7)


@pytest.mark.parametrize("seed,B,T,H,W,D,dtype,kw", [
    (90, 1, 3, 8, 8, 16, "f32", dict(tau_s=0.8, tau_t=0.8)),
    (91, 2, 3, 5, 6, 24, "bf16", dict(keep=0.5)),
    (92, 1, 2, 9, 9, 16, "bf16", dict(tau_s=0.2, tau_t=0.2)),   # nodes that the reduce takes from stored sums
    (93, 1, 3, 8, 8, 24, "f16", dict(tau_s=0.7, tau_t=0.7)),    # half-precision input and output
    (94, 1, 2, 17, 18, 16, "f32", dict(tau_s=0.3, tau_t=0.3)),  # P = 32: two pyramid levels above the 8x8 units
    (97, 2, 3, 14, 14, 24, "bf16", dict(tau_s=0.8, tau_t=0.7, root_grid=4)),  # 4x4 roots: 4x4 join blocks everywhere
    (96, 1, 150, 2, 2, 8, "f32", dict(tau_s=1.0, tau_t=-2.0)),  # four chains of 150 cells: clusters summed item by item
])
def test_emulated_kernels_match_the_oracle(emul, seed, B, T, H, W, D, dtype, kw):
    run_cpu, fake = emul
    feats = wl.generate(_variant(seed, B, T, H, W, D, dtype))
    r = run_cpu.run_cpu(feats, **kw)
    info = P.check_parity(fake, feats, r, **kw)
    assert info["K"] == r.K and int(r.counts.sum()) == feats[..., 0].size


@pytest.mark.parametrize("mode,order", [("topleft_only", "zscan"), ("most_similar", "raster"), ("first_passing", "zscan")])
def test_emulated_destination_rules_orders_and_positions(emul, mode, order):
    """Alternating coarse / fine frames (the rules differ there), rows in either scan, position indices."""
    run_cpu, fake = emul
    cfg = wl.Workload("v", 95, 1, 5, 8, 8, 16, "f32", 2, 0.05, 0.9)
    feats = wl.generate_alternating(cfg, 0.7)
    kw = dict(tau_s=0.9, tau_t=0.8)
    r = run_cpu.run_cpu(feats, match=P.MODES[mode], order=P.ORDERS[order], positions=True, **kw)
    info = P.check_parity(fake, feats, r, mode=mode, order=order, **kw)
    assert "merged_pos_err" in info


def test_emulated_budget_threshold_left_to_the_consumer_kernels(emul):
    """Without a host pointer for the threshold the value of the search is found by the kernels that use it:
    same partition, same clusters, same rows."""
    run_cpu, fake = emul
    feats = wl.generate(_variant(91, 2, 3, 5, 6, 24, "bf16"))
    a = run_cpu.run_cpu(feats, keep=0.5)
    b = run_cpu.run_cpu(feats, keep=0.5, defer_tau=True)
    assert (a.node_map == b.node_map).all() and (a.cluster_ids == b.cluster_ids).all()
    assert (a.parent == b.parent).all() and a.K == b.K
    np.testing.assert_array_equal(a.merged, b.merged)


def test_emulated_searches_without_weights_work_out_no_address_of_them(emul):
    """The elements of a temporal search have no weights: there is no table, and nothing is added to its absent address for
    the videos after the first."""
    run_cpu, _ = emul
    lib = run_cpu.load()
    run_cpu.run_cpu(wl.generate(_variant(91, 3, 3, 5, 6, 24, "bf16")), keep=0.5, lib=lib)
    assert not lib.hip_emul_off_null()


@pytest.mark.parametrize("kw", [dict(keep=0.5), dict(tau_s=0.95, tau_t=0.6)])
def test_emulated_temporal_pass_without_the_cell_dot_products(emul, kw):
    """With the option off the temporal pass computes every pair itself: same partition and clusters as with the
    cell-to-cell dot products of the spatial pass, and parity with the oracle either way."""
    run_cpu, fake = emul
    feats = wl.generate(_variant(98, 2, 4, 9, 7, 24, "bf16"))
    a = run_cpu.run_cpu(feats, **kw)
    for level in (0, 2):
        b = run_cpu.run_cpu(feats, cell_dots=level, **kw)
        assert (a.node_map == b.node_map).all() and (a.cluster_ids == b.cluster_ids).all() and a.K == b.K
        P.check_parity(fake, feats, b, **kw)
    P.check_parity(fake, feats, a, **kw)


@pytest.mark.parametrize("B", [2, 33])
def test_emulated_thresholds_named_by_the_caller_stay_for_later_calls(emul, B):
    """As a launch argument (up to 32) or copied: a later call without thresholds finds every video's own."""
    run_cpu, _ = emul
    feats = wl.generate(_variant(87, B, 2, 2, 4, 8, "f32"))
    rng = np.random.default_rng(B)
    r = run_cpu.run_cpu(feats, tau_s=rng.uniform(-0.5, 0.7, B), tau_t=rng.uniform(-0.5, 0.5, B), again=True)
    for a, b in zip(r.first, (r.node_map, r.node_level, r.cluster_ids)):
        assert (a == b.reshape(-1)).all()
    assert (r.node_level > 0).any() and (r.cluster_ids != r.node_map).any()


def _uniform_partition(T, H, W, levels):
    """Node map and levels of a video whose frame t consists of the aligned blocks of level levels[t] only."""
    nm = np.empty((1, T, H, W), np.int32)
    nl = np.empty((1, T, H, W), np.uint8)
    yy, xx = np.meshgrid(np.arange(H), np.arange(W), indexing="ij")
    for t, lv in enumerate(levels):
        nm[0, t] = t * H * W + ((yy >> lv) << lv) * W + ((xx >> lv) << lv)
        nl[0, t] = lv
    return nm, nl


def test_emulated_temporal_work_lists_at_their_largest(emul):
    """The temporal pass lists its work per frame pair by join level and walks every list with a fixed stride and
    a trip count known on entry. On a full 32 x 32 grid, frames of uniform level meet so that every list is as long
    as it can get: 256 regions of 2 x 2 (levels 0|1), 64 blocks of 4 x 4 (1|2 and 2|0), 16 staged sums with 256
    nodes of 2 x 2 under them (3|1), and 1024 single cells under one whole-frame node (5|0) or under sixteen
    8 x 8 nodes (0|3). Every pair similarity, edge, cluster and merged row is compared with the oracle."""
    run_cpu, fake = emul
    levels = [5, 0, 3, 1, 2, 0, 1]
    T, H, W, D = len(levels), 32, 32, 8
    feats = wl.generate(wl.Workload("v", 99, 1, T, H, W, D, "f32", 5, 0.3, 0.8))
    nm, nl = _uniform_partition(T, H, W, levels)
    from oracle import sttm_oracle as O
    sp = O.SpatialResult()
    sp.node_map, sp.node_level = nm, nl
    r = run_cpu.run_cpu(feats, tau_s=0.5, tau_t=0.3, node_map_override=(nm, nl))
    tm, _ = P.check_temporal(fake, feats, r, sp, 0.3)
    P.check_reduce(feats, r, tm, False)


@pytest.fixture(scope="module")
def large(emul):
    """The build in which every input takes the pyramid kernel of the large ones."""
    from tests.cpu_emul import build_cpu
    return emul[0].load(build_cpu.build(large=True))


@pytest.mark.parametrize("seed,B,T,H,W,D,dtype,kw", [
    (90, 1, 3, 8, 8, 16, "f32", dict(tau_s=0.8, tau_t=0.8)),
    (91, 2, 3, 5, 6, 24, "bf16", dict(keep=0.5)),
    (92, 1, 2, 9, 9, 16, "bf16", dict(tau_s=0.2, tau_t=0.2, cell_dots=0)),
    (93, 1, 3, 8, 8, 24, "f16", dict(tau_s=0.7, tau_t=0.7, cell_dots=2)),
    (94, 1, 2, 17, 18, 16, "f32", dict(tau_s=0.3, tau_t=0.3)),
    (97, 1, 2, 14, 14, 24, "bf16", dict(tau_s=0.8, tau_t=0.7, root_grid=4, cell_dots=2)),
    (98, 1, 3, 9, 7, 520, "bf16", dict(tau_s=0.95, tau_t=0.6)),     # a second chunk with one live lane
    (88, 3, 1, 13, 11, 24, "f16", dict(tau_s=0.6, tau_t=0.6)),      # single images: a three-dimensional grid
])
def test_emulated_pyramid_kernel_of_large_inputs(emul, large, seed, B, T, H, W, D, dtype, kw):
    """Inputs that a host-thread run can afford take k_pyramid_tiles; here k_pyramid_stats works on them instead: parity
    with the oracle, and every table and output the same bit for bit as from the other kernel. (What a table holds where
    nothing is defined is the workspace's filling, the same in both.)"""
    run_cpu, fake = emul
    small = run_cpu.load()
    feats = wl.generate(_variant(seed, B, T, H, W, D, dtype))
    r = []
    for lib, kernel, other in ((large, b"k_pyramid_stats", b"k_pyramid_tiles"), (small, b"k_pyramid_tiles", b"k_pyramid_stats")):
        grid = (ctypes.c_uint * 3)()
        lib.hip_emul_last_grid(None, None)
        r.append(run_cpu.run_cpu(feats, lib=lib, **kw))
        assert lib.hip_emul_last_grid(kernel, grid) and not lib.hip_emul_last_grid(other, grid)
    oracle_kw = {k: v for k, v in kw.items() if k != "cell_dots"}
    P.check_parity(fake, feats, r[0], **oracle_kw)
    for name, a in vars(r[0]).items():
        if isinstance(a, np.ndarray):
            np.testing.assert_array_equal(a, getattr(r[1], name), err_msg=name)


@pytest.mark.parametrize("seed,B,T,H,W,D,dtype,cell_dots", [
    (101, 1, 9, 5, 7, 24, "bf16", 2),      # two runs of one video: the second's first frame is read by the first as well
    (102, 1, 7, 9, 5, 264, "f32", 1),      # one run per column; a unit of one row, a second chunk of two lanes
    (103, 3, 5, 12, 4, 16, "f16", 2),      # runs across the ends of videos; a tile beyond the edge
    (104, 5, 2, 3, 3, 8, "bf16", 1),       # level 2 is the root's: no unit sums
])
def test_emulated_walk_through_runs_of_frames(emul, large, seed, B, T, H, W, D, dtype, cell_dots):
    """Runs of more frames than the block places need to come round (three), against the kernel without runs, bit for bit."""
    run_cpu, _ = emul
    feats = wl.generate(_variant(seed, B, T, H, W, D, dtype))
    a, b = (run_cpu.run_cpu(feats, lib=lib, tau_s=0.8, tau_t=0.7, cell_dots=cell_dots) for lib in (large, run_cpu.load()))
    for name, x in vars(a).items():
        if isinstance(x, np.ndarray):
            np.testing.assert_array_equal(x, getattr(b, name), err_msg=name)


@pytest.mark.parametrize("noise", [0.0, 0.003])
def test_emulated_search_among_many_elements_of_one_bin(emul, large, noise):
    """Similarities that crowd in a bin or two, equal ones among them (still content): listing the bin's elements and
    searching those gives the thresholds, the partition and the clusters that the search of a small input gives."""
    run_cpu, _ = emul
    rng = np.random.default_rng(11)
    feats = (rng.standard_normal(16) + noise * rng.standard_normal((2, 4, 8, 8, 16)).round(1)).astype(np.float32)
    feats[:, 2] = feats[:, 1]                              # a frame that repeats: its pairs are all alike
    a, b = (run_cpu.run_cpu(feats, lib=lib, keep=0.4) for lib in (large, run_cpu.load()))
    for name in ("tau_s", "tau_t", "node_map", "cluster_ids"):
        np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)


@pytest.mark.parametrize("B,T,H,W,keep", [
    (1, 4, 8, 8, 0.5),       # one workgroup lists the cells
    (2, 5, 16, 16, 0.3),     # several; the second video's list lies behind the first one's
])
def test_emulated_searches_can_be_recorded_and_replayed(emul, large, B, T, H, W, keep):
    """Statistics as ordinary calls, then a budget search and the call that uses its threshold recorded and replayed: what
    every replay gives, and the same calls made again afterwards, is what they gave when they were first made."""
    run_cpu, _ = emul
    D = 8
    feats = wl.generate(_variant(105, B, T, H, W, D, "f32"))
    N = B * T * H * W
    h, need = ctypes.c_void_p(), large.sttm_workspace_bytes(B, T, H, W, D, 0, 1)
    ws, x = run_cpu._aligned(need, garbage=True), run_cpu._aligned(feats.nbytes, 16)
    x[:] = feats.view(np.uint8).reshape(-1)
    nm, cl, nl = np.zeros(N, np.int32), np.zeros(N, np.int32), np.zeros(N, np.uint8)
    ptr, share = run_cpu._p, (ctypes.c_double * B)(*[keep] * B)
    shape = (0, B, T, H, W, D, 1)

    def chk(rc):
        assert rc == 0, large.sttm_last_error(h)

    assert large.sttm_create(ctypes.byref(h), 0, None) == 0
    chk(large.sttm_set_workspace(h, ptr(ws), ctypes.c_size_t(need)))

    def spatial():
        chk(large.sttm_budget_threshold(h, 0, share, None))
        chk(large.sttm_spatial_quadtree(h, ptr(x), *shape, None, ptr(nm), ptr(nl)))

    def temporal():
        chk(large.sttm_budget_threshold(h, 1, share, None))
        chk(large.sttm_temporal_merge(h, ptr(x), ptr(nm), ptr(nl), None, ptr(cl)))

    for stats, search, out in ((lambda: chk(large.sttm_spatial_stats(h, ptr(x), *shape)), spatial, nm),
                               (lambda: chk(large.sttm_temporal_stats(h, ptr(x), ptr(nm), ptr(nl))), temporal, cl)):
        stats()
        search()                                           # (the targets are on the device from here on)
        want = out.copy()
        stats()
        large.hip_emul_record(1)
        search()
        large.hip_emul_record(0)
        for again in range(4):
            out[:] = -1
            assert large.hip_emul_replay() > 1
            np.testing.assert_array_equal(out, want, err_msg=f"replay {again}")
        out[:] = -1
        search()
        np.testing.assert_array_equal(out, want)
        assert 1 < len(np.unique(want)) < N
    large.sttm_destroy(h)


def test_emulated_kernels_run_clean_under_address_and_undefined_behaviour_sanitizers():
    """The host-thread build with -fsanitize=address,undefined (any report aborts): both dtypes, fixed thresholds and
    a budget, every output in a heap block of its exact size, the workspace of exactly sttm_workspace_bytes(); once
    with the pyramid kernel of small inputs and once with that of large ones."""
    import subprocess
    from concurrent.futures import ThreadPoolExecutor
    from tests.cpu_emul import build_cpu

    def one(is_large):
        return subprocess.run([build_cpu.build_sanitized(large=is_large)], capture_output=True, text=True, timeout=600)

    with ThreadPoolExecutor(2) as pool:
        for r in pool.map(one, (False, True)):
            assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
            assert r.stdout.count("case ") == 2
            assert "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr


def test_emulated_contexts_leave_the_runtime_alone_when_they_go(emul):
    """Destroying a context must not call the runtime's host allocator: outside the relaxed capture mode that ends a
    stream capture running on any other stream, and a free waits for the work of every context. A block goes to the
    next context instead; of many idle ones only a bounded number is kept, the rest freed in the relaxed mode."""
    lib = emul[0].load()
    lib.sttm_destroy.argtypes = [ctypes.c_void_p]

    def pinned():
        out = (ctypes.c_int * 3)()
        lib.hip_emul_pinned(out)
        return list(out)

    def create(n):
        hs = [ctypes.c_void_p() for _ in range(n)]
        assert all(lib.sttm_create(ctypes.byref(h), 0, None) == 0 for h in hs)
        return hs

    def destroy(hs):
        assert all(lib.sttm_destroy(h) == 0 for h in hs)

    _, freed, unguarded = pinned()
    destroy(create(2))
    assert pinned()[1:] == [freed, unguarded]          # nothing freed, no call outside the relaxed mode
    allocated = pinned()[0]
    destroy(create(2))
    assert pinned() == [allocated, freed, unguarded]   # the same two blocks again
    destroy(create(200))
    allocated, freed, after = pinned()
    assert after == unguarded and 0 < allocated - freed <= 64


@pytest.mark.parametrize("B,T,cell_dots", [(1, 1, 1), (3, 1, 1), (1, 2, 0)])
def test_emulated_pyramid_grid_without_frame_pairs_has_no_idle_workgroups(emul, B, T, cell_dots):
    """Where no two workgroups share rows (single images, frame-to-frame products off) the pass is numbered plainly: as
    many workgroups as there are (frame, unit, chunk) triples, which the hardware deals to all dies in turn. A grid laid
    out in one range of frames per die would put a single image on one of the eight."""
    run_cpu, _ = emul
    H, W, D = 9, 10, 72                                # 4 units of 8x8, fp32: one chunk of 64 x 4 channels
    lib = run_cpu.load()
    lib.hip_emul_last_grid(None, None)
    run_cpu.run_cpu(wl.generate(_variant(89, B, T, H, W, D, "f32")), tau_s=0.5, tau_t=0.5, cell_dots=cell_dots, lib=lib)
    grid = (ctypes.c_uint * 3)()
    assert lib.hip_emul_last_grid(b"k_pyramid", grid)
    assert grid[0] * grid[1] * grid[2] == B * T * 4


def test_emulated_pass_issues_no_memset(emul):
    """A memset recorded into a graph has given wrong results on replays after the first: whatever a caller may capture
    clears memory in kernels, the work queues of the temporal pass on a new shape (its first call) among it."""
    run_cpu, _ = emul
    lib = run_cpu.load()
    before = lib.hip_emul_memsets()
    run_cpu.run_cpu(wl.generate(_variant(86, 1, 2, 3, 3, 8, "f32")), tau_s=0.5, tau_t=0.5, lib=lib)
    assert lib.hip_emul_memsets() == before


@pytest.mark.parametrize("H,W,dtype,cell_dots,levels", [
    (32, 32, "f32", 1, [5, 0, 3, 1, 2, 0, 1]),       # every kind of item, as many of each as there can be
    (13, 11, "bf16", 0, [2, 1, 0, 2, 4, 3, 1, 1]),   # tiles beyond the edge; equal levels count as well
    (9, 18, "f16", 1, [1, 5, 4, 3, 3, 0, 0, 2]),
])
def test_emulated_temporal_pass_with_and_without_a_plan(emul, large, H, W, dtype, cell_dots, levels):
    """The kernel that finds its work by itself against the one that is given a plan: all tables and outputs the same bit for
    bit, on partitions of uniform levels and on one that mixes them."""
    run_cpu, _ = emul
    T = len(levels)
    feats = wl.generate(_variant(106, 1, T, H, W, 8, dtype))
    for nm, nl in (_uniform_partition(T, H, W, levels), (None, None)):
        kw = dict(tau_s=0.7, tau_t=0.3, cell_dots=cell_dots)
        if nm is not None:
            kw["node_map_override"] = (nm, nl)
        a, b = (run_cpu.run_cpu(feats, lib=lib, **kw) for lib in (large, run_cpu.load()))
        for name, x in vars(a).items():
            if isinstance(x, np.ndarray):
                np.testing.assert_array_equal(x, getattr(b, name), err_msg=name)


@pytest.mark.parametrize("T,H,W", [
    (3, 16, 16),    # temporal pairs 512: the elements after the first 256 are a batch that is not full
    (10, 16, 16),   # 2304: those that were requested with the length, and one whole batch
])
def test_emulated_search_among_a_long_list(emul, T, H, W):
    """All similarities in one bin and listed: the thresholds are those of the search through all keys."""
    from tests.cpu_emul import build_cpu
    run_cpu, _ = emul
    rng = np.random.default_rng(T)
    feats = np.repeat(rng.standard_normal((1, 1, H, W, 8)), T, axis=1) + 0.0
    feats = (100 * rng.standard_normal(8) + feats + 1e-3 * rng.standard_normal(feats.shape)).astype(np.float32)
    a, b = (run_cpu.run_cpu(feats, lib=lib, keep=0.4) for lib in (run_cpu.load(build_cpu.build_listed()), run_cpu.load()))
    for name in ("tau_s", "tau_t", "node_map", "cluster_ids"):
        np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)


@pytest.mark.parametrize("B,T,H,W,D,least,most", [
    (1, 10, 8, 8, 8, 9, 10),           # about as many as there can be large clusters
    (1, 1, 8, 8, 8, 1, 1),
    (6, 25, 15, 20, 1280, 64, 192),    # of the few hundred there could be, few are there as a rule
    (32, 100, 6, 6, 256, 200, 256),    # a still scene: 1152 of them, one chunk
    (32, 27, 27, 27, 8, 250, 256),
    (1, 64, 14, 16, 8, 64, 221),
])
def test_emulated_combination_of_large_clusters_has_workgroups_for_them(emul, B, T, H, W, D, least, most):
    """Launched, not carried out: the workgroups of a chunk that walk the list of large clusters."""
    run_cpu, _ = emul
    lib, ptr, h = run_cpu.load(), run_cpu._p, ctypes.c_void_p()
    N = B * T * H * W
    x, merged = run_cpu._aligned(N * D * 2, 16), run_cpu._aligned(N * D * 2, 16)
    cluster, counts = np.zeros(N, np.int32), np.zeros(N, np.int32)
    offsets, grid = np.zeros(B + 1, np.int64), (ctypes.c_uint * 3)()
    assert lib.sttm_create(ctypes.byref(h), 0, None) == 0
    lib.hip_emul_last_grid(None, None)
    lib.hip_emul_record(1)
    try:
        assert lib.sttm_reduce_noalloc(h, ptr(x), 2, B, T, H, W, D, ptr(cluster), 2, ctypes.c_int64(N), ptr(merged), ptr(counts),
                                       None, ptr(offsets)) == 0, lib.sttm_last_error(h)
    finally:
        lib.hip_emul_record(0)
    assert lib.hip_emul_last_grid(b"k_reduce_big", grid) and least <= grid[0] <= most and grid[1] == (D + 511) // 512
    assert grid[0] % 2 == 1                                 # a cluster's chunks go to different dies
    lib.sttm_destroy(h)


@pytest.mark.parametrize("B,T,spatial,temporal", [
    (4, 64, False, False),
    (16, 64, False, True),     # 87,040 and 173,056 elements of all videos
    (16, 121, True, True),     # 10,285 and 20,449 a video
    (128, 16, False, True),    # 1360 a video: too few to be listed; 2704
    (1, 122, False, True),     # 20,618 of one video
])
def test_emulated_searches_of_a_batch_are_listed_where_all_its_elements_are_many(emul, B, T, spatial, temporal):
    """Launched, not carried out: whether a search has the elements of the picked bin listed depends on the elements of a
    video and, where every workgroup of the kernel that uses the threshold searches, on those of all videos."""
    run_cpu, _ = emul
    lib, ptr, h, H, D = run_cpu.load(), run_cpu._p, ctypes.c_void_p(), 13, 8
    N, need = B * T * H * H, lib.sttm_workspace_bytes(B, T, H, H, D, 0, 1)
    ws, x = run_cpu._aligned(need), run_cpu._aligned(N * D * 4, 16)
    nm, nl, grid = np.zeros(N, np.int32), np.zeros(N, np.uint8), (ctypes.c_uint * 3)()
    keep = (ctypes.c_double * B)(*[0.5] * B)

    def chk(rc):
        assert rc == 0, lib.sttm_last_error(h)

    def listed(stage, back=None):
        lib.hip_emul_last_grid(None, None)
        chk(lib.sttm_budget_threshold(h, stage, keep, back))
        return bool(lib.hip_emul_last_grid(b"k_select_list", grid))

    chk(lib.sttm_create(ctypes.byref(h), 0, None))
    chk(lib.sttm_set_workspace(h, ptr(ws), ctypes.c_size_t(need)))
    lib.hip_emul_record(1)
    try:
        chk(lib.sttm_spatial_stats(h, ptr(x), 0, B, T, H, H, D, 1))
        assert listed(0) == spatial
        chk(lib.sttm_spatial_quadtree(h, ptr(x), 0, B, T, H, H, D, 1, None, ptr(nm), ptr(nl)))
        chk(lib.sttm_temporal_stats(h, ptr(x), ptr(nm), ptr(nl)))
        assert listed(1) == temporal
        # one workgroup a video makes a search whose threshold is handed back
        assert listed(1, (ctypes.c_float * B)()) == (T * H * H > 20480)
    finally:
        lib.hip_emul_record(0)
    lib.sttm_destroy(h)


@pytest.mark.parametrize("noise", [0.0, 0.003])
def test_emulated_search_through_all_keys_of_a_bin_that_is_not_kept(emul, noise):
    """More elements in the picked bin than a search keeps, which are then read again from among all keys of their video: the
    thresholds of the search that keeps them."""
    from tests.cpu_emul import build_cpu
    run_cpu, _ = emul
    rng = np.random.default_rng(12)
    feats = (rng.standard_normal(16) + noise * rng.standard_normal((2, 3, 9, 7, 16)).round(1)).astype(np.float32)
    feats[:, 2] = feats[:, 1]                              # a frame that repeats: its pairs are all alike
    crowded = run_cpu.load(build_cpu.build_crowded())
    a, b, c = (run_cpu.run_cpu(feats, lib=lib, keep=0.4, defer_tau=later)
               for lib, later in ((crowded, False), (run_cpu.load(), False), (crowded, True)))
    for name in ("tau_s", "tau_t", "node_map", "cluster_ids"):
        np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)
    assert (c.node_map == a.node_map).all() and (c.cluster_ids == a.cluster_ids).all()


def test_emulated_search_through_all_keys_of_a_bin_that_is_not_kept_runs_clean_under_sanitizers():
    import subprocess
    from tests.cpu_emul import build_cpu
    r = subprocess.run([build_cpu.build_sanitized(), "still"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert r.stdout.count("case ") == 1 and "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr
