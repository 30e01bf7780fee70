"""The kernels for launches with both ends in HBM and for the host arena, at the sizes where one form hands over to the
next: chunks of whole KiB, chunks of whole 128-byte lines, ragged chunks, blocks of less than a wavefront, slots of
whole and of ragged jobs, with and without scales, layer-major and padded pools, descriptor lists inside and outside the
kernel arguments.  Gather, scatter (in both job orders) and move against the oracle, byte for byte."""
import numpy as np
import pytest

from adapters import GpuAdapter
from hostpool import HostPool
from oracle import kv_oracle as ko
from paper_2510_02758_amd import kvswap as kv
from paper_2510_02758_amd import workloads as W

pytestmark = pytest.mark.gpu

GEOMS = {
    "1KiB": W.Geometry(3, 1, 64, 8, "bf16", 96),                       # one full wavefront per chunk
    "1KiB_many": W.Geometry(1, 1, 64, 8, "bf16", 1800),                 # lists of 600 of 1800: sorted by digits for a scatter plane by plane
    "9KiB": W.Geometry(2, 4, 72, 16, "f16", 80),
    "1152B": W.Geometry(3, 1, 72, 8, "bf16", 96),                      # whole lines, no whole KiB; 432 vectors: lane per vector
    "2560B": W.Geometry(2, 2, 80, 8, "bf16", 96),                      # 640 vectors per block: the last job is full
    "128B": W.Geometry(5, 1, 16, 4, "bf16", 300),                      # 80 vectors per block
    "1040B": W.Geometry(5, 1, 65, 8, "bf16", 300),                     # ragged: no whole line
    "20528B": W.Geometry(3, 1, 5132, 2, "bf16", 40),                   # ragged and longer than 4 KiB: both orders of the scatter
    "16B": W.Geometry(1, 1, 8, 1, "bf16", 2000),                       # blocks of 32 bytes
    "fp8_1KiB": W.Geometry(2, 2, 64, 8, "fp8_e4m3", 96, scales=True),
    "fp8_4KiB_wide": W.Geometry(5, 32, 16, 8, "fp8_e4m3", 64, scales=True),     # 320 scale words: a full side job and a short one
    "fp8_640B": W.Geometry(6, 10, 16, 4, "fp8_e4m3", 96, scales=True),          # 480 vectors, a head count that is no power of two
    "fp8_256B": W.Geometry(2, 2, 16, 8, "fp8_e4m3", 200, scales=True),          # a block is exactly one wavefront
    "fp8_48B": W.Geometry(2, 2, 8, 3, "fp8_e4m3", 300, scales=True),
}


@pytest.mark.parametrize("layout", ["layer", "padded"])
@pytest.mark.parametrize("name", list(GEOMS))
def test_gather_scatter_move(gpu, name, layout):
    g = GEOMS[name]
    rng = np.random.default_rng(sum(map(ord, name)))
    for n, order in ((1, 0), (8, 0), (9, 0), (g.N // 3, 0), (g.N // 3, 2)):
        perm = rng.permutation(g.N).astype(np.int32)
        src, dst, mid = perm[:n], perm[n:2 * n], perm[2 * n:3 * n]
        tune = ((kv.KV_TUNE_SCATTER_ORDER, order),) if order else ()
        a, b = (HostPool(g, 0xB0B + n, layout, slots=n + 1) for _ in range(2))
        ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_STAGING_DEVICE, tune=tune)
        for lib in (ora, gpu_lib):
            assert lib.swap_out([7], [0, n], src, [n * g.B]) == ko.OK
            assert lib.swap_in([7], [0, n], dst) == ko.OK
            assert lib.move_blocks(dst, mid) == ko.OK
        assert np.array_equal(a.staging, b.staging), (name, n, "gather")
        assert np.array_equal(a.pool, b.pool), (name, n, "scatter or move")
        if g.scales:
            assert np.array_equal(a.scale, b.scale), (name, n, "scales")
        gpu_lib.close()


@pytest.mark.parametrize("geom", [(8, 1, 64, 8, "bf16"), (12, 1, 72, 8, "bf16"), (128, 2, 8, 3, "fp8_e4m3")], ids=["1KiB", "1152B", "fp8_48B"])
def test_moves_that_go_plane_by_plane(gpu, geom):
    """Moves over lists that are worth ordering, by digits: chunks of whole KiB, whole lines, ragged ones with scales."""
    g = W.Geometry(*geom, 4500, scales=geom[4] == "fp8_e4m3")
    n = 1400
    assert 3 * n <= g.N < 6 * n
    perm = np.random.default_rng(22).permutation(g.N).astype(np.int32)
    a, b = (HostPool(g, 0xB13, "layer", slots=1) for _ in range(2))
    ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_STAGING_DEVICE)
    assert ora.move_blocks(perm[:n], perm[n:2 * n]) == ko.OK and gpu_lib.move_blocks(perm[:n], perm[n:2 * n]) == kv.KV_OK
    assert ora.move_blocks(perm[n:2 * n], perm[2 * n:3 * n]) == ko.OK
    gpu_lib._push()
    assert gpu_lib.kp.move_blocks_noalloc(perm[n:2 * n], perm[2 * n:3 * n]) == kv.KV_OK
    gpu_lib._pull()
    assert np.array_equal(a.pool, b.pool) and (not g.scales or np.array_equal(a.scale, b.scale))
    gpu_lib.close()


@pytest.mark.parametrize("name", ["9KiB", "1040B", "fp8_1KiB", "fp8_48B"])
def test_bounce_buffer(gpu, name):
    """The copy-engine path's gather and scatter run the same kernels between the pool and the bounce buffer."""
    g = GEOMS[name]
    n = 21
    perm = np.random.default_rng(3).permutation(g.N).astype(np.int32)
    a, b = (HostPool(g, 0xB0C, "padded", slots=n) for _ in range(2))
    ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_PATH_DMA, bounce_slots=10)
    for lib in (ora, gpu_lib):
        assert lib.swap_out([1, 2], [0, 4, n], perm[:n], [4 * g.B, (n - 4) * g.B]) == ko.OK
        assert lib.swap_in([2, 1], [0, n - 4, n], perm[n:2 * n]) == ko.OK
    assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool)
    assert not g.scales or np.array_equal(a.scale, b.scale)
    gpu_lib.close()


@pytest.mark.parametrize("layout", ["layer", "padded"])
@pytest.mark.parametrize("name", list(GEOMS))
def test_host_arena(gpu, name, layout):
    """One block, a ragged list, and both directions in flight at once (the wider launches)."""
    g = GEOMS[name]
    rng = np.random.default_rng(1 + sum(map(ord, name)))
    for n in (1, g.N // 3):
        perm = rng.permutation(g.N).astype(np.int32)
        src, dst, more = perm[:n], perm[n:2 * n], perm[2 * n:2 * n + 1]
        a, b = (HostPool(g, 0xB0D + n, layout, slots=n + 2) for _ in range(2))
        ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_PATH_ZEROCOPY)
        assert ora.swap_out([7], [0, n], src, [n * g.B]) == ko.OK
        assert ora.swap_in([7], [0, n], dst) == ko.OK
        assert ora.swap_out([8], [0, 1], more, [g.B]) == ko.OK
        gpu_lib._push()
        kp = gpu_lib.kp
        assert kp.swap_out([7], [0, n], src, [n * g.B]) == kv.KV_OK
        assert kp.swap_in([7], [0, n], dst) == kv.KV_OK
        assert kp.swap_out([8], [0, 1], more, [g.B]) == kv.KV_OK
        gpu_lib._pull()
        assert np.array_equal(a.staging, b.staging), (name, n, "gather")
        assert np.array_equal(a.pool, b.pool), (name, n, "scatter")
        if g.scales:
            assert np.array_equal(a.scale, b.scale), (name, n, "scales")
        gpu_lib.close()


def test_lists_longer_than_the_kernel_arguments(gpu):
    """448 descriptors travel inside the arguments, 449 do not."""
    g = W.Geometry(1, 1, 16, 4, "bf16", 1400)
    perm = np.random.default_rng(9).permutation(g.N).astype(np.int32)
    for n in (448, 449):
        for flags in (kv.KV_STAGING_DEVICE, kv.KV_PATH_ZEROCOPY, kv.KV_PATH_DMA):
            a, b = (HostPool(g, 0xB0E, "layer", slots=n) for _ in range(2))
            ora, gpu_lib = a.oracle(), GpuAdapter(b, flags, bounce_slots=n)
            for lib in (ora, gpu_lib):
                assert lib.swap_out([1], [0, n], perm[:n], [n * g.B]) == ko.OK
                assert lib.swap_in([1], [0, n], perm[n:2 * n]) == ko.OK
            assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool), (n, flags)
            assert ora.move_blocks(perm[n:2 * n], perm[2 * n:3 * n]) == ko.OK
            gpu_lib._push()
            assert gpu_lib.kp.move_blocks_noalloc(perm[n:2 * n], perm[2 * n:3 * n]) == kv.KV_OK
            gpu_lib._pull()
            assert np.array_equal(a.pool, b.pool), (n, flags, "move")
            gpu_lib.close()


@pytest.mark.parametrize("n", [60, 61])
def test_lists_at_the_end_of_the_short_argument_block(gpu, n):
    """60 descriptors leave the arguments below 1 KiB, 61 take the long block, or an upload where they are a small move."""
    g = W.Geometry(1, 1, 64, 8, "bf16", 200)
    perm = np.random.default_rng(n).permutation(g.N).astype(np.int32)
    for flags in (kv.KV_STAGING_DEVICE, kv.KV_PATH_ZEROCOPY, kv.KV_PATH_DMA):
        a, b = (HostPool(g, 0xB0F, "layer", slots=n) for _ in range(2))
        ora, gpu_lib = a.oracle(), GpuAdapter(b, flags, bounce_slots=n)
        for lib in (ora, gpu_lib):
            assert lib.swap_out([1], [0, n], perm[:n], [n * g.B]) == ko.OK
            assert lib.swap_in([1], [0, n], perm[n:2 * n]) == ko.OK
            assert lib.move_blocks(perm[n:2 * n], perm[2 * n:3 * n]) == ko.OK
        assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool), flags
        assert ora.move_blocks(perm[2 * n:3 * n], perm[:n]) == ko.OK
        gpu_lib._push()
        assert gpu_lib.kp.move_blocks_noalloc(perm[2 * n:3 * n], perm[:n]) == kv.KV_OK
        gpu_lib._pull()
        assert np.array_equal(a.pool, b.pool), (flags, "move without allocation")
        gpu_lib.close()


@pytest.mark.parametrize("name", ["1KiB", "9KiB", "1040B", "fp8_4KiB_wide", "fp8_48B"])
def test_workgroup_cap(gpu, name):
    """Handles under KV_TUNE_MAX_WGS_DEVICE: lists inside the arguments and uploaded, both orders of the scatter."""
    g = GEOMS[name]
    rng = np.random.default_rng(5)
    for n, order in ((8, 0), (9, 0), (g.N // 3, 2)):
        perm = rng.permutation(g.N).astype(np.int32)
        src, dst, mid = perm[:n], perm[n:2 * n], perm[2 * n:3 * n]
        tune = ((kv.KV_TUNE_MAX_WGS_DEVICE, 3),) + (((kv.KV_TUNE_SCATTER_ORDER, order),) if order else ())
        a, b = (HostPool(g, 0xB10 + n, "padded", slots=n + 1) for _ in range(2))
        ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_STAGING_DEVICE, tune=tune)
        for lib in (ora, gpu_lib):
            assert lib.swap_out([7], [0, n], src, [n * g.B]) == ko.OK
            assert lib.swap_in([7], [0, n], dst) == ko.OK
            assert lib.move_blocks(dst, mid) == ko.OK
        assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool), (name, n, order)
        assert not g.scales or np.array_equal(a.scale, b.scale), (name, n, order)
        gpu_lib.close()


@pytest.mark.parametrize("arena", ["host", "device"])
@pytest.mark.parametrize("name,n", [("16B", 1), ("16B", 512), ("16B", 600), ("9KiB", 1), ("9KiB", 6), ("9KiB", 7), ("fp8_4KiB_wide", 2), ("fp8_48B", 90),
                                    ("1KiB", 60), ("1KiB_many", 61), ("1KiB_many", 449)])
def test_streams_hand_over_short_transfers(gpu, name, n, arena):
    """Short transfers tell the other stream by a number that they have finished: launches of one workgroup, of fewer jobs
    than workgroups, of more, of ragged slots (the host arena's two kinds of job), and lists of every kind of upload.  A chain of
    preemptions, resumptions and exchanges in which every call reads or overwrites what the one before it has moved, with
    nothing waited for in between."""
    g = GEOMS[name]
    rng = np.random.default_rng(n)
    a, b = (HostPool(g, 0xB11 + n, "layer", slots=2 * n) for _ in range(2))
    ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_STAGING_DEVICE if arena == "device" else kv.KV_PATH_ZEROCOPY)
    gpu_lib._push()
    kp, off = gpu_lib.kp, [0, n]
    tables = [rng.permutation(g.N)[:n].astype(np.int32) for _ in range(9)]
    for k in range(8):
        assert ora.swap_out([1], off, tables[k], [n * g.B]) == ko.OK
        assert kp.swap_out([1], off, tables[k], [n * g.B]) == kv.KV_OK
        assert ora.swap_in([1], off, tables[k + 1]) == ko.OK
        assert kp.swap_in([1], off, tables[k + 1]) == kv.KV_OK
    assert ora.swap_out([1], off, tables[8], [n * g.B]) == ko.OK
    assert kp.swap_out([1], off, tables[8], [n * g.B]) == kv.KV_OK
    for k in range(6):  # the set that is out takes the blocks of the one that goes
        out, back = 2 - k % 2, 1 + k % 2
        assert ora.swap_out([out], off, tables[8 - k], [n * g.B]) == ko.OK and ora.swap_in([back], off, tables[8 - k]) == ko.OK
        assert kp.evict_and_load([out], off, tables[8 - k], [n * g.B], [back], off, tables[8 - k]) == kv.KV_OK
    gpu_lib._pull()
    assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool)
    assert not g.scales or np.array_equal(a.scale, b.scale)
    gpu_lib.close()


@pytest.mark.parametrize("layers,n,order", [(12, 110, -1), (40, 70, 1)])
def test_pool_whose_planes_collide(gpu, layers, n, order):
    """Pools of 24 and 80 planes 4 MiB + 32 KiB apart: 70 of 258 blocks of 1.25 MiB go plane by plane out and in again, 110 of
    384 KiB, which are many in flight beside each other, do not."""
    g = W.Geometry(layers, 8, 128, 8, "bf16", 258)
    perm = np.random.default_rng(21).permutation(g.N).astype(np.int32)
    a, b = (HostPool(g, 0xB12, "layer", slots=n) for _ in range(2))
    ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_STAGING_DEVICE)
    for lib in (ora, gpu_lib):
        assert lib.swap_out([1, 2], [0, 40, n], perm[:n], [40 * g.B, (n - 40) * g.B]) == ko.OK
        assert lib.swap_in([2, 1], [0, n - 40, n], perm[n:2 * n]) == ko.OK
    assert gpu_lib.kp.stats()["scatter_order"] == order
    assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool)
    gpu_lib.close()


@pytest.mark.parametrize("arena", ["device", "host"])
@pytest.mark.parametrize("geom,n", [((4, 4, 64, 16, "f16"), 40), ((4, 4, 64, 16, "f16"), 300), ((5, 1, 65, 8, "bf16"), 150), ((5, 1, 16, 4, "bf16"), 150),
                                    ((2, 2, 8, 3, "fp8_e4m3"), 150)], ids=["8KiB", "8KiB_beyond_16MiB", "1040B", "128B", "fp8_48B"])
def test_calls_in_a_row_without_end_events(gpu, geom, n, arena):
    """Moves, allocation-free moves and transfers that depend on each other across the two streams, nothing waited for in
    between: short launches say by a number that they have finished."""
    g = W.Geometry(*geom, 3 * n + 5, scales=geom[4] == "fp8_e4m3")
    perm = np.random.default_rng(n).permutation(g.N).astype(np.int32)
    x, y, z, m = perm[:n], perm[n:2 * n], perm[2 * n:3 * n], n // 2
    a, b = (HostPool(g, 0xB20 + n, "layer", slots=n) for _ in range(2))
    ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_STAGING_DEVICE if arena == "device" else kv.KV_PATH_ZEROCOPY)
    gpu_lib._push()
    kp = gpu_lib.kp
    for turn in range(6):
        for lib, free in ((ora, ora.move_blocks), (kp, kp.move_blocks_noalloc)):
            assert lib.move_blocks(x, y) == ko.OK
            assert free(y, z) == ko.OK
            assert lib.swap_out([turn], [0, m], z[:m], [m * g.B]) == ko.OK
            assert lib.move_blocks(x[m:], z[:n - m]) == ko.OK                    # over what the swap-out reads
            assert lib.swap_in([turn], [0, m], x[n - m:]) == ko.OK               # over what the move reads
            assert free(x[n - m:], y[:m]) == ko.OK
            assert lib.swap_out([100], [0, m], y[:m], [m * g.B]) == ko.OK
            assert lib.swap_in([100], [0, m], x[:m]) == ko.OK
        if turn == 3:
            assert kp.req_wait(100) == kv.KV_OK and kp.req_poll(100) == 1
    gpu_lib._pull()
    assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool)
    assert not g.scales or np.array_equal(a.scale, b.scale)
    gpu_lib.close()


@pytest.mark.parametrize("arena", ["device", "host"])
def test_a_wait_ends_with_its_call(gpu, arena):
    """kv_req_wait and kv_last_stats of a call that finishes by number, with 60 ms of other work behind it on the same stream."""
    import torch
    g = W.Geometry(4, 4, 64, 16, "f16", 60)
    a, b = HostPool(g, 0xB40, "layer", slots=40), HostPool(g, 0xB40, "layer", slots=40)
    pool = torch.from_numpy(b.pool).to(gpu)
    slots = torch.zeros(40 * g.S, dtype=torch.uint8, device=gpu) if arena == "device" else torch.zeros(40 * g.S, dtype=torch.uint8).pin_memory()
    evict, load = torch.cuda.Stream(), torch.cuda.Stream()
    big = torch.zeros(2 << 30, dtype=torch.uint8, device=gpu)
    torch.cuda.synchronize()
    kp = kv.KVPool(g, pool, slots, evict_stream=evict, load_stream=load, flags=kv.KV_STAGING_DEVICE if arena == "device" else kv.KV_PATH_ZEROCOPY)
    ids = np.arange(60, dtype=np.int32)
    x, y, z = ids[:20], ids[20:40], ids[40:]
    off, tok = [0, 20], [20 * g.B]
    behind = torch.cuda.Event()
    for turn in range(4):
        assert kp.move_blocks(x, y) == kv.KV_OK and kp.swap_out([turn], off, y, tok) == kv.KV_OK
        with torch.cuda.stream(evict):
            for _ in range(80):
                big[:1 << 30].copy_(big[1 << 30:])
            behind.record()
        if turn % 2:
            assert kp.req_wait(turn) == kv.KV_OK
        else:
            st = kp.stats()
            assert st["op"] == 1 and 0 < st["ms_total"] < 20
        assert not behind.query(), "the wait has waited for what is behind its call"
        assert kp.req_poll(turn) == 1 and kp.io_stats()["inflight_calls"] == [0, 0]
        assert kp.swap_in([turn], off, z) == kv.KV_OK and kp.req_wait(turn) == kv.KV_OK
        assert kp.sync() == kv.KV_OK
        want = a.pool.reshape(2 * g.L, g.N, -1)
        want[:, y] = want[:, x]
        want[:, z] = want[:, x]
        assert np.array_equal(pool.cpu().numpy(), a.pool.reshape(-1).view(np.uint8))
        pool.view(2 * g.L, g.N, -1)[:, :20] += 1
        a.pool.reshape(2 * g.L, g.N, -1).view(np.uint8)[:, :20] += 1
        torch.cuda.synchronize()
    kp.close()


@pytest.mark.parametrize("geom,n", [((4, 4, 64, 16, "f16"), 27), ((1, 1, 72, 1, "bf16"), 57), ((2, 4, 64, 16, "fp8_e4m3"), 40), ((32, 8, 128, 16, "bf16"), 12)],
                         ids=["8KiB", "144B", "fp8", "24MiB"])
def test_the_host_reads_what_a_wait_says_is_there(gpu, geom, n):
    """The host arena is complete when a wait or a poll by number says so, over each build of the link kernel's gather."""
    import torch
    g = W.Geometry(*geom, 2 * n, scales=geom[4] == "fp8_e4m3")
    pool = torch.zeros(g.pool_bytes, dtype=torch.uint8, device=gpu)
    scale = torch.zeros(g.scale_bytes, dtype=torch.uint8, device=gpu) if g.scales else None
    slots = torch.zeros(n * g.S, dtype=torch.uint8).pin_memory()
    kp = kv.KVPool(g, pool, slots, scale=scale)
    ids, off, tok = np.arange(2 * n, dtype=np.int32), [0, n], [n * g.B]
    seen = slots.numpy()
    for turn in range(1, 60 if n * g.S > 1 << 20 else 250):
        for t in (pool, scale):
            if t is not None:
                t.fill_(turn)
        torch.cuda.synchronize()
        assert kp.move_blocks(ids[:1], ids[-1:]) == kv.KV_OK      # (the swap-out behind a call in flight has no end event)
        assert kp.swap_out([turn], off, ids[:n], tok) == kv.KV_OK
        if turn % 2:
            assert kp.req_wait(turn) == kv.KV_OK
        else:
            while not kp.req_poll(turn):
                pass
        assert (seen == turn).all(), turn
        assert kp.swap_in([turn], off, ids[n:]) == kv.KV_OK and kp.sync() == kv.KV_OK
    kp.close()


@pytest.mark.parametrize("geom,n", [((24, 4, 72, 16, "f16"), 701), ((20, 1, 72, 8, "bf16"), 6001), ((32, 4, 128, 8, "fp8_e4m3"), 1101)],
                         ids=["9KiB", "1152B", "fp8_4KiB"])
def test_lists_beyond_the_memory_side_cache(gpu, geom, n):
    """More than 256 MiB: the gather keeps the end of its list in the cache, the scatter begins there.  Against torch's own indexing."""
    import torch
    g = W.Geometry(*geom, 2 * n + 1, scales=geom[4] == "fp8_e4m3")
    assert n * g.S > 256 << 20
    gen = torch.Generator(device="cuda").manual_seed(n)
    pool = torch.randint(-2**62, 2**62, (g.pool_bytes // 8,), dtype=torch.int64, device="cuda", generator=gen).view(torch.uint8)
    scale = torch.randint(-2**62, 2**62, (g.scale_bytes // 8,), dtype=torch.int64, device="cuda", generator=gen).view(torch.uint8) if g.scales else None
    arena = torch.zeros(n * g.S, dtype=torch.uint8, device="cuda")
    perm = np.random.default_rng(n).permutation(g.N).astype(np.int32)
    src, dst = (torch.as_tensor(perm[k * n:(k + 1) * n].astype(np.int64), device="cuda") for k in (0, 1))
    planes = [t.view(2 * g.L, g.N, -1) for t in (pool, scale) if t is not None]
    before = [p.clone() for p in planes]
    torch.cuda.synchronize()
    kp = kv.KVPool(g, pool, arena, scale=scale, flags=kv.KV_STAGING_DEVICE)
    for turn in range(2):  # (the second scatter, where lists of 1024 blocks are timed both ways, goes plane by plane)
        assert kp.swap_out([7], [0, n], perm[:n], [n * g.B]) == kv.KV_OK
        assert kp.swap_in([7], [0, n], perm[n:2 * n]) == kv.KV_OK
        assert kp.sync() == kv.KV_OK
        at = 0
        for p, b in zip(planes, before):
            part = arena.view(n, g.S)[:, at:at + 2 * g.L * p.shape[2]].reshape(n, 2 * g.L, -1)
            at += 2 * g.L * p.shape[2]
            assert torch.equal(part, b[:, src].transpose(0, 1)), "gather"
            b[:, dst] = b[:, src]
            assert torch.equal(p, b), "scatter"
        pool.view(torch.int64).bitwise_xor_(0x5A5A)
        planes[0].copy_(pool.view(2 * g.L, g.N, -1))
        before[0].copy_(planes[0])
        torch.cuda.synchronize()
    kp.close()


@pytest.mark.parametrize("geom,n", [((1, 4, 72, 16, "f16"), 227), ((1, 4, 72, 16, "f16"), 229), ((3, 1, 72, 8, "bf16"), 607), ((3, 1, 72, 8, "bf16"), 610),
                                    ((1, 1, 64, 8, "bf16"), 2049), ((2, 2, 64, 8, "fp8_e4m3"), 1), ((2, 2, 64, 8, "fp8_e4m3"), 35),
                                    ((6, 10, 16, 4, "fp8_e4m3"), 37)],
                         ids=["9KiB_below_4MiB", "9KiB", "1152B_odd", "1152B", "1KiB", "fp8_1KiB_one", "fp8_1KiB", "fp8_640B"])
def test_workgroups_of_four_wavefronts(gpu, geom, n):
    """Counted launches from 4 MiB on, and all with scales, whose last workgroup has jobs for each number of its wavefronts and one or
    two for each of them: gather, scatter and move, block by block and plane by plane."""
    g = W.Geometry(*geom, 3 * n + 2, scales=geom[4] == "fp8_e4m3")
    perm = np.random.default_rng(n).permutation(g.N).astype(np.int32)
    for order in (0, 2):
        tune = ((kv.KV_TUNE_SCATTER_ORDER, order),) if order else ()
        a, b = (HostPool(g, 0xB30 + n, "layer", slots=n) for _ in range(2))
        ora, gpu_lib = a.oracle(), GpuAdapter(b, kv.KV_STAGING_DEVICE, tune=tune)
        for lib in (ora, gpu_lib):
            assert lib.swap_out([1], [0, n], perm[:n], [n * g.B]) == ko.OK
            assert lib.swap_in([1], [0, n], perm[n:2 * n]) == ko.OK
            assert lib.move_blocks(perm[n:2 * n], perm[2 * n:3 * n]) == ko.OK
        assert np.array_equal(a.staging, b.staging) and np.array_equal(a.pool, b.pool), order
        assert not g.scales or np.array_equal(a.scale, b.scale), order
        gpu_lib.close()


@pytest.mark.parametrize("geom,n", [((24, 4, 72, 16, "f16"), 191), ((20, 1, 72, 8, "bf16"), 1901), ((20, 3, 112, 1, "bf16"), 3201)], ids=["9KiB", "1152B", "672B"])
def test_longer_calls_in_a_row(gpu, geom, n):
    """The same with moves of 80 MiB and transfers of 40: beyond the sizes at which moves take two jobs a wavefront, and at which only
    calls of one launch store a number."""
    g = W.Geometry(*geom, 1)
    assert n * g.S > 64 << 20 and 32 << 20 < n // 2 * g.S < 48 << 20
    test_calls_in_a_row_without_end_events(gpu, geom, n, "device")
