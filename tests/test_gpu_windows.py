"""The window copies (store, streaming, shared and four-job retrieves) against
plain torch indexing, over segment sizes at the edges of the window copy's
range and over payloads on both sides of every size at which the launch shape
changes.  Copies move bytes, so every comparison is exact."""
import numpy as np
import pytest
import torch

import paper_2609_35065_amd as kv

pytestmark = pytest.mark.gpu

MIB = 1 << 20
# (block, heads, dim, elem): 496 B and 1 MiB segments take the generic copy; 512 B is the smallest window segment;
# 528 and 1,040 B leave rows that cross segments at every offset; the rest are 1.25, 4, 20, 32, 64 and 512 KiB
SHAPES = {"496": (1, 1, 248, 2), "512": (16, 1, 32, 1), "528": (33, 1, 16, 1), "1040": (13, 1, 40, 2), "1280": (16, 1, 80, 1),
          "4k": (16, 1, 128, 2), "20k": (16, 8, 80, 2), "32k": (16, 8, 128, 2), "64k": (16, 8, 128, 4),
          "512k": (128, 8, 128, 4), "1m": (256, 8, 128, 4)}


def _setup(shape, payload, slots_per_job, layout, pad, seed, layers=3, nseg=None):
    block, heads, dim, elem = shape
    seg = block * heads * dim * elem
    nseg = nseg or (16 if seg < 131072 else 2)
    slot = 2 * layers * nseg * seg
    n = max(1, payload // slot)
    slots = max(1, int(n * slots_per_job))
    nb = n * nseg + 3
    row = seg + pad
    strides = (nb * row, row) if layout == "kv_first" else (row, 2 * row)
    lo = kv.make_layout(layers, heads, dim, elem, block, block * nseg, nb, slots, *strides)
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def rand(nbytes):   # random words
        return torch.randint(-2**62, 2**62, (nbytes // 8,), dtype=torch.int64, device="cuda", generator=gen)

    pool = [rand(2 * nb * row) for _ in range(layers)]
    staging = rand(slots * slot)
    rng = np.random.default_rng(seed)
    bt = rng.permutation(nb)[:n * nseg].reshape(n, nseg).astype(np.int32)
    bt[0, nseg // 2] = -1          # segments that are skipped
    bt[n - 1, nseg - 1] = nb
    jobs = np.zeros((n, 4), np.int32)
    jobs[:, 0] = np.sort(rng.integers(0, slots, n)) if slots < n else np.arange(n)
    jobs[:, 1] = np.arange(n)
    if n > 4:
        jobs[2, 1] = n             # jobs that are skipped
        jobs[n - 2, 0] = slots
    ok = (jobs[:, 1] < n) & (jobs[:, 0] < slots)
    return lo, pool, staging, bt, jobs, ok, (layers, nseg, seg, nb, strides, slots)


def _expected(pool, staging, bt, jobs, ok, dims, store):
    layers, nseg, seg, nb, strides, slots = dims
    pool = [t.clone() for t in pool]
    staging = staging.clone()
    stg = staging.view(slots, layers, 2, nseg, seg // 8)
    j, i = np.nonzero(ok[:, None] & (bt >= 0) & (bt < nb))   # block tables: row r belongs to job r
    slot = torch.from_numpy(jobs[j, 0].astype(np.int64)).cuda()
    blk = torch.from_numpy(bt[j, i].astype(np.int64)).cuda()
    i = torch.from_numpy(i).cuda()
    for l in range(layers):
        for p in range(2):
            view = pool[l].as_strided((nb, seg // 8), (strides[1] // 8, 1), p * strides[0] // 8)
            if store:
                stg[slot, l, p, i] = view[blk]
            else:
                view[blk] = stg[slot, l, p, i]
    return pool, staging


def _check(shape, payload, op, layout, pad, seed, host=False, **dims):
    share = {"unit": 0.2, "quad": 0.2}.get(op, 1.0)
    lo, pool, staging, bt, jobs, ok, dims = _setup(SHAPES[shape], payload, share, layout, pad, seed, **dims)
    want_pool, want_staging = _expected(pool, staging, bt, jobs, ok, dims, op == "store")
    d_bt, d_jobs = torch.from_numpy(bt).cuda(), torch.from_numpy(jobs).cuda()
    at = staging
    if host:
        staging = torch.empty(staging.numel(), dtype=torch.int64, pin_memory=True).copy_(staging)
        want_staging = want_staging.cpu()
        at = kv.kv_host_device_pointer(staging.data_ptr())
    if op == "store":
        kv.kv_store_gather(lo, at, pool, d_bt, bt.shape[1], bt.shape[0], d_jobs, len(jobs))
    else:
        kind = {"unit": kv.KV_RETRIEVE_UNIT, "stream": kv.KV_RETRIEVE_STREAM, "quad": kv.KV_RETRIEVE_QUAD}[op]
        kv.kv_retrieve_scatter_as(kind, lo, at, pool, d_bt, bt.shape[1], bt.shape[0], d_jobs, len(jobs))
    torch.cuda.synchronize()
    assert torch.equal(staging, want_staging)
    for a, b in zip(pool, want_pool):
        assert torch.equal(a, b)


@pytest.mark.parametrize("op", ["store", "stream", "unit", "quad"])
@pytest.mark.parametrize("layout,pad", [("kv_first", 0), ("block_first", 48)])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_segment_sizes(shape, layout, pad, op):
    for payload in (1, 6 * MIB):
        _check(shape, payload, op, layout, pad, 7)


@pytest.mark.parametrize("op", ["store", "stream", "unit"])
@pytest.mark.parametrize("shape", ["1040", "4k", "20k", "32k"])
@pytest.mark.parametrize("mib", [23, 36, 60, 100, 600, 700, 1030])
def test_launch_shapes(mib, shape, op):
    _check(shape, mib * MIB, op, "kv_first", 16, 11)


@pytest.mark.parametrize("op", ["store", "stream", "unit"])
@pytest.mark.parametrize("shape,layers,nseg", [("512", 1, 1), ("1040", 1, 1), ("1040", 1, 3), ("4k", 1, 1), ("4k", 1, 5),
                                               ("20k", 1, 1), ("32k", 1, 1), ("64k", 1, 1)])
@pytest.mark.parametrize("mib", [3, 30, 1100])
def test_small_slots(mib, shape, layers, nseg, op):
    # slots below one workgroup's windows or one group, and no multiple of them (thousands of jobs)
    _check(shape, mib * MIB, op, "block_first", 0, 13, layers=layers, nseg=nseg)


@pytest.mark.parametrize("op", ["store", "stream", "unit"])
@pytest.mark.parametrize("shape", ["512", "1040", "4k", "20k", "32k", "64k"])
@pytest.mark.parametrize("mib", [1, 20, 60])
def test_host_memory(mib, shape, op):
    # staged chunks in host memory: one job, and payloads on both sides of the sizes at which the shape changes
    _check(shape, mib * MIB, op, "kv_first", 0, 17, host=True)


@pytest.mark.parametrize("shape", ["64k", "512k"])
@pytest.mark.parametrize("mib", [100, 700])
def test_planes_above_a_group(mib, shape):
    # planes of 1 MiB: groups of 256 windows, several jobs to a slot
    _check(shape, mib * MIB, "unit", "block_first", 0, 19)


@pytest.mark.parametrize("op", ["store", "stream"])
@pytest.mark.parametrize("shape", ["512", "528"])
@pytest.mark.parametrize("mib", [60, 1100])
def test_many_segments_a_window(mib, shape, op):
    # windows of 16 KiB over up to 33 segments: every lane of the address table in use
    _check(shape, mib * MIB, op, "kv_first", 0, 23)


@pytest.mark.parametrize("shape", ["4k", "32k"])
@pytest.mark.parametrize("host", [False, True])
def test_shared_retrieve_captured(host, shape):
    # The shared retrieve asks where the staged chunks lie before it launches: from device and from host memory,
    # eager and captured (replayed three times, with eager work and a synchronisation between).
    lo, pool, staging, bt, jobs, ok, dims = _setup(SHAPES[shape], 20 * MIB, 0.3, "kv_first", 0, 5)
    want, _ = _expected(pool, staging, bt, jobs, ok, dims, False)
    if host:
        pinned = torch.empty(staging.numel(), dtype=torch.int64, pin_memory=True)
        pinned.copy_(staging)
        src = kv.kv_host_device_pointer(pinned.data_ptr())
    else:
        src = staging
    d_bt, d_jobs = torch.from_numpy(bt).cuda(), torch.from_numpy(jobs).cuda()
    start = [t.clone() for t in pool]

    def run():
        kv.kv_retrieve_scatter(lo, src, pool, d_bt, bt.shape[1], bt.shape[0], d_jobs, len(jobs))

    def check():
        torch.cuda.synchronize()
        for a, b, c in zip(pool, want, start):
            assert torch.equal(a, b)
            a.copy_(c)

    run()
    check()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    for _ in range(3):
        g.replay()
        check()
