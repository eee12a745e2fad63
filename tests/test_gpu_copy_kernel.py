"""The copy kernel proper on pool->pool jobs. Most jobs that a test can afford go to the wave kernel, so these ask for the copy
kernel by its tile size (or by a chunk that the wave kernel does not take) and say by the statistics that they got it: every
alignment of both sides, the order ticket by ticket with and without an entry per tile in the descriptor table, its
counter pairs, and the tiles of one aligned tensor dealt out without a counter."""
import numpy as np
import pytest

from workloads import make_descs, FT_POOL
from workloads import format as fmt
from test_gpu_decode_log import _alloc, _check_job, _images_equal, _pair

pytestmark = pytest.mark.gpu
KiB, MiB = 1 << 10, 1 << 20


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2411_01830_amd import binding, harness
    assert torch.cuda.is_available()
    return binding, harness


def _piece(orc, eng, rng, n, f, ss, ds, rows=1, pitch=0):
    pitch = pitch if rows > 1 else n
    span = (rows - 1) * pitch + n + 48
    a, b = _alloc(orc, eng, span, rng), _alloc(orc, eng, span)
    return dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a + 16 + ss, dst=b + 16 + ds, row_bytes=n, rows=rows, src_pitch=pitch,
                dst_pitch=n if rows > 1 else pitch)


def test_every_alignment_pair_in_the_pool(gpu):
    """src % 16 x dst % 16 for pieces within a tile and over tiles; canaries around every destination."""
    binding, _ = gpu
    orc, eng, rng = _pair(gpu, 1 * MiB, 160 * MiB, 4 * KiB, 11)
    try:
        binding.set_tuning(eng.pool, 2, 0, 64 * KiB)
        for n in (1, 15, 16, 17, 255, 256, 257, 4095, 70001, 200017):
            print(f"case copy kernel alignments n={n}", flush=True)
            recs = [_piece(orc, eng, rng, n, (sa + da) % 3, sa, da) for sa in range(16) for da in range(16)]
            d = make_descs(recs)
            orc.wait(orc.submit(d, [1, 2, 3], 128 * KiB))
            jg = eng.submit(d, [1, 2, 3], 128 * KiB, fmt.FT_KEEP | fmt.FT_VALIDATE)
            eng.wait(jg)
            assert binding.job_stats(eng.pool, jg).cls[2].tile_bytes == 64 * KiB
            binding.job_release(eng.pool, jg)
            _images_equal(orc, eng)
            for off in list(orc.pool.allocs):
                orc.slab_free(off)
                eng.slab_free(off)
    finally:
        eng.close()


# name, (sizes, rows), pieces, functions, chunk, tile
ORDERS = [
    ("a piece per tile and more", ([60000, 65536, 131072], 1), 60, 4, 2 * MiB, 64 * KiB),
    ("an entry per tile", ([700, 3000, 9000], 1), 600, 5, 256 * KiB, 16 * KiB),
    ("an entry per tile, short rows", ([40, 300], 30), 600, 3, 128 * KiB, 43 * KiB),
    ("an entry per chunk, searched within it", ([5000, 9000], 1), 600, 3, 64 * KiB, 64 * KiB),
    ("chunks of two thirds of a tile", ([100000, 400000], 1), 40, 7, 100000 // 16 * 16, 48 * KiB),
]


@pytest.mark.parametrize("case", ORDERS, ids=[c[0] for c in ORDERS])
def test_decode_follows_the_order_in_the_pool(gpu, case):
    """Every ticket as the kernel decoded it against the order of the oracle cut into tiles."""
    binding, _ = gpu
    name, (sizes, rows), n, funcs, chunk, tile = case
    print(f"case copy kernel order: {name}", flush=True)
    orc, eng, rng = _pair(gpu, 1 * MiB, 128 * MiB, 4 * KiB, 17)
    try:
        binding.set_tuning(eng.pool, 2, 0, tile)
        recs = []
        for i in range(n):
            w = int(rng.choice(sizes))
            recs.append(_piece(orc, eng, rng, w, i % funcs, int(rng.integers(0, 16)) * (i % 3 == 0), 0, rows, w + 24))
        weights = [1 + 3 * f % 5 for f in range(funcs)]
        d = make_descs(recs)
        jo = orc.submit(d, weights, chunk)
        orc.wait(jo)
        for _ in range(2):
            jg = eng.submit(d, weights, chunk, fmt.FT_LOG | fmt.FT_VALIDATE)
            eng.wait(jg)
            st, seen = _check_job(binding, eng, orc, jg, jo, d, funcs, chunk, classes=(2,))
            tiles = -(-chunk // tile)
            assert st.cls[2].tile_bytes == (-(-chunk // tiles) + 15) // 16 * 16 and seen > 50
            binding.job_release(eng.pool, jg)
        _images_equal(orc, eng)
    finally:
        eng.close()


def test_counter_pairs_in_the_pool(gpu):
    """Jobs of a few tensors with more tiles than workgroups, one after the other on a counter pair that the kernel sets back
    itself, some kept meanwhile."""
    import torch
    binding, _ = gpu
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    orc, eng, rng = _pair(gpu, 1 * MiB, 192 * MiB, 1 * MiB, 23)
    try:
        binding.set_tuning(eng.pool, 2, 0, 64 * KiB)
        kept = []
        for case, n in enumerate([18 * MiB, 18 * MiB + 33, 24 * MiB, 17 * MiB + 4096, 20 * MiB + 1, 18 * MiB]):
            print(f"case copy kernel counter pair {case}", flush=True)
            d = make_descs([_piece(orc, eng, rng, n, 0, 0, 0), _piece(orc, eng, rng, n // 2, 1, case % 2, 3 * (case % 3))])
            jo = orc.submit(d, [1, 3], 2 * MiB)
            orc.wait(jo)
            jg = eng.submit(d, [1, 3], 2 * MiB, fmt.FT_KEEP)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg).cls[2]
            assert st.in_launch == 1 and st.workgroups == cus < st.tickets and st.tile_bytes == 64 * KiB
            assert eng.job_schedule(jg, 2) == orc.job_schedule(jo, 2)
            if case % 2:
                kept.append(jg)
            else:
                binding.job_release(eng.pool, jg)
            _images_equal(orc, eng)
            for off in list(orc.pool.allocs):
                orc.slab_free(off)
                eng.slab_free(off)
        for jg in kept:
            binding.job_release(eng.pool, jg)
    finally:
        eng.close()


# bytes, chunk, tile asked for (0: none)
DEALT = [(3 * MiB - 9, 512, 0), (20 * MiB + 4112, 2 * MiB, 16 * KiB), (33 * MiB - 9, 1 * MiB + 4112, 16 * KiB),
         (150 * MiB + 5, 2 * MiB, 32 * KiB), (129 * MiB, 1008, 0)]


@pytest.mark.parametrize("n,chunk,tile", DEALT)
def test_one_aligned_tensor_dealt_out_in_the_pool(gpu, n, chunk, tile):
    """Tiles under 64 KiB of one aligned tensor are shared out without a counter: up to 128 MiB with ordinary loads and
    stores, beyond that with nontemporal ones; ragged last tile and chunk, bytes around the destination stay."""
    import torch
    binding, harness = gpu
    print(f"case copy kernel deals out {n} bytes, chunk {chunk}, tile {tile}", flush=True)
    eng = harness.GpuEngine()
    try:
        eng.pool_create(2 * n // MiB * MiB + 4 * MiB, 1 * MiB)
        mem = eng.segments[0][0]
        mem.random_(0, 256, generator=torch.Generator("cuda").manual_seed(5))
        binding.set_tuning(eng.pool, 2, 0, tile)
        a, b = eng.slab_alloc(n + 64), eng.slab_alloc(n + 64)
        want = mem.clone()
        want[b + 32:b + 32 + n] = want[a + 16:a + 16 + n]
        d = make_descs([dict(func=0, src_space=FT_POOL, dst_space=FT_POOL, src=a + 16, dst=b + 32, row_bytes=n)])
        torch.cuda.synchronize()
        jg = eng.submit(d, [1], chunk, fmt.FT_KEEP)
        eng.wait(jg)
        st = binding.job_stats(eng.pool, jg).cls[2]
        assert st.in_launch == 1 and st.workgroups == torch.cuda.get_device_properties(0).multi_processor_count < st.tickets
        assert st.tile_bytes < 64 * KiB
        binding.job_release(eng.pool, jg)
        assert torch.equal(mem, want)
    finally:
        eng.close()
