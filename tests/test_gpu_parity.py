"""Parity of the HIP path with the CPU oracle, byte for byte, through the C ABI."""
import random

import numpy as np
import pytest

import oracle
from oracle import OracleEngine
from workloads import configs, runner, make_descs, FT_HOST, FT_POOL
from workloads import format as fmt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2411_01830_amd import binding, harness
    assert torch.cuda.is_available()
    return binding, harness


def _pool_image(eng):
    import torch
    return torch.cat([t for t, _ in eng.segments]).cpu().numpy()


def _compare_images(orc, eng):
    got_host = eng.host_np[:len(orc.host_mem)]
    assert np.array_equal(got_host, orc.host_mem), "host image differs"
    got_pool = _pool_image(eng)
    assert got_pool.shape == orc.pool_mem.shape
    if not np.array_equal(got_pool, orc.pool_mem):
        bad = np.flatnonzero(got_pool != orc.pool_mem)
        raise AssertionError(f"pool image differs at {len(bad)} bytes, first {bad[:8]}")


SCALED = [("tiny", 0.3), ("traffic", 0.2), ("feature", 0.02), ("contended", 0.01), ("large_mixed", 0.008)]


@pytest.mark.parametrize("name,scale", SCALED)
@pytest.mark.parametrize("path", ["kernel", "dma"])
def test_config_matches_oracle(gpu, name, scale, path):
    binding, harness = gpu
    print(f"case {name} scale {scale} path {path}", flush=True)
    plan = configs.CONFIGS[name](scale)
    orc = OracleEngine()
    rec_o = runner.run_plan(plan, orc)
    eng = harness.GpuEngine()
    flags = fmt.FT_VALIDATE | binding.FT_KEEP | (fmt.FT_PATH_DMA if path == "dma" else 0)
    try:
        rec_g = runner.run_plan(plan, eng, flags=flags)
        assert rec_g.alloc_off == rec_o.alloc_off
        assert rec_g.grows == rec_o.grows
        _compare_images(orc, eng)
        for jname, job in rec_g.jobs.items():
            for cls in (0, 1, 2):
                assert eng.job_schedule(job, cls) == orc.job_schedule(rec_o.jobs[jname], cls), (jname, cls)
            st = binding.job_stats(eng.pool, job)
            for cls in (0, 1, 2):
                assert st.cls[cls].payload_bytes == orc.job_class_bytes(rec_o.jobs[jname], cls)
            binding.job_release(eng.pool, job)
    finally:
        eng.close()


def _pair(gpu, host=1 << 20, pool=1 << 22, slab=4096, seed=0):
    _, harness = gpu
    orc, eng = OracleEngine(), harness.GpuEngine()
    rng = np.random.default_rng(seed)
    data = rng.integers(0, 256, host // 2, dtype=np.uint8)
    for e in (orc, eng):
        e.host_arena(host)
        e.pool_create(pool, slab)
        e.write_host(0, data)         # upper half of the arena keeps its fill: host destinations
    return orc, eng, rng


def _run_both(orc, eng, recs, w, C, flags=fmt.FT_VALIDATE):
    d = make_descs(recs)
    orc.wait(orc.submit(d, w, C))
    eng.wait(eng.submit(d, w, C, flags))
    _compare_images(orc, eng)


def test_every_alignment_pair(gpu):
    """src%16 x dst%16 for short, medium and long pieces, in all three classes; canaries
    around every destination are part of the compared image."""
    orc, eng, rng = _pair(gpu, host=1 << 25, pool=1 << 26, slab=16384)
    try:
        for n in (1, 7, 15, 16, 17, 31, 100, 255, 256, 257, 4095, 70001):
            recs = []
            hdst = (1 << 24)
            for sa in range(16):
                for da in range(16):
                    cls = (sa + da) % 3
                    span = n + 64
                    if cls == 0:      # host -> pool
                        b = orc.slab_alloc(span)
                        assert eng.slab_alloc(span) == b
                        recs.append(dict(func=(sa * 16 + da) % 3, src_space=FT_HOST, dst_space=FT_POOL,
                                         src=1024 + sa + 16 * int(rng.integers(0, 1000)), dst=b + 16 + da, row_bytes=n))
                    else:
                        a = orc.slab_alloc(span)
                        assert eng.slab_alloc(span) == a
                        fill = rng.integers(0, 256, span, dtype=np.uint8)
                        orc.write_pool(a, fill)
                        eng.write_pool(a, fill)
                        if cls == 1:  # pool -> host
                            recs.append(dict(func=1, src_space=FT_POOL, dst_space=FT_HOST, src=a + 16 + sa,
                                             dst=hdst + 16 + da, row_bytes=n))
                            hdst += (n + 48 + 15) // 16 * 16
                            assert hdst + n + 64 <= (1 << 25)
                        else:
                            b = orc.slab_alloc(span)
                            assert eng.slab_alloc(span) == b
                            recs.append(dict(func=2, src_space=FT_POOL, dst_space=FT_POOL, src=a + 16 + sa,
                                             dst=b + 16 + da, row_bytes=n))
            print(f"alignment case n={n} descs={len(recs)}", flush=True)
            _run_both(orc, eng, recs, [1, 2, 3], 4096)
            for off in list(orc.pool.allocs):
                orc.slab_free(off)
                eng.slab_free(off)
    finally:
        eng.close()


def test_random_pitched_descriptors(gpu):
    for seed in range(4):
        orc, eng, rng = _pair(gpu, host=1 << 23, pool=1 << 27, slab=16384, seed=seed)
        pyr = random.Random(seed)
        try:
            recs = []
            hdst = 1 << 22
            for i in range(60):
                rows = pyr.choice([1, 2, 5, 33, 200])
                rb = pyr.choice([1, 3, 16, 63, 64, 100, 255, 256, 257, 700, 1500, 3000])
                sp = rb + pyr.choice([0, 0, 1, 13, 64, 500])
                dp = rb + pyr.choice([0, 0, 1, 7, 64, 300])
                es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
                cls = pyr.choice([0, 1, 2, 2])
                if cls == 0:
                    if es + 16 > (1 << 22):
                        continue
                    b = orc.slab_alloc(ed + 32)
                    assert eng.slab_alloc(ed + 32) == b
                    recs.append(dict(func=i % 4, src_space=FT_HOST, dst_space=FT_POOL,
                                     src=pyr.randint(0, (1 << 22) - es - 1), dst=b + pyr.randint(0, 31),
                                     row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
                    continue
                a = orc.slab_alloc(es + 32)
                assert eng.slab_alloc(es + 32) == a
                fill = rng.integers(0, 256, es + 32, dtype=np.uint8)
                orc.write_pool(a, fill)
                eng.write_pool(a, fill)
                if cls == 1:
                    if hdst + ed + 64 > (1 << 23):
                        continue
                    recs.append(dict(func=i % 4, src_space=FT_POOL, dst_space=FT_HOST, src=a + pyr.randint(0, 31),
                                     dst=hdst + pyr.randint(0, 15), row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
                    hdst += ed + 32
                else:
                    b = orc.slab_alloc(ed + 32)
                    assert eng.slab_alloc(ed + 32) == b
                    recs.append(dict(func=i % 4, src_space=FT_POOL, dst_space=FT_POOL, src=a + pyr.randint(0, 31),
                                     dst=b + pyr.randint(0, 31), row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
            C = pyr.choice([16, 1024, 4096, 65536, 1 << 23])
            print(f"pitched seed={seed} descs={len(recs)} C={C}", flush=True)
            _run_both(orc, eng, recs, [1, 3, 2, 5], C)
        finally:
            eng.close()


def test_pitched_rows_at_the_limits_of_the_window_route(gpu):
    """pool->pool rows of 16 .. 4096 bytes move window by window; rows just outside take the other routines.
    Every row length at and around both limits and around a window's size, one to many rows (one pass of two,
    four and eight windows per lane, and several passes), equal and unequal pitches, random byte offsets on
    either side, and chunks small enough that tile boundaries cut rows. Whole pool image compared (the bytes
    between the rows of a destination are part of it)."""
    for seed, C in enumerate((16 * 1024, 1000 * 16, 1 << 21)):
        orc, eng, rng = _pair(gpu, host=1 << 20, pool=1 << 26, slab=16384, seed=100 + seed)
        pyr = random.Random(100 + seed)
        try:
            recs = []
            for rb in (15, 16, 17, 31, 32, 33, 47, 48, 4095, 4096, 4097):
                for rows in (2, 3, 40, 700):
                    if rb > 4000 and rows > 40:
                        rows = 300
                    sp = rb + pyr.choice([0, 1, 48, 333])
                    dp = rb + pyr.choice([0, 1, 48, 100])
                    es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
                    a = orc.slab_alloc(es + 32)
                    assert eng.slab_alloc(es + 32) == a
                    fill = rng.integers(0, 256, es + 32, dtype=np.uint8)
                    orc.write_pool(a, fill)
                    eng.write_pool(a, fill)
                    b = orc.slab_alloc(ed + 32)
                    assert eng.slab_alloc(ed + 32) == b
                    recs.append(dict(func=len(recs) % 3, src_space=FT_POOL, dst_space=FT_POOL, src=a + pyr.randint(0, 31),
                                     dst=b + pyr.randint(0, 31), row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
            print(f"window limits seed={seed} descs={len(recs)} C={C}", flush=True)
            _run_both(orc, eng, recs, [1, 2, 3], C)
        finally:
            eng.close()


def test_chunk_and_tile_shapes(gpu):
    """Chunks smaller than, equal to and not a multiple of the tile; tuned tile sizes."""
    binding, _ = gpu
    for C, tile in ((16, 0), (48, 32), (4096, 1000), (65536, 0), (65536 + 16, 0), (1 << 20, 4096), (3 << 16, 1 << 16)):
        orc, eng, rng = _pair(gpu, seed=C % 97)
        try:
            for cls in (0, 1, 2):
                binding.set_tuning(eng.pool, cls, 0, tile)
            recs = []
            for i in range(6):
                n = int(rng.integers(1, 200000))
                a = orc.slab_alloc(n)
                assert eng.slab_alloc(n) == a
                recs.append(dict(func=i % 2, src_space=FT_HOST, dst_space=FT_POOL, src=int(rng.integers(0, 300000)),
                                 dst=a, row_bytes=n))
            print(f"tile case C={C} tile={tile}", flush=True)
            _run_both(orc, eng, recs, [2, 1], C)
        finally:
            eng.close()


def test_jobs_on_one_stream_run_in_order(gpu):
    """host->pool then pool->pool of the same bytes then pool->host: each job reads what
    the previous one wrote, with no host synchronisation in between."""
    orc, eng, rng = _pair(gpu)
    try:
        n = 300001
        a = orc.slab_alloc(n); assert eng.slab_alloc(n) == a
        b = orc.slab_alloc(n); assert eng.slab_alloc(n) == b
        j1 = make_descs([dict(func=0, src_space=FT_HOST, dst_space=FT_POOL, src=5, dst=a, row_bytes=n)])
        j2 = make_descs([dict(func=0, src_space=FT_POOL, dst_space=FT_POOL, src=a, dst=b + 0, row_bytes=n)])
        j3 = make_descs([dict(func=0, src_space=FT_POOL, dst_space=FT_HOST, src=b, dst=(1 << 19) + 3, row_bytes=n)])
        for d in (j1, j2, j3):
            orc.wait(orc.submit(d, [1], 4096))
        jobs = [eng.submit(d, [1], 4096) for d in (j1, j2, j3)]
        for j in jobs:
            eng.wait(j)
        _compare_images(orc, eng)
        assert np.array_equal(eng.read_host((1 << 19) + 3, n), eng.read_host(5, n))
    finally:
        eng.close()


def test_busy_allocation_and_empty_job(gpu):
    binding, _ = gpu
    orc, eng, rng = _pair(gpu)
    try:
        a = eng.slab_alloc(1 << 20)
        d = make_descs([dict(func=0, src_space=FT_HOST, dst_space=FT_POOL, src=0, dst=a, row_bytes=1 << 19)])
        j = eng.submit(d, [1], 65536)
        with pytest.raises(binding.FtError) as ei:
            eng.slab_free(a)
        assert ei.value.code == fmt.FT_EBUSY
        eng.wait(j)
        eng.slab_free(a)
        j = eng.submit(make_descs([]), [1], 64)
        eng.wait(j)
    finally:
        eng.close()


def test_log_and_timing(gpu):
    binding, _ = gpu
    orc, eng, rng = _pair(gpu, pool=1 << 24)
    try:
        recs = []
        sizes = [700000, 500000, 900000]
        for f, n in enumerate(sizes):
            a = eng.slab_alloc(n)
            b = eng.slab_alloc(n)
            eng.write_pool(a, rng.integers(0, 256, n, dtype=np.uint8))
            recs.append(dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a, dst=b, row_bytes=n))
        d = make_descs(recs)
        j = eng.submit(d, [1, 2, 1], 65536, binding.FT_LOG | binding.FT_TIMING)
        eng.wait(j)
        st = binding.job_stats(eng.pool, j)
        log = binding.job_log(eng.pool, j, 2)
        assert len(log["bytes"]) == st.cls[2].tickets
        assert int(log["bytes"].sum()) == sum(sizes) == st.cls[2].payload_bytes
        for f, n in enumerate(sizes):
            assert int(log["bytes"][log["func"] == f].sum()) == n
        assert np.all(log["t_end_ns"] >= log["t_begin_ns"])
        assert st.cls[2].device_ms > 0
        span_ms = (int(log["t_end_ns"].max()) - int(log["t_begin_ns"].min())) / 1e6
        assert span_ms <= st.cls[2].device_ms * 1.5 + 0.5
        # which workgroup moved which ticket, and when each workgroup came and went (same clock)
        wg, t_in, t_out = binding.job_log_workgroups(eng.pool, j, 2, len(log["bytes"]))
        assert len(t_in) == st.cls[2].workgroups == len(t_out)
        assert int(wg.max()) < len(t_in)
        assert set(np.unique(wg).tolist()) == set(range(len(t_in)))       # no more workgroups than tickets
        assert np.all(t_out >= t_in)
        for g in range(len(t_in)):
            mine = wg == g
            assert int(log["t_begin_ns"][mine].min()) >= int(t_in[g])
            assert int(log["t_end_ns"][mine].max()) <= int(t_out[g])
        # workgroup b starts on ticket b
        assert wg[:len(t_in)].tolist() == list(range(len(t_in)))
        binding.job_release(eng.pool, j)
    finally:
        eng.close()


def test_plain_copy_kernel_copies(gpu):
    """The plain grid-stride copy that the benchmark uses as its yardstick, at a size with a ragged end."""
    import torch
    binding, _ = gpu
    n = (3 << 20) + 16 * 7
    a = torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda:0")
    b = torch.zeros(n + 64, dtype=torch.uint8, device="cuda:0")
    for wg in (0, 1, 256):
        b.zero_()
        binding.plain_copy(b.data_ptr(), a.data_ptr(), n, wg, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(b[:n], a) and int(b[n:].sum()) == 0


def test_plain_read_and_fill_kernels(gpu):
    """The two other yardsticks: the fill writes exactly its range, the read changes nothing."""
    import torch
    binding, _ = gpu
    n = (2 << 20) + 16 * 5
    st = torch.cuda.current_stream().cuda_stream
    b = torch.full((n + 64,), 7, dtype=torch.uint8, device="cuda:0")
    for wg in (0, 1, 300):
        b.fill_(7)
        binding.plain_fill(b.data_ptr() + 16, n, 0xC3C3C3C3, wg, st)
        torch.cuda.synchronize()
        assert int((b[16:16 + n] != 0xC3).sum()) == 0
        assert int((b[:16] != 7).sum()) == 0 and int((b[16 + n:] != 7).sum()) == 0
    before = b.clone()
    binding.plain_read(b.data_ptr(), n, 0, st)
    binding.plain_read(b.data_ptr(), 16, 64, st)
    torch.cuda.synchronize()
    assert torch.equal(b, before)
    with pytest.raises(binding.FtError) as err:
        binding.plain_fill(b.data_ptr() + 1, 16, 0, 0, st)
    assert err.value.code == fmt.FT_EINVAL


def test_small_jobs_take_the_launch_argument_path(gpu):
    """Single-class jobs of a few descriptors travel with the launch (tables as a kernel argument,
    one workgroup per ticket, the caller's stream). Same bytes and same order as the oracle for
    every class, 1-D and pitched, every alignment, several functions and weights, back to back."""
    binding, _ = gpu
    orc, eng, rng = _pair(gpu, host=1 << 24, pool=1 << 27, slab=16384, seed=77)
    pyr = random.Random(77)
    try:
        took = {0: 0, 1: 0, 2: 0}
        hdst = 1 << 23
        for case in range(90):
            cls = case % 3
            nfunc = pyr.choice([1, 1, 2, 3])
            recs = []
            for _ in range(pyr.choice([1, 1, 2, 5, 9])):
                rows = pyr.choice([1, 1, 1, 3, 40])
                rb = pyr.choice([1, 15, 16, 100, 4096, 20000, 70001]) if rows == 1 else pyr.choice([3, 64, 200, 1000])
                sp, dp = rb + pyr.choice([0, 5, 64]), rb + pyr.choice([0, 0, 9])
                es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
                sa, da = pyr.randrange(16), pyr.randrange(16)
                if cls == 0:
                    src, sspace = pyr.randrange(0, (1 << 23) - es - 16), FT_HOST
                else:
                    a = orc.slab_alloc(es + 32)
                    assert eng.slab_alloc(es + 32) == a
                    fill = rng.integers(0, 256, es + 32, dtype=np.uint8)
                    orc.write_pool(a, fill)
                    eng.write_pool(a, fill)
                    src, sspace = a + sa, FT_POOL
                if cls == 1:
                    dst, dspace = hdst + da, FT_HOST
                    hdst += (ed + 47) // 16 * 16
                    assert hdst < (1 << 24) - 100000
                else:
                    b = orc.slab_alloc(ed + 32)
                    assert eng.slab_alloc(ed + 32) == b
                    dst, dspace = b + da, FT_POOL
                recs.append(dict(func=pyr.randrange(nfunc), src_space=sspace, dst_space=dspace, src=src, dst=dst,
                                 row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
            w = [pyr.choice([1, 2, 5]) for _ in range(nfunc)]
            C = pyr.choice([4096, 65536, 2 << 20])
            d = make_descs(recs)
            jo = orc.submit(d, w, C)
            orc.wait(jo)
            jg = eng.submit(d, w, C, fmt.FT_VALIDATE | fmt.FT_KEEP | (fmt.FT_TIMING if case % 2 else 0))
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg)
            took[cls] += st.cls[cls].in_launch
            if st.cls[cls].in_launch:
                assert st.cls[cls].workgroups == st.cls[cls].tickets
            assert eng.job_schedule(jg, cls) == orc.job_schedule(jo, cls), case
            binding.job_release(eng.pool, jg)
            if case % 10 == 9:
                _compare_images(orc, eng)
        _compare_images(orc, eng)
        print("jobs that travelled with the launch, per class:", took, flush=True)
        assert all(v >= 15 for v in took.values()), took
    finally:
        eng.close()


def test_larger_single_class_jobs_reuse_the_self_resetting_counters(gpu):
    """Single-class jobs with more tickets than workgroups still travel with the launch, on a
    counter pair that the kernel itself sets back to zero: thirty jobs back to back (the same pair
    again and again), kept jobs holding a pair each meanwhile, all three classes, odd sizes. (Most of the pool->pool jobs
    here go to the wave kernel, which may need no pair; test_gpu_copy_kernel.py has the copy kernel's.)"""
    binding, _ = gpu
    orc, eng, rng = _pair(gpu, host=1 << 26, pool=3 << 27, slab=1 << 20, seed=79)
    pyr = random.Random(79)
    try:
        kept = []
        took = {0: 0, 1: 0, 2: 0}
        for case in range(30):
            cls = case % 3
            recs = []
            hdst = 1 << 25
            nfunc = pyr.choice([1, 2])
            for _ in range(pyr.choice([1, 2, 3])):
                n = pyr.choice([3 << 20, (5 << 20) + 17, (9 << 20) + 4096]) if cls != 2 else \
                    pyr.choice([17 << 20, (20 << 20) + 33, 24 << 20])
                sa, da = pyr.randrange(16), pyr.choice([0, 0, pyr.randrange(16)])
                if cls == 0:
                    src, sspace = pyr.randrange(0, (1 << 25) - n - 16), FT_HOST
                else:
                    a = orc.slab_alloc(n + 32)
                    assert eng.slab_alloc(n + 32) == a
                    fill = rng.integers(0, 256, n + 32, dtype=np.uint8)
                    orc.write_pool(a, fill)
                    eng.write_pool(a, fill)
                    src, sspace = a + sa, FT_POOL
                if cls == 1:
                    dst, dspace = hdst + da, FT_HOST
                    hdst += (n + 47) // 16 * 16
                    assert hdst + n < (1 << 26)
                else:
                    b = orc.slab_alloc(n + 32)
                    assert eng.slab_alloc(n + 32) == b
                    dst, dspace = b + da, FT_POOL
                recs.append(dict(func=pyr.randrange(nfunc), src_space=sspace, dst_space=dspace, src=src, dst=dst,
                                 row_bytes=n))
            w = [pyr.choice([1, 3]) for _ in range(nfunc)]
            d = make_descs(recs)
            jo = orc.submit(d, w, 2 << 20)
            orc.wait(jo)
            jg = eng.submit(d, w, 2 << 20, fmt.FT_KEEP)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg)
            took[cls] += st.cls[cls].in_launch
            assert st.cls[cls].in_launch == 1 and st.cls[cls].workgroups < st.cls[cls].tickets, (case, st.cls[cls].tickets)
            assert eng.job_schedule(jg, cls) == orc.job_schedule(jo, cls), case
            if case % 4 == 0:
                kept.append(jg)
            else:
                binding.job_release(eng.pool, jg)
            _compare_images(orc, eng)
            for off in list(orc.pool.allocs):
                orc.slab_free(off)
                eng.slab_free(off)
        for jg in kept:
            binding.job_release(eng.pool, jg)
        print("larger jobs that travelled with the launch, per class:", took, flush=True)
    finally:
        eng.close()


def test_one_aligned_tensor_is_dealt_out_without_a_counter(gpu):
    """One contiguous transfer between 16-byte aligned addresses (its length may be anything) which has more tiles than
    workgroups: the tiles are dealt out, no counter (Sec. 5.1: passing one tensor) - among the workgroups of the class's
    kernel over the host link, among the wavefronts of the wave kernel in the pool (test_gpu_copy_kernel.py has the copy kernel).
    Every class, lengths with a ragged last tile and a ragged last chunk, chunk sizes that are not a
    multiple of the tile, with and without timing; detached, such a job takes the ordinary route instead (it would
    hold the caller's stream); canaries around every destination."""
    binding, _ = gpu
    orc, eng, rng = _pair(gpu, host=1 << 26, pool=3 << 27, slab=1 << 20, seed=83)
    try:
        case = 0
        for cls in (0, 1, 2):
            sizes = [17 << 20, (20 << 20) + 4096 + 16, (33 << 20) - 9] if cls == 2 else \
                    [3 << 20, (5 << 20) + 48, (9 << 20) - 3]
            for n in sizes:
                for C in (2 << 20, (1 << 20) + 4096 + 16):
                    a = b = None
                    if cls == 0:
                        src, sspace = 4096 + 16 * case, FT_HOST
                    else:
                        a = orc.slab_alloc(n + 64)
                        assert eng.slab_alloc(n + 64) == a
                        fill = rng.integers(0, 256, n + 64, dtype=np.uint8)
                        orc.write_pool(a, fill)
                        eng.write_pool(a, fill)
                        src, sspace = a + 16, FT_POOL
                    if cls == 1:
                        dst, dspace = (1 << 25) + 32, FT_HOST
                    else:
                        b = orc.slab_alloc(n + 64)
                        assert eng.slab_alloc(n + 64) == b
                        dst, dspace = b + 32, FT_POOL
                    d = make_descs([dict(func=0, src_space=sspace, dst_space=dspace, src=src, dst=dst, row_bytes=n)])
                    flags = (fmt.FT_KEEP, fmt.FT_KEEP | fmt.FT_TIMING, fmt.FT_KEEP | fmt.FT_DETACHED)[case % 3]
                    jo = orc.submit(d, [3], C)
                    orc.wait(jo)
                    jg = eng.submit(d, [3], C, flags)
                    eng.wait(jg)
                    st = binding.job_stats(eng.pool, jg)
                    # a detached job of this size must not hold the caller's stream: it takes the ordinary route
                    assert st.cls[cls].in_launch == (0 if flags & fmt.FT_DETACHED else 1), (cls, n, C)
                    assert st.cls[cls].workgroups < st.cls[cls].tickets, (cls, n, C)
                    assert eng.job_schedule(jg, cls) == orc.job_schedule(jo, cls), (cls, n, C)
                    if flags & fmt.FT_TIMING:
                        assert st.cls[cls].device_ms > 0
                    binding.job_release(eng.pool, jg)
                    _compare_images(orc, eng)
                    for off in (a, b):
                        if off is not None:
                            orc.slab_free(off)
                            eng.slab_free(off)
                    case += 1
    finally:
        eng.close()


def test_detached_pool_to_pool_jobs_back_to_back_and_apart(gpu):
    """Detached jobs are independent: submitted back to back their pool->pool launches overlap on the class's two
    streams (a launch takes the other stream while the last one still runs), submitted apart they all take the
    first. Either way every byte is the oracle's; by their device times none of the launches submitted apart may
    overlap (how many of the back-to-back ones do depends on the host's pace and is only printed)."""
    import time
    binding, _ = gpu
    orc, eng, rng = _pair(gpu, host=1 << 20, pool=15 << 27, slab=1 << 20, seed=89)
    try:
        def job():
            recs = []
            for f in range(3):
                n = int(rng.integers(90 << 20, 100 << 20)) + int(rng.integers(0, 64))
                a, b = orc.slab_alloc(n + 32), orc.slab_alloc(n + 32)
                assert eng.slab_alloc(n + 32) == a and eng.slab_alloc(n + 32) == b
                fill = rng.integers(0, 256, n + 32, dtype=np.uint8)
                orc.write_pool(a, fill)
                eng.write_pool(a, fill)
                recs.append(dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a + int(rng.integers(0, 16)),
                                 dst=b + int(rng.integers(0, 16)), row_bytes=n))
            return make_descs(recs)
        import torch
        for apart in (False, True):
            descs = [job() for _ in range(3)]
            for d in descs:
                orc.wait(orc.submit(d, [1, 2, 4], 2 << 20))
            torch.cuda.synchronize()
            binding.timing_epoch(eng.pool, torch.cuda.current_stream().cuda_stream)
            handles = []
            for d in descs:
                handles.append(eng.submit(d, [1, 2, 4], 2 << 20, fmt.FT_KEEP | fmt.FT_DETACHED | fmt.FT_TIMING))
                if apart:
                    time.sleep(0.005)
            for h in handles:
                eng.wait(h)
            spans = []
            for h in handles:
                st = binding.job_stats(eng.pool, h)
                assert st.cls[2].in_launch == 0 and st.cls[2].end_ms > st.cls[2].begin_ms >= 0
                spans.append((st.cls[2].begin_ms, st.cls[2].end_ms))
                binding.job_release(eng.pool, h)
            overlaps = sum(1 for (b1, e1), (b2, e2) in zip(spans, spans[1:]) if b2 < e1)
            print("apart" if apart else "back to back", [(round(b, 3), round(e, 3)) for b, e in spans], flush=True)
            print("launches that began before the one before them had ended:", overlaps, flush=True)
            assert not apart or overlaps == 0, spans
            _compare_images(orc, eng)
            for off in list(orc.pool.allocs):
                orc.slab_free(off)
                eng.slab_free(off)
    finally:
        eng.close()


def test_short_rows_run_the_light_build_two_workgroups_per_unit(gpu):
    """A pool->pool job of over 16 MiB whose payload is mostly pitched rows of at most 2 KiB is launched with two workgroups
    of eight wavefronts per compute unit; one of long rows with one of sixteen. Gather into packed
    buffers, scatter out of them and pitched on both sides, row lengths 16 .. 1000 at every alignment, tiles that cut
    rows; bytes and order against the oracle."""
    import torch
    binding, _ = gpu
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    orc, eng, rng = _pair(gpu, host=1 << 20, pool=1 << 29, slab=1 << 16, seed=97)
    pyr = random.Random(97)
    try:
        for kind in ("gather", "scatter", "both", "long"):
            recs = []
            for i in range(32):
                rb = pyr.choice([4000, 8192]) if kind == "long" else pyr.choice([16, 17, 63, 64, 100, 160, 255, 256, 1000])
                rows = (1 << 20) // rb + pyr.randrange(7)
                sp = rb if kind == "scatter" else rb + pyr.choice([1, 16, 48])
                dp = rb if kind in ("gather", "long") else rb + pyr.choice([3, 16, 40])
                es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
                a, b = orc.slab_alloc(es + 32), orc.slab_alloc(ed + 32)
                assert eng.slab_alloc(es + 32) == a and eng.slab_alloc(ed + 32) == b
                fill = rng.integers(0, 256, es + 32, dtype=np.uint8)
                orc.write_pool(a, fill)
                eng.write_pool(a, fill)
                recs.append(dict(func=i % 3, src_space=FT_POOL, dst_space=FT_POOL, src=a + pyr.randrange(16),
                                 dst=b + pyr.randrange(16), row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
            d = make_descs(recs)
            jo = orc.submit(d, [1, 2, 3], 256 << 10)
            orc.wait(jo)
            jg = eng.submit(d, [1, 2, 3], 256 << 10, fmt.FT_VALIDATE | fmt.FT_KEEP)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg)
            print(kind, "tickets", st.cls[2].tickets, "workgroups", st.cls[2].workgroups, "tile", st.cls[2].tile_bytes, flush=True)
            assert st.cls[2].tickets > 2 * cus
            assert st.cls[2].workgroups == (cus if kind == "long" else 2 * cus), kind
            assert eng.job_schedule(jg, 2) == orc.job_schedule(jo, 2)
            binding.job_release(eng.pool, jg)
            _compare_images(orc, eng)
            for off in list(orc.pool.allocs):
                orc.slab_free(off)
                eng.slab_free(off)
    finally:
        eng.close()


def test_log_names_the_compute_unit_of_every_workgroup(gpu):
    """FT_LOG also records where a workgroup ran. A pool->pool launch of as many workgroups as the device has
    compute units occupies every unit once (two workgroups of sixteen wavefronts, here of misaligned tensors, do not fit one unit);
    one of two workgroups of eight wavefronts per unit, of short rows, occupies every unit twice."""
    import torch
    from collections import Counter
    binding, _ = gpu
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    orc, eng, rng = _pair(gpu, host=1 << 20, pool=3 << 27, slab=1 << 20, seed=101)
    try:
        n = 96 << 20
        a, b = orc.slab_alloc(n), orc.slab_alloc(n)
        assert eng.slab_alloc(n) == a and eng.slab_alloc(n) == b
        fill = rng.integers(0, 256, n, dtype=np.uint8)
        orc.write_pool(a, fill)
        eng.write_pool(a, fill)
        for rows, rb, per_unit in ((1, n // 2, 1), (n // 2 // 200, 200, 2)):
            recs = [dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a + f * (n // 2) + 3, dst=b + f * (n // 2) + 5,
                         row_bytes=rb - 16, rows=rows, src_pitch=rb, dst_pitch=rb - 16) for f in range(2)]
            d = make_descs(recs)
            orc.wait(orc.submit(d, [1, 2], 2 << 20))
            jg = eng.submit(d, [1, 2], 2 << 20, fmt.FT_LOG)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg)
            units = binding.job_log_units(eng.pool, jg, 2)
            assert len(units) == st.cls[2].workgroups == per_unit * cus
            count = Counter(int(u) for u in units)
            assert len(count) == cus and set(count.values()) == {per_unit}, sorted(count.values())[-4:]
            binding.job_release(eng.pool, jg)
            _compare_images(orc, eng)
    finally:
        eng.close()


def test_pool_to_host_stores_reach_the_link_while_the_kernel_runs(gpu):
    """The pool->host kernel writes its 16-byte stores through to the fabric as it issues them. Were they left in the
    L2, the workgroups would have issued their last store long before the launch ends (the L2 writes the lines back
    when the kernel finishes: 209 of 337 us on a job like this one). So: the workgroups' own record - first entry to
    last exit on the device clock - must cover nearly all of the dispatch's duration by its events. Bytes compared
    as everywhere."""
    binding, _ = gpu
    orc, eng, rng = _pair(gpu, host=1 << 25, pool=1 << 25, slab=1 << 16, seed=55)
    try:
        recs, hdst = [], 1 << 24
        for i in range(12):
            n = (1 << 20) + 16 * int(rng.integers(0, 4000)) + (i % 3)
            a = orc.slab_alloc(n + 32)
            assert eng.slab_alloc(n + 32) == a
            fill = rng.integers(0, 256, n + 32, dtype=np.uint8)
            orc.write_pool(a, fill)
            eng.write_pool(a, fill)
            recs.append(dict(func=i % 4, src_space=FT_POOL, dst_space=FT_HOST, src=a + (i % 5), dst=hdst + (i % 7), row_bytes=n))
            hdst += (n + 64 + 4095) // 4096 * 4096
        assert hdst <= 1 << 25
        d = make_descs(recs)
        orc.wait(orc.submit(d, [1, 1, 2, 2], 64 * 1024))
        covered = []
        for attempt in range(3):
            jg = eng.submit(d, [1, 1, 2, 2], 64 * 1024, fmt.FT_LOG | fmt.FT_TIMING)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg)
            _, t_in, t_out = binding.job_log_workgroups(eng.pool, jg, 1, st.cls[1].tickets)
            span_ms = (int(t_out.max()) - int(t_in.min())) / 1e6
            covered.append(span_ms / st.cls[1].device_ms)
            binding.job_release(eng.pool, jg)
        _compare_images(orc, eng)
        print(f"pool->host: workgroups at work for {[round(c, 3) for c in covered]} of the dispatch", flush=True)
        assert max(covered) >= 0.85, covered
    finally:
        eng.close()


def test_a_detached_pool_to_pool_job_does_not_wait_for_another_jobs_host_link_kernel(gpu):
    """Job A carries 128 MiB host->pool (2 ms on the link) and 1 GiB pool->pool, job B, submitted right behind it, 64 MiB
    pool->pool; both detached. B's launch may queue behind A's pool->pool launch but must be over long before A's
    host->pool kernel is: the library's streams share the process's few hardware queues, and a pool->pool launch put
    on a stream that shares one with the host->pool stream would run after that kernel instead of beside it."""
    import torch
    binding, _ = gpu
    MiB = 1 << 20
    orc, eng, rng = _pair(gpu, host=256 * MiB, pool=2432 * MiB, slab=MiB, seed=103)
    try:
        def alloc(n, fill):
            a = orc.slab_alloc(n)
            assert eng.slab_alloc(n) == a
            if fill:
                data = rng.integers(0, 256, n, dtype=np.uint8)
                orc.write_pool(a, data)
                eng.write_pool(a, data)
            return a
        h_dst, a_src, a_dst = alloc(128 * MiB, False), alloc(1024 * MiB, True), alloc(1024 * MiB, False)
        b_src, b_dst = alloc(64 * MiB, True), alloc(64 * MiB, False)
        job_a = make_descs([dict(func=0, src_space=FT_HOST, dst_space=FT_POOL, src=0, dst=h_dst, row_bytes=128 * MiB),
                            dict(func=1, src_space=FT_POOL, dst_space=FT_POOL, src=a_src, dst=a_dst, row_bytes=1024 * MiB)])
        job_b = make_descs([dict(func=0, src_space=FT_POOL, dst_space=FT_POOL, src=b_src, dst=b_dst, row_bytes=32 * MiB),
                            dict(func=1, src_space=FT_POOL, dst_space=FT_POOL, src=b_src + 32 * MiB, dst=b_dst + 32 * MiB,
                                 row_bytes=32 * MiB)])
        for d in (job_a, job_b):
            orc.wait(orc.submit(d, [1, 1], 2 * MiB))
        for attempt in range(2):        # the first pass also pays for first touches of fresh memory
            torch.cuda.synchronize()
            binding.timing_epoch(eng.pool, torch.cuda.current_stream().cuda_stream)
            flags = fmt.FT_KEEP | fmt.FT_DETACHED | fmt.FT_TIMING
            ja = eng.submit(job_a, [1, 1], 2 * MiB, flags)
            jb = eng.submit(job_b, [1, 1], 2 * MiB, flags)
            eng.wait(ja)
            eng.wait(jb)
            sa, sb = binding.job_stats(eng.pool, ja), binding.job_stats(eng.pool, jb)
            binding.job_release(eng.pool, ja)
            binding.job_release(eng.pool, jb)
        print("A host->pool", round(sa.cls[0].begin_ms, 3), round(sa.cls[0].end_ms, 3), "A pool->pool", round(sa.cls[2].begin_ms, 3),
              round(sa.cls[2].end_ms, 3), "B pool->pool", round(sb.cls[2].begin_ms, 3), round(sb.cls[2].end_ms, 3), flush=True)
        assert sa.cls[0].end_ms - sa.cls[0].begin_ms > 1.5
        assert sb.cls[2].end_ms < sa.cls[0].begin_ms + 0.5 * (sa.cls[0].end_ms - sa.cls[0].begin_ms)
        _compare_images(orc, eng)
    finally:
        eng.close()


def test_random_sequences_of_mixed_jobs(gpu):
    """Sixty jobs per seed, each a random mix of classes, sizes from bytes to MiB, pitched and plain,
    every alignment, random weights, chunk sizes, tile sizes and workgroup counts (tuned and default, so
    both launch routes are taken), allocations freed and taken again in between. After every tenth job
    the whole host image and the whole pool image are the oracle's."""
    binding, _ = gpu
    for seed in (101, 102, 103):
        orc, eng, rng = _pair(gpu, host=1 << 25, pool=1 << 28, slab=1 << 16, seed=seed)
        pyr = random.Random(seed)
        try:
            live = []
            for job in range(60):
                hdst = 1 << 24
                recs = []
                nfunc = pyr.choice([1, 2, 3, 6])
                classes = pyr.choice([[0], [1], [2], [0, 2], [0, 1, 2]])
                for _ in range(pyr.choice([1, 2, 4, 12])):
                    cls = pyr.choice(classes)
                    rows = pyr.choice([1, 1, 1, 2, 17, 120])
                    if rows == 1:
                        rb = pyr.choice([1, 9, 16, 250, 4096, 70000, 300001, (1 << 20) + 5, 3 << 20])
                    else:
                        rb = pyr.choice([2, 16, 31, 64, 190, 512, 1100, 5000])
                    sp = rb + pyr.choice([0, 0, 3, 64, 900])
                    dp = rb + pyr.choice([0, 0, 0, 5, 128])
                    es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
                    if cls == 0:
                        src, sspace = pyr.randrange(0, (1 << 24) - es), FT_HOST
                    else:
                        a = orc.slab_alloc(es + 32)
                        assert eng.slab_alloc(es + 32) == a
                        live.append(a)
                        fill = rng.integers(0, 256, es + 32, dtype=np.uint8)
                        orc.write_pool(a, fill)
                        eng.write_pool(a, fill)
                        src, sspace = a + pyr.randrange(32), FT_POOL
                    if cls == 1:
                        if hdst + ed + 64 > (1 << 25):
                            continue
                        dst, dspace = hdst + pyr.randrange(16), FT_HOST
                        hdst += (ed + 47) // 16 * 16
                    else:
                        b = orc.slab_alloc(ed + 32)
                        assert eng.slab_alloc(ed + 32) == b
                        live.append(b)
                        dst, dspace = b + pyr.randrange(32), FT_POOL
                    recs.append(dict(func=pyr.randrange(nfunc), src_space=sspace, dst_space=dspace, src=src, dst=dst,
                                     row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
                w = [pyr.choice([1, 1, 2, 3, 7]) for _ in range(nfunc)]
                C = pyr.choice([64, 4096, 65536, 1 << 20, 2 << 20])
                for cls in (0, 1, 2):
                    binding.set_tuning(eng.pool, cls, pyr.choice([0, 0, 1, 3, 64, 300]),
                                       pyr.choice([0, 0, 0, 16, 1000, 4096, 12272, 1 << 16]))
                d = make_descs(recs)
                jo = orc.submit(d, w, C)
                orc.wait(jo)
                jg = eng.submit(d, w, C, fmt.FT_KEEP | (fmt.FT_VALIDATE if job % 3 == 0 else 0))
                eng.wait(jg)
                for cls in (0, 1, 2):
                    assert eng.job_schedule(jg, cls) == orc.job_schedule(jo, cls), (seed, job, cls)
                binding.job_release(eng.pool, jg)
                if job % 10 == 9:
                    _compare_images(orc, eng)
                    pyr.shuffle(live)
                    for off in live[:len(live) * 2 // 3]:
                        orc.slab_free(off)
                        eng.slab_free(off)
                    live = live[len(live) * 2 // 3:]
            print(f"random sequence seed={seed} done", flush=True)
        finally:
            eng.close()


@pytest.mark.parametrize("weights", [[1000, 1, 4096, 3], [1, 1, 1, 1], [4000000000, 1, 1, 2], [7, 7, 7, 7], [3, 5, 1000003, 2]])
def test_device_order_with_extreme_weights(gpu, weights):
    """Weights that dwarf the chunk counts, equal weights, a weight near 2^32, weights with a common
    factor and a large prime: the order the device decodes (uploaded tables) is the oracle's, and so
    are the bytes."""
    orc, eng, rng = _pair(gpu, host=1 << 22, pool=1 << 24, slab=4096, seed=sum(weights) % 1000)
    try:
        C = 4096
        sizes = [3 * C - 5, 50 * C, 7 * C + 1, 200 * C - 4095]
        recs = []
        for f, n in enumerate(sizes):
            a = orc.slab_alloc(n)
            assert eng.slab_alloc(n) == a
            recs.append(dict(func=f, src_space=FT_HOST, dst_space=FT_POOL, src=int(rng.integers(0, 1 << 20)), dst=a,
                             row_bytes=n))
        d = make_descs(recs)
        jo = orc.submit(d, weights, C)
        orc.wait(jo)
        # a tuned workgroup count keeps the job on the route with uploaded tables and a counter
        from paper_2411_01830_amd import binding
        binding.set_tuning(eng.pool, 0, 7, 0)
        jg = eng.submit(d, weights, C, fmt.FT_KEEP | fmt.FT_VALIDATE)
        eng.wait(jg)
        assert eng.job_schedule(jg, 0) == orc.job_schedule(jo, 0)
        binding.job_release(eng.pool, jg)
        _compare_images(orc, eng)
    finally:
        eng.close()
