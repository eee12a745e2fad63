"""Jobs that are launched as a list of pieces: of runs, pool->pool at most 128 MiB or beyond that mostly misaligned, and over the host link, and of few pitched rows; none
whose schedule may be asked for. Bit-exact against the oracle (jobs beyond 128 MiB and lists in memory: against torch's copies) at the sizes where tiles, windows, the forms of the tables and the rule change."""
import numpy as np
import pytest

from oracle import OracleEngine
from workloads import make_descs, FT_POOL
from workloads import format as fmt
from test_host_logic import _host_sanitizer_run

KiB, MiB = 1 << 10, 1 << 20


def test_pieces_are_the_general_order_written_out(tmp_path):
    """tests/host/piece_tables.cpp: the pieces hold the bytes of the general walk in its order, and the kernels' arithmetic moves each
    byte once and nothing else."""
    _host_sanitizer_run(tmp_path, "piece_tables", ["ft_plan.cpp", "ft_pool.cpp"], ["1", "40"], "done 1..40")


def _runs(rng, n, sizes, funcs, odd=True):
    shift = (lambda: int(rng.integers(0, 16))) if odd else (lambda: 0)
    return [(int(sizes[i % len(sizes)] if len(sizes) >= n else rng.choice(sizes)), 1, 0, 0, i % funcs, shift(), shift()) for i in range(n)]


def _rows(rng, n, widths, total, funcs):
    out = []
    for i in range(n):
        rb = int(widths[i % len(widths)])
        out.append((rb, max(2, total // n // rb), rb + int(rng.integers(0, 50)), rb + int(rng.integers(0, 3)) * 7, i % funcs,
                    int(rng.integers(0, 16)), int(rng.integers(0, 16))))
    return out


def _tile(payload):
    return 2 * KiB if payload <= 10 * MiB else 4 * KiB if payload <= 20 * MiB else 8 * KiB


# name, pieces(rng): (row bytes, rows, src pitch, dst pitch, function, src shift, dst shift), weights, chunk, travels with its launch
# ("any": it may; None: not launched as pieces; "either": nor this, by a kernel of the same shape)
CASES = [
    ("one byte", lambda g: [(1, 1, 0, 0, 0, 3, 9)], [1], 2 * MiB, True),
    *[(f"one tensor of {n}", lambda g, n=n: [(n, 1, 0, 0, 0, 7, 4)], [1], 2 * MiB, True) for n in (15, 16, 17, 2047, 2048, 2049, 65536, 10 * MiB, 10 * MiB + 1, 20 * MiB + 1)],
    ("one aligned tensor", lambda g: [(64 * KiB, 1, 0, 0, 0, 0, 0)], [1], 2 * MiB, True),
    *[(f"{n} tensors of one function", lambda g, n=n: _runs(g, n, [1, 15, 16, 17, 127, 128, 129, 2047, 2048, 2049, 5000], 1), [1], 4 * KiB, n <= 240)
      for n in (2, 16, 17, 48, 49, 63, 64, 65, 128, 129, 192, 193, 240, 241)],
    ("lengths around a tile, aligned", lambda g: _runs(g, 60, [2032, 2048, 2064, 4096, 8176, 8192, 8208], 2, odd=False), [1, 1], 64 * KiB, True),
    ("chunks of 1 KiB", lambda g: _runs(g, 900, [1, 15, 16, 17, 1023, 1024, 1025], 3), [1, 2, 5], 1024, False),
    ("30 functions", lambda g: _runs(g, 70, [64, 5000, 9000], 30), list(range(1, 31)), 16 * KiB, True),
    ("1025 functions", lambda g: _runs(g, 2100, [64, 5000, 9000], 1025), [1] * 1025, 4 * KiB, False),
    ("5000 tensors", lambda g: _runs(g, 5000, [1, 60, 300, 700], 1), [1], 256 * KiB, False),
    ("tiles of 4 KiB", lambda g: _runs(g, 30, [400 * KiB, 500 * KiB + 5], 3), [1, 2, 4], 256 * KiB, True),
    ("tiles of 8 KiB", lambda g: _runs(g, 300, [80 * KiB + 3, 100 * KiB], 3), [1, 2, 4], 256 * KiB, False),
    ("few tensors in many chunks", lambda g: _runs(g, 20, [100 * KiB + 3, 100 * KiB], 4), [1, 2, 4, 1], 4 * KiB, "either"),
    ("over 20 MiB", lambda g: _runs(g, 30, [800 * KiB + 3, 1000 * KiB], 3), [1, 2, 4], 2 * MiB, True),
    ("chunks under 1 KiB", lambda g: _runs(g, 200, [300, 5000], 2), [1, 3], 512, None),
    ("rows of 16 bytes and a bit", lambda g: _rows(g, 14, [16, 17, 31, 32, 33, 47, 48], 2 * MiB, 2), [1, 2], 1 * MiB, True),
    ("rows cut by every chunk", lambda g: _rows(g, 10, [16, 17, 40, 100, 255, 2047, 2048], 400 * KiB, 3), [1, 2, 5], 1024, "either"),
    ("rows cut by every chunk, one function", lambda g: _rows(g, 16, [16, 17, 40, 100, 255, 2047, 2048], 200 * KiB, 1), [1], 1024, True),
    ("rows longer than a tile", lambda g: _rows(g, 6, [2049, 8193, 20000, 66000], 1 * MiB, 2), [3, 1], 1 * MiB, "any"),
    ("rows around a tile of 8 KiB", lambda g: _rows(g, 8, [4096, 4097, 8191, 8192, 8193, 8208], 22 * MiB, 2), [3, 1], 2 * MiB, "any"),
    ("rows and runs", lambda g: _rows(g, 20, [16, 100, 3000], 600 * KiB, 2) + _runs(g, 20, [1, 16, 5000, 70000], 2), [1, 2], 64 * KiB, "any"),
    ("100 pieces of few shapes", lambda g: [(100, 20, 160, 100, i % 2, i % 7, i % 5) for i in range(100)], [1, 1], 64 * KiB, True),
    ("200 pieces of few shapes", lambda g: [(100, 20, 160, 100, i % 2, i % 7, i % 5) for i in range(200)], [1, 1], 64 * KiB, "either"),
    ("70 shapes", lambda g: _rows(g, 70, list(range(16, 86)), 300 * KiB, 1), [1], 64 * KiB, "either"),
    ("single rows", lambda g: [(100, 2, 160, 100, i % 2, i % 7, i % 5) for i in range(30)], [1, 1], 1024, "any"),
    ("rows under 16 bytes", lambda g: _rows(g, 20, [1, 2, 3, 5, 8, 15], 100 * KiB, 2), [1, 2], 64 * KiB, None),
    ("rows between 1 MiB pitches", lambda g: [(100, 9, 1 << 20, 200, 0, 3, 5), (70, 5, 100, 1 << 20, 1, 1, 2), (50, 6, (1 << 20) + 1, 60, 0, 0, 0)],
     [1, 1], 64 * KiB, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_pieces_match_the_oracle(case):
    import torch
    from paper_2411_01830_amd import binding, harness
    name, pieces, weights, chunk, along = case
    print(f"case pieces: {name}", flush=True)
    rng = np.random.default_rng(len(name))
    orc, eng = OracleEngine(), harness.GpuEngine()
    try:
        for e in (orc, eng):
            e.host_arena(1 << 20)
            e.pool_create(96 * MiB, 4 * KiB)
        recs = []
        for rb, rows, sp, dp, f, ss, ds in pieces(rng):
            es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
            a, b = orc.slab_alloc(es + 16), orc.slab_alloc(ed + 16)
            assert eng.slab_alloc(es + 16) == a and eng.slab_alloc(ed + 16) == b
            fill = rng.integers(0, 256, es + 16, dtype=np.uint8)
            orc.write_pool(a, fill)
            eng.write_pool(a, fill)
            recs.append(dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a + ss, dst=b + ds, row_bytes=rb, rows=rows,
                             src_pitch=sp if rows > 1 else rb, dst_pitch=dp if rows > 1 else rb))
        before = torch.cat([t for t, _ in eng.segments]).clone()
        d = make_descs(recs)
        jo = orc.submit(d, weights, chunk)
        orc.wait(jo)
        payload = sum(r["row_bytes"] * r["rows"] for r in recs)

        def check(what):
            assert np.array_equal(torch.cat([t for t, _ in eng.segments]).cpu().numpy(), orc.pool_mem), what
            at = 0
            for t, _ in eng.segments:
                t.copy_(before[at:at + t.numel()])
                at += t.numel()
            torch.cuda.synchronize()

        for flags in (0, 0, fmt.FT_DETACHED, fmt.FT_TIMING):
            jg = eng.submit(d, weights, chunk, flags | fmt.FT_VALIDATE)
            eng.wait(jg)
            if flags & fmt.FT_TIMING:
                st = binding.job_stats(eng.pool, jg).cls[2]
                own = st.tile_bytes == _tile(payload) and st.workgroups == st.tickets
                if along is None:
                    assert not own
                elif along != "either":
                    assert own and (along == "any" or st.in_launch == along) and st.device_ms > 0, (st.tile_bytes, st.tickets, st.in_launch)
                assert eng.job_schedule(jg, 2) == orc.job_schedule(jo, 2)
                binding.job_release(eng.pool, jg)
            check(flags)
        torch.cuda.synchronize()
        if len(recs) < 600:
            eng.submit_static(d, weights, chunk, fmt.FT_VALIDATE)
            torch.cuda.synchronize()
            check("static")
    finally:
        eng.close()


@pytest.mark.gpu
def test_the_largest_job_of_pieces_and_the_next():
    """128 MiB goes as pieces, 16 bytes more by the copy kernel; a static submit captured into a graph is replayed on new bytes."""
    import torch
    from paper_2411_01830_amd import binding, harness
    print("case the largest job of pieces", flush=True)
    eng = harness.GpuEngine()
    try:
        eng.host_arena(1 << 20)
        eng.pool_create(320 * MiB, 4 * KiB)
        mem = eng.segments[0][0]
        g = torch.Generator("cuda").manual_seed(5)
        mem.random_(0, 256, generator=g)
        n = 64 * MiB
        src, dst = [eng.slab_alloc(n + 4096) for _ in range(2)], [eng.slab_alloc(n + 4096) for _ in range(2)]
        for more in (0, 16):
            recs = [dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=src[f] + 3 * f, dst=dst[f] + 5 * f, row_bytes=n + more * f) for f in range(2)]
            want = mem.clone()
            for r in recs:
                want[r["dst"]:r["dst"] + r["row_bytes"]] = mem[r["src"]:r["src"] + r["row_bytes"]]
            jg = eng.submit(make_descs(recs), [1, 2], 2 * MiB, fmt.FT_TIMING)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg).cls[2]
            assert (st.tile_bytes, st.workgroups == st.tickets) == ((8 * KiB, True) if more == 0 else (64 * KiB, False))
            binding.job_release(eng.pool, jg)
            assert torch.equal(mem, want)
            mem.random_(0, 256, generator=g)
        recs = [dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=src[f], dst=dst[f] + f, row_bytes=3 * MiB + f) for f in range(2)]
        d = make_descs(recs)
        s = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            binding.submit_static(eng.pool, d, [1, 2], 256 * KiB, 0, torch.cuda.current_stream().cuda_stream)
        for _ in range(3):
            mem.random_(0, 256, generator=g)
            want = mem.clone()
            for r in recs:
                want[r["dst"]:r["dst"] + r["row_bytes"]] = mem[r["src"]:r["src"] + r["row_bytes"]]
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(mem, want)
    finally:
        eng.close()


def test_lists_in_memory_read_back_as_they_were_written(tmp_path):
    """tests/host/packed_pieces.cpp: both forms of a list in memory, found by blocks and lengths as the kernels find them."""
    _host_sanitizer_run(tmp_path, "packed_pieces", ["ft_plan.cpp", "ft_pool.cpp"], [], "done")


@pytest.mark.gpu
@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("n", [241, 1024, 1025, 2730, 2731, 4096, 4097, 16384])
def test_lists_in_memory_of_every_size(n, far):
    """The blocks in the arguments (16, 64, 256), lists read in place and uploaded, sides close to each other and 4 GiB apart."""
    import torch
    from paper_2411_01830_amd import binding
    print(f"case lists in memory: {n}, far apart: {far}", flush=True)
    rng = np.random.default_rng(n)
    half = 16 * MiB
    mem = torch.empty((4 << 30) + half if far else 2 * half, dtype=torch.uint8, device="cuda")
    lo, hi = mem[:half], mem[-half:]
    pool = binding.pool_create(lo.data_ptr(), half, 4 * KiB, 0)
    try:
        binding.pool_grow(pool, hi.data_ptr(), half)
        binding.slab_alloc(pool, half)
        binding.slab_alloc(pool, half)
        sizes = rng.integers(1, 900 if n < 10000 else 400, n)
        # every third tensor from the other side; what one side reads the other's tensors do not write
        swap = np.arange(n) % 3 == 0
        at = np.concatenate([[0], np.cumsum(sizes + 17)[:-1]])
        assert at[-1] + 1000 < half // 2
        src = np.where(swap, half, 0) + at
        dst = np.where(swap, 0, half) + half // 2 + at + rng.integers(0, 2, n)
        d = make_descs([dict(func=0, src_space=FT_POOL, dst_space=FT_POOL, src=int(src[i]), dst=int(dst[i]), row_bytes=int(sizes[i])) for i in range(n)])
        for call in ("submit", "static"):
            lo.random_(0, 256)
            hi.random_(0, 256)
            before = torch.cat([lo, hi]).cpu().numpy()
            want = before.copy()
            for s, t, b in zip(src, dst, sizes):
                want[t:t + b] = before[s:s + b]
            if call == "submit":
                binding.wait(pool, binding.submit_transfers(pool, d, [1], 256 * KiB, 0, torch.cuda.current_stream().cuda_stream))
            elif n == 241:
                binding.submit_static(pool, d, [1], 256 * KiB, 0, torch.cuda.current_stream().cuda_stream)
            else:
                continue
            torch.cuda.synchronize()
            assert np.array_equal(torch.cat([lo, hi]).cpu().numpy(), want), call
    finally:
        binding.pool_destroy(pool)


@pytest.mark.gpu
@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("n,funcs,chunk", [(100, 8, 32 * KiB), (900, 2, 2 * KiB), (900, 1, 64 * KiB)])
def test_static_submits_of_lists_in_memory(n, funcs, chunk, far):
    """Lists that do not go along, in the library's own array: 12 and 20 bytes a piece, of fewer than 1024 pieces and of more (900 tensors in 450 places)."""
    import torch
    from paper_2411_01830_amd import binding
    print(f"case static lists: {n}, {funcs} functions, far apart: {far}", flush=True)
    rng = np.random.default_rng(n + funcs)
    sizes = rng.integers(900, 1100, n) if n == 900 else rng.integers(60 * KiB, 68 * KiB, n)
    room = -(-int(sizes.max() + 64) // 16) * 16
    half = -(-n * room // (1 << 20)) * (1 << 20)
    mem = torch.empty((4 << 30) + half if far else 2 * half, dtype=torch.uint8, device="cuda")
    lo, hi = mem[:half], mem[-half:]
    pool = binding.pool_create(lo.data_ptr(), half, 4 * KiB, 0)
    try:
        binding.pool_grow(pool, hi.data_ptr(), half)
        binding.slab_alloc(pool, half)
        binding.slab_alloc(pool, half)
        swap = np.arange(n) % 3 == 0  # these from the other side, into what is not read there
        at = np.arange(n) * room
        src, dst = np.where(swap, half, 0) + at + rng.integers(0, 16, n), np.where(swap, 0, half) + at + rng.integers(0, 16, n)
        d = make_descs([dict(func=i % funcs, src_space=FT_POOL, dst_space=FT_POOL, src=int(src[i]), dst=int(dst[i]), row_bytes=int(sizes[i])) for i in range(n)])
        stream = torch.cuda.current_stream().cuda_stream
        for call in ("static", "submit", "static"):
            lo.random_(0, 256)
            hi.random_(0, 256)
            before = torch.cat([lo, hi]).cpu().numpy()
            want = before.copy()
            for s, t, b in zip(src, dst, sizes):
                want[t:t + b] = before[s:s + b]
            if call == "static":
                binding.submit_static(pool, d, [1] * funcs, chunk, 0, stream)
            else:
                job = binding.submit_transfers(pool, d, [1] * funcs, chunk, fmt.FT_TIMING, stream)
                binding.wait(pool, job)
                st = binding.job_stats(pool, job).cls[2]
                if n == 900:
                    assert (st.tile_bytes, st.in_launch, st.workgroups == st.tickets) == (2 * KiB, 0, True)
                binding.job_release(pool, job)
            torch.cuda.synchronize()
            assert np.array_equal(torch.cat([lo, hi]).cpu().numpy(), want), call
    finally:
        torch.cuda.synchronize()
        binding.pool_destroy(pool)


@pytest.mark.gpu
@pytest.mark.parametrize("n,size", [(241, 200), (600, 150), (1500, 120)])
def test_a_list_read_in_place_is_the_one_that_was_written(n, size):
    """Thirty different lists one after the other in the same pinned buffer, each only waited for with ft_wait: none sees what an earlier one left in a cache."""
    import torch
    from paper_2411_01830_amd import binding
    print(f"case lists one after the other: {n} of {size}", flush=True)
    lists, half = 30, 16 * MiB
    mem = torch.zeros(2 * half, dtype=torch.uint8, device="cuda")
    pool = binding.pool_create(mem.data_ptr(), 2 * half, 4096, 0)
    try:
        binding.slab_alloc(pool, 2 * half)
        step = size + 37
        assert lists * n * step < half
        jobs = [binding.Transfers(make_descs([dict(func=0, src_space=FT_POOL, dst_space=FT_POOL, src=(k * n + i) * step, dst=half + (k * n + i) * step + 3,
                                                   row_bytes=size + (i + k) % 30) for i in range(n)]), [1]) for k in range(lists)]
        mask = torch.zeros(half, dtype=torch.bool)
        for k in range(lists):
            for i in range(n):
                at = (k * n + i) * step
                mask[at:at + size + (i + k) % 30] = True
        mask = mask.cuda()
        stream = torch.cuda.current_stream().cuda_stream
        for _ in range(4):
            mem[:half].random_(0, 256)
            mem[half:].zero_()
            torch.cuda.synchronize()
            for job in jobs:
                binding.wait(pool, binding.submit_transfers(pool, job, None, 2 * MiB, 0, stream))
            torch.cuda.synchronize()
            want = torch.where(mask, mem[:half], torch.zeros_like(mem[:half]))
            assert torch.equal(mem[half + 3:], want[:half - 3])
    finally:
        torch.cuda.synchronize()
        binding.pool_destroy(pool)


@pytest.mark.gpu
@pytest.mark.parametrize("shifts,pieces", [([(1, 5), (15, 3), (0, 116), (7, 123)], True), ([(1, 0), (15, 14), (0, 113), (7, 120)], True), ([(1, 0), (15, 14), (1, 16), (7, 32)], False),
                                           ([(3, 3), (0, 0), (1, 2), (5, 9)], False), ([(4, 0)], True), ([(0, 1)], True), ([(1, 0)], False)],
                         ids=["4 apart", "odd", "odd to aligned ones", "half odd", "one 4 apart", "one odd", "one odd to an aligned one"])
def test_streaming_pieces_at_odd_addresses(shifts, pieces):
    """Beyond 128 MiB jobs that are mostly misaligned in ways that are better off so go as pieces of 16 KiB, by submit and static; the first, last and inner tiles of runs."""
    import torch
    from paper_2411_01830_amd import binding
    print(f"case streaming pieces: {shifts}", flush=True)
    n = (132 * MiB) // len(shifts)
    slab = -(-(n + 256) // 4096) * 4096
    mem = torch.empty(2 * slab * len(shifts), dtype=torch.uint8, device="cuda")
    pool = binding.pool_create(mem.data_ptr(), mem.numel(), 4096, 0)
    try:
        at = [binding.slab_alloc(pool, slab) for _ in range(2 * len(shifts))]
        recs = [dict(func=i % 2, src_space=FT_POOL, dst_space=FT_POOL, src=at[2 * i] + s, dst=at[2 * i + 1] + t, row_bytes=n + i - 2)
                for i, (s, t) in enumerate(shifts)]
        d, weights = make_descs(recs), [1, 3][:len(shifts)]
        g = torch.Generator("cuda").manual_seed(3)
        stream = torch.cuda.current_stream().cuda_stream
        for call in ("submit", "static"):
            mem.random_(0, 256, generator=g)
            want = mem.clone()
            for r in recs:
                want[r["dst"]:r["dst"] + r["row_bytes"]] = mem[r["src"]:r["src"] + r["row_bytes"]]
            if call == "static":
                binding.submit_static(pool, d, weights, 1 * MiB, 0, stream)
            else:
                job = binding.submit_transfers(pool, d, weights, 1 * MiB, fmt.FT_TIMING, stream)
                binding.wait(pool, job)
                assert (binding.job_stats(pool, job).cls[2].tile_bytes == 16 * KiB) == pieces
                binding.job_release(pool, job)
            torch.cuda.synchronize()
            assert torch.equal(mem, want), call
    finally:
        torch.cuda.synchronize()
        binding.pool_destroy(pool)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [241, 300, 2730, 3000])
def test_streaming_pieces_of_lists_in_memory(n):
    """The same of more tensors than a launch holds: lists read in place, and uploaded ones of more than 2730 pieces. Sizes are odd, distances of every kind."""
    import torch
    from paper_2411_01830_amd import binding
    print(f"case streaming pieces of a list in memory: {n}", flush=True)
    total = 136 * MiB
    sizes = [total // n + (i * 7919) % 4099 - 2000 for i in range(n)]
    slab = -(-(max(sizes) + 32) // 4096) * 4096
    mem = torch.empty(2 * slab * n, dtype=torch.uint8, device="cuda")
    pool = binding.pool_create(mem.data_ptr(), mem.numel(), 4096, 0)
    try:
        src, dst = binding.slab_alloc(pool, slab * n), binding.slab_alloc(pool, slab * n)
        recs = [dict(func=i % 3, src_space=FT_POOL, dst_space=FT_POOL, src=src + i * slab + i % 16, dst=dst + i * slab + (5 * i + 3) % 16, row_bytes=b) for i, b in enumerate(sizes)]
        d = make_descs(recs)
        g = torch.Generator("cuda").manual_seed(n)
        stream = torch.cuda.current_stream().cuda_stream
        for flags in (fmt.FT_TIMING, 0):
            mem.random_(0, 256, generator=g)
            want = mem.clone()
            for r in recs:
                want[r["dst"]:r["dst"] + r["row_bytes"]] = mem[r["src"]:r["src"] + r["row_bytes"]]
            job = binding.submit_transfers(pool, d, [1, 2, 5], 2 * MiB, flags, stream)
            binding.wait(pool, job)
            if flags:
                st = binding.job_stats(pool, job).cls[2]
                assert (st.tile_bytes, st.in_launch, st.workgroups == st.tickets) == (16 * KiB, 0, True)
                binding.job_release(pool, job)
            torch.cuda.synchronize()
            assert torch.equal(mem, want), flags
    finally:
        torch.cuda.synchronize()
        binding.pool_destroy(pool)


# as above; the tiles are 1, 2 or 4 KiB, the workgroups at most 64 from the host and towards it 128, of more than 256 tiles 48
LINK_CASES = [
    ("one byte", lambda g: [(1, 1, 0, 0, 0, 3, 9)], [1], 2 * MiB, True),
    *[(f"one tensor of {n}", lambda g, n=n: [(n, 1, 0, 0, 0, 7, 4)], [1], 2 * MiB, True) for n in (15, 17, 1025, 32 * KiB, 32 * KiB + 1, 128 * KiB, 128 * KiB + 1, 3 * MiB)],
    ("one aligned tensor", lambda g: [(3 * MiB + 16, 1, 0, 0, 0, 0, 0)], [1], 2 * MiB, "to the host"),
    # (from the host as pieces where its kernel says itself when it is done, which one that is timed does not)
    ("one aligned tensor of 128 KiB", lambda g: [(128 * KiB, 1, 0, 0, 0, 0, 0)], [1], 2 * MiB, True),
    ("one aligned tensor of 128 KiB and 16", lambda g: [(128 * KiB + 16, 1, 0, 0, 0, 0, 0)], [1], 2 * MiB, "to the host"),
    ("one aligned tensor of 256 KiB", lambda g: [(256 * KiB, 1, 0, 0, 0, 0, 0)], [1], 2 * MiB, "to the host"),
    ("one aligned tensor of 256 KiB and 16", lambda g: [(256 * KiB + 16, 1, 0, 0, 0, 0, 0)], [1], 2 * MiB, "to the host"),
    *[(f"{n} tensors of one function", lambda g, n=n: _runs(g, n, [1, 15, 16, 17, 127, 4095, 4096, 4097, 9000], 1), [1], 4 * KiB, n <= 240) for n in (16, 48, 128, 129, 240, 241)],
    ("65 tiles of three functions", lambda g: [(4096, 1, 0, 0, i % 3, 0, 0) for i in range(65)], [1, 2, 5], 4 * KiB, True),
    ("129 tiles of three functions", lambda g: [(4096, 1, 0, 0, i % 3, 0, 0) for i in range(129)], [1, 2, 5], 4 * KiB, True),
    ("260 tiles of three functions", lambda g: [(4096, 1, 0, 0, i % 3, 0, 0) for i in range(260)], [1, 2, 5], 4 * KiB, False),
    ("tensors around 64 KiB", lambda g: _runs(g, 60, [60000, 65536, 70001, 100], 4), [1, 2, 5, 1], 64 * KiB, None),
    ("chunks of 1 KiB", lambda g: _runs(g, 900, [1, 15, 16, 17, 1023, 1024, 1025], 3), [1, 2, 5], 1024, False),
    ("chunks under 1 KiB", lambda g: _runs(g, 100, [300, 5000], 2), [1, 3], 512, "general"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", LINK_CASES, ids=[c[0] for c in LINK_CASES])
@pytest.mark.parametrize("to_host", [False, True])
def test_pieces_over_the_host_link(case, to_host):
    import torch
    from paper_2411_01830_amd import binding, harness
    name, pieces, weights, chunk, along = case
    print(f"case pieces over the host link: {name}, to the host: {to_host}", flush=True)
    rng = np.random.default_rng(len(name) + to_host)
    orc, eng = OracleEngine(), harness.GpuEngine()
    cls = 1 if to_host else 0
    try:
        host = 8 * MiB
        for e in (orc, eng):
            e.host_arena(host)
            e.pool_create(16 * MiB, 4 * KiB)
        data = rng.integers(0, 256, host, dtype=np.uint8)
        if not to_host:
            orc.write_host(0, data)
            eng.write_host(0, data)
        recs, at = [], 0
        for rb, rows, sp, dp, f, ss, ds in pieces(rng):
            a = orc.slab_alloc(rb + 16)
            assert eng.slab_alloc(rb + 16) == a
            if to_host:
                orc.write_pool(a, data[at:at + rb + 16])
                eng.write_pool(a, data[at:at + rb + 16])
            src, dst = (a + ss, at + ds) if to_host else (at + ss, a + ds)
            recs.append(dict(func=f, src_space=1 if to_host else 0, dst_space=0 if to_host else 1, src=src, dst=dst, row_bytes=rb))
            at += rb + 32
            assert at < host
        pool_before, host_before = torch.cat([t for t, _ in eng.segments]).clone(), eng.host_np.copy()
        d = make_descs(recs)
        jo = orc.submit(d, weights, chunk)
        orc.wait(jo)
        payload = sum(r["row_bytes"] for r in recs)
        for flags in (0, 0, fmt.FT_DETACHED, fmt.FT_TIMING, fmt.FT_TIMING):     # a counter has to be back at zero for the next launch
            jg = eng.submit(d, weights, chunk, flags | fmt.FT_VALIDATE)
            eng.wait(jg)
            if flags & fmt.FT_TIMING:
                st = binding.job_stats(eng.pool, jg).cls[cls]
                own = st.tile_bytes == (1024 if payload <= 32 * KiB else 2048 if payload <= 128 * KiB else 4096) and st.workgroups == min(st.tickets, (48 if st.tickets > 256 else 128) if to_host else 64)
                assert own == (along != "general" and (to_host or along != "to the host")), (st.tile_bytes, st.workgroups, st.tickets)
                assert along not in (True, False) or st.in_launch == (1 if along else 0)
                assert eng.job_schedule(jg, cls) == orc.job_schedule(jo, cls)
                binding.job_release(eng.pool, jg)
            assert np.array_equal(torch.cat([t for t, _ in eng.segments]).cpu().numpy(), orc.pool_mem), flags
            assert np.array_equal(eng.host_np[:len(orc.host_mem)], orc.host_mem), flags
            at = 0
            for t, _ in eng.segments:
                t.copy_(pool_before[at:at + t.numel()])
                at += t.numel()
            torch.cuda.synchronize()
            eng.host_np[:] = host_before
    finally:
        eng.close()


def test_inline_assembly_stores_of_the_piece_kernels_leave_no_hazard(tmp_path):
    """As for the other kernels: two wait states behind each store that is written through, its address in vector registers."""
    import os
    import re
    import subprocess
    from paper_2411_01830_amd import build
    out = tmp_path / "pieces.s"
    subprocess.run([build.hipcc(), "-x", "hip", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ft_pieces.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    lines = [re.sub(r"\s+", " ", l.split("//")[0]).strip() for l in open(out)]
    stores = [i for i, l in enumerate(lines) if l.startswith("global_store_dwordx4") and l.endswith(" sc1")]
    kernels = [l for l in lines if re.match(r"_ZN2ft20ft_link_piece_kernelILi2E\S*:", l)]
    assert len(kernels) >= 6 and len(stores) >= 4 * len(kernels)
    for i in stores:
        assert re.fullmatch(r"global_store_dwordx4 v\[\d+:\d+\], [va]\[\d+:\d+\], off (sc0 )?sc1", lines[i]), lines[i]
        assert lines[i + 1] == "s_nop 1", lines[i:i + 2]


def test_kernels_that_say_they_are_done_have_waited_for_their_stores(tmp_path):
    """In front of each word to the host a wait for every store, and nothing stored between the two. What is stored before it is of system scope, as the
    word is, or written back at that scope in front of the wait."""
    import os
    import re
    import subprocess
    from paper_2411_01830_amd import build
    out = tmp_path / "pieces.s"
    subprocess.run([build.hipcc(), "-x", "hip", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ft_pieces.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    lines = [re.sub(r"\s+", " ", l.split("//")[0]).strip() for l in open(out)]
    said = [i for i, l in enumerate(lines) if l.startswith("global_store_dwordx2") and l.endswith(" sc0 sc1")]
    kernels = [l for l in lines if re.match(r"_ZN2ft(15ft_piece_kernelILi4E|20ft_link_piece_kernel)\S*:", l)]
    assert len(said) == len(kernels) >= 20
    for l in lines:
        if re.match(r"_ZN2ft15ft_piece_kernel\S*:", l):
            assert ("DoneWords" in l) == ("ft_piece_kernelILi4E" in l), l
            # a launch with words has at most 640 tiles, so no more pieces, and lists of up to 1024 have a kernel of their own
            assert not re.search(r"ILi4E\S*PieceRefsILj(64|256)E", l), l
    for i in said:
        j = max(k for k in range(i) if lines[k] == "s_waitcnt vmcnt(0)" and lines[k - 1] == ";;#ASMSTART")
        assert not [l for l in lines[j:i] if re.match(r"(global|flat|buffer|scratch)_(store|atomic)", l)], lines[j:i + 1]
        begin = max(k for k in range(i) if lines[k].startswith("_ZN2ft"))
        stores = [k for k in range(begin, j) if re.match(r"(global|flat|buffer|scratch)_store", lines[k])]
        assert stores
        if "ft_piece_kernelILi4E" in lines[begin]:
            assert all(lines[k].endswith(" sc0 sc1") for k in stores), [lines[k] for k in stores]
        else:
            assert max(k for k in range(j) if lines[k] == "buffer_wbl2 sc0 sc1") > max(stores)


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["pool_to_pool", "host_to_pool", "pool_to_host"])
@pytest.mark.parametrize("sizes", [[5], [16], [64 * KiB + 3], [640 * 2 * KiB - 128], [640 * 2 * KiB + 1], [31, 700, 5000] * 25, [2 * KiB] * 70],
                         ids=["5", "16", "64K", "640 tiles", "641 tiles", "75 small", "70 jobs"])
def test_what_has_been_waited_for_is_there(where, sizes):
    """After ft_wait, with nothing else waited for, the bytes are read by the host, or first of all by a kernel on another stream, or by a copy to the host on it."""
    import torch
    from paper_2411_01830_amd import binding
    print(f"case waited for: {where} {len(sizes)} of {sizes[0]}", flush=True)
    g = torch.Generator("cuda").manual_seed(len(sizes))
    room = -(-(sum(sizes) + 64 * len(sizes)) // 4096) * 4096
    mem = torch.zeros(2 * room, dtype=torch.uint8, device="cuda")
    host = torch.zeros(room, dtype=torch.uint8, pin_memory=True)
    pool = binding.pool_create(mem.data_ptr(), 2 * room, 4 * KiB, 0)
    jobs, other = torch.cuda.Stream(), torch.cuda.Stream()
    try:
        binding.slab_alloc(pool, 2 * room)
        binding.host_window_add(pool, host.data_ptr(), room)
        starts = np.concatenate([[0], np.cumsum([n + 48 for n in sizes])[:-1]])
        src0, dst0 = (host.data_ptr() if where == "host_to_pool" else 0), (host.data_ptr() if where == "pool_to_host" else room)
        recs = [dict(func=0, src_space=0 if where == "host_to_pool" else 1, dst_space=0 if where == "pool_to_host" else 1, src=src0 + int(a) + 1,
                     dst=dst0 + int(a) + 1, row_bytes=n) for a, n in zip(starts, sizes)]
        lists = [[r] for r in recs] if len(recs) == 70 else [recs]
        lists = [binding.Transfers(make_descs(l), [1]) for l in lists]
        mask = torch.zeros(room, dtype=torch.bool, device="cuda")
        for a, n in zip(starts, sizes):
            mask[int(a) + 1:int(a) + 1 + n] = True
        seen, copied = torch.zeros(room, dtype=torch.uint8, device="cuda"), torch.zeros(room, dtype=torch.uint8, pin_memory=True)
        for k in range(16):
            data = torch.randint(0, 256, (room,), dtype=torch.uint8, device="cuda", generator=g)
            want = torch.where(mask, data, torch.zeros_like(data))
            (host if where == "host_to_pool" else mem[:room]).copy_(data)
            (host if where == "pool_to_host" else mem[room:]).zero_()
            wanted = want.cpu()
            torch.cuda.synchronize()
            handles = [binding.submit_transfers(pool, l, None, 2 * MiB, 0, jobs.cuda_stream) for l in lists]
            for h in handles:
                binding.wait(pool, h)
            if where == "pool_to_host":
                got = host.clone()
            elif k % 2 == 0:
                with torch.cuda.stream(other):
                    torch.bitwise_or(mem[room:], 0, out=seen)
                other.synchronize()
                got = seen.cpu()
            else:
                with torch.cuda.stream(other):
                    copied.copy_(mem[room:], non_blocking=True)
                other.synchronize()
                got = copied
            assert torch.equal(got, wanted)
            torch.cuda.synchronize()
    finally:
        torch.cuda.synchronize()
        binding.pool_destroy(pool)
