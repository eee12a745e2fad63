"""The kernel that gives every wavefront tiles of its own: pool->pool jobs of at most 16, 48 or 128 MiB and jobs of
pitched rows, host-link jobs of small pieces, at the sizes where its windows, its tiles and the rule that picks it change;
each case says by tile size and workgroups which kernel it got. Bit-exact against the oracle or plain strided copies."""
import os

import numpy as np
import pytest

from oracle import OracleEngine
from workloads import make_descs, FT_HOST, FT_POOL
from workloads import format as fmt
from test_host_logic import _host_sanitizer_run

KiB, MiB = 1 << 10, 1 << 20


def test_windows_and_decode_on_the_host(tmp_path):
    """tests/host/wave_tiles.cpp: the kernel's window arithmetic covers every piece and stays inside it; a ticket
    decoded by comparing 64 entries at a time names what the general walk names."""
    _host_sanitizer_run(tmp_path, "wave_tiles", ["ft_plan.cpp", "ft_pool.cpp"], ["1", "60"], "done 1..60")


def test_inline_assembly_stores_leave_no_hazard_to_the_scheduler(tmp_path):
    """The stores that are written through to the host are inline assembly, for which the compiler inserts no wait states: each
    has its two before its data may be overwritten, and none takes its address from a scalar register, which a vector
    instruction may have written within the five before."""
    import re
    import subprocess
    from paper_2411_01830_amd import build
    out = tmp_path / "kernels.s"
    subprocess.run([build.hipcc(), "-x", "hip", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ft_kernels.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    lines = [re.sub(r"\s+", " ", l.split("//")[0]).strip() for l in open(out)]
    stores = [i for i, l in enumerate(lines) if l.startswith("global_store_dwordx4") and l.endswith(" sc1")]
    assert len(stores) > 100
    for i in stores:
        assert re.fullmatch(r"global_store_dwordx4 v\[\d+:\d+\], [va]\[\d+:\d+\], off sc1", lines[i]), lines[i]
        assert lines[i + 1] == "s_nop 1", lines[i:i + 2]


def _runs(rng, n, sizes, funcs):
    """Contiguous pieces: (row_bytes, rows, src pitch, dst pitch, function, src shift, dst shift)."""
    return [(int(rng.choice(sizes)), 1, 0, 0, i % funcs, int(rng.integers(0, 16)), int(rng.integers(0, 16))) for i in range(n)]


def _rows(rng, n, widths, total, funcs):
    out = []
    for i in range(n):
        rb = int(rng.choice(widths))
        out.append((rb, max(2, total // n // rb), rb + int(rng.integers(0, 50)), rb + int(rng.integers(0, 3)) * 7, i % funcs,
                    int(rng.integers(0, 16)), int(rng.integers(0, 16))))
    return out


def _tile(chunk, want):
    """Bytes per tile when a chunk is cut into tiles of about `want` bytes."""
    n = -(-chunk // want)
    return (-(-chunk // n) + 15) // 16 * 16


def _wave_tile(payload, chunk):
    """The tile of a pool->pool launch of the wave kernel: about 4000 tiles of 2 .. 8 KiB."""
    t = payload // 4000
    return _tile(chunk, 2048 if t < 2048 else 8192 if t > 8192 else (t + 15) // 16 * 16)


# name, pieces(rng), weights, chunk, flags, kernel and workgroups of the pool->pool launch: the wave kernel with a workgroup per ticket or
# one or two per compute unit, or the copy kernel. Its tiles of 43 or 64 KiB tell the kernels apart where the chunk lets them,
# and where it does not its at most one workgroup per compute unit does.
CASES = [
    ("bytes around a window", lambda g: _runs(g, 200, [1, 15, 16, 17, 31, 32, 33, 1023, 1024, 1025], 3), [1, 2, 5], 4096, 0, "tickets"),
    ("bytes around a window, chunks of 1 KiB", lambda g: _runs(g, 900, [1, 15, 16, 17, 1023, 1024, 1025], 3), [1, 2, 5], 1024, 0, "tickets"),
    ("one tile and its edges", lambda g: _runs(g, 40, [2047, 2048, 2049, 8191, 8192, 8193, 8208], 2), [1, 1], 64 * KiB, 0, "tickets"),
    ("5000 descriptors of one function", lambda g: _runs(g, 5000, [1, 60, 300, 700], 1), [1], 256 * KiB, 0, "tickets"),
    ("256 functions", lambda g: _runs(g, 600, [64, 5000, 9000], 256), list(range(1, 257)), 4 * KiB, 0, "tickets"),
    ("1024 functions", lambda g: _runs(g, 2100, [64, 5000, 9000], 1024), [1 + f % 5 for f in range(1024)], 4 * KiB, 0, "tickets"),
    ("1025 functions", lambda g: _runs(g, 2100, [64, 5000, 9000], 1025), [1] * 1025, 4 * KiB, 0, None),
    ("chunks under 1 KiB", lambda g: _runs(g, 200, [300, 5000], 2), [1, 3], 512, 0, None),
    ("logged", lambda g: _runs(g, 60, [40, 3000, 70000], 4), [1, 2, 3, 4], 64 * KiB, fmt.FT_LOG, "tickets"),
    ("detached", lambda g: _runs(g, 60, [40, 3000, 70000], 4), [1, 2, 3, 4], 64 * KiB, fmt.FT_DETACHED, "tickets"),
    ("over 16 MiB", lambda g: _runs(g, 30, [600 * KiB, 700 * KiB + 5], 3), [1, 2, 4], 256 * KiB, 0, "one a unit"),
    ("rows of 16 bytes and a bit", lambda g: _rows(g, 20, [16, 17, 31, 32, 33], 2 * MiB, 2), [1, 2], 100000 // 16 * 16, 0, "tickets"),
    ("rows under 16 bytes", lambda g: _rows(g, 20, [1, 2, 3, 4, 5, 7, 8, 12, 15], 400 * KiB, 2), [1, 2], 64 * KiB, 0, None),
    ("rows longer than a tile", lambda g: _rows(g, 6, [8193, 20000, 66000], 4 * MiB, 2), [3, 1], 1 * MiB, 0, "tickets"),
    ("short rows over 16 MiB", lambda g: _rows(g, 24, [20, 100, 2000], 18 * MiB, 2), [3, 1], 256 * KiB, 0, "two a unit"),
    ("long rows over 16 MiB", lambda g: _rows(g, 12, [2100, 5760, 30001], 18 * MiB, 2), [3, 1], 256 * KiB, 0, "one a unit"),
    ("rows between 1 MiB pitches", lambda g: [(100, 9, 1 << 20, 200, 0, 3, 5), (70, 5, 100, 1 << 20, 1, 1, 2), (50, 6, (1 << 20) + 1, 60, 0, 0, 0)],
     [1, 1], 64 * KiB, 0, "tickets"),
    ("rows as far apart as a tile's 32 bits allow", lambda g: [(16, 3, ((1 << 32) - 1) // 516, 30, 0, 3, 5), (70, 5, 100, 1 << 20, 1, 1, 2)],
     [1, 1], 64 * KiB, 0, "tickets"),
    ("rows further apart", lambda g: [(16, 3, ((1 << 32) - 1) // 516 + 1, 30, 0, 3, 5), (70, 5, 100, 1 << 20, 1, 1, 2)],
     [1, 1], 64 * KiB, 0, None),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("beside_host_link", [False, True])
def test_wave_tiles_match_the_oracle(case, beside_host_link):
    import torch
    from paper_2411_01830_amd import binding, harness
    name, pieces, weights, chunk, flags, shape = case
    print(f"case wave tiles: {name}, host link beside: {beside_host_link}", flush=True)
    rng = np.random.default_rng(len(name) + beside_host_link)
    orc, eng = OracleEngine(), harness.GpuEngine()
    try:
        for e in (orc, eng):
            e.host_arena(1 << 20)
            e.pool_create(128 * MiB, 4 * KiB)
        data = rng.integers(0, 256, 1 << 19, dtype=np.uint8)
        orc.write_host(0, data)
        eng.write_host(0, data)
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
        if beside_host_link:
            b = orc.slab_alloc(200000)
            assert eng.slab_alloc(200000) == b
            recs.append(dict(func=0, src_space=FT_HOST, dst_space=FT_POOL, src=77, dst=b + 3, row_bytes=190001))
        d = make_descs(recs)
        jo = orc.submit(d, weights, chunk)
        orc.wait(jo)
        for _ in range(2):
            jg = eng.submit(d, weights, chunk, flags | fmt.FT_KEEP | fmt.FT_VALIDATE)
            eng.wait(jg)
            assert eng.job_schedule(jg, 2) == orc.job_schedule(jo, 2)
            st = binding.job_stats(eng.pool, jg).cls[2]
            cus = torch.cuda.get_device_properties(0).multi_processor_count
            own = [r for r in recs if r["src_space"] == FT_POOL]
            in_rows = sum(r["row_bytes"] * r["rows"] for r in own if r["rows"] > 1)
            if shape is None or (beside_host_link and st.payload_bytes > 16 * MiB and 2 * in_rows <= st.payload_bytes):
                short = sum(r["row_bytes"] * r["rows"] for r in own if r["rows"] > 1 and r["row_bytes"] <= 2048)
                want = _tile(chunk, 43 * KiB if 2 * short > st.payload_bytes else 64 * KiB), min(cus, st.tickets)
                assert want[0] != _wave_tile(st.payload_bytes, chunk) or cus < st.tickets     # the wave kernel would be seen
            else:
                units = 2 if beside_host_link or shape == "two a unit" else 1
                want = _wave_tile(st.payload_bytes, chunk), st.tickets if shape == "tickets" else units * cus
                assert want[0] != _tile(chunk, 64 * KiB) or cus < want[1]                     # and so would the copy kernel
            assert (st.tile_bytes, st.workgroups) == want, st.tickets
            if flags & fmt.FT_LOG:
                log = binding.job_log(eng.pool, jg, 2)
                assert int(log["bytes"].sum()) == st.payload_bytes and len(log["bytes"]) == st.tickets
            binding.job_release(eng.pool, jg)
        assert np.array_equal(torch.cat([t for t, _ in eng.segments]).cpu().numpy(), orc.pool_mem)
    finally:
        eng.close()


# name, pieces(rng), chunk, flags, the wave kernel with a workgroup per ticket (True), with 64 workgroups (False), or the class's
# own kernel (None); tiles of 1 and 4 KiB against its 8 and 16 KiB tell them apart
LINK_CASES = [
    ("bytes around a window", lambda g: _runs(g, 150, [1, 15, 16, 17, 31, 32, 33, 1023, 1024, 1025], 3), 4096, 0, True),
    ("one tensor", lambda g: _runs(g, 1, [65536 + 5], 1), 64 * KiB, 0, True),
    ("128 KiB and a byte of long pieces", lambda g: _runs(g, 2, [64 * KiB + 1], 2), 64 * KiB, 0, None),
    ("small pieces under 1 MiB", lambda g: _runs(g, 240, [3000, 4095, 4096], 3), 256 * KiB, fmt.FT_LOG, True),
    ("small pieces over 1 MiB", lambda g: _runs(g, 300, [3000, 4095, 4096, 4097], 3), 256 * KiB, 0, False),
    ("small pieces over 1 MiB, detached", lambda g: _runs(g, 300, [3000, 4095], 3), 256 * KiB, fmt.FT_DETACHED, False),
    ("rows apart on both sides", lambda g: _rows(g, 12, [16, 33, 100, 500, 2048], 1 * MiB, 2), 100000 // 16 * 16, 0, "rows"),
    ("narrow gathered rows", lambda g: [(w, 700, w + 40, w, i % 2, 3 * i % 16, 5 * i % 16) for i, w in enumerate([16, 17, 40, 63, 64])], 64 * KiB, 0, True),
    ("rows under 16 bytes", lambda g: _rows(g, 6, [1, 3, 9, 15], 40 * KiB, 2), 64 * KiB, 0, None),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", LINK_CASES, ids=[c[0] for c in LINK_CASES])
@pytest.mark.parametrize("to_host", [False, True])
def test_wave_tiles_on_the_host_link(case, to_host):
    """The same over the host link, each direction; what lies around every destination stays as it was."""
    import torch
    from paper_2411_01830_amd import binding, harness
    name, pieces, chunk, flags, tickets = case
    print(f"case wave tiles over the host link: {name}, to the host: {to_host}", flush=True)
    rng = np.random.default_rng(len(name) + to_host)
    orc, eng = OracleEngine(), harness.GpuEngine()
    cls = 1 if to_host else 0
    try:
        host = 8 * MiB
        for e in (orc, eng):
            e.host_arena(host)
            e.pool_create(32 * MiB, 4 * KiB)
        if not to_host:
            data = rng.integers(0, 256, host, dtype=np.uint8)
            orc.write_host(0, data)
            eng.write_host(0, data)
        recs, at = [], 0
        for rb, rows, sp, dp, f, ss, ds in pieces(rng):
            es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
            in_pool, on_host = (es, ed) if to_host else (ed, es)
            a = orc.slab_alloc(in_pool + 16)
            assert eng.slab_alloc(in_pool + 16) == a
            if to_host:
                fill = rng.integers(0, 256, in_pool + 16, dtype=np.uint8)
                orc.write_pool(a, fill)
                eng.write_pool(a, fill)
            src, dst = (a + ss, at + ds) if to_host else (at + ss, a + ds)
            recs.append(dict(func=f, src_space=FT_POOL if to_host else FT_HOST, dst_space=FT_HOST if to_host else FT_POOL, src=src,
                             dst=dst, row_bytes=rb, rows=rows, src_pitch=sp if rows > 1 else rb, dst_pitch=dp if rows > 1 else rb))
            at += on_host + 32
            assert at < host
        d = make_descs(recs)
        w = [2, 1, 5][:max(r["func"] for r in recs) + 1]
        jo = orc.submit(d, w, chunk)
        orc.wait(jo)
        for _ in range(2):
            jg = eng.submit(d, w, chunk, flags | fmt.FT_KEEP | fmt.FT_VALIDATE)
            eng.wait(jg)
            assert eng.job_schedule(jg, cls) == orc.job_schedule(jo, cls)
            st = binding.job_stats(eng.pool, jg).cls[cls]
            if tickets is None:
                own = 8 * KiB if to_host and st.payload_bytes <= 256 * KiB else 16 * KiB
                assert st.tile_bytes == _tile(chunk, own)
            else:
                each = tickets is True or (tickets == "rows" and st.payload_bytes <= 1 * MiB)
                assert st.tile_bytes == _tile(chunk, 1024 if st.payload_bytes <= 128 * KiB else 4096)
                assert st.workgroups == (st.tickets if each else min(64, st.tickets))
            if flags & fmt.FT_DETACHED:
                assert st.in_launch == 0     # it would hold the caller's stream
            if flags & fmt.FT_LOG:
                log = binding.job_log(eng.pool, jg, cls)
                assert int(log["bytes"].sum()) == st.payload_bytes and len(log["bytes"]) == st.tickets
            binding.job_release(eng.pool, jg)
        assert np.array_equal(torch.cat([t for t, _ in eng.segments]).cpu().numpy(), orc.pool_mem)
        assert np.array_equal(eng.host_np[:len(orc.host_mem)], orc.host_mem)
    finally:
        eng.close()


@pytest.mark.gpu
def test_static_submits_with_and_without_the_device_array():
    """ft_submit_static back to back: a job whose tables travel with its launch, one that goes through the library's
    device array, one tensor, and the first shape again, all on one stream with nothing in between."""
    import torch
    from paper_2411_01830_amd import harness
    print("case static submits with and without the device array", flush=True)
    rng = np.random.default_rng(5)
    orc, eng = OracleEngine(), harness.GpuEngine()
    try:
        for e in (orc, eng):
            e.host_arena(1 << 20)
            e.pool_create(96 * MiB, 4 * KiB)
        jobs = []
        for pieces, w in ((_runs(rng, 12, [5000, 70001], 3), [1, 2, 3]), (_runs(rng, 120, [100, 9000], 4), [4, 3, 2, 1]),
                          (_runs(rng, 1, [300001], 1), [1]), (_rows(rng, 10, [100, 4000], 1 * MiB, 2), [1, 5])):
            recs = []
            for rb, rows, sp, dp, f, ss, ds in pieces:
                es, ed = (rows - 1) * sp + rb, (rows - 1) * dp + rb
                a, b = orc.slab_alloc(es + 16), orc.slab_alloc(ed + 16)
                assert eng.slab_alloc(es + 16) == a and eng.slab_alloc(ed + 16) == b
                fill = rng.integers(0, 256, es + 16, dtype=np.uint8)
                orc.write_pool(a, fill)
                eng.write_pool(a, fill)
                recs.append(dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a + ss, dst=b + ds, row_bytes=rb, rows=rows,
                                 src_pitch=sp if rows > 1 else rb, dst_pitch=dp if rows > 1 else rb))
            jobs.append((make_descs(recs), w))
        torch.cuda.synchronize()
        for d, w in jobs:
            orc.wait(orc.submit(d, w, 64 * KiB))
            eng.submit_static(d, w, 64 * KiB, fmt.FT_VALIDATE)
        torch.cuda.synchronize()
        assert np.array_equal(torch.cat([t for t, _ in eng.segments]).cpu().numpy(), orc.pool_mem)
    finally:
        eng.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, fmt.FT_LOG])
def test_tiles_in_which_one_tensor_ends_and_the_next_begins(flags):
    """The copy kernel proper (asked for by its tile size) moves a full tile of two aligned tensors in one pass: lengths
    around a tile and around a vector, three tensors in a tile, a second one that is misaligned or pitched."""
    import torch
    from paper_2411_01830_amd import binding, harness
    print(f"case two tensors in a tile, flags {flags}", flush=True)
    rng = np.random.default_rng(9)
    orc, eng = OracleEngine(), harness.GpuEngine()
    try:
        for e in (orc, eng):
            e.host_arena(1 << 20)
            e.pool_create(160 * MiB, 4 * KiB)
        binding.set_tuning(eng.pool, 2, 0, 64 * KiB)
        sizes = [65536, 65520, 65552, 131072, 40000, 16, 32, 65536 - 32, 90000, 131056, 48, 65504, 77, 65536, 4096]
        recs = []
        for f in range(3):
            for i in range(60):
                n, rows = int(rng.choice(sizes)), 1
                shift = (0, 0)
                if f == 1 and i % 7 == 3:
                    shift = (int(rng.integers(0, 16)), int(rng.integers(0, 16)))
                if f == 2 and i % 5 == 2:
                    n, rows = 400, 30
                pitch = n + 48
                a, b = orc.slab_alloc(pitch * rows + 16), orc.slab_alloc(pitch * rows + 16)
                assert eng.slab_alloc(pitch * rows + 16) == a and eng.slab_alloc(pitch * rows + 16) == b
                fill = rng.integers(0, 256, pitch * rows + 16, dtype=np.uint8)
                orc.write_pool(a, fill)
                eng.write_pool(a, fill)
                recs.append(dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a + shift[0], dst=b + shift[1], row_bytes=n,
                                 rows=rows, src_pitch=pitch if rows > 1 else n, dst_pitch=pitch if rows > 1 else n))
        d = make_descs(recs)
        for chunk in (64 * KiB, 2 * MiB):
            jo = orc.submit(d, [1, 2, 3], chunk)
            orc.wait(jo)
            jg = eng.submit(d, [1, 2, 3], chunk, flags | fmt.FT_KEEP | fmt.FT_VALIDATE)
            eng.wait(jg)
            assert binding.job_stats(eng.pool, jg).cls[2].tile_bytes == 64 * KiB
            assert eng.job_schedule(jg, 2) == orc.job_schedule(jo, 2)
            binding.job_release(eng.pool, jg)
            assert np.array_equal(torch.cat([t for t, _ in eng.segments]).cpu().numpy(), orc.pool_mem)
    finally:
        eng.close()


def test_batches_of_tickets_on_the_host(tmp_path):
    """tests/host/ticket_batches.cpp: the protocol by which a workgroup's wavefronts share out the tickets behind the first
    round, run by threads: each ticket once, every wavefront ends, also beside one that is arbitrarily slow."""
    _host_sanitizer_run(tmp_path, "ticket_batches", [], ["1", "600"], "done 1..600")


def _move_with_torch(mem, host, rec):
    """One descriptor by plain strided torch copies; mem: the pool's bytes, host: pinned bytes."""
    view = lambda space, at, pitch: (mem if space == FT_POOL else host).as_strided((rec["rows"], rec["row_bytes"]), (pitch, 1), at)
    view(rec["dst_space"], rec["dst"], rec["dst_pitch"]).copy_(view(rec["src_space"], rec["src"], rec["src_pitch"]))


# name, link class, (row bytes, payload MiB) of a slow and of a fast function, chunk = tile, descriptors of each, flags
ORDER_CASES = [
    ("pool, short rows", 2, (16, 2000), 50, 8192, 4, 0),
    ("pool, short rows, uploaded tables", 2, (16, 2000), 50, 8192, 40, 0),
    ("pool, short rows, beyond the cache", 2, (16, 2000), 100, 8192, 4, 0),
    ("pool, long rows", 2, (2049, 60000), 50, 8192, 4, 0),
    ("pool, long rows, detached", 2, (2049, 60000), 50, 8192, 4, fmt.FT_DETACHED),
    ("host to pool", 0, (16, 2000), 8, 4096, 4, 0),
    ("pool to host", 1, (16, 2000), 8, 4096, 4, 0),
    ("pool to host, uploaded tables", 1, (16, 2000), 8, 4096, 40, 0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", ORDER_CASES, ids=[c[0] for c in ORDER_CASES])
def test_the_weighted_order_holds_whatever_the_tiles_cost(case):
    """Tickets drawn from the counter (kept jobs; others of that size may go as lists of pieces, whose order over the dies
    tests/host/piece_tables.cpp checks). Two functions of equal weight whose tiles alternate, one of them of slow tiles: when half of the tickets have been
    begun, half of those are the slow function's. A workgroup has at most the rest of one batch to begin, of which one
    function has at most one ticket more than the other: |A - B| <= workgroups, so the share is off by at most
    workgroups / tickets (and one per cent for tickets taken but not yet logged). Bytes against plain strided copies."""
    import torch
    from paper_2411_01830_amd import binding, harness
    name, cls, widths, mib, chunk, nd, flags = case
    print(f"case weighted order: {name}", flush=True)
    eng = harness.GpuEngine()
    try:
        eng.host_arena(64 * MiB)
        eng.pool_create(640 * MiB if mib == 50 else 1200 * MiB if mib == 100 else 64 * MiB, 4 * KiB)
        mem = eng.segments[0][0]
        mem.random_(0, 256, generator=torch.Generator("cuda").manual_seed(7))
        eng.host.random_(0, 256, generator=torch.Generator().manual_seed(8))
        recs, at = [], 32
        for f, rb in enumerate(widths):
            rows, pitch = mib * MiB // rb // nd, rb + 16 + f
            for _ in range(nd):
                extent = rows * pitch + 64
                a = eng.slab_alloc(extent) if cls != 0 else at
                b = eng.slab_alloc(extent) if cls != 1 else at
                at += extent if cls != 2 else 0
                recs.append(dict(func=f, src_space=FT_HOST if cls == 0 else FT_POOL, dst_space=FT_HOST if cls == 1 else FT_POOL, src=a + 1,
                                 dst=b + 2, row_bytes=rb, rows=rows, src_pitch=pitch, dst_pitch=pitch))
        assert at < 64 * MiB
        want_mem, want_host = mem.clone(), eng.host.clone()
        for r in recs:
            _move_with_torch(want_mem, want_host, r)
        torch.cuda.synchronize()
        shares = []
        for i in range(3):     # the counter has to be back at zero for the next launch
            if i == 2:
                flags |= fmt.FT_LOG
            jg = eng.submit(make_descs(recs), [1, 1], chunk, flags | fmt.FT_KEEP)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg).cls[cls]
            assert st.tile_bytes == chunk and st.workgroups * 8 < st.tickets
            if flags & fmt.FT_LOG:
                log = binding.job_log(eng.pool, jg, cls)
                assert int(log["bytes"].sum()) == st.payload_bytes
                first = np.argsort(log["t_begin_ns"], kind="stable")[:st.tickets // 2]
                shares.append(float((log["func"][first] == 0).mean()))
                assert abs(shares[-1] - 0.5) <= st.workgroups / st.tickets + 0.01, (shares, st.workgroups, st.tickets)
            binding.job_release(eng.pool, jg)
            assert torch.equal(mem, want_mem) and torch.equal(eng.host, want_host), i
        print(f"share of the slow function {shares}", flush=True)
    finally:
        eng.close()


# name, pieces(rng), beside the host link, chunk, workgroups per compute unit, tile
LARGE_CASES = [
    ("tensors over 16 MiB", lambda g: _runs(g, 50, [600 * KiB, 700 * KiB + 5], 3), False, 256 * KiB, 1, "wave"),
    ("one aligned tensor", lambda g: [(100 * MiB + 16, 1, 0, 0, 0, 0, 0)], False, 2 * MiB, 1, 8192),
    ("misaligned tensors over 48 MiB", lambda g: [(3 * MiB + i, 1, 0, 0, i % 3, i % 16, (i + 5) % 16) for i in range(20)], False, 2 * MiB, 1, 8192),
    ("aligned tensors over 48 MiB", lambda g: [(3 * MiB + 16 * i, 1, 0, 0, i % 3, 0, 0) for i in range(20)], False, 2 * MiB, 1, 64 * KiB),
    ("aligned tensors over 48 MiB, detached", lambda g: [(3 * MiB + 16 * i, 1, 0, 0, i % 3, 0, 0) for i in range(20)], False, 2 * MiB, 1, 64 * KiB),
    ("one aligned tensor beyond the cache", lambda g: [(150 * MiB + 16, 1, 0, 0, 0, 0, 0)], False, 2 * MiB, 1, 64 * KiB),
    ("short rows beyond the cache", lambda g: _rows(g, 24, [20, 100, 2000], 140 * MiB, 3), False, 256 * KiB, 2, 8192),
    ("long rows beyond the cache", lambda g: _rows(g, 12, [2100, 5761, 30001, 65535], 140 * MiB, 3), False, 1 * MiB, 1, 8192),
    ("rows of 64 KiB beyond the cache", lambda g: _rows(g, 12, [65536, 70001], 140 * MiB, 3), False, 1 * MiB, 1, 64 * KiB),
    ("misaligned tensors over 48 MiB beside the host link", lambda g: [(3 * MiB + i, 1, 0, 0, i % 3, i % 16, (i + 5) % 16) for i in range(20)], True, 2 * MiB, 1, 64 * KiB),
    ("rows beside the host link", lambda g: _rows(g, 12, [300, 5761, 30000], 40 * MiB, 3), True, 256 * KiB, 2, 8192),
    ("rows beyond the cache beside the host link", lambda g: _rows(g, 12, [300, 5761, 30000], 150 * MiB, 3), True, 1 * MiB, 1, 8192),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", LARGE_CASES, ids=[c[0] for c in LARGE_CASES])
def test_large_jobs_against_plain_copies(case):
    """Jobs of tens to hundreds of MiB, the whole pool compared with what plain strided copies make of it; the tile names the
    kernel that ran (the copy kernel proper has 43 and 64 KiB), the workgroups its form."""
    import torch
    from paper_2411_01830_amd import binding, harness
    name, pieces, beside, chunk, per_unit, tile = case
    print(f"case large job: {name}", flush=True)
    rng = np.random.default_rng(len(name))
    eng = harness.GpuEngine()
    try:
        eng.host_arena(8 * MiB)
        pcs = pieces(rng)
        eng.pool_create(sum(2 * ((rows * max(sp, dp, rb) + 16) // KiB // 4 + 2) * 4 * KiB for rb, rows, sp, dp, *_ in pcs) + 8 * MiB, 4 * KiB)
        mem = eng.segments[0][0]
        mem.random_(0, 256, generator=torch.Generator("cuda").manual_seed(3))
        eng.host.random_(0, 256, generator=torch.Generator().manual_seed(4))
        recs = []
        for rb, rows, sp, dp, f, ss, ds in pcs:
            sp, dp = (sp, dp) if rows > 1 else (rb, rb)
            a, b = eng.slab_alloc((rows - 1) * sp + rb + 16), eng.slab_alloc((rows - 1) * dp + rb + 16)
            recs.append(dict(func=f, src_space=FT_POOL, dst_space=FT_POOL, src=a + ss, dst=b + ds, row_bytes=rb, rows=rows, src_pitch=sp, dst_pitch=dp))
        if beside:
            b = eng.slab_alloc(4 * MiB)
            recs.append(dict(func=0, src_space=FT_HOST, dst_space=FT_POOL, src=5, dst=b + 3, row_bytes=4 * MiB - 77, rows=1, src_pitch=4 * MiB - 77, dst_pitch=4 * MiB - 77))
        want = mem.clone()
        for r in recs:
            _move_with_torch(want, eng.host, r)
        torch.cuda.synchronize()
        weights = [1 + f for f in range(1 + max(r["func"] for r in recs))]
        flags = fmt.FT_KEEP | (fmt.FT_DETACHED if "detached" in name else 0)
        for _ in range(2):
            jg = eng.submit(make_descs(recs), weights, chunk, flags)
            eng.wait(jg)
            st = binding.job_stats(eng.pool, jg).cls[2]
            tile = _wave_tile(st.payload_bytes, chunk) if tile == "wave" else tile
            assert (st.tile_bytes, st.workgroups) == (tile, per_unit * torch.cuda.get_device_properties(0).multi_processor_count)
            binding.job_release(eng.pool, jg)
            assert torch.equal(mem, want)
    finally:
        eng.close()
