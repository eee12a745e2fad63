"""The work that a user of the transfer engine has it do, case by case.

Every case goes through the Python binding of the C ABI: descriptors and weights are marshalled once
(`binding.Transfers`), the pool, the pinned windows and the allocations exist before the pass, as in a
serving process, and a pass submits, waits (where the entry point has a job to wait for) and hands back the
whole destination memory, gaps and canaries included. A pass only moves bytes, so outputs are equal or wrong.

Kinds of case:
  one     jobs of one contiguous tensor each, submitted one behind the other and waited for at the end
  batch   one job of many contiguous tensors of several weighted functions
  inout   such a job host->pool and the same tensors back pool->host
  rows    one job of pitched descriptors: windows cut out of larger row-major images
  wave    one job with host->pool and pool->pool traffic side by side
  ring    an open job whose host side is ordinary (pageable) memory: the circular pinned buffer
"""
import random

import torch

from paper_2411_01830_amd import binding as ft
from workloads import make_descs

HOST, POOL, PAGEABLE = 0, 1, 2
FT_OPEN = 1 << 6
KiB, MiB = 1 << 10, 1 << 20
CANARY = 0xA5
#: where -> (space of the source, space of the destination)
SPACES = {"pool_to_pool": (POOL, POOL), "host_to_pool": (HOST, POOL), "pool_to_host": (POOL, HOST),
          "pageable_to_pool": (PAGEABLE, POOL), "pool_to_pageable": (POOL, PAGEABLE)}
LARGEST = 1 << 30  # payload of the largest pool->pool case; the largest over the host link is `contended`


def listed():
    return [
        # the smallest call: one function hands one small tensor to the next
        {"name": "one_64k", "kind": "one", "where": "pool_to_pool", "tensors": 1, "lo": 64 * KiB, "hi": 64 * KiB,
         "odd": 0.0, "chunk": 2 * MiB, "shape": 1},
        # a server with 32 requests in flight: a job for each result, most results small, some at odd offsets
        {"name": "requests", "kind": "one", "where": "pool_to_pool", "tensors": 32, "lo": 4 * KiB, "hi": 1 * MiB,
         "odd": 0.25, "chunk": 2 * MiB, "shape": 2},
        # feature maps of single images (batch 1) passed between eight weighted functions
        {"name": "maps_batch1", "kind": "batch", "where": "pool_to_pool", "sizes": "maps1", "tensors": 64, "lo": 0, "hi": 0,
         "functions": 8, "odd": 0.0, "chunk": 2 * MiB, "call": "submit", "shape": 3},
        # the feature workload: 64 fp16 maps of batch 1, 8 or 32, weights 1:1:2:2:4:4:8:8, half a GiB
        {"name": "maps", "kind": "batch", "where": "pool_to_pool", "sizes": "maps", "tensors": 64, "lo": 0, "hi": 0,
         "functions": 8, "odd": 0.0, "chunk": 2 * MiB, "call": "submit", "shape": 4},
        # many small results (boxes, embeddings, cache blocks) gathered for the next stage in one job
        {"name": "small_tensors", "kind": "batch", "where": "pool_to_pool", "sizes": "log", "tensors": 1024,
         "lo": 1 * KiB, "hi": 64 * KiB, "functions": 4, "odd": 0.25, "chunk": 256 * KiB, "call": "submit", "shape": 5},
        # code that may not allocate (graph capture, tight loops): the static entry point, ordered by the stream alone
        {"name": "static", "kind": "batch", "where": "pool_to_pool", "sizes": "log", "tensors": 48, "lo": 64 * KiB,
         "hi": 2 * MiB, "functions": 4, "odd": 0.1, "chunk": 512 * KiB, "call": "static", "shape": 6},
        # the traffic workload's crops: 16 planar 1080p frames, 32 crops of 64..256 pixels a side each, two recognisers
        {"name": "crops", "kind": "rows", "where": "pool_to_pool", "images": 16, "planes": 3, "height": 1080, "pitch": 1920,
         "windows": 32, "rows_lo": 64, "rows_hi": 256, "row_lo": 64, "row_hi": 256, "form": "gather", "grid": False, "functions": 2,
         "chunk": 256 * KiB, "shape": 7},
        # interleaved 4K frames cut into quadrants for a detector
        {"name": "quadrants_4k", "kind": "rows", "where": "pool_to_pool", "images": 4, "planes": 1, "height": 2160,
         "pitch": 11520, "windows": 4, "rows_lo": 1080, "rows_hi": 1080, "row_lo": 5760, "row_hi": 5760, "form": "gather", "grid": True,
         "functions": 2, "chunk": 2 * MiB, "shape": 8},
        # the tiny workload: 32 inputs of 4 KiB..1 MiB to the pool, and as many results back to the host
        {"name": "inputs_and_results", "kind": "inout", "tensors": 32, "lo": 4 * KiB, "hi": 1 * MiB, "functions": 4,
         "odd": 0.0, "chunk": 64 * KiB, "shape": 9},
        # one wave of the large mixed workload: 64 transfers, both link classes at once, a tenth at odd offsets
        {"name": "wave", "kind": "wave", "tensors": 64, "bytes": 512 * MiB, "functions": 16, "odd": 0.1, "chunk": 2 * MiB,
         "shape": 10},
        # a model's inputs or weights out of ordinary memory, through the pinned ring
        {"name": "pageable_ring", "kind": "ring", "where": "pageable_to_pool", "tensors": 4, "bytes": 128 * MiB,
         "functions": 4, "chunk": 2 * MiB, "shape": 11},
        # the host link contended by sixteen weighted functions, 64 MiB each
        {"name": "contended", "kind": "batch", "where": "host_to_pool", "sizes": "log", "tensors": 16, "lo": 64 * MiB,
         "hi": 64 * MiB, "functions": 16, "odd": 0.0, "chunk": 512 * KiB, "call": "submit", "shape": 12},
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["one", "one", "batch", "batch", "batch", "rows", "rows", "inout", "wave", "ring"])
    shape = rng.randrange(100, 1 << 20)
    where = rng.choice(["pool_to_pool", "pool_to_pool", "host_to_pool", "pool_to_host"])
    odd = rng.choice([0.0, 0.1, 0.25, 1.0])
    chunk = rng.choice([64 * KiB, 256 * KiB, 512 * KiB, 2 * MiB])
    if kind == "one":
        n = rng.choice([1, 1, 1, _log(rng, 2, 64)])
        hi = _log(rng, 4 * KiB, 64 * MiB if n == 1 else 2 * MiB)
        return {"kind": "one", "where": where, "tensors": n, "lo": hi if n == 1 else max(256, hi // 64), "hi": hi,
                "odd": odd, "chunk": 2 * MiB, "shape": shape}
    if kind == "batch":
        n = _log(rng, 8, 2048)
        call = "static" if n <= 200 and rng.random() < 0.25 else "submit"
        most = min(64 * MiB, (LARGEST if where == "pool_to_pool" else 256 * MiB) // n)
        hi = _log(rng, 2 * KiB, most)
        sizes = "log" if rng.random() < 0.75 or n > 64 else rng.choice(["maps1", "maps"])
        if where != "pool_to_pool":
            sizes = "log"
        return {"kind": "batch", "where": where, "sizes": sizes, "tensors": n, "lo": max(256, hi // rng.choice([1, 8, 64])),
                "hi": hi, "functions": rng.randrange(1, 17), "odd": odd, "chunk": chunk, "call": call, "shape": shape}
    if kind == "rows":
        pitch = _log(rng, 512, 64 * KiB)
        row_hi = _log(rng, 16, pitch)
        height = _log(rng, 256, 4096)
        rows_hi = _log(rng, 16, height)
        images = max(1, min(16, (256 * MiB) // (3 * height * pitch)))
        most = (LARGEST // 2 if where == "pool_to_pool" else 128 * MiB) // (images * 3 * rows_hi * row_hi)
        return {"kind": "rows", "where": where, "images": images, "planes": rng.choice([1, 3]), "height": height,
                "pitch": pitch, "windows": max(1, min(32, most)), "rows_lo": max(1, rows_hi // 4), "rows_hi": rows_hi,
                "row_lo": max(16, row_hi // 4), "row_hi": row_hi, "form": rng.choice(["gather", "gather", "scatter", "both"]), "grid": False,
                "functions": rng.randrange(1, 5), "chunk": chunk, "shape": shape}
    if kind == "inout":
        hi = _log(rng, 8 * KiB, 8 * MiB)
        return {"kind": "inout", "tensors": rng.randrange(8, 65), "lo": max(1 * KiB, hi // 256), "hi": hi,
                "functions": rng.randrange(1, 9), "odd": odd, "chunk": rng.choice([64 * KiB, 512 * KiB]), "shape": shape}
    if kind == "wave":
        return {"kind": "wave", "tensors": rng.randrange(16, 129), "bytes": _log(rng, 16 * MiB, 512 * MiB),
                "functions": rng.randrange(2, 17), "odd": rng.choice([0.0, 0.1, 0.25]), "chunk": 2 * MiB, "shape": shape}
    return {"kind": "ring", "where": rng.choice(["pageable_to_pool", "pool_to_pageable"]), "tensors": rng.randrange(1, 9),
            "bytes": _log(rng, 16 * MiB, 128 * MiB), "functions": rng.randrange(1, 5), "chunk": 2 * MiB, "shape": shape}


# ---- shapes: functions of the case alone ------------------------------------------------------

def _sizes(case):
    rng = random.Random(case["shape"])
    n = case["tensors"]
    if case["kind"] == "ring":
        cuts = sorted(rng.randrange(1, case["bytes"]) for _ in range(n - 1))
        return [max(1, b - a) for a, b in zip([0] + cuts, cuts + [case["bytes"]])]
    if case["kind"] == "wave":
        raw = [min(max(rng.lognormvariate(0.0, 1.5), 0.002), 32.0) for _ in range(n)]
        scale = case["bytes"] / sum(raw)
        return [max(4 * KiB, int(r * scale)) // 16 * 16 for r in raw]
    if case.get("sizes") in ("maps", "maps1"):
        batches = [1, 8, 32] if case["sizes"] == "maps" else [1]
        return [2 * rng.choice(batches) * rng.choice([64, 256, 512]) * rng.choice([14, 28, 56]) ** 2 for _ in range(n)]
    sizes = [_log(rng, case["lo"], case["hi"]) for _ in range(n)]
    if case["odd"] == 0.0:
        sizes = [max(16, s // 16 * 16) for s in sizes]
    return sizes


def _weights(n):
    return [(1, 1, 2, 2, 4, 4, 8, 8)[f % 8] for f in range(n)]


def _windows(case):
    """(image, plane, first row, first byte, rows, row bytes) of every descriptor of a `rows` case."""
    rng = random.Random(case["shape"])
    out = []
    if case["grid"]:  # the image cut into equal parts
        across = case["pitch"] // case["row_hi"]
        return [(i, p, w // across * case["rows_hi"], w % across * case["row_hi"], case["rows_hi"], case["row_hi"])
                for i in range(case["images"]) for w in range(case["windows"]) for p in range(case["planes"])]
    if case["form"] == "gather":  # windows may overlap: they are only read
        for i in range(case["images"]):
            for _ in range(case["windows"]):
                r, b = rng.randint(case["rows_lo"], case["rows_hi"]), rng.randint(case["row_lo"], case["row_hi"])
                y, x = rng.randint(0, case["height"] - r), rng.randint(0, case["pitch"] - b)
                out += [(i, p, y, x, r, b) for p in range(case["planes"])]
        return out
    # windows that are written lie in cells of a grid of their own
    down, across = case["height"] // case["rows_hi"], case["pitch"] // case["row_hi"]
    cells = [(y, x) for y in range(down) for x in range(across)]
    for i in range(case["images"]):
        for y, x in rng.sample(cells, min(case["windows"], len(cells))):
            r, b = rng.randint(case["rows_lo"], case["rows_hi"]), rng.randint(case["row_lo"], case["row_hi"])
            out += [(i, p, y * case["rows_hi"], x * case["row_hi"], r, b) for p in range(case["planes"])]
    return out


# ---- state --------------------------------------------------------------------------------------

class State:
    """A pool over one device tensor, pinned and pageable host memory, and the jobs to submit."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.pool = None
        self.jobs = []       # (Transfers, chunk bytes, flags)
        self.outputs = []
        self.static = False
        self.one_by_one = False
        self.stream = torch.cuda.current_stream().cuda_stream

    def random_device(self, n):
        return torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=self.gen)

    def make_pool(self, nbytes, slab):
        n = -(-(nbytes + slab) // slab) * slab
        self.mem = torch.full((n,), CANARY, dtype=torch.uint8, device="cuda")
        self.pool = ft.pool_create(self.mem.data_ptr(), n, slab, self.mem.device.index or 0)

    def random_pool(self, lo, hi):
        if hi > lo:
            self.mem[lo:hi].copy_(self.random_device(hi - lo))

    def pinned(self, n, random_fill):
        t = torch.empty(n, dtype=torch.uint8, pin_memory=True)
        if random_fill:
            t.copy_(self.random_device(n))
        else:
            t.fill_(CANARY)
        ft.host_window_add(self.pool, t.data_ptr(), n)
        return t

    def pageable(self, n, random_fill):
        t = torch.empty(n, dtype=torch.uint8)
        if random_fill:
            t.copy_(self.random_device(n))
        else:
            t.fill_(CANARY)
        ft.pageable_window_add(self.pool, t.data_ptr(), n)
        return t

    def __del__(self):
        if self.pool is not None:
            ft.pool_destroy(self.pool)


def _up(v, a):
    return -(-v // a) * a


def _shifts(case, n):
    """Byte offsets of both sides of every tensor from a 16-byte boundary."""
    rng = random.Random(case["shape"] + 1)
    return [(rng.randint(1, 15), rng.randint(1, 15)) if rng.random() < case.get("odd", 0.0) else (0, 0) for _ in range(n)]


def _tensors(st, case, sizes, where):
    """Both sides of every tensor of a list, and which memory the results lie in: (src, dst) addresses and the output."""
    src_space, dst_space = SPACES[where]
    shifts = _shifts(case, len(sizes))
    room = [s + 16 for s in sizes]
    slab = 4 * KiB if max(sizes) < 256 * KiB else 256 * KiB
    in_pool = [space == POOL for space in (src_space, dst_space)]
    st.make_pool(sum(in_pool) * sum(_up(r, slab) for r in room), slab)
    sides = []
    for side, space in enumerate((src_space, dst_space)):
        if space == POOL:
            base = [ft.slab_alloc(st.pool, r) for r in room]
            lo, hi = base[0], base[-1] + _up(room[-1], slab)
            if side == 0:
                st.random_pool(lo, hi)
            else:
                out = st.mem[lo:hi]
        else:
            at, total = [], 0
            for r in room:
                at.append(total)
                total = _up(total + r, 4 * KiB)
            t = (st.pinned if space == HOST else st.pageable)(total, side == 0)
            base = [t.data_ptr() + a for a in at]
            if side == 0:
                st.source = t
            else:
                out = t
        sides.append([b + s[side] for b, s in zip(base, shifts)])
    return sides[0], sides[1], out


def _descs(src_space, dst_space, src, dst, sizes, functions):
    return [dict(func=i % functions, src_space=src_space, dst_space=dst_space, src=s, dst=d, row_bytes=n)
            for i, (s, d, n) in enumerate(zip(src, dst, sizes))]


def prepare(case, seed):
    st = State(seed)
    kind = case["kind"]
    if kind == "one":
        src, dst, out = _tensors(st, case, _sizes(case), case["where"])
        a, b = SPACES[case["where"]]
        for s, d, n in zip(src, dst, _sizes(case)):
            st.jobs.append((ft.Transfers(make_descs(_descs(a, b, [s], [d], [n], 1)), [1]), case["chunk"], 0))
        st.outputs = [out]
    elif kind in ("batch", "ring"):
        sizes = _sizes(case)
        src, dst, out = _tensors(st, case, sizes, case["where"])
        a, b = SPACES[case["where"]]
        nf = min(case["functions"], len(sizes))
        st.jobs = [(ft.Transfers(make_descs(_descs(a, b, src, dst, sizes, nf)), _weights(nf)), case["chunk"],
                    FT_OPEN if kind == "ring" else 0)]
        st.static = case.get("call") == "static"
        st.outputs = [out]
    elif kind == "inout":
        sizes = _sizes(case)
        shifts = _shifts(case, len(sizes))
        slab = 4 * KiB if max(sizes) < 256 * KiB else 256 * KiB
        st.make_pool(sum(_up(s + 16, slab) for s in sizes), slab)
        base = [ft.slab_alloc(st.pool, s + 16) for s in sizes]
        at, total = [], 0
        for s in sizes:
            at.append(total)
            total = _up(total + s + 16, 4 * KiB)
        st.source, back = st.pinned(total, True), st.pinned(total, False)
        src = [st.source.data_ptr() + a + s[0] for a, s in zip(at, shifts)]
        mid = [b + s[1] for b, s in zip(base, shifts)]
        dst = [back.data_ptr() + a + s[0] for a, s in zip(at, shifts)]
        nf = min(case["functions"], len(sizes))
        w = _weights(nf)
        st.jobs = [(ft.Transfers(make_descs(_descs(HOST, POOL, src, mid, sizes, nf)), w), case["chunk"], 0),
                   (ft.Transfers(make_descs(_descs(POOL, HOST, mid, dst, sizes, nf)), w), case["chunk"], 0)]
        st.one_by_one = True
        st.outputs = [st.mem, back]
    elif kind == "wave":
        sizes = _sizes(case)
        shifts = _shifts(case, len(sizes))
        rng = random.Random(case["shape"] + 2)
        from_host = [rng.random() < 0.6 for _ in sizes]
        slab = 64 * KiB
        st.make_pool(sum(_up(s + 16, slab) * (1 if h else 2) for s, h in zip(sizes, from_host)), slab)
        inside = [None if h else ft.slab_alloc(st.pool, s + 16) for s, h in zip(sizes, from_host)]
        dst = [ft.slab_alloc(st.pool, s + 16) for s in sizes]
        st.random_pool(0, dst[0])
        arena = max([64 * KiB] + [_up(s + 16, 4 * KiB) for s, h in zip(sizes, from_host) if h]) + 64 * MiB
        st.source = st.pinned(arena, True)
        descs = []
        for i, n in enumerate(sizes):
            at = st.source.data_ptr() + rng.randrange(0, (arena - n - 16) // 16) * 16 if from_host[i] else inside[i]
            descs.append(dict(func=i % case["functions"], src_space=HOST if from_host[i] else POOL, dst_space=POOL,
                              src=at + shifts[i][0], dst=dst[i] + shifts[i][1], row_bytes=n))
        st.jobs = [(ft.Transfers(make_descs(descs), _weights(case["functions"])), case["chunk"], 0)]
        st.outputs = [st.mem[dst[0]:]]
    else:
        _prepare_rows(st, case)
    return st


def _prepare_rows(st, case):
    """Windows of images: gathered into packed buffers, scattered out of them, or moved between two sets of images."""
    src_space, dst_space = SPACES[case["where"]]
    plane = case["height"] * case["pitch"]
    image = case["planes"] * plane
    wins = _windows(case)
    packed_at, run = [], 0
    for (_, _, _, _, r, b) in wins:
        packed_at.append(run)
        run = _up(run + r * b, 16)
    images = case["images"] * image
    extent = {"gather": (images, run), "scatter": (run, images), "both": (images, images)}[case["form"]]
    slab = 1 * MiB
    st.make_pool(sum(_up(e, slab) for e, s in zip(extent, (src_space, dst_space)) if s == POOL), slab)
    base = []
    for side, space in enumerate((src_space, dst_space)):
        if space == POOL:
            off = ft.slab_alloc(st.pool, extent[side])
            if side == 0:
                st.random_pool(off, off + extent[side])
            else:
                st.outputs = [st.mem[off:off + extent[side]]]
            base.append(off)
        else:
            t = st.pinned(extent[side], side == 0)
            if side == 0:
                st.source = t
            else:
                st.outputs = [t]
            base.append(t.data_ptr())
    descs = []
    nf = case["functions"]
    for k, (i, p, y, x, r, b) in enumerate(wins):
        in_image, in_packed = i * image + p * plane + y * case["pitch"] + x, packed_at[k]
        at = {"gather": (in_image, in_packed), "scatter": (in_packed, in_image), "both": (in_image, in_image)}[case["form"]]
        pitch = {"gather": (case["pitch"], b), "scatter": (b, case["pitch"]), "both": (case["pitch"], case["pitch"])}[case["form"]]
        descs.append(dict(func=k // case["planes"] % nf, src_space=src_space, dst_space=dst_space, src=base[0] + at[0],
                          dst=base[1] + at[1], row_bytes=b, rows=r, src_pitch=pitch[0], dst_pitch=pitch[1]))
    nf = min(nf, max(d["func"] for d in descs) + 1)
    st.jobs = [(ft.Transfers(make_descs(descs), _weights(nf)), case["chunk"], 0)]


def run(st):
    pool, stream = st.pool, st.stream
    if st.static:
        (tr, chunk, _), = st.jobs
        ft.submit_static(pool, tr.descs, tr.weights, chunk, 0, stream)
    elif st.one_by_one:
        for tr, chunk, flags in st.jobs:
            ft.wait(pool, ft.submit_transfers(pool, tr, None, chunk, flags, stream))
    else:
        handles = [ft.submit_transfers(pool, tr, None, chunk, flags, stream) for tr, chunk, flags in st.jobs]
        for h in handles:
            ft.wait(pool, h)
    return st.outputs


def work(case):
    if case["kind"] == "rows":
        payload = sum(w[4] * w[5] for w in _windows(case))
    else:
        payload = sum(_sizes(case)) * (2 if case["kind"] == "inout" else 1)
    return {"bytes": 2 * payload, "flops": 0}  # every byte is read once and written once


def tolerance(case):
    return "exact"
