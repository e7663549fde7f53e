"""Performance cases of the LeCo codec: the calls its users make, over the
sizes, column shapes, dtypes and options they make them with.

A case is a dict of plain values.  ``listed()`` gives the standing ones,
``draw(rng)`` another one from the same ranges, ``prepare(case, seed)`` what
a program has in hand before the call, ``run(state)`` one pass through the
public entry points, ``work(case)`` the bytes a pass cannot do without and
``exact(case, seed)`` the outputs that plain torch can state.

Column shapes (those of the benchmark, drawn on the device):
  line      1000 + 7 i + U{0..63}
  keys      sorted keys, cumulative sum of max(1, rint(lognormal(3, 1.5)))
  normal    sorted samples of N(2^30, 2^26)
  polyline  pieces of about 100,000 values, slopes U[0, 50), noise U{0..255}
  runs      runs of one value, geometric lengths with mean 64
  cosmos    two sines plus Gaussian noise
  cubic     blocks of 1000 .. 8000 values on random cubics, noise U{0..15}
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2306_15374_amd as leco

WIDTH = {"u32": 4, "u64": 8}
TORCH = {"u32": torch.int32, "u64": torch.int64}  # bit patterns of the unsigned values
DEV = "cuda"
TAU = 0.03  # split threshold of the variable partitions

_codec = None


def codec():
    """The program's one context."""
    global _codec
    if _codec is None:
        _codec = leco.Codec(0)
    return _codec


# ---- the cases -----------------------------------------------------------------

def listed():
    return [
        # one short column encoded as it arrives: latency and launches count
        dict(name="encode_small", kind="encode", data="line", dtype="u64", n=10_000, L=1024,
             regressor="ls"),
        # bulk load of a sorted key column, the benchmark's column and length
        dict(name="encode_keys", kind="encode", data="keys", dtype="u64", n=200_000_000, L=4096,
             regressor="ls"),
        # bulk load for the smallest blob of the line models
        dict(name="encode_minimax", kind="encode", data="line", dtype="u32", n=100_000_000, L=1024,
             regressor="minimax"),
        # bulk load of a non-linear signal with the higher-order models, at
        # the evaluation's partition length (no power of two)
        dict(name="encode_poly", kind="encode", data="cosmos", dtype="u32", n=100_000_000, L=1000,
             regressor="poly"),
        # a page of a resident column
        dict(name="decode_small", kind="decode", data="line", dtype="u64", n=1_000_000, L=1024,
             regressor="ls", span=10_000),
        # full scan of the benchmark's key column
        dict(name="decode_keys", kind="decode", data="keys", dtype="u64", n=200_000_000, L=4096,
             regressor="ls", span=0),
        # full scan of a 32-bit column whose partition length is no multiple
        # of a wavefront or a cache line
        dict(name="decode_odd", kind="decode", data="normal", dtype="u32", n=100_000_000, L=1000,
             regressor="ls", span=0),
        # full scan of variable partitions, 64 values each on average
        dict(name="decode_runs", kind="decode", data="runs", dtype="u32", n=100_000_000, L=0,
             regressor="ls", span=0),
        # point lookups at uniform positions of the key column
        dict(name="lookup_keys", kind="lookup", data="keys", dtype="u64", n=200_000_000, L=4096,
             regressor="ls", k=20_000_000),
        # a table of many uneven columns scanned in one launch
        dict(name="batch_decode", kind="batch", op="decode", cols=512),
        # requests of mixed sizes against resident columns
        dict(name="serve", kind="serve", cols=16, n=4_000_000, requests=48, range_exp=6.5),
        # variable partitions chosen for a column before its bulk load
        dict(name="partition", kind="partition", data="polyline", dtype="u32", n=10_000_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _column(rng, top):
    """A column shape, its dtype and a length of at most `top`."""
    data = rng.choice(["line", "keys", "normal", "cosmos", "cubic"])
    dtype = {"line": rng.choice(["u32", "u64"]), "keys": rng.choice(["u32", "u64"]), "normal": "u32",
             "cosmos": "u32", "cubic": "u64"}[data]
    if data == "keys" and dtype == "u32":
        top = min(top, 20_000_000)  # the keys stay below 2^31
    return dict(data=data, dtype=dtype, n=_log(rng, 2_000, top))


def _length(rng):
    """A partition length: a power of two or any."""
    return rng.choice([1 << rng.randint(7, 12), _log(rng, 100, 4096)])


def draw(rng):
    kind = rng.choice(["encode", "encode", "decode", "decode", "lookup", "batch", "serve", "partition"])
    if kind == "encode":
        return dict(kind=kind, **_column(rng, 100_000_000), L=_length(rng),
                    regressor=rng.choice(["ls", "minimax", "poly"]))
    if kind == "decode":
        if rng.random() < 0.25:  # variable partitions
            c = dict(data="runs", dtype="u32", n=_log(rng, 2_000, 100_000_000), L=0, regressor="ls")
        else:
            c = dict(**_column(rng, 100_000_000), L=_length(rng),
                     regressor=rng.choice(["ls", "ls", "minimax", "poly"]))
        return dict(kind=kind, **c, span=rng.choice([0, _log(rng, 1_000, c["n"])]))
    if kind == "lookup":
        c = _column(rng, 100_000_000)
        return dict(kind=kind, **c, L=_length(rng), regressor="ls", k=_log(rng, 100, 20_000_000))
    if kind == "batch":
        return dict(kind=kind, op=rng.choice(["decode", "filter", "encode"]), cols=_log(rng, 16, 512))
    if kind == "serve":
        return dict(kind=kind, cols=rng.randint(2, 32), n=_log(rng, 200_000, 4_000_000),
                    requests=rng.randint(8, 48), range_exp=round(rng.uniform(4.0, 6.5), 2))
    return dict(kind=kind, data=rng.choice(["polyline", "normal", "runs"]), dtype="u32",
                n=_log(rng, 20_000, 2_000_000))


# ---- columns -------------------------------------------------------------------

def _gen(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return g


def column(data, n, seed, dtype, device=DEV):
    g = _gen(seed, device)

    def randint(lo, hi, k):
        return torch.randint(lo, hi, (k,), generator=g, device=device, dtype=torch.int64)

    def uniform(k):
        return torch.rand(k, generator=g, device=device, dtype=torch.float64)

    def normal(k):
        return torch.randn(k, generator=g, device=device, dtype=torch.float64)

    if data == "line":
        v = torch.arange(n, dtype=torch.int64, device=device) * 7 + 1000
        v += randint(0, 64, n)
    elif data == "keys":
        v = torch.cumsum(torch.round(torch.exp(normal(n) * 1.5 + 3.0)).clamp_(min=1.0).to(torch.int64), 0)
    elif data == "normal":
        v = torch.round(normal(n) * 2.0**26 + 2.0**30).clamp_(0, 2**31 - 1).to(torch.int64)
        v = torch.sort(v).values
    elif data == "polyline":
        pieces = max(4, n // 100_000)
        cuts = torch.sort(randint(0, n, pieces)).values
        slope = uniform(pieces + 1) * 50.0
        piece = torch.bucketize(torch.arange(n, device=device), cuts, right=True)
        v = torch.floor(torch.cumsum(slope[piece], 0)).to(torch.int64) + randint(0, 256, n)
    elif data == "runs":
        k = n // 48 + 64  # more than enough runs of mean 64
        lens = torch.floor(torch.log1p(-uniform(k)) / math.log1p(-1.0 / 64.0)).to(torch.int64) + 1
        while int(lens.sum()) < n:
            lens = torch.cat([lens, lens])
        v = torch.repeat_interleave(randint(0, 1 << 32, len(lens)), lens)[:n]
        return torch.where(v < 2**31, v, v - 2**32).to(torch.int32)
    elif data == "cosmos":
        x = torch.arange(n, dtype=torch.float64, device=device) + 10.0
        w = 60.0 * math.pi
        v = torch.round((torch.sin(x / w) + torch.sin(3.0 * x / w) / 10.0) * 1e6 + normal(n) * 100.0 + 2.0**21)
        v = v.to(torch.int64)
    else:  # cubic
        k = n // 4000 + 8
        lens = randint(1000, 8000, k)
        while int(lens.sum()) < n:
            lens = torch.cat([lens, lens])
        k = len(lens)
        b, c, d = uniform(k) * 1000.0, uniform(k) * 0.1 - 0.05, uniform(k) * 2e-5 - 1e-5
        h = lens.to(torch.float64) - 1.0
        rise = b * h + c * h * h + d * h * h * h
        a = torch.cumsum(rise, 0) - rise + 2.0**40
        blk = torch.repeat_interleave(torch.arange(k, device=device), lens)[:n]
        t = (torch.arange(n, device=device) - (torch.cumsum(lens, 0) - lens)[blk]).to(torch.float64)
        v = torch.round(a[blk] + ((d[blk] * t + c[blk]) * t + b[blk]) * t).to(torch.int64) + randint(0, 16, n)
    return v.to(TORCH[dtype])


def _blob(col, case):
    """The column's blob, encoded as its owner does it once."""
    if case["L"]:
        return codec().encode(col, fixed_len=case["L"], regressor=case["regressor"])
    return codec().encode(col, starts=codec().partition(col, tau=TAU), regressor=case["regressor"])


def _span(case, seed):
    """[begin, end) of a decode."""
    n, span = case["n"], case["span"]
    if not span or span >= n:
        return 0, n
    b = int(np.random.default_rng(seed + 1).integers(0, n - span + 1))
    return b, b + span


def _positions(case, seed):
    g = _gen(seed + 1, DEV)
    return torch.randint(0, case["n"], (case["k"],), generator=g, device=DEV, dtype=torch.int64)


# ---- a table of columns ----------------------------------------------------------

def _table(case, seed):
    """Column specs: lognormal lengths (median 130,000, 1e3 .. 1e7), both
    dtypes, noisy lines at L 1024 and keys at L 4096.  The case fixes the
    sizes, the seed the values."""
    k = case["cols"]
    rng = np.random.default_rng(k)
    lens = np.clip(np.rint(np.exp(rng.normal(math.log(1.3e5), 1.7, k))), 1e3, 1e7).astype(int)
    kinds, wide = rng.integers(0, 2, k), rng.integers(0, 2, k)
    return [dict(data="keys" if kinds[i] else "line", dtype="u64" if wide[i] else "u32", n=int(lens[i]),
                 L=4096 if kinds[i] else 1024, seed=seed * 1000 + i, regressor="ls")
            for i in range(k)]


def _slots(sizes, align=256):
    """Byte offsets of buffers laid one after another, and their total."""
    at, offs = 0, []
    for s in sizes:
        offs.append(at)
        at += (s + align - 1) // align * align
    return offs, max(at, align)


def _table_out(specs):
    return _slots([s["n"] * WIDTH[s["dtype"]] for s in specs])


def _bounds(col):
    lo, hi = int(col[:1].item()), int(col[-1:].item())  # both shapes rise
    r = hi - lo
    return lo + r // 4, lo + 3 * r // 4


class Batch:
    """A batch handle with what its jobs point at."""

    def __init__(self, case, seed):
        specs = _table(case, seed)
        cols = [column(s["data"], s["n"], s["seed"], s["dtype"]) for s in specs]
        self.op = case["op"]
        self.handle = None
        self.size = torch.zeros(len(specs), dtype=torch.int64, device=DEV)
        if self.op == "encode":
            caps = [leco.leco_max_blob_bytes(s["n"], WIDTH[s["dtype"]],
                                             leco.make_partitioning(fixed_len=s["L"])[0]) for s in specs]
            offs, total = _slots(caps)
            self.cols = cols
            self.out = torch.zeros(total, dtype=torch.uint8, device=DEV)
            self.jobs = [leco.EncodeJob(c.data_ptr(), s["n"], WIDTH[s["dtype"]], 0, s["L"],
                                        self.out.data_ptr() + o, cap, self.size.data_ptr() + 8 * i, 0, 0)
                         for i, (s, c, o, cap) in enumerate(zip(specs, cols, offs, caps))]
            return
        offs, total = _table_out(specs)
        self.blobs = [_blob(c, s) for s, c in zip(specs, cols)]
        self.out = torch.zeros(total if self.op == "decode" else 8, dtype=torch.uint8, device=DEV)
        self.sums = torch.zeros(len(specs), 3, dtype=torch.int64, device=DEV)
        jobs = []
        for i, (s, c, b, o) in enumerate(zip(specs, cols, self.blobs, offs)):
            lo, hi = _bounds(c)
            decode = self.op == "decode"
            jobs.append(leco.DecodeJob(b.data_ptr(), b.numel(), s["n"],
                                       self.out.data_ptr() + o if decode else None, lo, hi,
                                       None if decode else self.sums[i].data_ptr()))
        self.handle = leco.leco_batch_create(codec().ctx, jobs)

    def run(self):
        if self.op == "encode":
            codec().check("leco_encode_batch", leco.leco_encode_batch(codec().ctx, self.jobs))
            return self.out, self.size
        what = leco.LECO_BATCH_DECODE if self.op == "decode" else leco.LECO_BATCH_FILTER
        codec().check("leco_batch_run", leco.leco_batch_run(self.handle, what))
        return self.out if self.op == "decode" else self.sums

    def __del__(self):
        if self.handle:
            torch.cuda.synchronize()
            leco.leco_batch_destroy(self.handle)


# ---- served requests ------------------------------------------------------------

def _served(case, seed):
    """Column specs and requests: half lookups of floor(2^U[0, 16]) uniform
    positions in device memory, half ranges of floor(10^U[3, range_exp])
    values.  The case fixes columns and sizes, the seed values and places."""
    rng, at = np.random.default_rng(case["requests"]), np.random.default_rng(seed)
    n = case["n"]
    specs = [dict(data="keys" if c % 2 else "line", dtype="u64", n=n, L=4096 if c % 2 else 1024,
                  seed=seed * 1000 + c, regressor="ls") for c in range(case["cols"])]
    reqs = []
    for _ in range(case["requests"]):
        c = int(rng.integers(0, len(specs)))
        if rng.integers(0, 2) == 0:
            k = int(2.0 ** rng.uniform(0, 16))
            reqs.append((c, at.integers(0, n, size=k)))
        else:
            ln = min(int(10.0 ** rng.uniform(3, case["range_exp"])), n)
            b = int(at.integers(0, n - ln + 1))
            reqs.append((c, b, b + ln))
    return specs, reqs


class _DeviceValues:
    """`count` 64-bit values in the server's memory, which stays with it as
    long as a tensor made of them does."""

    def __init__(self, server, ptr, count):
        self.server = server
        self.__cuda_array_interface__ = dict(shape=(count,), typestr="<i8", data=(ptr, False), version=2)


class Server:
    """A server over resident columns and one batch of requests to it."""

    def __init__(self, case, seed):
        specs, reqs = _served(case, seed)
        self.handle = None
        self.blobs = [_blob(column(s["data"], s["n"], s["seed"], s["dtype"]), s) for s in specs]
        self.pos = [torch.from_numpy(r[1]).to(DEV) if len(r) == 2 else None for r in reqs]
        self.reqs = (leco.Request * len(reqs))()
        for i, r in enumerate(reqs):
            if len(r) == 2:
                self.reqs[i] = leco.Request(leco.LECO_REQ_RANDOM_ACCESS_DEV, r[0], self.pos[i].data_ptr(),
                                            len(r[1]), 0, 0)
            else:
                self.reqs[i] = leco.Request(leco.LECO_REQ_RANGE, r[0], None, 0, r[1], r[2])
        torch.cuda.synchronize()  # the server reads positions on its own streams
        cfg = leco.ServerConfig(1 << 30, 256, 4, 1 << 16, 1 << 20, 0, 0, 0, 1 << 24)
        res = [leco.ResidentCol(b.data_ptr(), b.numel(), s["n"]) for b, s in zip(self.blobs, specs)]
        self.handle = leco.leco_server_start(codec().ctx, res, cfg)
        self.held = []

    def run(self):
        for t in self.held:  # the last pass's results are done with
            leco.leco_server_release(self.handle, t)
        st, tickets = leco.leco_server_submit_batch(self.handle, self.reqs)
        codec().check("leco_server_submit_batch", st)
        done = {}
        while len(done) < len(tickets):
            for c in leco.leco_server_poll(self.handle, len(tickets)):
                codec().check("request", c.status)
                done[c.ticket] = c
        self.held = tickets
        # valid until the tickets are released; each keeps the server alive
        return [torch.as_tensor(_DeviceValues(self, done[t].out_dev, done[t].count), device=DEV) for t in tickets]

    def __del__(self):
        if self.handle:
            leco.leco_server_stop(self.handle)


# ---- prepare and run -------------------------------------------------------------

class State:
    pass


def prepare(case, seed):
    if case["kind"] == "batch":
        return Batch(case, seed)
    if case["kind"] == "serve":
        return Server(case, seed)
    s = State()
    s.kind, s.case = case["kind"], case
    w = WIDTH[case["dtype"]]
    col = column(case["data"], case["n"], seed, case["dtype"])
    if s.kind == "partition":
        s.col = col
        s.params = leco.PartitionParams(TAU, 320, 1 << 20, 0, 0, 0)
        s.starts = np.zeros(case["n"] // 4 + 2, dtype=np.uint64)
    elif s.kind == "encode":
        s.col = col
        s.part, _ = leco.make_partitioning(fixed_len=case["L"], regressor=case["regressor"])
        s.cap = leco.leco_max_blob_bytes(case["n"], w, s.part)
        s.blob = torch.zeros(s.cap, dtype=torch.uint8, device=DEV)
        s.size = torch.zeros(1, dtype=torch.int64, device=DEV)
    else:
        s.blob = _blob(col, case)
        if s.kind == "decode":
            s.begin, s.end = _span(case, seed)
            s.out = torch.zeros(s.end - s.begin, dtype=TORCH[case["dtype"]], device=DEV)
        else:
            s.pos = _positions(case, seed)
            s.out = torch.zeros(case["k"], dtype=TORCH[case["dtype"]], device=DEV)
    return s


def run(s):
    if isinstance(s, (Batch, Server)):
        return s.run()
    c = codec()
    if s.kind == "partition":
        st, m = leco.leco_partition(c.ctx, s.col, s.case["n"], WIDTH[s.case["dtype"]], s.params, s.starts)
        c.check("leco_partition", st)
        return s.starts.view(np.int64), m
    if s.kind == "encode":
        c.check("leco_encode_async", leco.leco_encode_async(
            c.ctx, s.col, s.case["n"], WIDTH[s.case["dtype"]], s.part, s.blob, s.cap, s.size))
        return s.blob, s.size
    if s.kind == "lookup":
        c.check("leco_random_access", leco.leco_random_access(
            c.ctx, s.blob, s.blob.numel(), s.pos, s.case["k"], s.out))
    elif s.end - s.begin == s.case["n"]:
        c.check("leco_decode_all", leco.leco_decode_all(
            c.ctx, s.blob, s.blob.numel(), s.out, s.case["n"]))
    else:
        c.check("leco_decode_range", leco.leco_decode_range(
            c.ctx, s.blob, s.blob.numel(), s.begin, s.end, s.out))
    return s.out


# ---- work and exact values ---------------------------------------------------------

def _bytes_per_value(data, dtype, n, L, regressor):
    """Blob bytes per value, from least-squares fits of a few partitions."""
    if L == 0:
        return 40.0 / 64.0  # a record and a start per run
    if data == "normal":  # the middle of n sorted samples: exponential gaps
        gap = 2.0**26 * math.sqrt(2.0 * math.pi) / n
        v = np.floor(np.cumsum(np.random.default_rng(5).exponential(gap, (8, L)), axis=1))
    else:
        v = column(data, 8 * L, 5, dtype, "cpu").numpy().reshape(8, L).astype(np.float64)
    t = np.linspace(-1.0, 1.0, L)
    bits = []
    for y in v:
        r = y - np.polyval(np.polyfit(t, y, 3 if regressor == "poly" else 1), t)
        bits.append(math.ceil(math.log2(max(float(np.ptp(r)), 1.0) + 1.0)))
    return float(np.mean(bits)) / 8.0 + (48.0 if regressor == "poly" else 32.0) / L


def work(case):
    kind = case["kind"]
    if kind == "batch":
        mean = 1.3e5 * math.exp(1.7**2 / 2)
        out, blob = mean * 6.0, mean * (_bytes_per_value("line", "u64", 0, 1024, "ls") +
                                        _bytes_per_value("keys", "u64", 0, 4096, "ls")) / 2
        per = blob / 2 if case["op"] == "filter" else out + blob  # half the range lies inside the filter
        return {"bytes": case["cols"] * per, "flops": 0}
    if kind == "serve":
        n = case["n"]
        b = (_bytes_per_value("line", "u64", n, 1024, "ls") + _bytes_per_value("keys", "u64", n, 4096, "ls")) / 2
        e = case["range_exp"]
        lookups, values = (2**16 - 1) / (16 * math.log(2)), (10**e - 10**3) / ((e - 3) * math.log(10))
        return {"bytes": case["requests"] / 2 * (lookups * 24 + values * (8 + b)), "flops": 0}
    w, n = WIDTH[case["dtype"]], case["n"]
    if kind == "partition":
        return {"bytes": n * w, "flops": 0}
    if kind == "lookup":  # position, residual word, value
        return {"bytes": case["k"] * (16 + w), "flops": 0}
    b = _bytes_per_value(case["data"], case["dtype"], n, case["L"], case["regressor"])
    values = n if kind == "encode" or not case["span"] else min(case["span"], n)
    return {"bytes": values * (w + b), "flops": 0}


def exact(case, seed):
    """The values a decode or a lookup returns are the column's own; blobs
    and partition starts have no other definition than the codec's."""
    kind = case["kind"]
    if kind == "decode":
        b, e = _span(case, seed)
        return column(case["data"], case["n"], seed, case["dtype"])[b:e]
    if kind == "lookup":
        return column(case["data"], case["n"], seed, case["dtype"])[_positions(case, seed)]
    if kind == "batch" and case["op"] == "decode":
        specs = _table(case, seed)
        offs, total = _table_out(specs)
        out = torch.zeros(total, dtype=torch.uint8, device=DEV)
        for s, o in zip(specs, offs):
            v = column(s["data"], s["n"], s["seed"], s["dtype"]).view(torch.uint8)
            out[o:o + v.numel()] = v
        return out
    if kind == "batch" and case["op"] == "filter":
        rows = []
        for s in _table(case, seed):
            v = column(s["data"], s["n"], s["seed"], s["dtype"]).to(torch.int64)
            lo, hi = _bounds(v)
            v = v[(v >= lo) & (v < hi)]
            rows.append([int(v.sum()), 0, v.numel()])
        return torch.tensor(rows, dtype=torch.int64)
    if kind == "serve":
        specs, reqs = _served(case, seed)
        cols = [column(s["data"], s["n"], s["seed"], s["dtype"]) for s in specs]
        return [cols[r[0]][torch.from_numpy(r[1]).to(DEV)] if len(r) == 2 else cols[r[0]][r[1]:r[2]]
                for r in reqs]
    return None
