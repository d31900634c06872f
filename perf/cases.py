"""What a user of the library has it do, as cases that can be timed and checked.

A case is a dict of plain values.  Its "op" is the entry point used:

  step     adr_decode_step: append the new token, attend over the cached tokens (an executor's layer)
  attend   adr_kv_append then adr_decode_attention, the two calls on their own
  layer    adr_pack_qkv, adr_decode_step on views of the packed rows, adr_scatter_rows: a layer of the
           offloaded rows with both copies around it
  table    GraphTable.launch: a pre-recorded step over several layers, replayed for a batch that fills
           part of a recorded capacity
  merge    adr_lse_merge: combining the (o, lse) pairs of sequence-sharded requests

Lengths are the quantiles of the case's distribution, so that the tokens of a case (and with them its
work) are known from the case alone; the seed decides which request has which length, where the pages
lie and all values.  Values are N(0,1) rounded to bf16, as in the repository's workloads; pages no request
of the batch owns hold values too, as the other requests' pages of a pool in service do.  An fp8 pool has
one scale per page and kv-head, amax / 448.
"""
import math
import statistics

import numpy as np
import torch

import paper_2503_20552_amd as adr

_GQA = {"Hq": 32, "Hkv": 8, "d": 128}
_BASE = {"page": 16, "cache": "bf16", "out": "bf16", "lse": False, "part": 512, "bound": 0}


def listed():
    def case(name, op, **kw):
        return {"name": name, "op": op, **_BASE, **kw}

    return [
        # the smallest call of an executor: one offloaded request, under the bound the executor always passes
        case("single_request", "step", B=1, **_GQA, lengths="fixed_2000", bound=8192),
        # workload 1 of the repository: a few short requests, MHA heads of 64, one pass per request, fp32 out
        case("tiny_mha_d64", "attend", B=4, Hq=8, Hkv=8, d=64, lengths="uniform_1_512", part=0, out="f32", lse=True),
        # long requests kept on several executors: their partial results meet (3 shards each on average)
        case("merge_shards", "merge", B=96, **_GQA, parts=3),
        # the decode side's grouping, a small ragged batch of offloaded rows, and the rows put back
        case("layer_b37", "layer", B=37, **_GQA, lengths="lognormal_1000_16_4096"),
        # kernel pre-launching: eight layers replayed from a table recorded every 16 rows up to 64
        case("table_b40_8layers", "table", B=40, **_GQA, lengths="lognormal_1000_16_4096", bound=8192, layers=8,
             interval=16, capacity=64),
        # workload 2: Llama-2-7B-shaped MHA
        case("mha_b64", "step", B=64, Hq=32, Hkv=32, d=128, lengths="lognormal_1000_16_4096"),
        # workload 3, the benchmark: Llama-3-8B-shaped, 256 requests
        case("gqa_b256", "step", B=256, **_GQA, lengths="lognormal_1500_16_8192"),
        # the same batch over an fp8 cache
        case("gqa_b256_fp8", "step", B=256, **_GQA, lengths="lognormal_1500_16_8192", cache="fp8"),
        # workload 4: 70B-class heads (eight queries per kv-head), heavy-tailed lengths
        case("gqa_wide_b128", "step", B=128, Hq=64, Hkv=8, d=128, lengths="pareto_1.5_256_32768"),
        # workload 5: 512 requests, nine in ten short and the tenth very long: the largest
        case("skew_b512", "attend", B=512, **_GQA, lengths="skew_90_10"),
        # heads of 64 in groups of four, an ordinary batch
        case("gqa_d64_b128", "step", B=128, Hq=32, Hkv=8, d=64, lengths="lognormal_1500_16_8192"),
        # pages of 64 tokens, lse asked for, an odd batch
        case("page64_b75", "step", B=75, **_GQA, lengths="lognormal_1500_16_8192", page=64, out="f32", lse=True),
    ]


_MAX_TOKEN_BYTES = 3.0e9  # K + V a drawn case reads (the largest listed case reads 10.7e9)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["step", "attend", "layer", "table", "merge"], weights=[6, 3, 2, 2, 1])[0]
    if op == "merge":
        return {"op": op, **_BASE, "B": _log_int(rng, 1, 512), "Hq": rng.choice([8, 32, 40, 64]), "Hkv": 8,
                "d": rng.choice([64, 128, 128]), "parts": rng.randint(2, 9), "out": rng.choice(["bf16", "f32"]),
                "lse": rng.random() < 0.5}
    G = rng.choice([1, 2, 4, 4, 8])
    Hkv = rng.choice([4, 8, 8, 32] if G == 1 else [1, 2, 4, 8, 8])
    page = rng.choice([16, 16, 16, 32, 64])
    kind = rng.choice(["lognormal", "lognormal", "uniform", "pareto", "fixed"])
    mid = _log_int(rng, 100, 6000)
    lengths = {"lognormal": "lognormal_%d_16_%d" % (mid, min(8 * mid, 32768)), "uniform": "uniform_1_%d" % (2 * mid),
               "pareto": "pareto_1.5_%d_%d" % (max(mid // 4, 16), 32768), "fixed": "fixed_%d" % mid}[kind]
    case = {"op": op, **_BASE, "B": _log_int(rng, 1, 512), "Hq": G * Hkv, "Hkv": Hkv, "d": rng.choice([64, 128, 128, 128]),
            "lengths": lengths, "page": page, "cache": rng.choice(["bf16", "bf16", "fp8"]),
            "out": rng.choice(["bf16", "bf16", "f32"]), "lse": rng.random() < 0.3,
            "part": rng.choice([0, 256, 512, 512, 512, 1024])}
    if op == "table":
        case.update(layers=rng.randint(1, 4), interval=16, B=min(case["B"], 150))
        case["capacity"] = -(-case["B"] // 16) * 16 + 16 * rng.randint(0, 1)
    per_token = 2 * Hkv * case["d"] * (2 if case["cache"] == "bf16" else 1) * case.get("layers", 1)
    while case["B"] > 1 and int(_lengths(case).sum()) * per_token > _MAX_TOKEN_BYTES:
        case["B"] -= max(case["B"] // 10, 1)
    if op == "table":
        case["capacity"] = -(-case["B"] // 16) * 16 + 16 * rng.randint(0, 1)
    if rng.random() < 0.4 or op == "table":  # the bound a serving system passes instead of the batch's maximum
        case["bound"] = 1024 * -(-int(_lengths(case).max()) // 1024)
    return case


# ---- lengths, pages, values -----------------------------------------------------------------------

def _lengths(case):
    """Attended tokens of the case's requests (the new token included), ascending."""
    kind, *args = case["lengths"].split("_")
    B = case["B"]
    u = (np.arange(B) + 0.5) / B
    if kind == "fixed":
        L = np.full(B, int(args[0]))
    elif kind == "uniform":
        lo, hi = map(int, args)
        L = lo + np.floor(u * (hi - lo + 1))
    elif kind == "lognormal":
        median, lo, hi = map(int, args)
        z = np.array([statistics.NormalDist().inv_cdf(x) for x in u])
        L = np.clip(np.rint(median * np.exp(z)), lo, hi)
    elif kind == "pareto":
        alpha, lo, hi = float(args[0]), int(args[1]), int(args[2])
        L = np.clip(np.floor(lo * (1.0 - u) ** (-1.0 / alpha)), lo, hi)
    elif kind == "skew":
        long_ = max(B // 10, 1)
        L = np.concatenate([1 + np.floor(64 * (np.arange(B - long_) + 0.5) / max(B - long_, 1)),
                            32768 + np.floor(32769 * (np.arange(long_) + 0.5) / long_)])
    else:
        raise ValueError(kind)
    return L.astype(np.int64) + 1


def _bound(case):
    return case["bound"] or int(_lengths(case).max())


def _parts(case):
    """Partitions of each request of a merge case: parts - 2 .. parts + 2, at least one."""
    return np.maximum(case["parts"] - 2 + np.arange(case["B"]) % 5, 1)


class _Inputs:
    """Everything a case's calls take, from (case, seed) alone."""

    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed) * 7919 + 17)
        B, Hq, Hkv, d, page = case["B"], case["Hq"], case["Hkv"], case["d"], case["page"]
        L = rng.permutation(_lengths(case))
        need = -(-L // page)
        self.num_pages = int(1.5 * need.sum()) + 2
        width = -(-max(_bound(case), int(L.max())) // page)
        # physical pages of a request lie scattered over the pool; entries past its own name other pages
        ids = rng.permutation(self.num_pages)
        table = rng.integers(0, self.num_pages, size=(B, width))
        start = np.concatenate([[0], np.cumsum(need)])
        for b in range(B):
            table[b, :need[b]] = ids[start[b]:start[b + 1]]
        self.rows = case.get("capacity", B)
        pad = self.rows - B
        self.lens_host = np.concatenate([L, np.zeros(pad, dtype=np.int64)])
        self.table_host = np.concatenate([table, np.zeros((pad, width), dtype=np.int64)])
        self.table = torch.from_numpy(self.table_host.astype(np.int32)).cuda()
        self.lens = torch.from_numpy(self.lens_host.astype(np.int32)).cuda()
        self.q = self._randn(self.rows, Hq, d)
        self.k_new = self._randn(self.rows, Hkv, d)
        self.v_new = self._randn(self.rows, Hkv, d)
        self.caches = [self._cache(case) for _ in range(case.get("layers", 1))]
        self.order = torch.from_numpy(rng.permutation(2 * B)[:B].astype(np.int32)).cuda()  # places of the rows (layer)

    def _randn(self, *shape):
        return torch.randn(*shape, generator=self.gen, dtype=torch.bfloat16, device="cuda")

    def _cache(self, case):
        shape = (self.num_pages, case["page"], case["Hkv"], case["d"])
        if case["cache"] == "bf16":
            return adr.KVCache(self._randn(*shape), self._randn(*shape))
        both = []
        for _ in range(2):
            data = torch.empty(shape, dtype=torch.uint8, device="cuda")
            scale = torch.empty((shape[0], shape[2]), dtype=torch.float32, device="cuda")
            step = max(1, (1 << 28) // (shape[1] * shape[2] * shape[3]))
            for i in range(0, shape[0], step):
                x = self._randn(min(step, shape[0] - i), *shape[1:]).float()
                s = x.abs().amax(dim=(1, 3)) / 448.0
                scale[i:i + step] = s
                data[i:i + step] = (x / s[:, None, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
            both.append((data, scale))
        return adr.KVCache(both[0][0], both[1][0], both[0][1], both[1][1])


class _MergeInputs:
    def __init__(self, case, seed):
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed) * 7919 + 17)
        n = np.random.default_rng(seed).permutation(_parts(case))
        self.counts = n
        total = int(n.sum())
        self.o = torch.randn(total, case["Hq"], case["d"], generator=g, device="cuda")
        self.lse = 8.0 + torch.randn(total, case["Hq"], generator=g, device="cuda")
        self.offsets = torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int32)).cuda()


def _dtype(case):
    return torch.bfloat16 if case["out"] == "bf16" else torch.float32


class _State:
    def __init__(self, case):
        self.case, self.op, self.table = case, case["op"], None

    def __del__(self):
        if self.table is not None:
            self.table.destroy()


def prepare(case, seed):
    s = _State(case)
    B, Hq, Hkv, d = case["B"], case["Hq"], case["Hkv"], case["d"]
    if s.op == "merge":
        s.x = _MergeInputs(case, seed)
        rows = B
    else:
        s.x = x = _Inputs(case, seed)
        rows = x.rows
        s.bound, s.scale = _bound(case), 1.0 / math.sqrt(d)
        s.workspace = torch.empty(max(adr.adr_decode_workspace_bytes(rows, Hq, d, s.bound, case["part"]), 256),
                                  dtype=torch.uint8, device="cuda")
    s.out = torch.zeros((rows, Hq, d), dtype=_dtype(case), device="cuda")
    s.lse = torch.zeros((rows, Hq), dtype=torch.float32, device="cuda") if case["lse"] else None
    if s.op == "attend":
        s.positions = x.lens - 1
    if s.op == "layer":
        s.packed = torch.zeros((B, (Hq + 2 * Hkv) * d), dtype=torch.bfloat16, device="cuda")
        s.q = s.packed[:, :Hq * d].view(B, Hq, d)
        s.k_new = s.packed[:, Hq * d:(Hq + Hkv) * d].view(B, Hkv, d)
        s.v_new = s.packed[:, (Hq + Hkv) * d:].view(B, Hkv, d)
        s.out = torch.zeros((B, Hq, d), dtype=torch.bfloat16, device="cuda")  # the rows travel as bf16
        s.batch_out = torch.zeros((2 * B, Hq * d), dtype=torch.bfloat16, device="cuda")
    if s.op == "table":
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        s.table = adr.GraphTable(s.out, x.q, x.k_new, x.v_new, x.caches, x.table, x.lens, s.scale, s.bound,
                                 case["part"], s.workspace, case["interval"], x.rows, stream, lse=s.lse)
    return s


def run(s):
    x, part = s.x, s.case["part"]
    if s.op == "merge":
        adr.adr_lse_merge(s.out, x.o, x.lse, x.offsets, s.lse)
        return {"out": s.out, "lse": s.lse}
    cache = x.caches[0]
    if s.op == "step":
        adr.adr_decode_step(s.out, x.q, x.k_new, x.v_new, cache, x.table, x.lens, s.scale, s.bound, part, s.workspace,
                            s.lse)
    elif s.op == "attend":
        adr.adr_kv_append(cache, x.k_new, x.v_new, x.table, s.positions)
        adr.adr_decode_attention(s.out, x.q, cache, x.table, x.lens, s.scale, s.bound, part, s.workspace, s.lse)
    elif s.op == "layer":
        adr.adr_pack_qkv(s.packed, x.q, x.k_new, x.v_new)
        adr.adr_decode_step(s.out, s.q, s.k_new, s.v_new, cache, x.table, x.lens, s.scale, s.bound, part, s.workspace,
                            s.lse)
        adr.adr_scatter_rows(s.batch_out, s.out.view(s.out.shape[0], -1), x.order)
    else:
        s.table.launch(s.case["B"])
    return _outputs(s.out if s.op != "layer" else s.batch_out, s.lse, x.caches)


def _outputs(out, lse, caches):
    return {"out": out, "lse": lse, "caches": [[c.k, c.v, c.k_scale, c.v_scale] for c in caches]}


def work(case):
    B, Hq, Hkv, d = case["B"], case["Hq"], case["Hkv"], case["d"]
    out_bytes = B * Hq * (d * (2 if case["out"] == "bf16" or case["op"] == "layer" else 4) + (4 if case["lse"] else 0))
    if case["op"] == "merge":
        total = int(_parts(case).sum())
        return {"bytes": total * Hq * (d + 1) * 4 + 4 * (B + 1) + out_bytes, "flops": 2 * total * Hq * d}
    L, layers = _lengths(case), case.get("layers", 1)
    tokens, pages = int(L.sum()), int((-(-L // case["page"])).sum())
    kv = 2 * Hkv * (tokens * d * (2 if case["cache"] == "bf16" else 1) + (pages * 4 if case["cache"] == "fp8" else 0))
    new = 2 * B * Hkv * d * (2 + (2 if case["cache"] == "bf16" else 1))  # read, and written to the cache
    return {"bytes": layers * (kv + new + 4 * pages + 4 * B + B * Hq * d * 2 + out_bytes),
            "flops": layers * 4 * tokens * Hq * d}


def tolerance(case):
    # bf16 results are 1.7e-3 from the same in 64 bits (their rounding); two roundings of nearly equal numbers can
    # differ by a unit in the last place, 2^-8 to 2^-7 of the value.  fp32 results are 9e-6 from it (the weights
    # carry 16 bits).
    if case["out"] == "bf16" or case["op"] == "layer":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 4e-5, "max": 4e-4}


# ---- the same in 64 bits, in plain torch ----------------------------------------------------------------

def _append_exact(case, x, cache):
    rows = torch.from_numpy(np.nonzero(x.lens_host > 0)[0]).cuda()
    pos = torch.from_numpy(x.lens_host).cuda()[rows] - 1
    pages = torch.from_numpy(x.table_host).cuda()[rows, pos // case["page"]]
    slots = pos % case["page"]
    for data, new, scales in ((cache.k, x.k_new, cache.k_scale), (cache.v, x.v_new, cache.v_scale)):
        if case["cache"] == "bf16":
            data[pages, slots] = new[rows]
            continue
        v = new[rows].float()
        fresh = v.abs().amax(dim=2).clamp_min(2.0 ** -20) * (2.0 / 448.0)
        s = torch.where((slots == 0)[:, None], fresh, scales[pages])
        scales[pages] = s
        data[pages, slots] = (v * (1.0 / s)[:, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)


def _wide(data, scale, pages):
    """Pages of one cache as float64 [tokens, Hkv, d]."""
    if scale is None:
        v = data[pages].double()
    else:
        v = data[pages].view(torch.float8_e4m3fn).float().double() * scale[pages].double()[:, None, :, None]
    return v.reshape(-1, v.shape[2], v.shape[3])


def _attend_exact(case, x, cache):
    Hkv, d, page = case["Hkv"], case["d"], case["page"]
    G = case["Hq"] // Hkv
    out = torch.zeros((x.rows, case["Hq"], d), dtype=torch.float64, device="cuda")
    lse = torch.full((x.rows, case["Hq"]), -math.inf, dtype=torch.float64, device="cuda")
    table = x.table.long()
    for b in range(x.rows):
        L = int(x.lens_host[b])
        if not L:
            continue
        pages = table[b, :-(-L // page)]
        k = _wide(cache.k, cache.k_scale, pages)[:L].permute(1, 2, 0).contiguous()  # [Hkv, d, L]
        v = _wide(cache.v, cache.v_scale, pages)[:L].permute(1, 0, 2).contiguous()  # [Hkv, L, d]
        s = torch.matmul(x.q[b].double().view(Hkv, G, d), k) / math.sqrt(d)
        lse[b] = torch.logsumexp(s, dim=2).view(-1)
        out[b] = torch.matmul(torch.softmax(s, dim=2), v).view(-1, d)
    return out, lse


def exact(case, seed):
    if case["op"] == "merge":
        x = _MergeInputs(case, seed)
        B, n = case["B"], int(x.counts.max())
        at = x.offsets.long()[:-1, None] + torch.arange(n, device="cuda")[None]
        mine = torch.arange(n, device="cuda")[None] < torch.from_numpy(x.counts).cuda()[:, None]
        at = torch.where(mine, at, torch.zeros_like(at))
        ls = torch.where(mine[:, :, None], x.lse.double()[at], torch.full((), -math.inf, dtype=torch.float64, device="cuda"))
        out = (torch.softmax(ls, dim=1)[..., None] * x.o.double()[at]).sum(dim=1)
        return {"out": out, "lse": torch.logsumexp(ls, dim=1) if case["lse"] else None}
    x = _Inputs(case, seed)
    for cache in x.caches:
        _append_exact(case, x, cache)
    out, lse = _attend_exact(case, x, x.caches[-1])  # a table's layers share `out`: the last one's result stays
    if case["op"] == "layer":
        placed = torch.zeros((2 * case["B"], case["Hq"] * case["d"]), dtype=torch.float64, device="cuda")
        placed[x.order.long()] = out.view(case["B"], -1)
        out = placed
    return _outputs(out, lse if case["lse"] else None, x.caches)
