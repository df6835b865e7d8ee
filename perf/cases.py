"""Performance cases of the signalled + reordered GEMM path: what a program that
uses this package has it do, through the package's public entry points.

Four kinds of call:
  run      fo.run_overlapped: signalling GEMM on one stream, consumers of the
           wave groups on a second one, then the post-reorder (a plan of one
           group runs on the GEMM stream alone);
  gemm     fo.gemm_signal_reorder by itself: plain row-major output without
           counters, or a reordered, signalled output (after the counter reset
           that a caller owes each launch);
  consume  fo.consume_group: one contiguous segment, summed with a peer's
           partial or copied, with or without a counter to wait for;
  post     fo.post_reorder: row-major restore, fused with bias and RMSNorm.

All sizes are in elements; A is [M, K], W is [N, K], both K contiguous.
"""
import math

import numpy as np
import torch

import paper_2504_19519_amd as fo

CUS = 256                     # compute units the plans are made for
XCDS, BAND = 8, 4             # chiplets and band height of the XCD dispatch order
EPS = 1e-6
MAX_FLOPS = 2.0 * 8192 * 8192 * 3584
MAX_OUT = 8192 * 8192

_DTYPE = {"fp16": torch.float16, "bf16": torch.bfloat16}


def listed():
    def run(name, M, N, K, dtype, tile, pattern, dests, groups, post="none", order="xcd", unit="waves"):
        return {"name": name, "kind": "run", "M": M, "N": N, "K": K, "dtype": dtype, "tile_m": tile[0],
                "tile_n": tile[1], "order": order, "pattern": pattern, "dests": dests, "unit": unit,
                "groups": groups, "post": post}

    return [
        # the smallest run: four groups of four 64x64 tiles, all launches and handoffs
        run("ar_256x256x256", 256, 256, 256, "fp16", (64, 64), "tile", 0, "4,4,4,4", order="rowmajor", unit="tiles"),
        # one decode step of the long-prefill layer below: 64 tokens, reading the weight once
        run("ar_norm_64x4096x3584", 64, 4096, 3584, "bf16", (64, 64), "tile", 0, "1", "bias+norm+gamma"),
        # row-parallel linear shard, AllReduce with one peer, a single wave of tiles
        run("ar_2048x4096x4096", 2048, 4096, 4096, "fp16", (256, 128), "tile", 0, "1"),
        # a prompt length and a hidden size that only the 64x64 tile divides, ReduceScatter over four
        run("rs_1216x2880x1984", 1216, 2880, 1984, "bf16", (64, 64), "subtile", 4, "1,1,1,1"),
        # MLP down-projection shard (hidden 8192, FFN 28672/8), ReduceScatter over four
        run("rs_8192x8192x3584", 8192, 8192, 3584, "fp16", (256, 256), "subtile", 4, "2,1,1"),
        # long prefill, AllReduce, restore fused with bias and RMSNorm
        run("ar_norm_16384x4096x3584", 16384, 4096, 3584, "bf16", (256, 256), "tile", 0, "1,1,1,1", "bias+norm+gamma"),
        # MoE output projection, All-to-All to eight ranks, restore fused with RMSNorm; the last wave is 3/4 full
        run("a2a_norm_4096x7168x2048", 4096, 7168, 2048, "fp16", (256, 256), "subtoken", 8, "1,1", "norm"),
        # the GEMM without communication: chunked prefill through a plain linear layer
        {"name": "gemm_768x3840x4160", "kind": "gemm", "M": 768, "N": 3840, "K": 4160, "dtype": "bf16",
         "tile_m": 64, "tile_n": 64, "order": "xcd", "pattern": "rowmajor", "dests": 0, "unit": "waves",
         "groups": "3", "signal": False},
        # one group's AllReduce / ReduceScatter stand-in on a segment of ragged length, counter reached
        {"name": "consume_sum_8388613", "kind": "consume", "len": 2048 * 4096 + 5, "dtype": "fp16", "sum": True,
         "wait": True},
        # the All-to-All stand-in's copy of a whole buffer
        {"name": "consume_copy_29360128", "kind": "consume", "len": 4096 * 7168, "dtype": "bf16", "sum": False,
         "wait": False},
        # the restore alone after a ReduceScatter
        {"name": "post_8192x8192", "kind": "post", "M": 8192, "N": 8192, "dtype": "fp16", "tile_m": 256,
         "tile_n": 256, "pattern": "subtile", "dests": 4, "post": "none"},
        # a wide residual stream after an All-to-All: rows too wide to be held in one wave's registers
        {"name": "post_norm_1280x12288", "kind": "post", "M": 1280, "N": 12288, "dtype": "bf16", "tile_m": 256,
         "tile_n": 128, "pattern": "subtoken", "dests": 8, "post": "bias+norm+gamma"},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _tile(M, N):
    """The tile a caller takes: the largest that divides the output and leaves
    most of the compute units a tile."""
    if M % 256 == 0 and N % 256 == 0 and M * N >= 192 * 256 * 256:
        return 256, 256
    if M % 256 == 0 and N % 128 == 0 and M * N >= 96 * 256 * 128:
        return 256, 128
    return 64, 64


def draw(rng):
    kind = rng.choice(["run", "run", "run", "gemm", "consume", "post"])
    dtype = rng.choice(["fp16", "bf16"])
    if kind == "consume":
        return {"kind": kind, "len": int(_log(rng, 1 << 12, MAX_OUT)), "dtype": dtype,
                "sum": rng.random() < 0.5, "wait": rng.random() < 0.5}
    while True:
        M, N, K = _log(rng, 64, 16384), _log(rng, 256, 14336 if kind == "post" else 8192), 64 * round(_log(rng, 4, 112))
        m, n = (256 if M >= 1024 and rng.random() < 0.75 else 64), rng.choice([64, 128, 256, 256])
        M, N = m * max(1, round(M / m)), n * max(1, round(N / n))
        if M * N <= MAX_OUT and 2.0 * M * N * K <= MAX_FLOPS:
            break
    tile_m, tile_n = _tile(M, N)
    pattern = rng.choice(["tile", "subtile", "subtoken"])
    post = rng.choice(["none", "norm", "norm+gamma", "bias+norm+gamma"])
    dests = rng.choice([2, 4, 8]) if pattern == "subtile" else rng.randint(2, 8) if pattern == "subtoken" else 0
    if kind == "post":
        return {"kind": kind, "M": M, "N": N, "dtype": dtype, "tile_m": tile_m, "tile_n": tile_n,
                "pattern": pattern, "dests": dests, "post": post}
    T = -(-(M // tile_m) * (N // tile_n) // CUS)
    P = min(T, 4)
    groups = ",".join(str(T * (j + 1) // P - T * j // P) for j in range(P))
    case = {"kind": kind, "M": M, "N": N, "K": K, "dtype": dtype, "tile_m": tile_m, "tile_n": tile_n,
            "order": "xcd", "pattern": pattern, "dests": dests, "unit": "waves", "groups": groups}
    if kind == "run":
        return dict(case, post=post)
    if rng.random() < 0.5:
        return dict(case, signal=True)
    return dict(case, pattern="rowmajor", dests=0, signal=False)


# ---- inputs ---------------------------------------------------------------

_STREAMS = []


def _streams():
    """The program's one pair of streams, shared by all of its layers."""
    if not _STREAMS:
        _STREAMS.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    return _STREAMS


class _Draws:
    """Values of one case's inputs, from the seed alone."""

    def __init__(self, case, seed):
        self.dtype = _DTYPE[case["dtype"]]
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def activations(self, *shape, scale=1.0):
        return (torch.randn(*shape, generator=self.gen, device="cuda", dtype=torch.float32) * scale).to(self.dtype)

    def uniform(self, n, lo, hi):
        return (torch.rand(n, generator=self.gen, device="cuda", dtype=torch.float32) * (hi - lo) + lo).to(self.dtype)


def _routing(case, seed):
    """(slice -> destination buffer, row -> destination rank): host tables."""
    rng = np.random.default_rng(seed)
    perm = rng.permutation(case["dests"]).astype(np.int32) if case["pattern"] == "subtile" else None
    bucket = rng.integers(0, case["dests"], case["M"]).astype(np.int32) if case["pattern"] == "subtoken" else None
    return perm, bucket


def _sizes(case):
    if case["kind"] == "post":      # the restore does not depend on the grouping: one group
        return [-(-(case["M"] // case["tile_m"]) * (case["N"] // case["tile_n"]) // CUS)], "waves"
    return [int(s) for s in case["groups"].split(",")], case["unit"]


def _plan(case, seed):
    perm, bucket = _routing(case, seed)
    sizes, unit = _sizes(case)
    return fo.plan_groups(case["M"], case["N"], case.get("K", 64), dtype=case["dtype"], tile_m=case["tile_m"],
                          tile_n=case["tile_n"], order=case.get("order", "xcd"), group_m=BAND, num_xcds=XCDS,
                          num_cus=CUS, pattern=case["pattern"], num_dest=case["dests"], dest_perm=perm,
                          row_bucket=bucket, sizes=sizes, unit=unit)


def _inputs(case, seed):
    """The call's input tensors."""
    d = _Draws(case, seed)
    x = {}
    if case["kind"] == "consume":
        x["src"] = d.activations(case["len"])
        x["peer"] = d.activations(case["len"]) if case["sum"] else None
        return x
    M, N = case["M"], case["N"]
    if case["kind"] == "post":
        x["src"] = d.activations(M * N)
    else:
        x["A"], x["W"] = d.activations(M, case["K"]), d.activations(N, case["K"], scale=case["K"] ** -0.5)
    if case["kind"] == "run":
        # the peer's partial arrives in the reordered layout; an All-to-All has none
        x["peer"] = d.activations(M * N) if case["pattern"] != "subtoken" else None
    if case["kind"] != "gemm":
        x["bias"] = d.uniform(N, -0.1, 0.1) if "bias" in case["post"] else None
        x["gamma"] = d.uniform(N, 0.5, 1.5) if "gamma" in case["post"] else None
    return x


def prepare(case, seed):
    s = _inputs(case, seed)
    s.update(case=case, streams=_streams())
    dtype = _DTYPE[case["dtype"]]
    if case["kind"] == "consume":
        s["dst"] = torch.empty(case["len"], dtype=dtype, device="cuda")
        s["counter"] = torch.full((1,), 16, dtype=torch.int32, device="cuda") if case["wait"] else None
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        return s
    plan = s["plan"] = _plan(case, seed)
    s["table"] = torch.empty(plan.device_bytes // 4 + 4, dtype=torch.int32, device="cuda")
    plan.to_device(s["table"])
    n = case["M"] * case["N"]
    if case["kind"] != "post":
        s["C"] = torch.empty(n, dtype=dtype, device="cuda")
        s["counters"] = torch.zeros(plan.num_counters, dtype=torch.int32, device="cuda")
    if case["kind"] != "gemm":
        s["out"] = torch.empty(case["M"], case["N"], dtype=dtype, device="cuda")
    if case["kind"] == "run":
        s["dst"] = torch.empty(plan.dest_elems, dtype=dtype, device="cuda")
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()      # the plan's table has been copied
    return s


def run(s):
    case, (gemm_stream, comm_stream) = s["case"], s["streams"]
    if case["kind"] == "consume":
        fo.consume_group(s["src"], s["peer"], s["dst"], case["len"], case["dtype"], s["counter"],
                         16 if case["wait"] else 0, s["status"], gemm_stream)
        return {"dst": s["dst"]}
    plan, table = s["plan"], s["table"]
    if case["kind"] == "gemm":
        counters = s["counters"] if case["signal"] else None
        if case["signal"]:
            fo.reset_counters(counters, plan.P, gemm_stream)
        fo.gemm_signal_reorder(plan, table, s["A"], s["W"], s["C"], counters, gemm_stream)
        return {"C": s["C"]}
    norm = "norm" in case["post"]
    if case["kind"] == "post":
        fo.post_reorder(plan, table, s["src"], s["out"], s["bias"], s["gamma"], EPS, norm, gemm_stream)
        return {"out": s["out"]}
    fo.run_overlapped(plan, table, s["A"], s["W"], s["C"], s["peer"], s["dst"], s["out"], s["bias"], s["gamma"],
                      EPS, norm, s["counters"], s["status"], gemm_stream, comm_stream)
    return {"C": s["C"], "dst": s["dst"], "out": s["out"]}


def work(case):
    if case["kind"] == "consume":
        n = case["len"]
        return {"bytes": 2.0 * n * (3 if case["sum"] else 2), "flops": float(n) if case["sum"] else 0.0}
    M, N, K = case["M"], case["N"], case.get("K", 0)
    vectors = 2.0 * N * (("bias" in case.get("post", "")) + ("gamma" in case.get("post", "")))
    if case["kind"] == "post":
        return {"bytes": 2.0 * 2 * M * N + vectors, "flops": 0.0}
    operands = 2.0 * (M * K + N * K)
    if case["kind"] == "gemm":
        return {"bytes": operands + 2.0 * M * N, "flops": 2.0 * M * N * K}
    peer = 0.0 if case["pattern"] == "subtoken" else 2.0 * M * N
    return {"bytes": operands + peer + vectors + 3 * 2.0 * M * N, "flops": 2.0 * M * N * K}


def tolerance(case):
    # data movement and one correctly rounded sum per element: one right answer
    if case["kind"] == "consume" or (case["kind"] == "post" and case["post"] == "none"):
        return "exact"
    # the 16-bit results of fp32 sums in another order: three to four times
    # the distance of a whole run from the 64-bit result (2.9e-4, 2.7e-3)
    return {"rel": 1e-3} if case["dtype"] == "fp16" else {"rel": 8e-3}


# ---- the same in 64 bits ---------------------------------------------------

def _slots(case):
    """Dispatch position (slot) of every tile, tiles numbered row-major."""
    rows, cols = case["M"] // case["tile_m"], case["N"] // case["tile_n"]
    tiles = rows * cols
    p = np.arange(tiles)
    if case.get("order", "xcd") == "rowmajor":
        return p
    share, rest = -(-tiles // XCDS), tiles % XCDS or XCDS
    x, i = p % XCDS, p // XCDS
    q = np.where(x < rest, x * share + i, rest * share + (x - rest) * (share - 1) + i)
    first = q // (BAND * cols) * BAND
    height = np.minimum(rows - first, BAND)
    r = q % (BAND * cols)
    slot = np.empty(tiles, np.int64)
    slot[(first + r % height) * cols + r // height] = p
    return slot


def _places(case, seed):
    """For every output element (row-major): its place in the GEMM's reordered
    output and in the consumer's buffer."""
    M, N, bm, bn = case["M"], case["N"], case["tile_m"], case["tile_n"]
    i = np.arange(M * N, dtype=np.int64).reshape(M, N) if case["pattern"] == "rowmajor" else None
    if i is not None:
        return (torch.from_numpy(i.reshape(-1)).cuda(),) * 2
    slots = _slots(case)
    cols, tiles = N // bn, len(slots)
    row = np.arange(M)
    r = row % bm
    slot = slots.reshape(M // bm, cols)[row // bm]                 # [M, cols]
    perm, bucket = _routing(case, seed)
    if case["pattern"] == "tile":
        piece = dest = (slot * bm + r[:, None]) * bn
    elif case["pattern"] == "subtile":
        sizes, unit = _sizes(case)
        first = np.concatenate([[0], np.cumsum(sizes)]) * (CUS if unit == "waves" else 1)
        first = np.minimum(first, tiles)
        g = np.searchsorted(first, slot, side="right") - 1
        h = bm // case["dests"]
        k, rr = (r // h)[:, None], (r % h)[:, None]
        begin, count = first[g], first[g + 1] - first[g]
        piece = begin * bm * bn + ((k * count + slot - begin) * h + rr) * bn
        dest = (perm[k].astype(np.int64) * tiles * h + slot * h + rr) * bn
    else:
        # subtokens of pool b: by slot, then by row
        D = case["dests"]
        onehot = np.eye(D, dtype=np.int64)[bucket].reshape(M // bm, bm, D)
        rank = (np.cumsum(onehot, axis=1) - onehot).reshape(M, D)[row, bucket]
        per_slot = np.empty((tiles, D), np.int64)
        per_slot[slots] = np.repeat(onehot.sum(axis=1), cols, axis=0)
        before = np.cumsum(per_slot, axis=0) - per_slot
        pool = np.concatenate([[0], np.cumsum(per_slot.sum(axis=0))])
        piece = dest = (pool[bucket][:, None] + before[slot, bucket[:, None]] + rank[:, None]) * bn
    c = torch.arange(bn, device="cuda")
    return [(torch.from_numpy(np.ascontiguousarray(v)).cuda()[:, :, None] + c).reshape(-1) for v in (piece, dest)]


def exact(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "consume":
        return {"dst": x["src"].double() + (x["peer"].double() if case["sum"] else 0.0)}
    M, N = case["M"], case["N"]
    piece, dest = _places(case, seed)

    def placed(values, at):
        out = torch.empty(M * N, dtype=torch.float64, device="cuda")
        out[at] = values.reshape(-1)
        return out

    res = {}
    if case["kind"] == "post":
        h = x["src"].double()[dest].reshape(M, N)
    else:
        h = x["A"].double() @ x["W"].double().t()
        res["C"] = placed(h, piece)
        if case["kind"] == "gemm":
            return res
        if x["peer"] is not None:
            h = h + x["peer"].double()[piece].reshape(M, N)
        res["dst"] = placed(h, dest)
    if x["bias"] is not None:
        h = h + x["bias"].double()
    if "norm" in case["post"]:
        h = h / torch.sqrt((h * h).mean(dim=1, keepdim=True) + EPS)
        if x["gamma"] is not None:
            h = h * x["gamma"].double()
    res["out"] = h
    return res
