"""The work whose speed is followed: passes through the public entry points over the sizes they are used at.

A case is a dict of plain values. `path` says which entry point it goes through:
  gather   all-gather -> GEMM (ficco_run): shards in a device staging buffer or in pinned host memory land in A_dev over
           the copy engines while the GEMM multiplies what has landed. `schedule`: "pick" = what the library's own rule
           answers for the shape and the place of the shards, "fused" = one launch per step over `chunks` pieces per shard
  scatter  GEMM -> reduce-scatter (ficco_run, FICCO_DIR_GEMM_RS): row blocks of C stream out to the peers' buffers
  reduce   the receiving half of a reduce-scatter (ficco_rs_reduce): the peers' partial blocks arrive and are added
  experts  expert-parallel dispatch -> grouped GEMM (ficco_plan_grouped): unequal token counts per pair of GPUs
  static   the GEMM that allocates nothing (ficco_gemm_static), operands in place, weight given anew with every call

The run of a plan ends with ficco_query_stats(), as a caller's step does: the transfers are not ordered behind the work
on any stream, so a caller knows only from it that the buffers may be written again and that no wait has expired.
ficco_gemm_static() is ordinary work on a stream and is not waited for.

The weight, the plan and the buffers are laid out once (prepare); inputs are N(0,1) activations and N(0,1/K) weights in
bf16, so that outputs have unit variance.
"""
import math
import random

import torch

import paper_2512_10236_amd as F

# The largest all-gather product listed below; drawn cases stay under it.
MOST_FLOPS = 2 * 65536 * 4096 * 14336
STATIC_WEIGHT = F.FICCO_STATIC_MAX_WEIGHT_BYTES


def listed():
    return [
        # latency: the smallest workload of the repository, 1 GFLOP over four shards
        dict(name="gather_tiny", path="gather", M=512, K=1024, N=1024, shards=4, source="device", schedule="pick", chunks=0),
        # QKV share of an 8B-class model at TP=8: bound by its transfers
        dict(name="gather_qkv", path="gather", M=8192, K=4096, N=768, shards=8, source="device", schedule="pick", chunks=0),
        # the same with the shards in pinned host memory: bound by the host link
        dict(name="gather_qkv_host", path="gather", M=8192, K=4096, N=768, shards=8, source="host", schedule="pick", chunks=0),
        # FFN-up share of a 70B-class model at TP=8, the benchmark's default: bound by the GEMM
        dict(name="gather_ffn", path="gather", M=16384, K=8192, N=3584, shards=8, source="device", schedule="pick", chunks=0),
        # row-parallel projection at a small token count (M <= K): column pieces, re-laid out by the sender
        dict(name="gather_proj", path="gather", M=4096, K=16384, N=4096, shards=8, source="device", schedule="pick", chunks=0),
        # the widest product of the repository's sweep
        dict(name="gather_wide", path="gather", M=65536, K=4096, N=14336, shards=8, source="device", schedule="pick", chunks=0),
        # odd token count, and column and k extents that fill no tile
        dict(name="gather_ragged", path="gather", M=8 * 371, K=2880, N=1160, shards=8, source="device", schedule="pick", chunks=0),
        # one launch per step, the paper's own schedule, at a shape of the sweep
        dict(name="gather_fused", path="gather", M=4096, K=8192, N=3584, shards=8, source="device", schedule="fused", chunks=2),
        # the backward's direction: output blocks leave for eight peers as they are completed
        dict(name="scatter_ffn", path="scatter", M=16384, K=3584, N=8192, shards=8),
        # ... and the receiving GPU's half of it: 2048 x 8192 partial blocks of eight GPUs
        dict(name="reduce_ffn", path="reduce", M=16384, N=8192, shards=8, chunks=1),
        # 16384 tokens from eight peers to two local experts
        dict(name="experts", path="experts", M=16384, K=4096, N=7168, shards=8, experts=2, chunks=4),
        # a decode step's few rows against a weight share, in a loop that may not allocate
        dict(name="static_decode", path="static", M=64, K=4096, N=768),
    ]


def _log(rng, low, high):
    return math.exp(rng.uniform(math.log(low), math.log(high)))


def _rows(rng, low, high):
    """A row count: any integer, or half of the time a multiple of 64."""
    n = int(_log(rng, low, high))
    return max(64, n // 64 * 64) if rng.random() < 0.5 else n


def _k(rng, low=512, high=16384):
    return max(1, int(_log(rng, low, high)) // 64) * 64


def _n(rng, low=256, high=14336):
    """A column count: a multiple of 8, or half of the time of 64."""
    step = rng.choice([8, 64])
    return max(step, int(_log(rng, low, high)) // step * step)


def draw(rng):
    while True:
        path = rng.choices(["gather", "fused", "host", "scatter", "reduce", "experts", "static"], [9, 2, 1, 2, 2, 2, 3])[0]
        G = rng.choice([2, 4, 8, 8])
        if path == "static":
            K = _k(rng, 512, 8192)
            N = min(_n(rng, 64, 4096), STATIC_WEIGHT // (2 * K) // 8 * 8)
            c = dict(path="static", M=_rows(rng, 1, 8192), K=K, N=N)
        elif path == "reduce":
            c = dict(path="reduce", M=G * _rows(rng, 64, 4096), N=_n(rng, 512, 14336), shards=G, chunks=1)
        elif path == "experts":
            E = rng.choice([1, 2, 4, 8])
            c = dict(path="experts", M=_rows(rng, 1024, 32768), K=_k(rng, 1024, 8192), N=_n(rng, 512, 8192), shards=G, experts=E,
                     chunks=rng.choice([1, 2, 4]))
        elif path == "scatter":
            c = dict(path="scatter", M=G * _rows(rng, 128, 4096), K=_k(rng), N=_n(rng, 512, 14336), shards=G)
        elif path == "fused":
            chunks = rng.choice([1, 2, 4])
            c = dict(path="gather", M=G * chunks * _rows(rng, 64, 1024), K=_k(rng), N=_n(rng), shards=G, source="device", schedule="fused", chunks=chunks)
        else:
            c = dict(path="gather", M=G * _rows(rng, 64, 8192), K=_k(rng), N=_n(rng), shards=G, source="host" if path == "host" else "device",
                     schedule="pick", chunks=0)
        flops, moved = work(c)["flops"], c["M"] * c.get("K", c["N"]) * 2
        if flops <= MOST_FLOPS and moved <= (1 << 27 if c.get("source") == "host" else 1 << 29) and c["M"] * c["N"] * 2 <= 65536 * 14336 * 2:
            return c


def work(case):
    """What a pass cannot do without: sources read, landing buffers written, weight read, outputs written."""
    M, N = case["M"], case["N"]
    if case["path"] == "reduce":
        G = case["shards"]
        block = M // G * N
        # G-1 partial blocks cross into the landing buffer; G blocks are added into one
        return {"bytes": 2 * block * (2 * (G - 1) + 2), "flops": (G - 1) * block}
    K = case["K"]
    a, w, c = 2 * M * K, 2 * K * N, 2 * M * N
    if case["path"] == "experts":
        w *= case["experts"]
    moved = {"gather": 2 * a + w + c, "experts": 2 * a + w + c, "scatter": a + w + 2 * c, "static": a + w + c}[case["path"]]
    return {"bytes": moved, "flops": 2 * M * N * K}


def tolerance(case):
    if case["path"] == "reduce":
        return "exact"            # fp32 sums in a stated order, one rounding
    # bf16 results of fp32 sums: where the sum lands near the middle of two bf16 values, another order of summation
    # rounds it the other way, one step of 2^-8 to 2^-7 of the value. Against 64-bit sums: rel 2.5e-5 (K = 1024) to
    # 5.9e-5 (K = 16384), max 0.0078.
    return {"rel": 3e-4, "max": 0.016}


_streams = []


def streams():
    """A compute stream and a copy stream for the whole program."""
    if not _streams:
        _streams.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    return _streams


class State:
    """The buffers and the plan of one caller."""
    plan = None

    def __del__(self):
        if self.plan is not None:
            F.ficco_destroy(self.plan)


def _normal(g, rows, cols, scale=1.0):
    out = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
    step = max(1, (1 << 27) // cols)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        out[r:r + n] = torch.randn((n, cols), generator=g, device="cuda") * scale
    return out


def _counts(seed, peers, experts, total):
    """[peers][experts] token counts that sum to `total`: log-normal shares, as a router's choices are uneven."""
    rng = random.Random(seed)
    w = [[rng.lognormvariate(0.0, 0.6) for _ in range(experts)] for _ in range(peers)]
    s = sum(map(sum, w))
    n = [[int(x / s * total) for x in row] for row in w]
    for i in range(total - sum(map(sum, n))):
        n[i % peers][i // peers % experts] += 1
    return n


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    st = State()
    st.case, path = case, case["path"]
    M, N, K, G = case["M"], case["N"], case.get("K", 0), case.get("shards", 1)
    st.cs, st.xs = streams()
    if path == "reduce":
        st.P_src = _normal(g, M, N)
        st.P_dev = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
        st.own = _normal(g, M // G, N)
        st.out = torch.empty((M // G, N), dtype=torch.bfloat16, device="cuda")
        st.plan = F.ficco_plan(M, 64, N, G, case["chunks"], F.FICCO_FINE_PERSISTENT)
        torch.cuda.synchronize()
        return st
    A = _normal(g, M, K)
    experts = case.get("experts", 1)
    st.W = _normal(g, experts * K, N, K ** -0.5)
    st.C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    if path == "static":
        st.A_dev = A
        torch.cuda.synchronize()
        return st
    if path == "scatter":
        st.A_dev = A
        st.peers = [torch.empty((M // G, N), dtype=torch.bfloat16, device="cuda") for _ in range(G)]
        schedule, chunks = F.ficco_pick_schedule_rs(M, K, N, G)
        st.plan = F.ficco_plan(M, K, N, G, chunks, schedule)
        F.ficco_plan_set(st.plan, F.FICCO_OPT_DIRECTION, F.FICCO_DIR_GEMM_RS)
    else:
        st.A_dev = torch.empty((M, K), dtype=torch.bfloat16, device="cuda")
        st.A_src = A
        if path == "experts":
            st.plan = F.ficco_plan_grouped(K, N, _counts(seed, G, experts, M), case["chunks"], F.FICCO_FINE_PERSISTENT)
        elif case["schedule"] == "fused":
            st.plan = F.ficco_plan(M, K, N, G, case["chunks"], F.FICCO_FINE_FUSED)
        elif case["source"] == "host":
            st.A_src = torch.empty((M, K), dtype=torch.bfloat16, pin_memory=True).copy_(A)
            schedule, chunks = F.ficco_pick_schedule_layout(M, K, N, G, F.FICCO_LAYOUT_ROW_MAJOR_HOST)
            st.plan = F.ficco_plan(M, K, N, G, chunks, schedule)
        else:
            st.plan = F.ficco_plan(M, K, N, G, 1, F.FICCO_AUTO_ANY)
    torch.cuda.synchronize()
    F.ficco_pack_weight(st.plan, st.W, st.cs)
    return st


def run(st):
    path = st.case["path"]
    if path == "static":
        F.ficco_gemm_static(st.case["M"], st.case["K"], st.case["N"], st.A_dev, st.W, st.C, st.cs)
        return st.C
    if path == "reduce":
        F.ficco_rs_reduce(st.plan, st.case["shards"] // 2, st.P_src, st.P_dev, st.own, st.out, st.cs)
        F.ficco_query_stats(st.plan)
        return {"out": st.out, "landed": st.P_dev}
    if path == "scatter":
        F.ficco_run(st.plan, None, st.A_dev, st.W, st.C, st.peers, st.cs, st.xs)
        F.ficco_query_stats(st.plan)
        return {"C": st.C, "peers": st.peers}
    F.ficco_run(st.plan, st.A_src, st.A_dev, st.W, st.C, None, st.cs, st.xs)
    F.ficco_query_stats(st.plan)
    return {"C": st.C, "landed": st.A_dev}
