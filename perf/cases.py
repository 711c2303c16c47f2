"""What this library is timed on: one rank's share of the fused communication + GEMM operators, called as a
program that serves or trains a tensor-parallel model calls them (the ctypes binding, buffers made once, a new
epoch per call, the peers emulated on the same GPU).

Ranges that the listed cases stand for and that `draw` takes its sizes from: 16 to 8192 tokens over 2, 4 or 8
ranks; AllGather-GEMM with bf16 operands in both weight layouts and with fp8 operands, 256 to 6656 local
columns, contractions of 1024 to 16384; GEMM-ReduceScatter and GEMM + AllReduce with 1024 to 16384 columns and
local contractions of 256 to 4096, plain or with the scatter fused into the stores, one-shot or two-shot; MoE
AllGather + grouped GEMM with the experts sharded over the ranks or all local; MoE down-projection +
ReduceScatter.  Rows per rank, columns and contractions are odd multiples of the smallest step as often as not.
"""
import math

import torch

from paper_2605_02953_amd import binding as B

_DENSE = dict(world=8, rank=0)


def listed():
    return [
        # the smallest call there is: two ranks, one 128-row shard each, 256 columns; launches and latency
        dict(_DENSE, name="ag_small_bf16", op="ag", dtype="bf16", layout="nk", world=2, m_per_rank=128, n=256, k=256),
        # one decode step of 64 sequences through a bf16 up-projection (70B-class share): streams the weight once
        dict(_DENSE, name="ag_decode_bf16", op="ag", dtype="bf16", layout="nk", m_per_rank=8, n=3584, k=8192),
        # one decode step of 128 sequences with fp8 weights and activations
        dict(_DENSE, name="ag_decode_fp8", op="ag", dtype="fp8", layout="nk", m_per_rank=16, n=8192, k=8192),
        # a 1024-token chunk of a chunked prefill, 72B-class share (3696 columns are not a whole number of tiles)
        dict(_DENSE, name="ag_chunk_bf16", op="ag", dtype="bf16", layout="nk", m_per_rank=128, n=3696, k=8192),
        # 8192-token prefill / training forward, 70B-class up-projection share: the headline workload
        dict(_DENSE, name="ag_prefill_bf16", op="ag", dtype="bf16", layout="nk", m_per_rank=1024, n=3584, k=8192),
        # the same operator on ragged shards with the weight stored [k, n] (a backward pass, a foreign checkpoint)
        dict(_DENSE, name="ag_prefill_bf16_kn", op="ag", dtype="bf16", layout="kn", m_per_rank=997, n=3584, k=8192),
        # the headline sizes with fp8 operands
        dict(_DENSE, name="ag_prefill_fp8", op="ag", dtype="fp8", layout="nk", m_per_rank=1024, n=3584, k=8192),
        # one decode step of 128 sequences through the matching down-projection
        dict(_DENSE, name="rs_decode_bf16", op="rs", layout="nk", m_per_rank=16, n=8192, k=3584, chunks=1, form="plain"),
        # 8192-token prefill / training forward, down-projection + reduce-scatter, four row chunks per peer block
        dict(_DENSE, name="rs_prefill_bf16", op="rs", layout="nk", m_per_rank=1024, n=8192, k=3584, chunks=4, form="plain"),
        # the same GEMM with the all-reduce that a model without sequence parallelism needs
        dict(_DENSE, name="ar_prefill_bf16", op="ar", layout="nk", m_per_rank=1024, n=8192, k=3584, form="one"),
        # MoE up-projection with the experts sharded: 8192 tokens, top-2 of 64 experts, eight of them here
        dict(_DENSE, name="moe_ag", op="moe_ag", layout="nk", m_per_rank=1024, hidden=4096, inter=1536, experts=64, local=8, top_k=2),
        # MoE down-projection + reduce-scatter, every expert's slice of the intermediate size on the rank
        dict(_DENSE, name="moe_rs", op="moe_rs", layout="nk", m_per_rank=1024, hidden=2048, inter=192, experts=32, local=32, top_k=2, chunks=4),
    ]


# ------------------------------------------------------------------------------------------------ more cases
_MOST = {"ag": (4.9e11, 0.5e9), "rs": (4.9e11, 0.75e9), "ar": (4.9e11, 1.35e9), "moe_ag": (4.0e11, 0.45e9), "moe_rs": (4.0e11, 0.35e9)}


def _spread(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread over the logarithm."""
    return max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step) * step)


def _chunks(rng, rows):
    c = rng.choice([1, 2, 4])
    return c if rows % c == 0 else 1


def draw(rng):
    op = rng.choice(["ag", "ag", "ag", "ag", "rs", "rs", "ar", "ar", "moe_ag", "moe_rs"])
    while True:
        world = rng.choice([2, 4, 8, 8])
        m_per_rank = max(1, _spread(rng, 16, 8192) // world)
        case = dict(op=op, world=world, rank=rng.randrange(world), m_per_rank=m_per_rank, layout=rng.choice(["nk", "nk", "nk", "kn"]))
        if op == "ag":
            case.update(dtype=rng.choice(["bf16", "bf16", "fp8"]), n=_spread(rng, 256, 6656, 8), k=_spread(rng, 1024, 16384, 16))
            if case["dtype"] == "fp8":
                case["layout"] = "nk"     # the only one fp8 has
        elif op in ("rs", "ar"):
            case.update(n=_spread(rng, 1024, 16384, 8), k=_spread(rng, 256, 4096, 8))
            if op == "rs":
                case.update(chunks=_chunks(rng, m_per_rank), form=rng.choice(["plain", "plain", "fused"]))
            else:
                case["form"] = rng.choice(["one", "two"])
        else:
            experts = rng.choice([8, 16, 32, 60, 64])
            case.update(experts=experts, top_k=rng.choice([1, 2, 2, 4, 6]), hidden=_spread(rng, 1024, 8192, 8),
                        inter=_spread(rng, 128, 2048, 8))
            sharded = op == "moe_ag" and experts % world == 0 and rng.random() < 0.5
            case["local"] = experts // world if sharded else experts
            if op == "moe_rs":
                case.update(inter=max(64, case["inter"] // 64 * 8), chunks=_chunks(rng, m_per_rank))
        w = work(case)
        if w["flops"] <= _MOST[op][0] and w["bytes"] <= _MOST[op][1]:
            return case


# ------------------------------------------------------------------------------------------------ work
def _rows(case):
    """Rows that uniform routing sends to the local experts."""
    return case["world"] * case["m_per_rank"] * case["top_k"] * case["local"] // case["experts"]


def work(case):
    op, world, m_r = case["op"], case["world"], case["m_per_rank"]
    m = world * m_r
    if op == "ag":
        n, k, e = case["n"], case["k"], 1 if case["dtype"] == "fp8" else 2
        # the shards in, the gathered operand out, the weight in, the product out
        return {"bytes": e * (2 * m * k + n * k) + 2 * m * n, "flops": 2 * m * n * k}
    if op in ("rs", "ar"):
        n, k = case["n"], case["k"]
        own = 2 * (m * k + n * k + m * n)          # operands in, this rank's partial out
        if op == "rs":                             # the peers' blocks in and delivered, the reduced block out
            return {"bytes": own + 2 * (2 * (world - 1) + 1) * m_r * n, "flops": 2 * m * n * k}
        if case["form"] == "one":                  # every peer's partial in, the sum out
            return {"bytes": own + 2 * world * m * n, "flops": 2 * m * n * k}
        # the owned tiles of every peer's partial in and of every output out, the other tiles in and delivered
        share = m * n // world
        return {"bytes": own + 2 * (2 * world - 1) * share + 4 * (world - 1) * share, "flops": 2 * m * n * k}
    rows, hidden, inter, local = _rows(case), case["hidden"], case["inter"], case["local"]
    flops = 2 * rows * hidden * inter
    if op == "moe_ag":                             # tokens in and gathered, weights in, rows out, ids in
        return {"bytes": 4 * m * hidden + 2 * local * hidden * inter + 2 * rows * inter + 4 * m * case["top_k"], "flops": flops}
    # rows and weights in, the combined partial out, the peers' blocks in and delivered, the reduced block out
    return {"bytes": 2 * (rows * inter + local * hidden * inter + m * hidden + (2 * (world - 1) + 1) * m_r * hidden), "flops": flops}


def tolerance(case):
    """Outputs are bf16 after fp32 sums.  Four times what the listed cases measure against the same sums in 64 bits: the
    2-norm of the difference is 1.66e-3 to 1.76e-3 of the result's, which is one rounding to bf16; the largest difference
    is half a bf16 step (3.9e-3 of the value), and 5.2e-3 to 8.0e-3 where a bf16 partial is summed again (reduce-scatter,
    all-reduce, combine).  Gathered operands, counts, offsets and indices are whole numbers and stay as they are."""
    return {"rel": 7e-3, "max": 1.6e-2 if case["op"] in ("ag", "moe_ag") else 3.2e-2, "differ": 0.0}


# ------------------------------------------------------------------------------------------------ inputs
def _bf16(g, shape, std=1.0):
    x = torch.randn(shape, device="cuda", generator=g)
    return (x * std if std != 1.0 else x).to(torch.bfloat16)


def _fp8(g, shape, std, dim):
    """(e4m3 bytes, scales): N(0, std^2) over amax / 448, the amax taken over `dim` (None: the whole tensor)."""
    x = torch.randn(shape, device="cuda", generator=g) * std
    scale = (x.abs().amax() if dim is None else x.abs().amax(dim=dim, keepdim=True)) / 448.0
    q = (x / scale).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return q, scale.reshape(-1).float()


def _zeros(shape, dtype=torch.int32):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def _ok(status):
    if status != B.OK:
        raise RuntimeError(B.status_string(status))


def _routing(g, tokens, experts, top_k):
    """top_k distinct experts per token, uniformly: the first top_k of a random order."""
    return torch.rand((tokens, experts), device="cuda", generator=g).argsort(dim=1)[:, :top_k].to(torch.int32).contiguous()


def _weights(g, lead, rows, cols, layout, std):
    """A weight [.., k = cols, n = rows], stored [.., n, k] or [.., k, n]."""
    return _bf16(g, lead + ((rows, cols) if layout == "nk" else (cols, rows)), std)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    s = dict(case, epoch=0, b_layout=B.B_NK if case["layout"] == "nk" else B.B_KN, status=_zeros(B.STATUS_WORDS))
    world, rank, m_r = case["world"], case["rank"], case["m_per_rank"]
    m = world * m_r
    peers = lambda shape: [None if r == rank else _bf16(g, shape) for r in range(world)]   # noqa: E731
    if case["op"] == "ag":
        n, k, fp8 = case["n"], case["k"], case["dtype"] == "fp8"
        s["dt"] = B.FP8_E4M3 if fp8 else B.BF16
        s["a_scales"] = s["b_scales"] = None
        if fp8:
            quantised = [_fp8(g, (m_r, k), 1.0, None) for _ in range(world)]
            s["shards"] = [q for q, _ in quantised]
            s["a_scales"] = torch.cat([sc for _, sc in quantised]).contiguous()
            s["b"], s["b_scales"] = _fp8(g, (n, k), k ** -0.5, 1)
        else:
            s["shards"] = [_bf16(g, (m_r, k)) for _ in range(world)]
            s["b"] = _weights(g, (), n, k, case["layout"], k ** -0.5)
        # zero-filled once: decode-shaped problems exchange partial tiles behind the gathered operand
        s["workspace"] = _zeros(B.ag_gemm_workspace_bytes(m_r, n, k, world, s["dt"], s["b_layout"]), torch.uint8)
        s["gathered"] = s["workspace"][:m * k * (1 if fp8 else 2)].view(m, -1)
        s["signals"] = _zeros(B.signal_words(world, 1))
        s["c"] = _zeros((m, n), torch.bfloat16)
        if m <= 256:   # a decode loop marshals its call once and advances the epoch
            s["call"] = B.PreparedAgGemm(s["shards"], s["b"], s["b_layout"], s["c"], s["a_scales"], s["b_scales"], s["workspace"],
                                         s["signals"], s["status"], None, None, m_r, n, k, world, rank, s["dt"], B.EMULATE_PRODUCER)
    elif case["op"] in ("rs", "ar"):
        n, k = case["n"], case["k"]
        s["a"] = _bf16(g, (m, k))
        s["b"] = _weights(g, (), n, k, case["layout"], k ** -0.5)
        s["gemm_out"] = _zeros((m, n), torch.bfloat16)
        if case["op"] == "rs":
            s["peers"] = peers((m_r, n))
            s["signals"] = _zeros(B.signal_words(world, case["chunks"]))
            s["scatter"] = _zeros((world, m_r, n), torch.bfloat16)
            s["out"] = _zeros((m_r, n), torch.bfloat16)
            if case["form"] == "fused":   # the other ranks' buffers
                s["dsts"] = [s["scatter"] if r == rank else _zeros((world, m_r, n), torch.bfloat16) for r in range(world)]
        else:
            s["peers"] = peers((m, n))
            st, tiles = B.tile_config(3, m, n, k)
            _ok(st)
            s["signals"] = _zeros(B.signal_words(world, tiles["ntiles"]))
            s["out"] = _zeros((m, n), torch.bfloat16)
            if case["form"] == "two":     # the other ranks' outputs, and what they broadcast
                s["outs"] = [s["out"] if r == rank else _zeros((m, n), torch.bfloat16) for r in range(world)]
                s["reduced"] = peers((m, n))
    else:
        hidden, inter, experts, local, top_k = (case[x] for x in ("hidden", "inter", "experts", "local", "top_k"))
        assignments = m * top_k
        # room for twice the even share of the assignments, as a capacity factor of two gives
        max_rows = s["max_rows"] = min(assignments, 2 * _rows(case) + 256)
        ids = _routing(g, m, experts, top_k)
        s["records"] = _zeros(1 + 5 * B.moe_max_tiles(max_rows, local))
        if case["op"] == "moe_ag":
            s["begin"] = rank * local if local < experts else 0
            s["ids"] = ids
            s["shards"] = [_bf16(g, (m_r, hidden)) for _ in range(world)]
            s["w"] = _weights(g, (local,), inter, hidden, case["layout"], hidden ** -0.5)
            s["workspace"] = _zeros(B.moe_workspace_bytes(m_r, hidden, world), torch.uint8)
            s["gathered"] = s["workspace"][:m * hidden * 2].view(m, -1)
            s["y"] = _zeros((max_rows, inter), torch.bfloat16)
            s["counts"] = _zeros((world, experts))
            s["offsets"] = _zeros(local + 1)
            s["gather"] = _zeros(max_rows) - 1
            s["signals"] = _zeros(B.signal_words(world, 1))
        else:
            flat = ids.reshape(-1).long()
            # the assignments grouped by expert: what the AllGather + grouped GEMM before it leaves behind
            s["gather"] = torch.sort(flat, stable=True).indices.to(torch.int32).contiguous()
            s["offsets"] = _zeros(experts + 1)
            s["offsets"][1:] = torch.bincount(flat, minlength=experts).cumsum(0).to(torch.int32)
            s["gate"] = torch.rand(assignments, device="cuda", generator=g)
            s["h"] = _bf16(g, (max_rows, inter))
            s["w"] = _weights(g, (local,), hidden, inter, case["layout"], (inter * world) ** -0.5)
            s["y"] = _zeros((max_rows, hidden), torch.bfloat16)
            s["inverse"] = _zeros(assignments)
            s["combined"] = _zeros((m, hidden), torch.bfloat16)
            s["peers"] = peers((m_r, hidden))
            s["scatter"] = _zeros((world, m_r, hidden), torch.bfloat16)
            s["out"] = _zeros((m_r, hidden), torch.bfloat16)
            s["signals"] = _zeros(B.signal_words(world, case["chunks"]))
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    s["epoch"] += 1
    op, world, rank, m_r, mode = s["op"], s["world"], s["rank"], s["m_per_rank"], B.EMULATE_PRODUCER
    m = world * m_r
    if op == "ag":
        if "call" in s:
            _ok(s["call"](s["epoch"]))
        else:
            _ok(B.ag_gemm(s["shards"], s["b"], s["b_layout"], s["c"], s["a_scales"], s["b_scales"], s["workspace"], s["signals"],
                          s["status"], None, None, m_r, s["n"], s["k"], world, rank, s["dt"], s["epoch"], mode))
        return s["c"], s["gathered"]
    if op == "rs":
        if s["form"] == "fused":
            _ok(B.gemm_rs_fuse_scatter(s["a"], s["b"], s["b_layout"], s["dsts"], s["peers"], s["out"], s["signals"], s["status"], None,
                                       None, m, s["n"], s["k"], world, rank, s["chunks"], s["epoch"], mode))
            return s["out"], s["dsts"]
        _ok(B.gemm_rs(s["a"], s["b"], s["b_layout"], s["gemm_out"], s["peers"], s["scatter"], s["out"], s["signals"], s["status"],
                      None, None, m, s["n"], s["k"], world, rank, s["chunks"], s["epoch"], mode))
        return s["out"], s["gemm_out"], s["scatter"]
    if op == "ar":
        if s["form"] == "two":
            _ok(B.gemm_ar_two_shot(s["a"], s["b"], s["b_layout"], s["gemm_out"], s["peers"], s["outs"], s["reduced"], s["signals"],
                                   s["status"], None, m, s["n"], s["k"], world, rank, s["epoch"], mode))
            # of the other ranks' outputs the call writes the tiles this rank owns, and which those are is the tiling's affair
            return s["out"], s["gemm_out"]
        _ok(B.gemm_ar(s["a"], s["b"], s["b_layout"], s["gemm_out"], s["peers"], s["out"], s["signals"], s["status"], None, m, s["n"],
                      s["k"], world, rank, s["epoch"], mode))
        return s["out"], s["gemm_out"]
    if op == "moe_ag":
        _ok(B.moe_ag_grouped_gemm(s["shards"], s["ids"], s["w"], s["b_layout"], s["y"], s["counts"], s["offsets"], s["gather"],
                                  s["records"], s["workspace"], s["signals"], s["status"], None, m_r, s["hidden"], s["inter"],
                                  s["experts"], s["top_k"], s["begin"], s["local"], s["max_rows"], world, rank, s["epoch"], mode))
        return s["y"], s["counts"], s["offsets"], s["gather"], s["gathered"]
    _ok(B.moe_grouped_gemm_rs(s["h"], s["w"], s["b_layout"], s["gate"], s["gather"], s["offsets"], s["y"], s["inverse"], s["records"],
                              s["combined"], s["peers"], s["scatter"], s["out"], s["signals"], s["status"], None, m_r, s["hidden"],
                              s["inter"], s["experts"], s["top_k"], s["local"], s["max_rows"], world, rank, s["chunks"], s["epoch"], mode))
    return s["out"], s["combined"], s["scatter"]
