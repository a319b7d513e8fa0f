"""Performance cases: the work a serving program has this library do, through the public entry points.

Four kinds of case:
  linear   one projection on RAW (unpacked) factors, ``deinfer_lowrank_linear``: fp32 pairs, and 16-bit
           pairs that were not packed;
  block    the four calls of one decoder block on packed factors, back to back on one stream:
           qkv (handing out the rank-space cache rows t_k, t_v), o, gate/up + SiLU, down (or, non-GLU,
           the two layers with bias and activation);
  tp_rank  what one rank of an 8-way tensor-parallel group runs for such a block: the two stages of
           every sub-layer as separate calls (the exchange between them is not part of the library);
  kv       keys and values of cached tokens rebuilt from the paged low-rank cache: table of rotary
           angles, compacting copies, upward projections (the keys with the rotary epilogue).

Everything a program keeps between steps (packed weights, workspace, output buffers, the block plan) is
made by prepare(); weights ~ N(0, 0.02) and activations ~ N(0, 1) as in the benchmark configurations.
"""
import math

import torch

import paper_2604_17709_amd as dn
import synth_inputs as si

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
BLOCK_TOKENS = 16        # tokens per block of the paged cache
HEAD_DIM = 128
MAX_FLOPS = 3.0e12       # a drawn case stays below the largest listed one
MAX_FLOPS_RAW = 1.2e10   # ... and a drawn RAW case takes no longer (fp32 arithmetic)


def _rank(m, n, keep):
    """floor(keep m n / (m + n)): the rank that keeps this fraction of a weight's parameters."""
    return max(1, (round(keep * 1e6) * m * n) // (1000000 * (m + n)))


def _block(name, shape, T, dtype="bf16", act="silu", kind="block"):
    s = si.BLOCKS[shape]
    return {"name": name, "kind": kind, "hidden": s.hidden, "ffn": s.ffn, "kv": s.kv_width,
            "keep": s.keep_num / s.keep_den, "act": act, "dtype": dtype, "T": T}


def listed():
    return [
        # the small fp32 projection (a first call from a test or a tiny model): latency of two launches
        {"name": "f32_linear_T16", "kind": "linear", "d_in": 512, "d_out": 512, "r": 64, "dtype": "f32", "T": 16},
        # an fp32 checkpoint run as it is: one 7B-sized attention projection over a ragged batch of tokens
        {"name": "f32_linear_T201", "kind": "linear", "d_in": 4096, "d_out": 4096, "r": 1638, "dtype": "f32", "T": 201},
        # one user, one token: the latency of a 7B-shaped block
        _block("7b_decode_T1", "llama7b_keep80", 1),
        # a full decode batch of the same block
        _block("7b_decode_T64", "llama7b_keep80", 64),
        # a ragged decode batch, fp16, a model without GLU (biases, ReLU)
        _block("opt30b_decode_T37_f16", "opt30b_keep60", 37, dtype="f16", act="relu"),
        # the largest decode batch of a 70B-shaped layer with grouped kv heads
        _block("70b_decode_T128", "llama70b_keep40", 128),
        # one of eight tensor-parallel ranks at the same batch: many small launches
        _block("70b_tp8_rank_T128", "llama70b_keep40", 128, kind="tp_rank"),
        # a chunk of a chunked prefill
        _block("7b_chunk_T512", "llama7b_keep60", 512),
        # prefill of 4 x 2048 tokens
        _block("7b_prefill_T8192", "llama7b_keep60", 8192),
        # 16 x 512 prefill tokens and 64 decode tokens in one step
        _block("13b_mixed_T8256", "llama13b_keep60", 8256),
        # prefill of a 70B-shaped layer
        _block("70b_prefill_T4096", "llama70b_keep40", 4096),
        # 16 sequences of 512 cached tokens each rebuilt before attention
        {"name": "7b_kv_rebuild_T8192", "kind": "kv", "hidden": 4096, "kv": 4096, "keep": 0.8, "dtype": "bf16", "seqs": 16, "blocks": 32},
    ]


# ------------------------------------------------------------------------------------- drawn cases
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng):
    if rng.random() < 0.5:
        s = si.BLOCKS[rng.choice(sorted(si.BLOCKS))]
        return {"hidden": s.hidden, "ffn": s.ffn, "kv": s.kv_width, "act": "silu" if s.glu else rng.choice(["relu", "gelu"])}
    hidden = _log_int(rng, 64, 1024) * 8
    ffn = int(hidden * rng.uniform(2.6, 4.0)) // 8 * 8
    return {"hidden": hidden, "ffn": ffn, "kv": max(8, hidden // rng.choice([1, 1, 4, 8]) // 8 * 8), "act": rng.choice(["silu", "silu", "silu", "relu", "gelu"])}


def draw(rng):
    u = rng.random()
    if u < 0.14:
        c = {"kind": "linear", "d_in": _log_int(rng, 64, 4096), "d_out": _log_int(rng, 64, 4096),
             "dtype": rng.choice(["f32", "f32", "bf16", "f16"]), "T": _log_int(rng, 1, 2048)}
        c["r"] = _rank(c["d_in"], c["d_out"], rng.uniform(0.2, 0.9))
        c["T"] = max(1, min(c["T"], int(MAX_FLOPS_RAW / (2 * c["r"] * (c["d_in"] + c["d_out"])))))
        return c
    if u < 0.27:
        kv = rng.choice([1024, 1024, 4096, 5120])
        seqs = rng.choice([1, 2, 4, 8, 16, 32])
        return {"kind": "kv", "hidden": rng.choice([4096, 5120, 8192]), "kv": kv, "keep": round(rng.uniform(0.3, 0.9), 3),
                "dtype": rng.choice(["bf16", "bf16", "f16"]), "seqs": seqs, "blocks": max(1, _log_int(rng, 4, 512) // seqs)}
    c = {"kind": "tp_rank" if u < 0.37 else "block", "keep": round(rng.uniform(0.3, 0.9), 3), "dtype": rng.choice(["bf16", "bf16", "bf16", "f16"]),
         "T": _log_int(rng, 1, 128) if u < 0.32 or 0.37 <= u < 0.72 else _log_int(rng, 129, 8256)}
    c.update(_draw_shape(rng))
    if c["kind"] == "tp_rank":          # (shards of an eighth: widths whose eighths are whole groups of 8 columns)
        c["hidden"], c["ffn"], c["kv"] = (max(64, c[n] // 64 * 64) for n in ("hidden", "ffn", "kv"))
        c["act"] = "silu"
    c["T"] = max(1, min(c["T"], int(MAX_FLOPS / _flops_per_token(c))))
    return c


# ------------------------------------------------------------------------------------- shapes
def _projections(c):
    h, f, kv = c["hidden"], c["ffn"], c["kv"]
    p = {"q": (h, h), "k": (h, kv), "v": (h, kv), "o": (h, h), "gate": (h, f), "up": (h, f), "down": (f, h)}
    if c["act"] != "silu":
        del p["up"]
    return p


def _ranks(c):
    return {n: _rank(m, w, c["keep"]) for n, (m, w) in _projections(c).items()}


def _flops_per_token(c):
    r = _ranks(c)
    if c["kind"] == "tp_rank":
        return sum(2 * (_share(r[n]) * m + r[n] * (w // 8)) if n not in ("o", "down") else 2 * r[n] * (m // 8 + w)
                   for n, (m, w) in _projections(c).items())
    return sum(2 * r[n] * (m + w) for n, (m, w) in _projections(c).items())


def _share(r):
    return -(-r // 8)


def _pad8(n):
    return (n + 7) // 8 * 8


# ------------------------------------------------------------------------------------- prepare
class _Maker:
    def __init__(self, case, seed):
        self.dtype = DTYPES[case["dtype"]]
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, *shape, std=1.0):
        return (torch.randn(shape, generator=self.gen, device="cuda") * std).to(self.dtype)

    def rows(self, T, width, std=1.0):
        """Rank-space rows: a pitch of whole 16-byte chunks."""
        t = torch.zeros((T, _pad8(width)), dtype=self.dtype, device="cuda")[:, :width]
        t.copy_(self.normal(T, width, std=std))
        return t

    def room(self, T, width):
        return torch.zeros((T, _pad8(width)), dtype=self.dtype, device="cuda")[:, :width]

    def empty(self, *shape):
        return torch.empty(shape, dtype=self.dtype, device="cuda")

    def packed(self, d_in, r, d_out, std=0.02):
        p = dn.deinfer_pack_factors(dn.raw_pair(self.normal(d_in, r, std=std), self.normal(r, d_out, std=std)))
        torch.cuda.current_stream().synchronize()        # the raw factors are freed on return
        return p


def prepare(case, seed):
    return {"linear": _prepare_linear, "block": _prepare_block, "tp_rank": _prepare_tp, "kv": _prepare_kv}[case["kind"]](case, _Maker(case, seed), seed)


def _prepare_linear(c, mk, seed):
    pair = dn.raw_pair(mk.normal(c["d_in"], c["r"], std=1 / math.sqrt(c["d_in"])), mk.normal(c["r"], c["d_out"], std=1 / math.sqrt(c["r"])))
    return {"kind": "linear", "x": mk.normal(c["T"], c["d_in"]), "pair": pair, "y": mk.empty(c["T"], c["d_out"]),
            "ws": dn.Workspace(dn.deinfer_workspace_bytes(c["T"], [pair]))}


def _prepare_block(c, mk, seed):
    T, proj, r = c["T"], _projections(c), _ranks(c)
    p = {n: mk.packed(m, r[n], w) for n, (m, w) in proj.items()}
    s = {"kind": "block", "act": c["act"], "p": p, "x": mk.normal(T, c["hidden"]), "a": mk.normal(T, c["hidden"]), "m": mk.normal(T, c["hidden"]),
         "qkv": tuple(mk.empty(T, proj[n][1]) for n in ("q", "k", "v")), "t_k": mk.room(T, r["k"]), "t_v": mk.room(T, r["v"]),
         "o": mk.empty(T, c["hidden"]), "h": mk.empty(T, c["ffn"]), "y": mk.empty(T, c["hidden"])}
    if c["act"] != "silu":
        s["b1"], s["b2"] = mk.normal(c["ffn"], std=0.02), mk.normal(c["hidden"], std=0.02)
    groups = [[p["q"], p["k"], p["v"]], [p["o"]], [p["gate"], p["up"]] if c["act"] == "silu" else [p["gate"]], [p["down"]]]
    s["ws"] = dn.Workspace(max(dn.deinfer_workspace_bytes(T, g) for g in groups))
    return s


def _prepare_tp(c, mk, seed):
    T, r = c["T"], _ranks(c)
    h, f, kv = c["hidden"], c["ffn"], c["kv"]
    down = {n: mk.packed(h, _share(r[n]), 16) for n in ("q", "k", "v", "gate", "up")}          # this rank's columns of U
    down.update(o=mk.packed(h // 8, r["o"], 16), down=mk.packed(f // 8, r["down"], 16))        # this rank's rows of U
    up = {n: mk.packed(16, r[n], w) for n, w in (("q", h // 8), ("k", kv // 8), ("v", kv // 8), ("gate", f // 8), ("up", f // 8), ("o", h), ("down", h))}
    s = {"kind": "tp_rank", "d": down, "u": up, "x": mk.normal(T, h), "m": mk.normal(T, h), "a": mk.normal(T, h // 8),
         "t": {n: mk.rows(T, r[n], std=0.3) for n in up},                                      # rank-space rows after the exchange
         "td": {n: mk.room(T, _share(r[n]) if n not in ("o", "down") else r[n]) for n in up},
         "y": {n: mk.empty(T, up[n].d_out) for n in ("q", "k", "v", "o", "down")}, "h": mk.empty(T, f // 8)}
    groups = [[down["q"], down["k"], down["v"]], [down["gate"], down["up"]], [down["o"]], [down["down"]], [up["gate"], up["up"]]] + [[up[n]] for n in up]
    s["ws"] = dn.Workspace(max(dn.deinfer_workspace_bytes(T, g) for g in groups))
    return s


def _prepare_kv(c, mk, seed):
    r = _rank(c["hidden"], c["kv"], c["keep"])
    n_blocks, pitch = c["seqs"] * c["blocks"], _pad8(r)
    T, n_pool = n_blocks * BLOCK_TOKENS, 2 * n_blocks
    prompt = c["blocks"] * 3 // 4        # prompts got their blocks in one go, the rest came one by one
    table, held = si.paged_block_tables(seed, [prompt] * c["seqs"], [c["blocks"] - prompt] * c["seqs"], n_pool, recycled=n_pool // 8)
    plan, _, positions = dn.deinfer_kv_compact_plan(table, held, n_pool, n_blocks, BLOCK_TOKENS)
    s = {"kind": "kv", "block_bytes": BLOCK_TOKENS * pitch * 2, "r": r, "plan": torch.from_numpy(plan).cuda(), "positions": torch.from_numpy(positions).cuda(),
         "table": torch.empty((T, HEAD_DIM), dtype=torch.float32, device="cuda")}
    for n in ("k", "v"):
        pool = torch.zeros((n_pool * BLOCK_TOKENS, pitch), dtype=mk.dtype, device="cuda")
        pool[:, :r] = mk.normal(n_pool * BLOCK_TOKENS, r)
        s[n] = {"pool": pool, "rows": torch.zeros((T, pitch), dtype=mk.dtype, device="cuda"), "pair": mk.packed(16, r, c["kv"]), "out": mk.empty(T, c["kv"])}
    s["ws"] = dn.Workspace(max(dn.deinfer_workspace_bytes(T, [s[n]["pair"]]) for n in ("k", "v")))
    return s


# ------------------------------------------------------------------------------------- run
def run(s):
    return {"linear": _run_linear, "block": _run_block, "tp_rank": _run_tp, "kv": _run_kv}[s["kind"]](s)


def _run_linear(s):
    return dn.deinfer_lowrank_linear(s["x"], s["pair"], s["ws"], out=s["y"])


def _run_block(s):
    p, ws = s["p"], s["ws"]
    dn.deinfer_lowrank_qkv(s["x"], p["q"], p["k"], p["v"], ws, out=s["qkv"], t_k=s["t_k"], t_v=s["t_v"])
    dn.deinfer_lowrank_linear(s["a"], p["o"], ws, out=s["o"])
    if s["act"] == "silu":
        dn.deinfer_lowrank_gateup_silu(s["m"], p["gate"], p["up"], ws, out=s["h"])
        dn.deinfer_lowrank_down(s["h"], p["down"], ws, out=s["y"])
    else:
        dn.deinfer_lowrank_linear_act(s["m"], p["gate"], ws, bias=s["b1"], act=dn.ACT_RELU if s["act"] == "relu" else dn.ACT_GELU, out=s["h"])
        dn.deinfer_lowrank_linear_act(s["h"], p["down"], ws, bias=s["b2"], act=dn.ACT_NONE, out=s["y"])
    return {"qkv": s["qkv"], "t_k": s["t_k"], "t_v": s["t_v"], "o": s["o"], "h": s["h"], "y": s["y"]}


def _run_tp(s):
    d, u, t, td, y, ws = s["d"], s["u"], s["t"], s["td"], s["y"], s["ws"]
    dn.deinfer_lowrank_down_proj(s["x"], [d["q"], d["k"], d["v"]], ws, t_out=[td["q"], td["k"], td["v"]])
    for n in ("q", "k", "v"):
        dn.deinfer_lowrank_up(t[n], u[n], ws, out=y[n])
    dn.deinfer_lowrank_down_proj(s["a"], [d["o"]], ws, t_out=[td["o"]])
    dn.deinfer_lowrank_up(t["o"], u["o"], ws, out=y["o"])
    dn.deinfer_lowrank_down_proj(s["m"], [d["gate"], d["up"]], ws, t_out=[td["gate"], td["up"]])
    dn.deinfer_lowrank_up_glu_silu(t["gate"], t["up"], u["gate"], u["up"], ws, out=s["h"])
    dn.deinfer_lowrank_down_proj(s["h"], [d["down"]], ws, t_out=[td["down"]])
    dn.deinfer_lowrank_up(t["down"], u["down"], ws, out=y["down"])
    return {"t": td, "y": y, "h": s["h"]}


def _run_kv(s):
    k, v, ws = s["k"], s["v"], s["ws"]
    dn.deinfer_rope_table(s["positions"], HEAD_DIM, table=s["table"])
    dn.deinfer_kv_compact_copy(k["pool"], s["block_bytes"], s["plan"], k["rows"])
    dn.deinfer_lowrank_up_rope(k["rows"][:, :s["r"]], k["pair"], s["table"], ws, out=k["out"])
    dn.deinfer_kv_compact_copy(v["pool"], s["block_bytes"], s["plan"], v["rows"])
    dn.deinfer_lowrank_up(v["rows"][:, :s["r"]], v["pair"], ws, out=v["out"])
    return {"table": s["table"], "k": k["out"], "v": v["out"], "k_rows": k["rows"], "v_rows": v["rows"]}


# ------------------------------------------------------------------------------------- work, tolerance
def work(c):
    """Every factor element, input and output once; a result of one call that is another call's input is read once more."""
    if c["kind"] == "linear":
        es = 4 if c["dtype"] == "f32" else 2
        w = c["r"] * (c["d_in"] + c["d_out"])
        return {"bytes": es * (w + c["T"] * (c["d_in"] + c["d_out"])), "flops": 2.0 * c["T"] * w}
    if c["kind"] == "kv":
        r = _rank(c["hidden"], c["kv"], c["keep"])
        T = c["seqs"] * c["blocks"] * BLOCK_TOKENS
        return {"bytes": 2 * (2 * r * c["kv"] + 3 * 2 * T * r + 2 * T * c["kv"]) + 2 * 4 * T * HEAD_DIM, "flops": 2.0 * T * 2 * r * c["kv"]}
    T, r = c["T"], _ranks(c)
    if c["kind"] == "tp_rank":
        w = _flops_per_token(c) // 2
        rows = sum(r.values()) + sum(_share(r[n]) if n not in ("o", "down") else r[n] for n in r)
        cols = 2 * c["hidden"] + c["hidden"] // 8 + (c["hidden"] + 2 * c["kv"]) // 8 + 2 * c["hidden"] + 2 * (c["ffn"] // 8)
        return {"bytes": 2 * (w + T * (rows + cols)), "flops": 2.0 * T * w}
    w = _flops_per_token(c) // 2
    cols = 3 * c["hidden"] + c["hidden"] + 2 * c["kv"] + r["k"] + r["v"] + 2 * c["hidden"] + 2 * c["ffn"]
    return {"bytes": 2 * (w + T * cols), "flops": 2.0 * T * w}


def tolerance(c):
    """About four times what each kind of case differs by from the same path in 64 bits (storage roundings kept where the
    interface has them), or from itself with its sums in another order."""
    if c["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 1.2e-2, "max": 0.15} if c["dtype"] == "bf16" else {"rel": 1.5e-3, "max": 0.02}
