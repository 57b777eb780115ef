"""The work that a user of libburstattn has it do, as measurable cases.

Two families, as the library has two: the attention of one device on the ring (forward steps with their
online-softmax merge, D, backward steps) and the fused LM head + cross-entropy.  A case is a dict of
plain values:

  op "ring"     one device's pass over all KV shards.  direction "fwd", "bwd" or "train" (forward, then
                backward on its results).  aggregate "fused": the steps merge into the running state by
                themselves (ring.ring_forward); "merge": each step gives its own partial result (bf16) and
                the standalone merge folds it in, the last one also writing the bf16 copy.
  op "step"     one ring step alone: the local chunk against one visiting shard, as an outer loop that
                owns the communication calls it.
  op "lm_head"  one call over a device's tokens; entry "workspace" or "noalloc".

rows: tokens of a device's chunk; the sequence is rows * shards tokens long.
"""
import math

import torch

from paper_2509_19836_amd import binding as lib, ring, workloads as wl

PEAK_STATE_BYTES = 40e9      # inputs, buffers and results of a drawn case
MAX_DRAWN_FLOPS = 4.5e14     # just under the largest listed case


def _attn(name, **kw):
    case = dict(name=name, op="ring", direction="train", aggregate="fused", batch=1, q_heads=32, kv_heads=32,
                head_dim=128, rows=16384, shards=8, device=3, visiting=0, partition="zigzag", window=0, block_tokens=0,
                density=0.0, head_scale=False)
    case.update(kw)
    return case


def _lm(name, **kw):
    case = dict(name=name, op="lm_head", entry="workspace", tokens=16384, d_model=4096, vocab=32000, tile=8192,
                dh="bf16", grads=True)
    case.update(kw)
    return case


def listed():
    return [
        # the smallest ring of the benchmark definition: unit tests, toy models, debugging a distributed set-up
        _attn("ring_tiny_1k", q_heads=2, kv_heads=2, head_dim=64, rows=256, shards=4, device=1, partition="causal"),
        # fine-tuning at short context: several sequences, 64-wide heads, a chunk length that fits no tile
        _attn("ring_short_ragged", batch=4, q_heads=12, kv_heads=12, head_dim=64, rows=1500, shards=4, device=2,
              partition="causal"),
        # a head-parallel group in front of the ring leaves each device a few heads (64/8 heads over 4 devices)
        _attn("ring_few_heads", q_heads=16, kv_heads=2, rows=8192),
        # 128K tokens over 8 devices, the two directions on their own (inference prefill; backward of a
        # layer whose forward was checkpointed)
        _attn("ring_128k_fwd", direction="fwd"),
        _attn("ring_128k_bwd", direction="bwd"),
        # grouped-query attention at 256K tokens, one visiting shard
        _attn("step_gqa_256k", op="step", q_heads=64, kv_heads=8, rows=32768, device=5, visiting=2),
        # bidirectional attention over a batch, partial results merged by the standalone call
        _attn("ring_full_merge", direction="fwd", aggregate="merge", batch=2, rows=16384, shards=4, device=1,
              partition="full", head_scale=True),
        # the headline length: 1M tokens over 8 devices, one visiting shard
        _attn("step_1m", op="step", rows=131072, device=5, visiting=3),
        # sliding-window attention under the striped split
        _attn("ring_striped_window", partition="striped", window=32768),
        # block-wise sparse attention
        _attn("ring_block_sparse", density=0.25, block_tokens=512),
        # LM head + loss of a 128K-token sequence over 8 devices
        _lm("lm_head_16k"),
        # the entry point without a workspace argument: small sequence tiles, a ragged last one
        _lm("lm_head_noalloc_1k", entry="noalloc", tokens=1000, tile=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        if rng.random() < 0.3:
            entry = rng.choice(["workspace", "workspace", "noalloc"])
            case = _lm("", entry=entry, tokens=_log_int(rng, 64, 32768), d_model=256 * rng.choice([2, 3, 4, 8, 10, 16, 20]),
                       vocab=_log_int(rng, 8000, 130000 if entry == "workspace" else 40000),
                       tile=256 if entry == "noalloc" else 256 * rng.choice([4, 8, 16, 32]), dh=rng.choice(["bf16", "f32"]),
                       grads=rng.random() < 0.8)
            if entry == "noalloc":
                case["tokens"] = min(case["tokens"], 4096)
                if lib.burst_lm_head_workspace_bytes(_lm_shape(case)) > lib.burst_lm_head_static_scratch_bytes():
                    continue
        else:
            kv = rng.choice([1, 2, 4, 5, 8, 12, 16, 32])
            group = rng.choice([g for g in (1, 1, 2, 4, 8) if kv * g <= 64])
            partition = rng.choice(["full", "causal", "zigzag", "zigzag", "striped", "block_striped"])
            shards = rng.choice([1, 2, 4, 8])
            rows = _log_int(rng, 64, 131072)
            case = _attn("", op=rng.choice(["ring", "ring", "step"]), direction=rng.choice(["fwd", "bwd", "train", "train"]),
                         batch=rng.choice([1, 1, 2, 4]), q_heads=kv * group, kv_heads=kv, head_dim=rng.choice([64, 128, 128]),
                         rows=rows, shards=shards, device=rng.randrange(shards), partition=partition,
                         head_scale=rng.random() < 0.25)
            if case["direction"] == "fwd" and rng.random() < 0.3:
                case["aggregate"] = "merge"
            if partition == "zigzag":
                case["rows"] += rows & 1
                if rows >= 4096 and rng.random() < 0.25:      # block-sparse: pieces are whole blocks
                    case["block_tokens"] = 512 * rng.choice([1, 2])
                    case["rows"] = -(-rows // (2 * case["block_tokens"])) * 2 * case["block_tokens"]
                    case["density"] = rng.choice([0.1, 0.25, 0.5])
            elif partition == "block_striped":
                per = rng.choice([64, 256, 512])              # rows a device holds of each block
                case["block_tokens"] = per * shards
                case["rows"] = -(-rows // per) * per
            if partition != "full" and case["density"] == 0 and rows >= 1024 and rng.random() < 0.25:
                case["window"] = _log_int(rng, 256, rows * shards)
            # a visiting shard that every query row sees something of
            case["visiting"] = rng.randrange(case["device"] + 1)
            if case["op"] == "step" and (case["window"] or case["density"]):
                case["visiting"] = case["device"]
        w = work(case)
        if w["flops"] <= MAX_DRAWN_FLOPS and w["state"] <= PEAK_STATE_BYTES:
            del case["name"]
            return case


# ---- attention ---------------------------------------------------------------------------------------

def _order(case):
    return [case["visiting"]] if case["op"] == "step" else ring.ring_order(case["device"], case["shards"])


def _mask(case, j):
    return ring.fill_mask(case["partition"], case["device"], j, case["shards"], case["rows"] * case["shards"],
                          case["window"], case["block_tokens"])


def _pattern(case):
    """The global block pattern of a block-sparse model: part of the model, not of the data."""
    n = case["rows"] * case["shards"] // case["block_tokens"]
    return wl.block_sparse_pattern(n, case["density"], wl.BASE_SEED + 77)


def _block_mask(case, mask, pattern):
    pos = [ring.mask_positions(mask, side) for side in "qk"]
    return wl.local_block_mask(pattern, pos[0], pos[1], case["block_tokens"])


def _pairs(case):
    """Visible (query, key) pairs per head over the pass's steps."""
    pattern = _pattern(case) if case["density"] else None
    total = 0
    for j in _order(case):
        mask = _mask(case, j)
        if pattern is None:
            total += lib.burst_attn_visible_pairs(mask)
            continue
        R = case["block_tokens"]
        open_ = _block_mask(case, mask, pattern) != 0
        first_q, first_k = (ring.mask_positions(mask, side)[::R] for side in "qk")
        total += int((open_ & (first_q[:, None] > first_k[None, :])).sum()) * R * R
        total += int((open_ & (first_q[:, None] == first_k[None, :])).sum()) * R * (R + 1) // 2
    return total


def _prepare_attn(case, seed):
    B, n, Hq, Hkv, d = case["batch"], case["rows"], case["q_heads"], case["kv_heads"], case["head_dim"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    f32 = dict(device="cuda", dtype=torch.float32)

    def draw_tensor(heads, scaled=True):
        x = torch.randn(B, n, heads, d, generator=gen, **f32)
        if scaled and case["head_scale"]:
            x *= torch.empty(B, 1, heads, 1, **f32).uniform_(0.5, 2.0, generator=gen)
        return x.to(torch.bfloat16)

    order = _order(case)
    s = {"case": case, "order": order, "scale": d ** -0.5, "q": draw_tensor(Hq), "masks": {j: _mask(case, j) for j in order}}
    # shards that take no part in a single step are not in hand
    s["k"] = [draw_tensor(Hkv) if j in order else None for j in range(case["shards"])]
    s["v"] = [draw_tensor(Hkv) if j in order else None for j in range(case["shards"])]
    s["shape"] = lib.shape(B, Hq, Hkv, d, n, n, s["scale"])
    if case["density"]:
        pattern = _pattern(case)
        s["blocks"] = {j: torch.from_numpy(_block_mask(case, s["masks"][j], pattern)).cuda() for j in order}
        for j in order:
            lib.set_block_mask(s["masks"][j], s["blocks"][j], case["block_tokens"], case["block_tokens"])
    if case["direction"] != "bwd":
        s["o"], s["lse"] = torch.empty(B, n, Hq, d, **f32), torch.empty(B, Hq, n, **f32)
        if case["aggregate"] == "merge":
            s["o_part"] = torch.empty(B, n, Hq, d, device="cuda", dtype=torch.bfloat16)
            s["lse_part"] = torch.empty(B, Hq, n, **f32)
            s["o_cast"] = torch.empty(B, n, Hq, d, device="cuda", dtype=torch.bfloat16)
    else:
        # O and Lse of a forward pass over keys without structure: Lse about log(keys seen) + half the variance
        # of the scores, O about the mean of that many values
        seen = max(1.0, _pairs(case) / n)
        s["lse"] = math.log(seen) + 0.5 + 0.1 * torch.randn(B, Hq, n, generator=gen, **f32)
        s["o"] = torch.randn(B, n, Hq, d, generator=gen, **f32) * math.sqrt(math.e / (seen + math.e))
    if case["direction"] != "fwd":
        s["do"] = draw_tensor(Hq, scaled=False)
        s["d"] = torch.empty(B, Hq, n, **f32)
        s["dq"] = torch.empty(B, n, Hq, d, **f32)
        s["dk_all"], s["dv_all"] = (torch.empty(len(order), B, n, Hkv, d, **f32) for _ in range(2))
        at = {j: t for t, j in enumerate(order)}
        s["dk"] = [s["dk_all"][at[j]] if j in at else None for j in range(case["shards"])]
        s["dv"] = [s["dv_all"][at[j]] if j in at else None for j in range(case["shards"])]
    return s


def _forward(s):
    case = s["case"]
    s["o"].zero_()
    s["lse"].fill_(-math.inf)
    if case["aggregate"] == "merge":
        for j in s["order"]:
            lib.burst_attn_step_fwd(s["shape"], s["masks"][j], s["q"], s["k"][j], s["v"][j], o_part=s["o_part"],
                                    lse_part=s["lse_part"])
            lib.burst_attn_lse_merge(s["shape"], s["o"], s["lse"], s["o_part"], s["lse_part"],
                                     o_out_cast=s["o_cast"] if j == s["order"][-1] else None)
        return [s["o"], s["lse"], s["o_cast"]]
    if case["op"] == "ring" and not case["density"]:
        ring.ring_forward(case["device"], case["shards"], case["rows"] * case["shards"], case["partition"], s["scale"],
                          s["q"], s["k"], s["v"], s["o"], s["lse"], window=case["window"], N_blk=case["block_tokens"])
    else:
        for j in s["order"]:
            lib.burst_attn_step_fwd(s["shape"], s["masks"][j], s["q"], s["k"][j], s["v"][j], o_acc=s["o"], lse_acc=s["lse"])
    return [s["o"], s["lse"]]


def _backward(s):
    case = s["case"]
    if case["op"] == "step":      # gradients of this step alone: overwritten
        lib.burst_attn_preprocess_bwd(s["shape"], s["o"], s["do"], s["d"])
        j = s["order"][0]
        lib.burst_attn_step_bwd(s["shape"], s["masks"][j], s["q"], s["k"][j], s["v"][j], s["do"], s["lse"], s["d"],
                                dq=s["dq"], dk=s["dk"][j], dv=s["dv"][j])
    else:
        s["dq"].zero_()
        s["dk_all"].zero_()
        s["dv_all"].zero_()
        if case["density"]:
            lib.burst_attn_preprocess_bwd(s["shape"], s["o"], s["do"], s["d"])
            for j in s["order"]:
                lib.burst_attn_step_bwd(s["shape"], s["masks"][j], s["q"], s["k"][j], s["v"][j], s["do"], s["lse"], s["d"],
                                        dq=s["dq"], dk=s["dk"][j], dv=s["dv"][j],
                                        accumulate_flags=lib.BURST_ACC_DQ | lib.BURST_ACC_DK | lib.BURST_ACC_DV)
        else:
            ring.ring_backward(case["device"], case["shards"], case["rows"] * case["shards"], case["partition"], s["scale"],
                               s["q"], s["do"], s["o"], s["lse"], s["d"], s["k"], s["v"], s["dq"], s["dk"], s["dv"],
                               window=case["window"], N_blk=case["block_tokens"])
    return [s["d"], s["dq"], s["dk_all"], s["dv_all"]]


# ---- LM head -----------------------------------------------------------------------------------------

def _lm_shape(case):
    return lib.lm_head_shape(case["tokens"], case["d_model"], case["vocab"], case["tile"], 1.0 / case["tokens"])


def _prepare_lm(case, seed):
    N, d, v = case["tokens"], case["d_model"], case["vocab"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = {"case": case, "shape": _lm_shape(case)}
    s["h"] = torch.randn(N, d, device="cuda", generator=gen).to(torch.bfloat16)
    s["w"] = (torch.randn(v, d, device="cuda", generator=gen) * (2.0 / d ** 0.5)).to(torch.bfloat16)
    s["y"] = torch.randint(0, v, (N,), device="cuda", generator=gen)
    s["y"][: N // 50] = -100     # tokens without a loss (prompt, padding)
    s["loss"], s["lse"] = (torch.empty(N, device="cuda", dtype=torch.float32) for _ in range(2))
    s["dh"] = s["dw"] = None
    if case["grads"]:
        s["dh"] = torch.empty(N, d, device="cuda", dtype=torch.bfloat16 if case["dh"] == "bf16" else torch.float32)
        s["dw"] = torch.empty(v, d, device="cuda", dtype=torch.float32)
    if case["entry"] == "workspace":
        s["ws"] = torch.empty(lib.burst_lm_head_workspace_bytes(s["shape"]), dtype=torch.uint8, device="cuda")
    return s


def _run_lm(s):
    if s["case"]["entry"] == "workspace":
        lib.burst_lm_head_loss(s["shape"], s["h"], s["w"], s["y"], s["loss"], s["ws"], lse=s["lse"], d_h=s["dh"], d_w=s["dw"])
    else:
        lib.burst_lm_head_loss_noalloc(s["shape"], s["h"], s["w"], s["y"], s["loss"], lse=s["lse"], d_h=s["dh"], d_w=s["dw"])
    return [t for t in (s["loss"], s["lse"], s["dh"], s["dw"]) if t is not None]


# ---- what the measurement calls ----------------------------------------------------------------------

def prepare(case, seed):
    return (_prepare_lm if case["op"] == "lm_head" else _prepare_attn)(case, seed)


def run(state):
    case = state["case"]
    if case["op"] == "lm_head":
        return _run_lm(state)
    out = []
    if case["direction"] != "bwd":
        out += _forward(state)
    if case["direction"] != "fwd":
        out += _backward(state)
    return out


def work(case):
    """Bytes and floating-point operations of a pass (and the bytes a prepared state holds)."""
    if case["op"] == "lm_head":
        N, d, v = case["tokens"], case["d_model"], case["vocab"]
        nbytes = N * d * 2 + v * d * 2 + N * 8 + N * 8
        if case["grads"]:
            nbytes += N * d * (2 if case["dh"] == "bf16" else 4) + v * d * 4
        v_pad = (v + 255) // 256 * 256
        return {"bytes": nbytes, "flops": (6 if case["grads"] else 2) * N * d * v,
                "state": nbytes + (case["tile"] * v_pad * 6 if case["entry"] == "workspace" else 0)}
    B, n, Hq, Hkv, d = case["batch"], case["rows"], case["q_heads"], case["kv_heads"], case["head_dim"]
    fwd, bwd = case["direction"] != "bwd", case["direction"] != "fwd"
    q_el, kv_el, vec = B * n * Hq * d, len(_order(case)) * B * n * Hkv * d, B * n * Hq * 4
    nbytes = 2 * q_el + 2 * 2 * kv_el + 4 * q_el + vec           # q, k, v; O (written, or read by D) and Lse
    if case["aggregate"] == "merge":
        nbytes += 2 * q_el                                       # the bf16 copy
    if bwd:
        nbytes += 2 * q_el + vec + 4 * q_el + 2 * 4 * kv_el      # dO, D, dQ, dK, dV
    flops = _pairs(case) * B * Hq * d * ((4 if fwd else 0) + (10 if bwd else 0))
    return {"bytes": nbytes, "flops": flops, "state": nbytes + (2 * q_el + vec if case["aggregate"] == "merge" else 0)}


def tolerance(case):
    """About four times the error against the same path in 64 bits (at up to 4096 rows and 8000 words)."""
    if case["op"] == "lm_head":
        if not case["grads"]:
            return {"rel": 1e-5}                                  # fp32 sums: loss 5e-8, Lse 3e-8
        # dLogits is bf16 between two products (dH, dW 3.0e-4); a bf16 dH is rounded once more (1.7e-3)
        return {"rel": 6e-3 if case["dh"] == "bf16" else 1.2e-3}
    if case["direction"] == "fwd":
        # P is bf16 before the second product (O 1.6e-3); bf16 partial results add their own rounding (2.3e-3)
        return {"rel": 9e-3 if case["aggregate"] == "merge" else 6e-3}
    return {"rel": 1.2e-2}                                        # P and dS in bf16: dQ 1.7e-3, dV 2.5e-3, dK 3.0e-3 (4.0e-3 with head scales)
