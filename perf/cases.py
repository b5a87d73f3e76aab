"""The MoE layer calls whose speed this repository is judged by, and how to run each of them.

Every case is one ``ft_moe_forward`` (or ``ft_moe_forward_noalloc``) call of one MoE layer over a
GPU expert cache: routing, hit/miss split, grouped SwiGLU experts over the resident slots and the
combine.  The layers are the three the framework is configured for everywhere else (Qwen3-30B-A3B,
DeepSeek-V3 and DeepSeek-V4-Flash shapes; bf16, block-scaled fp8 and MXFP4 weights), at token
counts from a single decoding user to the largest prefill chunk, odd ones among them.
"""
from __future__ import annotations

import math

import torch

import paper_2608_16157_amd as ftm

BF16, FP8, MXFP4 = ftm.FT_DT_BF16, ftm.FT_DT_FP8E4M3FN_B128, ftm.FT_DT_MXFP4

# hidden, inter, experts, top-k, gating, weight type, shared expert
LAYERS = {
    "qwen3": (2048, 768, 128, 8, ftm.FT_GATE_SOFTMAX_TOPK_RENORM, BF16, False),
    "dsv3": (7168, 2048, 256, 8, ftm.FT_GATE_SIGMOID_TOPK_RENORM, FP8, True),
    "dsv4flash": (4096, 2048, 256, 6, ftm.FT_GATE_SIGMOID_TOPK_RENORM, MXFP4, False),
}
# (resident share of the experts, Zipf exponent of their popularity) in decode and in prefill, where
# the popularity of the DeepSeek layers is drawn anew every 1024 tokens
DECODE = {"qwen3": (0.5, 1.1), "dsv3": (0.25, 1.2), "dsv4flash": (0.25, 1.2)}
PREFILL = {"qwen3": (0.75, 0.0), "dsv3": (0.40, 1.2), "dsv4flash": (0.40, 1.2)}
SEGMENT = 1024
DECODE_MAX_TOKENS = 256   # larger calls are prompt chunks


def _case(layer, tokens, combine="ordered", act="exact", entry="forward", **kw):
    return {"layer": layer, "tokens": tokens, "combine": combine, "act": act, "entry": entry,
            "phase": "decode" if tokens <= DECODE_MAX_TOKENS else "prefill", **kw}


def listed():
    return [
        # one user decoding: four launches of a few microseconds each
        _case("qwen3", 1, name="qwen3_decode_1"),
        # an ordinary decode batch
        _case("qwen3", 32, name="qwen3_decode_32"),
        # a large continuous batch; the float32 atomic combine, for callers without need of
        # bit-reproducible sums
        _case("qwen3", 160, combine="atomic", name="qwen3_decode_160"),
        # a ragged prompt chunk, as chunked prefill hands them out
        _case("qwen3", 777, name="qwen3_chunk_777"),
        # a whole prompt
        _case("qwen3", 4096, name="qwen3_prefill_4096"),
        # decode batches of block-scaled fp8 experts with a shared expert
        _case("dsv3", 16, name="dsv3_decode_16"),
        _case("dsv3", 64, name="dsv3_decode_64"),
        # a short prompt chunk: many experts, few rows each
        _case("dsv3", 300, name="dsv3_chunk_300"),
        # the largest prompt chunk, and the default workload of bench.py
        _case("dsv3", 8192, name="dsv3_prefill_8192"),
        # the optional fp8-activation arithmetic
        _case("dsv3", 2048, act="fp8", name="dsv3_fp8act_2048"),
        # a few users decoding over MXFP4 experts, on the library's own scratch memory (the entry
        # point of serving loops that cannot allocate)
        _case("dsv4flash", 7, entry="noalloc", name="dsv4flash_decode_7"),
        # a ragged prompt chunk over MXFP4 experts
        _case("dsv4flash", 1500, name="dsv4flash_chunk_1500"),
    ]


def draw(rng):
    layer = rng.choice(sorted(LAYERS))
    tokens = min(8192, int(round(math.exp(rng.uniform(0.0, math.log(8192.0))))))
    act = "fp8" if layer == "dsv3" and rng.random() < 0.25 else "exact"
    combine = "atomic" if rng.random() < 0.25 else "ordered"
    return _case(layer, tokens, combine=combine, act=act)


# ------------------------------------------------------------------------------------- inputs

def _desc(case, n_slots, shared_slot):
    H, I, E, k, gating, wd, _ = LAYERS[case["layer"]]
    return dict(hidden=H, inter=I, n_experts=E, top_k=k, gating=gating, w_dtype=wd, x_dtype=BF16,
                n_slots=n_slots, shared_slot=shared_slot,
                combine=ftm.FT_COMBINE_ATOMIC if case["combine"] == "atomic" else ftm.FT_COMBINE_ORDERED,
                act_quant=ftm.FT_ACT_FP8_1x128_POW2 if case["act"] == "fp8" else ftm.FT_ACT_EXACT)


def _routing(case, g, device):
    """Router logits N(0, 1) - s ln(popularity rank) and the slot table: the most popular experts
    (of the first ranking) are resident, in random slots."""
    _, _, E, _, _, _, _ = LAYERS[case["layer"]]
    T = case["tokens"]
    frac, zipf = (DECODE if case["phase"] == "decode" else PREFILL)[case["layer"]]
    shifts = case["phase"] == "prefill" and zipf > 0
    n_seg = -(-T // SEGMENT) if shifts else 1
    perms = [torch.randperm(E, generator=g, device=device) for _ in range(n_seg)]
    n_res = int(frac * E + 1e-9)
    slots = torch.randperm(n_res, generator=g, device=device).to(torch.int32)
    slot_table = torch.full((E,), -1, dtype=torch.int32, device=device)
    slot_table[perms[0][:n_res]] = slots
    logits = torch.randn(T, E, generator=g, device=device)
    if zipf > 0:
        for s, p in enumerate(perms):
            bias = torch.empty(E, device=device)
            bias[p] = -zipf * torch.log(torch.arange(1, E + 1, dtype=torch.float32, device=device))
            logits[s * SEGMENT:(s + 1) * SEGMENT if n_seg > 1 else T] += bias
    return logits, slot_table, n_res


def _quant_fp8(w):
    """e4m3fn codes and one float32 scale (amax / 448) per 128 x 128 block."""
    r, c = w.shape
    blk = w.view(r // 128, 128, c // 128, 128)
    scale = blk.abs().amax(dim=(1, 3)) / 448.0
    q = (blk / scale[:, None, :, None]).clamp_(-448.0, 448.0)
    return q.view(r, c).to(torch.float8_e4m3fn).view(torch.uint8), scale


def _quant_mxfp4(w):
    """e2m1 code pairs (even element in the low nibble) and one e8m0 scale byte per 32 elements of
    a row, stored [C / 32][R]."""
    r, c = w.shape
    blk = w.view(r, c // 32, 32)
    byte = torch.floor(torch.log2(blk.abs().amax(dim=2))) - 2 + 127
    q = blk * torch.exp2(127 - byte)[:, :, None]
    a = q.abs()
    idx = ((a > 0.25).to(torch.uint8) + (a >= 0.75) + (a > 1.25) + (a >= 1.75) + (a > 2.5) + (a >= 3.5)
           + (a > 5))
    codes = (idx.to(torch.uint8) | (torch.signbit(q).to(torch.uint8) << 3)).view(r, c)
    return codes[:, 0::2] | (codes[:, 1::2] << 4), byte.to(torch.uint8).t()


def _banks(case, g, n_slots, device):
    """One expert per slot, weights N(0, 0.02) in the layer's format."""
    H, I, _, _, _, wd, _ = LAYERS[case["layer"]]
    kw = dict(device=device)
    if wd == BF16:
        b = {"w13": torch.empty(n_slots, 2 * I, H, dtype=torch.bfloat16, **kw),
             "w2": torch.empty(n_slots, H, I, dtype=torch.bfloat16, **kw), "s13": None, "s2": None}
    elif wd == FP8:
        b = {"w13": torch.empty(n_slots, 2 * I, H, dtype=torch.uint8, **kw),
             "w2": torch.empty(n_slots, H, I, dtype=torch.uint8, **kw),
             "s13": torch.empty(n_slots, 2 * I // 128, H // 128, **kw),
             "s2": torch.empty(n_slots, H // 128, I // 128, **kw)}
    else:
        b = {"w13": torch.empty(n_slots, 2 * I, H // 2, dtype=torch.uint8, **kw),
             "w2": torch.empty(n_slots, H, I // 2, dtype=torch.uint8, **kw),
             "s13": torch.empty(n_slots, H // 32, 2 * I, dtype=torch.uint8, **kw),
             "s2": torch.empty(n_slots, I // 32, H, dtype=torch.uint8, **kw)}
    for slot in range(n_slots):
        for w, s, rows, cols in (("w13", "s13", 2 * I, H), ("w2", "s2", H, I)):
            v = torch.randn(rows, cols, generator=g, **kw).mul_(0.02)
            if wd == BF16:
                b[w][slot] = v
            else:
                b[w][slot], b[s][slot] = (_quant_fp8 if wd == FP8 else _quant_mxfp4)(v)
    return b


def _inputs(case, seed):
    device = "cuda"
    H, _, _, _, _, _, shared = LAYERS[case["layer"]]
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    logits, slot_table, n_res = _routing(case, g, device)
    x = torch.randn(case["tokens"], H, generator=g, device=device).to(torch.bfloat16)
    n_slots = n_res + (1 if shared else 0)
    desc = _desc(case, n_slots, n_res if shared else -1)
    return desc, _banks(case, g, n_slots, device), logits, slot_table, x


# -------------------------------------------------------------------------------------- a pass

def prepare(case, seed):
    desc, banks, logits, slot_table, x = _inputs(case, seed)
    T = case["tokens"]
    return {"desc": desc, "banks": banks, "logits": logits, "slot_table": slot_table, "x": x, "T": T,
            "out": torch.empty(T, desc["hidden"], dtype=torch.float32, device="cuda"),
            "route": ftm.RouteBuffers(T, desc["top_k"], desc["n_experts"]),
            "ws": None if case["entry"] == "noalloc" else ftm.alloc_workspace(desc, T)}


_ROUTE_OUT = ("topk_ids", "topk_w", "topk_slot", "hit_pairs", "miss_pairs", "hit_off", "miss_off", "counts")


def run(state):
    s, r = state, state["route"]
    if s["ws"] is None:
        ftm.ft_moe_forward_noalloc(s["desc"], s["banks"], s["logits"], s["slot_table"], s["x"], s["T"],
                                   s["out"], r)
    else:
        ftm.ft_moe_forward(s["desc"], s["banks"], s["logits"], s["slot_table"], s["x"], s["T"], s["out"],
                           r, s["ws"])
    return {"out": s["out"], **{n: getattr(r, n) for n in _ROUTE_OUT}}


# -------------------------------------------------------------------- work, tolerance, reference

def work(case):
    """Each evaluated expert's weights once, the activations, logits and routing once; the flops of
    the evaluated pairs.  The routing is that of one draw of the case's distribution."""
    H, I, E, k, _, wd, shared = LAYERS[case["layer"]]
    T = case["tokens"]
    g = torch.Generator(device="cpu")
    g.manual_seed(1)
    logits, slot_table, _ = _routing(case, g, "cpu")
    ids = logits.topk(k, dim=1).indices
    hit = slot_table[ids] >= 0
    pairs = int(hit.sum()) + (T if shared else 0)
    experts = int(ids[hit].unique().numel()) + (1 if shared else 0)
    per_weight = {BF16: 2.0, FP8: 1.0 + 4.0 / 16384, MXFP4: 0.5 + 1.0 / 32}[wd]
    nbytes = experts * 3 * H * I * per_weight + T * (H * 2 + H * 4 + E * 4 + k * 20) + E * 12
    return {"bytes": int(nbytes), "flops": 6 * H * I * pairs}


def tolerance(case):
    # Measured against exact(), over all listed cases and some drawn ones: 2-norm up to 8e-5, largest
    # element 7e-3 of the output's root mean square.  h is rounded to bf16 between the projections,
    # so a sum taken in another order moves an element of h to the neighbouring bf16 value now and
    # then.  In the fp8-activation mode it may move to the neighbouring e4m3fn value, up to an
    # eighth of it: 1.2e-3 and 5e-2.
    if case["act"] == "fp8":
        return {"rel": 5e-3, "max": 0.25}
    return {"rel": 4e-4, "max": 3e-2}


_E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _weight64(case, banks, w, s, slot):
    wd = LAYERS[case["layer"]][5]
    q = banks[w][slot]
    if wd == BF16:
        return q.double()
    if wd == FP8:
        v = q.view(torch.float8_e4m3fn).to(torch.float32).double()
        return v * banks[s][slot].double().repeat_interleave(128, 0).repeat_interleave(128, 1)
    lut = torch.tensor(_E2M1 + tuple(-v for v in _E2M1), dtype=torch.float64, device=q.device)
    v = torch.stack((lut[(q & 15).long()], lut[(q >> 4).long()]), dim=2).flatten(1)
    return v * torch.exp2(banks[s][slot].t().double() - 127).repeat_interleave(32, 1)


def _act64(case, v):
    """Activations as the layer's definition holds them: bf16, and in the fp8 mode e4m3fn per row
    and 128 channels with the smallest power-of-two scale that keeps the codes within 448."""
    v = v.to(torch.float32).to(torch.bfloat16).double()
    if case["act"] != "fp8":
        return v
    b = v.view(v.shape[0], -1, 128)
    m, e = torch.frexp(b.abs().amax(dim=2, keepdim=True))
    scale = torch.exp2((e - 9 + (m > 0.875).to(e.dtype)).clamp(-127, 127).double())
    return ((b / scale).to(torch.float32).to(torch.float8_e4m3fn).to(torch.float32).double() * scale).flatten(1)


def exact(case, seed):
    H, I, E, k, gating, _, shared = LAYERS[case["layer"]]
    T = case["tokens"]
    desc, banks, logits, slot_table, x = _inputs(case, seed)
    val, ids = logits.double().sort(dim=1, descending=True, stable=True)
    val, ids = val[:, :k], ids[:, :k]
    if gating == ftm.FT_GATE_SOFTMAX_TOPK_RENORM:
        w = torch.softmax(val, dim=1)
    else:
        w = torch.sigmoid(val)
        w = w / w.sum(dim=1, keepdim=True)
    slot = slot_table[ids]
    # stable counting sort of the pairs by expert, hits and misses apart
    flat, hit = ids.flatten(), (slot >= 0).flatten()
    order = flat.sort(stable=True).indices
    lists, offs = [], []
    for sel in (hit, ~hit):
        p = order[sel[order]]
        cnt = torch.bincount(flat[p], minlength=E)
        lists.append(torch.cat((p, torch.full((T * k - p.numel(),), -1, device=p.device))).to(torch.int32))
        offs.append(torch.cat((torch.zeros(1, device=p.device), cnt.cumsum(0))).to(torch.int32))
    n_hit = int(hit.sum())
    counts = torch.tensor([n_hit, T * k - n_hit, flat[~hit].unique().numel(), 0], dtype=torch.int32)

    out = torch.zeros(T, H, dtype=torch.float64, device=x.device)
    xq = _act64(case, x)

    def expert(s, tok, gate):
        h13 = xq[tok] @ _weight64(case, banks, "w13", "s13", s).t()
        a, u = h13[:, :I], h13[:, I:]
        h = _act64(case, a * torch.sigmoid(a) * u)
        out.index_add_(0, tok, gate[:, None] * (h @ _weight64(case, banks, "w2", "s2", s).t()))

    for e in flat[hit].unique().tolist():
        p = lists[0][offs[0][e]:offs[0][e + 1]].long()
        expert(int(slot_table[e]), p // k, w.flatten()[p])
    if shared:
        expert(desc["shared_slot"], torch.arange(T, device=x.device), torch.ones(T, dtype=torch.float64, device=x.device))
    return {"out": out, "topk_ids": ids.flatten().to(torch.int32), "topk_w": w.flatten(),
            "topk_slot": slot.flatten().to(torch.int32), "hit_pairs": lists[0], "miss_pairs": lists[1],
            "hit_off": offs[0], "miss_off": offs[1], "counts": counts.to(x.device)}
