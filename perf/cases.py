"""Workloads of one Mixture-of-Experts layer, as a program that serves such layers calls it.

Layer shapes are this repository's presets (paper_2605_17889_amd/synth.py): `tiny`, the
Mixtral-8x7B and 8x22B shapes (few large experts), the Qwen3-30B-A3B and DeepSeek-V2-Lite shapes
(many small experts). Token counts run from one decoded token to whole prefill chunks. The call
forms are the public ones: the layer in one call, the layer as micro-batches, the layer with some
experts' weights in host memory, and its four stages called one by one.
"""
import math

import torch

from paper_2605_17889_amd import binding as B
from paper_2605_17889_amd import synth

# d_model, d_ff, experts, experts per token
SHAPES = {
    "tiny": (512, 1024, 8, 2),
    "mixtral8x7b": (4096, 14336, 8, 2),
    "mixtral8x22b": (6144, 16384, 8, 2),
    "qwen3_30b_a3b": (2048, 768, 128, 8),
    "deepseek_v2_lite": (2048, 1408, 64, 6),
}


def _case(shape, T, form="layer", bias="none", fp32_outputs=False, micro_tokens=0, streamed=0):
    d, f, E, k = SHAPES[shape]
    return {"shape": shape, "T": T, "d_model": d, "d_ff": f, "E": E, "k": k, "form": form,
            "bias": bias,                  # none | random | zipf (expert load ~ rank^-1.2)
            "fp32_outputs": fp32_outputs,  # expert outputs kept in fp32 until the combine
            "micro_tokens": micro_tokens,  # tokens per micro-batch (form "micro")
            "streamed": streamed}          # experts whose weights come from host memory


def _named(name, *args, **kw):
    return {"name": name, **_case(*args, **kw)}


def listed():
    return [
        # the smallest layer the repository knows, at its own batch: launches and latency
        _named("tiny_t256", "tiny", 256),
        # decode of a single sequence through many small experts: eight of 128 experts are touched
        _named("qwen3_decode_t1", "qwen3_30b_a3b", 1),
        # decode of a few dozen sequences, a ragged count: most experts hold zero to five rows
        _named("qwen3_decode_t37", "qwen3_30b_a3b", 37),
        # batched decode through large experts: all weights are read for a handful of rows each
        _named("mixtral8x7b_decode_t16", "mixtral8x7b", 16),
        # the same at the preset's batch: about 64 rows per expert
        _named("mixtral8x7b_decode_t256", "mixtral8x7b", 256),
        # a program that owns the exchange between the stages (expert parallelism, inspection)
        # calls them one by one, on a chunk of ordinary size; about 62 rows per expert
        _named("qwen3_stages_t1000", "qwen3_30b_a3b", 1000, form="stages", bias="random"),
        # prefill chunk of the 128-expert layer
        _named("qwen3_prefill_t8192", "qwen3_30b_a3b", 8192),
        # prefill of a ragged number of tokens, fp32 expert outputs for accuracy
        _named("deepseek_prefill_t5003_fp32", "deepseek_v2_lite", 5003, fp32_outputs=True),
        # the headline prefill chunk
        _named("mixtral8x22b_prefill_t8192", "mixtral8x22b", 8192),
        # the largest batch, with the expert load skewed as real routers skew it
        _named("mixtral8x22b_zipf_t16384", "mixtral8x22b", 16384, bias="zipf"),
        # the micro-batched form of the layer that coalescing is compared with
        _named("mixtral8x22b_micro_t1024_m256", "mixtral8x22b", 1024, form="micro", micro_tokens=256),
        # one expert's weights live in host memory and cross the link during the call
        _named("mixtral8x7b_streamed_t2048", "mixtral8x7b", 2048, form="streamed", streamed=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# largest token count drawn per shape; the largest listed case (8x22B, 16384 tokens) costs more
_MAX_T = {"tiny": 8192, "mixtral8x7b": 8192, "mixtral8x22b": 8192, "qwen3_30b_a3b": 16384,
          "deepseek_v2_lite": 16384}


def draw(rng):
    form = rng.choice(["layer"] * 7 + ["stages"] * 2 + ["micro", "streamed"])
    if form == "streamed":
        return _case("mixtral8x7b", _log_int(rng, 64, 4096), form=form, streamed=rng.randint(1, 2))
    shape = rng.choice(sorted(SHAPES))
    if form == "micro":
        m = _log_int(rng, 48, 1024)
        return _case(shape, rng.randint(m + 1, 5 * m), form=form, micro_tokens=m)
    bias = rng.choice(["none", "none", "random", "zipf"])
    T = _log_int(rng, 256 if bias == "zipf" else 1, _MAX_T[shape])
    return _case(shape, T, form=form, bias=bias, fp32_outputs=form == "layer" and rng.random() < 0.2)


def _zipf_bias(ctx, L, cfg):
    idx = torch.empty((cfg.T, cfg.k), dtype=torch.int32, device="cuda")
    w = torch.empty((cfg.T, cfg.k), dtype=torch.float32, device="cuda")

    def count_fn(bias):
        B.moe_route(ctx, L["x"], L["w_router"], bias.cuda(), cfg.T, idx, w)
        return torch.bincount(idx.view(-1).long(), minlength=cfg.E).cpu().tolist()

    # a few per cent off the target is as good a stand-in for a skewed load
    return synth.calibrate_expert_bias(cfg, count_fn, rel_tol=0.05, max_iter=60).cuda()


def prepare(case, seed):
    T, d, f, E, k = (case[n] for n in ("T", "d_model", "d_ff", "E", "k"))
    cfg = synth.LayerConfig(case["shape"], T, d, f, E, k, seed=seed % 1000003,
                            zipf_s=1.2 if case["bias"] == "zipf" else None)
    L = synth.make_layer(cfg, "cuda")
    ctx = B.MoeContext(T, d, f, E, k)
    if case["bias"] == "random":
        g = torch.Generator(device="cuda").manual_seed(seed % 1000003)
        L["bias"] = torch.randn(E, generator=g, device="cuda") * 0.3
    elif case["bias"] == "zipf":
        L["bias"] = _zipf_bias(ctx, L, cfg)
    if case["fp32_outputs"]:
        B.moe_set_expert_output_fp32(ctx, True)
    s = {"case": case, "ctx": ctx, "L": L, "y": torch.empty((T, d), dtype=torch.bfloat16, device="cuda")}
    n = case["streamed"]
    if n:
        for name in ("W1", "W3", "W2"):
            tail = torch.empty(L[name][E - n:].shape, dtype=torch.bfloat16, pin_memory=True)
            tail.copy_(L[name][E - n:])
            L[name + "_host"] = tail
            L[name] = L[name][:E - n].clone() if n < E else None
    if case["form"] == "stages":
        i32 = lambda *shape: torch.empty(shape, dtype=torch.int32, device="cuda")
        s.update(idx=i32(T, k), gate=torch.empty((T, k), dtype=torch.float32, device="cuda"),
                 counts=i32(E), offsets=i32(E + 1), perm=i32(T * k), inv_perm=i32(T * k),
                 x_perm=torch.empty((T * k, d), dtype=torch.bfloat16, device="cuda"),
                 y_perm=torch.empty((T * k, d), dtype=torch.bfloat16, device="cuda"))
    return s


def run(s):
    case, ctx, L, y = s["case"], s["ctx"], s["L"], s["y"]
    T, form = case["T"], case["form"]
    if form == "layer":
        B.moe_layer_forward(ctx, L["x"], L["w_router"], L["bias"], L["W1"], L["W3"], L["W2"], T, y)
        return y
    if form == "micro":
        B.moe_layer_forward_microbatched(ctx, L["x"], L["w_router"], L["bias"], L["W1"], L["W3"],
                                         L["W2"], T, case["micro_tokens"], y)
        return y
    if form == "streamed":
        B.moe_layer_forward_streamed(ctx, L["x"], L["w_router"], L["bias"], L["W1"], L["W3"], L["W2"],
                                     L["W1_host"], L["W3_host"], L["W2_host"], case["streamed"], T, y)
        return y
    B.moe_route(ctx, L["x"], L["w_router"], L["bias"], T, s["idx"], s["gate"])
    B.moe_permute(ctx, s["idx"], T, s["counts"], s["offsets"], s["perm"], s["inv_perm"], L["x"],
                  s["x_perm"])
    B.moe_expert_ffn(ctx, s["x_perm"], s["offsets"], T * case["k"], L["W1"], L["W3"], L["W2"],
                     s["y_perm"])
    B.moe_combine(ctx, s["y_perm"], s["inv_perm"], s["gate"], T, y)
    return {n: s[n] for n in ("idx", "gate", "counts", "offsets", "perm", "inv_perm", "x_perm",
                              "y_perm", "y")}


def work(case):
    T, d, f, E, k = (case[n] for n in ("T", "d_model", "d_ff", "E", "k"))
    # experts that receive a row, under uniform routing
    touched = lambda tokens: E * (1.0 - (1.0 - k / E) ** tokens)
    weights = 6.0 * d * f
    m = case["micro_tokens"]
    if m:      # micro-batches run one after the other, each through the experts it touches
        calls = [m] * (T // m) + ([T % m] if T % m else [])
        read = sum(touched(t) for t in calls) * weights
    else:
        read = touched(T) * weights
    bytes_ = read + 4.0 * d * E + 4.0 * T * d
    if case["form"] == "stages":       # the tensors that the stages hand over through the caller
        bytes_ += T * k * (2.0 * d * 4 + 4.0 * 9)
    return {"bytes": bytes_, "flops": 6.0 * T * k * d * f + 2.0 * T * d * E}


def tolerance(case):
    # Against the same layer in 64-bit arithmetic the outputs are off by 2.8e-3 to 2.9e-3 (2.3e-3
    # with fp32 expert outputs), single values by up to 1.4e-2 of the larger of themselves and the
    # root mean square: roundings to bf16. Routing tables are whole numbers and stay the same.
    return {"rel": 1.15e-2, "max": 6e-2}
