"""The work this library is timed on: prefills and decoding steps through its public entry points.

listed() names the cases, draw() gives further ones of the same ranges; prepare() makes what a serving
program holds before a request (the loaded model, the prompt, the buffers), run() serves the request once.

Models are the shapes of paper_2407_14057_amd.synth.  A program loads its model once and then serves
prompt after prompt, so a model is made once per process from a fixed seed and shared by all states; the
seed of prepare() makes the prompt.  Two things differ from the plain N(0, 0.02) draw, as in models that
are trained in earnest: the embedding rows have about unit variance (rows scaled by sqrt(d_model)), and
the two projections that write to the residual stream are scaled by a quarter of 1/sqrt(2 * n_layers), so
that a layer changes the stream by some per cent (a sixteenth for the 8-bit projections, whose rounding
steps are 16 times as wide).  Rounding differences between two correct implementations then stay of the
order of the data type instead of being amplified by every layer.

Which outputs come back: the logits; Eq. 1's scores of every layer before the first pruning layer; K and
V of the last of these layers.  The layers after a selection are represented by the logits: Eq. 1's scores
lie so close together that two correct implementations keep a few different tokens around the threshold,
and a single different token shifts all the packed rows behind it.  With 8-bit projections only the first
layer's scores, K and V come back beside the logits: from the second layer on a last-bit difference of an
input moves some 8-bit codes by 1/16 of their value, which K shows in full and the residual stream does not.
"""
import math

import torch

from paper_2407_14057_amd import binding as B
from paper_2407_14057_amd import synth

SHAPES = {"tiny": synth.TINY, "7b": synth.LLAMA7B, "xgen7b": synth.XGEN7B, "gqa8b": synth.GQA8B,
          "7b_fp8": synth.LLAMA7B_FP8}
PRUNED = "8:700,16:500,24:300"      # keep permille of the survivors on entry to a layer: the headline schedule
BATCH8 = ",".join(str(n) for n in synth.WORKLOADS["7b_batch8"].seqlens)

_models = {}


def listed():
    return [
        # the small model of the tests: a latency-bound prefill, about thirty small launches
        {"name": "tiny_512", "kind": "prefill", "model": "tiny", "lengths": "512", "schedule": "2:700,3:500"},
        # a short question, not pruned: the weights are read for few rows
        {"name": "7b_short_97", "kind": "prefill", "model": "7b", "lengths": "97", "schedule": ""},
        # an ordinary chat turn of odd length
        {"name": "7b_chat_613", "kind": "prefill", "model": "7b", "lengths": "613", "schedule": PRUNED},
        # the benchmark's own workload: a LongBench-sized prompt
        {"name": "7b_3376", "kind": "prefill", "model": "7b", "lengths": "3376", "schedule": PRUNED},
        # a long document with the harder schedule
        {"name": "7b_8192", "kind": "prefill", "model": "7b", "lengths": "8192", "schedule": "8:600,16:400,24:200"},
        # eight prompts of 1 k to 8 k tokens packed into one call
        {"name": "7b_batch8", "kind": "prefill", "model": "7b", "lengths": BATCH8, "schedule": PRUNED},
        # grouped-query attention, wider MLP, four times the vocabulary
        {"name": "gqa8b_3376", "kind": "prefill", "model": "gqa8b", "lengths": "3376", "schedule": PRUNED},
        # the 8-bit floating point projections
        {"name": "7b_3376_fp8", "kind": "prefill", "model": "7b_fp8", "lengths": "3376", "schedule": PRUNED},
        # decoding, small model: launches and host work
        {"name": "tiny_decode", "kind": "decode", "model": "tiny", "lengths": "512", "schedule": "2:700,3:500", "tokens": 16},
        # decoding after an unpruned prefill: one token row, bound by streaming weights and K,V
        {"name": "7b_decode_dense", "kind": "decode", "model": "7b", "lengths": "3376", "schedule": "", "tokens": 8},
        # decoding after a pruned prefill: the first steps revive many tokens from the Aux Cache
        {"name": "7b_decode_pruned", "kind": "decode", "model": "7b", "lengths": "2048", "schedule": PRUNED, "tokens": 4},
    ]


def draw(rng):
    """One more case: prompt lengths from a few tokens to 8192 (log-uniform), one to six prompts, schedules of one to three pruning layers."""
    kind = rng.choice(["prefill", "prefill", "prefill", "decode"])
    model = rng.choice(["7b", "7b", "7b", "xgen7b", "gqa8b", "7b_fp8", "tiny"])
    layers = SHAPES[model].n_layers
    top = 2048 if model == "tiny" else 8192 if kind == "prefill" else 4096

    def length():
        return max(16, min(top, int(round(math.exp(rng.uniform(math.log(16), math.log(top)))))))

    lengths = [length() for _ in range(rng.choice([1, 1, 1, 2, 3, 6]) if kind == "prefill" else 1)]
    while sum(lengths) > 16384:
        lengths.pop()
    schedule = ""
    if min(lengths) >= 256 and rng.random() < 0.8:      # a prompt of fewer tokens is not worth pruning
        at = sorted(rng.sample(range(layers // 4, layers), rng.randint(1, 2 if layers < 8 else 3)))
        keep = [50 * rng.randint(6, 18) for _ in at]
        if min(lengths) * math.prod(k / 1000.0 for k in keep) >= 96:
            schedule = ",".join("%d:%d" % pair for pair in zip(at, keep))
    case = {"kind": kind, "model": model, "lengths": ",".join(map(str, lengths)), "schedule": schedule}
    if kind == "decode":
        case["tokens"] = rng.randint(2, 8)
    return case


def _lengths(case):
    return [int(x) for x in case["lengths"].split(",")]


def _schedule(case):
    return [tuple(int(v) for v in x.split(":")) for x in case["schedule"].split(",") if x]


def _model(name):
    """The loaded model: as many as a program serves at a time stay loaded."""
    if name not in _models:
        while len(_models) > 1:
            _models.pop(next(iter(_models))).close()
        shape = SHAPES[name]
        w = synth.make_weights(shape, 1002, "cuda")
        w["embed"].mul_(math.sqrt(shape.d_model))
        for t in w["wo"] + w["w_down"]:
            t.mul_((0.0625 if shape.gemm_dtype == 1 else 0.25) / math.sqrt(2.0 * shape.n_layers))
        _models[name] = B.Model(shape.as_dict(), w)
        del w
        torch.cuda.empty_cache()
    return _models[name]


def _prefill(s):
    if len(s["lengths"]) == 1:
        res = B.lazyllm_prefill(s["model"].handle, s["ids"], None, s["lengths"][0], s["schedule"], 0, s["ws"], s["out"])
    else:
        res = B.lazyllm_prefill_varlen(s["model"].handle, s["ids"], None, s["cu"], s["cu_dev"], s["schedule"], 0,
                                       s["ws"], s["out"])
    return B.PrefillOutput(res, s["out"], s["model"].cfg)


def prepare(case, seed):
    model, lengths, schedule = _model(case["model"]), _lengths(case), _schedule(case)
    shape = SHAPES[case["model"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    ids = torch.randint(0, shape.vocab, (sum(lengths) + case.get("tokens", 0),), generator=g, device="cuda", dtype=torch.int32)
    cu = [0]
    for n in lengths:
        cu.append(cu[-1] + n)
    s = {"model": model, "lengths": lengths, "schedule": schedule, "ids": ids[:cu[-1]], "cu": cu,
         "cu_dev": torch.tensor(cu, dtype=torch.int32, device="cuda"),
         "ws": torch.empty(B.lazyllm_workspace_bytes(model.cfg, cu[-1], len(lengths), max(lengths)), dtype=torch.uint8, device="cuda"),
         "out": torch.empty(B.lazyllm_output_bytes(model.cfg, lengths, schedule, 0), dtype=torch.uint8, device="cuda"),
         # layers up to this one see every token of the prompt, and their K and V can be compared
         "full": 0 if shape.gemm_dtype == 1 else (schedule[0][0] if schedule else shape.n_layers) - 1}
    if case["kind"] == "decode":
        # the continuation is given (as when a candidate text is scored): one tensor per token
        s["tokens"] = [t.clone() for t in ids[cu[-1]:].split(1)]
        s["prefill"] = _prefill(s)
        s["ws"] = None                                   # a step has a workspace of its own
    return s


def run(s):
    full = s["full"]
    if "tokens" not in s:
        p = _prefill(s)
        return {"logits": p.logits, "scores": [p.scores(l) for l in range(full + 1)], "k": p.k(full), "v": p.v(full)}
    gen = B.Generation(s["model"], s["schedule"], s["prefill"], s["lengths"][0] + len(s["tokens"]))
    logits = [gen.step(t).logits.clone() for t in s["tokens"]]
    view = gen.view()
    gen.close()
    return {"logits": logits, "k": view["k"][full], "vt": view["vt"][full]}


def work(case):
    shape, schedule = SHAPES[case["model"]], dict(_schedule(case))
    d, kvd = shape.d_model, shape.kv_heads * shape.head_dim
    params = d * (d + 2 * kvd) + d * d + 3 * d * shape.d_ffn        # of one layer
    wbytes = 1 if shape.gemm_dtype == 1 and case["kind"] == "prefill" else 2
    rows = _lengths(case)
    weights = shape.n_layers * params * wbytes + shape.vocab * d * 2
    if case["kind"] == "decode":
        n, steps = rows[0], case["tokens"]
        bytes_, flops = steps * (weights + shape.vocab * 4), 0
        bytes_ += sum(2 * d * 2 for _ in range(steps))
        for l in range(shape.n_layers):
            before = n
            if l in schedule:
                n = max(1, -(-n * schedule[l] // 1000))
                bytes_ += 2 * (before - n) * d * 2                  # the Aux Cache moves into the state
            bytes_ += 2 * 2 * n * kvd * 2 + steps * 2 * n * kvd * 2  # K,V move into the state; a step reads them
            flops += steps * (2 * params + 4 * n * d)
        return {"bytes": bytes_, "flops": flops + steps * 2 * shape.vocab * d}
    bytes_ = weights + sum(rows) * (d * 2 + 4) + len(rows) * shape.vocab * 4
    flops = len(rows) * 2 * shape.vocab * d
    for l in range(shape.n_layers):
        if l in schedule:
            kept = [max(1, -(-n * schedule[l] // 1000)) for n in rows]
            bytes_ += (sum(rows) - sum(kept)) * (d * 2 + 4)          # the Aux Cache
            rows = kept
        bytes_ += sum(rows) * (2 * kvd * 2 + 4)                      # K, V, scores
        flops += sum(2 * n * params + 2 * n * (n + 1) * d for n in rows)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # Largest relative difference of any output between a prompt served alone and the same prompt in a batch (other
    # tile shapes, other splits of the sums), and under a relative change of 1e-3 of the embedding rows: 0.003 to
    # 0.009, 0.014 where few tokens survive the pruning (7b_chat_613); four times that, up to 0.03.
    return {"rel": 0.005 if case["model"] == "tiny" else 0.03}
