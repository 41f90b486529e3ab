"""The work a user of this framework has it do, as measurable cases.

A case is one call a training program makes again and again on one GPU: a whole iteration of a
Chimera worker (`chimera_run_worker_pipes` over its two stages), the forward, or the forward and
backward, of one pipeline stage, the embedding in front of the first stage, or the vocabulary head
and loss behind the last.  Everything goes through `paper_2107_06925_amd.binding`.

Weights, activations and gradients follow the recipe of `paper_2107_06925_amd.synth` (weights
N(0, 0.02), LayerNorm gains around 1, activations and upstream gradients N(0, 1)), drawn on the
GPU; token ids are spread over the logarithm of the vocabulary, as word frequencies are.
"""
import ctypes
import math

import torch

from paper_2107_06925_amd import binding as b
from paper_2107_06925_amd import synth

DEV = "cuda"
TORCH_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
LIB_DTYPE = {"f32": b.F32, "bf16": b.BF16}
ALGO = {"direct": b.DIRECT, "doubling": b.DOUBLING, "halving": b.HALVING}


# ---------------------------------------------------------------------- cases
def _worker(D, N, rank, layers, hidden, heads, seq, microbatch, causal, dtype, schedule="direct", gelu="tanh"):
    return {"kind": "worker", "schedule": schedule, "D": D, "N": N, "rank": rank, "layers": layers, "hidden": hidden,
            "heads": heads, "seq": seq, "microbatch": microbatch, "causal": causal, "gelu": gelu, "dtype": dtype}


def _configured(name, **over):
    c = synth.CONFIGS[name]
    return dict(_worker(c.D, c.N, 0, c.layers, c.hidden, c.heads, c.seq, c.microbatch, c.causal, c.dtype), **over)


def _stage(kind, layers, hidden, heads, seq, microbatch, causal, dtype, gelu="tanh"):
    return {"kind": kind, "layers": layers, "hidden": hidden, "heads": heads, "seq": seq, "microbatch": microbatch,
            "causal": causal, "gelu": gelu, "dtype": dtype}


def listed():
    return [
        # the smallest workload: 4 micro-batches through two stages of 2 blocks, float; every launch is tiny
        dict(_configured("tiny-gpt2-f32"), name="worker-tiny-f32"),
        # a small bf16 model, as in development and tests: two schedule units, launches and host time count
        dict(_worker(4, 8, 1, 2, 256, 4, 128, 2, True, "bf16"), name="worker-small-bf16"),
        # the three bf16 workloads: bidirectional, long causal chains of units (the largest), head dim 128
        dict(_configured("bert48-bf16"), name="worker-bert48"),
        dict(_configured("gpt2-1p3b-n32-bf16"), name="worker-gpt2-1p3b-n32"),
        dict(_configured("gpt2-deep-bf16"), name="worker-gpt2-deep"),
        # the memory-saving schedule: doubled forwards, backwards that recompute
        dict(_configured("bert48-bf16", schedule="doubling", N=8), name="worker-bert48-doubling"),
        # evaluation, or the measurement of a stage's forward time: nothing kept; the sequence length of the paper's GPT-2
        dict(_stage("stage_fwd", 6, 1600, 25, 632, 2, True, "bf16"), name="stage-fwd-seq632"),
        # one micro-batch forward and backward through the same stage, one sequence: ragged token count
        dict(_stage("stage_step", 6, 1600, 25, 632, 1, True, "bf16"), name="stage-step-seq632"),
        # odd sizes throughout, exact GeLU
        dict(_stage("stage_step", 3, 320, 5, 200, 2, True, "bf16", gelu="erf"), name="stage-step-ragged"),
        # float at an ordinary size
        dict(_stage("stage_step", 2, 1024, 16, 512, 2, False, "f32"), name="stage-step-f32"),
        # the two ends of the pipeline at the bench shape
        {"kind": "head", "tokens": 4096, "hidden": 1024, "vocab": 50304, "dtype": "bf16", "name": "head-loss"},
        {"kind": "embedding", "seq": 512, "microbatch": 8, "hidden": 1024, "vocab": 50304, "dtype": "bf16", "name": "embedding"},
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _block_shape(rng, dtype, max_hidden, max_tokens):
    # bf16: the two usual head sizes most of the time, the less usual ones now and then
    d = rng.choice((32, 64) if dtype == "f32" else (64, 64, 64, 64, 128, 128, 128, 32, 80, 96))
    usual = dtype == "bf16" and d in (64, 128)
    hidden = _spread(rng, 128, max_hidden if usual else min(max_hidden, 1280))
    heads = max(1, round(hidden / d))
    seq = _spread(rng, 64, min(2048 if usual else 640, max_tokens))
    if rng.random() < 0.4:                                    # often a round length
        seq = (seq + 32) // 64 * 64
    microbatch = max(1, min(_spread(rng, 1, 8), max_tokens // seq))
    return heads * d, heads, seq, microbatch


def draw(rng):
    kind = rng.choice(("worker", "worker", "worker", "worker", "stage_step", "stage_step", "stage_fwd", "head", "embedding"))
    if kind == "head":
        dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
        hidden = 8 * _spread(rng, 16, 256 if dtype == "bf16" else 96)
        return {"kind": kind, "tokens": _spread(rng, 128, 8192 if dtype == "bf16" else 2048), "hidden": hidden,
                "vocab": 8 * _spread(rng, 128, 8192), "dtype": dtype}
    if kind == "embedding":
        seq = _spread(rng, 32, 2048)
        return {"kind": kind, "seq": seq, "microbatch": max(1, min(32, _spread(rng, 128, 16384) // seq)),
                "hidden": 8 * _spread(rng, 16, 256), "vocab": _spread(rng, 1000, 65536), "dtype": rng.choice(("bf16", "bf16", "f32"))}
    dtype = rng.choice(("bf16", "bf16", "bf16", "bf16", "f32"))
    hidden, heads, seq, microbatch = _block_shape(rng, dtype, 2560 if dtype == "bf16" else 1024, 4096 if dtype == "bf16" else 1024)
    causal, gelu = rng.random() < 0.6, rng.choice(("tanh", "tanh", "erf"))
    layers = _spread(rng, 1, 12)
    if kind != "worker":
        return _stage(kind, layers, hidden, heads, seq, microbatch, causal, dtype, gelu)
    schedule = rng.choice(("direct", "direct", "direct", "direct", "doubling", "halving"))
    D = rng.choice((2, 4, 8))
    N = D * rng.choice((2, 4) if schedule == "doubling" else (1, 2, 4))
    if schedule == "halving":
        microbatch += microbatch % 2
    c = _worker(D, N, rng.randrange(D), layers, hidden, heads, seq, microbatch, causal, dtype, schedule, gelu)
    # no longer than the largest listed workload; float and the unusual head sizes run on slower units
    most = 60e12 if dtype == "bf16" and hidden // heads in (64, 128) else 0.3e12
    while work(c)["flops"] > most and c["layers"] > 1:
        c["layers"] -= 1
    while work(c)["flops"] > most and c["seq"] > 64:
        c["seq"] = max(64, c["seq"] * 3 // 4)
    return c


# -------------------------------------------------------------------- prepare
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(gen, *shape, dtype=torch.float32, std=1.0):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=gen)


def _ids(gen, n, vocab):
    u = torch.rand(n, device=DEV, generator=gen)
    return (torch.exp(u * math.log(vocab)).long() - 1).clamp_(0, vocab - 1).to(torch.int32)


def _make_stage(case, gen, slots, microbatch=None, keep=True, weights_of=None):
    H, L = case["hidden"], case["layers"]
    st = b.Stage(L, H, case["heads"], case["seq"], microbatch or case["microbatch"], LIB_DTYPE[case["dtype"]],
                 causal=case["causal"], gelu_erf=case["gelu"] == "erf", stash_slots=slots, keep=keep,
                 share_weights_of=weights_of)
    if weights_of is None:
        st.weights.normal_(0.0, 0.02, generator=gen)
        per_block = st.weights.view(L, -1)
        second = 2 * H + 3 * H * H + 3 * H + H * H + H          # ln2_g: behind ln1, w_qkv, b_qkv, w_o, b_o
        per_block[:, :H] += 1.0
        per_block[:, second:second + H] += 1.0
    return st


def _set_io(st, mb, x, y, dy, dx):
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    b.check(b.lib().chimera_stage_set_io(st.handle, mb, p(x), p(y), p(dy), p(dx)))


def prepare(case, seed):
    gen = _gen(seed)
    kind, tdt = case["kind"], TORCH_DTYPE[case["dtype"]]
    if kind == "embedding":
        S, H, V = case["seq"], case["hidden"], case["vocab"]
        M = S * case["microbatch"]
        return {"kind": kind, "seq": S, "tokens": _ids(gen, M, V), "wte": _randn(gen, V, H, dtype=tdt, std=0.02),
                "wpe": _randn(gen, S, H, dtype=tdt, std=0.02), "dx": _randn(gen, M, H, dtype=tdt),
                "x": torch.empty((M, H), dtype=tdt, device=DEV), "dwte": torch.zeros((V, H), device=DEV),
                "dwpe": torch.zeros((S, H), device=DEV)}
    if kind == "head":
        M, H, V = case["tokens"], case["hidden"], case["vocab"]
        need = b.lib().chimera_head_workspace_bytes(LIB_DTYPE[case["dtype"]], M, H, V)
        return {"kind": kind, "y": _randn(gen, M, H, dtype=tdt), "targets": _ids(gen, M, V), "scale": 1.0 / M,
                "g": 1.0 + _randn(gen, H, dtype=tdt, std=0.02), "b": _randn(gen, H, dtype=tdt, std=0.02),
                "w": _randn(gen, H, V, dtype=tdt, std=0.02), "dy": torch.empty((M, H), dtype=tdt, device=DEV),
                "dg": torch.zeros(H, device=DEV), "db": torch.zeros(H, device=DEV), "dw": torch.zeros((H, V), device=DEV),
                "loss": torch.zeros(1, device=DEV), "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}
    M, H = case["seq"] * case["microbatch"], case["hidden"]
    N = case.get("N", 1)
    x, dy = _randn(gen, N, M, H, dtype=tdt), _randn(gen, N, M, H, dtype=tdt)
    y, dx = torch.zeros_like(x), torch.zeros_like(x)
    s = {"kind": kind, "x": x, "dy": dy, "y": y, "dx": dx}
    if kind != "worker":
        st = _make_stage(case, gen, 1, keep=kind == "stage_step")
        _set_io(st, 0, x[0], y[0], dy[0], dx[0])
        return dict(s, stages=[st])
    algo, D, rank = ALGO[case["schedule"]], case["D"], case["rank"]
    ops = b.chimera_schedule_pipes(algo, D, N, 1, rank)
    need = b.stash_slots_needed_pipes(algo, D, N, 1, rank)
    stages = [_make_stage(case, gen, max(n, 1)) for n in need]
    doubled = []
    if algo == b.DOUBLING:
        s["y2"] = torch.zeros_like(y)
        doubled = [_make_stage(case, gen, 1, microbatch=2 * case["microbatch"], keep=False, weights_of=st) for st in stages]
    for o in ops:
        if o.kind == b.OP_F2:
            pair, out = x[o.mb:o.mb + 2], s["y2"][o.mb:o.mb + 2]
            _set_io(doubled[o.pipe], o.mb, pair, out, pair, out)
        elif o.kind in (b.OP_B, b.OP_BH1):
            _set_io(stages[o.pipe], o.mb, x[o.mb], y[o.mb], dy[o.mb], dx[o.mb])
    return dict(s, stages=stages, doubled=doubled, replay=(algo, rank, D, N))


# ------------------------------------------------------------------------ run
def run(s):
    kind = s["kind"]
    if kind == "embedding":
        b.chimera_op_embedding_fwd(s["tokens"], s["seq"], s["wte"], s["wpe"], s["x"])
        b.chimera_op_embedding_bwd(s["tokens"], s["seq"], s["dx"], s["dwte"], s["dwpe"])
        return {"x": s["x"], "dwte": s["dwte"], "dwpe": s["dwpe"]}
    if kind == "head":
        b.chimera_head_loss(s["y"], s["targets"], s["g"], s["b"], s["w"], s["scale"], s["dy"], s["dg"], s["db"], s["dw"],
                            s["loss"], workspace=s["ws"])
        return {k: s[k] for k in ("dy", "dg", "db", "dw", "loss")}
    stages = s["stages"]
    if kind == "stage_fwd":
        stages[0].fwd(0)
        return {"y": s["y"]}
    for st in stages:
        st.zero_grads()
    if kind == "stage_step":
        stages[0].fwd(0)
        stages[0].bwd(0)
    else:
        algo, rank, D, N = s["replay"]
        b.chimera_worker_bind_pipes(stages)
        if s["doubled"]:
            b.chimera_worker_bind_doubling(*s["doubled"])
        b.chimera_run_worker_pipes(algo, rank, D, N)
    out = {"y": s["y"], "dx": s["dx"], "grads": [st.grads for st in stages]}
    if "y2" in s:
        out["y2"] = s["y2"]
    return out


# ----------------------------------------------------------------------- work
def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    kind, H = case["kind"], case["hidden"]
    if kind == "embedding":
        M, V = case["seq"] * case["microbatch"], case["vocab"]
        # table rows the tokens touch (expected number); each gradient row is read and written
        rows = round(sum(1.0 - math.exp(-M / (math.log(V) * (i + 1))) for i in range(V)))
        return {"bytes": 4 * M + e * H * (rows + case["seq"] + 2 * M) + 8 * H * (rows + case["seq"]), "flops": 3 * M * H}
    if kind == "head":
        M, V = case["tokens"], case["vocab"]
        return {"bytes": e * (2 * M * H + H * V) + 8 * H * V, "flops": 6 * M * H * V}
    M, S, L, N = case["seq"] * case["microbatch"], case["seq"], case["layers"], case.get("N", 1)
    visible = (S + 1) / (2 * S) if case["causal"] else 1.0
    forward = L * (24 * M * H * H + 4 * M * S * H * visible)
    weights = L * (12 * H * H + 13 * H)
    if kind == "stage_fwd":
        return {"bytes": e * (weights + 2 * M * H), "flops": forward}
    stages = 2 if kind == "worker" else 1
    passes = 3 * N
    if case.get("schedule") == "doubling":
        D = case["D"]
        passes += N - (D if (N // D) % 2 else 0)         # forwards that the backwards recompute
    return {"bytes": stages * weights * (e + 4) + N * 4 * M * H * e, "flops": passes * forward}


def tolerance(case):
    if case["dtype"] == "f32" or case["kind"] == "embedding":
        return {"rel": 1e-5}
    return {"rel": 1e-2}
