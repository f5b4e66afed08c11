"""The work that a user of this framework has it do, as cases that can be timed.

A training program owns one `Stage` per GPU and, every iteration, has it interpret its instruction list on the
buffers of the iteration's micro-batches.  The cases are such iterations over the range the framework takes: the
fp32 configuration with a handful of tokens, one short sequence per micro-batch, the three bf16 stages of the
workload table, long and ragged sequences, an iteration after a failover (backward through the replica layers), the
wrap-around stage with the model's ends, and the optimizer step with the replica synchronisation that closes an
iteration.

Parameters and inputs follow the distributions of `synth` (matrices ~ N(0, 0.02^2), inputs ~ N(0, 1), upstream
gradients ~ N(0, 1) / sqrt(T H)), drawn on the device.
"""
import torch

from paper_2204_12013_amd import binding as B
from paper_2204_12013_amd import synth
from paper_2204_12013_amd.harness import StageHarness, WrapHarness

DEV = "cuda:0"
ENC, DEC = synth.ARCH_POST_LN_ENCODER, synth.ARCH_PRE_LN_CAUSAL
F32, BF16 = synth.DTYPE_FP32, synth.DTYPE_BF16
RC = {"lazy": B.RC_LFLB, "eager": B.RC_EFLB, "eager_backward": B.RC_EFEB}


def _case(name, kind, arch, dtype, hidden, heads, ffn, seq, micro_batch, n_own, n_shadow, P, stage_id, M,
          rc="eager", vocab=0):
    return {"name": name, "kind": kind, "arch": arch, "dtype": dtype, "hidden": hidden, "heads": heads, "ffn": ffn,
            "seq": seq, "micro_batch": micro_batch, "n_own": n_own, "n_shadow": n_shadow, "P": P,
            "stage_id": stage_id, "M": M, "rc": rc, "vocab": vocab}


def _from_table(name, workload, kind="iteration", rc="eager", vocab=0, **change):
    s = synth.CONFIGS[workload].replace(**change)
    return _case(name, kind, s.arch, s.dtype, s.hidden, s.heads, s.ffn, s.seq, s.micro_batch, s.n_own, s.n_shadow,
                 s.P, s.stage_id, s.M, rc, vocab)


def listed():
    return [
        # the fp32 configuration: 32 tokens a micro-batch, what a check of a new set-up runs
        _from_table("tiny_f32", "tiny"),
        # one short sequence per micro-batch through BERT-large layers: latency and weight traffic
        _from_table("one_short_sequence", "bert_large_stage", seq=128, micro_batch=1, n_own=2, n_shadow=2, M=4),
        # the headline workload: BERT-large stage, eager redundant forward on the second lane
        _from_table("bert_large_stage", "bert_large_stage"),
        # the same stage with redundancy off (the setting of a run on stable instances)
        _from_table("bert_large_no_redundancy", "bert_large_stage", rc="lazy"),
        # the GPT-2 stage, half of the table's micro-batches
        _from_table("gpt2_stage", "gpt2_1p5b_stage", M=8),
        # the large layer: matrix products of 2048 x 12288 x 49152, one layer and its replica
        _from_table("large_layer", "large_layer_stage", n_own=1, n_shadow=1, M=2),
        # sequences cut to their real length (333 tokens) instead of padded: token counts that divide by nothing
        _from_table("ragged_encoder", "bert_large_stage", seq=333, micro_batch=3, n_own=2, n_shadow=2, M=4),
        # one long document per micro-batch: attention over 8192 causal positions carries the time
        _case("long_context", "iteration", DEC, BF16, 1024, 16, 4096, 8192, 1, 2, 2, 4, 1, 2),
        # the iterations after a preemption: the stage runs its own and its victim's layers, both directions
        _from_table("after_failover", "bert_large_stage", kind="merged", n_own=3, n_shadow=3),
        # the last stage: LM head and loss behind its layers, the first stage's embedding and layers as replica
        _from_table("last_stage_wrap", "bert_large_stage", kind="wrap", stage_id=3, n_own=3, n_shadow=3,
                    vocab=synth.VOCAB["bert_large_stage"]),
        # the same for the decoder after the first stage was lost: both ends forward and backward
        _from_table("both_ends_merged", "gpt2_1p5b_stage", kind="wrap_merged", stage_id=7, n_own=1, n_shadow=1, M=4,
                    vocab=synth.VOCAB["gpt2_1p5b_stage"]),
        # the end of an iteration: Adam on the own parameters, the replica takes its owner's new values
        _from_table("optimizer_step", "bert_large_stage", kind="apply"),
    ]


# A drawn case's work stays below this many flops: a fifth of the largest listed case's.
_DRAW_FLOPS = 1.2e13


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    while True:
        kind = rng.choice(["iteration", "iteration", "iteration", "iteration", "merged", "wrap", "wrap_merged", "apply"])
        arch = rng.choice([ENC, DEC])
        if kind == "iteration" and rng.random() < 0.2:
            dtype, d = F32, rng.choice([32, 64])
            heads, seq, mb = rng.randint(1, 4), _log_int(rng, 8, 64), rng.randint(1, 4)
        else:
            dtype, d = BF16, rng.choice([64, 64, 128])
            heads = _log_int(rng, 4, 32) if d == 64 else _log_int(rng, 2, 24)
            seq, mb = _log_int(rng, 64, 4096), _log_int(rng, 1, 8)
            if rng.random() < 0.5:
                seq = max(64, seq // 64 * 64)          # padded to a multiple of 64, as many data loaders do
        hidden = heads * d
        # four times the width, or any other multiple of 8
        ffn = 4 * hidden if rng.random() < 0.7 else 8 * int(hidden * (2.0 + 2.5 * rng.random()) / 8)
        n_own = rng.randint(1, 4)
        n_shadow = n_own if rng.random() < 0.6 else rng.randint(1, 4)      # partitions may be uneven
        M = rng.randint(2, 8)
        P = rng.randint(2, 8)
        wrap = kind.startswith("wrap")
        stage_id = P - 1 if wrap else rng.randint(0, P - 2)
        rc = rng.choice(["lazy", "eager", "eager", "eager_backward"]) if kind == "iteration" else "eager"
        vocab = 8 * _log_int(rng, 128, 6288) if wrap else 0
        c = _case("", kind, arch, dtype, hidden, heads, ffn, seq, mb, n_own, n_shadow, P, stage_id, M, rc, vocab)
        del c["name"]
        if mb * seq <= 16384 and work(c)["flops"] <= _DRAW_FLOPS:
            return c


# ------------------------------------------------------------------------------------------- inputs

def _layers(gen, n, H, F, act):
    """n layers' parameters in one flat vector."""
    parts = []
    for _ in range(n):
        for name in synth.PARAM_NAMES:
            numel = 1
            for s in synth.param_shapes(H, F)[name]:
                numel *= s
            v = torch.randn(numel, generator=gen, device=DEV) * 0.02
            if name in ("g1", "g2"):
                v += 1.0
            parts.append(v.to(act))
    return torch.cat(parts)


def _zipf(gen, V, T):
    """Token ids with Zipf's law, as synth.zipf_ids gives them, drawn on the device."""
    p = torch.cumsum(1.0 / torch.arange(1, V + 1, device=DEV, dtype=torch.float64), 0)
    u = torch.rand(T, generator=gen, device=DEV, dtype=torch.float64) * p[-1]
    return torch.searchsorted(p, u).clamp_(max=V - 1).to(torch.int32)


def prepare(case, seed):
    kind, H, F = case["kind"], case["hidden"], case["ffn"]
    sc = synth.StageConfig("", case["arch"], case["dtype"], H, case["heads"], F, case["seq"], case["micro_batch"],
                           case["n_own"], case["n_shadow"], case["P"], case["stage_id"], case["M"], 0)
    T, M = sc.tokens, sc.M
    act = torch.bfloat16 if sc.dtype == BF16 else torch.float32
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    wrap = kind.startswith("wrap")
    cfg = B.make_cfg(sc, rc_mode=RC[case["rc"]], wrap=int(wrap))
    st = B.Stage(cfg, _layers(gen, sc.n_own, H, F, act), _layers(gen, sc.n_shadow, H, F, act))
    state = {"kind": kind, "stage": st, "step": 0}
    if kind == "apply":
        st.own_g.copy_(torch.randn(st.own_g.shape, generator=gen, device=DEV) * 1e-3)
        st.stage_optimizer_init()
        # the successor's parameters and optimizer state after its own update
        state["next_w"] = _layers(gen, sc.n_shadow, H, F, act)
        state["next_opt"] = torch.randn(st.shadow_opt.shape, generator=gen, device=DEV) * 1e-3
        torch.cuda.synchronize()
        return state
    x = [torch.randn(T, H, generator=gen, device=DEV).to(act) for _ in range(M)]
    g = [(torch.randn(T, H, generator=gen, device=DEV) / (T * H) ** 0.5).to(act) for _ in range(M)]
    if wrap:
        V = case["vocab"]
        sz = B.ends_query_sizes(cfg, V)
        ends = B.Ends(cfg, V, (torch.randn(int(sz.front_params), generator=gen, device=DEV) * 0.02).to(act),
                      (torch.randn(int(sz.back_params), generator=gen, device=DEV) * 0.02).to(act))
        ids = [_zipf(gen, V, T) for _ in range(M)]
        labels = [_zipf(gen, V, T) for _ in range(M)]
        state["ends"] = ends
        state["harness"] = WrapHarness(st, ends, x, ids, labels, g)
    else:
        # gradients at the stage's own output come from the live successor (a table), after a failover from BRC
        gy = [(torch.randn(T, H, generator=gen, device=DEV) / (T * H) ** 0.5).to(act) for _ in range(M)]
        state["harness"] = StageHarness(st, x, gz=g, gy_table=gy)
    if kind in ("merged", "wrap_merged"):
        # the successor was lost at the first hand-over of an earlier iteration
        st.stage_begin_iteration()
        st.failover_merge(0)
        st.stage_begin_iteration()
    state["program"] = st.stage_schedule()
    torch.cuda.synchronize()
    return state


def run(state):
    st = state["stage"]
    here = torch.cuda.current_stream()
    # the iteration is ordered after and before the program's other work on the device, never on the host
    st.stream_main.wait_stream(here)
    if state["kind"] == "apply":
        state["step"] += 1
        st.stage_apply(state["step"], lr=1e-4)
        st.stage_sync_replica(state["next_w"], state["next_opt"])
        here.wait_stream(st.stream_main)
        return {"own_w": st.own_w, "own_opt": st.own_opt, "shadow_w": st.shadow_w, "shadow_opt": st.shadow_opt}
    hz = state["harness"]
    hz.begin_iteration()
    hz.run(state["program"])
    st.stage_join()
    here.wait_stream(st.stream_main)
    out = {"y": hz.y, "gx": hz.gx, "own_g": st.own_g}
    frc = any(op == B.FRC for op, _, _, _ in state["program"])
    if frc:
        out["z"] = hz.z_frc
    if any(op == B.BRC for op, _, _, _ in state["program"]):
        out["shadow_g"] = st.shadow_g
    if state["kind"].startswith("wrap"):
        out["loss"], out["head_g"] = hz.loss, state["ends"].back_g
        if state["kind"] == "wrap_merged":
            out["front_g"] = state["ends"].front_g
    return out


# ----------------------------------------------------------------------------------- necessary work

def work(case):
    T, H, F, S, M = case["micro_batch"] * case["seq"], case["hidden"], case["ffn"], case["seq"], case["M"]
    e = 2 if case["dtype"] == BF16 else 4
    params = 4 * H * H + 2 * H * F + 9 * H + F
    own, shadow = params * case["n_own"], params * case["n_shadow"]
    if case["kind"] == "apply":
        # gradient, master weights and two moments in; the last three and the storage copy out; replica state in and out
        return {"bytes": own * (28 + e) + 2 * shadow * (12 + e), "flops": 12 * own}
    gemm = 2 * T * (4 * H * H + 2 * H * F)
    attn = 4 * T * S * H // (2 if case["arch"] == DEC else 1)
    fwd, bwd = gemm + attn, 2 * gemm + 5 * attn // 2
    act = T * H * e
    frc = case["rc"] != "lazy" or case["kind"] in ("merged", "wrap_merged")
    brc = case["rc"] == "eager_backward" or case["kind"] in ("merged", "wrap_merged")
    flops = M * case["n_own"] * (fwd + bwd)
    moved = own * (e + 4) + 4 * M * act                # weights in, gradients out; x, gy in, y, gx out
    if frc:
        flops += M * case["n_shadow"] * fwd
        moved += shadow * e + M * act
    if brc:
        flops += M * case["n_shadow"] * bwd
        moved += shadow * 4 + M * act
    if case["kind"].startswith("wrap"):
        V = case["vocab"]
        flops += 6 * M * T * H * V
        moved += H * V * (e + 4) + M * T * (H * e + 8)
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # About four times the distance from the same layers in the next wider arithmetic (fp64 for fp32 and for the
    # optimizer, fp32 storage for bf16), largest over outputs, input gradients and weight gradients.
    if case["kind"] == "apply":
        # measured 1.3e-5 (second moment); a bf16 weight at a tie may round the other way (2^-8)
        return {"rel": 5e-5, "max": 1e-2}
    if case["dtype"] == F32:
        # measured 1.6e-7 rel, 2.4e-6 max at 32 tokens; sums grow to a few hundred terms
        return {"rel": 1e-5, "max": 1e-4}
    # measured 0.5e-2 (2 layers) to 1.0e-2 (6 layers) rel, 0.06 to 0.13 max
    return {"rel": 2e-2, "max": 0.5}
