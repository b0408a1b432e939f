"""Performance cases of the stage library: what a training or evaluation program has it do.

A case is one iteration on one GPU through the public entry points of the binding: the gradient
accumulators are cleared, `mbs` microbatches go through the passes F, B and W of a chunk (or a whole
schedule is replayed), and the outputs, input gradients and parameter gradients come back.

    kind      "step"     F, B and W of every microbatch in turn
              "queued"   F and B of every microbatch, then ONE deferred W call for all of them
              "forward"  F alone, the unit given back (evaluation: nothing is differentiated)
              "replay"   schedule_replay of `schedule` for d simulated devices and n microbatches
"""
import math

import torch

import paper_2405_15362_amd as P
from paper_2405_15362_amd import runtime as R


def _case(name, kind, dtype, layers, hidden, heads, ffn, seq, microbatch=1, causal=True, mbs=1, schedule="", d=0, n=0):
    c = {"kind": kind, "dtype": dtype, "layers": layers, "hidden": hidden, "heads": heads, "ffn": ffn, "seq": seq,
         "microbatch": microbatch, "causal": causal, "mbs": mbs, "schedule": schedule, "d": d, "n": n}
    return {"name": name, **c} if name else c


def listed():
    return [
        # The smallest stage (the library's fp32 configuration): a handful of microseconds of work per
        # kernel, so launches and latency count.  One step, and a whole replay of 48 such passes.
        _case("step_f32_h256", "step", "f32", 1, 256, 4, 1024, 128),
        _case("replay_f32_h256", "replay", "f32", 1, 256, 4, 1024, 128, schedule="vhalf", d=2, n=4),
        # fp32 at a width where arithmetic counts: debugging a model in full precision.
        _case("step_f32_h1024", "step", "f32", 2, 1024, 16, 4096, 512),
        # A toy bf16 model with a short sequence, as in unit tests and smoke runs of a training script.
        _case("step_bf16_h256_s192", "step", "bf16", 2, 256, 2, 1024, 192),
        # Evaluation: several sequences of uneven length through four layers, nothing kept for backward.
        _case("forward_bf16_h1600_s1000", "forward", "bf16", 4, 1600, 25, 6400, 1000, microbatch=2),
        # An encoder (no mask) of moderate width, eight short sequences per microbatch, head size 64.
        _case("step_bf16_h1024_full_mb8", "step", "bf16", 2, 1024, 16, 4096, 512, microbatch=8, causal=False),
        # The small benchmark stage (1024 tokens of hidden 2048), and the same stage with a sequence
        # length that fills no tile.
        _case("step_bf16_h2048_s1024", "step", "bf16", 2, 2048, 16, 8192, 1024),
        _case("step_bf16_h2048_s1000", "step", "bf16", 2, 2048, 16, 8192, 1000),
        # Head size 112 (hidden 7168 over 64 heads), the widest model of the library's tests.
        _case("step_bf16_h7168_dh112", "step", "bf16", 1, 7168, 64, 28672, 1024),
        # Four layers of hidden 4096 with four microbatches whose W passes are deferred and run as one.
        _case("queued_bf16_h4096_x4", "queued", "bf16", 4, 4096, 32, 16384, 2048, mbs=4),
        # A memory-balanced schedule over four chunks of that layer, W right after B's turn.
        _case("replay_bf16_h4096", "replay", "bf16", 2, 4096, 32, 16384, 2048, schedule="vhalf", d=2, n=4),
        # The largest single-GPU stage: 4096 tokens of hidden 5120, attention-heavy.
        _case("step_bf16_h5120_s4096", "step", "bf16", 2, 5120, 40, 20480, 4096),
    ]


def _passes(c):
    """Chunk passes of each kind in one iteration (chunks x microbatches)."""
    return 2 * c["d"] * c["n"] if c["kind"] == "replay" else c["mbs"]


def _chunks(c):
    return 2 * c["d"] if c["kind"] == "replay" else 1


def _params_per_layer(c):
    h, f = c["hidden"], c["ffn"]
    return 4 * h * h + 2 * h * f + 9 * h + f


def _flops(c):
    t, h = c["seq"] * c["microbatch"], c["hidden"]
    gemm = 2 * t * h * (4 * h + 2 * c["ffn"])
    scores = 4 * t * c["seq"] * h // (2 if c["causal"] else 1)
    one = gemm + scores
    if c["kind"] != "forward":
        one += 2 * gemm + 2 * scores
    return c["layers"] * _passes(c) * one


def _bytes(c):
    e = 2 if c["dtype"] == "bf16" else 4
    params = _chunks(c) * c["layers"] * _params_per_layer(c)
    act = c["seq"] * c["microbatch"] * c["hidden"] * e
    ends = c["n"] if c["kind"] == "replay" else c["mbs"]
    if c["kind"] == "forward":
        return params * e + ends * 2 * act
    return params * (e + 4) + ends * 4 * act


def work(case):
    # weights read once, gradients written once, chunk inputs and outputs; the causal half of the scores;
    # backward counted as twice the forward
    return {"bytes": _bytes(case), "flops": _flops(case)}


def draw(rng):
    def spread(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    while True:
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        kind = rng.choices(("step", "queued", "forward", "replay"), (10, 4, 3, 3))[0]
        dh = rng.choice((64, 64, 128, 128, 128, 40, 80, 96, 112))
        hidden = dh * max(1, round(spread(64, 1280 if dtype == "f32" else 7168) / dh))
        ffn = 4 * hidden if rng.random() < 0.75 else 8 * round(hidden * rng.uniform(2.0, 4.5) / 8)
        microbatch = rng.choice((1, 1, 1, 2, 4, 8))
        # tokens are a multiple of 8; with 8 sequences per microbatch the sequence itself may be odd
        unit = 8 // microbatch
        seq = unit * max(1, round(spread(16, 768 if dtype == "f32" else 4096) / unit))
        mbs = {"step": rng.choice((1, 1, 2)), "queued": rng.randint(2, 8)}.get(kind, 1)
        c = _case("", kind, dtype, rng.randint(1, 4), hidden, hidden // dh, ffn, seq, microbatch, rng.random() < 0.8, mbs)
        if kind == "replay":
            c.update(schedule=rng.choice(("1f1b", "vzb", "vhalf", "vmin", "1f1bv")), d=rng.randint(1, 3), n=rng.randint(2, 6))
        # no more than the largest listed case costs: operations, and bytes of weights and gradients
        if _flops(c) <= (1.5e11 if dtype == "f32" else 3e13) and _bytes(c) <= 7e9:
            return c


class _State:
    """A program's context, chunks, microbatch tensors and schedule, given back with the object."""

    def __init__(self, case, seed):
        c, dt = case, R.torch_dtype(case["dtype"])
        gen = torch.Generator(device="cuda").manual_seed(seed)
        cfg = P.make_cfg(c["layers"], c["hidden"], c["heads"], c["ffn"], c["seq"], c["microbatch"], c["dtype"], c["causal"])
        self.case, self.schedule, ws, slabs = c, None, None, c["mbs"]
        if c["kind"] == "replay":
            self.schedule = P.pmc_schedule_build(c["schedule"], c["d"], c["n"])
            ws = P.pmc_replay_workspace_bytes(self.schedule, cfg)
            slabs = sum(a[0] for a in P.pmc_schedule_account(self.schedule, 1, 0))
        self.context = R.Context(cfg, slabs=slabs, workspace_bytes=ws)
        h, f, tokens = c["hidden"], c["ffn"], c["seq"] * c["microbatch"]
        shapes = ((h,), (h,), (h, 3 * h), (3 * h,), (h, h), (h,), (h,), (h,), (h, f), (f,), (f, h), (h,))
        # weights and biases N(0, 0.02^2), LayerNorm gains 1 + N(0, 0.02^2), activations and upstream gradients N(0, 1)
        self.params, self.flat_grads, self.grads, self.chunks = [], [], [], []
        for _ in range(_chunks(c)):
            params, grads, at = [], [], 0
            flat = torch.zeros(c["layers"] * sum(math.prod(s) for s in shapes), dtype=torch.float32, device="cuda")
            for _ in range(c["layers"]):
                for name, shape in zip(R.PARAM_NAMES, shapes):
                    p = torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, 0.02, generator=gen)
                    params.append(p + 1.0 if name in ("ln1_g", "ln2_g") else p)
                    grads.append(flat[at:at + p.numel()].view(shape))
                    at += p.numel()
            chunk = P.pmc_chunk_create(self.context.ctx, cfg)
            P.pmc_chunk_bind(chunk, params, grads)
            self.params.append(params)
            self.flat_grads.append(flat)
            self.grads.append(grads)
            self.chunks.append(chunk)
        count = c["n"] if c["kind"] == "replay" else c["mbs"]

        def normal():
            return torch.empty(tokens, h, dtype=dt, device="cuda").normal_(generator=gen)

        self.x = [normal() for _ in range(count)]
        self.y = [torch.empty_like(t) for t in self.x]
        if c["kind"] != "forward":
            self.dy = [normal() for _ in range(count)]
            self.dx = [torch.empty_like(t) for t in self.x]

    def __del__(self):
        for chunk in getattr(self, "chunks", ()):
            P.pmc_chunk_destroy(chunk)
        if getattr(self, "schedule", None) is not None:
            P.pmc_schedule_destroy(self.schedule)
        if hasattr(self, "context"):
            self.context.close()


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    kind, s = state.case["kind"], state
    if kind == "forward":
        for j, (x, y) in enumerate(zip(s.x, s.y)):
            P.stage_forward(s.chunks[0], j, x, y)
            P.stage_abandon(s.chunks[0], j)
        return {"y": s.y}
    for flat in s.flat_grads:
        flat.zero_()
    if kind == "replay":
        P.schedule_replay(s.context.ctx, s.schedule, s.chunks, s.x, s.dy, s.y, s.dx)
        return {"y": s.y, "dx": s.dx, "grads": s.flat_grads}
    for j in range(len(s.x)):
        P.stage_forward(s.chunks[0], j, s.x[j], s.y[j])
        P.stage_backward_input(s.chunks[0], j, s.dy[j], s.dx[j])
        if kind == "step":
            P.stage_backward_weight(s.chunks[0], [j])
    if kind == "queued":
        P.stage_backward_weight(s.chunks[0], range(len(s.x)))
    return {"y": s.y, "dx": s.dx, "grads": s.grads[0]}


def tolerance(case):
    # fp32 against the same passes in 64 bits: relative 8e-7 .. 1.5e-6, largest difference 2e-5.
    # bf16 with its sums in another order (other tile shapes, other attention splits): relative
    # 1.5e-3 (one or two narrow layers) .. 1e-2 (four layers of hidden 4096, one of 7168), largest
    # difference 0.12, mostly in the LayerNorm and bias gradients; against 64 bits 4e-3 .. 1.2e-2.
    # More than four layers in a row (replays) add up further.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-4}
    return {"rel": 2e-2 if _chunks(case) * case["layers"] <= 4 else 3e-2, "max": 0.45}
