"""The work that a user of this library has it do, as cases that can be timed and compared.

Four ways of calling it, all through paper_2405_18425_amd.binding:
  "path"   bigla_fwd, then locality_gate_fwd on its output: what bench.py calls a step (the gates are given)
  "call"   bigla_locality_fwd: the same two steps as one call
  "block"  gated_bigla_fwd, then locality_gate_fwd: the forward of a block from its input on, which also leaves
           the gates that the gradient needs
  "train"  bigla_fwd, then bigla_bwd: the token mixer's part of a training step, output and five gradients
"""
import math

import torch

from paper_2405_18425_amd import binding as vb

TAU = 16.0  # temperature of the forget gates
RANK = 16   # width of the gate producer's bottleneck


def _case(name, op, B, H, Hg, Wg, dk=64, dv=64, dtype="bf16", layout="bhld", mu=0.0):
    return {"name": name, "op": op, "B": B, "H": H, "Hg": Hg, "Wg": Wg, "dk": dk, "dv": dv, "dtype": dtype,
            "layout": layout, "mu": mu}


def listed():
    return [
        # the smallest configuration, in fp32: what a new installation is checked with; two launches
        _case("tiny_f32", "path", 1, 1, 8, 8, dk=16, dv=16, dtype="f32"),
        # one 224-pixel image through a block of the small model, token-major as projections emit it: latency
        _case("one_image_224_block", "block", 1, 6, 14, 14, layout="blhd"),
        # a batch at 224 pixels, tiny model: many short sequences
        _case("vig_t_224", "path", 64, 3, 14, 14),
        # the ImageNet training shape of the small model
        _case("vig_s_224_train", "train", 64, 6, 14, 14),
        # 512-pixel images, base model, slow decay: as many sequences as compute units, roughly
        _case("vig_b_512", "path", 16, 12, 32, 32, mu=2.0),
        # 1024-pixel images, small model, fast decay: few long sequences (bench.py's default)
        _case("vig_s_1024", "path", 8, 6, 64, 64, mu=-2.0),
        # training at that resolution
        _case("vig_s_1024_train", "train", 8, 6, 64, 64, mu=-2.0),
        # keys half as wide as values (the head shape of the published models), token-major, whole block
        _case("vig_s_1024_dk32_block", "block", 4, 6, 64, 64, dk=32, layout="blhd", mu=-1.0),
        # first and last stage of a hierarchical model at 224 pixels: two heads of 3136 tokens, sixteen of 49
        _case("stage1_56x56", "call", 16, 2, 56, 56),
        _case("stage4_7x7", "call", 64, 16, 7, 7),
        # a detection-style image whose grid is a multiple of nothing: ragged chunks, odd rows, training
        _case("ragged_37x53_train", "train", 3, 5, 37, 53, layout="blhd", mu=1.0),
        # full precision, for validating a training run
        _case("f32_224_train", "train", 4, 3, 14, 14, dtype="f32"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("path", "path", "call", "block", "block", "train", "train"))
    f32 = op in ("path", "train") and rng.random() < 0.15
    # the largest listed: 8 * 6 heads of 4096 tokens in bf16, and in fp32 short sequences in few heads
    most_tokens, side = (12 * 196, 14) if f32 else (8 * 6 * 4096, 64)
    while True:
        B, H = _log_int(rng, 1, 64), rng.choice((1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 16))
        Hg, Wg = _log_int(rng, 7, side), _log_int(rng, 7, side)
        if B * H * Hg * Wg <= most_tokens:
            break
    dk, dv = rng.choice((64, 64, 32)), 64
    if f32:
        dk = dv = rng.choice((16, 32, 64))
    case = _case("", op, B, H, Hg, Wg, dk, dv, "f32" if f32 else "bf16", rng.choice(("bhld", "blhd")),
                 round(rng.uniform(-2.0, 2.0), 1))
    del case["name"]
    return case


def _log_gates(shape, mu, gen, dtype):
    """log sigmoid(z) / tau with z ~ N(mu, 1)."""
    z = torch.randn(shape, generator=gen, device="cuda") + mu
    return (torch.nn.functional.logsigmoid(z) / TAU).to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    B, H, dk, dv = case["B"], case["H"], case["dk"], case["dv"]
    L = case["Hg"] * case["Wg"]
    op, layout = case["op"], case["layout"]

    def normal(shape, scale):
        return (torch.randn(shape, generator=gen, device="cuda") * scale).to(dtype)

    def heads(d):
        return (B, H, L, d) if layout == "bhld" else (B, L, H, d)

    s = {"case": case, "q": normal(heads(dk), 0.25), "k": normal(heads(dk), 0.25), "v": normal(heads(dv), 0.25)}
    if op == "block":
        D = H * dv
        s["x"] = normal((B, L, D), 1.0)
        s["w1"] = normal((RANK, D), D ** -0.5)
        s["w2"] = normal((2 * H * dk, RANK), RANK ** -0.5)
        s["b2"] = (torch.randn(2 * H * dk, generator=gen, device="cuda") + case["mu"]).to(dtype)
        s["g_fwd"], s["g_bwd"] = torch.empty_like(s["q"]), torch.empty_like(s["q"])
    else:
        s["g_fwd"] = _log_gates(heads(dk), case["mu"], gen, dtype)
        s["g_bwd"] = _log_gates(heads(dk), case["mu"], gen, dtype)
    if op == "train":
        s["d_out"] = normal(heads(dv), 1.0)
    else:
        s["conv_w"] = normal((H * dv, 3, 3), 0.1)
        s["conv_b"] = normal((H * dv,), 0.1) if op != "path" else None
        s["z"] = normal(heads(dv), 1.0)
        s["out"] = torch.empty_like(s["v"])
    s["o_global"] = torch.empty_like(s["v"])
    if op in ("path", "train"):
        code = vb.VIG_BF16 if case["dtype"] == "bf16" else vb.VIG_F32
        need = vb.bigla_workspace_bytes(B, H, L, dk, dv, code)
        s["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    c = s["case"]
    op, layout, Hg, Wg = c["op"], c["layout"], c["Hg"], c["Wg"]
    if op == "call":
        return vb.bigla_locality_fwd(s["q"], s["k"], s["v"], s["g_fwd"], s["g_bwd"], s["v"], s["conv_w"], s["z"], Hg, Wg,
                                     bias=s["conv_b"], out=s["out"], layout=layout)
    if op == "block":
        vb.gated_bigla_fwd(s["x"], s["w1"], s["w2"], s["q"], s["k"], s["v"], bias=s["b2"], tau=TAU, layout=layout,
                           out=s["o_global"], g_fwd=s["g_fwd"], g_bwd=s["g_bwd"])
    else:
        vb.bigla_fwd(s["q"], s["k"], s["v"], s["g_fwd"], s["g_bwd"], out=s["o_global"], workspace=s["workspace"],
                     layout=layout)
    if op == "train":
        return (s["o_global"], *vb.bigla_bwd(s["q"], s["k"], s["v"], s["g_fwd"], s["g_bwd"], s["d_out"], layout=layout))
    vb.locality_gate_fwd(s["v"], s["conv_w"], s["z"], s["o_global"], Hg, Wg, bias=s["conv_b"], out=s["out"], layout=layout)
    return (s["out"], s["g_fwd"], s["g_bwd"]) if op == "block" else s["out"]


def work(case):
    B, H, dk, dv, op = case["B"], case["H"], case["dk"], case["dv"], case["op"]
    L = case["Hg"] * case["Wg"]
    size = 2 if case["dtype"] == "bf16" else 4
    tokens = B * H * L
    # values per head and token: q, k, both gates; v and the output
    values = 4 * dk + 2 * dv
    # two directions of a state update and a readout, in the recurrence's own form
    flops = 8 * dk * dv
    if op == "train":
        values += 4 * dk + 2 * dv  # d_out in; dq, dk, dg_fwd, dg_bwd and dv out
        flops += 20 * dk * dv      # per direction: state, adjoint, dq, dk, dv
    else:
        values += dv               # gate logits (the convolution's input is v)
        flops += 25 * dv
    total, flop_total = tokens * values, tokens * flops
    if op == "block":
        D = H * dv
        total += B * L * D
        flop_total += B * L * 2 * RANK * (D + 2 * H * dk)
    return {"bytes": total * size, "flops": flop_total}


def tolerance(case):
    # Against the definition in 64 bits the listed cases show, in bf16, 2.2e-3 to 3.5e-3 and single values 0.012 to
    # 0.034 of the root mean square (the rounding of the result alone is 1.7e-3); two such results then differ by up to
    # 5e-3.  In fp32 the token-by-token kernels show 1.1e-7, the gate gradients (running sums over the sequence) 5.9e-7
    # and 2.8e-6; sums over chunks, with cumulative gates of ten nats in 32 bits, a few times that.
    return {"rel": 1e-2, "max": 0.15} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 5e-5}
