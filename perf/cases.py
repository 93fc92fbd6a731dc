"""Performance cases of the integerized ViT path: single linears, attention(+MLP) blocks and encoders,
from one image to the benchmark's full batches, each through the public entry points of
``paper_2504_18547_amd.vitq`` the way a user's program calls them.

Kinds of case
  linear    vq_quantize of fp32 tokens, then one reordered linear.  out: "acc_f32" (int32 accumulators
            and fp32), "f32", "packed" (requantized), "gelu" (GELU + requantized), "absorbed" (integer-only
            epilogue, packed).
  block     vq_quantize of LayerNormed fp32 tokens, then vq_attention_block (hidden == 0: attention only).
  encoder   vq_vit_encoder: a stack of pre-LayerNorm blocks on the fp32 residual stream.

Weights, biases and token distributions are those of ``workloads.py`` (weights N(0, std 0.02), biases
N(0, std 0.01), Q/K rows wider when ``sharp`` so that the quantized softmax is not degenerate); activation
steps are absmax-calibrated on one image in fp32, as a deployed model's would be.  Every result of the
library is a fixed sequence of integer and correctly rounded fp32 operations, so outputs compare exactly.
"""
import math

import torch

from paper_2504_18547_amd import vitq

STREAM_STEP_SIGMA = 3.5      # LayerNorm quantizers clip at 3.5 sigma (as bench.py's pre-LayerNorm block)


# ---- the cases ---------------------------------------------------------------------------------------

def _linear(name, M, K, Nout, bits_w, bits_a, out):
    return dict(name=name, kind="linear", M=M, K=K, Nout=Nout, bits_w=bits_w, bits_a=bits_a, out=out)


def _block(name, B, N, H, hidden, bits_w, bits_a, sharp=True, qkln=False):
    return dict(name=name, kind="block", B=B, N=N, H=H, hidden=hidden, bits_w=bits_w, bits_a=bits_a,
                sharp=sharp, qkln=qkln)


def _encoder(name, layers, B, N, H, hidden, bits_w, bits_a, qkln=False):
    return dict(name=name, kind="encoder", layers=layers, B=B, N=N, H=H, hidden=hidden, bits_w=bits_w,
                bits_a=bits_a, sharp=True, qkln=qkln)


def listed():
    return [
        # the ViT-S QKV projection of one image, accumulators and fp32 out: one small linear, all latency
        _linear("linear_vit_s_qkv_b1", 197, 384, 1152, 4, 4, "acc_f32"),
        # a linear of a pruned / odd-sized model: nothing is a multiple of a tile or of a packed word
        _linear("linear_ragged", 777, 1000, 1001, 4, 4, "f32"),
        # the integer-only form of the output projection (ViT-B, 64 images)
        _linear("absorbed_proj_b64", 64 * 197, 768, 768, 4, 4, "absorbed"),
        # interactive use: one image through a ViT-B block
        _block("block_vit_b_b1", 1, 197, 12, 3072, 4, 4),
        # attention-only ViT-S at its usual batch
        _block("attn_vit_s_b64", 64, 197, 6, 0, 4, 4),
        # the headline workload, weights as stated (near-uniform softmax)
        _block("block_vit_b_b256", 256, 197, 12, 3072, 4, 4, sharp=False),
        # the 8-bit model at the batch of its configuration
        _block("block_vit_b_b128_w8a8", 128, 197, 12, 3072, 8, 8),
        # 384-pixel ViT-L: long rows, the attention's other form
        _block("block_vit_l_577_b64", 64, 577, 16, 4096, 4, 4),
        # the same in 8 bits at a small, odd batch
        _block("block_vit_l_577_b9_w8a8", 9, 577, 16, 4096, 8, 8),
        # a whole ViT-B encoder for one image: the latency a caller waits for
        _encoder("encoder_vit_b_b1", 12, 1, 197, 12, 3072, 4, 4),
        # the same in throughput use
        _encoder("encoder_vit_b_b64", 12, 64, 197, 12, 3072, 4, 4),
        # the paper's own model and topology: DeiT-S tokens, 2-bit weights, LayerNorm quantizers on Q and K
        _encoder("encoder_deit_s_b50_w2a4_qkln", 12, 50, 198, 6, 1536, 2, 4, qkln=True),
    ]


MAX_FLOPS, MAX_SCORES, MAX_BYTES = 2.0e12, 3.0e8, 3.0e8     # bounds of a drawn case (below the largest listed ones)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost_ok(case):
    w = work(case)
    scores = case.get("layers", 1) * case["B"] * case["H"] * case["N"] ** 2 if case["kind"] != "linear" else 0
    return w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES and scores <= MAX_SCORES


def draw(rng):
    bits_w, bits_a = rng.choice([(4, 4), (4, 4), (4, 4), (3, 4), (2, 4), (8, 8)])
    kind = rng.choice(["linear", "linear", "block", "block", "block", "encoder", "encoder"])
    if kind == "linear":
        out = rng.choice(["acc_f32", "f32", "f32", "packed", "packed", "gelu", "absorbed"])
        K, Nout = _log_int(rng, 64, 4096), _log_int(rng, 16, 4096)
        if rng.random() < 0.5:
            K, Nout = (K + 63) // 64 * 64, (Nout + 63) // 64 * 64
        if out == "absorbed":
            Nout = (Nout + 15) // 16 * 16
        case = _linear("", _log_int(rng, 1, 50432), K, Nout, bits_w, bits_a, out)
        while not _cost_ok(case):
            case["M"] = case["M"] * 2 // 3
    else:
        N = rng.choice([197, 198, 577, _log_int(rng, 17, 577)])
        H = rng.choice([2, 3, 6, 6, 12, 12, 16])
        B = _log_int(rng, 1, 256)
        qkln = rng.random() < 0.25
        if kind == "block":
            hidden = rng.choice([0, 256 * H, 256 * H, 128 * H])
            case = _block("", B, N, H, hidden, bits_w, bits_a, sharp=rng.random() < 0.75, qkln=qkln)
        else:
            case = _encoder("", rng.choice([1, 2, 6, 12]), B, N, H, 256 * H, bits_w, bits_a, qkln=qkln)
        while not _cost_ok(case):
            case["B"] = max(1, case["B"] * 2 // 3)
    del case["name"]
    return case


# ---- what one pass cannot do without -------------------------------------------------------------------

def _storage(bits):
    return 2 if bits <= 2 else (4 if bits <= 4 else 8)


def work(case):
    """Integer multiply-adds (two operations each) of the matmuls; bytes of the fp32 / packed inputs and
    outputs and of the weights, each once (a chain's intermediates could stay on the chip)."""
    sw, sa = _storage(case["bits_w"]), _storage(case["bits_a"])
    if case["kind"] == "linear":
        M, K, Nout = case["M"], case["K"], case["Nout"]
        out = {"acc_f32": 8.0, "f32": 4.0}.get(case["out"], sa / 8)
        extra = Nout * 4.0 * (1 << case["bits_a"]) if case["out"] == "absorbed" else Nout * 8.0
        return dict(bytes=M * K * 4.0 + Nout * K * sw / 8 + M * Nout * out + extra, flops=2.0 * M * K * Nout)
    D, B, N, hidden = 64 * case["H"], case["B"], case["N"], case["hidden"]
    per_token = 3 * D * D + D * D + 2 * D * hidden + 2 * N * D
    weights = (4 * D * D + 2 * D * hidden) * sw / 8 + (5 * D + hidden) * 8.0
    L = case.get("layers", 1)
    return dict(bytes=B * N * D * 8.0 + L * weights, flops=2.0 * L * B * N * per_token)


def tolerance(case):
    return "exact"


# ---- what a user's program has in hand -----------------------------------------------------------------

def _step(t, qmax):
    """absmax step, rounded to three digits as a stored calibration would be."""
    return float("%.3g" % max(float(t.abs().max()) / qmax, 1e-6))


def _quantized_weight(w, bits):
    s = vitq.vq_weight_steps(w, bits)
    q = vitq.QMat.empty(w.shape[0], w.shape[1], bits)
    vitq.vq_quantize(w, 0.0, s, q)
    return q, s


def _prepare_linear(case, gen):
    M, K, Nout, ba = case["M"], case["K"], case["Nout"], case["bits_a"]
    qmax = float((1 << (ba - 1)) - 1)
    x = torch.randn(M, K, generator=gen, device="cuda")
    w = torch.randn(Nout, K, generator=gen, device="cuda") * 0.02
    bias = torch.randn(Nout, generator=gen, device="cuda") * 0.01
    wq, sw = _quantized_weight(w, case["bits_w"])
    s_x = 0.1 if (case["bits_w"], ba) == (4, 4) and case["out"] == "acc_f32" else 3.5 / qmax
    s_y = float("%.3g" % (3.5 * 0.02 * math.sqrt(K) / qmax))
    st = dict(kind="linear", out=case["out"], x=x, xq=vitq.QMat.empty(M, K, ba), s_x=s_x, wq=wq, sw=sw, bias=bias,
              s_y=s_y, acc=None, y=None, yq=None)
    if case["out"] == "acc_f32":
        st["acc"] = torch.empty(M, Nout, dtype=torch.int32, device="cuda")
    if case["out"] in ("acc_f32", "f32"):
        st["y"] = torch.empty(M, Nout, device="cuda")
    else:
        st["yq"] = vitq.QMat.empty(M, Nout, ba)
    if case["out"] == "absorbed":
        b_int, thr = vitq.vq_absorb_thresholds(s_x, sw.cpu().numpy(), bias.cpu().numpy(), [s_y], ba)
        st["b_int"], st["thr"] = torch.from_numpy(b_int).cuda(), torch.from_numpy(thr).cuda()
    return st


def _layer_norm(t):
    return torch.nn.functional.layer_norm(t, (t.shape[-1],), eps=1e-6)


def _float_attention(x, w, H):
    """fp32 Q, K, V and attention output of one image [N, D] (calibration only)."""
    N, D = x.shape
    q, k, v = (x @ w["qkv"].t() + w["b_qkv"]).view(N, 3, H, 64).permute(1, 2, 0, 3).contiguous()
    p = torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) * 0.125, dim=-1)
    return q, k, v, torch.matmul(p, v).permute(1, 0, 2).reshape(N, D)


def _layer(case, gen, x, preln):
    """Weights of one layer, their packed copies and the descriptor; x: one image's stream [N, D] in fp32,
    returned advanced by the layer."""
    H, N, hidden, bw, ba = case["H"], case["N"], case["hidden"], case["bits_w"], case["bits_a"]
    D = 64 * H
    qmax = float((1 << (ba - 1)) - 1)

    def randn(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")

    w = dict(qkv=randn(3 * D, D) * 0.02, b_qkv=randn(3 * D) * 0.01, proj=randn(D, D) * 0.02, b_proj=randn(D) * 0.01)
    if case["sharp"]:
        w["qkv"][: 2 * D] *= 0.08 * math.sqrt(384.0 / D) / 0.02
    if hidden:
        w.update(fc1=randn(hidden, D) * 0.02, b_fc1=randn(hidden) * 0.01, fc2=randn(D, hidden) * 0.02,
                 b_fc2=randn(D) * 0.01)
    xin = _layer_norm(x) if preln else x
    q, k, v, o = _float_attention(xin, w, H)
    attn = o @ w["proj"].t() + w["b_proj"]
    steps = dict(s_q=_step(q, qmax), s_k=_step(k, qmax), s_v=_step(v, qmax), s_o=_step(o, qmax), scale=0.125)
    ln = None
    if preln:
        steps["s_x"] = steps["s_x2"] = STREAM_STEP_SIGMA / qmax
        x = x + attn
        mlp_in = _layer_norm(x)
        ln = dict(g1=1 + 0.1 * randn(D), b1=0.05 * randn(D), g2=1 + 0.1 * randn(D), b2=0.05 * randn(D), eps=1e-6)
    else:
        steps["s_x"], steps["s_x2"] = _step(x, qmax), _step(attn, qmax)
        mlp_in = attn
    if hidden:
        h = torch.nn.functional.gelu(mlp_in @ w["fc1"].t() + w["b_fc1"], approximate="tanh")
        steps["s_h"] = _step(h, qmax)
        if preln:
            x = x + h @ w["fc2"].t() + w["b_fc2"]
    qk = None
    if case["qkln"]:
        qk = dict(gamma=1 + 0.2 * randn(2 * D), beta=0.1 * randn(2 * D), eps=1e-6)
        steps["s_q"] = steps["s_k"] = 3.0 / qmax
    packed = {}
    for nm in ("qkv", "proj", "fc1", "fc2"):
        if nm in w:
            packed["w_" + nm], packed["sw_" + nm] = _quantized_weight(w[nm], bw)
            packed["b_" + nm] = w["b_" + nm]
    desc = vitq.make_block_desc(dict(D=D, H=H, N=N, hidden=hidden), ba, ba, _storage(ba), packed, steps, qkln=qk)
    if preln:
        desc = vitq.make_preln_desc(desc, ln)
    return desc, steps, (packed, qk, ln), x


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["kind"] == "linear":
        return _prepare_linear(case, gen)
    B, N, D, ba = case["B"], case["N"], 64 * case["H"], case["bits_a"]
    M = B * N
    x = torch.randn(M, D, generator=gen, device="cuda")
    y = torch.empty(M, D, device="cuda")
    if case["kind"] == "block":
        x = _layer_norm(x)
        desc, steps, keep, _ = _layer(case, gen, x[:N], False)
        ws = torch.empty(vitq.vq_attention_block_workspace(desc, B), dtype=torch.uint8, device="cuda")
        return dict(kind="block", x=x, s_x=steps["s_x"], xq=vitq.QMat.empty(M, D, ba), desc=desc, B=B, y=y, ws=ws,
                    keep=keep)
    # the residual stream: a scale and a shift of its own for every token
    x = x * (0.5 + 2.5 * torch.rand(M, 1, generator=gen, device="cuda")) + (2 * torch.rand(M, 1, generator=gen, device="cuda") - 1)
    descs, keep, t = [], [], x[:N]
    for _ in range(case["layers"]):
        desc, _, held, t = _layer(case, gen, t, True)
        descs.append(desc)
        keep.append(held)
    ws = torch.empty(vitq.vq_vit_encoder_workspace(descs, B), dtype=torch.uint8, device="cuda")
    return dict(kind="encoder", descs=descs, x=x, B=B, y=y, ws=ws, keep=keep)


# ---- one pass --------------------------------------------------------------------------------------------

def run(state):
    s = state
    if s["kind"] == "encoder":
        vitq.vq_vit_encoder(s["descs"], s["x"], s["B"], s["y"], s["ws"])
        return s["y"]
    vitq.vq_quantize(s["x"], s["s_x"], None, s["xq"])
    if s["kind"] == "block":
        vitq.vq_attention_block(s["desc"], s["xq"], s["B"], s["y"], s["ws"])
        return s["xq"].data, s["y"]
    if s["out"] == "absorbed":
        vitq.vq_linear_absorbed(s["xq"], s["wq"], s["b_int"], s["thr"], None, s["yq"])
    else:
        vitq.vq_linear(s["xq"], s["s_x"], s["wq"], s["sw"], 1, s["bias"], int(s["out"] == "gelu"), s["acc"], s["y"],
                       s["s_y"], s["yq"])
    return [t for t in (s["acc"], s["y"], s["yq"].data if s["yq"] is not None else None) if t is not None]
