"""The work this library is used for, as cases that can be timed and compared.

Each case is one pass through the public entry points as a user's program
calls them: a linear layer on activation codes (generation and prompt
sizes, int8 and packed int4 weights, symmetric and asymmetric, 8- and 16-bit
activations), the quantizer with the gate/up projections, the logits of the
language-model head, a whole decoder block over a prompt, a decoder block's
generation step over a key/value cache, range learning forward and backward,
and the conversion of a weight matrix (smoothing scales, fold, pack).

Activations carry a few large channels, as the layers meet them in real
models; formats are static, as a calibrated deployment holds them.
"""
import math

import numpy as np
import torch

import paper_2408_13933_amd as mq
from paper_2408_13933_amd import workloads as wl
from paper_2408_13933_amd.block import BlockGPU

W_STD, B_STD = wl.W_STD, wl.B_STD
DIMS = wl.BLOCK_DIMS  # hidden 2048, 32 heads over 4 key/value heads of 64, feed-forward 5632

# Static float ranges of the block's stages for the inputs drawn here (unit
# rows with four channels 20 times as large): what a calibration would keep,
# the largest channels clipped where the codes have 8 bits.
RANGES = dict(h0=(-90.0, 95.0), x1=(-16.0, 18.0), q=(-4.5, 5.0), k=(-4.5, 5.0), v=(-4.0, 4.5),
              qr=(-5.0, 5.5), kr=(-5.0, 4.5), scores=(-32.0, 36.0), probs=(0.0, 1.0),
              ctx=(-1.5, 1.25), o=(-3.0, 3.5), h1=(-92.0, 97.0), x2=(-18.0, 16.0),
              gate=(-5.0, 5.5), up=(-5.5, 5.0), silu=(-0.2785, 5.5), mul=(-9.0, 8.0),
              down=(-5.0, 4.5), h2=(-94.0, 99.0))


def listed():
    return [
        # the smallest call: one linear over the 16 rows of a small batch in
        # generation, with bias, int8 to int8; launch and latency count
        dict(name="decode_16x2048x2048", kind="linear", M=16, K=2048, N=2048, w_bits=8,
             out_bits=8, a_bits=8, asym=False, bias=True),
        # one generated token's pass through a decoder block with 1531 tokens
        # in the cache (a chat in progress: the length is rarely round),
        # captured once and replayed as a serving loop does
        dict(name="generate_ctx1531", kind="generate", L=1531),
        # the logits of one generated token, 256000 words: weight bytes count
        dict(name="logits_m1_256000", kind="logits", M=1, K=2048, N=256000),
        # the logits of every position of a 512-token prompt (scoring)
        dict(name="logits_m512_256000", kind="logits", M=512, K=2048, N=256000),
        # float activations of a long prompt into codes and through gate and up
        dict(name="gate_up_2048x2048x5632", kind="gate_up", M=2048, K=2048, N=5632, out_bits=8),
        # a short prompt's down projection with a long reduction, 16-bit codes out
        dict(name="down_512x16384x2048", kind="linear", M=512, K=16384, N=2048, w_bits=8,
             out_bits=16, a_bits=8, asym=False, bias=False),
        # 4-bit weights (asymmetric per channel) in prompt encoding
        dict(name="w4_down_1024x5632x2048", kind="linear", M=1024, K=5632, N=2048, w_bits=4,
             out_bits=16, a_bits=8, asym=True, bias=False),
        # 16-bit activations, 8-bit weights: the setting that keeps activations wide
        dict(name="w8a16_gate_1024x2048x5632", kind="linear", M=1024, K=2048, N=5632, w_bits=8,
             out_bits=16, a_bits=16, asym=False, bias=False),
        # a whole decoder block over a 1024-token prompt
        dict(name="block_1024", kind="block", T=1024),
        # the same over a prompt whose length is no multiple of anything
        dict(name="block_777", kind="block", T=777),
        # range learning: the training form forward and backward on one
        # layer's activations
        dict(name="range_learning_2048x2048", kind="arl", M=2048, K=2048, bits=8),
        # converting one weight matrix: smoothing scales from calibration
        # activations, fold, one asymmetric 8-bit range per tensor
        dict(name="convert_5632x2048", kind="convert", M=2048, K=2048, N=5632, w_bits=8,
             per_tensor=True, asym=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A reduction length: a model dimension, a multiple of 64."""
    return max(1, int(round(_log(rng, lo, hi) / 64))) * 64


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "generate", "logits", "gate_up", "block",
                       "block", "arl", "convert"])
    if kind == "linear":
        a_bits = rng.choice([8, 8, 8, 16])
        w_bits = 8 if a_bits == 16 else rng.choice([8, 8, 4])
        asym = a_bits == 8 and rng.random() < 0.4
        K, N = _width(rng, 512, 16384), _log(rng, 256, 8192)
        M = min(_log(rng, 1, 2048), (1 << 36) // (K * N))  # bounds the largest products
        return dict(kind=kind, M=M, K=K, N=N, w_bits=w_bits, out_bits=rng.choice([8, 16]),
                    a_bits=a_bits, asym=asym, bias=rng.random() < 0.5)
    if kind == "generate":
        return dict(kind=kind, L=_log(rng, 64, 4096))
    if kind == "logits":
        return dict(kind=kind, M=_log(rng, 1, 512), K=_width(rng, 1024, 2048),
                    N=_log(rng, 32000, 256000))
    if kind == "gate_up":
        return dict(kind=kind, M=_log(rng, 16, 2048), K=_width(rng, 1024, 4096),
                    N=4 * _log(rng, 512, 4096), out_bits=rng.choice([8, 16]))
    if kind == "block":
        return dict(kind=kind, T=_log(rng, 48, 1024))
    if kind == "arl":
        return dict(kind=kind, M=_log(rng, 64, 4096), K=_width(rng, 512, 4096),
                    bits=rng.choice([4, 8, 16]))
    asym = rng.random() < 0.6
    K = _width(rng, 1024, 8192)
    return dict(kind=kind, M=_log(rng, 256, 2048), K=K, N=min(_log(rng, 512, 8192), (1 << 24) // K),
                w_bits=rng.choice([8, 8, 4]),
                per_tensor=asym and rng.random() < 0.5, asym=asym)


# ---------------------------------------------------------------------------
# Inputs.

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _acts(g, M, K):
    """fp32 activations: N(0, 1), four channels 20 times as large."""
    x = torch.randn(M, K, generator=g, device="cuda")
    ch = torch.randperm(K, generator=g, device="cuda")[:4]
    x[:, ch] *= 20.0
    return x


def _weights(g, N, K, asym=False):
    w = torch.randn(N, K, generator=g, device="cuda") * W_STD
    if asym:  # off-centre rows, so the zero-points spread over the grid
        w += (torch.rand(N, 1, generator=g, device="cuda") * 4.0 - 2.0) * W_STD
    return w


def _out_format(K, asym, bits):
    """Output format of a linear on _acts and _weights: skewed, so that the
    zero-point is not zero, a few outputs saturating."""
    energy = K + 4 * 399.0  # sum_k x^2 of one row
    sigma = W_STD * math.sqrt(energy * (7.0 / 3.0 if asym else 1.0))
    return mq.mq_act_params(-4.5 * sigma - 3 * B_STD, 5.5 * sigma + 3 * B_STD, bits)


def _linear_inputs(case, seed):
    g = _gen(seed)
    M, K, N = case["M"], case["K"], case["N"]
    x = _acts(g, M, K)
    w = _weights(g, N, K, case["asym"])
    bias = torch.randn(N, generator=g, device="cuda") * B_STD if case["bias"] else None
    s = dict(fa=mq.mq_act_params(-70.0, 80.0, case["a_bits"]),
             fy=_out_format(K, case["asym"], case["out_bits"]), bias=bias)
    s["a"] = mq.mq_quantize_act(x, *s["fa"], case["a_bits"])
    if case["asym"]:
        s["wq"], s["ws"], s["wz"], s["cs"] = mq.mq_pack_weights_asym(w, case["w_bits"])
        s["rowsum"] = mq.mq_act_rowsum(s["a"])
    else:
        s["wq"], s["ws"], s["cs"] = mq.mq_pack_weights(w, case["w_bits"])
    if case["a_bits"] == 8:
        nb = mq.mq_qlinear_workspace_bytes(M, K, N, case["w_bits"], case["out_bits"])
        s["work"] = torch.zeros(nb, dtype=torch.uint8, device="cuda") if nb else None
    return s


def _logits_inputs(case, seed):
    g = _gen(seed)
    x = _acts(g, case["M"], case["K"])
    s = dict(x=x, fa=mq.mq_act_params(-70.0, 80.0, 8), fy=_out_format(case["K"], False, 16))
    s["wq"], s["ws"], s["cs"] = mq.mq_pack_weights(_weights(g, case["N"], case["K"]), 8)
    nb = mq.mq_qlinear_workspace_bytes(case["M"], case["K"], case["N"], 8, 16)
    s["work"] = torch.zeros(nb, dtype=torch.uint8, device="cuda") if nb else None
    return s


def _gate_up_inputs(case, seed):
    g = _gen(seed)
    s = dict(x=_acts(g, case["M"], case["K"]), fa=mq.mq_act_params(-70.0, 80.0, 8))
    fy = _out_format(case["K"], False, case["out_bits"])
    s["linears"] = []
    for k in range(2):
        wq, ws, cs = mq.mq_pack_weights(_weights(g, case["N"], case["K"]), 8)
        s["linears"].append(dict(w_q=wq, w_scale=ws, w_colsum=cs, out_scale=fy[0] * (1 + k / 8),
                                 out_zp=fy[1]))
    return s


def _block_data(T, seed):
    g = _gen(seed)
    d = DIMS
    dim = dict(hidden=d["hidden"], kv=d["kv_heads"] * d["head_dim"], ffn=d["ffn"])
    h0 = _acts(g, T, d["hidden"])
    w = {n: _weights(g, dim[a], dim[b]) for n, a, b in wl.BLOCK_LINEARS}
    gamma = [torch.rand(d["hidden"], generator=g, device="cuda") + 0.5 for _ in range(2)]
    return h0, w, gamma


def _captured(fn):
    """fn's launches as a HIP graph (fn only enqueues work)."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fn()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    return graph


def _block_inputs(case, seed):
    h0, w, gamma = _block_data(case["T"], seed)
    data = wl.BlockData(case["T"], h0.cpu().numpy(), {n: v.cpu().numpy() for n, v in w.items()},
                        gamma[0].cpu().numpy(), gamma[1].cpu().numpy(), RANGES)
    block = BlockGPU(data)
    return dict(block=block, graph=_captured(block.run))


class _Step:
    """One generated token through a decoder block: the new key and value
    join the cache, the query attends to all L tokens."""

    def __init__(self, L, seed):
        from paper_2408_13933_amd.block import STAGE_BITS, formats
        d = DIMS
        H, G, D, hid, ffn = d["heads"], d["kv_heads"], d["head_dim"], d["hidden"], d["ffn"]
        self.L, self.H, self.G, self.D = L, H, G, D
        self.bits, self.fmt = STAGE_BITS, formats(RANGES, mq.mq_act_params)
        h0, w, self.gamma = _block_data(1, seed)
        self.w = {n: mq.mq_pack_weights(v, 8) for n, v in w.items()}
        self.h0 = mq.mq_quantize_act(h0, *self.fmt["h0"], 16)
        g = _gen(seed + 1000003)
        cap = (L + 63) // 64 * 64  # the cache's capacity
        keys = mq.mq_quantize_act(torch.randn(cap, G * D, generator=g, device="cuda") * 0.8,
                                  *self.fmt["kr"], 8)
        vals = mq.mq_quantize_act(torch.randn(G * D, cap, generator=g, device="cuda") * 0.8,
                                  *self.fmt["v"], 8)
        self.keys, self.vals = keys, vals  # [cap][G D] and [G D][cap]
        self.table = mq.mq_rope_table(1, D, base=d["rope_base"], pos0=L - 1)
        self.lut = mq.mq_lut_build(mq.LUT_SILU, *self.fmt["gate"], *self.fmt["silu"], 16)
        shapes = dict(x1=(1, hid), q=(1, H * D), k=(1, G * D), v=(1, G * D), qr=(1, H * D),
                      scores=(H, 1, L), probs=(H, 1, L), ctx=(1, H * D), o=(1, hid),
                      h1=(1, hid), x2=(1, hid), gate=(1, ffn), up=(1, ffn), mul=(1, ffn),
                      down=(1, hid), h2=(1, hid))
        self.out = {s: torch.empty(shp, device="cuda",
                                   dtype=torch.int8 if self.bits[s] == 8 else torch.int16)
                    for s, shp in shapes.items()}
        nb = max(mq.mq_attn_matmul_workspace_bytes(H, G, 1, L),
                 mq.mq_attn_matmul_workspace_bytes(H, G, 1, D))
        self.work = torch.empty(nb, dtype=torch.uint8, device="cuda")
        self.graph = _captured(self.step)

    def _group(self, stages, names, src):
        lin = []
        for st, n in zip(stages, names):
            wq, ws, cs = self.w[n]
            lin.append(dict(w_q=wq, w_scale=ws, w_colsum=cs, out_scale=self.fmt[st][0],
                            out_zp=self.fmt[st][1], out=self.out[st]))
        mq.mq_qlinear_group(self.out[src], lin, 8, *self.fmt[src], self.bits[stages[0]])

    def _linear(self, stage, name, src):
        wq, ws, cs = self.w[name]
        mq.mq_qlinear(self.out[src], wq, 8, ws, cs, *self.fmt[src], *self.fmt[stage],
                      self.bits[stage], out=self.out[stage])

    def step(self):
        f, o, L, H, G, D = self.fmt, self.out, self.L, self.H, self.G, self.D
        eps = DIMS["eps"]
        mq.mq_rmsnorm(self.h0, *f["h0"], self.gamma[0], eps, *f["x1"], 8, out=o["x1"])
        self._group(("q", "k"), ("q_proj", "k_proj"), "x1")
        self._linear("v", "v_proj", "x1")
        mq.mq_rope_apply(o["q"], H, *f["q"], *f["qr"], self.table, 16, out=o["qr"])
        mq.mq_rope_apply(o["k"], G, *f["k"], *f["kr"], self.table, 8, out=self.keys[L - 1:L])
        self.vals[:, L - 1].copy_(o["v"][0])
        mq.mq_attn_matmul(o["qr"].view(1, H, D).permute(1, 0, 2),
                          self.keys.view(-1, G, D)[:L].permute(1, 0, 2), *f["qr"], *f["kr"],
                          *f["scores"], 16, out=o["scores"], workspace=self.work)
        mq.mq_softmax(o["scores"].view(H, L), f["scores"][0] / D ** 0.5, f["scores"][1],
                      *f["probs"], 16, out=o["probs"].view(H, L))
        mq.mq_attn_matmul(o["probs"], self.vals.view(G, D, -1)[:, :, :L], *f["probs"], *f["v"],
                          *f["ctx"], 8, out=o["ctx"].view(1, H, D).permute(1, 0, 2),
                          workspace=self.work)
        self._linear("o", "o_proj", "ctx")
        mq.mq_add_rmsnorm(self.h0, *f["h0"], o["o"], *f["o"], *f["h1"], self.gamma[1], eps,
                          *f["x2"], 8, h=o["h1"], out=o["x2"])
        self._group(("gate", "up"), ("gate_proj", "up_proj"), "x2")
        mq.mq_lut_mul(o["gate"], self.lut, *f["silu"], o["up"], *f["up"], *f["mul"], 8,
                      out=o["mul"])
        self._linear("down", "down_proj", "mul")
        mq.mq_add_requant(o["h1"], *f["h1"], o["down"], *f["down"], *f["h2"], 16, out=o["h2"])


def _arl_inputs(case, seed):
    g = _gen(seed)
    x = _acts(g, case["M"], case["K"])
    grad = torch.randn(case["M"], case["K"], generator=g, device="cuda") * 1e-3
    # a learned range: narrower than the outlier channels, so that some clip
    alpha = 24.0 / (2 ** case["bits"] - 1)
    return dict(x=x, grad=grad, alpha=alpha, beta=-round(11.0 / alpha) + 0.25)


def _convert_inputs(case, seed):
    g = _gen(seed)
    return dict(x=_acts(g, case["M"], case["K"]),
                w=_weights(g, case["N"], case["K"], case["asym"]))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "generate":
        return dict(kind=kind, case=case, step=_Step(case["L"], seed))
    make = dict(linear=_linear_inputs, logits=_logits_inputs, gate_up=_gate_up_inputs,
                block=_block_inputs, arl=_arl_inputs, convert=_convert_inputs)[kind]
    return dict(make(case, seed), kind=kind, case=case)


def run(s):
    kind, c = s["kind"], s["case"]
    if kind == "linear":
        if c["a_bits"] == 16:
            return mq.mq_qlinear_a16(s["a"], s["wq"], 8, s["ws"], s["cs"], *s["fa"], *s["fy"],
                                     c["out_bits"], s["bias"])
        if c["asym"]:
            return mq.mq_qlinear_asym(s["a"], s["rowsum"], s["wq"], c["w_bits"], s["ws"], s["wz"],
                                      s["cs"], *s["fa"], *s["fy"], c["out_bits"], s["bias"],
                                      workspace=s["work"])
        return mq.mq_qlinear(s["a"], s["wq"], c["w_bits"], s["ws"], s["cs"], *s["fa"], *s["fy"],
                             c["out_bits"], s["bias"], workspace=s["work"])
    if kind == "logits":
        a = mq.mq_quantize_act(s["x"], *s["fa"], 8)
        return mq.mq_qlinear_dequant(a, s["wq"], 8, s["ws"], s["cs"], *s["fa"], *s["fy"], 16,
                                     workspace=s["work"])
    if kind == "gate_up":
        a = mq.mq_quantize_act(s["x"], *s["fa"], 8)
        return mq.mq_qlinear_group(a, s["linears"], 8, *s["fa"], c["out_bits"])
    if kind == "block":
        s["graph"].replay()
        o = s["block"].out
        return {k: o[k] for k in ("kr", "v", "probs", "ctx", "h1", "x2", "mul", "h2")}
    if kind == "generate":
        s["step"].graph.replay()
        st = s["step"]
        return {**{k: st.out[k] for k in ("probs", "ctx", "h1", "x2", "mul", "h2")},
                "keys": st.keys, "vals": st.vals}
    if kind == "arl":
        y = mq.mq_arl_forward(s["x"], s["alpha"], s["beta"], c["bits"])
        gx, grads = mq.mq_arl_backward(s["x"], s["grad"], s["alpha"], s["beta"], c["bits"])
        return y, gx, grads[:2]  # the rest of grads is scratch
    sv, x_max, w_max = mq.mq_smooth_scales(s["x"], s["w"], 0.5)
    w_hat = mq.mq_fold_weights(s["w"], sv)
    if c["asym"]:
        packed = mq.mq_pack_weights_asym(w_hat, c["w_bits"], c["per_tensor"])
    else:
        packed = mq.mq_pack_weights(w_hat, c["w_bits"])
    return (sv, x_max, w_max, w_hat) + tuple(packed)


# ---------------------------------------------------------------------------
# What a pass cannot do without: each input read once, each output written
# once, two operations per multiply-add (16-bit by 8-bit products count
# once).

def _linear_work(M, K, N, w_bits, out_bits, a_bits=8, asym=False, bias=False):
    per_col = 8 + 4 * asym + 4 * bias
    return (M * K * a_bits // 8 + N * K * w_bits // 8 + M * N * out_bits // 8 + N * per_col +
            4 * M * asym, 2.0 * M * N * K)


def _block_work(T, keys, causal):
    """The weights and the block's input and output once; with a cache, its
    bytes; attention over `keys` tokens per query (half of them hidden on
    average over a prompt)."""
    d = DIMS
    H, G, D, hid, ffn = d["heads"], d["kv_heads"], d["head_dim"], d["hidden"], d["ffn"]
    wk = hid * (2 * hid + 2 * G * D) + 3 * hid * ffn
    pairs = T * (T + 1) / 2 if causal else T * keys
    probs = 2 * H * T * keys  # written
    cache = 2 * keys * G * D
    out = T * (hid * 2 + hid * 2 + hid + hid + ffn)  # h1, h2, x2, ctx, mul
    return (wk + probs + cache + out + T * hid * 2,
            2.0 * T * wk + 4.0 * H * D * pairs)


def work(case):
    kind = case["kind"]
    if kind == "linear":
        b, f = _linear_work(case["M"], case["K"], case["N"], case["w_bits"], case["out_bits"],
                            case["a_bits"], case["asym"], case["bias"])
    elif kind == "logits":
        M, K, N = case["M"], case["K"], case["N"]
        b, f = M * K * 4 + N * K + N * 8 + M * N * 4, 2.0 * M * N * K
    elif kind == "gate_up":
        M, K, N = case["M"], case["K"], case["N"]
        b = M * K * 4 + 2 * N * (K + 8) + 2 * M * N * case["out_bits"] // 8
        f = 4.0 * M * N * K
    elif kind == "block":
        b, f = _block_work(case["T"], case["T"], True)
    elif kind == "generate":
        b, f = _block_work(1, case["L"], False)
    elif kind == "arl":
        n = case["M"] * case["K"]
        b, f = n * 16, n * 20.0  # x and g read, y and gx written
    else:
        x, w = case["M"] * case["K"], case["N"] * case["K"]
        b, f = 4 * x + 8 * w + w * case["w_bits"] // 8, x + 6.0 * w
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind in ("block", "generate"):
        # integer codes; the softmax goes through exp, whose last bit is
        # free, so a code may move one step at a rounding tie (none seen)
        return {"rel": 0.0, "differ": 1e-6}
    if kind == "arl":
        # the outputs and input gradients are fixed bit for bit; the two
        # parameter gradients are sums of fp64 terms in any order (2e-15 to
        # 1e-13 seen between orders, more where the sum cancels)
        return {"rel": 1e-12}
    return "exact"  # integer codes, single IEEE operations, or dequantized codes


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, from the definitions.

def _codes(v, fmt, bits):
    """clamp(rint(v / alpha) + zp) of fp64 values already divided by alpha."""
    lo, hi = -(1 << (bits - 1)), (1 << (bits - 1)) - 1
    return (torch.round(v.clamp(-1e9, 1e9)) + fmt[1]).clamp(lo, hi)


def _div32(a, b):
    """The correctly rounded fp32 quotient of fp32 values, as fp64 (the
    definitions divide once in fp32; a quotient rounded to fp64 first rounds
    to the same fp32)."""
    b = b.double() if isinstance(b, torch.Tensor) else np.float64(np.float32(b))
    return (a.double() / b).float().double()


def _quantize64(x, fmt, bits):
    return _codes(_div32(x, fmt[0]).clamp(-2.0 ** 20, 2.0 ** 20), fmt, bits)


def _requant64(c, scale_product, fy, bits):
    """The fixed-point rescale of integer sums c (fp64 holding integers,
    saturated to int32): M = M0 2^-sh, floor((c M0 + 2^(sh-1)) / 2^sh)."""
    c = c.clamp(-2.0 ** 31, 2.0 ** 31 - 1).to(torch.int64)
    f, e = np.frexp(np.atleast_1d(scale_product.cpu().numpy()) / np.float64(np.float32(fy[0])))
    m0 = np.rint(np.ldexp(f, 31)).astype(np.int64)
    e = np.where(m0 == 1 << 31, e + 1, e)
    m0 = np.where(m0 == 1 << 31, 1 << 30, m0)
    sh = 31 - e
    assert sh.min() >= 1 and sh.max() < 63
    m0, sh = (torch.as_tensor(v.astype(np.int64), device=c.device) for v in (m0, sh))
    r = (c * m0 + (torch.ones_like(sh) << (sh - 1))) >> sh
    lo, hi = -(1 << (bits - 1)), (1 << (bits - 1)) - 1
    return (r + fy[1]).clamp(lo, hi)


def _pack64(w, bits):
    q = 127 if bits == 8 else 7
    s = _div32(w.abs().amax(1), q)
    s = torch.where(s > 0, s, torch.ones_like(s))
    return torch.round(_div32(w, s[:, None]).clamp(-q, q)), s


def _asym_format64(lo, hi, bits):
    qmax = float(2 ** bits - 1)
    a = ((hi.double() - lo.double()) / qmax).float()
    a = torch.where(a > 0, a, torch.ones_like(a))
    z = torch.round(-lo.double() / a.double()).clamp(0, qmax) - 2 ** (bits - 1)
    return a, z


def _pack_asym64(w, bits, per_tensor=False):
    lo, hi = w.amin(1).clamp(max=0), w.amax(1).clamp(min=0)
    if per_tensor:
        lo, hi = lo.min().expand_as(lo), hi.max().expand_as(hi)
    a, z = _asym_format64(lo, hi, bits)
    half = 2 ** (bits - 1)
    q = (torch.round(_div32(w, a[:, None])) + z[:, None]).clamp(-half, half - 1)
    return q, a, z


def _matmul64(a, w):
    """a [M][K] times w [N][K]^T in fp64 (exact: integers below 2^53), in
    column blocks to bound the memory."""
    step = max(1, (1 << 28) // max(1, w.shape[1]))
    return torch.cat([a.double() @ w[i:i + step].double().T.contiguous()
                      for i in range(0, w.shape[0], step)], 1)


def _linear64(a, fa, wq, ws, fy, bits, wz=None, bias=None):
    prod = np.float64(np.float32(fa[0])) * ws.double()
    w = wq.double() if wz is None else wq.double() - wz[:, None]
    c = _matmul64(a.double() - fa[1], w)
    if bias is not None:
        c = c + torch.round((bias.double() / prod).clamp(-2.0 ** 30, 2.0 ** 30))
    return _requant64(c, prod, fy, bits)


def _block64(h0, w, gamma, keys=None, vals=None, pos0=0):
    """The block's stages as fp64 tensors of integer codes; keys and vals:
    the cached codes before this token ([n][G D] and [G D][n])."""
    from paper_2408_13933_amd.block import STAGE_BITS as B, formats
    d = DIMS
    H, G, D = d["heads"], d["kv_heads"], d["head_dim"]
    fm = formats(RANGES, mq.mq_act_params)

    def scale(st):
        return np.float64(np.float32(fm[st][0]))

    def real(o, st):
        return scale(st) * (o.double() - fm[st][1])

    def code(v, st):
        return _codes(v / scale(st), fm[st], B[st])

    def lin(x, src, name, st):
        q, s = packed[name]
        return _linear64(x, fm[src], q, s, fm[st], B[st]).double()

    def norm(x, st_in, gm, st):
        xi = x.double() - fm[st_in][1]
        a = scale(st_in)
        ms = a * a * (xi * xi).sum(1, keepdim=True) / x.shape[1] + np.float64(np.float32(d["eps"]))
        return code(a * xi * gm.double() / torch.sqrt(ms), st)

    def rope(x, heads, st_in, st):
        T = x.shape[0]
        u = real(x, st_in).view(T, heads, 2, D // 2)
        i = torch.arange(D // 2, dtype=torch.float64, device=x.device)
        inv = torch.pow(torch.full_like(i, d["rope_base"]), -2 * i / D)
        ang = (torch.arange(T, dtype=torch.float64, device=x.device) + pos0)[:, None] * inv
        c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
        y = torch.stack([u[:, :, 0] * c - u[:, :, 1] * s, u[:, :, 1] * c + u[:, :, 0] * s], 2)
        return code(y.reshape(T, heads * D), st)

    packed = {n: _pack64(v, 8) for n, v in w.items()}
    o = dict(h0=_quantize64(h0, fm["h0"], 16))
    o["x1"] = norm(o["h0"], "h0", gamma[0], "x1")
    q, k = lin(o["x1"], "x1", "q_proj", "q"), lin(o["x1"], "x1", "k_proj", "k")
    v = lin(o["x1"], "x1", "v_proj", "v")
    qr, kr = rope(q, H, "q", "qr"), rope(k, G, "k", "kr")
    o["kr"], o["v"] = kr, v
    if keys is not None:
        kr, v = torch.cat([keys.double(), kr]), torch.cat([vals.double().T, v])
    T, L = qr.shape[0], kr.shape[0]
    probs, ctx = [], []
    s1 = torch.tensor(scale("qr") * scale("kr"), dtype=torch.float64)
    s2 = torch.tensor(scale("probs") * scale("v"), dtype=torch.float64)
    sm = np.float64(np.float32(fm["scores"][0] / D ** 0.5))
    hidden = torch.ones(T, L, dtype=torch.bool, device=qr.device).triu(L - T + 1)
    for h in range(H):
        g = h // (H // G)
        a = qr[:, h * D:(h + 1) * D] - fm["qr"][1]
        b = kr[:, g * D:(g + 1) * D] - fm["kr"][1]
        sc = _requant64(_matmul64(a, b), s1, fm["scores"], 16).double()
        z = (sm * sc).masked_fill(hidden, -math.inf)
        e = torch.exp(z - z.amax(1, keepdim=True))
        p = code(e / e.sum(1, keepdim=True), "probs")
        probs.append(p)
        c = _matmul64(p - fm["probs"][1], (v[:, g * D:(g + 1) * D] - fm["v"][1]).T.contiguous())
        ctx.append(_requant64(c, s2, fm["ctx"], 8).double())
    o["probs"], o["ctx"] = torch.stack(probs), torch.cat(ctx, 1)
    ov = lin(o["ctx"], "ctx", "o_proj", "o")
    o["h1"] = code(real(o["h0"], "h0") + real(ov, "o"), "h1")
    o["x2"] = norm(o["h1"], "h1", gamma[1], "x2")
    gt, up = lin(o["x2"], "x2", "gate_proj", "gate"), lin(o["x2"], "x2", "up_proj", "up")
    gv = real(gt, "gate")
    su = code(gv / (1 + torch.exp(-gv)), "silu")
    o["mul"] = code(real(su, "silu") * real(up, "up"), "mul")
    dn = lin(o["mul"], "mul", "down_proj", "down")
    o["h2"] = code(real(o["h1"], "h1") + real(dn, "down"), "h2")
    return o


def _nibbles(q):
    q = q.to(torch.int64) & 15
    return (q[:, 0::2] | (q[:, 1::2] << 4)).to(torch.uint8)


def exact(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind == "linear":
        x = _acts(g, case["M"], case["K"])
        w = _weights(g, case["N"], case["K"], case["asym"])
        bias = torch.randn(case["N"], generator=g, device="cuda") * B_STD if case["bias"] else None
        fa = mq.mq_act_params(-70.0, 80.0, case["a_bits"])
        fy = _out_format(case["K"], case["asym"], case["out_bits"])
        q, s, z = (_pack_asym64(w, case["w_bits"]) if case["asym"]
                   else _pack64(w, case["w_bits"]) + (None,))
        return _linear64(_quantize64(x, fa, case["a_bits"]), fa, q, s, fy, case["out_bits"],
                         z, bias)
    if kind == "logits":
        x = _acts(g, case["M"], case["K"])
        fa, fy = mq.mq_act_params(-70.0, 80.0, 8), _out_format(case["K"], False, 16)
        q, s = _pack64(_weights(g, case["N"], case["K"]), 8)
        y = torch.cat([_linear64(_quantize64(x, fa, 8), fa, q[i:i + 32768], s[i:i + 32768], fy, 16)
                       .to(torch.int16) for i in range(0, case["N"], 32768)], 1)
        return (y.double() - fy[1]) * np.float64(np.float32(fy[0]))
    if kind == "gate_up":
        a = _acts(g, case["M"], case["K"])
        fa = mq.mq_act_params(-70.0, 80.0, 8)
        a = _quantize64(a, fa, 8)
        fy = _out_format(case["K"], False, case["out_bits"])
        return [_linear64(a, fa, *_pack64(_weights(g, case["N"], case["K"]), 8),
                          (fy[0] * (1 + k / 8), fy[1]), case["out_bits"]) for k in range(2)]
    if kind == "block":
        o = _block64(*_block_data(case["T"], seed))
        return {k: o[k] for k in ("kr", "v", "probs", "ctx", "h1", "x2", "mul", "h2")}
    if kind == "generate":
        st = _Step(case["L"], seed)  # for the cached codes only
        L = case["L"]
        keys, vals = st.keys.clone(), st.vals.clone()
        o = _block64(*_block_data(1, seed), keys[:L - 1], vals[:, :L - 1], pos0=L - 1)
        keys[L - 1], vals[:, L - 1] = o["kr"][0].to(torch.int8), o["v"][0].to(torch.int8)
        return {**{k: o[k] for k in ("probs", "ctx", "h1", "x2", "mul", "h2")}, "keys": keys,
                "vals": vals}
    if kind == "arl":
        s = _arl_inputs(case, seed)
        top = 2.0 ** case["bits"] - 1
        a, b = (np.float64(np.float32(s[k])) for k in ("alpha", "beta"))
        t = _div32(s["x"], s["alpha"])
        u = (torch.round(t).float() - torch.tensor(s["beta"], device="cuda")).double()
        c = u.clamp(0, top)
        inside = (u >= 0) & (u <= top)
        gr = s["grad"].double()
        ga = (gr * (c + b - torch.where(inside, t, torch.zeros_like(t)))).sum()
        gb = (gr * torch.where(inside, 0.0, float(a))).sum()
        return a * (c + b), torch.where(inside, gr, torch.zeros_like(gr)), torch.stack([ga, gb])
    s = _convert_inputs(case, seed)
    xm, wm = s["x"].abs().amax(0), s["w"].abs().amax(0)
    sv = torch.sqrt(xm.double()) / torch.sqrt(wm.double())
    w_hat = s["w"] * sv.float()
    if case["asym"]:
        q, a, z = _pack_asym64(w_hat, case["w_bits"], case["per_tensor"])
        extra = (z,)
    else:
        q, a = _pack64(w_hat, case["w_bits"])
        extra = ()
    cs = q.double().sum(1)
    return (sv, xm, wm, s["w"].double() * sv, q if case["w_bits"] == 8 else _nibbles(q), a,
            *extra, cs)
