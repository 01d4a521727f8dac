"""What the library is measured on: the calls a user of it makes, over the range of sizes and settings they are made with.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs, weights and buffers a user's program holds before the call
    run(state)          one pass through the public entry points, with everything it computes
    work(case)          bytes and operations the pass cannot do without
    tolerance(case)     how far another correct implementation may be off

Kinds of case:

    linear      one quantized linear layer applied to a batch of tokens (`DsfqLinear`)
    mlp         fc1 and fc2 of an MLP block, fc2 reading fc1's output with the GELU applied on the way (`pre_gelu`)
    mlp_apart   fc1 and fc2, each on its own resident input: the two halves without the activation between them
    block       the four linear layers of a transformer block with the LayerNorms in front of qkv and fc1 fused in
    asymmetric  one layer with affine activation codes (a zero point per token)
    prepare     making a layer: rotated statistic of a calibration batch, smoothing factor, weight codes (`DsfqLinear(...)`)
    calibrate   one refinement step of a layer's smoothing factor and weight steps: loss, derivatives, descent
    sampling    the two reductions over a sample's activations that choose a calibration set

Activations are heavy-tailed (Student-t, 3 degrees of freedom) with a few outlier channels and five large tokens per frame,
weights N(0, 0.02): the distributions of the repository's synthetic inputs, drawn on the device.
"""
import math

import torch

import paper_2509_21302_amd as q

DEV = "cuda:0"
FRAME = 1374            # tokens of a frame: 1369 patches and 5 special tokens
MOST_MACS = 137400 * 1024 * 4096      # of one layer: fc1 / fc2 at 100 frames
POWERS = (128, 256, 512, 1024, 2048, 4096, 8192)
PALEY = (768, 1536, 3072, 6144, 1280, 2560, 5120, 1792, 3584)


def listed():
    return [
        # the smallest layer anyone runs: 64 float32 tokens, 128 features; a call is launches and host work
        dict(name="tiny_f32", kind="linear", tokens=64, k=128, n=128, dtype="f32", bits=4, act_bits=4, bias=False),
        # one frame through a qkv layer: the frame-attention blocks of a single-image request
        dict(name="qkv_1_frame", kind="linear", tokens=FRAME, k=1024, n=3072, dtype="bf16", bits=4, act_bits=4, bias=True),
        # a token count and a width that fill no tile, as other image sizes and pruned layers have
        dict(name="ragged_2048", kind="linear", tokens=5207, k=2048, n=1040, dtype="bf16", bits=4, act_bits=4, bias=True),
        # the 768-wide layers of a base-size backbone (a Hadamard size 2^n * 12)
        dict(name="fc1_768_8_frames", kind="linear", tokens=8 * FRAME, k=768, n=3072, dtype="bf16", bits=4, act_bits=4, bias=True),
        # the MLP of a block over 8 frames, as the model runs it: fc1, GELU, fc2
        dict(name="mlp_8_frames", kind="mlp", tokens=8 * FRAME, k=1024, n=4096),
        # all linear layers of one block at global attention over 24 frames
        dict(name="block_24_frames", kind="block", tokens=24 * FRAME),
        # 100 frames, the throughput workload of the benchmark: fc1 and fc2 with their inputs resident
        dict(name="mlp_apart_100_frames", kind="mlp_apart", tokens=100 * FRAME, k=1024, n=4096, bits=4),
        # the 8-bit setting at 24 frames
        dict(name="mlp_apart_8bit_24_frames", kind="mlp_apart", tokens=24 * FRAME, k=1024, n=4096, bits=8),
        # affine activation codes at 8 frames
        dict(name="asymmetric_fc1_8_frames", kind="asymmetric", tokens=8 * FRAME, k=1024, n=4096),
        # quantizing a layer when a model is loaded: the largest weight, one calibration frame
        dict(name="prepare_fc2", kind="prepare", tokens=FRAME, k=4096, n=1024, bits=4),
        # one step of calibrating a layer on one frame, the step a calibration repeats for every layer
        dict(name="calibrate_qkv", kind="calibrate", tokens=FRAME, k=1024, n=3072, bits=4, static=False),
        # statistics of one 24-frame sample while a calibration set is chosen
        dict(name="sampling_24_frames", kind="sampling", frames=24, tokens=FRAME, k=1024),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _tokens(rng, k, n, lo=16, share=1.0):
    """Tokens of a call: whole frames, or any count (mostly odd sizes), while a layer costs no more than the largest listed one."""
    hi = max(lo, min(100 * FRAME, int(share * MOST_MACS) // (k * n)))
    t = _spread(rng, lo, hi)
    return t // FRAME * FRAME if t >= FRAME and rng.random() < 0.4 else t


def draw(rng):
    kind = rng.choice(["linear"] * 6 + ["mlp", "mlp_apart", "block", "asymmetric"] * 2 + ["prepare", "calibrate"] * 2 + ["sampling"])
    if kind == "linear":
        where = rng.random()
        k = rng.choice((1024, 2048, 4096)) if where < 0.6 else rng.choice(POWERS) if where < 0.8 else rng.choice(PALEY)
        n = 16 * _spread(rng, 8, 256)
        bits, act_bits = rng.choice([(4, 4)] * 5 + [(8, 8), (6, 6), (4, 8)])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        # float32 rows and the sizes beside 1024, 2048 and 4096 take the general rotation: a quarter of the largest layer
        share = 1.0 if dtype == "bf16" and k in (1024, 2048, 4096) else 0.25
        return dict(kind=kind, tokens=_tokens(rng, k, n, share=share), k=k, n=n, dtype=dtype, bits=bits, act_bits=act_bits, bias=rng.random() < 0.8)
    if kind == "block":
        return dict(kind=kind, tokens=_tokens(rng, 1024, 4096, share=0.4))
    if kind in ("mlp", "mlp_apart"):
        k, n = rng.choice([(1024, 4096)] * 3 + [(1024, 2048), (2048, 4096)])
        case = dict(kind=kind, tokens=_tokens(rng, k, n, share=0.8), k=k, n=n)
        return dict(case, bits=rng.choice([4, 4, 6, 8])) if kind == "mlp_apart" else case
    if kind == "asymmetric":
        k, n = rng.choice((1024, 2048, 4096)), 16 * _spread(rng, 8, 256)
        return dict(kind=kind, tokens=_tokens(rng, k, n), k=k, n=n)
    if kind == "prepare":
        k = rng.choice((1024, 2048, 4096))
        return dict(kind=kind, tokens=_spread(rng, 100, 4 * FRAME), k=k, n=128 * _spread(rng, 1, 32), bits=rng.choice([4, 4, 6, 8]))
    if kind == "calibrate":
        return dict(kind=kind, tokens=_spread(rng, 64, 2 * FRAME), k=rng.choice((128, 512, 1024, 1024, 2048, 4096)), n=16 * _spread(rng, 4, 256),
                    bits=rng.choice([4, 4, 6, 8]), static=rng.random() < 0.3)
    return dict(kind="sampling", frames=_spread(rng, 2, 100), tokens=_spread(rng, 200, FRAME), k=rng.choice((1024, 2048)))


# ---------------------------------------------------------------------------------------------------------------- inputs
class _Make:
    """Tensors from one seed, drawn on the device."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def normal(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV) * std

    def activations(self, tokens, k, dtype=torch.bfloat16):
        """[tokens, k]: Student-t body, 1 % outlier channels x 50, the first five tokens of every frame x 20."""
        out = torch.empty(tokens, k, dtype=dtype, device=DEV)
        channel = torch.ones(k, device=DEV)
        channel[torch.randperm(k, generator=self.g, device=DEV)[: max(1, k // 100)]] = 50.0
        for r in range(0, tokens, 8 * FRAME):
            rows = min(8 * FRAME, tokens - r)
            chi = self.normal(rows, k).square_()
            for _ in range(2):
                chi += self.normal(rows, k).square_()
            x = self.normal(rows, k).mul_(chi.mul_(1.0 / 3.0).rsqrt_()).mul_(channel)
            x[torch.arange(r, r + rows, device=DEV) % FRAME < 5] *= 20.0
            out[r : r + rows] = x
        return out

    def weights(self, n, k, dtype=torch.bfloat16):
        return self.normal(n, k, std=0.02).to(dtype)

    def bias(self, n):
        return self.normal(n, std=0.02).to(torch.bfloat16)

    def signs(self, k):
        return (torch.randint(0, 2, (k,), generator=self.g, device=DEV, dtype=torch.int8) * 2 - 1).contiguous()

    def layer(self, k, n, calibration, dtype=torch.bfloat16, bias=True, **settings):
        return q.DsfqLinear(self.weights(n, k, dtype), self.bias(n) if bias else None, self.signs(k), calibration, **settings)


def _gelu(x):
    return torch.nn.functional.gelu(x.float()).to(torch.bfloat16)


def prepare(case, seed):
    q.qvggt_init()
    make, kind, tokens = _Make(seed), case["kind"], case["tokens"]
    if kind == "linear":
        dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        X = make.activations(tokens, case["k"], dtype)
        layer = make.layer(case["k"], case["n"], X[:FRAME], dtype, case["bias"], bits=case["bits"], act_bits=case["act_bits"])
        return dict(case=case, X=X, layer=layer)
    if kind == "mlp":
        X = make.activations(tokens, case["k"])
        fc1 = make.layer(case["k"], case["n"], X[:FRAME])
        fc2 = make.layer(case["n"], case["k"], _gelu(fc1(X[:FRAME].contiguous())), pre_gelu=True)
        return dict(case=case, X=X, fc1=fc1, fc2=fc2)
    if kind == "mlp_apart":
        X, H = make.activations(tokens, case["k"]), make.activations(tokens, case["n"])
        return dict(case=case, X=X, H=H, fc1=make.layer(case["k"], case["n"], X[:FRAME], bits=case["bits"]),
                    fc2=make.layer(case["n"], case["k"], H[:FRAME], bits=case["bits"]))
    if kind == "block":
        d, h = 1024, 4096
        X, A, R = make.activations(tokens, d), make.activations(tokens, d), make.activations(tokens, d)      # block input, attention output, residual
        gamma, beta = [make.normal(d, std=0.1) + 1.0 for _ in range(2)], [make.normal(d, std=0.1) for _ in range(2)]

        def normed(x, i):
            return torch.nn.functional.layer_norm(x[:FRAME].float(), (d,), gamma[i], beta[i], 1e-5).to(torch.bfloat16)
        s = dict(case=case, X=X, A=A, R=R, gamma=gamma, beta=beta, qkv=make.layer(d, 3 * d, normed(X, 0)), proj=make.layer(d, d, A[:FRAME]),
                 fc1=make.layer(d, h, normed(R, 1)))
        s["fc2"] = make.layer(h, d, _gelu(s["fc1"](normed(R, 1))), pre_gelu=True)
        s["codes"] = torch.empty(q.qvggt_e2m3_bytes(tokens, d), dtype=torch.uint8, device=DEV)
        s["steps"] = torch.empty(tokens, dtype=torch.float32, device=DEV)
        return s
    if kind == "asymmetric":
        k, n = case["k"], case["n"]
        X = make.activations(tokens, k)
        layer = make.layer(k, n, X[:FRAME])
        sums = torch.empty(n, dtype=torch.float32, device=DEV)
        q.qvggt_weight_code_sums(layer.Wq, n, k, sums)
        return dict(case=case, X=X, layer=layer, sums=sums, codes=torch.empty(q.qvggt_e2m3_bytes(tokens, k), dtype=torch.uint8, device=DEV))
    if kind == "prepare":
        return dict(case=case, W=make.weights(case["n"], case["k"]), bias=make.bias(case["n"]), signs=make.signs(case["k"]),
                    calibration=make.activations(tokens, case["k"]))
    if kind == "calibrate":
        k, n = case["k"], case["n"]
        X, W, signs, bias = make.activations(tokens, k), make.weights(n, k), make.signs(k), make.bias(n)
        R, V = torch.empty(tokens, k, device=DEV), torch.empty(n, k, device=DEV)
        q.qvggt_rotate_rows(X, signs, R)
        q.qvggt_rotate_rows(W, signs, V)
        reference = X.float() @ W.float().t() + bias.float()
        # the starting point: the closed-form factor, absmax steps
        c = R.abs().amax(0).clamp_(min=1e-5).sqrt_() / V.abs().amax(0).clamp_(min=1e-5).sqrt_()
        qmax = float(2 ** (case["bits"] - 1) - 1)
        w_step = (V * c).abs().amax(1) / qmax
        x_step = ((R / c).abs().amax() / qmax).reshape(1) * 0.25 if case["static"] else None
        return dict(case=case, R=R, V=V, reference=reference, bias=bias, c=c, w_step=w_step, x_step=x_step,
                    workspace=torch.empty(q.qvggt_calib_workspace_bytes(tokens, n, k), dtype=torch.uint8, device=DEV))
    assert kind == "sampling", kind
    frames, count = case["frames"], tokens * case["k"]
    return dict(case=case, A=make.activations(frames * tokens, case["k"]).view(frames, count),
                workspace=torch.empty(q.qvggt_nfds_workspace_bytes(frames, count, q.QVGGT_BF16), dtype=torch.uint8, device=DEV))


# ------------------------------------------------------------------------------------------------------------------ a pass
def _f32(*shape):
    return torch.empty(*shape, dtype=torch.float32, device=DEV)


def _normed_linear(s, X, i, layer):
    """LayerNorm, then the layer, the normalisation inside the layer's first kernel."""
    tokens, d = X.shape
    Y = torch.empty(tokens, layer.N, dtype=torch.bfloat16, device=DEV)
    q.qvggt_layernorm_rotate_smooth_quant_e2m3(X, s["gamma"][i], s["beta"][i], 1e-5, layer.signs, layer.inv_smooth, s["codes"], s["steps"])
    q.qvggt_e2m3_gemm(s["codes"], s["steps"], layer.Wf, layer.w_scale, layer.bias, tokens, layer.N, d, Y)
    return Y


def run(s):
    case = s["case"]
    kind, tokens = case["kind"], case["tokens"]
    if kind == "linear":
        return s["layer"](s["X"])
    if kind == "mlp":
        hidden = s["fc1"](s["X"])
        return [hidden, s["fc2"](hidden)]
    if kind == "mlp_apart":
        return [s["fc1"](s["X"]), s["fc2"](s["H"])]
    if kind == "block":
        qkv = _normed_linear(s, s["X"], 0, s["qkv"])
        proj = s["proj"](s["A"])
        hidden = _normed_linear(s, s["R"], 1, s["fc1"])
        return [qkv, proj, hidden, s["fc2"](hidden)]
    if kind == "asymmetric":
        layer, step, zero = s["layer"], _f32(tokens), _f32(tokens)
        Y = torch.empty(tokens, layer.N, dtype=torch.bfloat16, device=DEV)
        q.qvggt_rotate_smooth_quant_asym_e2m3(s["X"], layer.signs, layer.inv_smooth, s["codes"], step, zero)
        q.qvggt_e2m3_gemm_shifted(s["codes"], step, zero, layer.Wf, layer.w_scale, s["sums"], layer.bias, tokens, layer.N, layer.K, Y)
        return [Y, step, zero]
    if kind == "prepare":
        layer = q.DsfqLinear(s["W"], s["bias"], s["signs"], s["calibration"], bits=case["bits"])
        return [layer.Wq, layer.Wf if layer.packed else layer.Wb, layer.w_scale, layer.inv_smooth]
    if kind == "calibrate":
        c, w_step = s["c"].clone(), s["w_step"].clone()
        loss, grad_c, grad_w = _f32(1), _f32(case["k"]), _f32(case["n"])
        grad_x = _f32(1) if case["static"] else None
        q.qvggt_calib_loss_grad(s["R"], s["V"], s["reference"], s["bias"], c, w_step, s["x_step"], case["bits"], loss, grad_c, grad_w, grad_x,
                                s["workspace"])
        q.qvggt_calib_descent_step(c, grad_c, 5e-3)
        q.qvggt_calib_descent_step(w_step, grad_w, 5e-2)
        return [loss, grad_c, grad_w, c, w_step] + ([grad_x] if case["static"] else [])
    A = s["A"]
    frames = A.shape[0]
    mean, var, corr = _f32(frames), _f32(frames), _f32(1, frames - 1)
    q.qvggt_nfds_moments(A, mean, var, s["workspace"])
    q.qvggt_nfds_frame_correlation(A.view(1, *A.shape), corr, s["workspace"])
    return [mean, var, corr]


# -------------------------------------------------------------------------------------------------------- what a pass needs
def _linear_work(tokens, k, n, bits=4, x_bytes=2, affine=False):
    """Input, weight codes, steps, multipliers, signs, bias read once, output written once; the products."""
    read = tokens * k * x_bytes + n * k * bits / 8 + 4 * n + 5 * k + 2 * n + (4 * n if affine else 0)
    return read + 2 * tokens * n + (8 * tokens if affine else 0), 2.0 * tokens * n * k


def work(case):
    kind, t, k, n = case["kind"], case["tokens"], case.get("k", 1024), case.get("n", 4096)
    if kind == "linear":
        parts = [_linear_work(t, k, n, case["bits"], 4 if case["dtype"] == "f32" else 2)]
    elif kind in ("mlp", "mlp_apart"):
        parts = [_linear_work(t, k, n, case.get("bits", 4)), _linear_work(t, n, k, case.get("bits", 4))]
    elif kind == "block":
        parts = [_linear_work(t, a, b) for a, b in ((1024, 3072), (1024, 1024), (1024, 4096), (4096, 1024))]
    elif kind == "asymmetric":
        parts = [_linear_work(t, k, n, affine=True)]
    elif kind == "prepare":      # weights and calibration rows read, two forms of the codes written; the rotations of both
        parts = [(2.0 * n * k + 2.0 * t * k + n * k * (1.25 if case["bits"] == 4 else 2.0) + 4 * n + 5 * k, (n + t) * k * math.log2(k))]
    elif kind == "calibrate":    # rotated activations, rotated weights and the reference output read; three products
        parts = [(4.0 * (t * k + n * k + t * n) + 12 * (k + n), 6.0 * t * n * k)]
    else:                        # the sample read once by each of the two reductions
        parts = [(2 * 2.0 * case["frames"] * t * k, 5.0 * case["frames"] * t * k)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    """About four times what the library was seen to be off from the same path in 64 bits (weights included), over the listed and
    some 40 drawn cases."""
    kind = case["kind"]
    if kind in ("linear", "mlp_apart", "asymmetric"):
        # outputs in bf16; a code on a rounding knife edge moves one row (activations) or one column (weights): rel 5.7e-4, and
        # 0.34 of the root mean square where that row is one of the large tokens
        return {"rel": 2.5e-3, "max": 0.95}
    if kind in ("mlp", "block"):
        # two quantizers in a row, and the normalised values rounded to bf16 in between: rel 4.7e-3 on the last layer
        return {"rel": 0.02, "max": 0.98}
    if kind == "prepare":
        # steps and multipliers 9e-8; codes on a knife edge: 2.5e-6 of them in a large layer, one or two in a small one
        return {"rel": 5e-7, "max": 2e-6, "differ": 1e-4}
    if kind == "calibrate":
        # the sums in 64 bits, codes as they are: rel 4.9e-6, 1.8e-5 of a single derivative
        return {"rel": 2e-5, "max": 1e-4}
    # sums in double, results rounded to float32 once
    return {"rel": 2e-7, "max": 4e-7}
