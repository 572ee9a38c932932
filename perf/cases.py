"""The work whose speed this repository watches: calls through the public
binding (``paper_2110_15456_amd``) as a program that trains or serves with BFP
makes them, over the range of sizes, widths, roundings and group sizes that
the benchmark, the tests and the paper's models span.

Kinds of case
  linear    the forward of a linear layer with its weights held in BFP: the
            FP32 input converted, then the BFP GEMM; FP32 output
  converted the same with the output converted to BFP in the GEMM's epilogue
            (the next layer's input)
  step      a training step of a linear layer, or of a convolution as its
            im2col GEMM: both groupings of X and dY (stochastic rounding), the
            GEMMs Y, dX and dW, and the weight update with both groupings of
            the new weights, into buffers held across steps
  quantize  one conversion of a tensor along any of its axes, and its inverse
  adaptive  the converter of the adaptive scheme, the choice of 2 or 4 bits
            from its sums, and the forward GEMM at that width
  packed    a linear layer with input and weights in the packed 3-bit-chunk
            storage

Inputs are drawn on the GPU from the seed: half-normal activations, N(0, 0.02)
weights, Laplace(0, 1e-4) gradients with 1% of the entries scaled by 100.
"""
from __future__ import annotations

import math

import torch

import paper_2110_15456_amd as fb

LR = 1e-3
ALPHA, BETA = 0.6, 0.3  # the adaptive scheme's threshold constants


def listed():
    return [
        # the smallest call: one 256-wide layer, where launches and the host show
        dict(name="linear_256", kind="linear", tokens=256, d_in=256, d_out=256, m_x=4, m_w=4, g=16),
        # a few tokens against the FFN up-projection's weights: serving
        dict(name="linear_few_tokens", kind="linear", tokens=16, d_in=4096, d_out=16384, m_x=4, m_w=4, g=16),
        # the QKV projection of a transformer block on a full batch of tokens
        dict(name="linear_qkv", kind="linear", tokens=8192, d_in=4096, d_out=12288, m_x=4, m_w=4, g=16),
        # the FFN up-projection at the lowest width, its output converted for the next layer
        dict(name="converted_ffn_up", kind="converted", tokens=8192, d_in=4096, d_out=16384, m_x=2, m_w=2, m_y=2,
             rounding="nearest"),
        # one FFN training step at the schedule's last width: the benchmark's largest step
        dict(name="step_ffn_m6", kind="step", tokens=8192, d_in=4096, d_out=16384, m=6),
        # one GPU's share of that step under 8-way data parallelism, at the schedule's first width
        dict(name="step_ffn_share_m2", kind="step", tokens=1024, d_in=4096, d_out=16384, m=2),
        # training steps of ResNet-18 convolutions at batch 256 (im2col): conv2_x, the widest
        # spread of M and N, and conv4_x
        dict(name="step_conv2_m2", kind="step", tokens=256 * 56 * 56, d_in=576, d_out=64, m=2),
        dict(name="step_conv4_m4", kind="step", tokens=256 * 14 * 14, d_in=2304, d_out=256, m=4),
        # the converter alone on 64M gradients with stochastic rounding
        dict(name="quantize_grads_64m", kind="quantize", outer=8192, length=8192, inner=1, g=16, m=4,
             rounding="stochastic", values="grads"),
        # a batch of weight matrices regrouped along their middle axis, ragged inner size, groups of 32
        dict(name="quantize_middle_axis", kind="quantize", outer=24, length=1056, inner=777, g=32, m=6,
             rounding="nearest", values="weights"),
        # the adaptive converter in front of the out-projection
        dict(name="adaptive_out_proj", kind="adaptive", tokens=8192, d_in=4096, d_out=4096, m_w=4),
        # the out-projection with both operands in packed storage
        dict(name="packed_out_proj", kind="packed", tokens=8192, d_in=4096, d_out=4096, m_x=4, m_w=4),
    ]


def _log(rng, lo, hi, multiple=1):
    """A size spread over the logarithm of [lo, hi], a multiple of `multiple`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(multiple, int(round(v / multiple)) * multiple)


def draw(rng):
    kind = rng.choice(["linear", "linear", "converted", "step", "step", "quantize", "quantize", "adaptive", "packed"])
    widths = [2, 4, 4, 6, 8]
    if kind == "quantize":
        g = rng.choice([8, 16, 16, 32])
        length = _log(rng, 64, 8192, 32)
        inner = rng.choice([1, 1, _log(rng, 16, 4096)])
        total = _log(rng, 1 << 14, 1 << 26)
        return dict(kind=kind, outer=max(1, total // (length * inner)), length=length, inner=inner, g=g,
                    m=rng.choice(widths), rounding=rng.choice(["nearest", "stochastic"]),
                    values=rng.choice(["half_normal", "weights", "grads"]))
    if kind == "step":
        tokens, d_in, d_out = _log(rng, 128, 200704, 16), _log(rng, 64, 4608, 16), _log(rng, 64, 16384, 16)
        while tokens * d_in * d_out > 8192 * 4096 * 8192 or tokens * max(d_in, d_out) > 1 << 28:
            tokens = max(128, tokens // 32 * 16)
        return dict(kind=kind, tokens=tokens, d_in=d_in, d_out=d_out, m=rng.choice([2, 4, 6]))
    tokens, d_in = _log(rng, 1, 16384), _log(rng, 64, 16384, 64)
    d_out = _log(rng, 64, 16384, 16)
    while tokens * d_in * d_out > 8192 * 4096 * 16384:
        tokens = max(1, tokens // 2)
    if kind == "linear":
        return dict(kind=kind, tokens=tokens, d_in=d_in, d_out=d_out + rng.choice([0, 0, 0, -7]), m_x=rng.choice(widths),
                    m_w=rng.choice(widths), g=rng.choice([16, 16, 16, 16, 32, 8, 64]))
    if kind == "converted":
        m = rng.choice([2, 4, 4, 6])
        return dict(kind=kind, tokens=tokens, d_in=d_in, d_out=d_out, m_x=m, m_w=rng.choice([2, 4, 6]), m_y=m,
                    rounding=rng.choice(["nearest", "stochastic"]))
    if kind == "adaptive":
        return dict(kind=kind, tokens=tokens, d_in=d_in, d_out=d_out, m_w=rng.choice([2, 4]))
    return dict(kind=kind, tokens=tokens, d_in=d_in, d_out=d_out, m_x=rng.choice([2, 4]), m_w=rng.choice([2, 4]))


# ---- inputs -------------------------------------------------------------


def _values(what, shape, gen):
    x = torch.empty(shape, dtype=torch.float32, device="cuda")
    if what == "half_normal":
        return x.normal_(generator=gen).abs_()
    if what == "weights":
        return x.normal_(0.0, 0.02, generator=gen)
    # gradients: Laplace(0, 1e-4), one entry in a hundred scaled by 100
    x.exponential_(1e4, generator=gen)
    u = torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-1.0, 1.0, generator=gen)
    x = torch.where(u.abs() < 0.01, 100.0 * x, x)
    return torch.where(u < 0, -x, x)


def _inputs(case, seed):
    """The case's FP32 inputs, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "quantize":
        shape = (case["outer"], case["length"], case["inner"])
        return dict(x=_values(case["values"], shape if case["inner"] > 1 else shape[:2], gen))
    T, I, O = case["tokens"], case["d_in"], case["d_out"]
    out = dict(x=_values("half_normal", (T, I), gen))
    if case["kind"] == "step":  # W as [in, out], as the update holds it
        out.update(w=_values("weights", (I, O), gen), dy=_values("grads", (T, O), gen))
    else:
        out["w"] = _values("weights", (O, I), gen)
    return out


def prepare(case, seed):
    v = _inputs(case, seed)
    s = dict(case=case, seed=seed, x=v["x"])
    kind = case["kind"]
    if kind == "step":
        T, I, O, m = case["tokens"], case["d_in"], case["d_out"], case["m"]
        e = fb.BFPTensor.empty
        dev = v["x"].device
        s.update(w=v["w"], dy=v["dy"], xa=e(T, I, 16, m, dev), xt=e(I, T, 16, m, dev), dya=e(T, O, 16, m, dev),
                 dyt=e(O, T, 16, m, dev), wk_new=e(I, O, 16, m, dev), wb_new=e(O, I, 16, m, dev),
                 y=torch.empty((T, O), device=dev), dx=torch.empty((T, I), device=dev),
                 dw=torch.empty((I, O), device=dev), w_new=torch.empty((I, O), device=dev))
        s["wk"], s["wb"] = fb.quantize_dual(v["w"], g=16, m=m)  # the last step's update left these
    elif kind == "packed":
        s["w"] = fb.quantize_packed(v["w"], m=case["m_w"])
    elif kind != "quantize":
        s["w"] = fb.quantize(v["w"], g=case.get("g", 16), m=case["m_w"])
    return s


# ---- one pass -----------------------------------------------------------


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "linear":
        a = fb.quantize(s["x"], g=case["g"], m=case["m_x"])
        return dict(y=fb.gemm(a, s["w"]))
    if kind == "converted":
        a = fb.quantize(s["x"], g=16, m=case["m_x"])
        t = fb.gemm_bfp(a, s["w"], case["m_y"], rounding=case["rounding"], seed=s["seed"])
        return dict(mant=t.mant, exp=t.exp)
    if kind == "step":
        m = case["m"]
        fb.quantize_dual(s["x"], m=m, out_rows=s["xa"], out_cols=s["xt"])
        fb.gemm(s["xa"], s["wb"], out=s["y"])
        fb.quantize_dual(s["dy"], m=m, rounding="stochastic", seed_rows=2 * s["seed"], seed_cols=2 * s["seed"] + 1,
                         out_rows=s["dya"], out_cols=s["dyt"])
        fb.gemm(s["dya"], s["wk"], out=s["dx"])
        fb.gemm(s["xt"], s["dyt"], out=s["dw"])
        fb.weight_update(s["w"], s["dw"], -LR, m=m, w_out=s["w_new"], out_rows=s["wk_new"], out_cols=s["wb_new"])
        return dict(y=s["y"], dx=s["dx"], dw=s["dw"], w=s["w_new"], wk_mant=s["wk_new"].mant, wk_exp=s["wk_new"].exp,
                    wb_mant=s["wb_new"].mant, wb_exp=s["wb_new"].exp)
    if kind == "quantize":
        axis = 1 if case["inner"] > 1 else -1
        t = fb.quantize(s["x"], group_axis=axis, g=case["g"], m=case["m"], rounding=case["rounding"], seed=s["seed"])
        return dict(mant=t.mant, exp=t.exp, values=fb.dequantize(t))
    if kind == "adaptive":
        t4, t2, sums = fb.quantize_adaptive(s["x"])
        m = fb.adaptive_mantissa(sums, fb.adaptive_threshold(ALPHA, BETA, 1, 2, 1, 2))
        return dict(mant4=t4.mant, mant2=t2.mant, exp=t4.exp, sums=sums, y=fb.gemm(t2 if m == 2 else t4, s["w"]))
    a = fb.quantize_packed(s["x"], m=case["m_x"])
    return dict(mant=a.mant, y=fb.gemm_packed(a, s["w"]))


# ---- what a pass cannot do without --------------------------------------


def _bits(m):
    """Stored bits per value without the exponent, by width."""
    return {2: 4, 4: 6, 6: 10, 8: 12}[m]


def _bfp(n, m, g=16):
    return n * (_bits(m) / 8.0 + 1.0 / g)


def work(case):
    kind = case["kind"]
    if kind == "quantize":
        n = case["outer"] * case["length"] * case["inner"]
        return dict(bytes=n * 8.0 + 2 * _bfp(n, case["m"], case["g"]), flops=0.0)
    T, I, O = case["tokens"], case["d_in"], case["d_out"]
    flops = 2.0 * T * I * O
    if kind == "linear":
        return dict(bytes=4.0 * T * I + _bfp(I * O, case["m_w"], case["g"]) + 4.0 * T * O, flops=flops)
    if kind == "converted":
        return dict(bytes=4.0 * T * I + _bfp(I * O, case["m_w"]) + _bfp(T * O, case["m_y"]), flops=flops)
    if kind == "step":
        # x, dy, w and both stored groupings of w in; y, dx, dw, the new w and its groupings out
        return dict(bytes=8.0 * T * (I + O) + 12.0 * I * O + 4 * _bfp(I * O, case["m"]), flops=3 * flops)
    if kind == "adaptive":
        return dict(bytes=4.0 * T * I + T * I * (0.75 + 0.5 + 1 / 16.0) + _bfp(I * O, case["m_w"]) + 4.0 * T * O,
                    flops=flops)
    packed = {2: 51 / 128.0, 4: 99 / 128.0}
    return dict(bytes=T * I * (4.0 + packed[case["m_x"]]) + I * O * packed[case["m_w"]] + 4.0 * T * O, flops=flops)


def tolerance(case):
    """FP32 sums over exact products in any order (and, of the updated weights'
    and of the converted output's codes, the few whose value sits within such a
    difference of a rounding boundary); conversions alone are exact."""
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] in ("converted", "step"):
        return {"rel": 2e-6, "max": 1e-4, "differ": 1e-4}
    return {"rel": 2e-6, "max": 1e-4}


# ---- the same in 64 bits ------------------------------------------------


def _noise(ngroups, g, seed):
    """Philox4x32-10 noise bytes [ngroups, g] of the stochastic rounding: key =
    the seed, counter = (group, group >> 32, t // 16, 0), byte t % 16 of the
    block."""
    mask = 0xFFFFFFFF
    gid = torch.arange(ngroups, dtype=torch.int64, device="cuda")

    def mulhilo(a, b):  # 32 x 32 -> (hi, lo); a: a constant, b: a tensor
        low = a * (b & 0xFFFF)
        mid = a * (b >> 16) + (low >> 16)
        return mid >> 16, ((mid & 0xFFFF) << 16) | (low & 0xFFFF)

    blocks = []
    for blk in range((g + 15) // 16):
        c = [gid & mask, gid >> 32, torch.full_like(gid, blk), torch.zeros_like(gid)]
        k0, k1 = seed & mask, (seed >> 32) & mask
        for _ in range(10):
            h0, l0 = mulhilo(0xD2511F53, c[0])
            h1, l1 = mulhilo(0xCD9E8D57, c[2])
            c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        blocks += [((w >> (8 * b)) & 0xFF).to(torch.uint8) for w in c for b in range(4)]
    return torch.stack(blocks[:g], dim=1)


def _bfp_values(x, m, g=16, rounding="nearest", seed=0, floor=None):
    """The values, in 64 bits, of x [rows, len] converted with groups of g along len."""
    rows, length = x.shape
    v = x.reshape(-1, g).double()
    e = torch.frexp(v.abs().amax(dim=1))[1] - 1  # exponent of the group's largest value
    e = torch.where(v.abs().amax(dim=1) == 0, torch.full_like(e, -127), e)
    if floor is not None:
        e = torch.clamp(e, min=floor)
    lsb = torch.ldexp(torch.ones_like(v[:, 0]), e - (m - 1))[:, None]
    a = v.abs() / lsb
    if rounding == "nearest":
        q = torch.floor(a + 0.5)
    else:
        q = torch.floor(torch.floor(a * 256.0) / 256.0 + _noise(v.shape[0], g, seed).double() / 256.0)
    q = torch.clamp(q, max=float(2 ** m - 1))
    return (torch.copysign(q, v) * lsb).reshape(rows, length)


def _matmul(a, b):
    """a . b^T in 64 bits, by rows so that it stays small in memory."""
    bt = b.t().contiguous()
    out = torch.empty((a.shape[0], bt.shape[1]), dtype=torch.float64, device=a.device)
    for r in range(0, a.shape[0], 65536):
        torch.mm(a[r:r + 65536], bt, out=out[r:r + 65536])
    return out


def exact(case, seed):
    kind = case["kind"]
    v = _inputs(case, seed)
    if kind == "quantize":
        x = v["x"] if case["inner"] == 1 else v["x"].transpose(1, 2).contiguous()
        x = x.reshape(-1, case["length"])
        return dict(mant=None, exp=None, values=_bfp_values(x, case["m"], case["g"], case["rounding"], seed))
    if kind == "converted":
        return None  # whole codes only
    if kind == "linear":
        return dict(y=_matmul(_bfp_values(v["x"], case["m_x"], case["g"]), _bfp_values(v["w"], case["m_w"], case["g"])))
    if kind == "step":
        m = case["m"]
        x, w, dy = v["x"], v["w"], v["dy"]
        wt, xt, dyt = w.t().contiguous(), x.t().contiguous(), dy.t().contiguous()
        y = _matmul(_bfp_values(x, m), _bfp_values(wt, m))
        dx = _matmul(_bfp_values(dy, m, 16, "stochastic", 2 * seed), _bfp_values(w, m))
        dw = _matmul(_bfp_values(xt, m), _bfp_values(dyt, m, 16, "stochastic", 2 * seed + 1))
        return dict(y=y, dx=dx, dw=dw, w=w.double() - LR * dw, wk_mant=None, wk_exp=None, wb_mant=None, wb_exp=None)
    if kind == "adaptive":
        x4 = _bfp_values(v["x"], 4)
        e = torch.frexp(v["x"].reshape(-1, 16).abs().amax(dim=1).double())[1] - 1
        lsb = torch.ldexp(torch.ones(e.shape, dtype=torch.float64, device=e.device), e - 3)[:, None]
        q = x4.reshape(-1, 16) / lsb
        x2 = (torch.copysign(torch.floor(q.abs() / 4.0), q) * 4.0 * lsb).reshape(x4.shape)
        num, den = (x4 - x2).abs().sum(), x2.abs().sum()
        x = x2 if float(num / den) < ALPHA - BETA * 0.5 - BETA * 0.5 else x4
        return dict(mant4=None, mant2=None, exp=None, sums=torch.stack([num, den]),
                    y=_matmul(x, _bfp_values(v["w"], case["m_w"])))

    def packed(x, m):  # the shared exponents are at least the tensor's largest minus 7
        top = int(torch.frexp(x.abs().amax().double())[1]) - 1
        return _bfp_values(x, m, floor=top - 7)

    return dict(mant=None, y=_matmul(packed(v["x"], case["m_x"]), packed(v["w"], case["m_w"])))
