"""The work that a user of this framework has it do, as cases to be timed.

Four kinds of call, each through the binding's public entry points with the
buffers a training program allocates once:

* ``linear``   backward of a linear layer: ``BackwardPlan.run`` (quantize dY,
               dX = dY W, dW = dY^T X).  With ``operands`` the step also
               quantizes that step's W and X per tensor (``sq_quantize_tensor``),
               as a program does that keeps no codes from the forward pass.
* ``conv``     one training step's integer work of a stride-1, same-size 3x3
               convolution: the layer input's quantizer onto the padded grid
               (``ConvBackwardPlan.quantize_input``), then the backward step
               (``ConvBackwardPlan.run``).
* ``l1bn``     one training step of a fully quantized L1 batch norm: quantize
               X, forward, backward.
* ``forward``  forward of a linear layer: per-output-channel W codes, X in
               ShiftQuant groups, Y = X W^T.

Every result is a whole number or one correctly rounded product of a whole
number and a scale with a fixed order of operations (include/shiftquant.h),
so any correct implementation gives the same bits: the tolerance is "exact".
"""
import math

import torch

from paper_2411_10948_amd import shiftquant as sq

DEVICE = "cuda"

# How the gradients are distributed (the recipes of the workloads module): a
# draw z scaled per channel by a log-normal sigma, some channels larger still.
RECIPES = {
    "resnet": {"z": "normal", "sigma": 1.0, "outliers": 0.02, "factor": 100.0},
    "mlp": {"z": "student_t3", "sigma": 1.5, "outliers": 0.0, "factor": 1.0},
    "large": {"z": "normal", "sigma": 2.0, "outliers": 0.005, "factor": 1000.0},
}


def listed():
    return [
        # the smallest layer a program trains: launches and latency are all of it
        {"name": "linear_256", "kind": "linear", "M": 256, "C_out": 256, "C_in": 256, "bits": 4, "groups": 4,
         "rounding": "nearest", "tiled": False, "operands": False, "recipe": "resnet"},
        # a 1000-way classifier on 2048 features, one batch of 256 images: sizes that no tile divides
        {"name": "classifier_2048x1000", "kind": "linear", "M": 256, "C_out": 1000, "C_in": 2048, "bits": 8,
         "groups": 4, "rounding": "nearest", "tiled": False, "operands": True, "recipe": "resnet"},
        # an attention projection over 16 sequences of 197 tokens: an odd row count, the default row-major codes
        {"name": "projection_197_tokens", "kind": "linear", "M": 16 * 197, "C_out": 768, "C_in": 768, "bits": 6,
         "groups": 4, "rounding": "nearest", "tiled": False, "operands": True, "recipe": "mlp"},
        # ResNet-50's 1x1 bottleneck convolution 1024 -> 256 at 14x14, batch 64: few channels, many rows
        {"name": "resnet50_conv1x1", "kind": "linear", "M": 64 * 14 * 14, "C_out": 256, "C_in": 1024, "bits": 4,
         "groups": 4, "rounding": "nearest", "tiled": True, "operands": False, "recipe": "resnet"},
        # a Transformer MLP's up-projection, 32 x 512 tokens, 6-bit gradients: the ordinary large layer
        {"name": "mlp_up_768x3072", "kind": "linear", "M": 32 * 512, "C_out": 3072, "C_in": 768, "bits": 6,
         "groups": 4, "rounding": "nearest", "tiled": True, "operands": False, "recipe": "mlp"},
        # the largest layer, stochastic rounding: the benchmark's own workload
        {"name": "linear_4096x11008_sr", "kind": "linear", "M": 8192, "C_out": 11008, "C_in": 4096, "bits": 6,
         "groups": 4, "rounding": "stochastic", "tiled": True, "operands": False, "recipe": "large"},
        # ResNet-18's four-bit 3x3 convolutions at batch 64: the first stage (many pixels, few channels) ...
        {"name": "conv3x3_56x56x64", "kind": "conv", "N": 64, "HW": 56, "C_out": 64, "C_in": 64, "bits": 4,
         "groups": 4, "rounding": "nearest", "recipe": "resnet"},
        # ... the second, with 6-bit stochastic gradients ...
        {"name": "conv3x3_28x28x128_sr", "kind": "conv", "N": 64, "HW": 28, "C_out": 128, "C_in": 128, "bits": 6,
         "groups": 4, "rounding": "stochastic", "recipe": "resnet"},
        # ... and the third: rows of 14 pixels, which no vector width divides
        {"name": "conv3x3_14x14x256", "kind": "conv", "N": 64, "HW": 14, "C_out": 256, "C_in": 256, "bits": 4,
         "groups": 4, "rounding": "nearest", "recipe": "resnet"},
        # ResNet-18's first-stage batch norm: the longest columns
        {"name": "l1bn_56x56x64", "kind": "l1bn", "M": 64 * 56 * 56, "C": 64, "bits": 8, "groups": 4,
         "rounding": "nearest", "recipe": "resnet"},
        # its third-stage batch norm: fewer rows than the reductions have room for
        {"name": "l1bn_14x14x256", "kind": "l1bn", "M": 64 * 14 * 14, "C": 256, "bits": 8, "groups": 4,
         "rounding": "nearest", "recipe": "resnet"},
        # the MLP up-projection's forward pass with that step's weights
        {"name": "forward_mlp_768x3072", "kind": "forward", "M": 32 * 512, "C_out": 3072, "C_in": 768, "bits": 6,
         "groups": 4, "recipe": "mlp"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A channel or row count: any whole number, or rounded to 64 as layers mostly are."""
    n = _log_int(rng, lo, hi)
    return n if rng.random() < 0.4 else max(64, (n + 32) // 64 * 64)


def draw(rng):
    kind = rng.choice(["linear", "linear", "conv", "conv", "l1bn", "forward"])
    bits = rng.choice([4, 6, 8])
    rounding = rng.choice(["nearest", "nearest", "stochastic"])
    recipe = rng.choice(sorted(RECIPES))
    common = {"kind": kind, "bits": bits, "groups": 4, "recipe": recipe}
    if kind in ("linear", "forward"):
        while True:
            M, C_out, C_in = _size(rng, 64, 16384), _size(rng, 64, 11008), _size(rng, 64, 4096)
            if M * C_out * C_in <= 8192 * 11008 * 4096 // 4 and M * C_out <= 16384 * 3072:
                break
        c = dict(common, M=M, C_out=C_out, C_in=C_in)
        if kind == "linear":
            c.update(rounding=rounding, tiled=rng.random() < 0.5, operands=rng.random() < 0.5)
        return c
    if kind == "conv":
        while True:
            c = dict(common, N=_log_int(rng, 1, 64), HW=_log_int(rng, 7, 56), C_out=_log_int(rng, 16, 512),
                     C_in=_log_int(rng, 16, 512), rounding=rounding)
            if rng.random() < 0.7:
                c["C_out"], c["C_in"] = ((c[k] + 15) // 16 * 16 for k in ("C_out", "C_in"))
            px = c["N"] * c["HW"] ** 2
            if px * max(c["C_out"], c["C_in"]) <= 64 * 56 * 56 * 64 and px * c["C_out"] * c["C_in"] <= 2 ** 30:
                return c
    while True:
        c = dict(common, M=_size(rng, 512, 64 * 56 * 56), C=_log_int(rng, 16, 256), rounding=rounding)
        if c["M"] * c["C"] <= 64 * 56 * 56 * 64:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEVICE)


def _grad(g, M, C, recipe):
    r = RECIPES[recipe]
    sigma = torch.exp(r["sigma"] * _randn(g, C))
    k = max(1, round(r["outliers"] * C)) if r["outliers"] else 0
    sigma[torch.randperm(C, generator=g, device=DEVICE)[:k]] *= r["factor"]
    z = _randn(g, M, C)
    if r["z"] == "student_t3":
        chi = _randn(g, M, C).square_()
        for _ in range(2):
            chi += _randn(g, M, C).square_()
        z /= (chi / 3.0).sqrt_().clamp_(min=1e-6)
    return z.mul_(sigma)


def _inputs(case, seed):
    """The fp32 tensors of a case, from the seed alone."""
    g = _generator(seed)
    kind = case["kind"]
    if kind == "linear":
        M, Co, Ci = case["M"], case["C_out"], case["C_in"]
        return {"dY": _grad(g, M, Co, case["recipe"]), "W": _randn(g, Co, Ci).mul_(0.02), "X": _randn(g, M, Ci)}
    if kind == "conv":
        M, Co, Ci = case["N"] * case["HW"] ** 2, case["C_out"], case["C_in"]
        return {"dY": _grad(g, M, Co, case["recipe"]), "W": _randn(g, Co, 9 * Ci).mul_(math.sqrt(2.0 / (9 * Ci))),
                "X": _randn(g, M, Ci).clamp_(min=0.0)}
    if kind == "l1bn":
        M, C = case["M"], case["C"]
        X = _randn(g, M, C).mul_(torch.exp(0.5 * _randn(g, C))).add_(0.5 * _randn(g, C))
        return {"X": X, "gamma": 1.0 + 0.2 * _randn(g, C), "beta": 0.2 * _randn(g, C),
                "dy": _grad(g, M, C, case["recipe"])}
    M, Co, Ci = case["M"], case["C_out"], case["C_in"]
    return {"X": _grad(g, M, Ci, case["recipe"]), "W": _randn(g, Co, Ci).mul_(0.02)}


def _params(case):
    mode = sq.ROUND_STOCHASTIC if case.get("rounding") == "stochastic" else sq.ROUND_NEAREST_EVEN
    return sq.Params.make(case["bits"], case["groups"], mode, 0, 0,
                          sq.LAYOUT_TILED if case.get("tiled") else sq.LAYOUT_ROWS)


def _bytes(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device=DEVICE)


def prepare(case, seed):
    st = {"case": case, "in": _inputs(case, seed), "params": _params(case)}
    p, t, kind = st["params"], st["in"], case["kind"]
    if kind == "linear":
        M, Co, Ci = case["M"], case["C_out"], case["C_in"]
        st["plan"] = sq.BackwardPlan(M, Co, Ci, p, device=DEVICE)
        st["wq_t"], st["xq_t"] = sq.code_matrix(Ci, Co, p.tiled, DEVICE), sq.code_matrix(Ci, M, p.tiled, DEVICE)
        st["ws"], st["xs"] = sq.new_scale(DEVICE), sq.new_scale(DEVICE)
        st["ws_w"] = _bytes(sq.sq_quantize_tensor_workspace_size(Co, Ci))
        st["ws_x"] = _bytes(sq.sq_quantize_tensor_workspace_size(M, Ci))
        if not case["operands"]:
            _linear_operands(st)   # the codes the forward pass left
    elif kind == "conv":
        N, HW, Co, Ci = case["N"], case["HW"], case["C_out"], case["C_in"]
        st["plan"] = sq.ConvBackwardPlan(N, HW, HW, Co, Ci, 3, 3, 1, 1, p, device=DEVICE)
        st["wq_t"], st["ws"] = sq.quantize_tensor(t["W"], 8)
    elif kind == "l1bn":
        M, C = case["M"], case["C"]
        st["xq"], st["xs"] = sq.code_matrix(M, C, False, DEVICE)[:, :C], sq.new_scale(DEVICE)
        for k, n in (("chan", C * sq.L1BN_CHANNEL_WORDS), ("layer", 16)):
            st[k] = torch.zeros(n, dtype=torch.int32, device=DEVICE)
        st["y"], st["dx"] = torch.empty_like(t["X"]), torch.empty_like(t["X"])
        st["dgamma"], st["dbeta"] = torch.empty_like(t["gamma"]), torch.empty_like(t["beta"])
        st["group"] = torch.empty(C, dtype=torch.uint8, device=DEVICE)
        st["gscale"] = sq.new_scale(DEVICE)
        st["ws_x"] = _bytes(sq.sq_quantize_tensor_workspace_size(M, C))
        st["ws_f"] = _bytes(sq.sq_l1bn_forward_workspace_size(M, C))
        st["ws_b"] = _bytes(sq.sq_l1bn_backward_workspace_size(M, C, p))
    else:
        M, Co, Ci = case["M"], case["C_out"], case["C_in"]
        lay_bytes, min_ld = sq.sq_grad_layout_size(Ci, p)
        st["xq"] = sq.code_matrix(M, min_ld, False, DEVICE)
        st["group"] = torch.empty(Ci, dtype=torch.uint8, device=DEVICE)
        st["xscale"] = sq.new_scale(DEVICE)
        st["layout"] = torch.zeros(lay_bytes // 4, dtype=torch.int32, device=DEVICE)
        st["wq"] = sq.code_matrix(Co, Ci, False, DEVICE)
        st["wscales"] = torch.zeros((Co, 4), dtype=torch.float32, device=DEVICE)
        st["Y"] = torch.empty((M, Co), dtype=torch.float32, device=DEVICE)
        st["ws_q"] = _bytes(sq.sq_quantize_grad_workspace_size(M, Ci, p))
        st["ws_c"] = _bytes(sq.sq_quantize_channels_workspace_size(Co, Ci, 0))
        st["ws_f"] = _bytes(sq.sq_gemm_dgrad_workspace_size(M, Ci, Co, p))
    return st


def _linear_operands(st):
    tr = 2 if st["params"].tiled else 1
    sq.sq_quantize_tensor(st["in"]["W"], 8, tr, st["wq_t"], st["ws"], st["ws_w"])
    sq.sq_quantize_tensor(st["in"]["X"], 8, tr, st["xq_t"], st["xs"], st["ws_x"])


def run(st):
    kind, t, p = st["case"]["kind"], st["in"], st["params"]
    if kind == "linear":
        if st["case"]["operands"]:
            _linear_operands(st)
        plan = st["plan"]
        dX, dW = plan.run(t["dY"], st["wq_t"], st["ws"], st["xq_t"], st["xs"])
        return dX, dW, plan.group, plan.scale
    if kind == "conv":
        plan = st["plan"]
        plan.quantize_input(t["X"])
        dX, dW = plan.run(t["dY"], st["wq_t"], st["ws"], plan.x_grid, plan.x_scale)
        return dX, dW, plan.group, plan.scale
    if kind == "l1bn":
        sq.sq_quantize_tensor(t["X"], 8, 0, st["xq"], st["xs"], st["ws_x"])
        sq.sq_l1bn_forward(st["xq"], st["xs"], t["gamma"], t["beta"], st["y"], st["chan"], st["layer"], st["ws_f"])
        sq.sq_l1bn_backward(t["dy"], p, st["xq"], st["chan"], st["layer"], st["dx"], st["dgamma"], st["dbeta"],
                            st["group"], st["gscale"], None, st["ws_b"])
        return st["y"], st["dx"], st["dgamma"], st["dbeta"], st["group"]
    M, Ci, Co = st["case"]["M"], st["case"]["C_in"], st["case"]["C_out"]
    sq.sq_quantize_channels(t["W"], 8, 0, False, st["wq"], st["wscales"], st["ws_c"])
    sq.sq_quantize_grad(t["X"], p, st["xq"], None, st["group"], st["xscale"], st["layout"], st["ws_q"])
    sq.sq_gemm_forward(st["xq"], st["layout"], st["group"], st["xscale"], st["wq"], st["wscales"], M, Ci, Co, p,
                       None, st["Y"], st["ws_f"])
    return st["Y"], st["group"], st["xscale"]


def work(case):
    kind = case["kind"]
    if kind in ("linear", "forward"):
        M, Co, Ci = case["M"], case["C_out"], case["C_in"]
        if kind == "forward":
            return {"bytes": 4 * (M * Ci + Co * Ci + M * Co), "flops": 2 * M * Co * Ci}
        b = 4 if case["operands"] else 1   # X and W in fp32, or their codes
        return {"bytes": 4 * M * Co + b * (M + Co) * Ci + 4 * (M + Co) * Ci, "flops": 4 * M * Co * Ci}
    if kind == "conv":
        px, Co, Ci = case["N"] * case["HW"] ** 2, case["C_out"], case["C_in"]
        return {"bytes": 4 * px * (Co + Ci) + 9 * Co * Ci + 4 * px * Ci + 36 * Co * Ci, "flops": 4 * px * 9 * Co * Ci}
    return {"bytes": 16 * case["M"] * case["C"], "flops": 20 * case["M"] * case["C"]}


def tolerance(case):
    return "exact"


# ---------------------------------------------------------------------------
# the same results in plain torch: codes as include/shiftquant.h defines them
# (fp32 products), everything after them in 64 bits
# ---------------------------------------------------------------------------
def _philox16(n, device):
    """The first n 16-bit uniforms of the Philox4x32-10 stream with key 0 and offset 0."""
    mask = 0xFFFFFFFF
    x = torch.arange((n + 7) // 8, dtype=torch.int64, device=device)
    c = [x & mask, x >> 32, torch.zeros_like(x), torch.zeros_like(x)]
    k0 = k1 = 0

    def mul(a, m):
        lo, hi = a * (m & 0xFFFF), a * (m >> 16)
        return (hi + (lo >> 16)) >> 16, ((hi << 16) + lo) & mask

    for _ in range(10):
        h0, l0 = mul(c[0], 0xD2511F53)
        h1, l1 = mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return torch.stack([h for w in c for h in (w & 0xFFFF, w >> 16)], 1).reshape(-1)[:n]


def _shift_codes(x, case):
    """(codes fp64, groups, scale) of ShiftQuant over the columns of x."""
    Q, ng = 2 ** (case["bits"] - 1) - 1, case["groups"]
    r = x.abs().amax(0)
    r_max = r.max()
    g = torch.zeros_like(r, dtype=torch.int64)
    for j in range(1, ng):
        g += (r * float(2 ** j) <= r_max).to(torch.int64)
    q32 = torch.full_like(r_max, Q)
    inv, step = q32 / r_max, r_max / q32
    v = x * (inv * torch.exp2(g.to(torch.float32)))
    if case.get("rounding") == "stochastic":
        low = v.floor()
        u = _philox16(v.numel(), x.device).reshape(v.shape).to(torch.float32)
        v = torch.where(u < (v - low) * 65536.0, low + 1.0, low)
    else:
        v = v.round()
    scale = torch.stack([r_max, inv, step, torch.zeros_like(inv)]).double()
    return v.clamp_(-Q, Q).double(), g, scale


def _tensor_codes(x, dim=None):
    """8-bit codes (fp64) and steps of x, one scale per tensor or per slice along dim."""
    a = x.abs().amax() if dim is None else x.abs().amax(dim, keepdim=True)
    q = torch.full_like(a, 127.0)
    return (x * (q / a)).round_().clamp_(-127, 127).double(), (a / q).double()


def exact(case, seed):
    t, kind = _inputs(case, seed), case["kind"]
    if kind == "l1bn":
        return _exact_l1bn(case, t)
    wq, ws = _tensor_codes(t["W"], 1 if kind == "forward" else None)
    q, g, scale = _shift_codes(t["X"] if kind == "forward" else t["dY"], case)
    lv = q * torch.exp2(-g.double())        # codes in units of the largest step
    if kind == "forward":
        return (lv @ wq.t()) * (scale[2] * ws.reshape(1, -1)), g, scale
    xq, xs = _tensor_codes(t["X"])
    if kind == "linear":
        return (lv @ wq) * (scale[2] * ws), (lv.t() @ xq) * (scale[2] * xs), g, scale
    N, HW, Co, Ci = case["N"], case["HW"], case["C_out"], case["C_in"]
    pad = torch.zeros((N, HW + 2, HW + 2, Ci), dtype=torch.float64, device=q.device)
    pad[:, 1:-1, 1:-1] = xq.reshape(N, HW, HW, Ci)
    dXp = torch.zeros_like(pad)
    dW = torch.empty((Co, 9, Ci), dtype=torch.float64, device=q.device)
    for r in range(3):
        for s in range(3):
            tap = wq[:, (3 * r + s) * Ci:(3 * r + s + 1) * Ci]
            dXp[:, r:r + HW, s:s + HW] += (lv @ tap).reshape(N, HW, HW, Ci)
            dW[:, 3 * r + s] = lv.t() @ pad[:, r:r + HW, s:s + HW].reshape(-1, Ci)
    return (dXp[:, 1:-1, 1:-1].reshape(-1, Ci) * (scale[2] * ws), dW.reshape(Co, -1) * (scale[2] * xs), g, scale)


def _round_div(a, b):
    """round half to even of a / b for whole a and b > 0, both int64."""
    f = torch.div(a, b, rounding_mode="floor")
    r = 2 * (a - f * b)
    return f + ((r > b) | ((r == b) & (f % 2 == 1))).to(f.dtype)


def _exact_l1bn(case, t):
    M = case["M"]
    q, sx = _tensor_codes(t["X"])
    mu = _round_div(q.sum(0).to(torch.int64), torch.tensor(M, device=q.device)).double()
    d = q - mu
    A = d.abs().sum(0)
    k = _round_div((127 * A).to(torch.int64), A.max().to(torch.int64)).clamp_(min=1).double()
    gamma, beta = (c * s for c, s in (_tensor_codes(t["gamma"]), _tensor_codes(t["beta"])))
    rho = 127.0 * M / (A.max() * k)
    y = d * (gamma * rho) + beta
    qg, g, scale = _shift_codes(t["dy"], case)
    delta = scale[2] * torch.exp2(-g.double())
    sgn = d.sign()
    dbeta = delta * qg.sum(0)
    dgamma = delta * (qg * d).sum(0) * rho
    lam = gamma * rho / sx
    dx = lam * (delta * qg - dbeta / M - dgamma / M * (sgn - sgn.sum(0) / M))
    return y, dx, dgamma, dbeta, g
