"""The framework's performance cases: what a program that uses it has it compute, one call
through a public entry point per case, over the sizes, storage types and options in use.

Entries ("entry" of a case):
  forward   paper_2208_05419_amd.filter_forward: out = x + filter(x).  "hs" (hidden units per
            block) may differ from the block size C / nb.
  backward  paper_2208_05419_amd.filter_backward: dx and the four parameter gradients.
  block     paper_2208_05419_amd.block_forward: one AFNO transformer block around the filter.
"""
import math

import torch

import paper_2208_05419_amd as afno

DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}


def _case(name, entry, B, H, W, C, nb, dtype, hs=0, keep=1.0, lam=0.01):
    return {"name": name, "entry": entry, "B": B, "H": H, "W": W, "C": C, "nb": nb, "hs": hs or C // nb,
            "dtype": dtype, "keep": keep, "lam": lam}


def listed():
    return [
        # a small grid: one forecast step of a toy or a regional model, where a call's launches count
        _case("forward_16x32_fp32", "forward", 1, 16, 32, 64, 4, "fp32"),
        # 0.25-degree fields in 8 x 8 patches, one sample at full precision: validation of a checkpoint
        _case("forward_90x180_fp32", "forward", 1, 90, 180, 768, 8, "fp32"),
        # the same grid in bf16, a batch of four: the throughput workload (serving, training forward)
        _case("forward_90x180_bf16", "forward", 4, 90, 180, 768, 8, "bf16"),
        # the same fields in 4 x 4 patches, eight wide blocks
        _case("forward_180x360_bf16_8_blocks", "forward", 1, 180, 360, 1024, 8, "bf16"),
        # the filter in the form of the paper: 32 narrow blocks on the 180 x 360 grid
        _case("forward_180x360_bf16_32_blocks", "forward", 1, 180, 360, 1024, 32, "bf16"),
        # part of an ensemble forecast with a hard cutoff: the lower half of the modes per axis
        _case("forward_ensemble_90x180_bf16", "forward", 32, 90, 180, 768, 8, "bf16", keep=0.5),
        # a block MLP twice as wide as its block
        _case("forward_hidden192_90x180_bf16", "forward", 4, 90, 180, 768, 8, "bf16", hs=192),
        # a regular grid of another size (1.4 degrees), two samples
        _case("forward_128x256_bf16", "forward", 2, 128, 256, 512, 8, "bf16"),
        # training: the gradient of the throughput workload
        _case("backward_90x180_bf16", "backward", 4, 90, 180, 768, 8, "bf16"),
        # training on the paper's grid and blocks
        _case("backward_180x360_bf16_32_blocks", "backward", 1, 180, 360, 1024, 32, "bf16"),
        # training at full precision on a 2.5-degree grid with blocks of 48
        _case("backward_72x144_fp32", "backward", 1, 72, 144, 384, 8, "fp32"),
        # a whole transformer block of the throughput workload
        _case("block_90x180_bf16", "block", 4, 90, 180, 768, 8, "bf16"),
    ]


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


_HEIGHTS = [n for n in range(12, 193) if _smooth(n)]
_WIDTHS = [n for n in range(12, 577, 2) if _smooth(n)]


def _log_choice(rng, values, low, high):
    """The one of the values nearest to a size drawn evenly over its logarithm."""
    t = math.exp(rng.uniform(math.log(low), math.log(high)))
    return min(values, key=lambda v: abs(math.log(v / t)))


def _fits(c):
    """Whether the entry point takes the case: a column of H x block (and H x hidden, and the
    backward's masks) with its transform buffer in the 160 KiB of one compute unit."""
    bs, hs, es = c["C"] // c["nb"], c["hs"], 4 if c["dtype"] == "fp32" else 2
    h16, pad = (c["H"] + 15) // 16 * 16, 4 if es == 4 else 8
    lds = h16 * (2 * bs + pad) * es + c["H"] * 8 * (33 if bs % 32 == 0 else 17) + 64
    if hs != bs:
        lds += h16 * (2 * hs + pad) * es
    if c["entry"] == "backward":
        lds += 2 * h16 * (bs // 16) * 4 + 64
    return lds <= 160 * 1024


def draw(rng):
    """A case of the ranges above: the entry points by their use, grids of 12 to 192 rows that are
    one to three times as wide (a global grid's two, and regional ones), blocks of 16 to 128
    channels, both storage types, cutoffs and hidden sizes."""
    while True:
        entry = rng.choices(["forward", "backward", "block"], [6, 3, 1])[0]
        dtype = "bf16" if entry == "block" or rng.random() < 0.65 else "fp32"
        bs = rng.choice([16, 32, 48, 64, 96, 128])
        nb = rng.choice([1, 2, 4, 6, 8, 12, 16, 32])
        C = bs * nb
        hs = bs
        if entry == "forward" and rng.random() < 0.25:
            hs = rng.choice([h for h in (bs // 2, 2 * bs, 4 * bs) if h % 16 == 0 and h <= 256])
        keep = 1.0 if rng.random() < 0.6 else round(rng.uniform(0.3, 0.95), 2)
        H = _log_choice(rng, _HEIGHTS, 12, 192)
        W = 2 * H if rng.random() < 0.5 else _log_choice(rng, _WIDTHS, H, 3 * H)
        if C > 1024 or (entry == "block" and C % 128):
            continue
        # elements of the token grid, from 2^15 up, and no dearer than the largest case listed
        top = {"forward": 48e6, "backward": 16e6, "block": 24e6}[entry] / (2.0 if dtype == "fp32" else 1.0)
        B = round(math.exp(rng.uniform(math.log(2.0 ** 15), math.log(top))) / (H * W * C))
        if not 1 <= B <= 32:
            continue
        case = _case("", entry, B, H, W, C, nb, dtype, hs=hs, keep=keep)
        del case["name"]
        if _fits(case):
            return case


def _kept(c):
    """Kept rows (|signed kh| < kept_h) and columns of the half spectrum."""
    H, W, f = c["H"], c["W"], c["keep"]
    kh, kw = math.floor((H // 2 + 1) * f), math.floor((W // 2 + 1) * f)
    rows = [k for k in range(H) if abs(k if k <= H // 2 else k - H) < kh]
    return rows, kw


def prepare(case, seed):
    c, dt = case, DTYPES[case["dtype"]]
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(1000003 * int(seed) + 17)
    B, H, W, C, nb, hs = (c[k] for k in ("B", "H", "W", "C", "nb", "hs"))
    bs = C // nb

    def normal(*shape, std=1.0, mean=0.0):
        return (mean + std * torch.randn(*shape, generator=g, device=dev)).to(dt)

    def signed(*shape):  # +-(1 to 1.5)
        r = torch.rand(*shape, generator=g, device=dev) - 0.5
        return ((1.0 + r.abs()) * torch.sign(r)).to(dt)

    s = {"case": dict(c)}
    # fields of zero mean whose channels (variables) differ in scale
    scale = 0.5 + 1.5 * torch.rand(C, generator=g, device=dev)
    x = torch.empty(B, H, W, C, dtype=dt, device=dev)
    for b in range(B):
        x[b] = (torch.randn(H, W, C, generator=g, device=dev) * scale).to(dt)
    s["x"] = x
    if c["entry"] == "backward":
        # weights at their initial scale, biases well away from the kinks of ReLU and softshrink: of a
        # mode within rounding of a kink either gradient is right, and a comparison would measure that choice
        w = {"w1": normal(nb, bs, hs, 2, std=0.02), "b1": signed(nb, hs, 2), "w2": normal(nb, hs, bs, 2, std=0.02),
             "b2": signed(nb, bs, 2)}
        s["g"] = torch.empty_like(x)
        for b in range(B):
            s["g"][b] = torch.randn(H, W, C, generator=g, device=dev).to(dt)
    else:
        # weights whose response is of the order of the tokens, as after training
        w = {"w1": normal(nb, bs, hs, 2, std=1.0 / math.sqrt(bs)), "b1": normal(nb, hs, 2, std=0.02),
             "w2": normal(nb, hs, bs, 2, std=1.0 / math.sqrt(hs)), "b2": normal(nb, bs, 2, std=0.02)}
    if c["entry"] == "block":
        w.update({"ln1_g": normal(C, std=0.1, mean=1.0), "ln1_b": normal(C, std=0.1), "ln2_g": normal(C, std=0.1, mean=1.0),
                  "ln2_b": normal(C, std=0.1), "wa": normal(C, 4 * C, std=1.0 / math.sqrt(C)), "ba": normal(4 * C, std=0.02),
                  "wb": normal(4 * C, C, std=0.5 / math.sqrt(C)), "bb": normal(C, std=0.02)})
    s["w"] = w
    return s


def run(state):
    c, w, x = state["case"], state["w"], state["x"]
    if c["entry"] == "forward":
        return afno.filter_forward(x, w["w1"], w["b1"], w["w2"], w["b2"], c["nb"], c["lam"], c["keep"])
    if c["entry"] == "backward":
        return afno.filter_backward(x, w["w1"], w["b1"], w["w2"], w["b2"], state["g"], c["nb"], c["lam"], c["keep"])
    return afno.block_forward(x, w, c["nb"], c["lam"], c["keep"])


def work(case):
    c = case
    B, H, W, C, nb, hs = (c[k] for k in ("B", "H", "W", "C", "nb", "hs"))
    bs, es, n = C // nb, 4 if c["dtype"] == "fp32" else 2, B * H * W * C
    rows, kw = _kept(c)
    modes = B * len(rows) * kw
    weights = nb * (4 * bs * hs + 2 * hs + 2 * bs)
    fft = 2.5 * n * math.log2(H * W)  # one real transform of the grid
    mlp = 16.0 * bs * hs * nb * modes  # both complex layers
    if c["entry"] == "forward":
        return {"bytes": (2 * n + weights) * es, "flops": 2 * fft + mlp}
    if c["entry"] == "backward":
        return {"bytes": (3 * n + weights) * es + 4 * weights, "flops": 3 * fft + 3 * mlp}
    return {"bytes": (2 * n + weights + 8 * C * C + 9 * C) * es, "flops": 2 * fft + mlp + 16.0 * n * C}


def tolerance(case):
    """About four times the largest error against exact() measured over the listed and 20 drawn
    cases: fp32 3.0e-7 forward and 9.6e-7 in the weight gradients' sums over the modes; bf16
    4.4e-3 (the spectrum, the hidden layer and the result rounded to 2^-9)."""
    return {"rel": 4e-6 if case["dtype"] == "fp32" else 1.8e-2}


def exact(case, seed):
    """The same outputs from dense transforms and products in float64 (complex128)."""
    c, s = case, prepare(case, seed)
    w = {k: v.double() for k, v in s["w"].items()}
    W, C = c["W"], c["C"]
    if c["entry"] == "backward":
        dx, sums = torch.empty(s["x"].shape, dtype=torch.float64, device=s["x"].device), None
        for b in range(c["B"]):
            dx[b], *grads = _exact_backward(c, w, s["x"][b].double(), s["g"][b].double())
            sums = grads if sums is None else [p + q for p, q in zip(sums, grads)]
        return {"dx": dx, **dict(zip(("dw1", "db1", "dw2", "db2"), sums))}
    out = torch.empty(s["x"].shape, dtype=torch.float64, device=s["x"].device)
    for b in range(c["B"]):
        x = s["x"][b].double()
        if c["entry"] == "forward":
            out[b] = x + _exact_filter(c, w, x)
            continue
        norm = lambda z, n: torch.nn.functional.layer_norm(z, (C,), w[n + "_g"], w[n + "_b"], 1e-6)  # noqa: E731
        t = norm(x, "ln1")
        v = x + t + _exact_filter(c, w, t)
        h = torch.nn.functional.gelu(norm(v, "ln2").reshape(-1, C) @ w["wa"] + w["ba"])
        out[b] = v + (h @ w["wb"] + w["bb"]).reshape(v.shape)
    return out


def _dft(n, rows, cols, device):
    """exp(-2 pi i r c / n) / sqrt(n), the angle reduced in whole numbers."""
    m = (torch.as_tensor(rows, device=device)[:, None] * torch.as_tensor(cols, device=device)[None]) % n
    a = m.double() * (-2.0 * math.pi / n)
    return torch.complex(torch.cos(a), torch.sin(a)) / math.sqrt(n)


def _spectrum(c, x):
    """Kept modes [rows, kw, C] of a real grid [H, W, C]."""
    rows, kw = _kept(c)
    H, W, C = x.shape
    fw, fh = _dft(W, range(kw), range(W), x.device), _dft(H, rows, range(H), x.device)
    s = torch.complex(torch.matmul(fw.real, x), torch.matmul(fw.imag, x))  # [H, kw, C]
    return (fh @ s.reshape(H, kw * C)).reshape(len(rows), kw, C)


def _column_weights(c, kw, device):
    return torch.tensor([1.0 if k == 0 or 2 * k == c["W"] else 2.0 for k in range(kw)], dtype=torch.float64, device=device)


def _grid(c, Y, weights):
    """The real grid [H, W, C] of kept modes [rows, kw, C] with the columns' weights."""
    rows, kw = _kept(c)
    H, W, C = c["H"], c["W"], c["C"]
    ih = _dft(H, range(H), rows, Y.device).conj()
    s = (ih @ Y.reshape(len(rows), kw * C)).reshape(H, kw, C)
    iw = _dft(W, range(W), range(kw), Y.device).conj() * weights
    return torch.matmul(iw.real.contiguous(), s.real.contiguous()) - torch.matmul(iw.imag.contiguous(), s.imag.contiguous())


def _layers(c, w, X):
    """Per block [nb, modes, .]: X, v = X w1 + b1, h = relu(v), o = h w2 + b2, and the complex weights."""
    nb, bs = c["nb"], c["C"] // c["nb"]
    cw = {k: torch.view_as_complex(w[k].contiguous()) for k in ("w1", "b1", "w2", "b2")}
    Xb = X.reshape(-1, nb, bs).transpose(0, 1).contiguous()
    v = torch.stack([Xb[k] @ cw["w1"][k] + cw["b1"][k] for k in range(nb)])
    h = torch.complex(torch.relu(v.real), torch.relu(v.imag))
    o = torch.stack([h[k] @ cw["w2"][k] + cw["b2"][k] for k in range(nb)])
    return Xb, v, h, o, cw


def _joined(t, like):
    return t.transpose(0, 1).reshape(like.shape)


def _exact_filter(c, w, x):
    X = _spectrum(c, x)
    o = _layers(c, w, X)[3]
    shrink = lambda t: torch.sign(t) * torch.relu(t.abs() - float(torch.tensor(c["lam"], dtype=torch.float32)))  # noqa: E731
    Y = _joined(torch.complex(shrink(o.real), shrink(o.imag)), X)
    return _grid(c, Y, _column_weights(c, X.shape[1], X.device))


def _exact_backward(c, w, x, g):
    nb, lam = c["nb"], float(torch.tensor(c["lam"], dtype=torch.float32))
    X = _spectrum(c, x)
    Xb, v, h, o, cw = _layers(c, w, X)
    ck = _column_weights(c, X.shape[1], X.device)
    dz = (_spectrum(c, g) * ck[None, :, None]).reshape(-1, nb, c["C"] // nb).transpose(0, 1)
    do = torch.complex(dz.real * (o.real.abs() > lam), dz.imag * (o.imag.abs() > lam))
    dh = torch.stack([do[k] @ cw["w2"][k].mH for k in range(nb)])
    dv = torch.complex(dh.real * (v.real > 0), dh.imag * (v.imag > 0))
    dX = torch.stack([dv[k] @ cw["w1"][k].mH for k in range(nb)])
    dx = g + _grid(c, _joined(dX, X), torch.ones_like(ck))
    pair = lambda t: torch.view_as_real(t.contiguous())  # noqa: E731
    dw1, dw2 = (pair(torch.stack([a[k].mH @ b[k] for k in range(nb)])) for a, b in ((Xb, dv), (h, do)))
    return dx, dw1, pair(dv.sum(1)), dw2, pair(do.sum(1))
