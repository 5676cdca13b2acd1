"""The work a user of this library has it do, as measurable cases.

A case is one call (or, for a layer step, one forward and backward) through the public entry points of
``paper_2509_25149_amd.binding``: quantizing an activation, a weight or a gradient, a linear layer's forward, a layer's
forward and backward, a weight gradient alone, the MXFP4 comparison format, and decoding a copy.  Sizes are those of
the 12B model's MLP (model dimension 5120, FFN dimension 20480, 8192 tokens), of the small parity configuration
(256 tokens, 512 -> 256) and of ragged layers in between; values are the synthetic stand-ins of ``synth.py``
(activations N(0, 1) with 0.1 % outliers, weights N(0, 0.02^2), gradients 1e-3 Student-t(3)).

``exact`` recomputes every case in plain torch: the quantizer's defining equations with one binary32 rounding per
operation (its results are whole bytes), everything after the codes in binary64.
"""
import torch

from paper_2509_25149_amd import binding as nv

RC = nv.LAYOUT_ROW | nv.LAYOUT_COL
TOKENS, D_MODEL, D_FFN = 8192, 5120, 20480      # the 12B model's MLP on one sequence


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # The smallest call there is in earnest: a layer input of the small configuration; launches and latency.
        dict(name="quantize_x_small", kind="quantize", operand="activation", tokens=256, d_in=512, d_out=0),
        # A layer input of the 12B model on its way into Fprop (row copy) and, rotated, into Wgrad (col copy).
        dict(name="quantize_x_12b", kind="quantize", operand="activation", tokens=TOKENS, d_in=D_MODEL, d_out=0),
        # A 12B weight once per optimizer step: 16x16 blocks, both orientations.
        dict(name="quantize_w_12b", kind="quantize", operand="weight", tokens=D_MODEL, d_in=D_FFN, d_out=0),
        # A 12B output gradient: stochastic rounding, both copies, the col copy rotated.
        dict(name="quantize_dy_12b", kind="quantize", operand="gradient", tokens=TOKENS, d_in=D_FFN, d_out=0),
        # One layer call of the small configuration.
        dict(name="forward_small", kind="forward", tokens=256, d_in=512, d_out=256),
        # Inference of the up-projection with a handful of sequences in flight: the weight's bytes count.
        dict(name="forward_few_tokens", kind="forward", tokens=64, d_in=D_MODEL, d_out=D_FFN),
        # A short prompt through an attention-sized projection, one tensor-level scale per token.
        dict(name="forward_row_scales", kind="forward_rows", tokens=512, d_in=D_MODEL, d_out=D_MODEL),
        # A weight gradient alone, FP32, 4096 tokens (the Wgrad parity configuration).
        dict(name="wgrad_4096", kind="wgrad", tokens=4096, d_in=D_MODEL, d_out=D_MODEL),
        # Training step of a layer none of whose sizes is a multiple of 64.
        dict(name="step_ragged", kind="step", tokens=1040, d_in=2064, d_out=1296),
        # Training step of the 12B model's up-projection on a full sequence: the largest.
        dict(name="step_12b", kind="step", tokens=TOKENS, d_in=D_MODEL, d_out=D_FFN),
        # Training step in the comparison format MXFP4 at an attention projection's size.
        dict(name="step_mx", kind="step_mx", tokens=4096, d_in=D_MODEL, d_out=D_MODEL),
        # A quantized activation decoded again (what a layer kept for its backward pass, or for inspection).
        dict(name="dequantize_12b", kind="dequantize", tokens=TOKENS, d_in=D_MODEL, d_out=0),
    ]


def _size(rng, lo, hi, multiple):
    """Log-uniform in [lo, hi]; half of the sizes odd multiples of the format's unit, half round ones."""
    n = lo * (hi / lo) ** rng.random()
    step = multiple if rng.random() < 0.5 else max(multiple, 256 if n >= 1024 else 64 if n >= 128 else 16)
    return min(hi, max(lo, int(round(n / step)) * step))


def draw(rng):
    kind = rng.choice(["quantize", "quantize", "forward", "forward", "forward_rows", "wgrad", "step", "step", "step_mx", "dequantize"])
    unit = 128 if kind == "step_mx" else 16
    case = dict(kind=kind, tokens=_size(rng, max(16, unit), TOKENS, unit), d_in=_size(rng, 256, D_MODEL, unit),
                d_out=_size(rng, 256, D_FFN, unit))
    if kind == "quantize":
        case["operand"] = rng.choice(["activation", "weight", "gradient"])
    if kind in ("quantize", "dequantize"):
        if case.get("operand", "activation") != "activation":
            case["d_in"] = case["d_out"]     # gradients and weights are as wide as the layer's output
        case["d_out"] = 0
    return case


# ---------------------------------------------------------------- inputs

def _generator(seed, which):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 8 + which)
    return g


def _activation(rows, cols, seed):
    g = _generator(seed, 0)
    x = torch.randn((rows, cols), generator=g, device="cuda", dtype=torch.float32)
    hit = torch.rand((rows, cols), generator=g, device="cuda") < 1e-3
    return torch.where(hit, x * 50.0, x).to(torch.bfloat16)


def _weight(rows, cols, seed):
    return (torch.randn((rows, cols), generator=_generator(seed, 1), device="cuda", dtype=torch.float32) * 0.02).to(torch.bfloat16)


def _gradient(rows, cols, seed):
    z = torch.randn((4, rows, cols), generator=_generator(seed, 2), device="cuda", dtype=torch.float32)
    chi = torch.sqrt((z[1] * z[1] + z[2] * z[2] + z[3] * z[3]) / 3.0).clamp_min(1e-12)
    return (z[0] / chi * 1e-3).to(torch.bfloat16)


def _seeds(seed):
    """Seeds of the sign diagonal and of the stochastic rounding."""
    return 2025 + seed, 0x5EED + 7 * seed


def _bytes(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")


# quantize calls: layout, block, rounding, rotation
_OPERANDS = {"activation": (RC, nv.BLOCK_1x16, nv.ROUND_RNE, True), "weight": (RC, nv.BLOCK_16x16, nv.ROUND_RNE, False),
             "gradient": (RC, nv.BLOCK_1x16, nv.ROUND_SR, True)}
_MAKE = {"activation": _activation, "weight": _weight, "gradient": _gradient}


def prepare(case, seed):
    """Inputs, the quantized weight and the buffers a program keeps from call to call."""
    kind, t, d_in, d_out = case["kind"], case["tokens"], case["d_in"], case["d_out"]
    rht, sr = _seeds(seed)
    st = dict(kind=kind, rht=rht, sr=sr)
    if kind == "quantize":
        layout, block, rounding, rot = _OPERANDS[case["operand"]]
        st.update(x=_MAKE[case["operand"]](t, d_in, seed), layout=layout, block=block, rounding=rounding, rot=rot,
                  q=nv.alloc_qtensor(t, d_in, layout), ws=_bytes(nv.quantized_sizes(t, d_in)[2]))
        return st
    if kind == "dequantize":
        st.update(q=nv.nvfp4_quantize(_activation(t, d_in, seed), nv.LAYOUT_ROW),
                  out=torch.empty((t, d_in), dtype=torch.bfloat16, device="cuda"))
        return st
    mx = kind == "step_mx"
    block = nv.BLOCK_MX32 if mx else nv.BLOCK_1x16
    if kind != "wgrad":
        st["qw"] = nv.nvfp4_quantize(_weight(d_in, d_out, seed), RC, nv.BLOCK_MX32 if mx else nv.BLOCK_16x16)
        st["y"] = torch.empty((t, d_out), dtype=torch.bfloat16, device="cuda")
    if kind in ("forward", "forward_rows"):
        layout = nv.LAYOUT_ROW | (nv.LAYOUT_ROW_SCALES if kind == "forward_rows" else 0)
        st.update(x=_activation(t, d_in, seed), layout=layout, qx=nv.alloc_qtensor(t, d_in, layout))
    elif kind == "wgrad":
        st.update(qx=nv.nvfp4_quantize(_activation(t, d_in, seed), nv.LAYOUT_COL, rht_on_col=True, rht_seed=rht),
                  qdy=nv.nvfp4_quantize(_gradient(t, d_out, seed), nv.LAYOUT_COL, rounding=nv.ROUND_SR, rht_on_col=True,
                                        rht_seed=rht, sr_seed=sr))
    else:
        st.update(x=_activation(t, d_in, seed), dy=_gradient(t, d_out, seed), qx=nv.alloc_qtensor(t, d_in, RC, block_dim=block),
                  qdy=nv.alloc_qtensor(t, d_out, RC, block_dim=block), dx=torch.empty((t, d_in), dtype=torch.bfloat16, device="cuda"))
    if kind in ("wgrad", "step", "step_mx"):
        st["dw"] = torch.empty((d_in, d_out), dtype=torch.float32, device="cuda")
    if not mx:
        st["ws"] = _bytes(max(nv.linear_workspace_bytes(t, d_in, d_out), nv.quantized_sizes(t, d_in)[2]))
    return st


# ---------------------------------------------------------------- one pass

def _copies(q):
    return [q.row_codes, q.row_scales, q.row_ts, q.col_codes, q.col_scales, q.col_ts]


def run(st):
    kind = st["kind"]
    if kind == "quantize":
        nv.nvfp4_quantize(st["x"], st["layout"], st["block"], st["rounding"], st["rot"], st["rht"], st["sr"], out=st["q"],
                          workspace=st["ws"])
        return _copies(st["q"])
    if kind == "dequantize":
        return nv.nvfp4_dequantize(st["q"], nv.COPY_ROW, out_dtype=nv.OUT_BF16, out=st["out"])
    if kind == "forward":
        return nv.nvfp4_linear_forward(st["x"], st["qw"], st["ws"], keep_for_backward=False, qx=st["qx"], y=st["y"])[0]
    if kind == "forward_rows":
        nv.nvfp4_quantize(st["x"], st["layout"], out=st["qx"], workspace=st["ws"])
        return nv.nvfp4_gemm(st["qx"], st["qw"], nv.OP_FPROP, nv.OUT_BF16, out=st["y"], workspace=st["ws"])
    if kind == "wgrad":
        return nv.nvfp4_gemm(st["qx"], st["qdy"], nv.OP_WGRAD, nv.OUT_F32, out=st["dw"], workspace=st["ws"])
    if kind == "step":
        y, qx = nv.nvfp4_linear_forward(st["x"], st["qw"], st["ws"], True, st["rht"], qx=st["qx"], y=st["y"])
        dx, _ = nv.nvfp4_linear_backward(st["dy"], qx, st["qw"], st["dw"], st["ws"], accumulate_dw=False, sr_seed=st["sr"],
                                         qdy=st["qdy"], dx=st["dx"])
        return [y, dx, st["dw"]]
    nv.nvfp4_quantize(st["x"], RC, nv.BLOCK_MX32, nv.ROUND_RNE, True, st["rht"], out=st["qx"])
    nv.nvfp4_gemm(st["qx"], st["qw"], nv.OP_FPROP, nv.OUT_BF16, out=st["y"])
    nv.nvfp4_quantize(st["dy"], RC, nv.BLOCK_MX32, nv.ROUND_SR, True, st["rht"], st["sr"], out=st["qdy"])
    nv.nvfp4_gemm(st["qdy"], st["qw"], nv.OP_DGRAD, nv.OUT_BF16, out=st["dx"])
    nv.nvfp4_gemm(st["qx"], st["qdy"], nv.OP_WGRAD, nv.OUT_F32, out=st["dw"])
    return [st["y"], st["dx"], st["dw"]]


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Each input read once, each result written once; 2 M N K per product, a few operations per quantized element."""
    kind, t, d_in, d_out = case["kind"], case["tokens"], case["d_in"], case["d_out"]
    copy = 1 / 2 + (1 / 32 if kind == "step_mx" else 1 / 16)      # bytes per element of a quantized copy
    nx, nw, ny = t * d_in, d_in * d_out, t * d_out
    if kind == "quantize":
        return dict(bytes=nx * (2 + 2 * copy) + 16, flops=nx * (4 if case["operand"] == "weight" else 9))
    if kind == "dequantize":
        return dict(bytes=nx * (2 + copy) + 4, flops=2 * nx)
    if kind in ("forward", "forward_rows"):
        return dict(bytes=2 * nx + copy * nw + 2 * ny, flops=2 * t * d_in * d_out)
    if kind == "wgrad":
        return dict(bytes=copy * (nx + ny) + 4 * nw, flops=2 * t * d_in * d_out)
    return dict(bytes=2 * (nx + ny) + 2 * copy * nw + 2 * (nx + ny) + 4 * nw, flops=6 * t * d_in * d_out)


def tolerance(case):
    """Codes, scales, tensor scales and decoded values are one defined sequence of roundings.  Products accumulate in
    FP32; where they leave as bf16 that rounding (2^-9 of a value at the most) is all that shows."""
    kind = case["kind"]
    if kind in ("quantize", "dequantize"):
        return "exact"
    if kind == "wgrad":
        return {"rel": 1e-6}      # measured 3e-8 to 6e-8 against binary64 here, 4e-7 at the longest sums (20480)
    return {"rel": 7e-3}          # measured 1.7e-3 against binary64


# ---------------------------------------------------------------- the same in plain torch

_CHUNK = 1 << 24      # elements worked on at a time


def _mulhilo(m, x):
    """High and low word of the 64-bit product of two 32-bit words (held in int64)."""
    p0, p1 = m * (x & 0xFFFF), m * (x >> 16)
    s = p1 + (p0 >> 16)
    return s >> 16, ((s & 0xFFFF) << 16) | (p0 & 0xFFFF)


def _philox(c0, c1, c2, c3, key):
    c = [torch.as_tensor(v, dtype=torch.int64, device="cuda") for v in (c0, c1, c2, c3)]
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, c[0])
        h1, l1 = _mulhilo(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _halves(words):
    """[.., 8] 16-bit draws of Philox calls: word t serves elements 2t (low half) and 2t + 1 (high half)."""
    return torch.stack([h for w in words for h in (w & 0xFFFF, w >> 16)], dim=-1).to(torch.int32)


def _signs(seed, d):
    w = _philox(0, 0, 0, 0xFFFFFFFF, seed)
    return torch.tensor([-1.0 if (int(w[i // 32]) >> (i % 32)) & 1 else 1.0 for i in range(d)], device="cuda")


def _rotate(v, seed, d):
    """Groups of d along the last dimension: sign diagonal, Walsh-Hadamard butterfly, 1 / sqrt(d), each one binary32 operation."""
    v = v.reshape(*v.shape[:-1], -1, d) * _signs(seed, d)
    h = 1
    while h < d:
        p = v.reshape(*v.shape[:-1], d // (2 * h), 2, h)
        a, b = p[..., 0, :], p[..., 1, :]
        v = torch.stack([a + b, a - b], dim=-2).reshape(v.shape)
        h *= 2
    norm = torch.tensor(d ** -0.5, dtype=torch.float64).to(torch.float32).item()
    return (v * norm).flatten(-2)


def _e2m1(v, draws):
    """E2M1 codes of scaled binary32 values: nearest (ties to the even code), or up when position + draw >= 1."""
    m = v.abs()
    if draws is None:
        idx = ((m > 0.25).byte() + (m >= 0.75).byte() + (m > 1.25).byte() + (m >= 1.75).byte() + (m > 2.5).byte() +
               (m >= 3.5).byte() + (m > 5.0).byte())
    else:
        grid = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0, 8.0], device="cuda")
        lo = sum((m >= g).int() for g in (0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0))
        base, step = grid[lo], grid[(lo + 1)] - grid[lo]
        p = ((m.double() - base.double()) / step.double() * 65536.0).floor().clamp_max(65535.0).to(torch.int32)
        idx = torch.where(lo == 7, lo, lo + ((p + draws) >= 65536).int()).byte()
    return idx + torch.signbit(v).byte() * 8


class _Ref:
    """One quantized copy: codes and scale bytes as stored, the tensor scale, decoded values on demand."""

    def __init__(self, codes, scales, ts, block):
        self.codes, self.scales, self.ts, self.block = codes, scales, ts, block

    def decoded(self):
        """value(code) * block scale * s_dec in binary64."""
        table = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64, device="cuda")
        n = self.codes.shape[0]
        nib = torch.stack([self.codes & 15, self.codes >> 4], dim=-1).reshape(n, -1)
        s = (torch.exp2(self.scales.double() - 127.0) if self.block == 32 else self.scales.view(torch.float8_e4m3fn).double())
        out = torch.empty(nib.shape, dtype=torch.float64, device="cuda")
        step = max(1, _CHUNK // nib.shape[1])
        for r in range(0, n, step):
            v = table[nib[r:r + step].int()]
            out[r:r + step] = (v.reshape(v.shape[0], -1, self.block) * s[r:r + step, :, None]).flatten(1)
        sd = self.ts[:n, None] if self.ts.numel() > 2 else self.ts[0]
        return out * sd.double()


def _ref_copy(x, col, mx=False, block2d=False, sr=None, rht=None, per_row=False):
    """Eq. 1-4 for one copy of the bf16 tensor x: one binary32 rounding per operation."""
    v = (x.t() if col else x).contiguous()
    outer, inner = v.shape
    blk = 32 if mx else 16
    step = max(16, _CHUNK // inner // 16 * 16)
    rows = lambda r: _rotate(v[r:r + step].float(), rht, blk) if rht is not None else v[r:r + step].float()
    if mx:
        s_enc = s_dec = amax = None
        ts = torch.tensor([1.0, 0.0], device="cuda")
    else:
        amax = torch.cat([rows(r).abs().amax(dim=1) for r in range(0, outer, step)])
        amax = amax if per_row else amax.amax().reshape(1)
        s_enc = (2688.0 / amax.double()).float()
        s_enc = torch.where(amax == 0, torch.ones_like(amax), s_enc.clamp_max(3.4028234663852886e38))
        s_dec = (1.0 / s_enc.double()).float()
        ts = torch.cat([s_dec, amax])
        s_enc, s_dec = s_enc.expand(outer), s_dec.expand(outer)
    codes, scales = [], []
    for r in range(0, outer, step):
        w = rows(r)
        n = w.shape[0]
        b = w.reshape(n, -1, blk)
        top = b.abs().amax(dim=2)
        if block2d:
            top = top.reshape(n // 16, 16, -1).amax(dim=1, keepdim=True).expand(-1, 16, -1).reshape(n, -1)
        sixth = (top.double() / 6.0).float()
        if mx:
            mant, ex = torch.frexp(sixth.double())      # sixth = mant * 2^ex, mant in [0.5, 1): up to a power of two
            e = torch.where(sixth == 0, torch.full_like(ex, -127), torch.where(mant == 0.5, ex - 1, ex)).clamp(-127, 127)
            byte = (e + 127).to(torch.uint8)
            enc = torch.exp2(-e.double()).float()
        else:
            s8 = (sixth.double() * s_enc[r:r + n, None].double()).float().clamp_max(448.0).to(torch.float8_e4m3fn)
            byte = s8.view(torch.uint8)
            den = (s8.double() * s_dec[r:r + n, None].double()).float()
            enc = torch.where(den == 0, torch.zeros_like(den), (1.0 / den.double()).float())
        scaled = (b * enc[..., None]).reshape(n, inner)
        draws = None
        if sr is not None:
            i = torch.arange(r, r + n, device="cuda")
            k = torch.arange(inner // 8, device="cuda")
            if mx and col:      # this copy's own draws: counter (row / 8, column, 1, 0)
                draws = _halves(_philox(k[None, :].expand(n, -1), i[:, None].expand(-1, inner // 8), 1, 0, sr)).reshape(n, inner)
            elif col:           # element (row, column) of the tensor: counter (column / 8, row, 0, 0)
                g0, g1 = r // 8, (r + n + 7) // 8
                rr = torch.arange(inner, device="cuda")
                gg = torch.arange(g0, g1, device="cuda")
                d = _halves(_philox(gg[None, :].expand(inner, -1), rr[:, None].expand(-1, g1 - g0), 0, 0, sr))
                draws = d.reshape(inner, -1)[:, r - 8 * g0:r - 8 * g0 + n].t()
            else:
                draws = _halves(_philox(k[None, :].expand(n, -1), i[:, None].expand(-1, inner // 8), 0, 0, sr)).reshape(n, inner)
        c = _e2m1(scaled, draws)
        codes.append(c[:, 0::2] | (c[:, 1::2] << 4))
        scales.append(byte)
    return _Ref(torch.cat(codes), torch.cat(scales), ts, blk)


def exact(case, seed):
    kind, t, d_in, d_out = case["kind"], case["tokens"], case["d_in"], case["d_out"]
    rht, sr = _seeds(seed)
    if kind == "quantize":
        op = case["operand"]
        x = _MAKE[op](t, d_in, seed)
        kw = dict(block2d=op == "weight", sr=sr if op == "gradient" else None)
        row, col = _ref_copy(x, False, **kw), _ref_copy(x, True, rht=None if op == "weight" else rht, **kw)
        return [row.codes, row.scales, row.ts, col.codes, col.scales, col.ts]
    if kind == "dequantize":
        return _ref_copy(_activation(t, d_in, seed), False).decoded()
    product = lambda a, b: a.decoded() @ b.decoded().t()
    x, mx = _activation(t, d_in, seed), kind == "step_mx"
    if kind == "wgrad":
        return product(_ref_copy(x, True, rht=rht), _ref_copy(_gradient(t, d_out, seed), True, sr=sr, rht=rht))
    w = _weight(d_in, d_out, seed)
    y = product(_ref_copy(x, False, mx=mx, per_row=kind == "forward_rows"), _ref_copy(w, True, mx=mx, block2d=not mx))
    if kind in ("forward", "forward_rows"):
        return y
    dy = _gradient(t, d_out, seed)
    dx = product(_ref_copy(dy, False, mx=mx, sr=sr), _ref_copy(w, False, mx=mx, block2d=not mx))
    dw = product(_ref_copy(x, True, mx=mx, rht=rht), _ref_copy(dy, True, mx=mx, sr=sr, rht=rht))
    return [y, dx, dw]
