"""The calls whose speed is measured: what a program does that decomposes a model's linear layers (error tables over
quantization configurations, the decomposition itself), stores and reloads the quantized component, and runs the
decomposed layers forward, for one sequence, a few sequences and long prompts.

Sizes are those of the repository's workloads (the 768 x 768 matrix, RoBERTa-Large and LLaMA-2 linear layers) and, where
drawn, generic sizes between them.  Inputs have the distributions of gen.py (Student-t noise, a planted decaying low-rank
part, outlier columns, heavy feature columns in the activations), drawn on the GPU because they are made many times."""
from __future__ import annotations

import math
from statistics import NormalDist

import torch

from paper_2311_12023_amd import lq

DEV = "cuda"


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(231112023 + seed)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _weight(g, d, k, planted, outliers=True):
    """0.02 * Student-t(5) noise, 0.1 % of the columns times 20, plus a planted part with singular values 0.8^i."""
    w = torch.empty((d, k), device=DEV)
    for lo in range(0, d, 2048):                       # in strips: the largest matrix has 235 M weights
        part = w[lo:lo + 2048]
        chi = torch.zeros_like(part)
        for _ in range(5):
            chi.addcmul_(z := _randn(g, *part.shape), z)
        torch.div(_randn(g, *part.shape).mul_(0.02 * math.sqrt(5.0)), chi.sqrt_(), out=part)
    if outliers:
        w[:, torch.randperm(k, generator=g, device=DEV)[:max(1, round(0.001 * k))]] *= 20.0
    if planted:
        u = torch.linalg.qr(_randn(g, d, planted))[0]
        v = torch.linalg.qr(_randn(g, k, planted))[0]
        w.addmm_(u * 0.8 ** torch.arange(planted, device=DEV), v.T)
    return w


def _fisher(g, n):
    return torch.exp(_randn(g, n))                     # squares of log-normal row / column gradient scales


def _activations(g, m, d):
    x = _randn(g, m, d)
    x[:, torch.randperm(d, generator=g, device=DEV)[:max(1, d // 256)]] *= 8.0
    return x


_CODEBOOKS = {}


def _codebook(bits):
    """NormalFloat codes: normal quantiles of 2^(b-1) probabilities up to 1/2 and 2^(b-1) + 1 from there, 1/2 once."""
    if bits not in _CODEBOOKS:
        half, delta, inv = 1 << (bits - 1), 0.5 * (1 / 30 + 1 / 32), NormalDist().inv_cdf
        q = [inv(delta + (0.5 - delta) * i / (half - 1)) for i in range(half - 1)] + [0.0]
        q += [inv(0.5 + (0.5 - delta) * i / half) for i in range(1, half + 1)]
        _CODEBOOKS[bits] = torch.tensor([v / q[-1] for v in q], dtype=torch.float64).float().to(DEV)
    return _CODEBOOKS[bits]


def _quantize(flat, c):
    """Quantize in plain torch: -> (codes int64, scale_idx uint8, v fp32 rounded to b2)."""
    code = _codebook(c["bits"])
    mid = (code[1:].double() + code[:-1].double()) / 2
    absmax = flat.reshape(-1, c["block"]).abs().amax(1)
    inv = torch.where(absmax > 0, 1.0 / absmax, torch.zeros_like(absmax)).repeat_interleave(c["block"])
    codes = torch.bucketize((flat * inv).double(), mid)
    nb, b1 = absmax.numel(), c["scale_block"]
    ng = -(-nb // b1)
    v = torch.zeros(ng * b1, device=flat.device)
    v[:nb] = absmax
    v = v.reshape(ng, b1).amax(1)
    top = 2 ** (c["scale_bits"] - 1) - 1
    sigma = (v / top).repeat_interleave(b1)[:nb]
    idx = torch.where(sigma > 0, absmax / sigma, torch.zeros_like(sigma)).round().clamp(0, top)
    cast = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}[c["v_dtype"]]
    return codes, idx.to(torch.uint8), v.to(cast).float()


def _pack(codes, bits):
    """Little-endian bit stream, code j in bits [j * bits, (j + 1) * bits); the number of codes is a multiple of 8."""
    c = codes.reshape(-1, 8)
    word = sum(c[:, j] << (j * bits) for j in range(8))            # 8 codes are `bits` bytes; 8 bits wrap into the sign
    return torch.stack([((word >> (8 * b)) & 255).to(torch.uint8) for b in range(bits)], 1).reshape(-1)


def _dequantize64(codes, idx, v, c):
    top = 2 ** (c["scale_bits"] - 1) - 1
    scale = idx.double() * (v.double() / top).repeat_interleave(c["scale_block"])[:idx.numel()]
    return _codebook(c["bits"])[codes].double() * scale.repeat_interleave(c["block"])


def _cfg(c):
    return lq.config(c["bits"], c["block"], c["scale_block"], c["scale_bits"], c["v_dtype"])


def _grid(c):
    """The first `cells` of a fixed shuffle of bits x B0 x B1 (so that few cells still mix code widths)."""
    blocks = [(b0, b1) for b0 in (16, 32, 64) for b1 in ((256,) if c["cells"] <= 9 else (16, 64, 256))]
    bits = (2, 3, 4) if c["cells"] <= 9 else (2, 3, 4, 8)
    full = [(b, *blk) for b in bits for blk in blocks]
    return [full[(7 * i) % len(full)] for i in range(c["cells"])]


# ---------------------------------------------------------------- the cases

NF3 = dict(bits=3, block=64, scale_block=256, scale_bits=8, v_dtype="fp32")
NF4 = dict(bits=4, block=64, scale_block=256, scale_bits=8, v_dtype="bf16")


def listed():
    return [
        # the smallest matrix of the workloads, stored quantized: one short launch
        dict(name="quantize_768", kind="quantize", d=768, k=768, **NF3),
        # the largest one, as when a 70B model's MLP weights are quantized: streaming
        dict(name="quantize_8192x28672", kind="quantize", d=8192, k=28672, **NF4),
        # a stored weight expanded for a program that wants it dense; a ragged code width and small blocks
        dict(name="dequantize_4096x11008", kind="dequantize", d=4096, k=11008,
             bits=3, block=16, scale_block=64, scale_bits=8, v_dtype="fp16"),
        # decoding one token of one sequence through a decomposed attention projection, without a workspace
        dict(name="forward_1_row", kind="forward", m=1, d=4096, k=4096, rank=64, precision=0, static=True, **NF4),
        # decoding two dozen sequences together through an up projection
        dict(name="forward_24_rows", kind="forward", m=24, d=4096, k=11008, rank=64, precision=0, static=False, **NF4),
        # a prompt of odd length through a down projection, fp32-grade products
        dict(name="forward_1000_rows", kind="forward", m=1000, d=11008, k=4096, rank=64, precision=0, static=False, **NF4),
        # a training batch of 4096 tokens in bf16 through a 3-bit layer
        dict(name="forward_4096_rows_bf16", kind="forward", m=4096, d=4096, k=4096, rank=64, precision=1, static=False,
             **NF3),
        # the low-rank factors of a pretrained weight on their own (cold start of the randomized SVD)
        dict(name="factorize_4096", kind="factorize", d=4096, k=4096, rank=64, weighted=False),
        # one small matrix decomposed from start to finish with 8-bit codes
        dict(name="decompose_768", kind="decompose", d=768, k=768, rank=8, weighted=False, iters=5, bits=8, block=64,
             scale_block=256, scale_bits=8, v_dtype="fp32"),
        # one MLP weight with Fisher weights, the chosen configuration applied
        dict(name="decompose_4096x11008_fisher", kind="decompose", d=4096, k=11008, rank=64, weighted=True, iters=10,
             **NF3),
        # a small encoder layer's row of the error table
        dict(name="table_1024x4096_9", kind="table", d=1024, k=4096, rank=8, weighted=False, iters=10, cells=9),
        # an attention projection's row of the error table, the whole grid: what a model's search spends its time on
        dict(name="table_4096_36", kind="table", d=4096, k=4096, rank=64, weighted=False, iters=10, cells=36),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["quantize", "dequantize", "forward", "forward", "forward", "factorize", "decompose", "table", "table"])
    c = dict(kind=kind)
    if kind != "factorize":
        c.update(bits=rng.choice([2, 3, 4, 8]), block=rng.choice([16, 32, 64]), scale_block=rng.choice([16, 64, 256]),
                 scale_bits=8, v_dtype=rng.choice(["fp32", "bf16", "fp16"]))
    if kind in ("quantize", "dequantize"):
        return dict(c, d=int(_log(rng, 256, 8192)), k=64 * int(_log(rng, 12, 448)))
    if kind == "forward":
        m = int(_log(rng, 1, 4097))
        static = m <= 4 and rng.random() < 0.5
        return dict(c, m=m, d=32 * int(_log(rng, 24, 345)), k=64 * int(_log(rng, 12, 173)),
                    rank=rng.choice([0, 8, 16, 33, 64]) if not static else 64, precision=rng.choice([0, 0, 1]), static=static)
    small = rng.random() < 0.5
    d, k = (int(_log(rng, 512, 2048)), 64 * int(_log(rng, 8, 64))) if small else (int(_log(rng, 2048, 4097)),
                                                                                    64 * int(_log(rng, 32, 65)))
    c.update(d=d, k=k, rank=rng.choice([8, 16]) if small else rng.choice([32, 64]))
    if kind == "factorize":
        return dict(c, weighted=rng.random() < 0.3)
    c.update(weighted=rng.random() < 0.3, iters=rng.choice([3, 5, 10]))
    if kind == "table":
        for name in ("bits", "block", "scale_block", "scale_bits", "v_dtype"):
            del c[name]
        c.update(cells=rng.choice([5, 9, 18, 27, 36]))
    return c


def prepare(c, seed):
    g, kind = _gen(seed), c["kind"]
    d, k = c["d"], c["k"]
    s = dict(case=c)
    if kind == "quantize":
        s.update(x=_weight(g, d, k, 0).reshape(-1), cfg=_cfg(c))
    elif kind in ("dequantize", "forward"):
        codes, s["idx"], s["v"] = _quantize(_weight(g, d, k, 0).reshape(-1), c)
        s.update(codes=_pack(codes, c["bits"]), cfg=_cfg(c))
        del codes
        if kind == "forward":
            s["x"] = _activations(g, c["m"], d)
            s["l1"] = _randn(g, d, c["rank"]) * 0.05 if c["rank"] else None
            s["l2"] = _randn(g, c["rank"], k) * 0.05 if c["rank"] else None
            if not c["static"]:
                s["ws"] = lq.matmul_workspace(c["m"], d, k, c["rank"])
    else:
        s["w"] = _weight(g, d, k, 2 * c["rank"] if c["rank"] <= 16 else 64, outliers=c["rank"] > 16)
        s["row_w"], s["col_w"] = (_fisher(g, d), _fisher(g, k)) if c["weighted"] else (None, None)
        if kind == "factorize":
            need = lq._lib.lq_factorize_workspace_bytes(d, k, c["rank"], None)
        elif kind == "decompose":
            need = lq._lib.lq_decompose_workspace_bytes(d, k, c["rank"], None)
            s["cfg"] = _cfg(c)
        else:
            s["cfgs"] = [lq.config(*t) for t in _grid(c)]
            need = lq._lib.lq_error_table_workspace_bytes(d, k, c["rank"], c["cells"], None)
        s["ws"] = torch.empty(need + 256, dtype=torch.uint8, device=DEV)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "quantize":
        return lq.nf_quantize(s["x"], s["cfg"])
    if kind == "dequantize":
        return lq.nf_dequantize(s["codes"], s["idx"], s["v"], c["d"] * c["k"], s["cfg"])
    if kind == "forward":
        if c["static"]:
            return lq.matmul_few_rows_static(s["x"], s["codes"], s["idx"], s["v"], s["cfg"], c["k"], s["l1"], s["l2"])
        return lq.matmul(s["x"], s["codes"], s["idx"], s["v"], s["cfg"], c["k"], s["l1"], s["l2"],
                         precision=c["precision"], workspace=s["ws"])
    if kind == "factorize":
        l1, l2, sigma = lq.factorize(s["w"], c["rank"], s["row_w"], s["col_w"], seed=1, workspace=s["ws"])
        return {"low_rank": l1 @ l2, "sigma": sigma}   # the sign of a pair of singular vectors is free, their product is not
    if kind == "decompose":
        o = lq.decompose(s["w"], c["rank"], s["cfg"], c["iters"], row_w=s["row_w"], col_w=s["col_w"], seed=1,
                         workspace=s["ws"], want_dense=True)
        if c["bits"] == 8:
            return {"low_rank": o["L1"] @ o["L2"], "Q": o["Q"], "sigma": o["sigma"], "trace": list(o["trace"])}
        # With coarse codes a difference of rounding in the first iteration (1e-6) flips codes that move the next singular
        # vectors, which flip more: two correct runs end 5 to 10 % apart in Q (measured between fp32 and split products),
        # and yet within 3e-3 in the singular values and 2e-4 in the errors.  These are what can be compared.
        return {"sigma": o["sigma"], "trace": list(o["trace"])}
    err, storage, trace = lq.error_table(s["w"], c["rank"], s["cfgs"], c["iters"], row_w=s["row_w"], col_w=s["col_w"],
                                         seed=1, workspace=s["ws"], want_trace=True)
    return {"err_sq": err, "storage": storage, "trace": [trace[:, t] for t in range(c["iters"])]}


def _stored_bytes(c):
    n = c["d"] * c["k"]
    return n * c["bits"] / 8 + n / c["block"] + 4 * math.ceil(n / (c["block"] * c["scale_block"]))


def work(c):
    d, k, kind = c["d"], c["k"], c["kind"]
    n = d * k
    if kind in ("quantize", "dequantize"):
        return {"bytes": 4 * n + _stored_bytes(c), "flops": 4 * n}
    if kind == "forward":
        m, r = c["m"], c["rank"]
        return {"bytes": _stored_bytes(c) + 4 * (m * d + m * k + r * (d + k)), "flops": 2 * m * n + 2 * m * r * (d + k)}
    r = c["rank"]
    factors = 4 * r * (d + k)
    if kind == "factorize":
        return {"bytes": 4 * n + factors + 4 * n, "flops": 4 * n * r + 2 * n * r}
    # an iteration: one application of A and of its transpose to r vectors, L1 L2, and the quantizer
    cells = c.get("cells", 1)
    out = 8 * cells * (c["iters"] + 2) if kind == "table" else factors + 8 * n
    return {"bytes": 4 * n + out, "flops": cells * c["iters"] * (6 * n * r + 10 * n)}


def tolerance(c):
    kind = c["kind"]
    if kind in ("quantize", "dequantize"):
        return "exact"
    if kind == "forward":
        if c["precision"] == 1 and c["m"] > 8:
            return {"rel": 1e-2}
        return {"rel": 2e-5} if c["m"] > 8 else {"rel": 1e-6}
    # Four times what fp32 products, split products and a tighter cold start differ by on the listed cases.
    if kind == "factorize":
        return {"rel": 2e-3, "max": 0.03}
    if kind == "decompose":
        return {"rel": 0.03, "max": 0.99} if c["bits"] == 8 else {"rel": 8e-3, "max": 0.02}
    return {"rel": 1e-3, "max": 4e-3}


def _top64(a, rank):
    """The rank leading singular values and the best rank-r approximation of `a` (float64): subspace iteration far past
    float32 accuracy, orthonormalised twice by Cholesky."""
    g = _gen(5)
    l = min(4 * rank + 32, *a.shape)
    y = torch.randn(a.shape[1], l, generator=g, device=a.device, dtype=torch.float64)

    def ortho(y):
        for _ in range(2):
            y = torch.linalg.solve_triangular(torch.linalg.cholesky(y.T @ y), y.T, upper=False).T
        return y.contiguous()

    y = ortho(y)
    last = None
    for it in range(400):
        b = ortho(a @ y)
        y = a.T @ b
        if it % 40 == 39:
            s = torch.linalg.svdvals(y.cpu())[:rank]
            if last is not None and float(((s - last) / s).abs().max()) < 1e-13:
                break
            last = s
        y = ortho(y)
    b = ortho(a @ y)
    u, s, vt = torch.linalg.svd((b.T @ a).cpu(), full_matrices=False)
    u, s, vt = (t[..., :rank].to(a.device) if t is not vt else t[:rank].to(a.device) for t in (u, s, vt))
    return s, (b @ (u * s)) @ vt


def exact(c, seed):
    kind = c["kind"]
    s = prepare(c, seed) if kind in ("quantize", "dequantize", "forward", "factorize") else None
    if kind == "quantize":
        return None, None, _quantize(s["x"], c)[2]
    if kind in ("dequantize", "forward"):
        codes = _quantize(_weight(_gen(seed), c["d"], c["k"], 0).reshape(-1), c)[0]
        q = _dequantize64(codes, s["idx"], s["v"], c)
        if kind == "dequantize":
            return q
        q = q.reshape(c["d"], c["k"])
        y = s["x"].double() @ q
        return y + (s["x"].double() @ s["l1"].double()) @ s["l2"].double() if c["rank"] else y
    if kind == "factorize":
        rw, cw = (s["row_w"].double().sqrt()[:, None], s["col_w"].double().sqrt()) if c["weighted"] else (1.0, 1.0)
        sigma, low = _top64(rw * s["w"].double() * cw, c["rank"])
        return {"low_rank": low / rw / cw, "sigma": sigma}
    # The errors of a decomposition have no value that 64 bits determine to better than fp32 products do: the first
    # iteration's jumps by 1e-6 to 1e-5 where a block scale rounds to the other index (measured between fp32 products, split
    # products and float64 on several seeds), and the later ones amplify that.  The SVD inside is covered by "factorize".
    if kind == "decompose":
        return None
    cells = [dict(NF3, bits=b, block=b0, scale_block=b1) for b, b0, b1 in _grid(c)]
    storage = [c["d"] * c["k"] * (f["bits"] + 8 / f["block"] + 32 / (f["block"] * f["scale_block"])) for f in cells]
    return {"err_sq": None, "storage": torch.tensor(storage, dtype=torch.float64), "trace": [None] * c["iters"]}
