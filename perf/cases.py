"""Workloads for timing the library through its Python binding.

A case is a dict of plain values; `kind` says which entry points it goes through:

  apply    perq_permute_rotate_quant: T rows of d channels, blocks of b, one of the 4-bit formats.
           perm "none" is P = I (the permutation merged into the weights), "given" hands over the
           calibrated permutation, "prepared" also the form perq_perm_prepare makes of it.  pad > 0
           are rows that lie `pad` elements further apart than they are wide.
  stat     perq_colabs_mean / perq_colabs_absmax over T calibration rows.
  diagnose what a study of one layer runs on a batch: the fp32 rotation output, its 4-bit form, the
           quantization error and the block statistics of every token.
  product  the quantized product of T activation rows and N weight rows (perq_w4a4_gemm_ref,
           perq_w4a4_mxfp4_gemm_ref), codes and scales in hand.

Activations are heavy tailed with one channel in a hundred fifty times larger, the law of the
repository's synthetic workloads; permutations are the calibrated ones (Algorithm 1).
"""
import math

import numpy as np
import torch

from paper_2601_22347_amd import binding

MOST_ELEMENTS = 65536 * 8192        # T * d of the largest listed apply case
MOST_PRODUCT = 2048 * 4096 * 4096   # T * N * d of the largest listed product


def listed():
    return [
        # one step of token generation for a batch of sixteen: launch and latency
        {"name": "decode_16x4096", "kind": "apply", "T": 16, "d": 4096, "b": 128, "fmt": "int4", "perm": "prepared", "pad": 0},
        # one prompt of 2048 tokens at the Llama3-1B down projection
        {"name": "prompt_2048x8192", "kind": "apply", "T": 2048, "d": 8192, "b": 32, "fmt": "int4", "perm": "prepared", "pad": 0},
        # a ragged batch whose rows are a slice of a wider tensor, at a width that is no power of two,
        # with the asymmetric quantizer of the paper's INT4 results
        {"name": "slice_4001x3072_asym", "kind": "apply", "T": 4001, "d": 3072, "b": 128, "fmt": "int4_asym", "perm": "given", "pad": 64},
        # the Llama3-8B widths at throughput batch size: hidden state, and down projection with large blocks
        {"name": "batch_32768x4096", "kind": "apply", "T": 32768, "d": 4096, "b": 128, "fmt": "int4", "perm": "prepared", "pad": 0},
        {"name": "batch_32768x14336_b2048", "kind": "apply", "T": 32768, "d": 14336, "b": 2048, "fmt": "int4", "perm": "prepared", "pad": 0},
        # MXFP4 with its natural block size on the longest batch
        {"name": "batch_65536x8192_mxfp4", "kind": "apply", "T": 65536, "d": 8192, "b": 32, "fmt": "mxfp4", "perm": "prepared", "pad": 0},
        # narrow rows, full-vector rotation, permutation merged away
        {"name": "narrow_16384x2048_mxfp4", "kind": "apply", "T": 16384, "d": 2048, "b": 2048, "fmt": "mxfp4", "perm": "none", "pad": 0},
        # the full-vector rotation of a width that is no power of two (14336 = 2^9 * 28)
        {"name": "full_32768x14336", "kind": "apply", "T": 32768, "d": 14336, "b": 14336, "fmt": "int4", "perm": "none", "pad": 0},
        # the calibration statistic of Algorithm 1 over 4096 tokens
        {"name": "calibrate_4096x8192", "kind": "stat", "T": 4096, "d": 8192, "stat": "mean"},
        # the per-token quantities of the paper's analysis for one layer and 2048 tokens
        {"name": "diagnose_2048x8192", "kind": "diagnose", "T": 2048, "d": 8192, "b": 32, "fmt": "int4", "perm": "given"},
        # the 4-bit product those codes are for, in both formats
        {"name": "product_int4_2048", "kind": "product", "T": 2048, "N": 4096, "d": 4096, "fmt": "int4"},
        {"name": "product_mxfp4_2048", "kind": "product", "T": 2048, "N": 2048, "d": 8192, "fmt": "mxfp4"},
    ]


WIDTHS = (512, 1024, 1536, 2048, 2560, 2880, 3072, 3584, 4096, 5120, 6144, 7168, 8192, 9728, 11008, 12288, 14336, 16384, 28672, 32768)
FULL_WIDTHS = {3072: 12, 3584: 28, 6144: 12, 7168: 28, 9728: 76, 12288: 12, 14336: 28, 28672: 28}
FORMATS = ("int4", "int4", "mxfp4", "mxfp4", "int4_asym", "fp4_token", "fp4_token7")


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_block(rng, d):
    top = d & -d                                   # largest power of two that divides the row
    return 1 << rng.randint(4, top.bit_length() - 1)


def draw(rng):
    kind = rng.choice(("apply", "apply", "apply", "apply", "apply", "stat", "diagnose", "product"))
    d = rng.choice(WIDTHS)
    if kind == "apply":
        T = _log_uniform(rng, 1, min(65536, MOST_ELEMENTS // d))
        b = d if d in FULL_WIDTHS and rng.random() < 0.3 else _draw_block(rng, d)
        perms = ["none", "given"]
        if d >= 4096 and d % 512 == 0 and b <= 4096 and b & (b - 1) == 0:
            perms += ["prepared", "prepared"]
        return {"kind": kind, "T": T, "d": d, "b": b, "fmt": rng.choice(FORMATS), "perm": rng.choice(perms),
                "pad": 0 if rng.random() < 0.75 else 8 * rng.randint(1, 64)}
    if kind == "stat":
        return {"kind": kind, "T": _log_uniform(rng, 16, 32768), "d": d, "stat": rng.choice(("mean", "mean", "absmax"))}
    if kind == "diagnose":
        return {"kind": kind, "T": _log_uniform(rng, 16, max(16, (1 << 26) // d)), "d": d, "b": _draw_block(rng, d),
                "fmt": rng.choice(FORMATS), "perm": rng.choice(("none", "given"))}
    T, N = _log_uniform(rng, 1, 4096), _log_uniform(rng, 64, 14336)
    T = max(1, min(T, MOST_PRODUCT // (N * d)))
    return {"kind": kind, "T": T, "N": N, "d": d, "fmt": rng.choice(("int4", "mxfp4"))}


# ---- inputs --------------------------------------------------------------------------------------
def _rows(T, d, pad, seed):
    """bf16 [T, d] on the GPU: Student-t(3) entries, one channel in a hundred times 50, within +-1e4."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62))
    gain = torch.ones(d, device="cuda")
    gain[torch.randperm(d, generator=g, device="cuda")[:max(1, d // 100)]] = 50.0
    x = torch.empty((T, d + pad), dtype=torch.bfloat16, device="cuda")
    step = max(1, (1 << 26) // d)
    for r in range(0, T, step):
        n = min(T, r + step) - r
        block = torch.randn((n, d), generator=g, device="cuda")
        spread = torch.zeros_like(block)
        for _ in range(3):
            spread.addcmul_(*[torch.randn((n, d), generator=g, device="cuda")] * 2)
        block.mul_(spread.div_(3.0).clamp_(min=1e-6).rsqrt_()).mul_(gain).clamp_(-1.0e4, 1.0e4)
        x[r:r + n, :d] = block.to(torch.bfloat16)
        if pad:
            x[r:r + n, d:] = 7.0
    return x[:, :d]


def _calibrated(x, b):
    """The permutation of Algorithm 1 for these rows' channel means (host, int32)."""
    a = x[:2048].to(torch.float64).abs().mean(dim=0).to(torch.float32)
    return binding.perq_massdiff_perm(a.cpu().numpy(), b)


def _codes(rows, d, fmt, gen):
    """Quantized N(0, 1) rows: (codes uint8 [rows, d/2], scales) as the formats lay them out."""
    v = torch.randn((rows, d), generator=gen, device="cuda")
    if fmt == "int4":
        scales = v.abs().amax(dim=1) / 7.0
        q = torch.round(v / scales[:, None]).clamp_(-7, 7).to(torch.int32) & 15
    else:
        grid = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0], device="cuda")
        e = torch.floor(torch.log2(v.view(rows, d // 32, 32).abs().amax(dim=2).clamp_(min=1e-20))) - 2.0
        scales = (e + 127.0).clamp_(0, 254).to(torch.uint8)
        u = v.view(rows, d // 32, 32) / torch.exp2(e)[:, :, None]
        mag = torch.bucketize(u.abs().reshape(rows, d), (grid[1:] + grid[:-1]) / 2.0).to(torch.int32)
        q = mag + 8 * ((v < 0) & (mag > 0)).to(torch.int32)
    q = q.view(rows, d // 2, 2)
    return (q[:, :, 0] | (q[:, :, 1] << 4)).to(torch.uint8).contiguous(), scales.contiguous()


def prepare(case, seed):
    s = dict(case)
    if case["kind"] == "product":
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed) * 2654435761 % (1 << 62))
        s["a"] = _codes(case["T"], case["d"], case["fmt"], g)
        s["w"] = _codes(case["N"], case["d"], case["fmt"], g)
        return s
    s["x"] = _rows(case["T"], case["d"], case.get("pad", 0), seed)
    s["perm_dev"] = s["placement"] = None
    if case.get("perm", "none") != "none":
        perm = _calibrated(s["x"], case["b"])
        s["perm_dev"] = torch.from_numpy(perm).cuda()
        if case["perm"] == "prepared":
            s["placement"] = binding.placement_to_device(binding.perq_perm_prepare(perm, case["b"])[0])
    return s


def run(s):
    kind = s["kind"]
    if kind == "apply":
        return binding.perq_permute_rotate_quant(s["x"], s["perm_dev"], s["b"], s["fmt"], placement=s["placement"])
    if kind == "stat":
        return binding.perq_colabs_mean(s["x"]) if s["stat"] == "mean" else binding.perq_colabs_absmax(s["x"])
    if kind == "product":
        f = binding.perq_w4a4_gemm_ref if s["fmt"] == "int4" else binding.perq_w4a4_mxfp4_gemm_ref
        return f(*s["a"], *s["w"])
    y = binding.perq_permute_rotate_f32(s["x"], s["perm_dev"], s["b"])
    codes, scales = binding.perq_permute_rotate_quant(s["x"], s["perm_dev"], s["b"], s["fmt"])
    error = binding.perq_quant_error(y, codes, scales, s["fmt"])
    stats = binding.perq_block_diagnostics(s["x"], s["perm_dev"], s["b"])
    return y, codes, scales, error, stats


# ---- what a pass cannot do without ------------------------------------------------------------------
def _scale_bytes(rows, d, fmt):
    return rows * d // 32 if fmt == "mxfp4" else rows * (8 if fmt == "int4_asym" else 4)


def work(case):
    T, d, fmt = case["T"], case["d"], case.get("fmt")
    if case["kind"] == "stat":
        return {"bytes": 2 * T * d + 4 * d, "flops": T * d}
    if case["kind"] == "product":
        N = case["N"]
        return {"bytes": (T + N) * d // 2 + _scale_bytes(T + N, d, fmt) + 4 * T * N, "flops": 2 * T * N * d}
    size = 2 * T * d + T * d // 2 + _scale_bytes(T, d, fmt) + (4 * d if case["perm"] != "none" else 0)
    flops = T * d * (math.ceil(math.log2(case["b"])) + 4)
    if case["kind"] == "diagnose":
        size += 4 * T * d + (3 + 4) * 4 * T
        flops += 8 * T * d
    return {"bytes": size, "flops": flops}


def tolerance(case):
    # measured against exact(): floats up to 7e-8 (norm) and 3e-7 (largest), bytes up to 2.5e-6 of them
    if case["kind"] == "stat":
        # fp32 partial sums (the maximum is exact)
        return "exact" if case["stat"] == "absmax" else {"rel": 3e-7, "max": 2e-6}
    if case["kind"] == "product":
        # int4: exact integer sums and two roundings; mxfp4: fp32 sums of d exact products
        return {"rel": 3e-7, "max": 4e-6}
    # fp32 sums of up to b terms, then rounding to 4 bits: a sum in another order moves a value across
    # a rounding boundary now and then (two bytes of a small output)
    return {"rel": 3e-7, "max": 2e-6, "differ": max(1e-5, 2.0 / (case["T"] * case["d"] // 2))}


# ---- the same in 64 bits ----------------------------------------------------------------------------
def _base(m):
    """Paley's Hadamard matrix of order 12, 28 or 76 (type I over m - 1, else type II over m / 2 - 1)."""
    prime = all((m - 1) % k for k in range(2, int(math.sqrt(m)) + 1)) and (m - 1) % 4 == 3
    p = m - 1 if prime else m // 2 - 1
    squares = {i * i % p for i in range(1, p)}
    chi = np.array([0] + [1 if i in squares else -1 for i in range(1, p)])
    q = np.array([[chi[(i - j) % p] for j in range(p)] for i in range(p)])
    c = np.zeros((p + 1, p + 1), dtype=int)
    c[0, 1:], c[1:, 1:] = 1, q
    c[1:, 0] = -1 if prime else 1
    if prime:
        return c + np.eye(m, dtype=int)
    return np.kron(c, [[1, 1], [1, -1]]) + np.kron(np.eye(p + 1, dtype=int), [[1, -1], [-1, -1]])


def _rotated(x, perm, b):
    """fp64 [rows, d]: the rows permuted and every block of b rotated."""
    v = x.to(torch.float64)
    if perm is not None:
        v = v[:, perm.long()]
    rows, d = v.shape
    m = 1
    if b & (b - 1):
        t = b
        while t % 2 == 0:
            t //= 2
        m = 4 * t
        v = (v.reshape(-1, m) @ torch.from_numpy(_base(m)).to(v)).view(rows, d)
    h = m
    while h < b:
        v = v.view(-1, 2, h)
        v = torch.stack((v[:, 0] + v[:, 1], v[:, 0] - v[:, 1]), dim=1)
        h *= 2
    return v.view(rows, d) / math.sqrt(b)


def _e2m1(v):
    """Nearest e2m1 magnitude (ties to the even code, saturating), zero always +0: (value, nibble)."""
    a = v.abs()
    step = torch.where(a < 2.0, 0.5, torch.where(a < 4.0, 1.0, 2.0)).to(v)
    mag = (torch.round(a / step) * step).clamp_(max=6.0)
    code = torch.where(mag < 2.0, 2.0 * mag, torch.where(mag < 4.0, mag + 2.0, mag / 2.0 + 4.0)).to(torch.int32)
    return torch.where(v < 0, -mag, mag), code + 8 * ((v < 0) & (mag > 0)).to(torch.int32)


def _quantized(y, fmt):
    """fp64 y -> (codes uint8, scales, value the codes stand for)."""
    rows, d = y.shape
    if fmt == "mxfp4":
        g = y.view(rows, d // 32, 32)
        top = g.abs().amax(dim=2)
        e = (torch.frexp(top)[1] - 1 - 2 + 127).clamp_(0, 254)
        e = torch.where(top > 0, e, 0)
        unit = torch.exp2(e.to(y) - 127.0)[:, :, None]
        value, q = _e2m1(g / unit)
        value, q, scales = (value * unit).view(rows, d), q.view(rows, d), e.to(torch.uint8)
    elif fmt == "int4_asym":
        lo, hi = y.amin(dim=1, keepdim=True), y.amax(dim=1, keepdim=True)
        unit = (hi - lo) / 15.0
        safe = torch.where(unit > 0, unit, 1.0)
        zero = torch.where(unit > 0, torch.round(lo / safe), 0.0)
        c = torch.where(unit > 0, (torch.round(y / safe) - zero).clamp_(0, 15), 0.0)
        value, q, scales = unit * (c + zero), c.to(torch.int32), torch.cat((unit, zero), dim=1)
    else:
        unit = y.abs().amax(dim=1, keepdim=True) / {"int4": 7.0, "fp4_token": 6.0, "fp4_token7": 7.0}[fmt]
        u = y / torch.where(unit > 0, unit, 1.0)
        if fmt == "int4":
            c = torch.round(u).clamp_(-7, 7)
            value, q = unit * c, c.to(torch.int32) & 15
        else:
            c, q = _e2m1(u)
            value = unit * c
        scales = unit.view(rows)
    q = q.view(rows, d // 2, 2)
    return (q[:, :, 0] | (q[:, :, 1] << 4)).to(torch.uint8), scales, value


def _decoded(codes, scales, fmt):
    q = torch.stack((codes & 15, codes >> 4), dim=2).view(codes.shape[0], -1).long()
    if fmt == "int4":
        return ((q ^ 8) - 8).to(torch.float64) * scales.to(torch.float64)[:, None]
    grid = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]
    v = torch.tensor(grid + [-u for u in grid], dtype=torch.float64, device=codes.device)[q]
    return (v.view(v.shape[0], -1, 32) * torch.exp2(scales.to(torch.float64) - 127.0)[:, :, None]).view(v.shape)


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "product":
        return _decoded(*s["a"], s["fmt"]) @ _decoded(*s["w"], s["fmt"]).T
    x, step = s["x"], max(1, (1 << 26) // case["d"])
    parts = [x[r:r + step] for r in range(0, x.shape[0], step)]
    if case["kind"] == "stat":
        if case["stat"] == "absmax":
            return torch.stack([p.to(torch.float64).abs().amax(dim=0) for p in parts]).amax(dim=0)
        return sum(p.to(torch.float64).abs().sum(dim=0) for p in parts) / x.shape[0]
    got = []
    for p in parts:
        y = _rotated(p, s["perm_dev"], case["b"])
        codes, scales, value = _quantized(y, case["fmt"])
        if case["kind"] == "apply":
            got.append((codes, scales))
            continue
        v = p.to(torch.float64).abs()
        v = v if s["perm_dev"] is None else v[:, s["perm_dev"].long()]
        error = torch.stack(((y - value).norm(dim=1), y.norm(dim=1), y.abs().amax(dim=1)), dim=1)
        block = v.view(v.shape[0], -1, case["b"]).sum(dim=2).amax(dim=1)
        stats = torch.stack((v.amax(dim=1), v.sum(dim=1), block, y.abs().amax(dim=1)), dim=1)
        got.append((y, codes, scales, error, stats))
    return tuple(torch.cat(c) for c in zip(*got))
