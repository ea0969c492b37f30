"""HIP library vs CPU oracle, element by element, through the C ABI (needs an MI355X)."""
import math
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity  # noqa: E402
import prepared_form  # noqa: E402
from oracle import perq_oracle as orc  # noqa: E402
from paper_2601_22347_amd import binding, synth  # noqa: E402

pytestmark = pytest.mark.gpu

ALGOS = ["butterfly", "mfma", "auto"]


def mfma_covers(d, b):
    """Shapes the matrix-core kernel accepts; everything else must come back UNSUPPORTED."""
    return d % 512 == 0 and b <= 4096


def _torch():
    import torch
    return torch


def run_gpu(x_bits, perm, b, fmt, algo="auto", want_y=True, ldx=None):
    """One call of the fused path (+ the fp32 test entry) on cuda:0; NumPy results."""
    torch = _torch()
    T, d = x_bits.shape
    if ldx is None:
        x = binding.bits_to_device(x_bits)
    else:
        buf = torch.zeros((max(T, 1), ldx), dtype=torch.bfloat16, device="cuda")
        buf[:T, :d] = binding.bits_to_device(x_bits)
        x = buf[:T, :d]
    perm_t = None if perm is None else torch.from_numpy(np.ascontiguousarray(perm, dtype=np.int32)).cuda()
    codes, scales = binding.perq_permute_rotate_quant(x, perm_t, b, fmt, algo=algo)
    y = binding.perq_permute_rotate_f32(x, perm_t, b, algo=algo) if want_y else None
    torch.cuda.synchronize()
    return codes.cpu().numpy(), scales.cpu().numpy(), (None if y is None else y.cpu().numpy())


def assert_parity(x_bits, perm, b, fmt, algo="auto", rotate=None, ldx=None, label=""):
    print(f"[case] {label} T={x_bits.shape[0]} d={x_bits.shape[1]} b={b} fmt={fmt} algo={algo} "
          f"perm={'yes' if perm is not None else 'no'}", flush=True)
    if algo == "mfma" and not mfma_covers(x_bits.shape[1], b):
        with pytest.raises(binding.PerqError) as ei:
            run_gpu(x_bits, perm, b, fmt, algo=algo, ldx=ldx)
        assert ei.value.status == binding.PERQ_ERR_UNSUPPORTED
        return None
    codes, scales, y = run_gpu(x_bits, perm, b, fmt, algo=algo, ldx=ldx)
    rep = parity.compare_apply(x_bits, perm, b, fmt, codes, scales, y, rotate=rotate)
    print("       ", rep.summary(), flush=True)
    assert rep.ok(), (rep.summary(), rep.notes[:5])
    return rep


# ---- configs[0]: tiny, identity and greedy perm ------------------------------------------
@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_tiny_identity_and_greedy(fmt, algo):
    wl = synth.tiny()
    x = wl.apply_rows()
    assert_parity(x, None, 16, fmt, algo, label="tiny/identity")
    a = orc.colabs_mean(orc.bf16_bits_to_f64(wl.calib_rows())).astype(np.float32)
    perm = binding.perq_massdiff_perm(a, 16)
    assert_parity(x, perm, 16, fmt, algo, label="tiny/greedy")


# ---- structured inputs with closed-form answers --------------------------------------------
@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("d,b", [(256, 16), (256, 256), (1024, 64), (4096, 4096), (2048, 128)])
def test_structured_rows(d, b, algo):
    rng = np.random.default_rng(d + b)
    rows = []
    for pos in (0, b - 1, d - 1, d // 2 + 3):
        r = np.zeros(d); r[pos] = -3.5; rows.append(r)               # one-hot
    rows.append(np.ones(d) * 0.75)                                    # all equal
    rows.append(np.zeros(d))                                          # all zero
    base = rng.standard_normal(d)
    rows += [base, -base, base * 2.0 ** 10, base * 2.0 ** -10]        # sign flip, power-of-two scaling
    rows.append(np.where(np.arange(d) % 2 == 0, 1.0, -1.0))           # alternating signs
    x = synth.f64_to_bf16_bits(np.array(rows))
    if algo == "mfma" and not mfma_covers(d, b):
        pytest.skip("shape not covered by the matrix-core kernel")
    for fmt in ("int4", "mxfp4"):
        codes, scales, y = run_gpu(x, None, b, fmt, algo)
        rep = parity.compare_apply(x, None, b, fmt, codes, scales, y)
        assert rep.ok(), (rep.summary(), rep.notes[:5])
        # one-hot row: every output of the hit block has magnitude 3.5/sqrt(b), others are 0
        blk = y[0].reshape(d // b, b)
        assert np.allclose(np.abs(blk[0]), 3.5 / np.sqrt(b), rtol=1e-6) and np.all(blk[1:] == 0)
        # all-equal row: (0.75*sqrt(b), 0, ..., 0) per block; all-zero row: zeros and zero scale
        assert np.allclose(y[4].reshape(d // b, b)[:, 0], 0.75 * np.sqrt(b), rtol=1e-6)
        assert np.all(y[4].reshape(d // b, b)[:, 1:] == 0)
        assert np.all(codes[5] == 0) and np.all(scales[5] == 0)
        # sign flip negates INT4 codes; scaling by 2^k keeps the codes
        if fmt == "int4":
            c = parity.unpack_nibbles(codes).astype(np.int16); c = np.where(c >= 8, c - 16, c)
            assert np.array_equal(c[6], -c[7])
            assert np.array_equal(c[6], c[8]) and np.array_equal(c[6], c[9])
            assert scales[8] == scales[6] * 2.0 ** 10 and scales[9] == scales[6] * 2.0 ** -10
        else:
            assert np.array_equal(codes[6], codes[8]) and np.array_equal(codes[6], codes[9])
            assert np.array_equal(scales[8].astype(int), scales[6].astype(int) + 10)


# ---- shapes: several tiles, ragged tails, row strides, permutations -------------------------
SHAPES = [
    # (T, d, b list)
    (37, 256, [16, 32, 64, 128, 256]),
    (19, 1024, [16, 32, 256, 512, 1024]),
    (13, 3072, [16, 32, 64, 1024]),          # nt = 96: not a power of two
    (21, 2048, [32, 2048]),
    (24, 2048, [32, 128, 1024, 2048]),       # rows of d < 4096 stored back to back: several to a wave
    (40, 1024, [16, 64, 1024]),
    (64, 512, [32, 512]),
    (69, 512, [32, 512]),                    # rows left over: a wave that is not full
    (27, 2048, [32, 2048]),                  # (b >= 1024 with a permutation: a launch of its own for the last row)
    (9, 8192, [16, 32, 64, 128, 2048, 4096, 8192]),
    (5, 14336, [32, 128, 512, 1024, 2048]),
    (6, 20480, [256, 1024, 4096]),           # 8-wave groups, ragged last tile
    (3, 32768, [16, 2048, 4096, 32768]),
]


@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("T,d,bs", SHAPES)
def test_shapes_against_oracle(T, d, bs, algo):
    rng = np.random.default_rng(1000 + d)
    x = synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, d)) * np.exp(rng.uniform(-3, 3, size=(T, 1))))
    x[:, rng.choice(d, size=max(1, d // 100), replace=False)] = synth.f64_to_bf16_bits(
        rng.standard_normal((T, max(1, d // 100))) * 60)
    perm = rng.permutation(d).astype(np.int32)
    for b in bs:
        rotate = orc.fwht_f64 if b > 4096 else None
        for fmt in ("int4", "mxfp4"):
            assert_parity(x, None, b, fmt, algo, rotate=rotate, label="shape/identity")
            assert_parity(x, perm, b, fmt, algo, rotate=rotate, label="shape/perm")


@pytest.mark.parametrize("algo", ALGOS)
def test_row_stride_and_special_perms(algo):
    rng = np.random.default_rng(7)
    T, d = 11, 512
    x = synth.f64_to_bf16_bits(rng.standard_normal((T, d)))
    assert_parity(x, None, 32, "int4", algo, ldx=d + 64, label="ldx")
    assert_parity(x, np.arange(d, dtype=np.int32), 32, "int4", algo, label="identity-as-perm")
    assert_parity(x, np.arange(d, dtype=np.int32)[::-1].copy(), 64, "mxfp4", algo, ldx=d + 8, label="reverse")
    # a permutation followed by its inverse is the identity path on the un-permuted data
    perm = rng.permutation(d).astype(np.int32)
    if algo == "mfma" and not mfma_covers(d, 128):
        return
    xp = x[:, perm]
    c1, s1, y1 = run_gpu(xp, np.argsort(perm).astype(np.int32), 128, "int4", algo)
    c2, s2, y2 = run_gpu(x, None, 128, "int4", algo)
    assert np.array_equal(c1, c2) and np.array_equal(s1, s2) and np.array_equal(y1, y2)


def test_empty_and_single_row():
    torch = _torch()
    x = torch.zeros((0, 256), dtype=torch.bfloat16, device="cuda")
    codes, scales = binding.perq_permute_rotate_quant(x, None, 16, "int4")
    assert codes.shape == (0, 128) and scales.shape == (0,)
    bits = synth.f64_to_bf16_bits(np.random.default_rng(3).standard_normal((1, 4096)))
    assert_parity(bits, None, 128, "int4", label="single-row")
    assert_parity(bits, None, 32, "mxfp4", label="single-row")


def test_deterministic_across_launches():
    bits = synth.llama1b_down().apply_rows(0, 300)
    a = run_gpu(bits, None, 128, "int4", want_y=False)
    b_ = run_gpu(bits, None, 128, "int4", want_y=False)
    assert np.array_equal(a[0], b_[0]) and np.array_equal(a[1], b_[1])


# ---- reduced-T versions of configs[1..4]: every (d, b, fmt) the workloads name ---------------
def _calibrated_perm(wl, b):
    a = orc.colabs_mean(orc.bf16_bits_to_f64(wl.calib_rows())).astype(np.float32)
    return binding.perq_massdiff_perm(a, b)


@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("name", ["llama1b_down", "block_vs_full", "llama8b_d4096", "llama8b_d14336",
                                  "calib_apply"])
def test_workload_slices(name, algo):
    wl = synth.ALL[name]()
    rows = 160 if wl.d <= 8192 else 96
    x = wl.apply_rows(0, rows)
    if wl.massive_rows.size:                      # include a x200 row
        r = int(wl.massive_rows[0])
        x = np.concatenate([x, wl.apply_rows(r, r + 1)])
    for b in wl.block_sizes:
        perm = _calibrated_perm(wl, b) if wl.calib_tokens else None
        assert_parity(x, perm, b, wl.fmt, algo, label=name)


# ---- perq_colabs_mean ---------------------------------------------------------------------------
@pytest.mark.parametrize("M,d", [(256, 256), (2048, 8192), (4096, 8192), (1000, 14336), (3, 32)])
def test_colabs_mean(M, d):
    rng = np.random.default_rng(M + d)
    bits = synth.f64_to_bf16_bits(rng.standard_t(3, size=(M, d)))
    got = binding.perq_colabs_mean(binding.bits_to_device(bits))
    _torch().cuda.synchronize()
    got = got.cpu().numpy()
    want = orc.colabs_mean(orc.bf16_bits_to_f64(bits))
    # fp32 accumulation of non-negative terms, at most 32 rows per slice at these M, then a
    # reduction in double: relative error below 33 * 2^-24
    assert np.all(np.abs(got - want) <= 33 * 2.0**-24 * want + 1e-30)
    again = binding.perq_colabs_mean(binding.bits_to_device(bits)).cpu().numpy()
    assert np.array_equal(got, again)
    # constant-magnitude columns are exact
    const = synth.f64_to_bf16_bits(np.sign(rng.standard_normal((M, d))) * (1 + np.arange(d) % 7))
    got = binding.perq_colabs_mean(binding.bits_to_device(const)).cpu().numpy()
    assert np.array_equal(got, (1 + np.arange(d) % 7).astype(np.float32))


# ---- enough rows for the run-time schedule of the matrix-core kernels --------------------------
# With at least two units per worker (a workgroup; in mfma_kernel with d <= 4096 a wave) they deal their
# rows through ticket counters; every row is checked against the oracle, ragged tails included.
DYNAMIC_SHAPES = [
    # (T, d, b, fmt, perm)
    # block_kernel: two waves a row, one, four, eight
    (4099, 4096, 128, "int4", True),
    (4099, 4096, 32, "mxfp4", False),
    (4611, 2048, 64, "mxfp4", True),
    (8200, 2048, 64, "mxfp4", True),
    (8200, 2048, 2048, "mxfp4", False),
    (2051, 8192, 32, "mxfp4", True),
    (1030, 14336, 2048, "int4", False),
    # mfma_kernel
    (4500, 4096, 4096, "int4", True),     # a wave per row, shared address table
    (4500, 4096, 2048, "int4", True),
    (8201, 2048, 2048, "mxfp4", True),    # two rows folded into one tile, the last one by itself
    (2051, 8192, 4096, "mxfp4", True),    # two rows per workgroup
    (1030, 14336, 128, "int4", True),     # one row per workgroup, ragged last tile, row maximum across waves
    (530, 20480, 1024, "int4", True),     # eight-wave workgroups, one staging buffer
]


@pytest.mark.parametrize("T,d,b,fmt,with_perm", DYNAMIC_SHAPES)
def test_run_time_schedule_all_rows(T, d, b, fmt, with_perm):
    rng = np.random.default_rng(T + d + b)
    x = synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, d)) * np.exp(rng.uniform(-2, 2, size=(T, 1))))
    perm = rng.permutation(d).astype(np.int32) if with_perm else None
    print(f"[case] run-time schedule T={T} d={d} b={b} fmt={fmt} perm={with_perm}", flush=True)
    codes, scales, _ = run_gpu(x, perm, b, fmt, "mfma", want_y=False)
    rep = parity.compare_apply(x, perm, b, fmt, codes, scales, None)
    print("       ", rep.summary(), flush=True)
    assert rep.ok(), (rep.summary(), rep.notes[:5])


# (block_kernel, mfma_kernel with a wave and with a workgroup as worker)
@pytest.mark.parametrize("T,d,b", [(4200, 4096, 128), (4200, 4096, 2048), (1100, 14336, 128)])
def test_run_time_schedule_counters_come_back_to_zero(T, d, b):
    """Many launches in a row on one stream, i.e. on one set of ticket counters: a counter that a
    launch left non-zero would hand the next launch the wrong rows."""
    torch = _torch()
    print(f"[case] counters T={T} d={d} b={b}", flush=True)
    rng = np.random.default_rng(99)
    x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_normal((T, d))))
    perm = torch.from_numpy(rng.permutation(d).astype(np.int32)).cuda()
    ref = None
    for i in range(150):
        codes, scales = binding.perq_permute_rotate_quant(x, perm, b, "int4", algo="mfma")
        if ref is None:
            ref = (codes.clone(), scales.clone())
        elif i % 10 == 9 or i >= 140:
            assert torch.equal(codes, ref[0]) and torch.equal(scales, ref[1]), f"launch {i} differs"
    torch.cuda.synchronize()


def test_run_time_schedule_both_kernels_in_turn_on_one_stream():
    """block_kernel and mfma_kernel draw from the counters of their stream alike, with grids, workers and numbers of
    tickets of their own: every launch finds them at zero, whichever came before."""
    torch = _torch()
    rng = np.random.default_rng(98)
    calls = []
    for T, d, b, fmt, with_perm in ((4200, 4096, 128, "int4", True), (4300, 4096, 2048, "int4", True), (9000, 3072, 128, "int4_asym", True),
                                    (1100, 14336, 128, "mxfp4", True), (1500, 14336, 512, "fp4_token", False), (2100, 8192, 4096, "int4", True)):
        x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_normal((T, d))))
        perm = torch.from_numpy(rng.permutation(d).astype(np.int32)).cuda() if with_perm else None
        x3 = x[:3].contiguous()                    # (too few units to draw for)
        calls.append((x, perm, b, fmt, binding.perq_permute_rotate_quant(x, perm, b, fmt, algo="mfma")))
        few = binding.perq_permute_rotate_quant(x3, perm, b, fmt, algo="mfma")
        assert torch.equal(few[0], calls[-1][4][0][:3]) and torch.equal(few[1], calls[-1][4][1][:3])
    order = [int(k) for k in rng.integers(0, len(calls), size=120)]
    got = [binding.perq_permute_rotate_quant(*calls[k][:4], algo="mfma") for k in order]
    torch.cuda.synchronize()
    for i, k in enumerate(order):
        assert torch.equal(got[i][0], calls[k][4][0]) and torch.equal(got[i][1], calls[k][4][1]), f"launch {i}, call {k}"


# ---- the two per-token formats of Appendix B: asymmetric INT4, FP4 with a real scale -------------
TOKEN_FORMAT_SHAPES = [
    # (T, d, b list)
    (37, 256, [16, 64, 256]),
    (19, 1024, [32, 1024]),
    (13, 3072, [16, 1024]),
    (9, 4096, [128, 4096]),
    (7, 8192, [32, 2048, 8192]),
    (5, 14336, [128, 2048]),                 # ragged last tile: absent sub-blocks must not enter min / max
    (4, 20480, [256, 4096]),
    # narrow rows stored back to back, T a multiple of 4096 / d: several to a wave, the row extremes then exchanged inside 8 or 16
    # lanes of a half-wave pair (block_kernel), and rows of 2048 two to a 4096-wide one for b >= 1024 with a permutation (mfma_kernel)
    (24, 2048, [32, 128, 512, 1024, 2048]),
    (40, 1024, [16, 64, 256, 1024]),
    (64, 512, [32, 128, 512]),
    # the same with rows left over that do not fill the last wave, or 4096-wide row (a second launch)
    (25, 2048, [128, 2048]),
    (43, 1024, [64]),
    (67, 512, [32]),
]


@pytest.mark.parametrize("fmt", ["int4_asym", "fp4_token", "fp4_token7"])
@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("T,d,bs", TOKEN_FORMAT_SHAPES)
def test_token_formats_against_oracle(T, d, bs, algo, fmt):
    rng = np.random.default_rng(2000 + d)
    x = rng.standard_t(4, size=(T, d)) * np.exp(rng.uniform(-3, 3, size=(T, 1)))
    x[: T // 2] += 0.4 * np.exp(rng.uniform(-3, 3, size=(T // 2, 1)))         # off-centre rows
    x[-1] = np.abs(x[-1]) + 0.5                                                # an all-positive row
    x = synth.f64_to_bf16_bits(x)
    perm = rng.permutation(d).astype(np.int32)
    for b in bs:
        rotate = orc.fwht_f64 if b > 4096 else None
        assert_parity(x, None, b, fmt, algo, rotate=rotate, label="token-format/identity")
        assert_parity(x, perm, b, fmt, algo, rotate=rotate, label="token-format/perm")


@pytest.mark.parametrize("fmt", ["int4_asym", "fp4_token", "fp4_token7"])
def test_token_formats_structured_rows(fmt):
    d, b = 1024, 64
    rows = [np.zeros(d), np.full(d, 0.75), np.full(d, -2.0)]
    r = np.zeros(d); r[5] = 3.0; rows.append(r)
    r = np.zeros(d); r[700] = -1.5; rows.append(r)
    rows.append(np.where(np.arange(d) % 2 == 0, 1.0, -1.0))
    x = synth.f64_to_bf16_bits(np.array(rows))
    for algo in ALGOS:
        codes, scales, y = run_gpu(x, None, b, fmt, algo)
        rep = parity.compare_apply(x, None, b, fmt, codes, scales, y)
        assert rep.ok(), (algo, rep.summary(), rep.notes[:5])
        assert np.all(codes[0] == 0) and np.all(scales[0] == 0)              # all-zero row


@pytest.mark.parametrize("fmt,T,d,b,with_perm", [("int4_asym", 4099, 4096, 128, True), ("fp4_token", 4099, 4096, 128, True),
                                                  ("int4_asym", 1030, 14336, 128, False), ("fp4_token", 2051, 8192, 32, True)])
def test_token_formats_run_time_schedule(fmt, T, d, b, with_perm):
    rng = np.random.default_rng(T + d + b + 1)
    x = synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, d)) * np.exp(rng.uniform(-2, 2, size=(T, 1))) + 0.1)
    perm = rng.permutation(d).astype(np.int32) if with_perm else None
    codes, scales, _ = run_gpu(x, perm, b, fmt, "mfma", want_y=False)
    rep = parity.compare_apply(x, perm, b, fmt, codes, scales, None)
    print("       ", rep.summary(), flush=True)
    assert rep.ok(), (rep.summary(), rep.notes[:5])


# ---- asymmetric INT4 on rows that are a large offset plus a small spread ----------------------------
@pytest.mark.parametrize("d,b,algo", [(4096, 128, "mfma"), (4096, 4096, "mfma"), (14336, 2048, "mfma"),
                                      (1024, 64, "butterfly"), (3072, 768, "auto"), (8192, 8192, "auto")])
def test_int4_asym_offset_rows(d, b, algo):
    """One value at the head of every block and tiny values elsewhere: the rotated row is a constant
    plus a spread of a few fp32 steps to a few thousand, and the zero point reaches 10^7.  Against the
    oracle under the stated tolerance (which is wider than a step on such rows), and, as properties of
    the device's own fp32 outputs: every code decodes to within half a step (plus the fp32 rounding of
    the offset) of its value, the row minimum has code 0 and the maximum 14 or 15."""
    rng = np.random.default_rng(d + b)
    T = 48
    x = np.zeros((T, d))
    eps = 2.0 ** -rng.integers(14, 23, size=(T, 1)).astype(np.float64)          # spread from coarse to a few steps
    x[:] = eps * rng.standard_normal((T, d))
    if b & (b - 1) == 0:
        x[:, ::b] = 16.0 * np.where(rng.random((T, 1)) < 0.5, -1.0, 1.0)
    else:
        x[:, ::b] = 16.0                                                        # (first row of a Paley base: all ones)
    x[T - 1] = 0.0
    x[T - 1, ::b] = 16.0                                                        # exactly constant after the rotation
    x_bits = synth.f64_to_bf16_bits(x)
    print(f"[case] int4_asym offset rows d={d} b={b} algo={algo}", flush=True)
    codes, scales, y = run_gpu(x_bits, None, b, "int4_asym", algo)
    rep = parity.compare_apply(x_bits, None, b, "int4_asym", codes, scales, y)
    print("       ", rep.summary(), flush=True)
    assert rep.ok(), (rep.summary(), rep.notes[:5])
    c = parity.unpack_nibbles(codes).astype(np.float64)
    s, z = scales[:, 0].astype(np.float64), scales[:, 1].astype(np.float64)
    y = y.astype(np.float64)
    lo, hi = y.min(axis=1), y.max(axis=1)
    assert np.all(np.abs(z[:-1]) > 1e3) and np.all(np.abs(z) < 2.0 ** 28) and np.all(z == np.rint(z))
    exact_z = np.abs(z) < 2.0 ** 24                # (a zero point is handed over as a float: exact up to 2^24)
    assert exact_z.sum() >= T // 2
    # (the fp32 test output is the kernel's value times fl(1/sqrt(b)), rounded once more: each end of
    #  the row carries up to a step of the offset's fp32 grid)
    assert np.all(np.abs(s - (hi - lo) / 15.0) <= 1e-5 * s + 4.0 * 2.0 ** -24 * np.abs(y).max(axis=1) / 15.0)
    dq = s[:, None] * (c + z[:, None])
    slack = 0.5 * s[:, None] * (1 + 1e-3) + 6.0 * 2.0 ** -24 * np.abs(y)
    worst = (np.abs(dq - y) - slack).max(axis=1)
    worst[T - 1] = 0.0                                       # (the constant row has no step: nothing decodes)
    worst[~exact_z] = 0.0
    assert np.all(worst <= 0), (int(np.argmax(worst)), float(worst.max()), float(s[np.argmax(worst)]))
    rows = np.arange(T - 1)
    assert np.all(c[rows, y[:-1].argmin(axis=1)] == 0) and np.all(c[rows, y[:-1].argmax(axis=1)] >= 14)
    assert np.all(c[T - 1] == 0) and s[T - 1] == 0 and z[T - 1] == 0            # constant row


# ---- fp32 output: stored by quads of lanes; rows of fewer than four lanes, of a multiple and not ------
@pytest.mark.parametrize("d,b", [(32, 32), (64, 16), (96, 32), (128, 64), (160, 32), (352, 32), (512, 256), (1536, 512),
                                 (4096, 128), (4608, 512), (8192, 4096), (14336, 2048), (10240, 1024)])
@pytest.mark.parametrize("algo", ["butterfly", "mfma"])
def test_f32_output_fills_its_rows_and_nothing_else(d, b, algo):
    torch = _torch()
    if algo == "mfma" and not mfma_covers(d, b):
        return
    print(f"[case] f32 rows d={d} b={b} algo={algo}", flush=True)
    rng = np.random.default_rng(d + b)
    for T in (1, 5):
        x_bits = synth.f64_to_bf16_bits(rng.standard_normal((T, d)))
        perm = rng.permutation(d).astype(np.int32)
        buf = torch.full((T * d + 64,), 7.5, device="cuda")
        binding.perq_permute_rotate_f32(binding.bits_to_device(x_bits), torch.from_numpy(perm).cuda(), b,
                                        y=buf[:T * d].view(T, d), algo=algo)
        X = orc.bf16_bits_to_f64(x_bits)
        want = orc.block_hadamard(orc.permute_channels(X, perm), b)
        got = buf[:T * d].view(T, d).cpu().numpy().astype(np.float64)
        # log2(b) + 1 fp32 roundings of values no larger than the row's l1 norm over sqrt(b)
        assert np.all(np.abs(got - want) <= 1e-5 * np.linalg.norm(X, axis=1, keepdims=True))
        assert bool((buf[T * d:] == 7.5).all())


# ---- the line between the two general kernels: calls on either side of it -------------------------
@pytest.mark.parametrize("d,b,rows,with_perm", [(3072, 64, 1366, False), (2560, 512, 1639, False), (3584, 16, 2341, False),
                                                (3072, 128, 2731, True), (4096, 128, 1024, False), (4096, 64, 513, True),
                                                (8192, 128, 1024, True), (6144, 2048, 342, True), (5120, 1024, 1639, False),
                                                (10240, 64, 410, True), (5120, 32, 3277, True), (5120, 32, 4916, False),
                                                (5120, 32, 4916, True), (7168, 16, 2341, True),
                                                (8192, 256, 1536, False), (512, 128, 4352, True), (2048, 64, 8192, False),
                                                (1024, 128, 6144, False), (1024, 512, 2056, True)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4", "int4_asym"])
def test_few_rows_and_many_take_either_kernel(d, b, rows, with_perm, fmt):
    rng = np.random.default_rng(d + b + rows)
    x_bits = synth.f64_to_bf16_bits(rng.standard_t(4, size=(rows, d)))
    perm = rng.permutation(d).astype(np.int32) if with_perm else None
    for T in (rows - 1, rows):          # (strided rows are not folded)
        assert_parity(x_bits[:T], perm, b, fmt, ldx=d + 24 if T == rows and d >= 2560 else None, label="few or many rows")
    if with_perm and d >= 4096:          # the prepared form goes where the plain call goes
        torch = _torch()
        pt, place = torch.from_numpy(perm).cuda(), binding.placement_to_device(binding.perq_perm_prepare(perm, b)[0])
        for T in (rows - 1, rows):
            x = binding.bits_to_device(x_bits[:T])
            for p, q in zip(binding.perq_permute_rotate_quant(x, pt, b, fmt),
                            binding.perq_permute_rotate_quant(x, pt, b, fmt, placement=place)):
                assert torch.equal(p, q)


# the lines of rows of three tiles and more
@pytest.mark.parametrize("d,b,rows,with_perm", [(12288, 1024, 257, True), (14336, 128, 513, True), (9728, 64, 513, True), (9728, 16, 513, True),
                                                (12288, 16, 1025, True), (14336, 256, 513, False), (16384, 64, 768, False), (9728, 32, 863, False),
                                                (22528, 2048, 513, False), (28672, 64, 257, False), (20480, 4096, 257, False), (25600, 32, 656, False),
                                                (17920, 64, 257, True), (24576, 32, 513, True), (20480, 1024, 3, True), (25600, 16, 3, True)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_few_wide_rows_and_many_take_either_kernel(d, b, rows, with_perm, fmt):
    test_few_rows_and_many_take_either_kernel(d, b, rows, with_perm, fmt)


# ---- a kernel chosen by the caller: a row's bits do not depend on how many rows come with it ------------
@pytest.mark.parametrize("d,b", [(1024, 64), (2048, 2048), (3072, 32), (4096, 128), (4096, 4096), (8192, 32), (14336, 512), (20480, 16)])
@pytest.mark.parametrize("algo", ["butterfly", "mfma"])
def test_rows_alone_and_among_others(d, b, algo):
    torch = _torch()
    rng = np.random.default_rng(d + b)
    few = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_t(4, size=(67, d))))
    many = few.repeat((1 << 24) // d // 67 + 2, 1)
    for perm in (None, torch.from_numpy(rng.permutation(d).astype(np.int32)).cuda()):
        print(f"[case] few and many rows d={d} b={b} algo={algo}", flush=True)
        for fmt in ("int4", "mxfp4", "int4_asym", "fp4_token"):
            want = binding.perq_permute_rotate_quant(many, perm, b, fmt, algo=algo)
            for T in (1, 7, 67):
                for got, full in zip(binding.perq_permute_rotate_quant(few[:T], perm, b, fmt, algo=algo), want):
                    assert torch.equal(got, full[:T]) and torch.equal(got, full[67:67 + T]), (T, fmt)
        y = binding.perq_permute_rotate_f32(many, perm, b, algo=algo)
        assert torch.equal(binding.perq_permute_rotate_f32(few, perm, b, algo=algo), y[:67])


# ---- rows that are no multiple of a load instruction: staged at a pitch of whole instructions ----------
# AUTO takes the matrix-core kernel for every such width from 2^26 elements on.  The rows repeat with a
# period of 32, and a row's output does not depend on its place: the first 32 go to the oracle, the others
# have to equal them bit for bit.
@pytest.mark.parametrize("d,b,with_perm", [
    # (block_kernel up to b = 64, mfma_kernel above)
    (2592, 32, True), (2880, 64, True), (2880, 32, False), (3040, 16, True), (3552, 32, True),   # two waves a row
    (5152, 32, True), (7648, 16, False), (7424, 256, True),                                       # three and four; two rows a group
    (11008, 256, True), (11008, 64, False), (15904, 32, True),                                    # one row of four tiles; six and eight
    (17440, 32, True), (28800, 128, True), (31776, 16, True),                                     # nine to sixteen; eight waves
    (4064, 32, True), (8160, 32, True), (16352, 16, False), (32736, 32, True)])                   # no room for the zeros: butterflies
@pytest.mark.parametrize("fmt", ["int4", "mxfp4", "int4_asym", "fp4_token"])
def test_ragged_rows_in_bulk(d, b, with_perm, fmt):
    torch = _torch()
    rng = np.random.default_rng(d + b)
    few = synth.f64_to_bf16_bits(rng.standard_t(4, size=(32, d)))
    T = (1 << 26) // d + 3
    perm = rng.permutation(d).astype(np.int32) if with_perm else None
    pt = None if perm is None else torch.from_numpy(perm).cuda()
    x = torch.zeros((T, d + 8), dtype=torch.bfloat16, device="cuda")[:, :d]
    x.copy_(binding.bits_to_device(few).repeat(T // 32 + 1, 1)[:T])
    print(f"[case] ragged rows T={T} d={d} b={b} fmt={fmt} perm={with_perm}", flush=True)
    codes, scales = binding.perq_permute_rotate_quant(x, pt, b, fmt)
    y = binding.perq_permute_rotate_f32(x, pt, b)
    for out in (codes, scales, y):
        assert torch.equal(out, out[:32].repeat(T // 32 + 1, *[1] * (out.dim() - 1))[:T])
    rep = parity.compare_apply(few, perm, b, fmt, codes[:32].cpu().numpy(), scales[:32].cpu().numpy(), y[:32].cpu().numpy())
    assert rep.ok(), (rep.summary(), rep.notes[:5])


# ---- the codes consumed: W4A4 product with P and the rotation merged into the weights -----------
@pytest.mark.parametrize("T,N,d,b", [(70, 50, 256, 32), (33, 130, 4096, 128), (5, 3, 1024, 1024),
                                     # rotations that are not symmetric matrices (base 12) or not powers of two
                                     (20, 24, 3072, 3072), (9, 17, 3584, 896), (6, 5, 2432, 2432),
                                     (7, 9, 8192, 8192)])
def test_w4a4_gemm_against_oracle_and_unrotated_product(T, N, d, b):
    torch = _torch()
    rng = np.random.default_rng(T + N + d)
    x_bits = synth.f64_to_bf16_bits(rng.standard_t(5, size=(T, d)))
    wt_bits = synth.f64_to_bf16_bits(rng.standard_normal((N, d)) * 0.05)        # rows of W^T
    perm = rng.permutation(d).astype(np.int32)
    perm_t = torch.from_numpy(perm).cuda()
    xa, wa = binding.bits_to_device(x_bits), binding.bits_to_device(wt_bits)
    ca, sa = binding.perq_permute_rotate_quant(xa, perm_t, b, "int4")
    cw, sw = binding.perq_permute_rotate_quant(wa, perm_t, b, "int4")
    out = binding.perq_w4a4_gemm_ref(ca, sa, cw, sw).cpu().numpy().astype(np.float64)
    # (1) the integer product itself, on operands that the oracle quantized: its codes and scales go
    # to the device, the library's product of them must equal the oracle's (exact sums, two fp32
    # multiplications)
    rot = orc.fwht_f64 if (b > 4096 and b & (b - 1) == 0) else orc.block_hadamard
    ra, rw = orc.perq_apply(x_bits, perm, b, "int4", rotate=rot), orc.perq_apply(wt_bits, perm, b, "int4", rotate=rot)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = binding.perq_w4a4_gemm_ref(dev(ra["packed"]), dev(ra["scales"]), dev(rw["packed"]), dev(rw["scales"]))
    acc, want = orc.w4a4_matmul(ra["codes"], ra["scales"], rw["codes"], rw["scales"])
    got = got.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - want) <= 4e-7 * np.abs(want) + 1e-30)
    # (2) it stands for X W: within the two operands' INT4 error bounds of the unrotated product
    X, Wt = orc.bf16_bits_to_f64(x_bits), orc.bf16_bits_to_f64(wt_bits)
    s_a, s_w = sa.cpu().numpy().astype(np.float64), sw.cpu().numpy().astype(np.float64)
    ey, ew = np.sqrt(d) * s_a / 2, np.sqrt(d) * s_w / 2
    ny, nw = np.linalg.norm(X, axis=1), np.linalg.norm(Wt, axis=1)
    bound = ey[:, None] * nw[None, :] + ny[:, None] * ew[None, :] + ey[:, None] * ew[None, :]
    assert np.all(np.abs(out - X @ Wt.T) <= bound * (1 + 1e-4))
    # (3) and the rotation really cancels: pre-quantization outputs of both sides multiply to X W
    y = binding.perq_permute_rotate_f32(xa, perm_t, b).cpu().numpy().astype(np.float64)
    wy = binding.perq_permute_rotate_f32(wa, perm_t, b).cpu().numpy().astype(np.float64)
    ref = X @ Wt.T
    assert np.all(np.abs(y @ wy.T - ref) <= 1e-5 * ny[:, None] * nw[None, :] * 2)


@pytest.mark.parametrize("T,N,d,b", [(70, 50, 256, 32), (33, 130, 4096, 128), (5, 3, 1024, 1024), (9, 40, 3584, 896),
                                     (37, 33, 96, 32)])
def test_w4a4_mxfp4_gemm_on_the_scaled_matrix_unit(T, N, d, b):
    """The packed MXFP4 output (codes and scale bytes) goes into gfx950's scaled fp4 matrix instruction
    as it is; the product equals the oracle's product of the decoded operands."""
    torch = _torch()
    rng = np.random.default_rng(T * 7 + N + d)
    x_bits = synth.f64_to_bf16_bits(rng.standard_t(5, size=(T, d)) * np.exp(rng.uniform(-6, 6, size=(T, 1))))
    wt_bits = synth.f64_to_bf16_bits(rng.standard_normal((N, d)) * 0.05)        # rows of W^T
    perm = rng.permutation(d).astype(np.int32)
    # (1) the product itself, on operands that the oracle quantized
    ra, rw = orc.perq_apply(x_bits, perm, b, "mxfp4"), orc.perq_apply(wt_bits, perm, b, "mxfp4")
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = binding.perq_w4a4_mxfp4_gemm_ref(dev(ra["packed"]), dev(ra["scales"]), dev(rw["packed"]), dev(rw["scales"]))
    got = got.cpu().numpy().astype(np.float64)
    want = orc.w4a4_mxfp4_matmul(ra["codes"], ra["scales"], rw["codes"], rw["scales"])
    da, dw = np.abs(orc.dequant_mxfp4(ra["codes"], ra["scales"])), np.abs(orc.dequant_mxfp4(rw["codes"], rw["scales"]))
    # exact products, fp32 sums in the unit's own order: d rounding errors of 2^-24 on the sum of magnitudes
    assert np.all(np.abs(got - want) <= d * 2.0 ** -24 * (da @ dw.T) + 1e-37)
    # (2) end to end on the library's own output: it stands for X W within the format's error
    xa, wa = binding.bits_to_device(x_bits), binding.bits_to_device(wt_bits)
    perm_t = torch.from_numpy(perm).cuda()
    ca, sa = binding.perq_permute_rotate_quant(xa, perm_t, b, "mxfp4")
    cw, sw = binding.perq_permute_rotate_quant(wa, perm_t, b, "mxfp4")
    out = binding.perq_w4a4_mxfp4_gemm_ref(ca, sa, cw, sw).cpu().numpy().astype(np.float64)
    X, Wt = orc.bf16_bits_to_f64(x_bits), orc.bf16_bits_to_f64(wt_bits)
    # an element is off by at most a quarter of its group's maximum (half a step of the coarsest e2m1
    # interval), so each operand keeps most of its norm; a loose bound is enough to catch a wrong layout
    ny, nw = np.linalg.norm(X, axis=1), np.linalg.norm(Wt, axis=1)
    assert np.all(np.abs(out - X @ Wt.T) <= 0.6 * ny[:, None] * nw[None, :])
    assert np.corrcoef(out.ravel(), (X @ Wt.T).ravel())[0, 1] > 0.97


# every branch of the products' choice of tile, each at ragged edges of rows, columns and contraction
# (rows of a superstage of 1024 codes or less never reach the loop over whole superstages: every tile shape that
# runs it is here with several of them, with rows that end there and rows that go on for one, two or four stages)
@pytest.mark.parametrize("T,N,d", [(1, 1, 32), (3, 70, 96), (515, 700, 64), (515, 700, 96), (515, 700, 128),     # one wave per tile
                                   (33, 70, 128), (5, 3, 1056), (64, 130, 4096),      # few tiles: contraction cut among waves
                                   (31, 65, 8224),                                    # the same sizes, long rows
                                   (513, 700, 1024), (449, 577, 2880), (449, 577, 4096),                # 64 x 64 tiles
                                   (1540, 1537, 1312), (1700, 1300, 544), (1540, 1537, 2880), (1540, 1537, 3328), (1540, 1537, 4096),  # 128 x 128
                                   (2177, 2177, 416), (2177, 2177, 2016), (2060, 2177, 2080),      # 128 x 128 twice a CU; 128 x 256
                                   (2060, 2177, 2880), (2060, 2177, 3328), (2060, 2177, 4096),
                                   (2060, 2177, 5152), (2060, 2177, 6016), (2060, 2177, 6144), (2690, 3330, 2912)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_w4a4_products_over_tiles_and_remainders(T, N, d, fmt):
    torch = _torch()
    print(f"[case] product {fmt} T={T} N={N} d={d}", flush=True)
    rng = np.random.default_rng(T + 3 * N + d)
    codes = lambda n: rng.integers(0, 256, size=(n, d // 2), dtype=np.uint8)           # all sixteen codes, -8 among them
    nib = lambda c: np.stack([c & 15, c >> 4], axis=2).reshape(c.shape[0], d)
    ca, cw = codes(T), codes(N)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = torch.full((T, N + 3), 7.5, device="cuda")                                  # rows further apart than they are wide
    if fmt == "int4":
        sa, sw = (rng.uniform(0.01, 2.0, size=n).astype(np.float32) for n in (T, N))
        binding.perq_w4a4_gemm_ref(dev(ca), dev(sa), dev(cw), dev(sw), out=out[:, :N])
        val = lambda c: ((nib(c).astype(np.int64) ^ 8) - 8).astype(np.float64)
        acc = val(ca) @ val(cw).T                                                     # exact: below 2^53
        want = (acc.astype(np.float32) * sa[:, None] * sw[None, :]).astype(np.float32)  # (the sums are below 2^24)
        assert np.array_equal(out[:, :N].cpu().numpy(), want)
    else:
        ea, ew = (rng.integers(110, 140, size=(n, d // 32), dtype=np.uint8) for n in (T, N))
        binding.perq_w4a4_mxfp4_gemm_ref(dev(ca), dev(ea), dev(cw), dev(ew), out=out[:, :N])
        a, w = orc.dequant_mxfp4(nib(ca), ea), orc.dequant_mxfp4(nib(cw), ew)
        got = out[:, :N].cpu().numpy().astype(np.float64)
        # exact products; d fp32 additions, each off by at most 2^-24 of the sum of magnitudes
        assert np.all(np.abs(got - a @ w.T) <= d * 2.0 ** -24 * (np.abs(a) @ np.abs(w).T))
    assert bool((out[:, N:] == 7.5).all())


# few tiles: four and eight waves, one row of tiles and several, rows of one stage, of stages that the waves share unevenly, cut rows
@pytest.mark.parametrize("T,N,d", [(1, 33, 160), (32, 16500, 288), (32, 16500, 4128), (17, 9000, 2336), (130, 3300, 2080), (130, 3300, 4096),
                                   (64, 2048, 2304), (33, 100, 2048), (300, 1500, 1088)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_w4a4_products_of_few_tiles(T, N, d, fmt):
    test_w4a4_products_over_tiles_and_remainders(T, N, d, fmt)


# one row of tiles on either side of the line (MXFP4), three and four of them to a CU (INT4), tiles that columns fill in part
@pytest.mark.parametrize("T,N,d", [(32, 8224, 3200), (32, 8224, 3616), (32, 8224, 3552), (130, 4900, 2080), (96, 8320, 2080), (33000, 120, 1056)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_w4a4_products_where_the_choice_changes(T, N, d, fmt):
    test_w4a4_products_over_tiles_and_remainders(T, N, d, fmt)


# MXFP4 rows of less than a superstage: one stage to four, whole ones and cut ones, several rounds of tiles; the last one is not
@pytest.mark.parametrize("T,N,d", [(2700, 3330, 160), (2700, 3330, 256), (1540, 1537, 288), (2700, 3330, 512), (1540, 1537, 544), (1540, 1537, 768),
                                   (2700, 3330, 992), (1540, 1537, 992), (1540, 1537, 1024)])
def test_w4a4_mxfp4_products_of_short_rows(T, N, d):
    test_w4a4_products_over_tiles_and_remainders(T, N, d, "mxfp4")
    test_w4a4_products_repeat_bit_for_bit(T, N, d, "mxfp4")


# ---- rows that end in several stages of a partial superstage: the waits count the loads that are there ----
@pytest.mark.parametrize("T,N,d", [(449, 577, 2880), (513, 700, 1312), (1540, 1537, 800), (2177, 2177, 2016),
                                   (1540, 1537, 2880), (1540, 1537, 4096), (2060, 2177, 2880), (2060, 2177, 4096),
                                   (2060, 2177, 6016), (2060, 2177, 6144)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_w4a4_products_repeat_bit_for_bit(T, N, d, fmt):
    torch = _torch()
    g = torch.Generator(device="cuda").manual_seed(T + d)
    ca, cw = (torch.randint(0, 256, (n, d // 2), dtype=torch.uint8, device="cuda", generator=g) for n in (T, N))
    if fmt == "int4":
        sa, sw = (torch.rand(n, device="cuda", generator=g) + 0.1 for n in (T, N))
        call = binding.perq_w4a4_gemm_ref
    else:
        sa, sw = (torch.randint(120, 131, (n, d // 32), dtype=torch.uint8, device="cuda", generator=g) for n in (T, N))
        call = binding.perq_w4a4_mxfp4_gemm_ref
    first = call(ca, sa, cw, sw)
    flush = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
    for k in range(50):
        flush.fill_(k)                  # twice the last-level cache: the operands come from memory
        assert torch.equal(call(ca, sa, cw, sw), first)


@pytest.mark.parametrize("T,N,d", [(300, 640, 1152), (300, 640, 2944), (1024, 1408, 1024), (1024, 1408, 4224), (2176, 2304, 2176),
                                   (2176, 2304, 3072)])
def test_w4a4_mxfp4_scale_bytes_at_any_address(T, N, d):
    """Scale bytes at an odd address go through registers, at a dword into LDS directly: the same sums, bit for bit.
    Output rows of whole 128-byte lines and others are stored differently: the same values."""
    torch = _torch()
    print(f"[case] scale bytes T={T} N={N} d={d}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d)
    ca, cw = (torch.randint(0, 256, (n, d // 2), dtype=torch.uint8, device="cuda", generator=g) for n in (T, N))
    ea, ew = (torch.randint(110, 140, (n, d // 32), dtype=torch.uint8, device="cuda", generator=g) for n in (T, N))
    want = binding.perq_w4a4_mxfp4_gemm_ref(ca, ea, cw, ew)

    def at(t, shift):
        room = torch.zeros(t.numel() + 16, dtype=torch.uint8, device="cuda")
        room[shift:shift + t.numel()] = t.flatten()
        return room[shift:shift + t.numel()].view(t.shape)
    for sa, sw in ((1, 0), (0, 2), (3, 3), (4, 8)):
        assert torch.equal(binding.perq_w4a4_mxfp4_gemm_ref(ca, at(ea, sa), cw, at(ew, sw)), want)
    out = torch.full((T, N + 5), 7.5, device="cuda")
    binding.perq_w4a4_mxfp4_gemm_ref(ca, ea, cw, ew, out=out[:, :N])
    assert torch.equal(out[:, :N], want) and bool((out[:, N:] == 7.5).all())
    a, w = (orc.dequant_mxfp4(np.stack([c & 15, c >> 4], axis=2).reshape(len(c), d), e)
            for c, e in ((ca[:64].cpu().numpy(), ea[:64].cpu().numpy()), (cw.cpu().numpy(), ew.cpu().numpy())))
    # exact products; d fp32 additions, each off by at most 2^-24 of the sum of magnitudes
    assert np.all(np.abs(want[:64].cpu().numpy().astype(np.float64) - a @ w.T) <= d * 2.0 ** -24 * (np.abs(a) @ np.abs(w).T))


@pytest.mark.parametrize("d,b", [(64, 16), (512, 32), (1024, 512), (2048, 64), (4096, 128), (4096, 4096)])
@pytest.mark.parametrize("perm", [False, True])
def test_butterflies_few_rows_to_a_workgroup(d, b, perm):
    """How many rows a workgroup of the butterflies takes follows from T; a row's bits do not."""
    torch = _torch()
    g = torch.Generator(device="cuda").manual_seed(d + b)
    x = torch.randn((3000, d), device="cuda", generator=g).to(torch.bfloat16)
    pt = torch.randperm(d, device="cuda", generator=g).to(torch.int32) if perm else None
    call = lambda v, fmt: binding.perq_permute_rotate_quant(v, pt, b, fmt, algo="butterfly")
    want = {fmt: call(x, fmt) for fmt in ("int4", "mxfp4", "int4_asym")}
    y, st = binding.perq_permute_rotate_f32(x, pt, b, algo="butterfly"), binding.perq_block_diagnostics(x, pt, b)
    for T in (1, 2, 3, 127, 255, 256, 257, 511, 513, 1021, 2049):
        print(f"[case] butterflies T={T} d={d} b={b}", flush=True)
        for fmt, (codes, scales) in want.items():
            c, s = call(x[:T], fmt)
            assert torch.equal(c, codes[:T]) and torch.equal(s, scales[:T])
        assert torch.equal(binding.perq_permute_rotate_f32(x[:T], pt, b, algo="butterfly"), y[:T])
        assert torch.equal(binding.perq_block_diagnostics(x[:T], pt, b), st[:T])


# one launch (2, 3, 17, 32, 33, 40, 48 slices of rows) and two (41, 49, 64, 65), one tile of columns, a cut one and as many as fit
@pytest.mark.parametrize("M,d", [(129, 256), (192, 8), (1088, 520), (2048, 512), (2049, 504), (2560, 520), (2561, 520), (3072, 1544), (3073, 1544),
                                 (4096, 512), (4097, 512), (300, 32768), (300, 32776), (4000, 4104), (2200, 3840)])
@pytest.mark.parametrize("stat", ["mean", "absmax"])
def test_column_statistics_in_one_launch(M, d, stat):
    """Against 64 bits; every call gives the same bits, with other streams' calls beside it and replayed from a graph
    (which takes two launches) too."""
    torch = _torch()
    print(f"[case] column {stat} M={M} d={d}", flush=True)
    call = binding.perq_colabs_mean if stat == "mean" else binding.perq_colabs_absmax
    g = torch.Generator(device="cuda").manual_seed(M + d)
    xs = [torch.randn((M, d), device="cuda", generator=g).to(torch.bfloat16) for _ in range(3)]
    want = [call(x) for x in xs]
    for x, w in zip(xs, want):
        v = x.double().abs()
        ref = v.mean(dim=0) if stat == "mean" else v.amax(dim=0)
        r = max(8, -(-M // max(1, 512 // -(-d // 2048))))                 # terms of an fp32 sum, as documented
        assert bool(((w.double() - ref).abs() <= (0.0 if stat == "absmax" else (r + 1) * 2.0 ** -24) * ref).all())
    streams = [torch.cuda.Stream() for _ in xs]
    torch.cuda.synchronize()
    for _ in range(20):
        got = []
        for s, x in zip(streams, xs):
            with torch.cuda.stream(s):
                got.append(call(x))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call(xs[0])
    for _ in range(3):
        out.zero_()
        graph.replay()
        call(xs[1])
        torch.cuda.synchronize()
        assert torch.equal(out, want[0])


def test_buffers_of_a_call_belong_to_its_stream():
    """With stream=, outputs and workspaces are blocks of that stream, and of the current one where it is not given:
    a workspace ends with the call, and a block of another stream could be handed out again while the call still runs."""
    torch = _torch()
    x = torch.randn((4096, 2048), device="cuda").to(torch.bfloat16)
    want = [binding.perq_colabs_mean(x), binding.perq_colabs_absmax(x), *binding.perq_permute_rotate_quant(x, None, 128, "int4"),
            binding.perq_permute_rotate_f32(x, None, 128), binding.perq_block_diagnostics(x, None, 128)]
    codes, scales, y = want[2], want[3], want[4]
    want += [binding.perq_quant_error(y, codes, scales, "int4"), binding.perq_w4a4_gemm_ref(codes[:300], scales[:300], codes[:400], scales[:400])]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for st in (side, None, torch.cuda.current_stream()):
        torch.cuda.memory._record_memory_history("all", context=None, max_entries=10000, clear_history=True)
        try:
            got = [binding.perq_colabs_mean(x, stream=st), binding.perq_colabs_absmax(x, stream=st),
                   *binding.perq_permute_rotate_quant(x, None, 128, "int4", stream=st),
                   binding.perq_permute_rotate_f32(x, None, 128, stream=st), binding.perq_block_diagnostics(x, None, 128, stream=st),
                   binding.perq_quant_error(y, codes, scales, "int4", stream=st),
                   binding.perq_w4a4_gemm_ref(codes[:300], scales[:300], codes[:400], scales[:400], stream=st)]
            trace = torch.cuda.memory._snapshot()["device_traces"][torch.cuda.current_device()]
        finally:
            torch.cuda.memory._record_memory_history(None)
        allocs = [e["stream"] for e in trace if e["action"] == "alloc"]
        assert len(allocs) == len(got) + 2                                           # two workspaces
        assert set(allocs) == {(st or torch.cuda.current_stream()).cuda_stream}
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_w4a4_gemm_argument_checks():
    torch = _torch()
    a = torch.zeros((4, 16), dtype=torch.uint8, device="cuda")
    s = torch.ones(4, device="cuda")
    out = binding.perq_w4a4_gemm_ref(a, s, a[:0], s[:0])
    assert out.shape == (4, 0)
    with pytest.raises(ValueError):
        binding.perq_w4a4_gemm_ref(a, s, torch.zeros((4, 8), dtype=torch.uint8, device="cuda"), s)


# one slice or several, column tiles of 256 and their remainders, streaming loads from 256 MiB on
@pytest.mark.parametrize("M,d", [(1, 8), (7, 248), (64, 256), (65, 264), (127, 2056), (128, 14336), (129, 520), (577, 4096),
                                 (1030, 8), (33, 40000), (2049, 65536)])
def test_statistics_over_slices_and_column_tiles(M, d):
    torch = _torch()
    print(f"[case] statistics M={M} d={d}", flush=True)
    rng = np.random.default_rng(M + d)
    bits = synth.f64_to_bf16_bits(rng.standard_normal((min(M, 600), d)) * np.exp(rng.uniform(-2, 2, size=(1, d))))
    bits = np.tile(bits, (-(-M // bits.shape[0]), 1))[:M]
    wide = torch.full((M, d + 16), 1.0e4, dtype=torch.bfloat16, device="cuda")       # strided rows, loud padding
    wide[:, :d] = binding.bits_to_device(bits)
    out = torch.full((d + 8,), -1.0, device="cuda")
    a = np.zeros(d)
    top = np.zeros(d)
    for r in range(0, M, 600):
        x = np.abs(orc.bf16_bits_to_f64(bits[r:r + 600]))
        a, top = a + x.sum(axis=0) / M, np.maximum(top, x.max(axis=0))
    got = binding.perq_colabs_mean(wide[:, :d], out=out[:d]).cpu().numpy().astype(np.float64)
    r = max(8, -(-M // max(1, 512 // -(-d // 2048))))                                # the documented bound
    assert np.all(np.abs(got - a) <= (r + 1) * 2.0 ** -24 * a)
    assert np.array_equal(binding.perq_colabs_absmax(wide[:, :d], out=out[:d]).cpu().numpy().astype(np.float64), top)
    assert bool((out[d:] == -1.0).all())


# A fp32 sum that starts with a 1 loses every later value below half its last place, so rows of ones that are followed
# by rows of such values show how many rows a sum takes in: the documented number r at most, also where the
# widths do not divide evenly.
@pytest.mark.parametrize("M,d", [(4096, 28672), (32768, 28672), (4096, 43776), (4096, 8192), (33333, 256), (1000, 140000)])
def test_mean_of_rows_that_one_sum_would_lose(M, d):
    torch = _torch()
    r = max(8, -(-M // max(1, 512 // -(-d // 2048))))
    for step in (-(-M // max(1, 512 // -(-d // 256))), 8 * r, r):
        print(f"[case] statistics M={M} d={d} ones every {step} rows", flush=True)
        v = torch.full((M,), 2.0 ** -24 * (1 - 2.0 ** -8), dtype=torch.bfloat16)
        v[(torch.arange(M) % step) < 8] = 1.0
        x = v.cuda()[:, None].expand(M, d).contiguous()
        a = float(v.double().mean())
        got = binding.perq_colabs_mean(x).double()
        assert float((got - a).abs().max()) <= (r + 1) * 2.0 ** -24 * a
        assert bool((binding.perq_colabs_absmax(x) == 1.0).all())


def test_mean_of_values_near_the_top_of_the_range():
    """Sums of r rows fit fp32 here, sums of more do not."""
    torch = _torch()
    for M, d in ((1024, 256), (4096, 520), (130, 8192)):
        x = torch.full((M, d), 3.0e37, dtype=torch.bfloat16, device="cuda")
        got = binding.perq_colabs_mean(x).double()
        assert bool(((got - x[0].double()).abs() <= 9 * 2.0 ** -24 * x[0].double()).all()), (M, d)


# ---- ablation permutations and the per-token diagnostics (Appendix C; Section 3) ------------------
def test_colabs_absmax_is_exact():
    wl = synth.llama1b_down()
    bits = wl.calib_rows()[:700]
    got = binding.perq_colabs_absmax(binding.bits_to_device(bits)).cpu().numpy()
    assert np.array_equal(got.astype(np.float64), orc.colabs_max(orc.bf16_bits_to_f64(bits)))


@pytest.mark.parametrize("T,d,bs", [(37, 256, [16, 32, 64, 256]), (9, 4096, [16, 128, 2048, 4096]), (5, 14336, [32, 2048]),
                                     (3, 8192, [4096, 8192]), (4, 32768, [1024, 32768])])
def test_block_diagnostics_against_oracle(T, d, bs):
    rng = np.random.default_rng(3000 + d)
    x = rng.standard_t(3, size=(T, d))
    x[:, rng.choice(d, size=max(1, d // 100), replace=False)] *= 50
    bits = synth.f64_to_bf16_bits(x)
    xd = binding.bits_to_device(bits)
    torch = _torch()
    perm = rng.permutation(d).astype(np.int32)
    for b in bs:
        for pm in (None, perm):
            pt = None if pm is None else torch.from_numpy(pm).cuda()
            got = binding.perq_block_diagnostics(xd, pt, b).cpu().numpy().astype(np.float64)
            want = orc.block_diagnostics(bits, pm, b) if b <= 4096 else None
            if want is None:         # explicit H_b too large: same quantities with the fast transform
                X = orc.bf16_bits_to_f64(bits); Xp = orc.permute_channels(X, pm)
                want = np.stack([np.abs(X).max(1), np.abs(X).sum(1), np.abs(Xp).reshape(T, d // b, b).sum(2).max(1),
                                 np.abs(orc.fwht_f64(Xp, b)).max(1)], axis=1)
            l2 = np.linalg.norm(orc.bf16_bits_to_f64(bits), axis=1)
            assert np.array_equal(got[:, 0], want[:, 0])
            assert np.allclose(got[:, 1], want[:, 1], rtol=2e-6) and np.allclose(got[:, 2], want[:, 2], rtol=2e-6)
            assert np.all(np.abs(got[:, 3] - want[:, 3]) <= 1e-5 * l2)
            assert np.all(got[:, 3] <= got[:, 2] / np.sqrt(b) * (1 + 1e-5))        # Proposition 2 on the device numbers


@pytest.mark.parametrize("d,b", [(64, 16), (64, 32), (128, 128), (96, 32), (512, 64), (2080, 32), (4096, 16), (4096, 32), (4096, 512), (8192, 64), (8192, 256), (11008, 256),
                                 (9728, 16), (14336, 128), (28672, 64), (28672, 2048)])
@pytest.mark.parametrize("perm", [False, True])
def test_block_diagnostics_as_exact_as_the_butterflies(d, b, perm):
    """The largest rotated value of a row: the butterflies' for b = 16 and 64 and for rows of 64 and 128 through a permutation, elsewhere
    no further from 64 bits than theirs."""
    torch = _torch()
    print(f"[case] statistics d={d} b={b} perm={perm}", flush=True)
    T = (1 << 24) // d
    g = torch.Generator(device="cuda").manual_seed(d + b)
    x = torch.randn((T, d), device="cuda", generator=g)
    x /= torch.stack([torch.randn((T, d), device="cuda", generator=g) for _ in range(3)]).square().mean(dim=0).clamp(min=1e-6).sqrt()
    x[:, torch.randperm(d, device="cuda", generator=g)[:max(1, d // 100)]] *= 50.0
    x = x.clamp(-1e4, 1e4).to(torch.bfloat16)
    p = torch.randperm(d, device="cuda", generator=g).to(torch.int32) if perm else None
    got = binding.perq_block_diagnostics(x, p, b)[:, 3]
    theirs = binding.perq_permute_rotate_f32(x, p, b, algo="butterfly").abs().amax(dim=1)
    if b in (16, 64) or (perm and d in (64, 128)):
        assert torch.equal(got, theirs)
    v = x.double() if p is None else x.double()[:, p.long()]
    h = 1
    while h < b:
        v = v.reshape(-1, 2, h)
        v = torch.stack((v[:, 0] + v[:, 1], v[:, 0] - v[:, 1]), dim=1)
        h *= 2
    want = v.reshape(T, d).abs().amax(dim=1) / b ** 0.5
    error = [float((((o.double() - want) / want) ** 2).mean() ** 0.5) for o in (got, theirs)]
    print(f"       error {error[0]:.3e}, butterflies {error[1]:.3e}", flush=True)
    # (the mean ratio over many such inputs is 1.000 - 1.002 where the scale is a power of two, and below 1 elsewhere; a root mean square
    # over T >= 512 rows scatters by 1 / sqrt(2 T), 3 % at most)
    assert error[0] <= 1.03 * error[1]


def test_calibrated_permutations_ranked_by_the_bound():
    """MassDiff against identity / random / absmax / ZigZag on the calibrated synthetic law: the mean
    Proposition 2 bound over apply tokens, from the device diagnostics."""
    torch = _torch()
    wl = synth.llama1b_down()
    b = 32
    cal = binding.bits_to_device(wl.calib_rows())
    a = binding.perq_colabs_mean(cal).cpu().numpy()
    amx = binding.perq_colabs_absmax(cal).cpu().numpy()
    x = binding.bits_to_device(wl.apply_rows(0, 512))
    perms = {"identity": None, "massdiff": binding.perq_massdiff_perm(a, b), "absmax": binding.perq_perm_sorted(amx),
             "zigzag": binding.perq_perm_zigzag(amx, b), "random": binding.perq_perm_random(wl.d, 2026)}
    bound = {}
    for name, pm in perms.items():
        pt = None if pm is None else torch.from_numpy(pm).cuda()
        dg = binding.perq_block_diagnostics(x, pt, b).cpu().numpy()
        bound[name] = float((dg[:, 2] / np.sqrt(b) / dg[:, 0]).mean())
    print("mean normalised Prop. 2 bound:", bound, flush=True)
    assert bound["massdiff"] < bound["identity"] and bound["massdiff"] <= bound["zigzag"] * 1.02
    assert bound["absmax"] > bound["massdiff"]            # sorting concentrates the heavy channels in one block
    assert bound["random"] >= bound["massdiff"]           # a shuffle spreads them by chance only


# ---- the fused call with a placement prepared for the permutation -------------------------------------
def _in_bulk(x):
    """x over and over, 2^25 elements and more: with a permutation and d >= 4096 the matrix-core kernel takes so
    many whatever b is, and reads the prepared form."""
    return x.repeat((1 << 25) // x.numel() + 1, 1)


@pytest.mark.parametrize("T,d,b,fmt", [(300, 4096, 128, "int4"), (4200, 4096, 128, "int4"), (300, 4096, 4096, "int4"),
                                       (2100, 8192, 32, "mxfp4"), (1030, 14336, 128, "int4"), (1030, 14336, 2048, "int4_asym"),
                                       (270, 14336, 512, "fp4_token"), (530, 20480, 1024, "int4"), (600, 12288, 64, "mxfp4"),
                                       (1, 4096, 16, "int4"), (3, 8192, 1024, "mxfp4"), (2050, 8192, 32, "int4"),
                                       (5, 12288, 4096, "int4"), (77, 14336, 2048, "int4"), (130, 32768, 256, "int4"),
                                       (9, 24576, 4096, "fp4_token"), (2, 16384, 64, "int4_asym")])
def test_prepared_placement_gives_the_plain_call_bit_for_bit(T, d, b, fmt):
    """The prepared form only moves work out of the launch (operand offsets worked out once per
    permutation) and, on wide rows, decides where the row's pieces sit in LDS between the staging loads
    and the operand reads of one launch: the form of perq_perm_prepare, and any other valid one, must
    not change a bit."""
    torch = _torch()
    rng = np.random.default_rng(T + d + b)
    x_bits = synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, d)) * np.exp(rng.uniform(-2, 2, size=(T, 1))))
    perm = rng.permutation(d).astype(np.int32)
    x = binding.bits_to_device(x_bits)
    perm_t = torch.from_numpy(perm).cuda()
    print(f"[case] prepared placement T={T} d={d} b={b} fmt={fmt}", flush=True)
    plain = binding.perq_permute_rotate_quant(x, perm_t, b, fmt)
    table, before, after, reads = binding.perq_perm_prepare(perm, b)
    assert after < before
    rows = min(T, 128)
    got = binding.perq_permute_rotate_quant(x, perm_t, b, fmt, placement=binding.placement_to_device(table))
    torch.cuda.synchronize()
    assert torch.equal(got[0], plain[0]) and torch.equal(got[1], plain[1])          # (few rows: the form may be ignored)
    # many rows: the kernel that reads the form, against the same kernel chosen without one
    bulk = _in_bulk(x)
    want = binding.perq_permute_rotate_quant(bulk, perm_t, b, fmt, algo="mfma")
    got = binding.perq_permute_rotate_quant(bulk, perm_t, b, fmt, placement=binding.placement_to_device(table))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    # ... and it does read it: the form of another permutation gives other codes
    other = binding.placement_to_device(binding.perq_perm_prepare(np.roll(perm, 1), b)[0])
    assert not torch.equal(binding.perq_permute_rotate_quant(bulk, perm_t, b, fmt, placement=other)[0], want[0])
    # a random valid form: the 8 pieces of every 128-byte line shuffled
    G = d // 8
    slot_of = np.concatenate([8 * w + rng.permutation(8) for w in range(G // 8)]).astype(np.int64)
    rnd = prepared_form.assemble(perm, slot_of)
    assert binding.perq_perm_prepared_validate(rnd, perm)
    got = binding.perq_permute_rotate_quant(bulk, perm_t, b, fmt, placement=binding.placement_to_device(rnd))
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    # and against the oracle
    rep = parity.compare_apply(x_bits[:rows], perm, b, fmt, got[0][:rows].cpu().numpy(), got[1][:rows].cpu().numpy())
    assert rep.ok(), (rep.summary(), rep.notes[:5])


def test_prepared_form_on_seeded_random_shapes():
    """Forty seeded shapes (row widths in steps of 512 from 4096 to 32768, every block size that divides
    them, every format, 1 to 300 rows, alone and over and over until the matrix-core kernel takes them): the
    prepared call equals the plain call and that kernel without the form, bit for bit."""
    torch = _torch()
    rng = np.random.default_rng(20260)
    fmts = ["int4", "mxfp4", "int4_asym", "fp4_token"]
    for case in range(40):
        d = 512 * int(rng.integers(8, 65))
        bs = [b for b in (16, 32, 64, 128, 256, 512, 1024, 2048, 4096) if d % b == 0]
        b = int(bs[rng.integers(len(bs))])
        T = int(rng.integers(1, 301))
        fmt = fmts[case % 4]
        print(f"[case] prepared form, seeded shape {case}: T={T} d={d} b={b} fmt={fmt}", flush=True)
        x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, d))))
        perm = rng.permutation(d).astype(np.int32)
        perm_t = torch.from_numpy(perm).cuda()
        form = binding.placement_to_device(binding.perq_perm_prepare(perm, b)[0])
        plain = binding.perq_permute_rotate_quant(x, perm_t, b, fmt)
        got = binding.perq_permute_rotate_quant(x, perm_t, b, fmt, placement=form)
        torch.cuda.synchronize()
        assert torch.equal(got[0], plain[0]) and torch.equal(got[1], plain[1]), (T, d, b, fmt)
        bulk = _in_bulk(x)
        want = binding.perq_permute_rotate_quant(bulk, perm_t, b, fmt, algo="mfma")
        got = binding.perq_permute_rotate_quant(bulk, perm_t, b, fmt, placement=form)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (bulk.shape[0], d, b, fmt)


def test_prepared_placement_is_ignored_where_no_such_gather_runs():
    torch = _torch()
    rng = np.random.default_rng(77)
    # (the last three: too few rows for the kernel that reads the form)
    for T, d, b in ((50, 2048, 128), (40, 8192, 8192), (30, 3072, 768), (16, 4096, 128), (300, 8192, 32), (200, 14336, 128)):
        x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_normal((T, d))))
        perm_t = torch.from_numpy(rng.permutation(d).astype(np.int32)).cuda()
        junk = torch.full((binding.load().perq_perm_prepared_bytes(d),), 0x7F, dtype=torch.uint8, device="cuda")
        plain = binding.perq_permute_rotate_quant(x, perm_t, b, "int4")
        got = binding.perq_permute_rotate_quant(x, perm_t, b, "int4", placement=junk)
        torch.cuda.synchronize()
        assert torch.equal(got[0], plain[0]) and torch.equal(got[1], plain[1])


# ---- per-token quantization error (Section 3) ---------------------------------------------------------
@pytest.mark.parametrize("d,b", [(256, 16), (2048, 64), (4096, 128), (4096, 4096), (3072, 768)])
def test_quant_error_against_oracle_and_worst_case_bound(d, b):
    torch = _torch()
    rng = np.random.default_rng(d * 3 + b)
    T = 70
    x = rng.standard_t(3, size=(T, d))
    x[:, rng.choice(d, size=max(1, d // 100), replace=False)] *= 40.0
    x[T - 1] = 0.0                                                    # an all-zero token: no error, no norm
    x_bits = synth.f64_to_bf16_bits(x)
    perm = rng.permutation(d).astype(np.int32)
    xd = binding.bits_to_device(x_bits)
    perm_t = torch.from_numpy(perm).cuda()
    y = binding.perq_permute_rotate_f32(xd, perm_t, b)
    Y = orc.block_hadamard(orc.permute_channels(orc.bf16_bits_to_f64(x_bits), perm), b)
    for fmt in ("int4", "mxfp4", "int4_asym", "fp4_token", "fp4_token7"):
        print(f"[case] quant error d={d} b={b} fmt={fmt}", flush=True)
        codes, scales = binding.perq_permute_rotate_quant(xd, perm_t, b, fmt)
        got = binding.perq_quant_error(y, codes, scales, fmt).cpu().numpy().astype(np.float64)
        want = orc.quant_error(Y, fmt)
        assert np.all(np.abs(got - want) <= 1e-4 * want + 1e-30), (fmt, np.abs(got - want).max())
        assert np.all(got[T - 1] == 0.0)
        if fmt == "int4":
            # Section 3 on the device's own numbers: ||y - Q(y)||_2 <= sqrt(d) / (2^4 - 2) ||y||_inf
            assert np.all(got[:, 0] <= math.sqrt(d) / 14.0 * got[:, 2] * (1 + 1e-5))


def test_quant_error_of_codes_scales_and_rows_that_are_not_aligned():
    """Codes and e8m0 bytes at odd addresses, y at 8 modulo 16: what the entry point takes beside the aligned case."""
    torch = _torch()
    g = torch.Generator(device="cuda").manual_seed(4)
    for T, d in ((5, 32), (9, 96), (70, 4128)):
        y = torch.randn((T, d), device="cuda", generator=g)
        for fmt in ("int4", "mxfp4", "int4_asym", "fp4_token"):
            print(f"[case] quant error, not aligned T={T} d={d} fmt={fmt}", flush=True)
            codes, scales = binding.alloc_outputs(T, d, fmt, "cuda")
            codes.random_(0, 256, generator=g)
            if fmt == "mxfp4":
                scales.random_(100, 140, generator=g)
            else:
                scales.uniform_(0.1, 2.0, generator=g)
            want = binding.perq_quant_error(y, codes, scales, fmt)
            off = lambda t, k: torch.empty(t.numel() + k, dtype=t.dtype, device="cuda")[k:].view(t.shape).copy_(t)
            got = binding.perq_quant_error(off(y, 2), off(codes, 1), off(scales, 1) if fmt != "int4_asym" else scales, fmt)
            assert torch.equal(got, want)


# long and short calls on either side of the lines between the two kernels, rows of one tile, two, three and more, folded, ragged
@pytest.mark.parametrize("T,d,b", [(2048, 8192, 32), (1024, 14336, 128), (600, 14336, 128), (40, 28672, 64), (1600, 9728, 16), (6000, 3072, 128),
                                   (900, 16384, 2048), (300, 12288, 1024), (2048, 4096, 64), (4096, 2048, 64), (1500, 11008, 256)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_fp32_output_is_what_the_codes_were_made_from(T, d, b, fmt):
    """AUTO takes one of the two kernels for both calls of an input."""
    torch = _torch()
    print(f"[case] one kernel T={T} d={d} b={b} fmt={fmt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d)
    x = torch.randn((T, d), device="cuda", generator=g).to(torch.bfloat16)
    perm = torch.randperm(d, device="cuda", generator=g).to(torch.int32)
    for p in (perm, None):
        codes, scales = binding.perq_permute_rotate_quant(x, p, b, fmt)
        y = binding.perq_permute_rotate_f32(x, p, b)
        same = []
        for algo in ("butterfly", "mfma") if d % 512 == 0 else ("butterfly",):
            c, s = binding.perq_permute_rotate_quant(x, p, b, fmt, algo=algo)
            same.append((torch.equal(c, codes) and torch.equal(s, scales), torch.equal(binding.perq_permute_rotate_f32(x, p, b, algo=algo), y)))
        if d % 512 == 0:
            assert (True, True) in same, same
        else:                                     # (no explicit call of the other kernel: it is the one that the butterflies are not)
            assert same[0][0] == same[0][1] or fmt == "mxfp4", same


# ---- the ticket counters under concurrency and graph replay ------------------------------------------
# (block_kernel, mfma_kernel with a wave and with a workgroup as worker, one of each)
@pytest.mark.parametrize("shapes", [((6000, 4096, 128, "int4"), (2100, 8192, 32, "mxfp4")), ((6000, 4096, 2048, "int4"), (1100, 14336, 128, "int4")),
                                    ((4300, 4096, 4096, "int4"), (1500, 14336, 512, "mxfp4"))])
def test_run_time_schedule_on_two_streams_and_in_a_graph(shapes):
    """Every stream has a counter set of its own, so launches that overlap on two streams never draw
    from the same counters; a launch that is being captured takes the fixed split and can be replayed
    beside eager launches: every result equals the eager one."""
    torch = _torch()
    rng = np.random.default_rng(123)
    cases = []
    for T, d, b, fmt in shapes:
        print(f"[case] two streams T={T} d={d} b={b} fmt={fmt}", flush=True)
        x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_normal((T, d))))
        perm = torch.from_numpy(rng.permutation(d).astype(np.int32)).cuda()
        ref = binding.perq_permute_rotate_quant(x, perm, b, fmt, algo="mfma")
        cases.append((x, perm, b, fmt, ref))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    sets = [binding.perq_schedule_set(st) for st in streams]
    assert sets[0] != sets[1] and min(sets) >= 0
    assert sets == [binding.perq_schedule_set(st) for st in streams]            # a stream keeps its set
    outs = [[], []]
    for rep in range(40):
        for k, st in enumerate(streams):
            x, perm, b, fmt, ref = cases[k]
            codes, scales = binding.alloc_outputs(x.shape[0], x.shape[1], fmt, x.device)
            with torch.cuda.stream(st):
                binding.perq_permute_rotate_quant(x, perm, b, fmt, codes=codes, scales=scales, stream=st, algo="mfma")
            outs[k].append((codes, scales))
    torch.cuda.synchronize()
    for k in range(2):
        ref = cases[k][4]
        for i, (codes, scales) in enumerate(outs[k]):
            assert torch.equal(codes, ref[0]) and torch.equal(scales, ref[1]), f"stream {k} launch {i}"
    # graph: capture one launch, replay it with eager launches in between
    x, perm, b, fmt, ref = cases[0]
    codes, scales = binding.alloc_outputs(x.shape[0], x.shape[1], fmt, x.device)
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        binding.perq_permute_rotate_quant(x, perm, b, fmt, codes=codes, scales=scales, stream=st, algo="mfma")   # warm
        st.synchronize()
        with torch.cuda.graph(g, stream=st):
            assert binding.perq_schedule_set(torch.cuda.current_stream()) == -1   # capturing: fixed split
            binding.perq_permute_rotate_quant(x, perm, b, fmt, codes=codes, scales=scales,
                                              stream=torch.cuda.current_stream(), algo="mfma")
    other = torch.cuda.Stream()
    for rep in range(4):
        codes.fill_(0xAA); scales.fill_(-1.0)
        torch.cuda.synchronize()
        # the replay runs beside eager launches of the same shape on another stream
        with torch.cuda.stream(other):
            e1 = binding.perq_permute_rotate_quant(x, perm, b, fmt, stream=other, algo="mfma")
        g.replay()
        with torch.cuda.stream(other):
            e2 = binding.perq_permute_rotate_quant(x, perm, b, fmt, stream=other, algo="mfma")
        torch.cuda.synchronize()
        assert torch.equal(codes, ref[0]) and torch.equal(scales, ref[1]), f"replay {rep}"
        for e in (e1, e2):
            assert torch.equal(e[0], ref[0]) and torch.equal(e[1], ref[1]), f"eager beside replay {rep}"
        eager = binding.perq_permute_rotate_quant(x, perm, b, fmt, algo="mfma")
        torch.cuda.synchronize()
        assert torch.equal(eager[0], ref[0])


def test_prepared_form_and_chunked_kernel_in_a_graph():
    """A captured launch with a prepared form (its table reads are waited for by count) and a captured
    launch of the chunked kernel (its grid comes from an occupancy query) replay to the eager result,
    with eager work between the replays."""
    torch = _torch()
    rng = np.random.default_rng(321)
    st = torch.cuda.Stream()
    for T, d, b, fmt, prepared in ((1100, 8192, 64, "int4", True), (300, 14336, 2048, "int4_asym", True),
                                   (500, 12288, 12288, "int4", False), (260, 16384, 8192, "mxfp4", False)):
        print(f"[case] graph T={T} d={d} b={b} fmt={fmt} prepared={prepared}", flush=True)
        x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, d))))
        perm_np = rng.permutation(d).astype(np.int32) if prepared else None
        perm = torch.from_numpy(perm_np).cuda() if prepared else None
        form = binding.placement_to_device(binding.perq_perm_prepare(perm_np, b)[0]) if prepared else None
        ref = binding.perq_permute_rotate_quant(x, perm, b, fmt, algo="mfma" if prepared else "auto")
        if prepared:          # the form is read
            other = binding.placement_to_device(binding.perq_perm_prepare(np.roll(perm_np, 1), b)[0])
            assert not torch.equal(binding.perq_permute_rotate_quant(x, perm, b, fmt, placement=other)[0], ref[0])
        codes, scales = binding.alloc_outputs(T, d, fmt, x.device)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(st):
            binding.perq_permute_rotate_quant(x, perm, b, fmt, codes=codes, scales=scales, stream=st, placement=form)   # warm
            st.synchronize()
            with torch.cuda.graph(g, stream=st):
                binding.perq_permute_rotate_quant(x, perm, b, fmt, codes=codes, scales=scales,
                                                  stream=torch.cuda.current_stream(), placement=form)
        for rep in range(3):
            codes.fill_(0x55); scales.fill_(3)
            eager = binding.perq_permute_rotate_quant(x, perm, b, fmt, placement=form)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(codes, ref[0]) and torch.equal(scales, ref[1]), f"replay {rep}"
            assert torch.equal(eager[0], ref[0]) and torch.equal(eager[1], ref[1])


def test_column_statistics_take_no_set_of_the_row_schedule():
    """A stream that only computes statistics, of columns or of blocks, leaves the 64 sets of the fused path to others."""
    torch = _torch()
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    raw = []
    for _ in range(4):
        h = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(h)) == 0
        raw.append(h)
    streams = [torch.cuda.ExternalStream(h.value) for h in raw]
    x = torch.randn((1024, 2048), device="cuda").to(torch.bfloat16)
    want = binding.perq_colabs_mean(x)
    torch.cuda.synchronize()
    first = binding.perq_schedule_set(streams[0])
    got = [binding.perq_colabs_mean(x, stream=st) for st in streams[1:3]]
    many = torch.zeros((20000, 2048), device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for st in streams[1:3]:
        binding.perq_block_diagnostics(many, None, 128, stream=st)
    last = binding.perq_schedule_set(streams[3])
    torch.cuda.synchronize()
    assert all(torch.equal(g, want) for g in got)
    assert first >= 0 and last == first + 1
    del streams
    for h in raw:
        assert hip.hipStreamDestroy(h) == 0


def test_reset_leaves_the_column_statistics_of_other_streams_alone():
    torch = _torch()
    xs = [torch.randn((4096, 8192), device="cuda").to(torch.bfloat16) for _ in range(2)]
    want = [binding.perq_colabs_mean(x) for x in xs]
    st, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    got = []
    for k in range(60):
        with torch.cuda.stream(st):
            got.append(binding.perq_colabs_mean(xs[k % 2]))
        for _ in range(3):
            binding.perq_reset_schedule(other)
    torch.cuda.synchronize()
    assert all(torch.equal(g, want[k % 2]) for k, g in enumerate(got))
    # on its own stream a reset comes after what was queued before it
    with torch.cuda.stream(st):
        binding.perq_reset_schedule(st)
        assert torch.equal(binding.perq_colabs_mean(xs[0]), want[0])


def test_reset_leaves_the_block_statistics_of_other_streams_alone():
    """A launch whose counters went back to zero under it would leave them off zero, and the next one would skip rows."""
    torch = _torch()
    x = torch.randn((30000, 4096), device="cuda").to(torch.bfloat16)
    want = binding.perq_block_diagnostics(x, None, 128)
    st, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    got = []
    for k in range(40):
        out = torch.full_like(want, -1.0)
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st):
            got.append(binding.perq_block_diagnostics(x, None, 128, out=out))
        for _ in range(6):
            binding.perq_reset_schedule(other)
    torch.cuda.synchronize()
    assert all(torch.equal(g, want) for g in got)
    with torch.cuda.stream(st):
        binding.perq_reset_schedule(st)
        assert torch.equal(binding.perq_block_diagnostics(x, None, 128), want)
    torch.cuda.synchronize()


@pytest.mark.parametrize("b", [128, 2048])          # (block_kernel, mfma_kernel)
def test_run_time_schedule_more_streams_than_counter_sets_and_reset(b):
    """The 65th stream of a device gets no counter set: its launches take the fixed split.  All
    streams launch at once; every result equals the reference.  perq_reset_schedule leaves the
    counters usable."""
    torch = _torch()
    rng = np.random.default_rng(321)
    T, d, fmt = 4300, 4096, "int4"
    x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_normal((T, d))))
    perm = torch.from_numpy(rng.permutation(d).astype(np.int32)).cuda()
    ref = binding.perq_permute_rotate_quant(x, perm, b, fmt, algo="mfma")
    torch.cuda.synchronize()
    # (torch hands out streams from a pool of 32; 80 distinct ones come from the runtime itself)
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    raw = []
    for _ in range(80):
        h = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(h)) == 0
        raw.append(h)
    streams = [torch.cuda.ExternalStream(h.value) for h in raw]
    sets = [binding.perq_schedule_set(st) for st in streams]
    with_set = [s for s in sets if s >= 0]
    assert len(set(with_set)) == len(with_set) and max(sets) <= 63          # one set per stream
    assert sets.count(-1) >= 80 - 64                                         # the late-comers have none
    outs = []
    for st in streams:
        codes, scales = binding.alloc_outputs(T, d, fmt, x.device)
        with torch.cuda.stream(st):
            binding.perq_permute_rotate_quant(x, perm, b, fmt, codes=codes, scales=scales, stream=st, algo="mfma")
        outs.append((codes, scales))
    torch.cuda.synchronize()
    for i, (codes, scales) in enumerate(outs):
        assert torch.equal(codes, ref[0]) and torch.equal(scales, ref[1]), f"stream {i} (set {sets[i]})"
    binding.perq_reset_schedule()
    again = binding.perq_permute_rotate_quant(x, perm, b, fmt, algo="mfma")
    torch.cuda.synchronize()
    assert torch.equal(again[0], ref[0]) and torch.equal(again[1], ref[1])
    del streams
    for h in raw:
        assert hip.hipStreamDestroy(h) == 0


# ---- edges of the run-time schedule: exactly two units per worker, one more, strided rows, long T ----
@pytest.mark.parametrize("b", [64, 2048])          # (block_kernel, mfma_kernel)
@pytest.mark.parametrize("T", [4095, 4096, 4097, 4160])
def test_run_time_schedule_threshold_edges(T, b):
    """d = 4096 has room for 2048 workers (of two waves, of one): T = 4096 is the first size on the ticket path (mfma_kernel:
    no row left to draw), T = 4095 the last on the fixed stride."""
    rng = np.random.default_rng(T)
    d = 4096
    x = synth.f64_to_bf16_bits(rng.standard_normal((T, d)) * np.exp(rng.uniform(-1, 1, size=(T, 1))))
    perm = rng.permutation(d).astype(np.int32)
    for fmt in ("int4", "mxfp4"):
        for _ in range(2):                          # twice: the counters must be back at zero
            codes, scales, _y = run_gpu(x, perm, b, fmt, "mfma", want_y=False)
            rep = parity.compare_apply(x, perm, b, fmt, codes, scales, None)
            assert rep.ok(), (T, fmt, rep.summary(), rep.notes[:5])


@pytest.mark.parametrize("b", [128, 4096])         # (block_kernel, mfma_kernel)
def test_run_time_schedule_with_a_row_stride(b):
    rng = np.random.default_rng(5)
    T, d = 2300, 8192
    x = synth.f64_to_bf16_bits(rng.standard_normal((T, d)))
    perm = rng.permutation(d).astype(np.int32)
    codes, scales, _y = run_gpu(x, perm, b, "int4", "mfma", want_y=False, ldx=d + 512)
    rep = parity.compare_apply(x, perm, b, "int4", codes, scales, None)
    assert rep.ok(), (rep.summary(), rep.notes[:5])


@pytest.mark.parametrize("b", [128, 2048])         # (block_kernel, mfma_kernel)
def test_long_launch_sampled_rows(b):
    """T = 131072 rows of 4096, 60 and more tickets to a worker: sampled rows against the oracle, every row's scale against
    the identity |y|_inf = |scale| * 7 <= |x|_2."""
    torch = _torch()
    T, d = 131072, 4096
    g = torch.Generator(device="cuda"); g.manual_seed(11)
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    perm = np.random.default_rng(12).permutation(d).astype(np.int32)
    perm_t = torch.from_numpy(perm).cuda()
    codes, scales = binding.perq_permute_rotate_quant(x, perm_t, b, "int4", algo="mfma")
    rows = np.unique(np.concatenate([np.arange(40), T - 1 - np.arange(40), np.random.default_rng(13).choice(T, 120, replace=False)]))
    rt = torch.from_numpy(rows).cuda()
    x_bits = x[rt].view(torch.int16).cpu().numpy().view(np.uint16)
    rep = parity.compare_apply(x_bits, perm, b, "int4", codes[rt].cpu().numpy(), scales[rt].cpu().numpy(), None)
    assert rep.ok(), (rep.summary(), rep.notes[:5])
    l2 = x.float().norm(dim=1)
    assert torch.all(scales > 0) and torch.all(scales * 7 <= l2 * (1 + 1e-5))
    nib = codes.view(torch.uint8)
    lo, hi = nib & 0xF, nib >> 4
    assert torch.all(((lo == 7) | (lo == 9) | (hi == 7) | (hi == 9)).any(dim=1))       # every row reaches +-7


# ---- block sizes 2^k' * 28 (the non-power-of-two rotation of Appendix A.1) ----------------------
def _heavy_rows(T, d, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_t(3, size=(T, d)).clip(-1e4, 1e4)
    x[:, rng.choice(d, max(d // 100, 1), replace=False)] *= 50.0
    return synth.f64_to_bf16_bits(x)


@pytest.mark.parametrize("d,bs", [(3584, [28, 112, 896, 3584]), (7168, [56, 1792, 7168]),
                                  (14336, [28, 224, 3584, 7168, 14336]),
                                  # base 12 (chunks of 3072): k' = 1 .. 10
                                  (3072, [24, 48, 768, 1536, 3072]), (6144, [96, 3072, 6144]),
                                  (12288, [24, 192, 1536, 3072, 6144, 12288]),
                                  # base 76 (chunks of 2432): k' = 0 .. 7
                                  (2432, [76, 152, 608, 1216, 2432]), (4864, [304, 2432, 4864]),
                                  (9728, [76, 1216, 2432, 4864, 9728]),
                                  # rows of eight chunks: workgroups of eight waves (base 28; the powers of
                                  # two above 4096 take the same kernel with H_32 as base)
                                  (28672, [28, 3584, 7168, 14336, 28672]), (32768, [8192, 16384, 32768])])
@pytest.mark.parametrize("with_perm", [False, True])
def test_nonpo2_rotation_against_oracle(d, bs, with_perm):
    T = (5 if d >= 28672 else 13) if d >= 9728 else 21      # ragged against 1, 2 and 4 rows per workgroup pass
    x = _heavy_rows(T, d, 900 + d)
    perm = np.random.default_rng(d).permutation(d).astype(np.int32) if with_perm else None
    for b in bs:
        rotate = orc.fwht_f64 if (b > 4096 and b & (b - 1) == 0) else None
        for fmt in (["int4", "mxfp4"] if b not in (bs[0], bs[-1]) else ["int4", "mxfp4", "int4_asym", "fp4_token"]):
            assert_parity(x, perm, b, fmt, "auto", rotate=rotate, label="nonpo2")


def test_nonpo2_structured_rows_and_many_rows():
    d, b = 14336, 14336
    H28 = orc.paley_hadamard(28).astype(np.float64)
    # one-hot rows: every output has magnitude |c| / sqrt(b); row a*28 + r of H_512 (x) H_28
    T = 6
    x = np.zeros((T, d))
    hot = [0, 27, 28, 5000, 14335, 7168]
    for t, i in enumerate(hot):
        x[t, i] = 2.0 ** (t - 2)
    bits = synth.f64_to_bf16_bits(x)
    torch = _torch()
    y = binding.perq_permute_rotate_f32(binding.bits_to_device(bits), None, b).cpu().numpy().astype(np.float64)
    for t, i in enumerate(hot):
        a, r = divmod(i, 28)
        aa = np.arange(512)
        sylv = 1.0 - 2.0 * (np.array([bin(a & v).count("1") for v in aa]) & 1)
        want = (sylv[:, None] * H28[r][None, :]).reshape(d) * 2.0 ** (t - 2) / np.sqrt(b)
        assert np.allclose(y[t], want, rtol=1e-6, atol=0), (t, i)
    # all-zero rows, a constant row, and more rows than one pass of the grid covers
    x = np.zeros((3, d)); x[1] = 1.0
    for fmt in ("int4", "mxfp4", "int4_asym", "fp4_token"):
        assert_parity(synth.f64_to_bf16_bits(x), None, b, fmt, "auto", label="nonpo2/zero+const")
    big = _heavy_rows(1100, d, 77)
    codes, scales = binding.perq_permute_rotate_quant(binding.bits_to_device(big), None, b, "int4")
    torch.cuda.synchronize()
    rows = np.r_[0:8, 505:520, 1017:1032, 1092:1100]
    rep = parity.compare_apply(big[rows], None, b, "int4", codes.cpu().numpy()[rows], scales.cpu().numpy()[rows])
    print("       ", rep.summary(), flush=True)
    assert rep.ok(), rep.summary()


def test_nonpo2_argument_checks():
    torch = _torch()
    x = torch.zeros((4, 14336), dtype=torch.bfloat16, device="cuda")
    # 14336 = 2^9 * 28 only: a base of 12 or 76 does not divide it, and 7 * 2^k with k < 2 is no Hadamard order
    with pytest.raises(binding.PerqError) as ei:
        binding.perq_permute_rotate_quant(x, None, 14, "int4")
    assert ei.value.status == binding.PERQ_ERR_INVALID_ARG
    # known base, width the kernels do not cover (1, 2 or 4 chunks of 3072 for the base of 12)
    x12 = torch.zeros((4, 1536), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(binding.PerqError) as ei:
        binding.perq_permute_rotate_quant(x12, None, 1536, "int4")
    assert ei.value.status == binding.PERQ_ERR_UNSUPPORTED
    # a base the library can build (20 = 19 + 1) but has no kernel for
    x20 = torch.zeros((4, 20 * 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(binding.PerqError) as ei:
        binding.perq_permute_rotate_quant(x20, None, 20 * 64, "int4")
    assert ei.value.status == binding.PERQ_ERR_UNSUPPORTED
    # order 4 * 9 = 36 = 2 * (17 + 1) exists by the second construction, 4 * 23 = 92 by neither
    x92 = torch.zeros((4, 92 * 8), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(binding.PerqError) as ei:
        binding.perq_permute_rotate_quant(x92, None, 92, "int4")
    assert ei.value.status == binding.PERQ_ERR_INVALID_ARG
    # the rotation kernels named explicitly do not take these block sizes
    for algo in ("butterfly", "mfma"):
        with pytest.raises(binding.PerqError) as ei:
            binding.perq_permute_rotate_quant(x, None, 14336, "int4", algo=algo)
        assert ei.value.status == binding.PERQ_ERR_UNSUPPORTED


def test_nonpo2_row_stride_single_row_empty_and_repeat():
    torch = _torch()
    for d, b in [(14336, 14336), (6144, 1536), (9728, 9728)]:
        x = _heavy_rows(9, d, 31 + d)
        # rows at a pitch larger than d (a view into a wider buffer)
        assert_parity(x, None, b, "int4", "auto", ldx=d + 64, label="nonpo2/stride")
        perm = np.random.default_rng(5).permutation(d).astype(np.int32)
        assert_parity(x, perm, b, "mxfp4", "auto", ldx=d + 8, label="nonpo2/stride+perm")
        # one row (three of a pass's four chunk slots stay empty when a row has one or two chunks)
        assert_parity(x[:1], None, b, "int4_asym", "auto", label="nonpo2/one row")
        # no rows: nothing is read or written
        xe = torch.empty((0, d), dtype=torch.bfloat16, device="cuda")
        codes, scales = binding.perq_permute_rotate_quant(xe, None, b, "int4")
        assert codes.shape[0] == 0 and scales.shape[0] == 0
        # the same call twice gives the same bytes
        xd = binding.bits_to_device(x)
        c1, s1 = binding.perq_permute_rotate_quant(xd, None, b, "fp4_token")
        c2, s2 = binding.perq_permute_rotate_quant(xd, None, b, "fp4_token")
        torch.cuda.synchronize()
        assert torch.equal(c1, c2) and torch.equal(s1, s2)


# ---- a permutation arranged for the LDS gather is a permutation like any other -------------------
@pytest.mark.parametrize("d,b,fmt", [(4096, 128, "int4"), (14336, 128, "int4"), (14336, 2048, "mxfp4"),
                                     (8192, 32, "mxfp4"), (4096, 4096, "int4_asym"), (16384, 1024, "fp4_token")])
def test_arranged_permutation(d, b, fmt):
    rng = np.random.default_rng(d * 3 + b)
    a = np.exp(rng.normal(0, 1.5, d)).astype(np.float32)
    greedy = binding.perq_massdiff_perm(a, b)
    assert np.array_equal(greedy, orc.massdiff_greedy(a.astype(np.float64), b))
    perm = binding.perq_perm_arrange(greedy, b)
    assert not np.array_equal(perm, greedy)
    x = _heavy_rows(11, d, 77 + d)
    for algo in ("mfma", "auto"):
        assert_parity(x, perm, b, fmt, algo, label="arranged perm")


# ---- rows of extreme magnitude ------------------------------------------------------------------
@pytest.mark.parametrize("d,b", [(256, 16), (512, 512), (4096, 128), (4096, 4096), (8192, 32), (2048, 2048),
                                 (3584, 3584), (8192, 8192)])
def test_rows_from_subnormal_to_huge(d, b):
    """Rows scaled by 2^-132 ... 2^110: bf16 subnormals (the quotient 7 / max of a per-token format is
    then beyond fp32), the smallest normals, and values whose block sums stay just inside fp32."""
    rng = np.random.default_rng(d + b)
    exps = [-132, -131, -130, -128, -126, -125, -120, -110, -101, -100, -99, -64, 0, 64, 100, 110]
    x = rng.standard_normal((len(exps), d)) * (2.0 ** np.array(exps, dtype=np.float64))[:, None]
    bits = synth.f64_to_bf16_bits(x)
    rotate = orc.fwht_f64 if (b > 4096 and b & (b - 1) == 0) else None
    for fmt in ("int4", "mxfp4", "int4_asym", "fp4_token"):
        for algo in ALGOS:
            if algo == "butterfly" and b & (b - 1):
                continue
            if algo == "mfma" and (b & (b - 1) or b > 4096):
                continue
            assert_parity(bits, None, b, fmt, algo, rotate=rotate, label="extreme magnitudes")


# ---- a seeded sweep over shapes, block sizes, formats, permutations and row pitches ---------------
def _random_cases(n, seed):
    rng = np.random.default_rng(seed)
    widths = [64, 256, 320, 512, 1536, 2048, 2432, 3072, 3584, 4096, 4864, 5120, 6144, 7168, 8192, 9728, 12288,
              14336, 16384, 28672, 32768]
    cases = []
    while len(cases) < n:
        d = int(rng.choice(widths))
        # block sizes the library takes for this width: powers of two, and 2^k' * {12, 28, 76} on the
        # widths of the three bases
        bs = [b for b in (16, 32, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384, 32768) if b <= d and d % b == 0]
        for base, chunk in ((28, 3584), (12, 3072), (76, 2432)):
            if d in (chunk, 2 * chunk, 4 * chunk) or (base == 28 and d == 8 * chunk):
                bs += [base << k for k in range(12) if (base << k) >= 16 and (base << k) <= d and d % (base << k) == 0]
        if d % 32 != 0 or not bs:
            continue
        b = int(rng.choice(bs))
        T = int(rng.integers(1, 48 if d < 20000 else 12))
        fmt = str(rng.choice(["int4", "mxfp4", "int4_asym", "fp4_token"]))
        with_perm = bool(rng.integers(0, 2))
        pad = int(rng.choice([0, 0, 8, 64, 1000]))
        cases.append((T, d, b, fmt, with_perm, pad, int(rng.integers(1 << 30))))
    return cases


@pytest.mark.parametrize("T,d,b,fmt,with_perm,pad,seed", _random_cases(72, 20260122))
def test_seeded_sweep(T, d, b, fmt, with_perm, pad, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_t(3, size=(T, d)).clip(-1e4, 1e4) * np.exp(rng.uniform(-4, 4, size=(T, 1)))
    x[:, rng.choice(d, size=max(1, d // 64), replace=False)] *= 40.0
    if T > 2:
        x[1] = 0.0                                   # an all-zero row
    bits = synth.f64_to_bf16_bits(x)
    perm = rng.permutation(d).astype(np.int32) if with_perm else None
    rotate = orc.fwht_f64 if (b > 4096 and b & (b - 1) == 0) else None
    assert_parity(bits, perm, b, fmt, "auto", rotate=rotate, ldx=(d + pad) if pad else None, label="sweep")


@pytest.mark.parametrize("d,b,fmt,with_perm", [(3584, 3584, "int4", False), (7168, 1792, "mxfp4", True),
                                               (3072, 3072, "int4_asym", True), (6144, 6144, "fp4_token", False),
                                               (2432, 2432, "mxfp4", False), (4864, 4864, "int4", True),
                                               (8192, 8192, "int4", True), (16384, 16384, "mxfp4", False),
                                               (28672, 28672, "int4", False), (32768, 16384, "mxfp4", True)])
def test_chunked_kernels_more_rows_than_one_pass_of_the_grid(d, b, fmt, with_perm):
    """Every workgroup comes round several times (4, 2 or 1 rows per pass); sampled rows against the oracle."""
    torch = _torch()
    chunk = next(c for c in (3584, 3072, 2432, 4096) if d % c == 0)      # positions per wave chunk
    rows_per_pass = max(1, 4 // (d // chunk))                            # a workgroup takes 4 (or 8) chunks per pass
    T = int(512 * rows_per_pass * 2.5) + 3
    print(f"[many] d={d} b={b} fmt={fmt} T={T}", flush=True)
    x = _heavy_rows(T, d, 4000 + d)
    perm = np.random.default_rng(d + 1).permutation(d).astype(np.int32) if with_perm else None
    perm_t = None if perm is None else torch.from_numpy(perm).cuda()
    codes, scales = binding.perq_permute_rotate_quant(binding.bits_to_device(x), perm_t, b, fmt)
    torch.cuda.synchronize()
    rng = np.random.default_rng(3)
    rows = np.unique(np.r_[0:6, T - 6:T, rng.choice(T, size=40, replace=False),
                           512 * rows_per_pass - 2:512 * rows_per_pass + 3])
    rotate = orc.fwht_f64 if (b > 4096 and b & (b - 1) == 0) else None
    rep = parity.compare_apply(x[rows], perm, b, fmt, codes.cpu().numpy()[rows], scales.cpu().numpy()[rows],
                               rotate=rotate)
    print("       ", rep.summary(), flush=True)
    assert rep.ok(), (rep.summary(), rep.notes[:5])


# ---- the matrix-core kernel of half the tile ---------------------------------------------------------
# rows that share a wave (512), are packed several to a unit from 512 units on (1536, 3072), leave a wave part empty (2880, which only
# AUTO takes, from 2^22 elements on), fill one, two, three, four, eight and sixteen waves; every number of stages
@pytest.mark.parametrize("T,d,b", [(70, 512, 16), (33, 1024, 32), (1457, 2880, 64), (11, 512, 128), (2051, 1536, 512), (1027, 3072, 256), (19, 1024, 1024),
                                   (7, 4096, 64), (9, 5120, 1024), (3, 6144, 2048), (4, 8192, 128), (3, 11264, 256), (2, 16384, 512), (2, 28672, 512), (2, 32768, 512)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4", "int4_asym", "fp4_token"])
def test_half_tile_kernel_at_the_edges_of_its_shapes(T, d, b, fmt):
    rng = np.random.default_rng(T + d + b)
    x = rng.standard_t(3, size=(T, d))
    x[:, rng.choice(d, size=max(1, d // 100), replace=False)] *= 50
    x[T // 2] *= 2.0 ** -115                                   # a row whose step leaves the usual range
    bits = synth.f64_to_bf16_bits(x)
    for perm in (None, rng.permutation(d).astype(np.int32)) if d % 512 == 0 else (None,):
        assert_parity(bits, perm, b, fmt, algo="mfma" if d % 512 == 0 else "auto", label="half tile")


# as above, in launches long enough for the run-time schedule (units of two and more to every workgroup) and its limit on
# waves, against launches of a few rows: (.., 14336, 64) is the other matrix-core kernel's from 2^26 elements on, same bits
@pytest.mark.parametrize("T,d,b,fmt,perms", [(70001, 512, 128, "int4", "ni"), (14001, 3072, 32, "int4_asym", "ni"), (2101, 14336, 64, "int4", "ni"), (1537, 16384, 64, "int4", "ni"),
                                             (50003, 1536, 512, "int4_asym", "ni"), (14001, 3072, 64, "mxfp4", "ni"),
                                             (9001, 4096, 512, "fp4_token", "nip"), (5003, 8192, 2048, "mxfp4", "nip"), (4001, 8192, 32, "int4", "nip"),
                                             (1501, 16384, 512, "int4", "nip"), (4701, 14336, 64, "int4", "ip"), (1101, 28672, 512, "mxfp4", "nip")])
def test_half_tile_kernel_long_and_short_launches_give_the_same_bits(T, d, b, fmt, perms):
    torch = _torch()
    print(f"[case] long and short T={T} d={d} b={b} fmt={fmt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(d + b)
    x = torch.randn((T, d), device="cuda", generator=g).to(torch.bfloat16)
    perm = torch.randperm(d, device="cuda", generator=g).to(torch.int32)
    form = binding.placement_to_device(binding.perq_perm_prepare(perm.cpu().numpy(), b)[0]) if "p" in perms else None
    for kind in perms:
        # (a prepared form is AUTO's, which these numbers of rows take to the matrix cores)
        p, how = None if kind == "n" else perm, {"placement": form} if kind == "p" else {"algo": "mfma"}
        codes, scales = binding.perq_permute_rotate_quant(x, p, b, fmt, **how)
        y, stats = binding.perq_permute_rotate_f32(x, p, b, algo="mfma"), binding.perq_block_diagnostics(x, p, b)
        for at in (slice(0, 3), slice(T // 2, T // 2 + 5), slice(T - 7, T)):
            c, s = binding.perq_permute_rotate_quant(x[at].contiguous(), p, b, fmt, algo="mfma")
            assert torch.equal(c, codes[at]) and torch.equal(s, scales[at]), (kind, at)
            assert torch.equal(binding.perq_permute_rotate_f32(x[at], p, b, algo="mfma"), y[at]), (kind, at)
            assert torch.equal(binding.perq_block_diagnostics(x[at], p, b), stats[at]), (kind, at)


# a permutation as given, launches of a unit to every workgroup that fits and of one less or more than that or than half of it:
# the same bits as in two calls, which have other workgroups
@pytest.mark.parametrize("T,d,b", [(1024, 4096, 32), (1025, 4096, 128), (2047, 4096, 64), (2048, 4096, 512), (2049, 4096, 32), (8193, 512, 128),
                                   (16384, 512, 128), (16389, 512, 32), (513, 8192, 128), (1024, 8192, 512), (512, 14336, 512), (257, 28672, 64)])
def test_half_tile_kernel_launches_of_one_unit_to_a_workgroup(T, d, b):
    torch = _torch()
    print(f"[case] one unit to a workgroup T={T} d={d} b={b}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + b)
    x = torch.randn((T, d), device="cuda", generator=g)
    x[:, torch.randperm(d, device="cuda", generator=g)[:max(1, d // 100)]] *= 1000.0        # (sums that round)
    x = x.to(torch.bfloat16)
    perm = torch.randperm(d, device="cuda", generator=g).to(torch.int32)
    calls = [lambda v, fmt=fmt: binding.perq_permute_rotate_quant(v, perm, b, fmt, algo="mfma") for fmt in ("int4", "mxfp4", "int4_asym")]
    calls += [lambda v: (binding.perq_permute_rotate_f32(v, perm, b, algo="mfma"),), lambda v: (binding.perq_block_diagnostics(v, perm, b),)]
    cut = T // 3
    for call in calls:
        for whole, head, tail in zip(call(x), call(x[:cut]), call(x[cut:])):
            assert torch.equal(whole[:cut], head) and torch.equal(whole[cut:], tail)


# the prepared form of rows wider than 8192 in launches of a unit or two to a workgroup: read, and the bits of the plain call
@pytest.mark.parametrize("T,d,b", [(520, 9728, 64), (600, 9728, 512), (513, 14336, 512), (700, 14336, 64), (100, 28672, 32), (257, 28672, 512), (64, 32768, 16)])
@pytest.mark.parametrize("fmt", ["int4", "mxfp4"])
def test_half_tile_kernel_reads_the_prepared_form_of_few_wide_rows(T, d, b, fmt):
    torch = _torch()
    print(f"[case] few wide rows, prepared T={T} d={d} b={b} fmt={fmt}", flush=True)
    rng = np.random.default_rng(T + d + b)
    x = binding.bits_to_device(synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, d))))
    perm = rng.permutation(d).astype(np.int32)
    perm_t = torch.from_numpy(perm).cuda()
    form, other = (binding.placement_to_device(binding.perq_perm_prepare(p, b)[0]) for p in (perm, np.roll(perm, 1)))
    want = binding.perq_permute_rotate_quant(x, perm_t, b, fmt, algo="mfma")
    got = binding.perq_permute_rotate_quant(x, perm_t, b, fmt, placement=form)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert not torch.equal(binding.perq_permute_rotate_quant(x, perm_t, b, fmt, placement=other)[0], want[0])


# ---- AUTO's line between the butterflies and the matrix cores ------------------------------------------
# The matrix unit cuts every term of a sum of eight off at half an ulp of the largest, which butterflies do not: below the line
# AUTO's outputs are the butterflies', bit for bit, and above it those of the matrix cores.  (T, d, b, pad, permutation, which):
# each class of the line from both sides where it has two, with rows that it never takes (widths below 2560 that do not pack
# into 4096, rows that lie apart), short rows through a permutation between 6.3 and 11 million elements, and one row.
@pytest.mark.parametrize("T,d,b,pad,perm,which", [
    (70, 64, 16, 0, True, "butterfly"), (333, 96, 32, 0, False, "butterfly"), (2051, 1536, 512, 0, False, "butterfly"),
    (2051, 1536, 256, 0, True, "butterfly"), (3001, 2048, 128, 64, True, "butterfly"), (5, 2048, 64, 0, False, "butterfly"),
    (6145, 1024, 32, 0, True, "butterfly"), (65536, 1024, 32, 0, True, "mfma"), (20155, 512, 16, 0, True, "butterfly"),
    (8191, 2048, 64, 0, False, "butterfly"), (8192, 2048, 64, 0, False, "mfma"), (512, 4096, 64, 0, True, "butterfly"),
    (513, 4096, 64, 0, True, "mfma"), (16, 4096, 128, 0, True, "butterfly"), (1023, 4096, 256, 0, False, "butterfly"),
    (1024, 4096, 256, 0, False, "mfma"), (2730, 3072, 128, 0, True, "butterfly"), (2731, 3072, 128, 0, True, "mfma"),
    (1024, 8192, 32, 0, True, "butterfly"), (2048, 8192, 32, 0, True, "mfma"), (1, 14336, 2048, 0, False, "butterfly"),
    (512, 14336, 512, 0, True, "butterfly"), (513, 14336, 512, 0, True, "mfma"), (256, 28672, 64, 0, False, "butterfly"),
    (257, 28672, 64, 0, False, "mfma"), (1, 28672, 64, 0, True, "mfma"), (1500, 2880, 64, 0, False, "mfma"),
    (1400, 2880, 64, 0, False, "butterfly"), (700, 11008, 256, 0, False, "butterfly"), (16, 8192, 4096, 0, False, "butterfly")])
def test_auto_takes_the_butterflies_below_its_line(T, d, b, pad, perm, which):
    torch = _torch()
    print(f"[case] line T={T} d={d} b={b} pad={pad} perm={perm} {which}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + b)
    x = torch.randn((T, d + pad), device="cuda", generator=g)
    x[:, torch.randperm(d, device="cuda", generator=g)[:max(1, d // 100)]] *= 1000.0        # (sums that round)
    x = x.to(torch.bfloat16)[:, :d]
    p = torch.randperm(d, device="cuda", generator=g).to(torch.int32) if perm else None
    y = binding.perq_permute_rotate_f32(x, p, b)
    butterflies = binding.perq_permute_rotate_f32(x, p, b, algo="butterfly")
    if which == "butterfly":
        assert torch.equal(y, butterflies)
    else:
        assert not torch.equal(y, butterflies)
        if d % 512 == 0:
            assert torch.equal(y, binding.perq_permute_rotate_f32(x, p, b, algo="mfma"))
    for fmt in ("int4", "mxfp4"):
        codes, scales = binding.perq_permute_rotate_quant(x, p, b, fmt)
        if which == "butterfly" or d % 512 == 0:
            c, s = binding.perq_permute_rotate_quant(x, p, b, fmt, algo=which)
            assert torch.equal(codes, c) and torch.equal(scales, s), fmt


# ---- the lines between the two matrix-core kernels: the same bits on either side ------------------------
# Up to b = 64 they form the same sums in the same order, so the number of rows may decide.  (T: the first number of rows that is
# mfma_kernel's for some format; rows of 2560 .. 4095, also of no multiple of 512, of no whole tile and of whole tiles past 8192.)
@pytest.mark.parametrize("T,d", [(39322, 2560), (34953, 2880), (32768, 3072), (28087, 3584), (4682, 14336), (2341, 28672), (1756, 28672), (10923, 12288), (8192, 16384)])
@pytest.mark.parametrize("b,fmt", [(16, "int4"), (32, "int4_asym"), (64, "fp4_token"), (32, "mxfp4")])
def test_the_same_bits_on_either_side_of_the_matrix_core_kernels_lines(T, d, b, fmt):
    torch = _torch()
    print(f"[case] same bits T={T} d={d} b={b} fmt={fmt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + b)
    x = torch.randn((T, d), device="cuda", generator=g)
    x[:, torch.randperm(d, device="cuda", generator=g)[:max(1, d // 100)]] *= 1000.0        # (sums that round)
    x = x.to(torch.bfloat16)
    perm = torch.randperm(d, device="cuda", generator=g).to(torch.int32)
    long = binding.perq_permute_rotate_quant(x, perm, b, fmt)
    short = binding.perq_permute_rotate_quant(x[:T - 1], perm, b, fmt)
    assert torch.equal(long[0][:-1], short[0]) and torch.equal(long[1][:-1], short[1])
    if d >= 4096:
        form = binding.placement_to_device(binding.perq_perm_prepare(perm.cpu().numpy(), b)[0])
        for n in (T - 1, T):
            codes, scales = binding.perq_permute_rotate_quant(x[:n], perm, b, fmt, placement=form)
            assert torch.equal(codes, long[0][:n]) and torch.equal(scales, long[1][:n])
    del long, short
    y = binding.perq_permute_rotate_f32(x, perm, b)
    assert torch.equal(y[:-1], binding.perq_permute_rotate_f32(x[:T - 1], perm, b))


# ---- how far the matrix cores' sums are from 64 bits -----------------------------------------------------
# perq.h gives the mean ratio to the butterflies' error by block size and the range of the means of a width; `most` is the top of the
# range.  Single inputs scatter further (b = 16: 1.0 to 3, few sums round at all), the mean of these 24 by a fifth of that.
@pytest.mark.parametrize("b,most", [(16, 1.36), (32, 1.03), (64, 1.24), (128, 1.08), (512, 1.08), (2048, 1.08)])
def test_error_of_the_matrix_cores_stays_where_the_header_has_it(b, most):
    torch = _torch()
    ratios = []
    for d in (4096, 8192, 14336):
        for seed in range(4):
            g = torch.Generator(device="cuda").manual_seed(d + b + 7 * seed)
            T = (1 << 23) // d
            x = torch.randn((T, d), device="cuda", generator=g)
            x /= torch.stack([torch.randn((T, d), device="cuda", generator=g) for _ in range(3)]).square().mean(dim=0).clamp(min=1e-6).sqrt()
            x[:, torch.randperm(d, device="cuda", generator=g)[:max(1, d // 100)]] *= 50.0
            x = x.clamp(-1e4, 1e4).to(torch.bfloat16)
            perm = torch.randperm(d, device="cuda", generator=g).to(torch.int32)
            for p in (None, perm):
                v = x.double() if p is None else x.double()[:, p.long()]
                h = 1
                while h < b:
                    v = v.reshape(-1, 2, h)
                    v = torch.stack((v[:, 0] + v[:, 1], v[:, 0] - v[:, 1]), dim=1)
                    h *= 2
                want = v.reshape(T, d) / b ** 0.5
                error = [float((binding.perq_permute_rotate_f32(x, p, b, algo=algo).double() - want).norm() / want.norm()) for algo in ("mfma", "butterfly")]
                print(f"[case] error d={d} b={b} perm={p is not None}: {error[0]:.3e}, butterflies {error[1]:.3e}", flush=True)
                # (each of log2(b) stages and the scale round to 2^-24 of a norm that they keep)
                assert error[0] < (math.log2(b) + 1) * 2.0 ** -24
                ratios.append(error[0] / error[1])
    print("       mean ratio", sum(ratios) / len(ratios), min(ratios), max(ratios), flush=True)
    assert sum(ratios) / len(ratios) <= most


# Blocks of 1024 and 2048 that begin with their largest channels, as the calibrated permutations fill them: the matrix cores contract
# the middle bits of a position first, so large values meet in four roundings where the butterflies round them eleven times.  (Ratio of the
# two errors of a row's step 0.82 - 0.91 over such inputs; a root mean square over T >= 512 rows scatters by 1 / sqrt(2 T), 3 % at most.)
@pytest.mark.parametrize("d,b", [(2048, 1024), (4096, 2048), (5120, 1024), (6144, 2048), (7168, 1024), (8192, 1024), (8192, 2048), (14336, 2048)])
def test_large_blocks_that_begin_with_their_largest_channels(d, b):
    torch = _torch()
    T = (1 << 24) // d
    g = torch.Generator(device="cuda").manual_seed(d + b)
    x = torch.randn((T, d), device="cuda", generator=g)
    x /= torch.stack([torch.randn((T, d), device="cuda", generator=g) for _ in range(3)]).square().mean(dim=0).clamp(min=1e-6).sqrt()
    x[:, torch.randperm(d, device="cuda", generator=g)[:max(1, d // 100)]] *= 50.0
    x = x.clamp(-1e4, 1e4).to(torch.bfloat16)
    perm = binding.perq_massdiff_perm(binding.perq_colabs_mean(x).cpu().numpy(), b)
    p = torch.from_numpy(perm).cuda()
    v, h = x.double()[:, p.long()], 1
    while h < b:
        v = v.reshape(-1, 2, h)
        v = torch.stack((v[:, 0] + v[:, 1], v[:, 0] - v[:, 1]), dim=1)
        h *= 2
    want = v.reshape(T, d).abs().amax(dim=1) / b ** 0.5 / 7.0
    error = {}
    for algo in ("auto", "mfma", "butterfly"):
        step = binding.perq_permute_rotate_quant(x, p, b, "int4", algo=algo)[1]
        error[algo] = float((((step.double() - want) / want) ** 2).mean() ** 0.5)
    print(f"[case] largest first d={d} b={b}: {error}", flush=True)
    assert error["auto"] == error["mfma"] <= 1.03 * 0.91 * error["butterfly"]


# d = b = 1024 with a permutation: four rows to a 4096-wide one for MXFP4 and fp32 output, one to a tile for the formats with a step
# per token, rows left over and rows that lie apart; one kernel by name for all of them
@pytest.mark.parametrize("T,pad", [(1, 0), (3, 0), (4, 0), (5, 0), (1027, 0), (9, 64)])
def test_rows_of_one_block_of_1024_folded_and_not(T, pad):
    torch = _torch()
    rng = np.random.default_rng(T + pad)
    bits = synth.f64_to_bf16_bits(rng.standard_t(4, size=(T, 1024)))
    perm = rng.permutation(1024).astype(np.int32)
    for fmt in ("int4", "mxfp4", "int4_asym", "fp4_token"):
        assert_parity(bits, perm, 1024, fmt, algo="mfma", ldx=1024 + pad if pad else None, label="one block of 1024")
    x, p = binding.bits_to_device(bits), torch.from_numpy(perm).cuda()
    y = binding.perq_permute_rotate_f32(x, p, 1024, algo="mfma")
    assert torch.equal(binding.perq_permute_rotate_f32(x[T // 2:], p, 1024, algo="mfma"), y[T // 2:])
    if T >= 4:
        assert torch.equal(binding.perq_permute_rotate_f32(x, p, 1024), y) and torch.equal(*(binding.perq_permute_rotate_quant(x, p, 1024, "mxfp4", algo=a)[0] for a in ("auto", "mfma")))


# ---- outputs under a mode of the dispatcher ---------------------------------------------------------------
def test_a_mode_of_the_dispatcher_sees_the_buffers_of_a_call():
    torch = _torch()
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        def __init__(self):
            super().__init__()
            self.ops = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.ops.append(str(func))
            return func(*args, **(kwargs or {}))

    x = torch.randn((40, 512), device="cuda").to(torch.bfloat16)
    want = binding.perq_permute_rotate_quant(x, None, 32, "int4")
    with Seen() as seen:
        got = binding.perq_permute_rotate_quant(x, None, 32, "int4")
        stats = binding.perq_block_diagnostics(x, None, 32)
    assert seen.ops.count("aten.empty.memory_format") == 3, seen.ops
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(stats, binding.perq_block_diagnostics(x, None, 32))
    traced = torch.jit.trace(lambda t: binding.perq_permute_rotate_quant(t, None, 32, "int4")[0], x, check_trace=False)
    assert "aten::empty" in str(traced.graph)
