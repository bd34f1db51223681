"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the same seeded inputs.

Quantization, packing and dequantization must match bit for bit.  The product must satisfy, per
element, |Y_gpu - Y_ref| <= 1e-5 * sum_b |term_b| (the fp32 accumulation over blocks may run in any
order; the block terms themselves are exact) and ||Y_gpu - Y_ref||_F <= 1e-5 * ||Y_ref||_F.
"""
import numpy as np
import pytest
import torch

from oracle import mx_oracle as orc
from paper_2307_15517_amd import inputs, mx

pytestmark = pytest.mark.gpu
MAT_LAYOUT = mx.MX_LAYOUT_MATRIX

DEV = "cuda:0"
TOL = 1e-5
F32_TINY = 2.0 ** -149        # one fp32 subnormal step: the output grid itself


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    return t.detach().cpu().numpy()


def say(*a):
    print(*a, flush=True)


# ----------------------------------------------------------------------------------------------
def quantize_gpu(x, block, w, e=8, rounding=mx.MX_RNE, axis=1):
    f = mx.fmt(block, w, e, rounding)
    mant, exps = mx.quantize(dev(x), f, axis)
    torch.cuda.synchronize()
    return host(mant), host(exps)


def check_quantize(x, block, w, e=8, rounding=mx.MX_RNE, axis=1):
    q, ex = orc.quantize(x, block, w, e, rounding, axis)
    want_m = orc.pack_bits(q, w).reshape(-1)
    mant, exps = quantize_gpu(x, block, w, e, rounding, axis)
    assert np.array_equal(exps, ex.reshape(-1)), "exponent bytes differ"
    assert np.array_equal(mant, want_m), "mantissa bytes differ"


def special_values(rng, rows, cols):
    """Zeros, subnormals, huge and tiny magnitudes, exact ties, saturating maxima."""
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    x *= np.exp2(rng.integers(-12, 12, size=(rows, 1))).astype(np.float32)
    flat = x.reshape(-1)
    n = flat.size
    idx = rng.permutation(n)
    k = n // 16
    flat[idx[:k]] = 0.0
    flat[idx[k:2 * k]] = (rng.integers(-64, 65, size=k) * 0.5).astype(np.float32)          # ties
    flat[idx[2 * k:3 * k]] = np.float32(1.9999999) * np.exp2(rng.integers(-3, 3, size=k))  # saturate
    x[0, :] = 0.0                                                                            # zero blocks
    if rows > 2:
        x[1, :] = (rng.standard_normal(cols) * 1e-41).astype(np.float32)                     # subnormals
        x[2, :] = (rng.standard_normal(cols) * 1e37).astype(np.float32)                      # near fp32 max
    if rows > 4:
        x[3, :] = (rng.standard_normal(cols) * 2e-38).astype(np.float32)                     # around 2^-126
        x[4, ::3] = np.float32(2.0 ** -149)
    return x


@pytest.mark.parametrize("w", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("block", [8, 16, 32, 64])
def test_quantize_bit_exact_all_formats(w, block):
    rng = np.random.default_rng(1000 * w + block)
    say("quantize w", w, "block", block)
    x = special_values(rng, 37, 5 * 64)                 # 37 rows: ragged tail of the last wave
    for rounding in (mx.MX_RNE, mx.MX_RTZ):
        check_quantize(x, block, w, 8, rounding)
    check_quantize(x[:5], block, w, 4)                  # narrow exponent: clamps both ways
    check_quantize(x[:5], block, w, 2)


def test_quantize_strided_rows_and_batch():
    rng = np.random.default_rng(5)
    big = special_values(rng, 3 * 24, 256 + 64)
    f = mx.fmt(32, 6)
    xb = dev(big).reshape(3, 24, 320)[:, :17, :256]      # batch 3, 17 rows of 256 inside padded storage
    mant = torch.empty(mx.mx_mant_bytes(3, 17, 256, f), dtype=torch.uint8, device=DEV)
    exps = torch.empty(mx.mx_exps_bytes(3, 17, 256, f), dtype=torch.uint8, device=DEV)
    mx.mx_quantize(xb, 3, 17, 256, xb.stride(1), xb.stride(0), 1, f, mant, exps)
    torch.cuda.synchronize()
    xs = big.reshape(3, 24, 320)[:, :17, :256].reshape(-1, 256)
    q, ex = orc.quantize(xs, 32, 6)
    assert np.array_equal(host(exps), ex.reshape(-1))
    assert np.array_equal(host(mant), orc.pack_bits(q, 6).reshape(-1))
    # a 4-byte aligned but not 16-byte aligned base pointer
    flat = dev(np.concatenate([np.zeros(1, np.float32), big[:8, :256].reshape(-1)]))
    mant2 = torch.empty(mx.mx_mant_bytes(1, 8, 256, f), dtype=torch.uint8, device=DEV)
    exps2 = torch.empty(mx.mx_exps_bytes(1, 8, 256, f), dtype=torch.uint8, device=DEV)
    mx.mx_quantize(flat.data_ptr() + 4, 1, 8, 256, 256, 0, 1, f, mant2, exps2)
    torch.cuda.synchronize()
    q, ex = orc.quantize(big[:8, :256], 32, 6)
    assert np.array_equal(host(exps2), ex.reshape(-1))
    assert np.array_equal(host(mant2), orc.pack_bits(q, 6).reshape(-1))


@pytest.mark.parametrize("block,w", [(16, 4), (16, 8), (32, 5), (8, 3), (64, 6)])
def test_quantize_axis0(block, w):
    rng = np.random.default_rng(77 + w)
    x = special_values(rng, 4 * 64, 131)                 # 131 columns: ragged
    check_quantize(x, block, w, axis=0)


@pytest.mark.parametrize("block,w,cols", [(16, 4, 130), (16, 8, 32), (32, 5, 66), (8, 3, 2), (64, 6, 34)])
def test_quantize_axis0_two_row_blocks(block, w, cols):
    """Blocks of (block rows of x, 2 columns): the canonical form of the transposed matrix with two-row blocks."""
    rng = np.random.default_rng(177 + w)
    x = special_values(rng, 5 * 64, cols)                # 320 rows: two row tiles of the kernel, the second ragged
    x[:, 1::2] *= np.exp2(rng.integers(-6, 1, size=(1, cols // 2))).astype(np.float32)   # neighbours of unequal size
    for rounding in (mx.MX_RNE, mx.MX_RTZ):
        f = mx.fmt(block, w, 8, rounding, block_rows=2)
        mant, exps = mx.quantize(dev(x), f, axis=0)
        torch.cuda.synchronize()
        q, ex = orc.quantize(np.ascontiguousarray(x.T), block, w, 8, rounding, block_rows=2)
        assert np.array_equal(host(exps), ex.reshape(-1)), "exponent bytes differ"
        assert np.array_equal(host(mant), orc.pack_bits(q, w).reshape(-1)), "mantissa bytes differ"


def test_quantize_workload_shapes():
    """The activation tensors of the LLM-shaped workloads at full size."""
    for case in inputs.single_linear() + inputs.opt125m_layer() + inputs.llama7b_prefill()[:1] + \
            inputs.llama13b_decode(8)[:2]:
        say("quantize", case.name)
        x, wt = inputs.make(case)
        check_quantize(x, case.block, case.wx)
        check_quantize(wt[:512], case.block, case.ww)


def test_quantize_and_dequantize_beyond_32_bit_offsets():
    """2^31 + 2^21 elements (8.6 GB of fp32 in, 2.1 GB of mantissas out): element and byte offsets that do not fit
    32 bits.  The input is one seeded tile of 256 rows repeated down the tensor, so every repetition must come out
    as the tile's own quantization, which is checked against the oracle."""
    rng = np.random.default_rng(31)
    cols, tile_rows = 8192, 256
    reps = 2 ** 31 // (cols * tile_rows) + 1
    tile = (rng.standard_normal((tile_rows, cols)) * np.exp2(rng.integers(-8, 8, size=(tile_rows, 1)))).astype(np.float32)
    f = mx.fmt(32, 8)
    td = dev(tile)
    m_tile, e_tile = mx.quantize(td, f)
    q, ex = orc.quantize(tile, 32, 8)
    assert np.array_equal(host(e_tile), ex.reshape(-1)) and np.array_equal(host(m_tile), orc.pack_bits(q, 8).reshape(-1))
    xd = td.repeat(reps, 1)
    assert xd.numel() > 2 ** 31
    mant, exps = mx.quantize(xd, f)
    torch.cuda.synchronize()
    assert bool((mant.view(reps, -1) == m_tile.view(1, -1)).all()), "mantissas of a repetition differ"
    assert bool((exps.view(reps, -1) == e_tile.view(1, -1)).all()), "exponents of a repetition differ"
    y = mx.dequantize(mant, exps, 1, reps * tile_rows, cols, f)
    y_tile = mx.dequantize(m_tile, e_tile, 1, tile_rows, cols, f)
    torch.cuda.synchronize()
    assert np.array_equal(host(y_tile)[0].astype(np.float64), orc.dequantize(q, ex, 32, 8))
    assert bool((y.view(reps, -1) == y_tile.view(1, -1)).all()), "values of a repetition differ"
    del xd, mant, exps, y
    torch.cuda.empty_cache()


def test_quantize_is_deterministic_and_ignores_stale_output():
    rng = np.random.default_rng(6)
    x = dev(special_values(rng, 64, 1024))
    f = mx.fmt(32, 8)
    a = mx.quantize(x, f)
    b = mx.quantize(x, f)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("block,w", [(8, 2), (16, 4), (32, 8), (64, 7), (16, 3), (32, 6), (16, 5)])
def test_dequantize_exact(block, w):
    rng = np.random.default_rng(w * 10 + block)
    rows, cols = 19, 4 * 64
    q = rng.integers(-(2 ** (w - 1)), 2 ** (w - 1), size=(rows, cols)).astype(np.int8)   # incl. the unused code
    ex = rng.integers(0, 248, size=(rows, cols // block)).astype(np.uint8)   # values stay below fp32 max
    f = mx.fmt(block, w)
    y = mx.dequantize(dev(orc.pack_bits(q, w).reshape(-1)), dev(ex.reshape(-1)), 1, rows, cols, f)
    torch.cuda.synchronize()
    want = orc.dequantize(q, ex, block, w)
    got = host(y)[0].astype(np.float64)
    exact = np.abs(want) >= 2.0 ** -149
    assert np.array_equal(got[exact], want[exact])
    assert np.all(np.abs(got[~exact] - want[~exact]) <= 2.0 ** -149)


@pytest.mark.parametrize("block,w", [(16, 4), (16, 8), (32, 4), (32, 8), (64, 4), (16, 6), (32, 3), (64, 7),
                                     (16, 2), (16, 5), (32, 7)])
def test_pack_unpack_roundtrip(block, w):
    rng = np.random.default_rng(block + w)
    f = mx.fmt(block, w)
    for rows, cols in [(33, 5 * block), (64, 8 * block), (1, block)]:
        mant = rng.integers(0, 256, size=mx.mx_mant_bytes(2, rows, cols, f)).astype(np.uint8)
        exps = rng.integers(0, 256, size=mx.mx_exps_bytes(2, rows, cols, f)).astype(np.uint8)
        packed = mx.pack(dev(mant), dev(exps), 2, rows, cols, f)
        m2, e2 = mx.unpack(packed, 2, rows, cols, f)
        torch.cuda.synchronize()
        assert np.array_equal(host(m2), mant) and np.array_equal(host(e2), exps)


# ----------------------------------------------------------------------------------------------
# Two-row blocks: the paper's block shape (block, 2), e.g. MXInt((16,2),8,7)
# ----------------------------------------------------------------------------------------------
@pytest.mark.parametrize("block", [8, 16, 32, 64])
def test_quantize_two_row_blocks_bit_exact(block):
    rng = np.random.default_rng(700 + block)
    for w in range(2, 9):
        f = mx.fmt(block, w, 8, mx.MX_RNE if w % 2 else mx.MX_RTZ, block_rows=2)
        x = special_values(rng, 2 * 34, 3 * 64).reshape(2, 34, 3 * 64)
        q, ex = zip(*(orc.quantize(x[b], block, w, 8, f.rounding, block_rows=2) for b in range(2)))
        mant, exps = mx.quantize(dev(x), f)
        torch.cuda.synchronize()
        assert exps.numel() == 2 * 17 * (3 * 64 // block)
        assert np.array_equal(host(exps), np.stack(ex).reshape(-1)), "exponent bytes differ"
        assert np.array_equal(host(mant), np.stack([orc.pack_bits(qq, w) for qq in q]).reshape(-1)), "mantissa bytes differ"
        # and back: the same values as the oracle's, both rows of a pair reading the pair's exponent
        y = mx.dequantize(mant, exps, 2, 34, 3 * 64, f)
        torch.cuda.synchronize()
        ref = np.stack([orc.dequantize(q[b], orc.row_exps(ex[b], 2), block, w) for b in range(2)])
        fine = np.abs(ref) >= 2.0 ** -126           # below that fp32 itself rounds
        assert np.array_equal(host(y).astype(np.float64)[fine], ref[fine])
    # strided rows
    f = mx.fmt(block, 8, block_rows=2)
    big = rng.standard_normal((20, 4 * 64 + 8)).astype(np.float32)
    xd = dev(big)
    mant = torch.empty(mx.mx_mant_bytes(1, 20, 4 * 64, f), dtype=torch.uint8, device=DEV)
    exps = torch.empty(mx.mx_exps_bytes(1, 20, 4 * 64, f), dtype=torch.uint8, device=DEV)
    mx.mx_quantize(xd, 1, 20, 4 * 64, 4 * 64 + 8, 0, 1, f, mant, exps)
    q, ex = orc.quantize(big[:, :4 * 64], block, 8, block_rows=2)
    torch.cuda.synchronize()
    assert np.array_equal(host(mant), orc.pack_bits(q, 8).reshape(-1)) and np.array_equal(host(exps), ex.reshape(-1))


@pytest.mark.parametrize("layout", [mx.MX_LAYOUT_FRAGMENT, mx.MX_LAYOUT_MATRIX])
@pytest.mark.parametrize("block,w", [(16, 8), (16, 4), (16, 5), (32, 8), (32, 4), (64, 6)])
def test_two_row_blocks_pack_roundtrip_and_fused(layout, block, w):
    rng = np.random.default_rng(720 + block + w)
    f = mx.fmt(block, w, block_rows=2)
    for batch, rows, cols in [(1, 70, 5 * 64), (2, 34, 8 * 64), (1, 256, 1024)]:
        x = (rng.standard_normal((batch, rows, cols)) * np.exp2(rng.integers(-6, 6, size=(batch, rows, 1)))).astype(np.float32)
        xd = dev(x)
        mant, exps = mx.quantize(xd, f)
        n = mx.mx_packed_bytes(batch, rows, cols, f, layout)
        packed = torch.zeros(n, dtype=torch.uint8, device=DEV)       # zeroed: the layouts leave their tail padding alone
        fused = torch.zeros(n, dtype=torch.uint8, device=DEV)
        mx.mx_pack(mant, exps, batch, rows, cols, f, layout, packed)
        m2, e2 = mx.unpack(packed, batch, rows, cols, f, layout)
        mx.mx_quantize_pack(xd, batch, rows, cols, cols, rows * cols, f, layout, fused)
        torch.cuda.synchronize()
        assert torch.equal(m2, mant) and torch.equal(e2, exps), "pack/unpack round trip"
        assert torch.equal(fused, packed), "fused quantize+pack differs from quantize, then pack"


def test_paper_type_linear_two_row_blocks():
    """The paper's own types on a linear layer (Fig. 2b): activations MXInt((16,2),8,7), weights
    MXInt((16,2),8,3), on both layouts; the product kernels see per-row exponents and do not change."""
    case = inputs.opt125m_layer()[2]
    x, wt = inputs.make(case)
    fa, fb = mx.fmt(16, 8, block_rows=2), mx.fmt(16, 4, block_rows=2)
    qa, ea = orc.quantize(x, 16, 8, block_rows=2)
    qb, eb = orc.quantize(wt, 16, 4, block_rows=2)
    y_ref, mag = orc.gemm(qa, orc.row_exps(ea, 2), 8, qb, orc.row_exps(eb, 2), 4, 16, want_mag=True)
    for layout in (mx.MX_LAYOUT_FRAGMENT, MAT_LAYOUT):
        A = mx.quantize_pack(dev(x), fa, layout)
        B = mx.quantize_pack(dev(wt), fb, layout)
        y = mx.gemm(A, fa, B, fb, case.M, case.N, case.K, layout=layout)
        torch.cuda.synchronize()
        say("two-row blocks, layout", layout, "worst", check_product(host(y)[0], y_ref, mag, "paper types"))


def test_two_row_blocks_rejections():
    f2 = mx.fmt(16, 8, block_rows=2)
    buf = torch.zeros(1 << 16, dtype=torch.uint8, device=DEV)
    xf = torch.zeros((8, 64), dtype=torch.float32, device=DEV)
    out = torch.zeros(1 << 16, dtype=torch.uint8, device=DEV)
    assert mx.mx_quantize(xf, 1, 7, 64, 64, 0, 1, f2, buf, out, check=False) == mx.MX_ERR_BAD_ARG          # odd rows
    assert mx.mx_quantize(xf, 1, 32, 15, 16, 0, 0, f2, buf, out, check=False) == mx.MX_ERR_BAD_ARG         # along the rows: odd columns
    assert mx.mx_cast(buf, buf, 1, 8, 64, f2, mx.fmt(16, 4), out, out, check=False) == mx.MX_ERR_BAD_ARG                     # block_rows differ
    assert mx.mx_quantize(xf, 1, 8, 64, 64, 0, 1, mx.fmt(16, 8, block_rows=3), buf, out, check=False) == mx.MX_ERR_BAD_ARG
    y = torch.zeros((2, 64), dtype=torch.float32, device=DEV)
    assert mx.mx_linear(xf, 1, 64, 64, f2, buf, buf, 64, mx.fmt(16, 4), mx.MX_LAYOUT_FRAGMENT, y, 64,
                        check=False) == mx.MX_ERR_BAD_ARG                                                  # odd rows
    assert mx.mx_exps_bytes(1, 8, 64, f2) == 4 * 4 and mx.mx_exps_bytes(1, 7, 64, f2) == 0


# ----------------------------------------------------------------------------------------------
# Width cast inside the format (bit-exact against the oracle's integer cast)
# ----------------------------------------------------------------------------------------------
def check_cast(q, ex, block, ws, wd, es=8, ed=8, rounding=mx.MX_RNE, batch=1, block_rows=1):
    rows, cols = q.shape[-2], q.shape[-1]
    q2 = q.reshape(-1, cols)
    want_q, want_e = orc.cast(q2, ex.reshape(-1, cols // block), block, ws, wd, es, ed, rounding, block_rows=block_rows)
    fs, fd = mx.fmt(block, ws, es, block_rows=block_rows), mx.fmt(block, wd, ed, rounding, block_rows=block_rows)
    mant = dev(orc.pack_bits(q2, ws).reshape(-1))
    got_m, got_e = mx.cast(mant, dev(ex.reshape(-1)), batch, rows, cols, fs, fd)
    torch.cuda.synchronize()
    assert np.array_equal(host(got_e), want_e.reshape(-1)), "exponent bytes differ"
    assert np.array_equal(host(got_m), orc.pack_bits(want_q, wd).reshape(-1)), "mantissa bytes differ"


@pytest.mark.parametrize("block", [8, 16, 32, 64])
def test_cast_all_width_pairs(block):
    rng = np.random.default_rng(900 + block)
    for ws in range(2, 9):
        for wd in range(2, 9):
            rows, cols = 37, 5 * 64 + (block if block < 32 else 0)      # for small blocks the tensor ends inside a 32-element run
            q = rng.integers(-(2 ** (ws - 1)), 2 ** (ws - 1), size=(rows, cols)).astype(np.int8)   # every code
            q[::4] //= 8                                                # blocks that are not normalised
            q[3] = 0                                                    # zero blocks
            ex = rng.integers(0, 256, size=(rows, cols // block)).astype(np.uint8)
            check_cast(q, ex, block, ws, wd, rounding=mx.MX_RNE if (ws + wd) % 2 else mx.MX_RTZ)


def test_cast_exponent_widths_batch_and_workload_shape():
    rng = np.random.default_rng(950)
    # narrower and wider exponent fields: clamping on the way down, rebasing on the way up
    for es, ed in [(8, 4), (4, 8), (8, 2), (5, 7)]:
        q = rng.integers(-127, 128, size=(2 * 20, 256)).astype(np.int8)
        ex = rng.integers(0, 2 ** es, size=(2 * 20, 256 // 32)).astype(np.uint8)
        check_cast(q.reshape(2, 20, 256), ex, 32, 8, 4, es, ed, batch=2)
    # the prefill activations: 8-bit quantizer output narrowed to 4 bits, and widened back
    case = inputs.llama7b_prefill()[0]
    x, _ = inputs.make(case, 512)
    q8, e8 = orc.quantize(x, case.block, 8)
    check_cast(q8, e8, case.block, 8, 4)
    q4, e4 = orc.cast(q8, e8, case.block, 8, 4)
    check_cast(q4, e4, case.block, 4, 8)
    # cast of the quantizer's own output on the GPU equals quantizing to the narrow format's grid of the wide values
    f8, f4 = mx.fmt(case.block, 8), mx.fmt(case.block, 4)
    m8, x8 = mx.quantize(dev(x), f8)
    m4, x4 = mx.cast(m8, x8, 1, x.shape[0], x.shape[1], f8, f4)
    torch.cuda.synchronize()
    assert np.array_equal(host(m4), orc.pack_bits(q4, 4).reshape(-1)) and np.array_equal(host(x4), e4.reshape(-1))


@pytest.mark.parametrize("block", [8, 16, 32, 64])
def test_cast_two_row_blocks(block):
    rng = np.random.default_rng(960 + block)
    for ws, wd in [(8, 4), (4, 8), (6, 3), (3, 7), (5, 5), (8, 8), (2, 2)]:
        rows, cols = 2 * 19, (6 * 64 if block == 64 else 5 * 64 + 32)
        q = rng.integers(-(2 ** (ws - 1)), 2 ** (ws - 1), size=(2, rows, cols)).astype(np.int8)
        q[:, ::4] //= 8
        q[:, 6:8] = 0
        ex = rng.integers(0, 256, size=(2, rows // 2, cols // block)).astype(np.uint8)
        check_cast(q, ex, block, ws, wd, rounding=mx.MX_RTZ if ws == 6 else mx.MX_RNE, batch=2, block_rows=2)


@pytest.mark.parametrize("block,cols", [(8, 40), (16, 48), (16, 16), (8, 8), (16, 5 * 16)])
def test_cast_two_row_blocks_any_column_count(block, cols):
    """Two-row blocks whose rows are not whole runs of 32 elements: all 49 width pairs, both roundings."""
    rng = np.random.default_rng(970 + cols)
    rows = 2 * 7
    for ws in range(2, 9):
        q = rng.integers(-(2 ** (ws - 1)), 2 ** (ws - 1), size=(2, rows, cols)).astype(np.int8)
        q[:, ::4] //= 8
        q[:, 6:8] = 0
        ex = rng.integers(0, 256, size=(2, rows // 2, cols // block)).astype(np.uint8)
        for wd in range(2, 9):
            check_cast(q, ex, block, ws, wd, rounding=mx.MX_RTZ if (ws + wd) % 3 == 0 else mx.MX_RNE, batch=2, block_rows=2)
    check_cast(q, ex, block, 8, 4, es=8, ed=4, batch=2, block_rows=2)        # exponent clamped both ways


def test_cast_rejects_bad_arguments():
    f8, f4 = mx.fmt(32, 8), mx.fmt(32, 4)
    buf = torch.zeros(4096, dtype=torch.uint8, device=DEV)
    out = torch.zeros(4096, dtype=torch.uint8, device=DEV)
    assert mx.mx_cast(buf, buf, 1, 4, 64, f8, mx.fmt(16, 4), out, out, check=False) == mx.MX_ERR_BAD_ARG   # block differs
    assert mx.mx_cast(buf, buf, 1, 4, 64, f8, f4, buf, out, check=False) == mx.MX_ERR_BAD_ARG               # in place
    assert mx.mx_cast(buf, buf, 1, 4, 48, f8, f4, out, out, check=False) == mx.MX_ERR_BAD_ARG               # cols % block
    assert mx.mx_cast(buf, buf, 0, 4, 64, f8, f4, out, out, check=False) == mx.MX_OK                        # empty


# ----------------------------------------------------------------------------------------------
def gpu_operand(q, ex, block, w, batch=1, layout=mx.MX_LAYOUT_FRAGMENT):
    f = mx.fmt(block, w)
    rows, cols = q.shape[-2], q.shape[-1]
    mant = dev(orc.pack_bits(q.reshape(-1, cols), w).reshape(-1))
    return mx.pack(mant, dev(ex.reshape(-1)), batch, rows, cols, f, layout), f


def product_magnitude(qa, ea, wa, qb, eb, wb, block):
    """sum_k |qa_k * qb_k| * 2^(block exponents): the size of the individual products (numpy only)."""
    M, K = qa.shape
    N = qb.shape[0]
    nb = K // block
    a = np.abs(qa.astype(np.float64)).reshape(M, nb, block) * np.ldexp(1.0, ea.astype(int) - 127 - (wa - 2))[:, :, None]
    b = np.abs(qb.astype(np.float64)).reshape(N, nb, block) * np.ldexp(1.0, eb.astype(int) - 127 - (wb - 2))[:, :, None]
    return a.reshape(M, K) @ b.reshape(N, K).T


def check_product(y_gpu, y_ref, mag, what="", mag_elem=None):
    """|err| <= 1e-5 * sum_b |term_b|.  With mag_elem (matrix-core layout on adversarial exponent
    spreads only) the bound gains 1e-6 * sum_k |product_k|: that path's accumulator keeps 24 bits below
    the largest single product of an instruction, not below the block sums."""
    y_gpu = y_gpu.astype(np.float64)
    err = np.abs(y_gpu - y_ref)
    bound = TOL * mag + F32_TINY
    if mag_elem is not None:
        bound = bound + 1e-6 * mag_elem
    worst = float((err / np.maximum(mag, 1e-300)).max()) if err.size else 0.0
    assert np.all(err <= bound), "%s: worst element error %.3g of sum|terms|" % (what, worst)
    ref_norm = np.linalg.norm(y_ref)
    if ref_norm > 0 and mag_elem is None:
        assert np.linalg.norm(y_gpu - y_ref) <= TOL * ref_norm + F32_TINY, what
    return worst


def run_case(case, M=None, rows=None, layout=mx.MX_LAYOUT_FRAGMENT, fused=False):
    """Quantize on the GPU (checked bit-exact elsewhere), pack, multiply; compare with the oracle
    applied to the same fp32 inputs.  rows=(a,b): only that row window is computed by the oracle.
    fused: the activations go through mx_quantize_pack (the path the benchmark times)."""
    x, wt = inputs.make(case, M)
    m = x.shape[0]
    fa, fb = mx.fmt(case.block, case.wx), mx.fmt(case.block, case.ww)
    if fused:
        A = mx.quantize_pack(dev(x), fa, layout)
    else:
        am, ae = mx.quantize(dev(x), fa)
        A = mx.pack(am, ae, 1, m, case.K, fa, layout)
    bm, be = mx.quantize(dev(wt), fb)
    B = mx.pack(bm, be, 1, case.N, case.K, fb, layout)
    y = mx.gemm(A, fa, B, fb, m, case.N, case.K, layout=layout)
    torch.cuda.synchronize()
    qa, ea = orc.quantize(x, case.block, case.wx)
    qb, eb = orc.quantize(wt, case.block, case.ww)
    r0, r1 = (0, m) if rows is None else rows
    y_ref, mag = orc.gemm(qa, ea, case.wx, qb, eb, case.ww, case.block, rows=(r0, r1), want_mag=True)
    return check_product(host(y)[0][r0:r1], y_ref[r0:r1], mag[r0:r1], case.name)


def test_gemm_single_linear_full():
    for case in inputs.single_linear():
        say("gemm", case.name, "worst", run_case(case))


def test_gemm_opt125m_layer_full():
    for case in inputs.opt125m_layer():
        say("gemm", case.name, "worst", run_case(case))


def test_gemm_llama7b_reduced_m256_full_output():
    case = inputs.llama7b_prefill()[0]
    say("gemm", case.name, "M=256 worst", run_case(case, M=256))


@pytest.mark.parametrize("idx", [0, 1, 2])
def test_gemm_llama7b_full_size_sampled_rows(idx):
    case = inputs.llama7b_prefill()[idx]
    # the int8 path at M = 2048 (a slow kernel at this size); the oracle computes a 256-row window
    say("gemm", case.name, "rows 900..1156 worst", run_case(case, rows=(900, 1156)))


@pytest.mark.parametrize("M", [1, 4, 8])
def test_gemv_llama13b_decode_full(M):
    for case in inputs.llama13b_decode(M):
        say("gemv", case.name, "M", M, "worst", run_case(case))


@pytest.mark.parametrize("M", [1, 2, 3, 8])
def test_linear_against_oracle_and_the_three_call_chain(M):
    """mx_linear (one launch, K slices added in slice order) against the oracle on the whole output, against
    quantize + pack + product (same block terms, another order of the fp32 additions), twice for the same bits,
    and with the workspace's counters left at zero."""
    case = inputs.llama13b_decode(M)[0]
    x, wt = inputs.make(case)
    fa, fb = mx.fmt(case.block, case.wx), mx.fmt(case.block, case.ww)
    bm, be = mx.quantize(dev(wt), fb)
    B = mx.pack(bm, be, 1, case.N, case.K, fb)
    xd = dev(x)
    am, ae = mx.quantize(xd, fa)
    A = mx.pack(am, ae, 1, M, case.K, fa)
    y1 = mx.gemm(A, fa, B, fb, M, case.N, case.K)[0]
    scratch = mx.linear_workspace(M, case.K, case.N, fa, fb, DEV)
    y2 = torch.full((M, case.N), 3.0, dtype=torch.float32, device=DEV)
    y3 = torch.full((M, case.N), 5.0, dtype=torch.float32, device=DEV)
    mx.mx_linear(xd, M, case.K, case.K, fa, scratch, B, case.N, fb, mx.MX_LAYOUT_FRAGMENT, y2, case.N)
    mx.mx_linear(xd, M, case.K, case.K, fa, scratch, B, case.N, fb, mx.MX_LAYOUT_FRAGMENT, y3, case.N)
    torch.cuda.synchronize()
    assert torch.equal(y2, y3)            # the sum over the slices has a fixed order: identical bits
    assert int(scratch[:16384].max()) == 0
    y_ref, mag = orc.linear(x, wt, case.block, case.wx, case.ww, want_mag=True)
    check_product(host(y2), y_ref, mag, "linear M %d" % M)
    assert np.all(np.abs(host(y1).astype(np.float64) - host(y2)) <= 2e-5 * mag + 2.0 ** -149)


@pytest.mark.parametrize("block,wx,ww,M,e,rounding", [(16, 5, 4, 5, 8, mx.MX_RNE), (32, 2, 8, 8, 8, mx.MX_RTZ),
                                                       (64, 8, 3, 3, 5, mx.MX_RNE), (16, 7, 6, 4, 4, mx.MX_RTZ)])
def test_linear_rows_3_to_8_formats_and_alignment(block, wx, ww, M, e, rounding):
    """mx_linear for 3..8 rows over block sizes, widths, narrow exponents and truncation, with K not a whole
    number of chunks, for rows that are 16-byte aligned (one launch) and rows that are not (quantize, then the
    decode product: identical bits to quantize + pack + product)."""
    rng = np.random.default_rng(block * 100 + wx)
    K, N = 7 * block, 100
    xpad = (rng.standard_normal((M, K + 4)) * np.exp2(rng.integers(-6, 7, size=(M, 1)))).astype(np.float32)
    wt = (rng.standard_normal((N, K)) * 0.05).astype(np.float32)
    fa, fb = mx.fmt(block, wx, e, rounding), mx.fmt(block, ww, e, rounding)
    bm, be = mx.quantize(dev(wt), fb)
    B = mx.pack(bm, be, 1, N, K, fb)
    xd = dev(xpad)
    scratch = mx.linear_workspace(M, K, N, fa, fb, DEV)
    ys = []
    for off in (0, 1):                                   # element offset 1: rows not 16-byte aligned
        xv = xd[:, off:off + K]
        am, ae = mx.quantize(xv, fa)
        A = mx.pack(am, ae, 1, M, K, fa)
        y1 = mx.gemm(A, fa, B, fb, M, N, K)[0]
        y2 = torch.full((M, N), 3.0, dtype=torch.float32, device=DEV)
        mx.mx_linear(xv, M, K, K + 4, fa, scratch, B, N, fb, mx.MX_LAYOUT_FRAGMENT, y2, N)
        torch.cuda.synchronize()
        if off:                           # unaligned rows take the two-launch form: the same kernels as y1
            assert torch.equal(y1, y2)
        y_ref, mag = orc.linear(xpad[:, off:off + K], wt, block, wx, ww, e, rounding, want_mag=True)
        check_product(host(y2), y_ref, mag, "linear block %d off %d" % (block, off))


@pytest.mark.parametrize("M,block,wx,ww", [(2, 16, 8, 4), (4, 16, 8, 4), (8, 32, 6, 5), (6, 64, 8, 8)])
def test_linear_two_row_activation_blocks(M, block, wx, ww):
    """mx_linear with the paper's (block, 2) shape for the activations (rows 2p and 2p+1 of x share their
    exponents) and for the weights: the oracle's product of the two-row quantizations."""
    rng = np.random.default_rng(block + M)
    K, N = 9 * block, 100
    x = (rng.standard_normal((M, K)) * np.exp2(rng.integers(-6, 7, size=(M, 1)))).astype(np.float32)
    wt = (rng.standard_normal((N, K)) * 0.05).astype(np.float32)
    fa, fb = mx.fmt(block, wx, block_rows=2), mx.fmt(block, ww, block_rows=2)
    B = mx.quantize_pack(dev(wt), fb, mx.MX_LAYOUT_FRAGMENT)
    scratch = mx.linear_workspace(M, K, N, fa, fb, DEV)
    y = torch.full((M, N), 3.0, dtype=torch.float32, device=DEV)
    mx.mx_linear(dev(x), M, K, K, fa, scratch, B, N, fb, mx.MX_LAYOUT_FRAGMENT, y, N)
    torch.cuda.synchronize()
    qa, ea = orc.quantize(x, block, wx, block_rows=2)
    qb, eb = orc.quantize(wt, block, ww, block_rows=2)
    y_ref, mag = orc.gemm(qa, orc.row_exps(ea, 2), wx, qb, orc.row_exps(eb, 2), ww, block, want_mag=True)
    check_product(host(y), y_ref, mag, "two-row linear M %d block %d" % (M, block))
    assert not np.array_equal(orc.row_exps(ea, 2), orc.quantize(x, block, wx)[1])     # the shape matters here


@pytest.mark.parametrize("M,K,block", [(3, 300 * 64, 16), (8, 270 * 128, 32), (1, 64, 16), (2, 5 * 256, 64)])
def test_gemv_long_and_short_k(M, K, block):
    """Decode path beyond what the streaming kernel keeps in LDS (falls back to the looping kernel),
    and at a single chunk."""
    rng = np.random.default_rng(K + M)
    N = 70
    qa, ea = random_operand(rng, M, K, block, 8, 118, 132)
    qb, eb = random_operand(rng, N, K, block, 4, 118, 132)
    A, fa = gpu_operand(qa, ea, block, 8)
    B, fb = gpu_operand(qb, eb, block, 4)
    y = mx.gemm(A, fa, B, fb, M, N, K)
    torch.cuda.synchronize()
    y_ref, mag = orc.gemm(qa, ea, 8, qb, eb, 4, block, want_mag=True)
    check_product(host(y)[0], y_ref, mag, "gemv M=%d K=%d block=%d" % (M, K, block))


def random_operand(rng, rows, K, block, w, elo, ehi):
    qmax = 2 ** (w - 1) - 1
    q = rng.integers(-qmax - 1, qmax + 1, size=(rows, K)).astype(np.int8)     # includes the code -2^(w-1)
    ex = rng.integers(elo, ehi, size=(rows, K // block)).astype(np.uint8)
    return q, ex


@pytest.mark.parametrize("block", [16, 32, 64])
def test_gemm_all_width_pairs_ragged_shapes(block):
    rng = np.random.default_rng(block)
    M, N, K = 45, 70, 5 * block                     # ragged in M, N and in the 4-block chunking of K
    for wa in range(2, 9):
        for wb in range(2, 9):
            qa, ea = random_operand(rng, M, K, block, wa, 100, 150)
            qb, eb = random_operand(rng, N, K, block, wb, 100, 150)
            A, fa = gpu_operand(qa, ea, block, wa)
            B, fb = gpu_operand(qb, eb, block, wb)
            y = mx.gemm(A, fa, B, fb, M, N, K)
            torch.cuda.synchronize()
            y_ref, mag = orc.gemm(qa, ea, wa, qb, eb, wb, block, want_mag=True)
            check_product(host(y)[0], y_ref, mag, "wa=%d wb=%d block=%d" % (wa, wb, block))
    say("all width pairs ok, block", block)


@pytest.mark.parametrize("M", [1, 5, 8, 9, 40])
def test_gemm_extreme_exponents_and_batch(M):
    rng = np.random.default_rng(M)
    N, K, block, batch = 50, 256, 16, 3
    ya, yr, mg = [], [], []
    qa = np.stack([random_operand(rng, M, K, block, 8, 0, 256)[0] for _ in range(batch)])
    qb = np.stack([random_operand(rng, N, K, block, 4, 0, 256)[0] for _ in range(batch)])
    # exponent bytes over the full range (both clamps included), arranged so that every block term
    # stays inside fp32: the two operands' bytes of a block sum to about 255
    base = rng.integers(0, 256, size=(batch, 1, K // block))
    ea = (base + rng.integers(-5, 6, size=(batch, M, K // block))).clip(0, 255).astype(np.uint8)
    eb = (255 - base + rng.integers(-20, 21, size=(batch, N, K // block))).clip(0, 255).astype(np.uint8)
    A, fa = gpu_operand(qa, ea, block, 8, batch)
    B, fb = gpu_operand(qb, eb, block, 4, batch)
    y = mx.gemm(A, fa, B, fb, M, N, K, batch=batch)
    torch.cuda.synchronize()
    for b in range(batch):
        y_ref, mag = orc.gemm(qa[b], ea[b], 8, qb[b], eb[b], 4, block, want_mag=True)
        check_product(host(y)[b], y_ref, mag, "batch %d" % b)


def test_gemm_special_structures():
    rng = np.random.default_rng(99)
    block, K, M = 32, 256, 40
    qa, ea = random_operand(rng, M, K, block, 8, 110, 140)
    # identity weights (code 2^(w-2), E = 0 is the value 1.0): the product returns the dequantized left operand
    wb = 4
    qb = (np.eye(K, dtype=np.int8) * 2 ** (wb - 2)).astype(np.int8)
    eb = np.full((K, K // block), 127, np.uint8)
    A, fa = gpu_operand(qa, ea, block, 8)
    B, fb = gpu_operand(qb, eb, block, wb)
    y = mx.gemm(A, fa, B, fb, M, K, K)
    torch.cuda.synchronize()
    assert np.array_equal(host(y)[0].astype(np.float64), orc.dequantize(qa, ea, block, 8))
    # K = 0: an empty sum
    y0 = mx.gemm(A, fa, B, fb, M, K, 0)
    torch.cuda.synchronize()
    assert not host(y0).any()
    # output with a leading dimension larger than N leaves the gap untouched
    out = torch.full((M, K + 8), 7.0, dtype=torch.float32, device=DEV)
    mx.mx_gemm(1, M, K, K, A, fa, B, fb, mx.MX_LAYOUT_FRAGMENT, out, K + 8, 0)
    torch.cuda.synchronize()
    assert np.array_equal(host(out)[:, K:], np.full((M, 8), 7.0, np.float32))
    assert np.array_equal(host(out)[:, :K], host(y)[0])


@pytest.mark.parametrize("M", [1, 2, 4])
@pytest.mark.parametrize("block", [16, 32, 64])
def test_gemv_block_halves_that_cancel(M, block):
    """A block with a large exponent whose two half-block dots cancel exactly, next to blocks 2^20 times
    smaller that carry the result: the block dot has to be an exact integer before it is scaled (the decode
    kernels hold the halves of a block in different lanes).  The result must be that of the small blocks."""
    rng = np.random.default_rng(block + M)
    K, N, wa, wb = 8 * block, 70, 8, 4
    qa, ea = random_operand(rng, M, K, block, wa, 100, 104)
    qb, eb = random_operand(rng, N, K, block, wb, 100, 104)
    for blk in (0, 5):                                   # the cancelling blocks: a = c everywhere, b = +7 then -7
        qa[:, blk * block:(blk + 1) * block] = rng.integers(20, 120, size=(M, 1))
        qb[:, blk * block:blk * block + block // 2] = 7
        qb[:, blk * block + block // 2:(blk + 1) * block] = -7
        ea[:, blk] = 120
        eb[:, blk] = 120
    A, fa = gpu_operand(qa, ea, block, wa)
    B, fb = gpu_operand(qb, eb, block, wb)
    y = mx.gemm(A, fa, B, fb, M, N, K)
    torch.cuda.synchronize()
    y_ref, mag = orc.gemm(qa, ea, wa, qb, eb, wb, block, want_mag=True)
    check_product(host(y)[0], y_ref, mag, "cancelling halves M %d block %d" % (M, block))
    # the half-block terms are 2^40 times the bound: a kernel that adds them in fp32 cannot pass
    half = 7.0 * 20 * (block // 2) * 2.0 ** (240 - 254 - (wa - 2) - (wb - 2))
    assert half > 1e9 * mag.max()


def test_gemm_output_beyond_32_bit_offsets():
    """32768 x 65600 outputs (2^31 + 2^21 elements, 8.6 GB): output offsets that do not fit 32 bits, through the
    block-scaled, the bfloat16 and the int8 tiled kernels; the oracle takes windows of rows at both ends."""
    rng = np.random.default_rng(32)
    M, N, K = 32768, 65600, 64
    x = rng.standard_normal((M, K)).astype(np.float32)
    wt = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    assert Y.numel() > 2 ** 31
    for layout, block in ((MAT, 32), (MAT, 16), (mx.MX_LAYOUT_FRAGMENT, 32)):
        fa, fb = mx.fmt(block, 8), mx.fmt(block, 4)
        A = mx.quantize_pack(dev(x), fa, layout)
        B = mx.quantize_pack(dev(wt), fb, layout)
        Y.fill_(7.0)
        mx.mx_gemm(1, M, N, K, A, fa, B, fb, layout, Y, N, M * N)
        torch.cuda.synchronize()
        qa, ea = orc.quantize(x, block, 8)
        qb, eb = orc.quantize(wt, block, 4)
        for r0, r1 in ((0, 6), (16380, 16390), (M - 6, M)):
            y_ref, mag = orc.gemm(qa[r0:r1], ea[r0:r1], 8, qb, eb, 4, block, want_mag=True)
            check_product(host(Y[r0:r1]), y_ref, mag, "layout %d block %d rows %d.." % (layout, block, r0))
            assert not np.any(host(Y[r0:r1]) == 7.0)
    del Y
    torch.cuda.empty_cache()


def test_packed_operand_beyond_32_bit_offsets():
    """A right operand of 196608 x 45056 weights: 35 GB of fp32 into mx_quantize_pack, 6.9 GB (matrix layout) and
    4.7 GB (fragment layout) packed -- byte offsets beyond 32 bits inside the operand, through the fused quantizer,
    the prefill kernel, the tiled int8 kernel and the decode kernels.  The weights are one seeded tile of 512 rows
    repeated, so output column n must equal column n mod 512, and the first 512 columns are checked against the
    oracle."""
    rng = np.random.default_rng(33)
    N, K, T_ = 196608, 45056, 512
    tile = (rng.standard_normal((T_, K)) * 0.02).astype(np.float32)
    wd = dev(tile).repeat(N // T_, 1)
    assert wd.numel() * 0.75 > 2 ** 32
    qb, eb = orc.quantize(tile, 32, 4)
    fa, fb = mx.fmt(32, 8), mx.fmt(32, 4)
    for layout, Ms in ((MAT, (64,)), (mx.MX_LAYOUT_FRAGMENT, (1, 8, 40))):
        B = mx.quantize_pack(wd, fb, layout)
        assert B.numel() > 2 ** 32
        for M in Ms:
            x = rng.standard_normal((M, K)).astype(np.float32)
            A = mx.quantize_pack(dev(x), fa, layout)
            y = mx.gemm(A, fa, B, fb, M, N, K, layout=layout)[0]
            torch.cuda.synchronize()
            assert bool((y.view(M, N // T_, T_) == y[:, :T_].reshape(M, 1, T_)).all()), "columns of a repetition differ"
            qa, ea = orc.quantize(x, 32, 8)
            y_ref, mag = orc.gemm(qa, ea, 8, qb, eb, 4, 32, want_mag=True)
            check_product(host(y[:, :T_]), y_ref, mag, "layout %d M %d" % (layout, M))
        del B
    del wd
    torch.cuda.empty_cache()


def test_gemm_is_deterministic():
    case = inputs.opt125m_layer()[0]
    x, wt = inputs.make(case)
    fa, fb = mx.fmt(case.block, case.wx), mx.fmt(case.block, case.ww)
    A = mx.pack(*mx.quantize(dev(x), fa), 1, case.M, case.K, fa)
    B = mx.pack(*mx.quantize(dev(wt), fb), 1, case.N, case.K, fb)
    y1 = mx.gemm(A, fa, B, fb, case.M, case.N, case.K)
    y2 = mx.gemm(A, fa, B, fb, case.M, case.N, case.K)
    torch.cuda.synchronize()
    assert torch.equal(y1, y2)


def oracle_probabilities(Q, K, block, wq, wk, dim):
    """fp32 probabilities [heads, Sq, Sk] for the second product of the unfused attention tests, from the
    oracle's scores (float64 softmax, held as fp32): an input of both sides that owes nothing to the kernels."""
    out = np.empty((Q.shape[0], Q.shape[1], K.shape[1]), np.float32)
    for hd in range(Q.shape[0]):
        oq, oqe = orc.quantize(Q[hd], block, wq)
        ok, oke = orc.quantize(K[hd], block, wk)
        z = orc.gemm(oq, oqe, wq, ok, oke, wk, block) / np.sqrt(dim)
        z -= z.max(axis=1, keepdims=True)
        np.exp(z, out=z)
        z /= z.sum(axis=1, keepdims=True)
        out[hd] = z
    return out


@pytest.mark.parametrize("seed", [0, 3])
def test_attention_shaped_products_mixed_widths(seed):
    """Reduced form of the mixed-precision attention workload: per head Q K^T (blocks of 16 along the head
    dimension) and P V (blocks of 16 along the sequence: V is quantized along its strided axis), every
    tensor with its own width drawn by seed, batched over the heads."""
    heads, seq, dim, block = 4, 256, 128, 16
    wq, wk, wp, wv = inputs.attention_widths(seed)
    Q, K, V = inputs.attention_qkv(seed, heads, seq, dim)
    say("attention widths", wq, wk, wp, wv)
    fq, fk, fp_, fv = (mx.fmt(block, w) for w in (wq, wk, wp, wv))
    # scores = Q K^T
    qm, qe = mx.quantize(dev(Q), fq)
    km, ke = mx.quantize(dev(K), fk)
    A = mx.pack(qm, qe, heads, seq, dim, fq)
    B = mx.pack(km, ke, heads, seq, dim, fk)
    S = mx.gemm(A, fq, B, fk, seq, seq, dim, batch=heads)
    torch.cuda.synchronize()
    Ph = oracle_probabilities(Q, K, block, wq, wk, dim)               # fp32, outside the MXInt path
    P = dev(Ph)
    # out = P V: P blocked along its rows' sequence axis, V along the sequence (its strided axis)
    pm, pe = mx.quantize(P, fp_)
    vm, ve = mx.quantize(dev(V), fv, axis=0)                          # canonical form of V^T: [heads, dim, seq]
    A2 = mx.pack(pm, pe, heads, seq, seq, fp_)
    B2 = mx.pack(vm, ve, heads, dim, seq, fv)
    O = mx.gemm(A2, fp_, B2, fv, seq, dim, seq, batch=heads)
    torch.cuda.synchronize()
    for hd in range(heads):
        oq, oqe = orc.quantize(Q[hd], block, wq)
        ok, oke = orc.quantize(K[hd], block, wk)
        s_ref, s_mag = orc.gemm(oq, oqe, wq, ok, oke, wk, block, want_mag=True)
        check_product(host(S)[hd], s_ref, s_mag, "scores head %d" % hd)
        op, ope = orc.quantize(Ph[hd], block, wp)
        ov, ove = orc.quantize(V[hd], block, wv, axis=0)
        assert np.array_equal(host(pm).reshape(heads, -1)[hd], orc.pack_bits(op, wp).reshape(-1))
        assert np.array_equal(host(vm).reshape(heads, -1)[hd], orc.pack_bits(ov, wv).reshape(-1))
        assert np.array_equal(host(ve).reshape(heads, -1)[hd], ove.reshape(-1))
        o_ref, o_mag = orc.gemm(op, ope, wp, ov, ove, wv, block, want_mag=True)
        check_product(host(O)[hd], o_ref, o_mag, "output head %d" % hd)


def test_bound_call_matches_direct_call():
    """mx.bound marshals once and re-issues the same entry-point call: same bytes as the direct call."""
    case = inputs.llama13b_decode(1)[0]
    x, wt = inputs.make(case)
    fa, fb = mx.fmt(case.block, case.wx), mx.fmt(case.block, case.ww)
    bm, be = mx.quantize(dev(wt), fb)
    B = mx.pack(bm, be, 1, case.N, case.K, fb)
    xd = dev(x)
    scratch = mx.linear_workspace(1, case.K, case.N, fa, fb, DEV)
    y1 = torch.zeros((1, case.N), dtype=torch.float32, device=DEV)
    y2 = torch.zeros_like(y1)
    mx.mx_linear(xd, 1, case.K, case.K, fa, scratch, B, case.N, fb, mx.MX_LAYOUT_FRAGMENT, y1, case.N)
    call = mx.bound("mx_linear", xd, 1, case.K, case.K, fa, scratch, B, case.N, fb, mx.MX_LAYOUT_FRAGMENT, y2, case.N)
    call()
    call()
    torch.cuda.synchronize()
    assert np.array_equal(host(y1), host(y2))
    bad = mx.bound("mx_linear", xd, 1, case.K + 1, case.K, fa, scratch, B, case.N, fb, mx.MX_LAYOUT_FRAGMENT, y2, case.N)
    with pytest.raises(mx.MxError):
        bad()


def test_attention_full_size_sampled_heads_and_rows():
    """The attention workload at its full size (32 heads, 2048 positions, head dimension 128) through the
    fused quantize+pack path the benchmark times; the oracle computes two heads on a 32-row window."""
    heads, seq, dim, block, seed = 32, 2048, 128, 16, 0
    wq, wk, wp, wv = inputs.attention_widths(seed)
    Q, K, V = inputs.attention_qkv(seed, heads, seq, dim)
    fq, fk, fp_, fv = (mx.fmt(block, w) for w in (wq, wk, wp, wv))
    A = mx.quantize_pack(dev(Q), fq)
    B = mx.quantize_pack(dev(K), fk)
    S = mx.gemm(A, fq, B, fk, seq, seq, dim, batch=heads)
    Ph = oracle_probabilities(Q, K, block, wq, wk, dim)
    A2 = mx.quantize_pack(dev(Ph), fp_)
    vm, ve = mx.quantize(dev(V), fv, axis=0)
    B2 = mx.pack(vm, ve, heads, dim, seq, fv)
    O = mx.gemm(A2, fp_, B2, fv, seq, dim, seq, batch=heads)
    torch.cuda.synchronize()
    r0, r1 = 1500, 1532
    for hd in (0, 31):
        oq, oqe = orc.quantize(Q[hd], block, wq)
        ok, oke = orc.quantize(K[hd], block, wk)
        s_ref, s_mag = orc.gemm(oq, oqe, wq, ok, oke, wk, block, rows=(r0, r1), want_mag=True)
        say("scores head", hd, "worst", check_product(host(S[hd, r0:r1]), s_ref[r0:r1], s_mag[r0:r1], "scores"))
        op, ope = orc.quantize(Ph[hd], block, wp)
        ov, ove = orc.quantize(V[hd], block, wv, axis=0)
        o_ref, o_mag = orc.gemm(op, ope, wp, ov, ove, wv, block, rows=(r0, r1), want_mag=True)
        say("output head", hd, "worst", check_product(host(O[hd, r0:r1]), o_ref[r0:r1], o_mag[r0:r1], "output"))


# ----------------------------------------------------------------------------------------------
# The block-scaled matrix-core layout (block 32 / 64) and the product kernel that reads it
# ----------------------------------------------------------------------------------------------
MAT = mx.MX_LAYOUT_MATRIX


@pytest.mark.parametrize("block,w", [(32, 2), (32, 3), (32, 4), (32, 5), (32, 6), (32, 7), (32, 8), (64, 4), (64, 8),
                                     (16, 2), (16, 3), (16, 4), (16, 5), (16, 6), (16, 7), (16, 8)])
def test_matrix_pack_unpack_roundtrip(block, w):
    rng = np.random.default_rng(200 + block + w)
    f = mx.fmt(block, w)
    for rows, cols in [(70, 5 * 64), (32, 64), (1, 64), (129, 9 * 64), (33, 7 * 16)][:5 if block == 16 else 4]:
        # every code, including -2^(w-1); exponent bytes over the layout's range: up to 250 for the
        # block-scaled form, [w - 1, 253] for the bfloat16 form of block 16
        lo, hi = (w - 1, 254) if block == 16 else (0, 251)
        mant = rng.integers(0, 256, size=mx.mx_mant_bytes(2, rows, cols, f)).astype(np.uint8)
        exps = rng.integers(lo, hi, size=mx.mx_exps_bytes(2, rows, cols, f)).astype(np.uint8)
        packed = mx.pack(dev(mant), dev(exps), 2, rows, cols, f, MAT)
        m2, e2 = mx.unpack(packed, 2, rows, cols, f, MAT)
        torch.cuda.synchronize()
        assert np.array_equal(host(m2), mant) and np.array_equal(host(e2), exps)


@pytest.mark.parametrize("layout", [mx.MX_LAYOUT_FRAGMENT, MAT])
@pytest.mark.parametrize("block,w,rounding", [(32, 8, mx.MX_RNE), (32, 4, mx.MX_RNE), (64, 6, mx.MX_RTZ),
                                              (32, 3, mx.MX_RTZ), (64, 8, mx.MX_RNE), (32, 5, mx.MX_RNE),
                                              (16, 8, mx.MX_RNE), (16, 4, mx.MX_RTZ), (16, 7, mx.MX_RNE)])
def test_quantize_pack_equals_quantize_then_pack(layout, block, w, rounding):
    rng = np.random.default_rng(300 + block + w)
    f = mx.fmt(block, w, 8, rounding)
    for batch, rows, cols in [(1, 70, 5 * 64), (2, 33, 8 * 64), (1, 256, 1024)]:
        x = special_values(rng, batch * rows, cols).reshape(batch, rows, cols)
        x = np.clip(x, -1e30, 1e30)                      # the matrix layout stops at exponent byte 250
        xd = dev(x)
        n = mx.mx_packed_bytes(batch, rows, cols, f, layout)
        p1 = torch.zeros(n, dtype=torch.uint8, device=DEV)
        p2 = torch.zeros(n, dtype=torch.uint8, device=DEV)
        mant, exps = mx.quantize(xd, f)
        mx.mx_pack(mant, exps, batch, rows, cols, f, layout, p1)
        mx.mx_quantize_pack(xd, batch, rows, cols, cols, rows * cols, f, layout, p2)
        torch.cuda.synchronize()
        assert torch.equal(p1, p2), (layout, block, w, batch, rows, cols)


def test_matrix_gemm_llama7b_reduced_m256_full_output():
    case = inputs.llama7b_prefill()[0]
    say("matrix gemm", case.name, "M=256 worst", run_case(case, M=256, layout=MAT))
    say("matrix gemm fused", case.name, "M=256 worst", run_case(case, M=256, layout=MAT, fused=True))


@pytest.mark.parametrize("idx", [0, 1, 2])
def test_matrix_gemm_llama7b_full_size_whole_output(idx):
    """The benchmark's launch configuration (M = 2048, fused quantize+pack, matrix layout): every element of
    the output against the oracle under the plain criterion |err| <= 1e-5 * sum_b |term_b|."""
    case = inputs.llama7b_prefill()[idx]
    worst = run_case(case, layout=MAT, fused=True)
    say("matrix gemm", case.name, "whole output, worst err / sum|terms|", worst)
    assert worst <= 1e-5


@pytest.mark.parametrize("N,wa", [(32 * 256 + 300, 8), (32 * 256 + 128, 4), (64 * 256 + 1, 6)])
def test_matrix_gemm_more_than_one_round_of_tiles_ragged_n(N, wa):
    """M = 2048 with N a little over whole rounds of resident workgroups (two workgroups per compute unit, banded
    tile order, a ragged last column of tiles; one- and two-piece left operands).  Whole output."""
    rng = np.random.default_rng(N + wa)
    M, K, block = 2048, 256, 32
    x = (rng.standard_normal((M, K)) * np.exp2(rng.integers(-3, 4, size=(M, 1)))).astype(np.float32)
    wt = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    fa, fb = mx.fmt(block, wa), mx.fmt(block, 4)
    y = mx.gemm(mx.quantize_pack(dev(x), fa, MAT), fa, mx.quantize_pack(dev(wt), fb, MAT), fb, M, N, K, layout=MAT)
    torch.cuda.synchronize()
    y_ref, mag = orc.linear(x, wt, block, wa, 4, want_mag=True)
    say("ragged rounds, N", N, "worst", check_product(host(y)[0], y_ref, mag, "ragged rounds N=%d" % N))


def test_check_finite_agrees_with_what_the_oracle_refuses():
    """mx_check_finite on a strided batch (rows and matrices with gaps, a ragged last piece of 1024 columns): finite
    data pass, and a NaN or an infinity of either sign planted anywhere (first and last element included), which the
    oracle's quantizer refuses, is reported; values in the gaps are not looked at."""
    rng = np.random.default_rng(77)
    batch, rows, cols = 3, 37, 2050
    big = rng.standard_normal((batch, rows + 2, cols + 30)).astype(np.float32)
    big[:, rows:, :] = np.nan                                   # outside the tensor: rows past the end ...
    big[:, :, cols:] = np.inf                                   # ... and the gap behind every row
    bd = dev(big)
    view = bd[:, :rows, :cols]
    assert view.stride(-1) == 1 and not view.is_contiguous()
    assert mx.check_finite(view)
    assert mx.check_finite(dev(np.full((5, 16), 3.0e38, np.float32)))          # large is not infinite
    assert mx.check_finite(dev(np.full((5, 16), 1.0e-45, np.float32)))         # nor is a subnormal
    spots = [(0, 0, 0), (batch - 1, rows - 1, cols - 1), (1, 17, 1023), (1, 17, 1024), (2, 0, 2049)]
    for (b, r, c), bad in zip(spots, [np.nan, np.inf, -np.inf, -np.nan, np.inf]):
        keep = float(big[b, r, c])
        bd[b, r, c] = float(bad)
        assert not mx.check_finite(view), (b, r, c, bad)
        one = big[b, :rows, :cols - 2].copy()
        one[r, min(c, cols - 3)] = bad
        with pytest.raises(ValueError):
            orc.quantize(one, 32, 8)
        bd[b, r, c] = keep
        assert mx.check_finite(view)


@pytest.mark.parametrize("wa,wb,block", [(8, 4, 32), (3, 4, 64), (8, 6, 32), (4, 8, 64)])
def test_matrix_gemm_block_exponents_change_with_every_group_of_k_steps(wa, wb, block):
    """A small product (the form whose waves split K and load operands and scales straight from global memory) repeated many
    times, the magnitude of both operands moving by a few binades from one group of four K steps (256 elements) to the
    next, so that scales of the wrong group show in every element.  All four piece combinations of the block-scaled kernel;
    whole output, every repetition.  The forms that copy scales through LDS, where they could be read before they have
    landed, are run the same way by test_matrix_product_on_long_k in test_gpu_tiles.py."""
    rng = np.random.default_rng(17 * wa + wb)
    M, N, K = 100, 300, 13 * 256
    grp = np.repeat(np.arange(K // 256), 256)
    x = (rng.standard_normal((M, K)) * np.exp2(((5 * grp) % 11) - 5.0)).astype(np.float32)
    wt = (rng.standard_normal((N, K)) * 0.02 * np.exp2(((3 * grp) % 7) - 3.0)).astype(np.float32)
    fa, fb = mx.fmt(block, wa), mx.fmt(block, wb)
    A, B = mx.quantize_pack(dev(x), fa, MAT), mx.quantize_pack(dev(wt), fb, MAT)
    y_ref, mag = orc.linear(x, wt, block, wa, wb, want_mag=True)
    worst = 0.0
    for rep in range(40):
        y = mx.gemm(A, fa, B, fb, M, N, K, layout=MAT)
        torch.cuda.synchronize()
        worst = max(worst, check_product(host(y)[0], y_ref, mag, "k-group scales, repetition %d" % rep))
    say("k-group scales", wa, wb, block, "worst", worst)


@pytest.mark.parametrize("block", [16, 32, 64])
@pytest.mark.parametrize("spread", ["window", "adversarial"])
def test_matrix_gemm_all_width_pairs_ragged_shapes(block, spread):
    """Random mantissas and independent random block exponents.  In rows and columns 0..9 about half of the
    blocks are made to cancel exactly (+qmax, -qmax against two equal weights) while holding the largest
    products, and the other blocks, which carry the result, sit at the bottom of the exponent range.
    window: the exponent sums Ea + Eb of an output's blocks span at most 24 - wa - wb binades.  The matrix
      instruction keeps 24 bits below its largest single product and a product of two mantissa pieces has at most
      wa + wb - 1 bits (16h * 16h' can pass the product of the mantissas themselves by a binade), so nothing a
      smaller block contributed is pushed out: the plain criterion must hold.
    adversarial: over 50 binades the matrix-core path is bounded against the size of the individual products
      (see check_product)."""
    rng = np.random.default_rng(400 + block)
    M, N, K = 45, 70, 5 * 64
    nb = K // block
    for wa in range(2, 9):
        for wb in range(2, 9):
            if spread == "window":
                D = 24 - wa - wb
                sa = (2 * D + 2) // 3
                sb = D - sa
                hia, hib = 128, 122
            else:
                sa = sb = 50
                hia = hib = 150
            qa, ea = random_operand(rng, M, K, block, wa, hia - sa, hia + 1)
            qb, eb = random_operand(rng, N, K, block, wb, hib - sb, hib + 1)
            cancel = rng.random(nb) < 0.5
            ea[:10], eb[:10] = hia - sa, hib - sb
            for j in np.nonzero(cancel)[0]:
                qa[:10, j * block:(j + 1) * block] = 0
                qa[:10, j * block] = 2 ** (wa - 1) - 1
                qa[:10, j * block + 1] = -(2 ** (wa - 1) - 1)
                qb[:10, j * block:j * block + 2] = 2 ** (wb - 1) - 1
                ea[:10, j], eb[:10, j] = hia, hib
            A, fa = gpu_operand(qa, ea, block, wa, layout=MAT)
            B, fb = gpu_operand(qb, eb, block, wb, layout=MAT)
            y = mx.gemm(A, fa, B, fb, M, N, K, layout=MAT)
            torch.cuda.synchronize()
            y_ref, mag = orc.gemm(qa, ea, wa, qb, eb, wb, block, want_mag=True)
            me = None if spread == "window" else product_magnitude(qa, ea, wa, qb, eb, wb, block)
            check_product(host(y)[0], y_ref, mag, "matrix wa=%d wb=%d block=%d" % (wa, wb, block), me)
    say("matrix layout: all width pairs ok, block", block, spread)


@pytest.mark.parametrize("M,N", [(300, 520), (257, 130), (64, 64)])
def test_matrix_gemm_tiles_batch_wide_exponents(M, N):
    """Several workgroup tiles with ragged edges, a batch, and exponent bytes over the layout's whole
    range (0..250), arranged so that every block term stays inside fp32."""
    rng = np.random.default_rng(M + N)
    K, block, batch = 7 * 64, 32, 2
    qa = np.stack([random_operand(rng, M, K, block, 8, 0, 1)[0] for _ in range(batch)])
    qb = np.stack([random_operand(rng, N, K, block, 4, 0, 1)[0] for _ in range(batch)])
    base = rng.integers(0, 251, size=(batch, 1, K // block))
    ea = (base + rng.integers(-5, 6, size=(batch, M, K // block))).clip(0, 250).astype(np.uint8)
    eb = (250 - base + rng.integers(-20, 21, size=(batch, N, K // block))).clip(0, 250).astype(np.uint8)
    A, fa = gpu_operand(qa, ea, block, 8, batch, MAT)
    B, fb = gpu_operand(qb, eb, block, 4, batch, MAT)
    y = mx.gemm(A, fa, B, fb, M, N, K, batch=batch, layout=MAT)
    y0 = mx.gemm(A, fa, B, fb, M, N, 0, batch=batch, layout=MAT)
    torch.cuda.synchronize()
    assert not host(y0).any()
    for b in range(batch):
        y_ref, mag = orc.gemm(qa[b], ea[b], 8, qb[b], eb[b], 4, block, want_mag=True)
        me = product_magnitude(qa[b], ea[b], 8, qb[b], eb[b], 4, block)
        check_product(host(y)[b], y_ref, mag, "matrix batch %d" % b, me)


def test_matrix_gemm_block16_workloads_full_output():
    """Block 16 in the matrix layout (bfloat16 form): the single linear and the OPT-125M layer, whole
    outputs, through mx_quantize + mx_pack and through the fused mx_quantize_pack."""
    for case in inputs.single_linear() + inputs.opt125m_layer():
        say("matrix gemm b16", case.name, "worst", run_case(case, layout=MAT),
            "fused", run_case(case, layout=MAT, fused=True))


@pytest.mark.parametrize("M,N", [(300, 520), (257, 130), (64, 64)])
def test_matrix_gemm_block16_tiles_batch_wide_exponents(M, N):
    """Block 16: several workgroup tiles with ragged edges, a batch, K that is not a multiple of the
    K step, exponent bytes over the bfloat16 form's range, every block term inside fp32."""
    rng = np.random.default_rng(M + N + 16)
    K, block, batch = 7 * 64 + 16, 16, 2
    qa = np.stack([random_operand(rng, M, K, block, 8, 0, 1)[0] for _ in range(batch)])
    qb = np.stack([random_operand(rng, N, K, block, 4, 0, 1)[0] for _ in range(batch)])
    base = rng.integers(10, 245, size=(batch, 1, K // block))
    ea = (base + rng.integers(-3, 4, size=(batch, M, K // block))).clip(7, 253).astype(np.uint8)
    eb = (254 - base + rng.integers(-3, 4, size=(batch, N, K // block))).clip(7, 253).astype(np.uint8)
    A, fa = gpu_operand(qa, ea, block, 8, batch, MAT)
    B, fb = gpu_operand(qb, eb, block, 4, batch, MAT)
    y = mx.gemm(A, fa, B, fb, M, N, K, batch=batch, layout=MAT)
    y0 = mx.gemm(A, fa, B, fb, M, N, 0, batch=batch, layout=MAT)
    y2 = mx.gemm(A, fa, B, fb, M, N, K, batch=batch, layout=MAT)
    torch.cuda.synchronize()
    assert not host(y0).any()
    assert torch.equal(y, y2)
    for b in range(batch):
        y_ref, mag = orc.gemm(qa[b], ea[b], 8, qb[b], eb[b], 4, block, want_mag=True)
        me = product_magnitude(qa[b], ea[b], 8, qb[b], eb[b], 4, block)
        check_product(host(y)[b], y_ref, mag, "matrix b16 batch %d" % b, me)


def test_matrix_attention_full_size_sampled_heads_and_rows():
    """The attention workload at full size on the matrix layout (block 16, bfloat16 form), fused
    quantize+pack for Q, K, P and quantize along the sequence + pack for V."""
    heads, seq, dim, block, seed = 32, 2048, 128, 16, 0
    wq, wk, wp, wv = inputs.attention_widths(seed)
    Q, K, V = inputs.attention_qkv(seed, heads, seq, dim)
    fq, fk, fp_, fv = (mx.fmt(block, w) for w in (wq, wk, wp, wv))
    A = mx.quantize_pack(dev(Q), fq, MAT)
    B = mx.quantize_pack(dev(K), fk, MAT)
    S = mx.gemm(A, fq, B, fk, seq, seq, dim, batch=heads, layout=MAT)
    Ph = oracle_probabilities(Q, K, block, wq, wk, dim)
    A2 = mx.quantize_pack(dev(Ph), fp_, MAT)
    vm, ve = mx.quantize(dev(V), fv, axis=0)
    B2 = mx.pack(vm, ve, heads, dim, seq, fv, MAT)
    O = mx.gemm(A2, fp_, B2, fv, seq, dim, seq, batch=heads, layout=MAT)
    torch.cuda.synchronize()
    r0, r1 = 1500, 1532
    for hd in (0, 31):
        oq, oqe = orc.quantize(Q[hd], block, wq)
        ok, oke = orc.quantize(K[hd], block, wk)
        s_ref, s_mag = orc.gemm(oq, oqe, wq, ok, oke, wk, block, rows=(r0, r1), want_mag=True)
        say("scores head", hd, "worst", check_product(host(S[hd, r0:r1]), s_ref[r0:r1], s_mag[r0:r1], "scores"))
        op, ope = orc.quantize(Ph[hd], block, wp)
        ov, ove = orc.quantize(V[hd], block, wv, axis=0)
        o_ref, o_mag = orc.gemm(op, ope, wp, ov, ove, wv, block, rows=(r0, r1), want_mag=True)
        say("output head", hd, "worst", check_product(host(O[hd, r0:r1]), o_ref[r0:r1], o_mag[r0:r1], "output"))


def check_quantized_output(q_g, e_g, q_o, e_o, y, mag, block, w, block_rows):
    """The fused output quantizer decides integers from fp32 sums that differ from the oracle's within the
    product tolerance, so codes may differ where a value sits on a rounding or binade boundary.  Checked:
    (1) every block exponent is the binade of a block maximum within the tolerance; (2) every mantissa is a
    correct rounding (or saturation) of a value within the tolerance; (3) all but a sliver equal the oracle's."""
    tol = TOL * mag + 2.0 ** -22 * np.abs(y) + F32_TINY
    M, N = y.shape
    nb = N // block
    qmax = 2 ** (w - 1) - 1
    Eg = orc.row_exps(e_g, block_rows).astype(np.int64) - 127                          # [M, nb]
    blk = lambda a: a.reshape(M // block_rows, block_rows, nb, block).transpose(0, 2, 1, 3).reshape(M // block_rows, nb, -1)
    hi = blk(np.abs(y) + tol).max(axis=2)
    lo = np.maximum(blk(np.abs(y) - tol), 0).max(axis=2)
    Eb = e_g.astype(np.int64) - 127                                                    # [M/R, nb]
    zero = e_g == 0
    assert np.all(hi[zero] < 2.0 ** -126), "zero exponent byte on a block that is not (nearly) zero"
    nz = ~zero
    assert np.all(np.ldexp(1.0, Eb[nz]) <= hi[nz]) and np.all(lo[nz] < np.ldexp(2.0, Eb[nz])), "block exponent off"
    unit = np.repeat(np.ldexp(1.0, Eg - (w - 2)), block, axis=1)
    xhat = q_g.astype(np.float64) * unit
    near = np.abs(xhat - y) <= 0.5 * unit + tol
    sat = (np.abs(q_g) == qmax) & (np.abs(y) >= (qmax - 0.5) * unit - tol)
    assert np.all(near | sat), "a mantissa is not a rounding of the value: worst %g units" % float(
        (np.abs(xhat - y) / unit)[~(near | sat)].max())
    same = np.mean((q_g == q_o) & np.repeat(orc.row_exps(e_g == e_o, block_rows), block, axis=1))
    assert same >= 0.999, "only %.4f of the codes equal the oracle's" % same
    return float(same)


@pytest.mark.parametrize("block,block_rows,wx,wo", [(16, 1, 8, 8), (16, 1, 8, 4), (16, 2, 8, 8), (16, 2, 8, 5),
                                                    (32, 1, 8, 8), (32, 1, 8, 4), (32, 2, 4, 6), (64, 1, 8, 8),
                                                    (64, 2, 3, 3)])
def test_gemm_q_bias_and_output_quantizer(block, block_rows, wx, wo):
    """mx_gemm_q: product + MXInt bias + output quantizer in one kernel, against the oracle's emulated
    linear layer, and bit for bit against mx_gemm, the fp32 bias add and mx_quantize_pack run one by one."""
    rng = np.random.default_rng(40 + wo + block_rows + block)
    ww, wbias = 4, 4
    for M, K, N in [(128, 768, 3072), (70, 7 * 64, 64 * 11), (300, 5 * 64, 64 * 9)]:
        x = rng.standard_normal((M, K)).astype(np.float32)
        wt = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
        bias = (rng.standard_normal(N) * 0.1).astype(np.float32)
        fa, fb = mx.fmt(block, wx, block_rows=block_rows), mx.fmt(block, ww, block_rows=block_rows)
        fbias, fo = mx.fmt(block, wbias), mx.fmt(block, wo, block_rows=block_rows)
        A = mx.quantize_pack(dev(x), fa, MAT)
        B = mx.quantize_pack(dev(wt), fb, MAT)
        bm, be = mx.quantize(dev(bias.reshape(1, N)), fbias)
        n_out = mx.mx_packed_bytes(1, M, N, fo, MAT)
        out = torch.zeros(n_out, dtype=torch.uint8, device=DEV)
        mx.mx_gemm_q(1, M, N, K, A, fa, B, fb, MAT, bm, be, fbias, fo, out)
        # the same, one kernel after the other
        y = mx.gemm(A, fa, B, fb, M, N, K, layout=MAT)[0]
        yb = y + mx.dequantize(bm, be, 1, 1, N, fbias)[0]
        ref = torch.zeros(n_out, dtype=torch.uint8, device=DEV)
        mx.mx_quantize_pack(yb.contiguous(), 1, M, N, N, 0, fo, MAT, ref)
        out2 = torch.zeros(n_out, dtype=torch.uint8, device=DEV)
        mx.mx_gemm_q(1, M, N, K, A, fa, B, fb, MAT, None, None, fbias, fo, out2)          # no bias
        ref2 = torch.zeros(n_out, dtype=torch.uint8, device=DEV)
        mx.mx_quantize_pack(y.contiguous(), 1, M, N, N, 0, fo, MAT, ref2)
        torch.cuda.synchronize()
        assert torch.equal(out, ref), "fused output differs from gemm, bias add, quantize+pack"
        assert torch.equal(out2, ref2), "fused output without bias differs from gemm, quantize+pack"
        # against the oracle
        q_o, e_o, y_ref, mag = orc.linear_q(x, wt, bias, block, wx, ww, wbias, wo, block_rows=block_rows)
        mg, eg = mx.unpack(out, 1, M, N, fo, MAT)
        torch.cuda.synchronize()
        q_g = orc.unpack_bits(host(mg).reshape(M, -1), N, wo)
        e_g = host(eg).reshape(M // block_rows, N // block)
        say("gemm_q", (M, K, N), "codes equal to the oracle's:", check_quantized_output(
            q_g, e_g, q_o, e_o, y_ref, mag, block, wo, block_rows))
    f16, f32_ = mx.fmt(16, 8), mx.fmt(32, 8)
    buf = torch.zeros(1 << 20, dtype=torch.uint8, device=DEV)
    assert mx.mx_gemm_q(1, 32, 64, 64, buf, f32_, buf, f32_, MAT, None, None, f32_, f32_, buf, check=False) == mx.MX_ERR_UNSUPPORTED   # 8-bit right operand
    assert mx.mx_gemm_q(1, 32, 64, 64, buf, f16, buf, f16, MAT, None, None, f16, f32_, buf, check=False) == mx.MX_ERR_UNSUPPORTED    # forms differ
    assert mx.mx_gemm_q(1, 32, 64, 64, buf, f16, buf, f16, mx.MX_LAYOUT_FRAGMENT, None, None, f16, f16, buf, check=False) == mx.MX_ERR_UNSUPPORTED
    assert mx.mx_gemm_q(1, 32, 72, 64, buf, f16, buf, f16, MAT, None, None, f16, f16, buf, check=False) == mx.MX_ERR_BAD_ARG
    assert mx.mx_gemm_q(1, 32, 64, 64, buf, f16, buf, f16, MAT, buf, None, f16, f16, buf, check=False) == mx.MX_ERR_BAD_ARG


def test_matrix_gemm_identity_and_determinism():
    rng = np.random.default_rng(500)
    block, K, M = 32, 256, 40
    qa, ea = random_operand(rng, M, K, block, 8, 110, 140)
    qb = (np.eye(K, dtype=np.int8) * 4).astype(np.int8)            # 1.0 at w = 4: code 2^(w-2), E = 0
    eb = np.full((K, K // block), 127, np.uint8)
    A, fa = gpu_operand(qa, ea, block, 8, layout=MAT)
    B, fb = gpu_operand(qb, eb, block, 4, layout=MAT)
    y = mx.gemm(A, fa, B, fb, M, K, K, layout=MAT)
    y2 = mx.gemm(A, fa, B, fb, M, K, K, layout=MAT)
    torch.cuda.synchronize()
    assert np.array_equal(host(y)[0].astype(np.float64), orc.dequantize(qa, ea, block, 8))
    assert torch.equal(y, y2)


# ----------------------------------------------------------------------------------------------
# mx_attention: both products and the quantizer of the probabilities in one kernel
# ----------------------------------------------------------------------------------------------
def attention_bound(info, wp, wv, scale, rounding, e=8, block=16):
    """Bound on |O_kernel - O_oracle| per element, from the oracle's intermediate values only.

    The kernel's probabilities are fp32 values P(1 + d) with |d| <= eps: hardware exp2/log2 and the
    rounding of their arguments (<= 1e-5 for arguments up to a few hundred), plus the fp32 accumulation
    error of the scores (<= 1e-6 of sum|terms|, far inside the product tolerance) carried through exp
    and through the normalisation.
    A mantissa of P^ can therefore differ from the oracle's by one step where P / step is within eps of a
    rounding boundary, and a whole block by up to two steps where its maximum is within eps of a power of
    two.  Those deviations times |V^|, plus the product tolerance of the second product, bound the output.
    Returns (bound [R, D], fraction of mantissas that may differ)."""
    P = info["P"].astype(np.float32).astype(np.float64)
    R, Sk = P.shape
    bias = 2 ** (e - 1) - 1
    # d P_k / P_k = dz_k - sum_j P_j dz_j with |dz| <= |scale| * 1e-6 * sum|terms| of that score
    dz = abs(scale) * 1e-6 * info["S_mag"]
    eps = 1e-5 + dz + (info["P"] * dz).sum(axis=1, keepdims=True)
    E = info["pe"].astype(np.int64) - bias                                   # [R, Sk/block]
    step = np.repeat(np.ldexp(1.0, E - (wp - 2)), block, axis=1)
    x = P / step
    edge = np.floor(x) + 0.5 if rounding == orc.RNE else np.round(x)        # nearest rounding boundary
    may = (np.abs(x - edge) <= eps * np.maximum(x, 1.0)) & (x < 2 ** (wp - 1))
    if rounding == orc.RTZ:
        may &= x >= 0.5                                                      # nothing below zero to fall to
    amax = P.reshape(R, -1, block).max(axis=2)
    eps_b = eps.reshape(R, -1, block).max(axis=2)
    if info.get("block_rows", 1) == 2:                                       # the block spans rows 2t and 2t+1
        amax = np.repeat(np.maximum(amax[0::2], amax[1::2]), 2, axis=0)
        eps_b = np.repeat(np.maximum(eps_b[0::2], eps_b[1::2]), 2, axis=0)
    frac = amax / np.ldexp(1.0, E)                                           # in [1, 2) unless the exponent is clamped
    amb = ((np.abs(frac - 1.0) <= 2 * eps_b) | (np.abs(frac - 2.0) <= 4 * eps_b)) & (amax > 0)
    dev_ = np.where(may, step, 0.0) + np.repeat(np.where(amb, 2.0, 0.0), block, axis=1) * step
    vabs = np.abs(orc.dequantize(info["vq"], info["ve"], block, wv, e)).T    # [Sk, D]
    pabs = np.abs(orc.dequantize(info["pq"], info["pe"], block, wp, e))
    bound = TOL * info["O_mag"] + 1e-6 * (pabs @ vabs) + dev_ @ vabs + F32_TINY
    return bound, float(may.mean() + amb.mean())


def run_attention(Q, K, V, widths, scale, heads_checked=None, rows=None, rounding=mx.MX_RNE, e_pv=8, max_maybe=1e-2,
                  block_rows=1):
    """Q [H,Sq,D], K, V [H,Sk,D] float32 numpy.  Returns the worst error as a fraction of its bound."""
    wq, wk, wp, wv = widths
    H, Sq, D = Q.shape
    Sk = K.shape[1]
    fq, fk = mx.fmt(16, wq, 8, rounding, block_rows), mx.fmt(16, wk, 8, rounding, block_rows)
    fp_, fv = mx.fmt(16, wp, e_pv, rounding, block_rows), mx.fmt(16, wv, e_pv, rounding, block_rows)
    A = mx.quantize_pack(dev(Q), fq, MAT)
    B = mx.quantize_pack(dev(K), fk, MAT)
    if block_rows == 1:
        vm, ve = mx.quantize(dev(V), fv, axis=0)                             # canonical form of V^T
        Bv = mx.pack(vm, ve, H, D, Sk, fv, MAT)
    else:                                                                    # two columns of V share exponents
        Bv = torch.empty((mx.mx_packed_bytes(H, D, Sk, fv, MAT),), dtype=torch.uint8, device=DEV)
        mx.mx_quantize_pack_axis0(dev(V), H, Sk, D, D, Sk * D, fv, MAT, Bv)
    O = torch.full((H, Sq, D + 4), 7.0, dtype=torch.float32, device=DEV)     # row pitch > D: the gap must survive
    mx.mx_attention(H, Sq, Sk, D, A, fq, B, fk, Bv, fv, fp_, scale, MAT, O, D + 4, Sq * (D + 4))
    torch.cuda.synchronize()
    Oh = host(O)
    assert np.all(Oh[:, :, D:] == 7.0)
    worst = 0.0
    for hd in (range(H) if heads_checked is None else heads_checked):
        # the oracle re-quantizes V with exp_bits e_pv; Q and K keep 8 exponent bits
        o_ref, info = orc.attention(Q[hd], K[hd], V[hd], 16, wq, wk, wp, wv, scale, 8, rounding, rows, block_rows, e_pv=e_pv)
        r0, r1 = info["rows"]
        bound, maybe = attention_bound(info, wp, wv, scale, rounding, e_pv)
        assert maybe < max_maybe, "the tolerance would excuse too many mantissas (%.3g)" % maybe
        err = np.abs(Oh[hd, r0:r1, :D].astype(np.float64) - o_ref[r0:r1])
        ratio = err / bound
        assert np.all(ratio <= 1.0), "head %d: worst error %.3g of its bound (widths %s)" % (hd, ratio.max(), widths)
        # the tolerance is far below the size of the result: a wrong key order, row or scale cannot pass
        if max_maybe <= 1e-2:
            assert np.median(bound) < 1e-3 * np.abs(o_ref[r0:r1]).max()
        worst = max(worst, float(ratio.max()))
    return worst


@pytest.mark.parametrize("seed", [0, 1, 2, 3, 4, 5, 6, 7])
def test_attention_fused_reduced_workload(seed):
    """The attention workload at reduced size, widths drawn by seed; 300 queries (ragged last tile of 32 and
    of the workgroup's 256) against 272 keys (a ragged tile of 32 keys)."""
    heads, Sq, Sk, dim = 3, 300, 272, 128
    widths = inputs.attention_widths(seed)
    Q, _, _ = inputs.attention_qkv(seed, heads, Sq, dim)
    _, K, V = inputs.attention_qkv(seed + 50, heads, Sk, dim)
    say("attention widths", widths, "worst/bound", run_attention(Q, K, V, widths, dim ** -0.5))


@pytest.mark.parametrize("Sq,Sk,dim", [(1, 16, 16), (33, 48, 32), (64, 2080, 64), (40, 96, 96), (257, 32, 48),
                                        (96, 160, 112)])
def test_attention_fused_shapes(Sq, Sk, dim):
    rng = np.random.default_rng(Sq * 1000 + Sk)
    Q = rng.standard_normal((2, Sq, dim)).astype(np.float32)
    K = rng.standard_normal((2, Sk, dim)).astype(np.float32)
    V = (rng.standard_normal((2, Sk, dim)) * rng.choice([0.01, 1.0, 30.0], size=(2, 1, dim))).astype(np.float32)
    say("worst/bound", run_attention(Q, K, V, (8, 8, 6, 5), 0.7 * dim ** -0.5))


@pytest.mark.parametrize("rounding,e_pv,wp", [(mx.MX_RTZ, 8, 5), (mx.MX_RNE, 4, 8), (mx.MX_RNE, 8, 2), (mx.MX_RTZ, 5, 3)])
def test_attention_fused_rounding_and_exponent_width_of_p(rounding, e_pv, wp):
    """Truncation for P and V; a narrow exponent for P and V (probabilities below 2^-bias share the lowest
    exponent and lose their low bits); ternary probabilities."""
    rng = np.random.default_rng(77)
    Q = rng.standard_normal((2, 70, 64)).astype(np.float32)
    K = rng.standard_normal((2, 144, 64)).astype(np.float32)
    V = rng.standard_normal((2, 144, 64)).astype(np.float32)
    say("worst/bound", run_attention(Q, K, V, (7, 7, wp, 6), 0.5, rounding=rounding, e_pv=e_pv))


@pytest.mark.parametrize("scale", [-0.3, 0.0, 1e-3, 2.0])
def test_attention_fused_scales(scale):
    """Negative scale (the smallest score gets the largest probability), zero (uniform probabilities whatever the
    scores), a tiny and a large one; 144 keys: a ragged last tile of 32."""
    rng = np.random.default_rng(91)
    Q = rng.standard_normal((2, 70, 64)).astype(np.float32)
    K = rng.standard_normal((2, 144, 64)).astype(np.float32)
    V = rng.standard_normal((2, 144, 64)).astype(np.float32)
    say("scale", scale, "worst/bound", run_attention(Q, K, V, (8, 7, 6, 5), scale, max_maybe=5e-2))
    if scale == 0.0:                                     # and the probabilities are exactly 1/144 in the oracle
        _, info = orc.attention(Q[0], K[0], V[0], 16, 8, 7, 6, 5, scale)
        assert np.all(info["P"] == 1.0 / 144)


def test_attention_fused_peaked_and_flat_rows():
    """Rows whose softmax is one-hot (a key matching the query by a wide margin), rows with all scores
    equal, and ordinary rows, in one call: the exact cases of the oracle's pins, through the kernel.  Their
    probabilities are powers of two, i.e. they sit exactly on the quantizer's exponent boundary, so for
    those 32 rows the bound allows either exponent (two steps per element)."""
    rng = np.random.default_rng(8)
    Sq, Sk, dim = 64, 64, 64
    K = rng.standard_normal((1, Sk, dim)).astype(np.float32)
    Q = rng.standard_normal((1, Sq, dim)).astype(np.float32)
    Q[0, :16] = 0.0                                      # flat rows: P = 1/64 exactly
    Q[0, 16:32] = 40.0 * K[0, rng.permutation(Sk)[:16]]  # peaked rows
    V = rng.standard_normal((1, Sk, dim)).astype(np.float32)
    say("worst/bound", run_attention(Q, K, V, (8, 8, 7, 8), 1.0, max_maybe=0.6))


@pytest.mark.parametrize("Sq,Sk,dim,widths", [(300, 272, 128, (8, 8, 6, 5)), (34, 48, 32, (7, 6, 5, 3)),
                                               (130, 2080, 64, (8, 4, 8, 8)), (2, 16, 16, (8, 8, 2, 4))])
def test_attention_fused_two_row_blocks(Sq, Sk, dim, widths):
    """Every tensor in the paper's block shape (16, 2) (Section 3, the MASE IR example; Section 4.1): pairs of queries share the exponents of
    Q and of the probabilities, pairs of keys those of K, pairs of columns those of V.  Row scales differ
    from query to query, so the pair's exponent is often set by the neighbour."""
    rng = np.random.default_rng(Sq + Sk)
    Q = (rng.standard_normal((2, Sq, dim)) * rng.choice([0.2, 1.0, 4.0], size=(2, Sq, 1))).astype(np.float32)
    K = rng.standard_normal((2, Sk, dim)).astype(np.float32)
    V = (rng.standard_normal((2, Sk, dim)) * rng.choice([0.01, 1.0, 30.0], size=(2, 1, dim))).astype(np.float32)
    for rounding in (mx.MX_RNE, mx.MX_RTZ):
        say("worst/bound", run_attention(Q, K, V, widths, dim ** -0.5, rounding=rounding, block_rows=2))
    # and it is not the one-row result: the exponents of P differ
    _, i1 = orc.attention(Q[0], K[0], V[0], 16, *widths, dim ** -0.5)
    _, i2 = orc.attention(Q[0], K[0], V[0], 16, *widths, dim ** -0.5, block_rows=2)
    assert not np.array_equal(i1["pe"], i2["pe"])


@pytest.mark.parametrize("Sq,Sk,dim,widths,rounding,R", [(70, 288, 64, (8, 8, 6, 5), mx.MX_RNE, 1), (33, 64, 128, (7, 6, 5, 3), mx.MX_RTZ, 1),
                                                          (130, 2080, 32, (8, 4, 8, 8), mx.MX_RNE, 1),
                                                          (70, 288, 64, (8, 8, 6, 5), mx.MX_RNE, 2), (34, 64, 96, (7, 6, 4, 3), mx.MX_RTZ, 2)])
def test_attention_fused_blocks_of_32(Sq, Sk, dim, widths, rounding, R):
    """All four tensors quantized in blocks of 32 (the block size of the paper's MXInt8 comparisons).  The
    packed operands enter as the block-16 tensors of the same values (each exponent byte repeated for its two
    runs of 16); the probabilities are quantized in blocks of 32 keys inside the kernel.  R = 2: blocks of
    (32, 2), two rows sharing each exponent, in all four tensors."""
    wq, wk, wp, wv = widths
    rng = np.random.default_rng(Sq + Sk + 1)
    H = 2
    Q = rng.standard_normal((H, Sq, dim)).astype(np.float32)
    K = (rng.standard_normal((H, Sk, dim)) * rng.choice([0.3, 1.0, 3.0], size=(H, 1, dim))).astype(np.float32)
    V = (rng.standard_normal((H, Sk, dim)) * rng.choice([0.01, 1.0, 30.0], size=(H, Sk, 1))).astype(np.float32)
    scale = dim ** -0.5

    def operand(x, w):                                   # x [H, rows, cols], blocks of 32 along cols
        rows, cols = x.shape[1:]
        mant, exps = [], []
        for hd in range(H):
            q, ex = orc.quantize(x[hd], 32, w, 8, rounding, block_rows=R)
            mant.append(orc.pack_bits(q, w).reshape(-1))
            exps.append(np.repeat(orc.row_exps(ex, R), 2, axis=1).reshape(-1))
        f16 = mx.fmt(16, w, 8, rounding)
        return mx.pack(dev(np.concatenate(mant)), dev(np.concatenate(exps)), H, rows, cols, f16, MAT), f16

    A, fq = operand(Q, wq)
    B, fk = operand(K, wk)
    Bv, fv = operand(np.ascontiguousarray(V.transpose(0, 2, 1)), wv)
    fp_ = mx.fmt(32, wp, 8, rounding, block_rows=R)
    O = torch.empty((H, Sq, dim), dtype=torch.float32, device=DEV)
    mx.mx_attention(H, Sq, Sk, dim, A, fq, B, fk, Bv, fv, fp_, scale, MAT, O, dim, Sq * dim)
    torch.cuda.synchronize()
    for hd in range(H):
        o_ref, info = orc.attention(Q[hd], K[hd], V[hd], 32, wq, wk, wp, wv, scale, 8, rounding, block_rows=R)
        bound, maybe = attention_bound(info, wp, wv, scale, rounding, 8, block=32)
        assert maybe < 1e-2
        ratio = np.abs(host(O)[hd].astype(np.float64) - o_ref) / bound
        assert np.all(ratio <= 1.0), "head %d: worst error %.3g of its bound" % (hd, ratio.max())
        assert np.median(bound) < 1e-3 * np.abs(o_ref).max()
    # blocks of 16 give other exponents for the probabilities: the block size matters at these inputs
    _, i16 = orc.attention(Q[0], K[0], V[0], 16, wq, wk, wp, wv, scale, 8, rounding)
    _, i32 = orc.attention(Q[0], K[0], V[0], 32, wq, wk, wp, wv, scale, 8, rounding)
    assert not np.array_equal(np.repeat(i32["pe"], 2, axis=1), i16["pe"])


def test_attention_fused_full_size_sampled_heads_and_rows():
    """32 heads x 2048 x 2048 x 128, widths of seed 0, in the launch the benchmark times; the oracle takes two
    heads and a window of query rows each."""
    heads, seq, dim, seed = 32, 2048, 128, 0
    Q, K, V = inputs.attention_qkv(seed, heads, seq, dim)
    for hd, rows in ((0, (0, 40)), (31, (1990, 2048))):
        w = run_attention(Q, K, V, inputs.attention_widths(seed), dim ** -0.5, heads_checked=[hd], rows=rows)
        say("head", hd, "rows", rows, "worst/bound", w)


def test_attention_rejections():
    f = mx.fmt(16, 8)
    buf = torch.zeros(1 << 20, dtype=torch.uint8, device=DEV)
    O = torch.zeros((64, 128), dtype=torch.float32, device=DEV)
    call = lambda Sq=64, Sk=64, D=128, fq=f, fk=f, fv=f, fp_=f, layout=MAT, scale=1.0, ldo=128: mx.mx_attention(
        1, Sq, Sk, D, buf, fq, buf, fk, buf, fv, fp_, scale, layout, O, ldo, 64 * 128, check=False)
    assert call() == mx.MX_OK
    assert call(Sk=0) == mx.MX_ERR_BAD_ARG
    assert call(Sk=40) == mx.MX_ERR_BAD_ARG                 # not whole blocks of keys
    assert call(D=120) == mx.MX_ERR_BAD_ARG
    assert call(ldo=64) == mx.MX_ERR_BAD_ARG
    assert call(scale=float("nan")) == mx.MX_ERR_BAD_ARG
    assert call(fk=mx.fmt(32, 8)) == mx.MX_ERR_BAD_ARG      # Q and K must share the block size
    assert call(fq=mx.fmt(32, 4), fk=mx.fmt(32, 4), D=128) == mx.MX_ERR_UNSUPPORTED
    assert call(fp_=mx.fmt(32, 8)) == mx.MX_OK              # probabilities in blocks of 32 keys
    assert call(fp_=mx.fmt(64, 8)) == mx.MX_ERR_UNSUPPORTED
    assert call(fp_=mx.fmt(32, 8), Sk=48) == mx.MX_ERR_BAD_ARG
    assert call(fv=mx.fmt(32, 8)) == mx.MX_ERR_BAD_ARG     # P's block must be a multiple of V's
    assert call(layout=mx.MX_LAYOUT_FRAGMENT) == mx.MX_ERR_UNSUPPORTED
    assert call(D=256, ldo=256) == mx.MX_ERR_UNSUPPORTED
    f2 = mx.fmt(16, 8, block_rows=2)
    assert call(fp_=f2, fv=f2) == mx.MX_OK                 # two-row blocks: whole pairs of queries
    assert call(Sq=63, fp_=f2) == mx.MX_ERR_BAD_ARG
    assert call(Sq=63, fq=f2) == mx.MX_ERR_BAD_ARG
    assert call(Sq=0) == mx.MX_OK
    torch.cuda.synchronize()


# ----------------------------------------------------------------------------------------------
# Block Minifloat / Block Logarithm quantizer: bit-exact against the oracle
# ----------------------------------------------------------------------------------------------
def run_minifloat(x, block, e, m, rounding=mx.MX_RNE):
    rows, cols = x.shape[-2:]
    batch = 1 if x.ndim == 2 else x.shape[0]
    f = mx.mx_minifloat_format(block, e, m, rounding)
    xd = dev(x)
    codes = torch.full((batch * rows * cols,), 0xAA, dtype=torch.uint8, device=DEV)
    shared = torch.full((batch * rows * (cols // block),), 0xAA, dtype=torch.uint8, device=DEV)
    mx.mx_quantize_minifloat(xd, batch, rows, cols, cols, rows * cols, f, codes, shared)
    y = torch.empty((batch, rows, cols), dtype=torch.float32, device=DEV)
    mx.mx_dequantize_minifloat(codes, shared, batch, rows, cols, f, y)
    torch.cuda.synchronize()
    x3 = x.reshape(batch, rows, cols)
    for b in range(batch):
        oc, osh = orc.quantize_minifloat(x3[b], block, e, m, rounding)
        assert np.array_equal(host(shared).reshape(batch, rows, -1)[b], osh), "shared bytes differ"
        assert np.array_equal(host(codes).reshape(batch, rows, cols)[b], oc), "codes differ"
        assert np.array_equal(host(y)[b].astype(np.float64), orc.dequantize_minifloat(oc, osh, block, e, m))


@pytest.mark.parametrize("block", [8, 16, 32, 64])
@pytest.mark.parametrize("e,m", [(4, 3), (3, 4), (7, 0), (2, 0), (1, 6), (5, 2)])
def test_minifloat_quantizer_bit_exact(block, e, m):
    rng = np.random.default_rng(block * 100 + 10 * e + m)
    rows, cols = 37, 5 * block                           # ragged against the 256-thread workgroups
    x = (rng.standard_normal((rows, cols)) * np.exp2(rng.integers(-12, 12, size=(rows, 1)))).astype(np.float32)
    x[0] = 0.0
    x[1, ::3] = 0.0
    x[2] = np.exp2(rng.integers(-8, 8, size=cols)).astype(np.float32)                    # exact powers of two
    x[3] = (1.5 * np.exp2(rng.integers(-8, 8, size=cols))).astype(np.float32)            # ties of the m = 0 format
    x[4] = (rng.integers(0, 2 ** (m + 2), size=cols) * 2.0 ** -(m + 1) - 1.0).astype(np.float32)   # half steps: ties
    x[5] = (rng.standard_normal(cols) * 1e-39).astype(np.float32)                        # fp32 subnormals
    x[6] = (rng.standard_normal(cols) * 3e38).clip(-3.4e38, 3.4e38).astype(np.float32)   # top of the fp32 range
    x[7, :block] = 1.0
    x[7, 0] = np.float32(2.0) - np.float32(2.0 ** -(m + 1))                              # maximum exactly at the carry midpoint
    for rounding in (mx.MX_RNE, mx.MX_RTZ):
        run_minifloat(x, block, e, m, rounding)


def test_minifloat_workload_shape_and_batch():
    """The prefill activation shape (2048 x 4096, Student-t with outlier channels) in BMF(32, 4, 3) and
    BL(32, 7), and a batch of small matrices."""
    case = inputs.llama7b_prefill()[0]
    x, _ = inputs.make(case)
    run_minifloat(x, 32, 4, 3)
    run_minifloat(x, 32, 7, 0)
    rng = np.random.default_rng(4)
    run_minifloat(rng.standard_normal((3, 9, 64)).astype(np.float32), 16, 3, 2)


def test_minifloat_rejections():
    x = torch.zeros((4, 64), dtype=torch.float32, device=DEV)
    c = torch.zeros(256, dtype=torch.uint8, device=DEV)
    s = torch.zeros(16, dtype=torch.uint8, device=DEV)
    q = lambda f, cols=64, xx=x, stride=64: mx.mx_quantize_minifloat(xx, 1, 4, cols, stride, 4 * 64, f, c, s, check=False)
    F = mx.mx_minifloat_format
    assert q(F(16, 4, 3, 0)) == mx.MX_OK
    assert q(F(16, 4, 4, 0)) == mx.MX_ERR_BAD_ARG            # 1 + 4 + 4 bits do not fit a byte
    assert q(F(16, 0, 3, 0)) == mx.MX_ERR_BAD_ARG
    assert q(F(12, 4, 3, 0)) == mx.MX_ERR_BAD_ARG
    assert q(F(16, 4, 3, 2)) == mx.MX_ERR_BAD_ARG
    assert q(F(16, 4, 3, 0), cols=40) == mx.MX_ERR_BAD_ARG   # not whole blocks
    assert q(F(16, 4, 3, 0), xx=x.view(-1)[1:], cols=48, stride=48) == mx.MX_ERR_UNSUPPORTED   # rows not 16-byte aligned
    torch.cuda.synchronize()


# ----------------------------------------------------------------------------------------------
# mx_quantize_pack_axis0: blocks down the columns, packed as the transposed operand
# ----------------------------------------------------------------------------------------------
@pytest.mark.parametrize("rows,cols,w,rounding,e", [(64, 128, 8, mx.MX_RNE, 8), (272, 96, 3, mx.MX_RNE, 8),
                                                    (16, 16, 5, mx.MX_RTZ, 8), (2080, 130, 6, mx.MX_RNE, 5),
                                                    (48, 33, 2, mx.MX_RTZ, 4)])
def test_quantize_pack_axis0_equals_quantize_then_pack(rows, cols, w, rounding, e):
    """Same bytes as mx_quantize (axis 0) followed by mx_pack -- padding included -- and the canonical form
    recovered by mx_unpack is the oracle's; ragged tiles, unaligned row pitch, narrow exponents, a batch."""
    rng = np.random.default_rng(rows + cols)
    batch = 3
    x = (rng.standard_normal((batch, rows, cols + 3)) * np.exp2(rng.integers(-10, 10, size=(batch, 1, cols + 3)))).astype(np.float32)
    x[0, :16, 0] = 0.0
    f = mx.fmt(16, w, e, rounding)
    xd = dev(x)
    xv = xd[:, :, :cols]
    vm, ve = mx.quantize(xv, f, axis=0)
    want = mx.pack(vm, ve, batch, cols, rows, f, MAT)
    got = torch.full((mx.mx_packed_bytes(batch, cols, rows, f, MAT),), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mx_quantize_pack_axis0(xv, batch, rows, cols, cols + 3, rows * (cols + 3), f, MAT, got)
    torch.cuda.synchronize()
    # a packed matrix is its fragments, its exponent bytes, and alignment padding up to 256 bytes that no one writes
    valid = ((cols + 31) // 32) * (((rows + 31) // 32 + 1) // 2 * 2) * 2048 + cols * (rows // 16)
    per = mx.mx_packed_bytes(1, cols, rows, f, MAT)
    assert per == (valid + 255) // 256 * 256
    assert torch.equal(got.view(batch, per)[:, :valid], want.view(batch, per)[:, :valid])
    assert bool((got.view(batch, per)[:, valid:] == 0x5A).all())
    um, ue = mx.unpack(got, batch, cols, rows, f, MAT)
    torch.cuda.synchronize()
    for b in range(batch):
        oq, oe = orc.quantize(x[b, :, :cols], 16, w, e, rounding, axis=0)
        assert np.array_equal(host(um).reshape(batch, -1)[b], orc.pack_bits(oq, w).reshape(-1))
        assert np.array_equal(host(ue).reshape(batch, -1)[b], oe.reshape(-1))


@pytest.mark.parametrize("rows,cols,w,rounding", [(64, 128, 8, mx.MX_RNE), (272, 96, 3, mx.MX_RTZ), (2080, 130, 6, mx.MX_RNE),
                                                   (16, 2, 4, mx.MX_RNE)])
def test_quantize_pack_axis0_two_row_blocks(rows, cols, w, rounding):
    """Blocks of (16 keys, 2 columns): the bytes of mx_quantize_pack on the transposed matrix with two-row
    blocks, and the canonical form recovered by mx_unpack is the oracle's quantization of x^T."""
    rng = np.random.default_rng(rows * 7 + cols)
    batch = 2
    x = (rng.standard_normal((batch, rows, cols)) * np.exp2(rng.integers(-10, 10, size=(batch, 1, cols)))).astype(np.float32)
    x[0, :16, :2] = 0.0
    f = mx.fmt(16, w, 8, rounding, block_rows=2)
    want = mx.quantize_pack(dev(np.ascontiguousarray(x.transpose(0, 2, 1))), f, MAT)
    got = torch.full((mx.mx_packed_bytes(batch, cols, rows, f, MAT),), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mx_quantize_pack_axis0(dev(x), batch, rows, cols, cols, rows * cols, f, MAT, got)
    torch.cuda.synchronize()
    valid = ((cols + 31) // 32) * (((rows + 31) // 32 + 1) // 2 * 2) * 2048 + cols * (rows // 16)
    per = mx.mx_packed_bytes(1, cols, rows, f, MAT)
    assert torch.equal(got.view(batch, per)[:, :valid], want.view(batch, per)[:, :valid])
    um, ue = mx.unpack(got, batch, cols, rows, f, MAT)
    torch.cuda.synchronize()
    for b in range(batch):
        oq, oe = orc.quantize(np.ascontiguousarray(x[b].T), 16, w, 8, rounding, block_rows=2)
        assert np.array_equal(host(um).reshape(batch, -1)[b], orc.pack_bits(oq, w).reshape(-1))
        assert np.array_equal(host(ue).reshape(batch, -1)[b], oe.reshape(-1))
    assert mx.mx_quantize_pack_axis0(dev(x), batch, rows, cols - 1, cols, rows * cols, f, MAT, got, check=False) == mx.MX_ERR_BAD_ARG


def test_quantize_pack_axis0_workload_and_rejections():
    heads, seq, dim = 32, 2048, 128
    _, _, V = inputs.attention_qkv(0, heads, seq, dim)
    f = mx.fmt(16, 3)
    Vd = dev(V)
    vm, ve = mx.quantize(Vd, f, axis=0)
    want = mx.pack(vm, ve, heads, dim, seq, f, MAT)
    got = torch.empty_like(want)
    mx.mx_quantize_pack_axis0(Vd, heads, seq, dim, dim, seq * dim, f, MAT, got)
    torch.cuda.synchronize()
    assert torch.equal(got, want)             # 128 * 128 exponent bytes: no alignment padding at this shape
    call = lambda ff, layout=MAT, rows=seq: mx.mx_quantize_pack_axis0(Vd, heads, rows, dim, dim, seq * dim, ff, layout, got, check=False)
    assert call(mx.fmt(32, 4)) == mx.MX_ERR_UNSUPPORTED
    assert call(f, mx.MX_LAYOUT_FRAGMENT) == mx.MX_ERR_UNSUPPORTED
    assert call(f, rows=seq - 8) == mx.MX_ERR_BAD_ARG       # not whole blocks down the columns
    torch.cuda.synchronize()


# ----------------------------------------------------------------------------------------------
# The entry points allocate nothing and touch only the caller's stream: a graph can capture them
# ----------------------------------------------------------------------------------------------
def test_calls_captured_in_a_graph_replay_the_same_bits():
    """A decode step (mx_linear at one row, and at four rows through both of its entry points: K slices, arrival
    counters that every launch leaves at zero), a prefill product and an attention call captured into one graph;
    every replay, with eager work and synchronisation in between, gives the eager bits."""
    cases = inputs.llama13b_decode(1)[:2]
    work = []
    for c in cases:
        x, wt = inputs.make(c)
        fa, fb = mx.fmt(c.block, c.wx), mx.fmt(c.block, c.ww)
        bm, be = mx.quantize(dev(wt), fb)
        work.append((dev(x), c, fa, mx.linear_workspace(1, c.K, c.N, fa, fb, DEV),
                     mx.pack(bm, be, 1, c.N, c.K, fb), fb, torch.zeros((1, c.N), dtype=torch.float32, device=DEV)))
    rng = np.random.default_rng(12)
    f8, f4, f16 = mx.fmt(32, 8), mx.fmt(32, 4), mx.fmt(16, 6)
    X = dev(rng.standard_normal((256, 512)).astype(np.float32))
    W = mx.quantize_pack(dev((rng.standard_normal((384, 512)) * 0.05).astype(np.float32)), f4, MAT)
    A = torch.zeros(mx.mx_packed_bytes(1, 256, 512, f8, MAT), dtype=torch.uint8, device=DEV)
    Y = torch.zeros((256, 384), dtype=torch.float32, device=DEV)
    Q, K, V = (dev(rng.standard_normal((2, 96, 64)).astype(np.float32)) for _ in range(3))
    Qp, Kp = (torch.zeros(mx.mx_packed_bytes(2, 96, 64, f16, MAT), dtype=torch.uint8, device=DEV) for _ in range(2))
    Vp = torch.zeros(mx.mx_packed_bytes(2, 64, 96, f16, MAT), dtype=torch.uint8, device=DEV)
    O = torch.zeros((2, 96, 64), dtype=torch.float32, device=DEV)
    c4 = inputs.llama13b_decode(4)[0]
    x4 = dev(inputs.make(c4)[0])
    fa4, fb4 = mx.fmt(c4.block, c4.wx), mx.fmt(c4.block, c4.ww)
    ws4 = mx.linear_workspace(4, c4.K, c4.N, fa4, fb4, DEV)
    Y4a, Y4b = (torch.zeros((4, c4.N), dtype=torch.float32, device=DEV) for _ in range(2))

    def step():
        for xd, c, fa, scratch, B, fb, y in work:
            mx.mx_linear(xd, 1, c.K, c.K, fa, scratch, B, c.N, fb, mx.MX_LAYOUT_FRAGMENT, y, c.N)
        mx.mx_linear(x4, 4, c4.K, c4.K, fa4, ws4, work[0][4], c4.N, fb4, mx.MX_LAYOUT_FRAGMENT, Y4a, c4.N)
        mx.mx_linear_static_workspace(x4, 4, c4.K, c4.K, fa4, work[0][4], c4.N, fb4, mx.MX_LAYOUT_FRAGMENT, Y4b, c4.N)
        mx.mx_quantize_pack(X, 1, 256, 512, 512, 0, f8, MAT, A)
        mx.mx_gemm(1, 256, 384, 512, A, f8, W, f4, MAT, Y, 384, 256 * 384)
        mx.mx_quantize_pack(Q, 2, 96, 64, 64, 96 * 64, f16, MAT, Qp)
        mx.mx_quantize_pack(K, 2, 96, 64, 64, 96 * 64, f16, MAT, Kp)
        mx.mx_quantize_pack_axis0(V, 2, 96, 64, 64, 96 * 64, f16, MAT, Vp)
        mx.mx_attention(2, 96, 96, 64, Qp, f16, Kp, f16, Vp, f16, f16, 0.125, MAT, O, 64, 96 * 64)

    outs = [w[-1] for w in work] + [Y, O, Y4a, Y4b]
    step()
    torch.cuda.synchronize()
    want = [o.clone() for o in outs]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            step()
    for rep in range(4):
        for o in outs:
            o.fill_(float(rep + 1))                     # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert torch.equal(o, w), "replay %d differs" % rep
