"""The forms of the product kernels that are chosen by size, at the sizes where each can go wrong."""
import numpy as np
import pytest
import torch

from oracle import mx_oracle as orc
from paper_2307_15517_amd import mx
from test_gpu_parity import attention_bound, check_cast, check_product, gpu_operand, host, random_operand, run_attention, run_minifloat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,block,wa,wb", [
    (9, 32, 64, 16, 8, 4),             # one chunk of K: fifteen of the sixteen waves have none
    (16, 40, 17 * 64, 16, 8, 4),       # the tile's upper rows do not exist; one wave has a second chunk
    (17, 33, 48, 16, 5, 7),            # one row in the upper half, a partial chunk
    (33, 1, 9 * 128, 32, 6, 5),        # one column, eight waves and one chunk more
    (64, 64, 3 * 256, 64, 8, 8),
    (40, 32 * 270, 128, 16, 8, 4),     # 540 tiles: eight waves each
    (70, 32 * 350 + 5, 64, 16, 4, 4),  # one chunk under 1053 tiles: 128 x 128 instead
    (40, 32 * 530 + 5, 336, 16, 4, 4), # 1062 tiles: four waves each, one with a second chunk
])
def test_fragment_product_tiles_and_waves(M, N, K, block, wa, wb):
    """Block exponents on both sides of the range in which the scales are built by an integer instruction (bytes 96 to
    159), the other way for whole operands, and zero blocks (byte 0) among ordinary ones."""
    rng = np.random.default_rng(M * N + K)
    for lo, hi in ((96, 160), (94, 99), (157, 162)):
        qa, ea = random_operand(rng, M, K, block, wa, lo, hi)
        qb, eb = random_operand(rng, N, K, block, wb, 100, 150)
        zero = rng.random(ea.shape) < 0.1
        ea[zero] = 0
        qa.reshape(M, K // block, block)[zero] = 0
        A, fa = gpu_operand(qa, ea, block, wa)
        B, fb = gpu_operand(qb, eb, block, wb)
        y = mx.gemm(A, fa, B, fb, M, N, K)
        torch.cuda.synchronize()
        y_ref, mag = orc.gemm(qa, ea, wa, qb, eb, wb, block, want_mag=True)
        check_product(host(y)[0], y_ref, mag, "%dx%dx%d bytes %d..%d" % (M, N, K, lo, hi - 1))


@pytest.mark.parametrize("M,N,K,block,wa,wb", [
    (40, 32 * 400, 3 * 128, 32, 8, 4),      # 800 tiles, two waves each, one with a second chunk
    (33, 32 * 150, 5 * 128 + 32, 32, 5, 6), # 300 tiles, four waves each
    (50, 32 * 270, 3 * 256, 64, 6, 5),      # 540 tiles, two waves each
    (40, 32 * 200, 41 * 64, 16, 8, 6),      # 400 tiles, eight waves each
    (20, 96, 20 * 64, 16, 6, 8), (20, 96, 20 * 128, 32, 4, 3), (20, 96, 20 * 128, 32, 7, 8),   # sums without the bias
])
def test_fragment_product_block_sums_with_a_bias(M, N, K, block, wa, wb):
    """The largest block sums there are, of either sign, and sums of zero, with the exponents of both operands at the ends of
    the range in which the scales are built by integer adds, and just past them."""
    rng = np.random.default_rng(M + N + K + wa)
    qa, _ = random_operand(rng, M, K, block, wa, 100, 101)
    qb, _ = random_operand(rng, N, K, block, wb, 100, 101)
    ma, mb = (1 << (wa - 1)) - 1, (1 << (wb - 1)) - 1
    qa[::3], qb[::3] = ma, mb                    # every product the largest
    qa[1::3, ::2], qa[1::3, 1::2] = ma, -ma      # block sums of zero against constant rows
    qb[2::3] = -mb
    for (alo, ahi), (blo, bhi) in (((96, 98), (96, 98)), ((158, 160), (158, 160)), ((96, 98), (158, 160)), ((159, 161), (95, 97))):
        ea = rng.integers(alo, ahi, size=(M, K // block)).astype(np.uint8)
        eb = rng.integers(blo, bhi, size=(N, K // block)).astype(np.uint8)
        A, fa = gpu_operand(qa, ea, block, wa)
        B, fb = gpu_operand(qb, eb, block, wb)
        y = mx.gemm(A, fa, B, fb, M, N, K)
        torch.cuda.synchronize()
        y_ref, mag = orc.gemm(qa, ea, wa, qb, eb, wb, block, want_mag=True)
        check_product(host(y)[0], y_ref, mag, "%dx%dx%d bytes %d %d" % (M, N, K, alo, blo))


MAT = mx.MX_LAYOUT_MATRIX
# (row tiles, column tiles) of 32, from the smallest tile with K split over the waves to a partial second round of the larger
# ones.  K is short in the tests that take these, which moves some to smaller tiles: MATRIX_FORMS_LONG_K has every form.
MATRIX_FORMS = [(1, 2), (2, 200), (4, 200), (4, 400), (4, 900), (3, 1500), (4, 2400)]


@pytest.mark.parametrize("rt,ct", MATRIX_FORMS)
@pytest.mark.parametrize("block,wa,wb,K", [(16, 8, 4, 48), (16, 6, 3, 32 * 9), (32, 8, 4, 64 * 9), (32, 4, 3, 96),
                                           (32, 5, 6, 64 * 3), (64, 3, 8, 64)])
def test_matrix_product_forms(rt, ct, block, wa, wb, K):
    """Ragged rows and columns, waves without a K step or with one more than others; exponent sums span fewer than
    24 - wa - wb binades, so the sums are exact up to the final additions."""
    M, N = rt * 32 - 13, ct * 32 - 5
    if K * ct > 64 * 1500:
        K = {16: 48, 32: 96, 64: 64}[block]
    rng = np.random.default_rng(M * 31 + N + K)
    qa, ea = random_operand(rng, M, K, block, wa, 122, 126)
    qb, eb = random_operand(rng, N, K, block, wb, 120, 123)
    A, fa = gpu_operand(qa, ea, block, wa, layout=MAT)
    B, fb = gpu_operand(qb, eb, block, wb, layout=MAT)
    y = torch.full((M, N + 3), 7.0, device="cuda")
    mx.mx_gemm(1, M, N, K, A, fa, B, fb, MAT, y, N + 3, 0)
    torch.cuda.synchronize()
    y = host(y)
    assert (y[:, N:] == 7.0).all(), "columns past N written"
    y_ref, mag = orc.gemm(qa, ea, wa, qb, eb, wb, block, want_mag=True)
    check_product(y[:, :N], y_ref, mag, "%dx%dx%d block %d" % (M, N, K, block))


@pytest.mark.parametrize("rt,ct", [(1, 3), (2, 200), (4, 200), (4, 400), (4, 900), (4, 2400)])
@pytest.mark.parametrize("block,wx,wo", [(16, 8, 6), (32, 8, 8), (64, 6, 4), (32, 4, 8)])
def test_matrix_product_forms_quantized_output(rt, ct, block, wx, wo):
    """mx_gemm_q in the forms up to 64 x 256 and 128 x 128, without a bias and with a short K, against mx_gemm of the same
    operands quantized afterwards: with exact sums (few binades, 24 bits hold them) the packed bytes are the same, padding
    rows and columns included.  (All forms, with the rest of the ending: test_matrix_quantized_output_on_long_k.)"""
    M, N, K = rt * 32 - 13, ct * 32 - (block if block < 64 else 0), 2 * block
    N -= N % block
    rng = np.random.default_rng(M * 31 + N)
    qa, ea = random_operand(rng, M, K, block, wx, 124, 126)
    qb, eb = random_operand(rng, N, K, block, 4, 120, 122)
    A, fa = gpu_operand(qa, ea, block, wx, layout=MAT)
    B, fb = gpu_operand(qb, eb, block, 4, layout=MAT)
    fo = mx.fmt(block, wo)
    out = torch.full((mx.mx_packed_bytes(1, M, N, fo, MAT),), 255, dtype=torch.uint8, device="cuda")
    mx.mx_gemm_q(1, M, N, K, A, fa, B, fb, MAT, None, None, fb, fo, out)
    want = torch.full_like(out, 255)
    y = mx.gemm(A, fa, B, fb, M, N, K, layout=MAT)
    mx.mx_quantize_pack(y, 1, M, N, N, 0, fo, MAT, want)
    torch.cuda.synchronize()
    assert np.array_equal(host(out), host(want))


@pytest.mark.parametrize("dim", [32, 64, 80, 128])
@pytest.mark.parametrize("heads,Sq,Sk", [(2, 33, 16), (3, 7, 272), (12, 702, 272), (10, 702, 272), (12, 702, 336), (100, 258, 48)])
def test_attention_forms(heads, Sq, Sk, dim):
    """A workgroup per 32 queries and 32 columns, per 32 queries, per 128 queries: a ragged last tile of queries and of
    keys, waves without a key tile, both rounding modes, one- and two-row blocks, both signs of the scale."""
    rng = np.random.default_rng(heads * 1000 + Sk + dim)
    Q = rng.standard_normal((heads, Sq, dim)).astype(np.float32)
    K = rng.standard_normal((heads, Sk, dim)).astype(np.float32)
    V = (rng.standard_normal((heads, Sk, dim)) * rng.choice([0.01, 1.0, 30.0], size=(heads, 1, dim))).astype(np.float32)
    for rounding, rows, scale in ((mx.MX_RNE, 1, dim ** -0.5), (mx.MX_RTZ, 2 if Sq % 2 == 0 else 1, -0.7 * dim ** -0.5)):
        run_attention(Q, K, V, (8, 7, 6, 5), scale, heads_checked=[0, heads - 1], rounding=rounding, block_rows=rows)


def attention_output(Q, K, V, widths, scale):
    heads, Sq, dim = Q.shape
    Sk = K.shape[1]
    fq, fk, fp, fv = (mx.fmt(16, w) for w in widths)
    Bv = torch.empty((mx.mx_packed_bytes(heads, dim, Sk, fv, MAT),), dtype=torch.uint8, device="cuda")
    mx.mx_quantize_pack_axis0(torch.from_numpy(V).cuda(), heads, Sk, dim, dim, Sk * dim, fv, MAT, Bv)
    O = torch.empty((heads, Sq, dim), device="cuda")
    mx.mx_attention(heads, Sq, Sk, dim, mx.quantize_pack(torch.from_numpy(Q).cuda(), fq, MAT), fq,
                    mx.quantize_pack(torch.from_numpy(K).cuda(), fk, MAT), fk, Bv, fv, fp, scale, MAT, O, dim, Sq * dim)
    torch.cuda.synchronize()
    return host(O)


def run_attention_of_scale_zero(Q, K, V, widths, heads_checked, rows=None):
    """Every probability is 1 / Sk.  Where that is a power of two the row statistic, exact or a last place above it, decides
    between it and the largest mantissa one exponent below, for a whole row: all of a row has to be one of the two."""
    Sk, (wp, wv) = K.shape[1], widths[2:]
    if Sk & (Sk - 1):
        run_attention(Q, K, V, widths, 0.0, heads_checked=heads_checked, rows=rows)
        return
    O = attention_output(Q, K, V, widths, 0.0)[:, slice(*rows) if rows else slice(None)]
    below = (2 ** (wp - 1) - 1) / 2 ** (wp - 1) / Sk
    for hd in heads_checked:
        v = orc.dequantize(*orc.quantize(V[hd].T.copy(), 16, wv), 16, wv).astype(np.float64)
        bound = 1e-5 * np.abs(v).sum(axis=1) / Sk                           # fp32 sums, as every product's
        exact, less = (np.abs(O[hd] - p * v.sum(axis=1)) <= bound for p in (1 / Sk, below))
        assert (exact.all(axis=1) | less.all(axis=1)).all(), hd


@pytest.mark.parametrize("dim", [32, 64, 80, 128])
@pytest.mark.parametrize("heads,Sq,Sk", [(3, 7, 528), (3, 33, 1024), (2, 40, 1040), (2, 1, 2048), (2, 5, 2064), (12, 702, 784),
                                         (12, 702, 1200), (24, 702, 768), (40, 800, 1296)])
def test_attention_with_kept_scores(heads, Sq, Sk, dim):
    """17 to 64 key tiles and one more, waves with all their tiles, with fewer and with none, a ragged last one; a workgroup per
    32 columns and per 32 queries, one to four rounds of them; both rounding modes, two-row blocks, a scale below and of zero."""
    Q, K, V = long_attention_inputs(heads, Sq, Sk, dim)
    some = dict(heads_checked=[0, heads - 1], rows=(max(0, Sq - 34), Sq))
    run_attention(Q, K, V, (8, 7, 6, 5), dim ** -0.5, **some)
    run_attention(Q, K, V, (7, 8, 5, 6), -0.7 * dim ** -0.5, rounding=mx.MX_RTZ, block_rows=2 if Sq % 2 == 0 else 1, **some)
    run_attention_of_scale_zero(Q, K, V, (8, 7, 8, 6), **some)


@pytest.mark.parametrize("dim", [16, 48, 80, 128])
@pytest.mark.parametrize("heads,Sq,Sk", [(3, 1, 16), (3, 16, 256), (2, 5, 272), (5, 3, 512), (2, 13, 784), (2, 16, 2032), (2, 2, 2048),
                                         (130, 2, 304), (300, 1, 48)])
def test_attention_of_up_to_sixteen_queries(heads, Sq, Sk, dim):
    """One to 64 key tiles, waves with all their tiles, with fewer and with none, a ragged last one; a workgroup per 32 columns and
    per head; both rounding modes, two-row blocks, a narrow exponent of P and V, a scale below and of zero."""
    Q, K, V = long_attention_inputs(heads, Sq, Sk, dim)
    some = dict(heads_checked=[0, heads - 1])
    run_attention(Q, K, V, (8, 7, 6, 5), dim ** -0.5, **some)
    run_attention(Q, K, V, (7, 8, 5, 6), -0.7 * dim ** -0.5, rounding=mx.MX_RTZ, block_rows=2 if Sq % 2 == 0 else 1, **some)
    run_attention(Q, K, V, (8, 7, 8, 6), dim ** -0.5, e_pv=4, **some)
    run_attention_of_scale_zero(Q, K, V, (8, 7, 8, 6), **some)


def test_fragment_product_past_one_grid_dimension():
    """131072 x 131072 results, 64 GiB: 2^24 tiles of 32 x 32, more than the work items of one grid dimension hold as
    workgroups of 256.  Every element is written, sampled rows and columns (first and last among them) are right."""
    n, K, block = 131072, 2048, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    f = mx.fmt(block, 4)
    x = torch.randn((n, K), generator=g, device="cuda")
    w = torch.randn((n, K), generator=g, device="cuda")
    A, B = mx.quantize_pack(x, f), mx.quantize_pack(w, f)
    idx = torch.tensor([0, 31, 32, 4097, 65535, 65536, 99999, n - 1], device="cuda")
    xs, ws = host(x[idx]), host(w[idx])
    del x, w
    y = torch.full((n, n), float("nan"), device="cuda")
    mx.mx_gemm(1, n, n, K, A, f, B, f, mx.MX_LAYOUT_FRAGMENT, y, n, 0)
    torch.cuda.synchronize()
    for r in range(0, n, 8192):
        assert not torch.isnan(y[r:r + 8192]).any(), "rows %d.. not written" % r
    y_ref, mag = orc.linear(xs, ws, block, 4, 4, want_mag=True)
    check_product(host(y[idx][:, idx]), y_ref, mag, "64 GiB result")


@pytest.mark.parametrize("M,N,K,block,wa,wb,batch", [
    (1300, 4100, 128, 16, 8, 4, 1),        # two chunks of K: 363 tiles of 128 x 128, both edges ragged
    (2048 - 13, 4096 - 5, 64 + 32, 32, 6, 5, 1),
    (190, 257, 64, 32, 7, 3, 20),          # 120 tiles over a batch, the last columns one wide
    (2048 - 13, 4096 - 5, 3 * 256 + 64, 64, 8, 7, 1),
    (700, 1000, 256, 64, 3, 6, 2),         # 96 tiles, one chunk
    (1024, 4096, 3 * 256, 64, 5, 2, 2),    # 512 tiles, no edge
])
def test_fragment_product_large_tiles(M, N, K, block, wa, wb, batch):
    """The 128 x 128 form: widths that are spread from 2, 3, 5, 6 and 7 bits, exponents over 60 binades, zero blocks, ragged
    edges, batches.  Sampled rows (edges of tiles and of the matrix) over all columns, and nothing past N written."""
    rng = np.random.default_rng(M + N + K)
    rows = np.unique(np.concatenate([[0, 31, 32, 127, 128, M - 1], rng.integers(0, M, 10)]))
    ops = []
    for b in range(batch):
        qa, ea = random_operand(rng, M, K, block, wa, 90, 151)
        qb, eb = random_operand(rng, N, K, block, wb, 100, 161)
        zero = rng.random(ea.shape) < 0.1
        ea[zero] = 0
        qa.reshape(M, K // block, block)[zero] = 0
        ops.append((qa, ea, qb, eb))
    cat = lambda k: np.stack([o[k] for o in ops])
    A, fa = gpu_operand(cat(0), cat(1), block, wa, batch=batch)
    B, fb = gpu_operand(cat(2), cat(3), block, wb, batch=batch)
    y = torch.full((batch, M, N + 3), 7.0, device="cuda")
    mx.mx_gemm(batch, M, N, K, A, fa, B, fb, mx.MX_LAYOUT_FRAGMENT, y, N + 3, M * (N + 3))
    torch.cuda.synchronize()
    assert (y[:, :, N:] == 7.0).all(), "columns past N written"
    assert not (y[:, :, :N] == 7.0).all(dim=2).any(), "rows not written"
    for b, (qa, ea, qb, eb) in enumerate(ops):
        y_ref, mag = orc.gemm(qa[rows], ea[rows], wa, qb, eb, wb, block, want_mag=True)
        check_product(host(y[b, rows, :N]), y_ref, mag, "large tiles, batch entry %d" % b)


def test_fragment_product_with_short_k_runs_at_the_rate_of_its_stores():
    """One chunk of K under a 1.6 GB result: the product is a store of its result and little else.  With 32 x 32 tiles
    whose waves divide K it took 4.1 times a fill of the same buffer, with 128 x 128 tiles 0.9."""
    batch, M, N, K = 32, 2304, 5504, 32
    fa, fb = mx.fmt(32, 8), mx.fmt(32, 4)
    A = mx.quantize_pack(torch.randn((batch, M, K), device="cuda"), fa)
    B = mx.quantize_pack(torch.randn((batch, N, K), device="cuda"), fb)
    y = torch.empty((batch, M, N), device="cuda")
    product = mx.bound("mx_gemm", batch, M, N, K, A, fa, B, fb, mx.MX_LAYOUT_FRAGMENT, y, N, M * N)

    def best(call):
        times = []
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            call()
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)
    fill = best(lambda: y.fill_(1.0))
    assert best(product) < 2.0 * fill


@pytest.mark.parametrize("block,wx,M,N,K,batch", [(32, 4, 40, 32, 512, 1), (32, 8, 40, 32, 512, 1), (64, 8, 300, 64, 1088, 8),
                                                  (32, 3, 736, 64, 864, 32), (32, 4, 1400, 96, 800, 24), (64, 7, 2100, 320, 576, 16)])
def test_quantized_output_with_few_columns(block, wx, M, N, K, batch):
    """Narrow results, most of whose layout is padding (columns to 256, row tiles to an even number): the padding bytes are
    those of mx_quantize_pack, with a bias, over a batch, in the split form and in each staged one."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    fx, fw, fo = mx.fmt(block, wx), mx.fmt(block, 3), mx.fmt(block, wx, block_rows=2 if M % 4 == 0 else 1)
    # integers that every product and sum holds exactly, so that the two ways to the result agree in every bit
    x = torch.randint(-3, 4, (batch, M, K), generator=g, device="cuda").float()
    w = torch.randint(-3, 4, (batch, N, K), generator=g, device="cuda").float()
    x[:, :, ::block] = 3.0
    w[:, :, ::block] = 3.0
    bias = torch.randint(-3, 4, (1, N), generator=g, device="cuda").float()
    bias[:, ::block] = 3.0
    A, B = mx.quantize_pack(x, fx, MAT), mx.quantize_pack(w, fw, MAT)
    out = torch.full((mx.mx_packed_bytes(batch, M, N, fo, MAT),), 255, dtype=torch.uint8, device="cuda")
    mx.mx_gemm_q(batch, M, N, K, A, fx, B, fw, MAT, *mx.quantize(bias, fw), fw, fo, out)
    y = mx.gemm(A, fx, B, fw, M, N, K, batch=batch, layout=MAT) + bias
    torch.cuda.synchronize()
    assert torch.equal(y, x.double().matmul(w.double().transpose(1, 2).contiguous()).float() + bias)
    want = torch.full_like(out, 255)
    mx.mx_quantize_pack(y, batch, M, N, N, M * N, fo, MAT, want)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


def best_time(call):
    """Shortest of twelve launches, ms."""
    times = []
    for _ in range(12):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        call()
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end))
    return min(times)


def test_quantized_output_takes_no_product_for_padding():
    """64 columns in a layout of 256: the fused call does the work of the plain product, not that of four times its
    columns (1.7 times the plain product's time when the padding tiles took a product, 1.0 without)."""
    batch, M, N, K = 32, 736, 64, 10880
    f = mx.fmt(64, 4)
    A = mx.quantize_pack(torch.randn((batch, M, K), device="cuda"), f, MAT)
    B = mx.quantize_pack(torch.randn((batch, N, K), device="cuda"), f, MAT)
    y = torch.empty((batch, M, N), device="cuda")
    out = torch.empty(mx.mx_packed_bytes(batch, M, N, f, MAT), dtype=torch.uint8, device="cuda")
    plain = mx.bound("mx_gemm", batch, M, N, K, A, f, B, f, MAT, y, N, M * N)
    fused = mx.bound("mx_gemm_q", batch, M, N, K, A, f, B, f, MAT, None, None, f, f, out)
    assert best_time(fused) < 1.4 * best_time(plain)


def test_a_smaller_matrix_product_is_not_the_slower_one():
    """A size whose 128 x 256 tiles fill a second round in most of its places, beside one that fills it: with the tile of half
    the width and twice the operand traffic the smaller product had taken 1.25 times as long as the larger one (0.94 now)."""
    M, larger, N, K = 3687, 4096, 3922, 7152
    fa, fb = mx.fmt(16, 6), mx.fmt(16, 4)
    A = mx.quantize_pack(torch.randn((larger, K), device="cuda"), fa, MAT)
    B = mx.quantize_pack(torch.randn((N, K), device="cuda"), fb, MAT)
    y = torch.empty((larger, N), device="cuda")
    times = [best_time(mx.bound("mx_gemm", 1, m, N, K, A, fa, B, fb, MAT, y, N, 0)) for m in (M, larger, M, larger)]
    assert min(times[0], times[2]) < 1.1 * min(times[1], times[3]), times


@pytest.mark.parametrize("M", [1, 2, 5])
@pytest.mark.parametrize("wx,ww", [(8, 5), (4, 6), (6, 7), (8, 8)])
def test_decode_rings_of_wide_records(M, wx, ww):
    """Blocks of 64 with 5 to 8 bits on few columns: sixteen waves with rings of three or two chunks, on K of fewer chunks
    than waves, of one more than a turn of all rings and of a partial last chunk."""
    rng = np.random.default_rng(100 * M + 10 * wx + ww)
    N = 70
    for K in (64, 256 * 5, 256 * 49 + 128):
        x = (rng.standard_normal((M, K)) * np.exp2(rng.integers(-6, 7, size=(M, K // 64)).repeat(64, axis=1))).astype(np.float32)
        wt = (rng.standard_normal((N, K)) * 0.05).astype(np.float32)
        fx, fw = mx.fmt(64, wx), mx.fmt(64, ww)
        xd = torch.from_numpy(x).cuda()
        A, B = mx.quantize_pack(xd, fx), mx.quantize_pack(torch.from_numpy(wt).cuda(), fw)
        y = torch.full((2, M, N), 3.0, device="cuda")
        mx.mx_linear(xd, M, K, K, fx, mx.linear_workspace(M, K, N, fx, fw, "cuda"), B, N, fw, mx.MX_LAYOUT_FRAGMENT, y[0], N)
        mx.mx_gemm(1, M, N, K, A, fx, B, fw, mx.MX_LAYOUT_FRAGMENT, y[1], N, 0)
        torch.cuda.synchronize()
        y_ref, mag = orc.linear(x, wt, 64, wx, ww, want_mag=True)
        for k in (0, 1):
            check_product(host(y[k]), y_ref, mag, "M %d K %d widths %d %d" % (M, K, wx, ww))


@pytest.mark.parametrize("M,K,N,block,wx,ww,rounding", [
    (3, 48, 33, 16, 8, 8, mx.MX_RNE),          # one column group, four parts: one partial chunk, three of the waves have none
    (5, 37 * 16, 100, 16, 2, 4, mx.MX_RTZ),    # one group, eight parts of two chunks, the last ones short, a partial chunk
    (6, 70 * 64, 41 * 32 + 5, 16, 8, 4, mx.MX_RNE),   # one group, eight parts, five slices, the last one short
    (5, 24 * 128, 669, 32, 6, 5, mx.MX_RTZ),   # one group, four parts, six slices
    (6, 179 * 32, 2075, 32, 6, 5, mx.MX_RNE),  # two groups, four parts, six slices, half a column of workgroups, a partial chunk
    (8, 13 * 32, 13007, 32, 8, 2, mx.MX_RNE),  # two groups, four parts, one slice, half a column
    (8, 8 * 128, 20000, 32, 8, 2, mx.MX_RNE),  # four groups, two parts, one slice, a column with one group of the four
    (8, 80 * 64, 432 * 32, 16, 8, 4, mx.MX_RNE),      # four groups, two parts, four slices
    (8, 80 * 64, 13889, 16, 8, 4, mx.MX_RNE),  # the same with three of the four groups in the last column
    (4, 45 * 32, 2000, 32, 6, 8, mx.MX_RNE),   # one group, eight parts, one slice
    (7, 17 * 64, 321, 64, 8, 7, mx.MX_RNE),
    # one and two rows: the dot-product kernel
    (1, 45 * 32, 2000, 32, 8, 5, mx.MX_RNE), (1, 64, 31, 64, 4, 8, mx.MX_RTZ), (2, 81 * 64, 5120, 16, 8, 4, mx.MX_RNE),
])
def test_decode_splits_and_scales(M, K, N, block, wx, ww, rounding):
    """One to eight rows in every form of the split.  Block exponents at the ends of the range in which the block sums take
    two multiply-adds (activations -63 to 64, weights -31 to 32), one past them, and blocks of zeros on both sides."""
    rng = np.random.default_rng(M * K + N)
    x0 = rng.standard_normal((M, K)).astype(np.float32)
    w0 = rng.standard_normal((N, K)).astype(np.float32)
    x0.reshape(M, -1, block)[rng.random((M, K // block)) < 0.1] = 0.0
    w0.reshape(N, -1, block)[rng.random((N, K // block)) < 0.02] = 0.0
    fx, fw = mx.fmt(block, wx, 8, rounding), mx.fmt(block, ww, 8, rounding)

    def blocks_at(a, exponents):                 # every block's largest value gets one of these exponents
        v = a.reshape(a.shape[0], -1, block)
        e = np.frexp(np.abs(v).max(axis=2, keepdims=True))[1] - 1
        return np.ldexp(v, rng.choice(exponents, size=e.shape) - e).reshape(a.shape).astype(np.float32)

    for xe, we in (([-2, 3], [-6, -5]), ([-63, -62], [-31, -30]), ([63, 64], [31, 32]), ([-64, -63], [-31, -30]), ([64, 65], [0, 1]),
                   ([0, 1], [-32, 33])):
        x, wt = blocks_at(x0, xe), blocks_at(w0, we)
        xd = torch.from_numpy(x).cuda()
        B = mx.quantize_pack(torch.from_numpy(wt).cuda(), fw)
        y = torch.full((2, M, N), 3.0, device="cuda")
        ws = mx.linear_workspace(M, K, N, fx, fw, "cuda")
        for k in (0, 1):                         # the counters are left at zero, the order of arrival does not matter
            mx.mx_linear(xd, M, K, K, fx, ws, B, N, fw, mx.MX_LAYOUT_FRAGMENT, y[k], N)
        torch.cuda.synchronize()
        assert torch.equal(y[0], y[1]) and int(ws[:16384].max()) == 0
        cols = np.unique(np.r_[0, N - 1, rng.integers(0, N, size=200)])
        y_ref, mag = orc.linear(x, wt[cols], block, wx, ww, rounding=rounding, want_mag=True)
        check_product(host(y[0])[:, cols], y_ref, mag, "M %d exponents %s %s" % (M, xe, we))


def spread(g, rows, K, block):
    """Blocks whose exponents lie far enough apart that a sum over them is rounded: another order shows in its bits."""
    x = torch.randn((rows, K // block, block), generator=g, device="cuda")
    return (x * torch.exp2(torch.randint(-8, 9, (rows, K // block, 1), generator=g, device="cuda").float())).reshape(rows, K)


@pytest.mark.parametrize("K,N,block,wx,ww", [
    (81 * 64, 5120, 16, 8, 4),
    (33 * 128, 2000, 32, 8, 8),
    (9 * 256, 1100, 64, 6, 4),
    (5 * 256 + 64, 70, 64, 4, 8),
])
def test_decode_of_one_and_two_rows_keeps_nothing_between_workgroups(K, N, block, wx, ww):
    """At one and two rows no workgroup waits for another's sums: the bits of a row are those of the product of packed
    operands, with one row or two, aligned or not, and a workspace that other calls are using is neither read nor written."""
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    fx, fw = mx.fmt(block, wx), mx.fmt(block, ww)
    rows, w = spread(g, 2, K, block), spread(g, N, K, block)
    shifted = torch.zeros((2, K + 4), device="cuda")
    shifted[:, 1:K + 1] = rows
    B = mx.quantize_pack(w, fw)
    want = mx.gemm(mx.quantize_pack(rows, fx), fx, B, fw, 2, N, K)[0]
    ws = mx.linear_workspace(2, K, N, fx, fw, "cuda")

    def linear(M, x, stride):
        y = torch.full((M, N), 3.0, device="cuda")
        mx.mx_linear(x, M, K, stride, fx, ws, B, N, fw, mx.MX_LAYOUT_FRAGMENT, y, N)
        return y
    for M in (1, 2):
        assert torch.equal(linear(M, rows, K), want[:M]), "%d rows" % M
        assert torch.equal(linear(M, shifted[:, 1:], K + 4), want[:M]), "%d rows, not aligned" % M
    ws.fill_(0xAB)
    for M in (1, 2):
        assert torch.equal(linear(M, rows, K), want[:M]), "%d rows, workspace in use" % M
    assert int(ws.min()) == int(ws.max()) == 0xAB


@pytest.mark.parametrize("K,N,block,wx,ww", [
    (80 * 64, 5120, 16, 8, 4), (80 * 64, 13824, 16, 8, 4), (86 * 128, 4096, 32, 6, 5), (32 * 128, 11008, 32, 6, 5),
    (12 * 256, 1100, 64, 6, 4), (30 * 128, 3000, 32, 8, 8),
])
def test_decode_rows_have_the_same_bits_with_three_to_eight_of_them(K, N, block, wx, ww):
    """The split of K follows from the weights alone: a sequence gets the same sums, added in the same order, in a batch of
    three as in one of eight, wherever its row lies."""
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    fx, fw = mx.fmt(block, wx), mx.fmt(block, ww)
    x = spread(g, 8, K, block)
    B = mx.quantize_pack(spread(g, N, K, block), fw)
    ws = mx.linear_workspace(8, K, N, fx, fw, "cuda")
    y8 = torch.full((8, N), 3.0, device="cuda")
    mx.mx_linear(x, 8, K, K, fx, ws, B, N, fw, mx.MX_LAYOUT_FRAGMENT, y8, N)
    for M in (3, 4, 5, 6, 7):
        for first in (0, 8 - M):
            y = torch.full((M, N), 3.0, device="cuda")
            mx.mx_linear(x[first:], M, K, K, fx, ws, B, N, fw, mx.MX_LAYOUT_FRAGMENT, y, N)
            assert torch.equal(y, y8[first:first + M]), "%d rows from row %d" % (M, first)


@pytest.mark.parametrize("K,N,block,ww,parts,slices,part", [
    (11008, 4096, 32, 8, 2, 8, 6), (5504, 2860, 32, 8, 4, 4, 3), (4096, 4096, 32, 5, 4, 4, 2),
    (5120, 12643, 64, 2, 4, 1, 5), (4736, 12316, 64, 3, 4, 1, 5), (4672, 11773, 64, 4, 4, 1, 5), (3072, 768, 64, 8, 4, 3, 1),
])
def test_decode_sums_are_added_in_the_order_of_the_split(K, N, block, ww, parts, slices, part):
    """The bits of a result are those of the split of K that the rule has for these weights: runs of `part` records of four
    blocks added one after the other, `parts` runs to a slice, the slices in their order.  How many records a wave keeps
    in flight is none of it."""
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    fx, fw = mx.fmt(block, 8), mx.fmt(block, ww)
    x, w = spread(g, 3, K, block), spread(g, N, K, block)
    y = torch.full((3, N), 3.0, device="cuda")
    mx.mx_linear(x, 3, K, K, fx, mx.linear_workspace(3, K, N, fx, fw, "cuda"), mx.quantize_pack(w, fw), N, fw, mx.MX_LAYOUT_FRAGMENT, y, N)
    cols = np.r_[0:48, N - 48:N]
    (qa, ea), (qb, eb) = orc.quantize(host(x), block, 8), orc.quantize(host(w[torch.from_numpy(cols).cuda()]), block, ww)
    dots = np.einsum("mkb,nkb->kmn", *(q.reshape(len(q), -1, block).astype(np.int64) for q in (qa, qb)))
    scale = ea.T[:, :, None].astype(int) + eb.T[:, None, :].astype(int) - 2 * 127 - (8 - 2) - (ww - 2)
    terms = np.ldexp(dots.astype(np.float32), scale)                         # exact
    chunks = -(-K // (4 * block))
    total = np.zeros((3, len(cols)), np.float32)
    for sl in range(slices):
        first, last = sl * part * parts, min(chunks, (sl + 1) * part * parts)
        in_slice = None
        for p in range(parts):
            acc = np.zeros_like(total)
            for t in terms[4 * min(last, first + p * part):4 * min(last, first + (p + 1) * part)]:
                acc = acc + t
            in_slice = acc if p == 0 else in_slice + acc
        total = total + in_slice
    assert last == chunks
    assert np.array_equal(host(y)[:, cols], total)


@pytest.mark.parametrize("rows,cols", [(512, 1024), (8193, 64), (1, 16)])
def test_minifloat_dequantizer_forms(rows, cols):
    """One item per thread up to 2^19 elements, four past that; the last workgroup full, ragged, and alone."""
    rng = np.random.default_rng(rows)
    x = (rng.standard_normal((rows, cols)) * np.exp2(rng.integers(-20, 20, size=(rows, 1)))).astype(np.float32)
    x[rng.random(x.shape) < 0.05] = 0.0
    for block, e, m in ((16, 4, 3), (8, 7, 0), (16, 1, 6)):
        run_minifloat(x, block, e, m)


def long_attention_inputs(heads, Sq, Sk, dim):
    rng = np.random.default_rng(heads * 1000 + Sk + dim)
    Q = rng.standard_normal((heads, Sq, dim)).astype(np.float32)
    K = rng.standard_normal((heads, Sk, dim)).astype(np.float32)
    V = (rng.standard_normal((heads, Sk, dim)) * rng.choice([0.01, 1.0, 30.0], size=(heads, 1, dim))).astype(np.float32)
    return Q, K, V


@pytest.mark.parametrize("heads,Sq,Sk,dim", [
    (100, 258, 352, 32), (100, 258, 368, 32),      # 900 tiles of 32 queries, eleven key tiles and twelve with a ragged one
    (100, 258, 352, 64), (100, 258, 368, 64),
    (100, 258, 352, 80), (100, 258, 368, 128),
    (500, 258, 352, 64), (500, 258, 368, 48),      # 4500: heads of 33 to 64 without the lag of the second product
    (500, 258, 1056, 64),                          # and with it from 33 key tiles on
    (100, 258, 32, 64), (100, 258, 64, 128), (100, 258, 16, 96), (60, 100, 32, 128),    # one and two key tiles
])
def test_attention_of_128_queries_per_workgroup(heads, Sq, Sk, dim):
    """The key loop past its prologue, with every stage of the ring reused, odd and even numbers of key tiles and a ragged
    last one, a ragged last workgroup of queries; both rounding modes, two-row blocks, a narrow exponent of P and V."""
    Q, K, V = long_attention_inputs(heads, Sq, Sk, dim)
    some = dict(heads_checked=[0, heads // 2, heads - 1])
    run_attention(Q, K, V, (8, 7, 6, 5), dim ** -0.5, rows=(Sq - 34, Sq), **some)
    run_attention(Q, K, V, (7, 8, 5, 6), -0.7 * dim ** -0.5, rows=(0, 34), rounding=mx.MX_RTZ, block_rows=2, **some)
    run_attention(Q, K, V, (8, 7, 8, 6), dim ** -0.5, rows=(Sq - 34, Sq), e_pv=4, **some)


@pytest.mark.parametrize("dim", [32, 64, 128])
@pytest.mark.parametrize("tops", [
    (0, 5, 40, 42, 61, 62, 100, 60, 130, 110, 0),      # rises below and past 20 binades, in odd and even tiles, then falls
    (130, 0, 0, 0, 120, 0, 0, 100, 0, 0, 149),         # a first tile above all until the last, masked, one
    (-90, -110, -71, -100, -69, -50, -49, -48, -29, -28, -27),
])
def test_attention_row_maximum_that_moves(tops, dim):
    """128 queries per workgroup: the sum so far is rescaled whenever a key tile raises the maximum.  tops: the largest score of
    each key tile in binades, the two signs of the scale."""
    heads, Sq, Sk = 100, 258, 336
    rng = np.random.default_rng(dim + abs(tops[1]))
    u = np.full(dim, dim ** -0.5, np.float32)
    Q = (u + 0.02 * rng.standard_normal((heads, Sq, dim))).astype(np.float32)
    top = np.repeat(np.array(tops, np.float32), 32)[:Sk] - 8 * rng.random((heads, Sk)).astype(np.float32)
    K = (np.log(2) / 0.25 * top[:, :, None] * u + 0.1 * rng.standard_normal((heads, Sk, dim))).astype(np.float32)
    V = rng.standard_normal((heads, Sk, dim)).astype(np.float32)
    some = dict(heads_checked=[0, heads - 1], max_maybe=5e-2)
    run_attention(Q, K, V, (8, 8, 6, 5), 0.25, rows=(Sq - 34, Sq), **some)
    run_attention(Q, -K, V, (8, 8, 8, 5), -0.25, rows=(0, 34), block_rows=2, **some)


@pytest.mark.parametrize("heads,Sq,Sk,dim", [(2, 33, 1040, 128), (2, 40, 2032, 64), (3, 5, 1040, 128), (2, 16, 528, 64)])
@pytest.mark.parametrize("tops", [(0, 5, 40, 42, 61, 62, 100, 60), (130, 0, 0, 120, 0, 100, 0, 149), (-90, -110, -71, -69, -50, -48, -29, -27)])
def test_attention_row_maximum_that_moves_with_few_queries(heads, Sq, Sk, dim, tops):
    """The same where eight waves take the key tiles in turn and keep the scores, 33 queries and more and up to sixteen: the tiles
    of a wave rise or fall by tops, one step ahead from wave to wave, the last one is ragged."""
    rng = np.random.default_rng(dim + Sk + abs(tops[1]))
    tile = np.arange(Sk) // 32
    u = np.full(dim, dim ** -0.5, np.float32)
    Q = (u + 0.02 * rng.standard_normal((heads, Sq, dim))).astype(np.float32)
    top = np.array(tops, np.float32)[(tile // 8 + tile) % 8] - 8 * rng.random((heads, Sk)).astype(np.float32)
    K = (np.log(2) / 0.25 * top[:, :, None] * u + 0.1 * rng.standard_normal((heads, Sk, dim))).astype(np.float32)
    V = rng.standard_normal((heads, Sk, dim)).astype(np.float32)
    run_attention(Q, K, V, (8, 8, 6, 5), 0.25, max_maybe=5e-2)
    run_attention(Q, -K, V, (8, 8, 8, 5), -0.25, block_rows=2 if Sq % 2 == 0 else 1, max_maybe=5e-2)


# One shape of every form of the attention kernels: 128 queries per workgroup, split, kept scores and up to sixteen queries, with
# all columns of the result and with 32 of them per workgroup
ATTENTION_KERNELS = [(100, 258, 352, 128), (100, 258, 352, 64), (100, 32, 544, 64), (100, 32, 512, 128), (100, 32, 1024, 128),
                     (60, 32, 2048, 128), (200, 32, 1200, 64), (200, 16, 1024, 128), (100, 16, 608, 64), (40, 13, 2048, 128)]


@pytest.mark.parametrize("heads,Sq,Sk,dim", ATTENTION_KERNELS)
def test_attention_of_a_query_does_not_depend_on_the_others(heads, Sq, Sk, dim):
    """The same bits whether the queries beside it are ordinary ones or have a maximum that rises by 25 binades from key tile to
    key tile (element 0, which is zero in the others)."""
    Q, K, V = long_attention_inputs(heads, Sq, Sk, dim)
    Q[:, :, 0] = 0.0
    K[:, :, 0] = np.arange(Sk) // 32
    others = np.arange(Sq) % 3 == 1
    jump = Q.copy()
    jump[:, others, 0] = 25 * np.log(2) * dim ** 0.5
    alone, beside = (attention_output(q, K, V, (8, 7, 8, 6), dim ** -0.5)[:, ~others] for q in (Q, jump))
    assert np.array_equal(alone.view(np.uint32), beside.view(np.uint32))


@pytest.mark.parametrize("heads,Sq,Sk,dim", ATTENTION_KERNELS)
def test_attention_probability_just_below_a_power_of_two(heads, Sq, Sk, dim):
    """Two keys of score 0 and one, in an earlier tile, d = 19.6 to 19.97 binades below: the row sum is 2 + 2^-d, the two
    probabilities 1/2 less a relative 2^-(d+1), which 8 bits hold as 127/256.  In fp32 the logarithm of that sum is 1 + 7e-7 or
    more, at least five of its last places above 1, as long as the exponentials are taken against the row maximum; against the
    earlier key it is rounded near d + 1, where 7e-7 is less than half a last place, and 128/256 comes out."""
    c = 19.97 / 127                                      # of the exponent in binades
    far, near = -4.0 * 127, np.array([-125.0, -126.0, -127.0], np.float32)
    tops = (8 * 32 + 1, (16 if Sk > 16 * 32 else 9) * 32 + 2)    # with eight waves on the key tiles: those of the first one's wave
    Q, K, V = (np.zeros((heads, n, dim), np.float32) for n in (Sq, Sk, Sk))
    Q[:, :, 0] = 1.0
    K[:, :, 0] = far
    K[:, 0, 0] = near[np.arange(heads) % 3]
    K[:, tops, 0] = 0.0
    V[:, tops] = 1.0
    O = attention_output(Q, K, V, (8, 8, 8, 8), c * np.log(2))
    assert (O == 2 * 127 / 256).all(), (O != 2 * 127 / 256).mean()


@pytest.mark.parametrize("heads,Sq,Sk,dim,R", [(100, 258, 352, 128, 1), (100, 258, 384, 64, 2), (100, 258, 352, 96, 2), (500, 258, 352, 64, 1),
                                               (100, 258, 64, 32, 1)])
def test_attention_of_128_queries_in_blocks_of_32(heads, Sq, Sk, dim, R):
    """P in blocks of 32 keys, one whole key tile, with all tensors quantized in blocks of 32 (entered as blocks of 16)."""
    Q, K, V = long_attention_inputs(heads, Sq, Sk, dim)
    wq, wk, wp, wv = 8, 7, 6, 5

    def operand(x, w, axis):
        mant, exps = mx.quantize(torch.from_numpy(x).cuda(), mx.fmt(32, w, block_rows=R), axis)
        rows, cols = (x.shape[1], x.shape[2]) if axis == 1 else (x.shape[2], x.shape[1])
        if R == 2:
            exps = exps.view(heads, rows // 2, cols // 32).repeat_interleave(2, dim=1).reshape(-1)
        f = mx.fmt(16, w)
        return mx.pack(mant, exps.repeat_interleave(2), heads, rows, cols, f, MAT), f
    A, fq = operand(Q, wq, 1)
    B, fk = operand(K, wk, 1)
    Bv, fv = operand(V, wv, 0)
    fp = mx.fmt(32, wp, block_rows=R)
    O = torch.empty((heads, Sq, dim), device="cuda")
    mx.mx_attention(heads, Sq, Sk, dim, A, fq, B, fk, Bv, fv, fp, dim ** -0.5, MAT, O, dim, Sq * dim)
    torch.cuda.synchronize()
    for hd in (0, heads // 2, heads - 1):
        for rows in ((0, 34), (Sq - 34, Sq)):
            o_ref, info = orc.attention(Q[hd], K[hd], V[hd], 32, wq, wk, wp, wv, dim ** -0.5, 8, mx.MX_RNE, rows, R)
            bound, maybe = attention_bound(info, wp, wv, dim ** -0.5, mx.MX_RNE, 8, block=32)
            assert maybe < 1e-2
            r0, r1 = rows
            assert (np.abs(host(O[hd, r0:r1]).astype(np.float64) - o_ref[r0:r1]) <= bound).all(), (hd, rows)


@pytest.mark.parametrize("heads,Sq,Sk,dim,R", [(3, 6, 352, 128, 1), (3, 12, 1024, 64, 2), (2, 34, 1024, 128, 2), (2, 33, 1056, 64, 1)])
def test_attention_of_few_queries_in_blocks_of_32(heads, Sq, Sk, dim, R):
    """The same with one to sixteen queries and with kept scores."""
    Q, K, V = long_attention_inputs(heads, Sq, Sk, dim)
    A, B = mx.quantize_pack(torch.from_numpy(Q).cuda(), mx.fmt(16, 8), MAT), mx.quantize_pack(torch.from_numpy(K).cuda(), mx.fmt(16, 7), MAT)
    mant, exps = mx.quantize(torch.from_numpy(V).cuda(), mx.fmt(32, 5), 0)
    Bv = mx.pack(mant, exps.repeat_interleave(2), heads, dim, Sk, mx.fmt(16, 5), MAT)
    O = torch.empty((heads, Sq, dim), device="cuda")
    mx.mx_attention(heads, Sq, Sk, dim, A, mx.fmt(16, 8), B, mx.fmt(16, 7), Bv, mx.fmt(16, 5), mx.fmt(32, 6, block_rows=R), dim ** -0.5, MAT,
                    O, dim, Sq * dim)
    torch.cuda.synchronize()
    for hd in (0, heads - 1):
        # Q and K enter the oracle as what blocks of 16 made of them, at a width that holds every one of these values
        q, k = (orc.dequantize(*orc.quantize(x[hd], 16, w), 16, w).astype(np.float32) for x, w in ((Q, 8), (K, 7)))
        s64 = q.astype(np.float64) @ k.astype(np.float64).T * dim ** -0.5
        P = np.exp(s64 - s64.max(axis=1, keepdims=True))
        P = (P / P.sum(axis=1, keepdims=True)).astype(np.float32)
        rows = np.arange(Sq) if R == 1 else np.arange(Sq) ^ 1
        amax = np.maximum(P, P[rows]).reshape(Sq, -1, 32).max(axis=2)
        E = np.floor(np.log2(amax.astype(np.float64)))
        step = np.repeat(np.ldexp(1.0, (E - 4).astype(int)), 32, axis=1)
        x = P / step
        pq = np.minimum(np.round(x), 31) * step
        vabs = np.abs(orc.dequantize(*orc.quantize(V[hd].T.copy(), 32, 5), 32, 5))
        v = orc.dequantize(*orc.quantize(V[hd].T.copy(), 32, 5), 32, 5)
        # eps: 1e-5 of the fp32 softmax and 1e-6 of the terms of a score (below 9 in sum).  A probability that close to a tie may
        # take the neighbouring mantissa, a block maximum that close to a power of two the neighbouring exponent (two steps)
        eps = 2e-5
        frac = np.repeat(amax / np.ldexp(1.0, E.astype(int)), 32, axis=1)
        may = (np.abs(x - np.floor(x) - 0.5) <= eps * np.maximum(x, 1)) + 2.0 * ((frac < 1 + eps) | (frac > 2 - 2 * eps))
        assert may.mean() < 1e-2
        bound = 1e-5 * pq @ vabs.T + (may * step) @ vabs.T + 1e-12
        assert (np.abs(O[hd].cpu().numpy().astype(np.float64) - pq @ v.T) <= bound).all(), hd


@pytest.mark.parametrize("block", [8, 16, 32, 64])
def test_cast_to_nearest_by_any_shift(block):
    """Every width pair, code and tie; blocks of zeros and of one sign; a narrow destination exponent makes the shift anything from
    the widest left one to the widest right one; the tensor ends inside a run of 32 elements for small blocks."""
    rng = np.random.default_rng(970 + block)
    rows, cols = 33, 5 * 64 + (block if block < 32 else 0)
    for ws in range(2, 9):
        for wd in range(2, 9):
            q = rng.integers(-(2 ** (ws - 1)), 2 ** (ws - 1), size=(rows, cols)).astype(np.int8)
            q[::4] //= 2 ** (ws // 2)
            q[3] = 0
            q[5], q[6] = np.maximum(q[5], 0), -(2 ** (ws - 1))
            check_cast(q, rng.integers(0, 256, size=(rows, cols // block)).astype(np.uint8), block, ws, wd)
            ex = rng.integers(112, 144, size=(rows, cols // block)).astype(np.uint8)
            check_cast(q, ex, block, ws, wd, ed=3)


# The forms of the matrix-layout product, (row tiles, column tiles) of 32 and what they select, with K of long_k.  Blocks of 32
# and 64 with pieces of the left by pieces of the right operand; a quantized result takes what 2 x 1 and 1 x 1 take.  "copy":
# with copy waves, "x 2": two workgroups per compute unit.  (Forms that need another K: test_matrix_product_with_deep_stages.)
#                2 x 1             1 x 1             1 x 2             2 x 2             blocks of 16
MATRIX_FORMS_LONG_K = [
    (1, 100),  # 32 x 32, K split over the waves, in all of them
    (2, 200),  # 32 x 64, K split
    (4, 240),  # 64 x 128         128 x 128         128 x 128         64 x 128          64 x 64, K split
    (4, 400),  # the same                                                               64 x 128
    (4, 900),  # 64 x 256         128 x 128         128 x 128         128 x 128 copy    128 x 128
    (4, 1600), # 128 x 256 copy   128 x 256 copy    128 x 256 copy    128 x 128 x 2     128 x 256
    (4, 2400), # 64 x 256         128 x 128         128 x 128         64 x 128          128 x 128: a second round little filled
    (20, 830), # 128 x 256 x 2    128 x 256 x 2     128 x 256 copy    128 x 128 x 2     128 x 256 x 2
]


def exact_operands(g, batch, M, N, K):
    """Small integers whose scale moves by binades from one group of 256 along K to the next, differently on the two sides:
    every product and every sum is a whole number below 2^24, so any order of additions gives the same fp32 result, and a
    scale byte, a stage or a fragment of another K step shows in it."""
    grp = torch.arange(K, device="cuda") // 256
    x = torch.randint(-3, 4, (batch, M, K), generator=g, device="cuda").float() * torch.exp2(((5 * grp) % 4).float())
    w = torch.randint(-3, 4, (batch, N, K), generator=g, device="cuda").float() * torch.exp2(((3 * grp) % 3).float())
    return x, w


def long_k(block):
    """Block 32/64: 30 steps of 64 (29 and a half with blocks of 32), eight groups of four with padding, six turns of five
    stages.  Block 16: 35 steps of 32, the last one half filled, more than five turns of six stages."""
    return {16: 32 * 34 + 16, 32: 64 * 29 + 32, 64: 64 * 30}[block]


@pytest.mark.parametrize("rt,ct", MATRIX_FORMS_LONG_K)
@pytest.mark.parametrize("block,wa,wb", [(16, 8, 4), (32, 8, 4), (64, 6, 3), (32, 4, 3), (64, 3, 8), (32, 5, 6)])
def test_matrix_product_on_long_k(rt, ct, block, wa, wb):
    """Whole results of every form and every combination of mantissa pieces, ragged in rows and columns, ten
    launches each."""
    M, N, K = rt * 32 - 13, ct * 32 - 5, long_k(block)
    g = torch.Generator(device="cuda")
    g.manual_seed(rt * ct)
    x, w = exact_operands(g, 1, M, N, K)
    fa, fb = mx.fmt(block, wa), mx.fmt(block, wb)
    A, B = mx.quantize_pack(x, fa, MAT), mx.quantize_pack(w, fb, MAT)
    want = torch.mm(x[0].double(), w[0].t().double()).float()
    assert want.abs().max() < 2.0 ** 24
    for rep in range(10):
        y = torch.full((M, N + 3), float("nan"), device="cuda")
        mx.mx_gemm(1, M, N, K, A, fa, B, fb, MAT, y, N + 3, 0)
        torch.cuda.synchronize()
        assert torch.equal(y[:, :N], want), "launch %d" % rep
        assert torch.isnan(y[:, N:]).all(), "columns past N written"


@pytest.mark.parametrize("rt,ct", [(r, c // 2) for r, c in MATRIX_FORMS_LONG_K])
@pytest.mark.parametrize("block,wa,wo,rows", [(16, 8, 8, 2), (16, 5, 4, 1), (32, 8, 8, 2), (64, 8, 6, 1), (32, 6, 4, 2), (64, 4, 8, 2),
                                              (32, 3, 4, 1)])
def test_matrix_quantized_output_on_long_k(rt, ct, block, wa, wo, rows):
    """mx_gemm_q over a batch of two in every form, with an MXInt bias and one- and two-row blocks
    of the result, one- and two-piece operands and results: byte for byte what mx_quantize_pack makes of product + bias,
    padding rows and columns included, five launches each."""
    batch, M, K = 2, rt * 32 - 14, long_k(block)
    N = (ct * 32 - 8) // block * block
    g = torch.Generator(device="cuda")
    g.manual_seed(rt * ct + wa)
    x, w = exact_operands(g, batch, M, N, K)
    bias = torch.randint(-3, 4, (1, N), generator=g, device="cuda").float() * 64.0
    fa, fb, fo = mx.fmt(block, wa), mx.fmt(block, 4), mx.fmt(block, wo, block_rows=rows)
    A, B = mx.quantize_pack(x, fa, MAT), mx.quantize_pack(w, fb, MAT)
    y = torch.stack([torch.mm(x[b].double(), w[b].t().double()) for b in range(batch)]).float() + bias
    assert y.abs().max() < 2.0 ** 24
    want = torch.full((mx.mx_packed_bytes(batch, M, N, fo, MAT),), 255, dtype=torch.uint8, device="cuda")
    mx.mx_quantize_pack(y, batch, M, N, N, M * N, fo, MAT, want)
    mant, exps = mx.quantize(bias, fb)
    for rep in range(5):
        out = torch.full_like(want, 255)
        mx.mx_gemm_q(batch, M, N, K, A, fa, B, fb, MAT, mant, exps, fb, fo, out)
        torch.cuda.synchronize()
        assert torch.equal(out, want), "launch %d" % rep


@pytest.mark.parametrize("rt,ct,steps,batch", [
    (4, 400, 52, 1), (4, 400, 61, 1), (4, 400, 55, 1), (4, 200, 55, 2),         # eight stages: 64 x 128 and 128 x 128 with one piece
    (5, 390, 57, 1), (5, 195, 57, 2),                       # the same, 64 x 256 beside it, six stages with two pieces on both sides
    (11, 344, 33, 1), (11, 344, 35, 1), (11, 344, 40, 1), (11, 172, 35, 2),     # 64 x 384 with six stages
    (8, 400, 24, 1),                                        # short K: 64 x 128 and 128 x 128
    (4, 400, 20, 3),                                        # past a batch of two: two pieces on both sides take 128 x 256
])
@pytest.mark.parametrize("block,wa,wb", [(32, 8, 4), (64, 4, 3), (32, 7, 6), (64, 3, 8)])
def test_matrix_product_with_deep_stages(rt, ct, steps, batch, block, wa, wb):
    """The forms with six and eight stages and copy waves (64 x 128, 128 x 128, 64 x 384) and others that this K selects:
    numbers of K steps that fill the last group of four, leave it with one and with three, every stage and every slot of the
    scales reused, alone and over a batch; the quantized ending, whose work the copy waves share, where there is one."""
    M, N, K = rt * 32 - 13, (ct * 32 - 8) // block * block, 64 * steps - (32 if block == 32 else 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(rt * ct + steps)
    x, w = exact_operands(g, batch, M, N, K)
    fa, fb = mx.fmt(block, wa), mx.fmt(block, wb)
    A, B = mx.quantize_pack(x, fa, MAT), mx.quantize_pack(w, fb, MAT)
    want = torch.stack([torch.mm(x[b].double(), w[b].t().double()) for b in range(batch)]).float()
    assert want.abs().max() < 2.0 ** 24
    for rep in range(5):
        y = torch.full((batch, M, N + 3), float("nan"), device="cuda")
        mx.mx_gemm(batch, M, N, K, A, fa, B, fb, MAT, y, N + 3, M * (N + 3))
        torch.cuda.synchronize()
        assert torch.equal(y[:, :, :N], want), "launch %d" % rep
        assert torch.isnan(y[:, :, N:]).all(), "columns past N written"
    if wb > 4:
        return
    bias = torch.randint(-3, 4, (1, N), generator=g, device="cuda").float() * 64.0
    mant, exps = mx.quantize(bias, fb)
    for wo in (8, 4):
        fo = mx.fmt(block, wo)
        packed = torch.full((mx.mx_packed_bytes(batch, M, N, fo, MAT),), 255, dtype=torch.uint8, device="cuda")
        mx.mx_quantize_pack(want + bias, batch, M, N, N, M * N, fo, MAT, packed)
        for rep in range(3):
            out = torch.full_like(packed, 255)
            mx.mx_gemm_q(batch, M, N, K, A, fa, B, fb, MAT, mant, exps, fb, fo, out)
            torch.cuda.synchronize()
            assert torch.equal(out, packed), "width %d, launch %d" % (wo, rep)
