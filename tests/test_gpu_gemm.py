"""GPU parity of the decoder inside a matrix product for many tokens (bof4_gemm) against the oracle, which multiplies
the decoded bfloat16 matrix with x in binary64.

Every product of two bfloat16 numbers is exact in binary32, so the kernels' only roundings are those of their
additions: at most one per column inside the matrix cores' accumulation chain and a few where chains, waves and column
splits are added up - under (cols + 64) roundings of relative size 2^-24 against the sum of the magnitudes of the terms
(an outlier counts with its value: it takes its placeholder's place before the product).  Where every partial sum is a
binary32 number (small integers times powers of two) the result must equal the oracle's bit for bit: that case catches
a term that is dropped, doubled or paired with the wrong x, however small."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_06653_amd import binding, inputs
from test_gpu_parity import cb_for, make_weights
from test_gpu_gemv import dev_i64, dev_u16, quantized, rand_x
from test_host_gemm_plan import rules  # noqa: F401 (a fixture: the host's choice of the kernel)

pytestmark = pytest.mark.gpu
DEV = "cuda"
U = 2.0 ** -24


def run_gpu(cb, codes, scales, oi, ov, rows, cols, block, x):
    cd = torch.from_numpy(codes).to(DEV)
    sd = dev_u16(scales)
    k = 0 if oi is None else int(oi.size)
    packed = binding.bof4_gemm_pack(cd, sd, rows, cols, block)
    if k:
        tab = binding.bof4_gemm_outlier_table(cd, sd, rows, cols, block, cb, dev_i64(oi), dev_u16(ov))
        y = binding.bof4_gemm(packed, rows, cols, cb, x.to(DEV), tab, k)
    else:
        y = binding.bof4_gemm(packed, rows, cols, cb, x.to(DEV))
    torch.cuda.synchronize()
    return y.cpu().numpy().astype(np.float64)


def check(cb, codes, scales, oi, ov, rows, cols, block, x):
    xb = inputs.bits(x).reshape(x.shape)
    st, y_o, a = oracle.gemm(codes, scales, rows, cols, block, cb, xb, oi, ov)
    assert st == oracle.OK
    y_g = run_gpu(cb, codes, scales, oi, ov, rows, cols, block, x)
    assert y_g.shape == y_o.shape
    err = np.abs(y_g - y_o)
    assert np.all(err <= (cols + 64) * U * a + 1e-37), float(np.max(err / (a + 1e-300)))
    return y_g, y_o


@pytest.mark.parametrize("block", [32, 64, 128, 256])
@pytest.mark.parametrize("opq", [0, 1])
@pytest.mark.parametrize("n_tokens", [1, 7, 32, 40, 96, 130, 224])
def test_gemm_parity(block, opq, n_tokens):
    # two row tiles, the second with 5 rows; 36 chunks of 64 columns over 4 workgroups each; token tiles (of 32) taken
    # four, two or one at a time
    rows, cols = 37, 2304
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, opq, seed=900 + block)
    check(cb, codes, scales, oi if opq else None, ov if opq else None, rows, cols, block, rand_x(n_tokens, cols, 7))


@pytest.mark.parametrize("rows,cols", [(1, 32), (3, 64), (130, 6144), (65, 4096 + 2048 + 1024), (33, 32768),
                                       (16390, 128), (16390, 32)])
def test_gemm_shapes(rows, cols):
    """Half a chunk, one chunk, many; the last two have hundreds of row tiles, so that one workgroup takes all columns of
    its rows and writes the result itself."""
    cb, codes, scales, oi, ov = quantized(rows, cols, 32, 0, 1, seed=31 + rows)
    packed_x = 32 * ((cols + 63) // 64 * 64) * 2 + cols * 32 * 2  # in product order, and as much again, 32 token slots
    extra = binding.bof4_gemm_workspace_bytes(rows, cols, 5) - packed_x
    assert 0 <= extra < 512 if (rows > 16000 or cols < 1024) else extra >= 2 * 32 * rows * 4
    check(cb, codes, scales, oi, ov, rows, cols, 32, rand_x(5, cols, 11))


def _random_cases(count, seed):
    rng = np.random.default_rng(seed)
    cases = []
    for i in range(count):
        block = int(rng.choice([32, 64, 128, 256]))
        wide = i % 4 == 3  # every fourth case has 8192 or more columns: two tiles of rows per wave above 32 tokens
        cols = block * int(rng.integers(8192 // block, 8192 // block + 6) if wide else rng.integers(1, 3072 // block + 1))
        rows = int(rng.integers(1, 40 if wide else 200))
        n_tokens = int(rng.choice([1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 200]))
        cases.append((rows, cols, block, n_tokens, int(rng.integers(0, 2)), int(rng.integers(0, 2))))
    return cases


@pytest.mark.parametrize("rows,cols,block,n_tokens,signed,opq", _random_cases(24, seed=2025))
def test_gemm_random_shapes(rows, cols, block, n_tokens, signed, opq):
    """Shapes, block sizes and token counts drawn once from a seeded generator: ragged row tiles, half chunks, every
    number of token tiles per launch."""
    w = make_weights(rows, cols, seed=rows * 7 + cols, outliers=False)
    cb = cb_for(block, signed)
    T = oracle.opq_threshold(0.9, block) if opq else 0.0
    st, codes, scales, oi, ov, k = oracle.quantize(inputs.bits(w), block, cb, signed, opq_T=T)
    assert st == oracle.OK
    lst = (oi, ov) if (opq and k) else (None, None)
    check(cb, codes, scales, lst[0], lst[1], rows, cols, block, rand_x(n_tokens, cols, seed=cols + n_tokens))


@pytest.mark.parametrize("rows,cols,n_tokens", [(33, 32768, 40), (70, 8192, 130), (16390, 128, 70)])
def test_gemm_with_two_tiles_of_rows_per_wave(rows, cols, n_tokens):
    """More than 32 tokens on a matrix with 8192 or more rows or columns: a wave multiplies two tiles of 32 rows with
    every word of x it reads.  Row counts that leave the second tile nearly empty, absent (an odd number of tiles)
    or ragged."""
    cb, codes, scales, oi, ov = quantized(rows, cols, 64, 1, 1, seed=41 + rows)
    check(cb, codes, scales, oi, ov, rows, cols, 64, rand_x(n_tokens, cols, 13))
    check(cb, codes, scales, None, None, rows, cols, 64, rand_x(n_tokens, cols, 14))


@pytest.mark.parametrize("rows,cols,n_tokens", [(70, 1536, 33), (16390, 128, 9), (16390, 128, 45), (70, 8192, 33)])
def test_gemm_is_exact_where_every_partial_sum_is_a_binary32_number(rows, cols, n_tokens):
    """Levels k / 8, constants 2^e, x small integers, list values multiples of 1 / 8: every product and every sum of
    them is a multiple of 2^-9 below 2^15, so no addition rounds, in any order.  (The last two cases take two tiles
    of rows per wave.)"""
    block = 32
    rng = np.random.default_rng(rows)
    cb = (np.arange(16) - 8) / 8.0
    codes = rng.integers(0, 256, rows * cols // 2, dtype=np.uint8)
    top, xmax = (3, 4) if cols <= 2048 else (1, 2)  # |product| <= 2^(top - 1) * xmax, times cols below 2^15
    scales = (2.0 ** rng.integers(-6, top, rows * cols // block)).astype(np.float16).view(np.uint16)
    x = torch.from_numpy(rng.integers(-xmax, xmax + 1, (n_tokens, cols)).astype(np.float32)).to(torch.bfloat16)
    xb = inputs.bits(x).reshape(x.shape)
    oi = np.sort(rng.choice(rows * cols, rows * cols // 300, replace=False)).astype(np.int64)
    ov = (rng.integers(-32, 33, oi.size) / 8.0).astype(np.float16).view(np.uint16)
    for lst in ((None, None), (oi, ov)):
        st, y_o, _ = oracle.gemm(codes, scales, rows, cols, block, cb, xb, *lst)
        assert st == oracle.OK
        y_g = run_gpu(cb, codes, scales, lst[0], lst[1], rows, cols, block, x)
        assert np.array_equal(y_g, y_o)


@pytest.mark.parametrize("n_tokens", [7, 100])
def test_gemm_dense_outlier_rows_take_several_rounds_and_empty_rows_none(n_tokens):
    """A hand-made list: a third of the weights of rows 4..11 (thousands of entries per row), single entries in the
    first and last column elsewhere, nothing in most rows; values unrelated to the codes; a codebook without a zero
    level, so every placeholder decodes to something."""
    rows, cols, block = 40, 6144, 64
    cb, codes, scales, _, _ = quantized(rows, cols, block, 1, 0, seed=77)
    cb = cb + 0.013 * np.linspace(-1, 1, 16) ** 2 + 0.004
    rng = np.random.default_rng(5)
    mask = np.zeros((rows, cols), dtype=bool)
    mask[4:12] = rng.random((8, cols)) < 0.33
    mask[20, 0] = True
    mask[39, cols - 1] = True
    oi = np.flatnonzero(mask.reshape(-1)).astype(np.int64)
    ov = (rng.standard_normal(oi.size).astype(np.float32) * 0.3).astype(np.float16).view(np.uint16)
    x = rand_x(n_tokens, cols, 3)
    y_g, y_o = check(cb, codes, scales, oi, ov, rows, cols, block, x)
    y_none = run_gpu(cb, codes, scales, None, None, rows, cols, block, x)
    touched = np.zeros(rows, dtype=bool)
    touched[4:12] = touched[20] = touched[39] = True
    assert np.array_equal(y_g[:, ~touched], y_none[:, ~touched])  # rows without entries: the dense result, bit for bit
    assert np.max(np.abs(y_g[:, 4:12] - y_none[:, 4:12])) > 1e-3  # the list matters


@pytest.mark.parametrize("rows,cols,k", [(1, 4160, 1), (3, 2112, 2), (17, 8192, 3), (33, 6176, 5), (33, 6176, 3000),
                                         (64, 32768, 4), (40, 64, 2560)])
def test_gemm_list_with_few_entries_and_with_all_positions(rows, cols, k):
    """Row counts for which the list's offsets cover 1, 2, 16 or 32 chunks of 64 columns each (they have to fit the table's
    size), with the matrix's first and last position always listed; the last case lists every position."""
    block = 32
    cb, codes, scales, _, _ = quantized(rows, cols, block, 1, 0, seed=85)
    rng = np.random.default_rng(k)
    oi = rng.choice(rows * cols, k, replace=False)
    oi[: min(k, 2)] = [rows * cols - 1, 0][: min(k, 2)]
    oi = np.unique(oi).astype(np.int64)
    ov = (rng.standard_normal(oi.size).astype(np.float32)).astype(np.float16).view(np.uint16)
    check(cb, codes, scales, oi, ov, rows, cols, block, rand_x(5, cols, 3))


def test_gemm_outlier_table_of_2_to_the_29_rows():
    """More row tiles than a launch of one workgroup of 256 lanes per tile can hold (2^32 lanes): the offsets before and
    behind the entries of the first, a middle and the last tile, and the entries themselves."""
    rows, cols, block = 1 << 29, 32, 32
    codes = torch.zeros(rows * cols // 2, dtype=torch.uint8, device=DEV)
    scales = torch.zeros(rows * cols // block, dtype=torch.float16, device=DEV)
    mid = (1 << 20) * 32 * cols  # the first row tile that a workgroup takes in its second turn
    oi = np.array([5, mid + 33, rows * cols - 1], dtype=np.int64)
    ov = np.array([1.0, 2.0, 3.0], dtype=np.float16)
    tab = binding.bof4_gemm_outlier_table(codes, scales, rows, cols, block, np.linspace(-1, 1, 16), dev_i64(oi),
                                          torch.from_numpy(ov).to(DEV)).view(torch.int32)
    n_tiles = rows // 32
    want = torch.ones(n_tiles + 1, dtype=torch.int32, device=DEV)  # one chunk of columns: one group
    want[0], want[(1 << 20) + 1:], want[-1] = 0, 2, 3
    assert torch.equal(tab[: n_tiles + 1], want)
    at = (rows + 1 + 1) // 2 * 2  # behind one offset per row and the closing one, 8-byte aligned
    place = [5, 1 * 8 + 1, 3 * 512 + 31 * 8 + 7]  # j * 512 + lane * 8 + column % 8: (row, column) (0, 5), (1, 1), (31, 31)
    bits16 = [0x3F80, 0x4000, 0x4040]
    assert tab[at: at + 3].tolist() == [b | p << 16 for b, p in zip(bits16, place)]


@pytest.mark.parametrize("rows,cols,n_tokens", [(70, 4096, 40), (300, 4096, 400)])
def test_gemm_told_another_list_length_than_its_table_was_made_for(rows, cols, n_tokens):
    """Both kernels, row counts for which the offsets' grouping is bound by the table's size: a longer length changes
    nothing, a shorter one (the entries of the first row tile) leaves the other rows without a list."""
    block = 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, 1, seed=87)
    cd, sd = torch.from_numpy(codes).to(DEV), dev_u16(scales)
    tab = binding.bof4_gemm_outlier_table(cd, sd, rows, cols, block, cb, dev_i64(oi), dev_u16(ov))
    packed = binding.bof4_gemm_pack(cd, sd, rows, cols, block)
    x = rand_x(n_tokens, cols, 5).to(DEV)
    k, first = int(oi.size), int(np.searchsorted(oi, 32 * cols))
    assert 64 < first < k
    y = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k)
    assert torch.equal(binding.bof4_gemm(packed, rows, cols, cb, x, tab, k + 12345), y)
    y_first = binding.bof4_gemm(packed, rows, cols, cb, x, tab, first)
    only = [t[:first] for t in (dev_i64(oi), dev_u16(ov))]
    tab_first = binding.bof4_gemm_outlier_table(cd, sd, rows, cols, block, cb, *[t.contiguous() for t in only])
    assert torch.equal(y_first, binding.bof4_gemm(packed, rows, cols, cb, x, tab_first, first))
    assert torch.equal(y_first[:, :32], y[:, :32]) and not torch.equal(y_first, y)


@pytest.mark.parametrize("rows,cols,n_tokens,share", [
    (1, 512, 257, 0.02), (255, 544, 385, 0.01), (257, 1056, 300, 0.01), (520, 512, 512, 0.0), (40, 640, 260, 1.0),
    (33, 6176, 250, 0.004), (96, 8256, 640, 0.01), (256, 13024, 244, 0.006), (16390, 512, 255, 0.001),
    (1, 512, 700, 0.02), (40, 640, 600, 1.0), (33, 6176, 400, 0.004)])
def test_gemm_wide_tile(rows, cols, n_tokens, share):
    """The tile of 256 rows x 128 tokens: one row more and less than a tile, row tiles and token tiles that are absent,
    half chunks of columns, columns split over up to 16 workgroups with 8 to 13 steps each, sums cut after every chunk and
    less often; lists with no, few and (share 1) all positions, and row counts whose offsets cover several chunks each.
    (1 x 512, 40 x 640 and 33 x 6176 are there twice: the fewer tokens go to the other kernel.)  The bound is that of
    every product here."""
    block = 32
    cb, codes, scales, _, _ = quantized(rows, cols, block, 1, 0, seed=91)
    cb = cb + 0.004  # no zero level: every placeholder decodes to something
    rng = np.random.default_rng(rows + cols)
    oi = ov = None
    if share > 0:
        oi = np.sort(rng.choice(rows * cols, int(rows * cols * share), replace=False)).astype(np.int64)
        ov = (rng.standard_normal(oi.size).astype(np.float32)).astype(np.float16).view(np.uint16)
    check(cb, codes, scales, oi, ov, rows, cols, block, rand_x(n_tokens, cols, 3))


def _rms_error_and_bound(rows, cols, n_tokens, listed, chain, split, seed=7):
    """The root mean square error of a product of random codes, over that of the results (binary64 on the GPU); and what
    gemm_kernel makes of it where every entry of the list is added apart from the decoded matrix.  `chain` chunks are 4 *
    chain additions in a row inside the matrix cores, then come eight waves and `split` workgroups; each rounds what has
    been added up so far (2^-24 / sqrt(3), over sqrt(2) for where in its binade a number lies: mean square U^2 / 6).
    The matrix cores also truncate, with one sign: (additions in a row)^2 / 375 roundings more, from dense products of 4 to
    112 in a row, which this formula gives to 4 % from 16 on and to 8 % below.  Listed positions carry half of the
    sums' energy here; added apart, to the sum of one of the `split` workgroups, they halve what is rounded before that
    and add 2.5 roundings (a few terms, then one addition of the two sums); of the additions over the workgroups they are in
    half, as much as the rest's energy is in all.  10 % is for the sample of 10^5 results and more."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    block, n = 64, rows * cols
    codes = torch.randint(0, 256, (n // 2,), generator=g, device=DEV, dtype=torch.uint8)
    scales = (torch.rand(n // block, generator=g, device=DEV) * 0.1 + 0.05).to(torch.float16)
    cb = cb_for(block, 1)
    oi = ov = tab = None
    w = binding.bof4_dequantize(codes, scales, n, block, cb)
    k = n // 150 if listed else 0
    if k:
        oi = torch.unique(torch.randint(0, n, (k,), generator=g, device=DEV))
        k = oi.numel()
        sigma = float(w.double().pow(2).mean().sqrt()) * (n / k) ** 0.5
        ov = (torch.randn(k, generator=g, device=DEV) * sigma).to(torch.float16)
        tab = binding.bof4_gemm_outlier_table(codes, scales, rows, cols, block, cb, oi, ov)
        w = binding.bof4_dequantize(codes, scales, n, block, cb, oi, ov)
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, block)
    x = torch.randn((n_tokens, cols), generator=g, device=DEV).to(torch.bfloat16)
    y = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k).double()
    ref = x.double() @ w.reshape(rows, cols).double().T
    roundings = 4 * chain / 2 + (4 * chain) ** 2 / 375 + 35 / 8
    if listed:
        roundings = roundings / 2 + 2.5
    bound = 1.1 * U / 6 ** 0.5 * (roundings + split / 2) ** 0.5
    print(f"rms error {float((y - ref).norm() / ref.norm()):.3e}, bound {bound:.3e}")
    return float((y - ref).norm() / ref.norm()), bound


@pytest.mark.parametrize("rows,cols,n_tokens,chain,split", [
    (6176, 2112, 20, 5, 1), (12288, 4096, 32, 8, 1), (12288, 4096, 100, 8, 1), (8192, 28672, 8, 28, 2),
    (12320, 2112, 70, 5, 1), (4096, 4096, 100, 4, 2), (16384, 1024, 100, 2, 1), (8000, 1024, 40, 2, 1)])
def test_gemm_with_a_list_rounds_no_more_than_with_the_list_added_apart(rows, cols, n_tokens, chain, split):
    """Both ways of cutting the chain of additions (a second set of accumulators; two runs), odd and even numbers of
    chunks per wave."""
    err, bound = _rms_error_and_bound(rows, cols, n_tokens, True, chain, split)
    assert err <= bound, (err, bound)


@pytest.mark.parametrize("listed", [False, True])
@pytest.mark.parametrize("rows,cols,n_tokens,chain,split", [
    (1024, 1024, 400, 1, 2), (4096, 4096, 640, 4, 2), (4096, 11008, 256, 8, 3), (8192, 8192, 512, 8, 2),
    (28672, 512, 256, 1, 1), (500, 28672, 400, 3, 24), (22016, 4096, 256, 8, 1)])
def test_gemm_wide_tile_rounds_no_more_than_the_other_kernel(rows, cols, n_tokens, chain, split, listed):
    """The tile of 256 rows x 128 tokens, whose workgroups take all columns or an eighth and more of them, against the
    bound of gemm_kernel, whose waves take `chain` chunks each."""
    err, bound = _rms_error_and_bound(rows, cols, n_tokens, listed, chain, split)
    assert err <= bound, (err, bound)


@pytest.mark.parametrize("rows,cols,n_tokens,steps,share", [
    (57344, 8192, 128, 128, 0.006), (24576, 6144, 256, 96, 0.03), (4096, 11008, 2000, 172, 0.006),
    (8192, 8192, 512, 64, 0.0), (16390, 12320, 128, 65, 0.01), (10240, 8192, 120, 22, 0.006)])
def test_gemm_wide_tile_many_steps(rows, cols, n_tokens, steps, share):
    """Up to `steps` chunks of 64 columns per workgroup: the list's offsets are read 64 at a time, two and three times; a tile
    with more than 64 entries; several runs of each chain; one group of 128 tokens, and matrices of more than 2^27
    weights.  Each result against binary64 on the GPU, with the bound of every product here."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + cols)
    block, n = 32, rows * cols
    codes = torch.randint(0, 256, (n // 2,), generator=g, device=DEV, dtype=torch.uint8)
    scales = (torch.rand(n // block, generator=g, device=DEV) * 0.1 + 0.05).to(torch.float16)
    cb = cb_for(block, 1) + 0.004
    oi = ov = tab = None
    k = int(n * share)
    if k:
        oi = torch.unique(torch.randint(0, n, (k,), generator=g, device=DEV))
        k = oi.numel()
        ov = torch.randn(k, generator=g, device=DEV).to(torch.float16)
        tab = binding.bof4_gemm_outlier_table(codes, scales, rows, cols, block, cb, oi, ov)
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, block)
    x = torch.randn((n_tokens, cols), generator=g, device=DEV).to(torch.bfloat16)
    y = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k)
    w = binding.bof4_dequantize(codes, scales, n, block, cb, oi, ov).reshape(rows, cols)
    for r0 in range(0, rows, 8192):
        wd = w[r0: r0 + 8192].double()
        ref, mag = x.double() @ wd.T, x.double().abs() @ wd.abs().T
        worst = float(((y[:, r0: r0 + 8192].double() - ref).abs() / mag).max())
        assert worst <= (cols + 64) * U, (r0, worst / U)


@pytest.mark.parametrize("rows,cols,n_tokens,share,split,wide_split", [
    (4100, 4128, 2001, 0.006, 1, 2), (8001, 1056, 2500, 0.0, 1, 1), (28700, 512, 1900, 0.04, 1, 1),
    (33000, 4160, 1000, 0.002, 1, 1), (4099, 8224, 900, 0.006, 3, 3), (500, 28672, 400, 0.01, 16, 16)])
def test_gemm_decoded_first(rows, cols, n_tokens, share, split, wide_split):
    """Products large enough for the matrix to be decoded first: ragged row tiles, row groups and token groups, half chunks,
    step counts of every remainder in the loop, tiles with more than 64 entries and with none, two slabs, columns split over
    workgroups.  Against binary64 on the GPU with the bound of every product here; and where both split the columns alike,
    bit for bit what the 256 x 128 tile makes of the codes, which a workspace without room for the decoded matrix gets."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + cols)
    block, n = 32, rows * cols
    codes = torch.randint(0, 256, (n // 2,), generator=g, device=DEV, dtype=torch.uint8)
    scales = (torch.rand(n // block, generator=g, device=DEV) * 0.1 + 0.05).to(torch.float16)
    cb = cb_for(block, 1) + 0.004
    oi = ov = tab = None
    k = int(n * share)
    if k:
        oi = torch.unique(torch.randint(0, n // 2, (k,), generator=g, device=DEV))  # (none in the lower half of the rows)
        k = oi.numel()
        ov = torch.randn(k, generator=g, device=DEV).to(torch.float16)
        tab = binding.bof4_gemm_outlier_table(codes, scales, rows, cols, block, cb, oi, ov)
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, block)
    x = torch.randn((n_tokens, cols), generator=g, device=DEV).to(torch.bfloat16)
    need = binding.bof4_gemm_workspace_bytes(rows, cols, n_tokens)
    chunks, n_pad = (cols + 63) // 64, (n_tokens + 31) // 32 * 32
    parts = n_pad * chunks * 128 + (split - 1) * n_tokens * rows * 4  # x in product order, partial results
    assert need > parts + min(n * 2, 120 << 20)  # room for the decoded matrix, or a slab of it
    ws = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
    out = torch.full((n_tokens + 2, rows), float("nan"), device=DEV)
    y = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k, out=out[1:-1], ws=ws[:need])
    assert bool((ws[need:] == 0xFF).all()) and bool(out[0].isnan().all()) and bool(out[-1].isnan().all())
    assert torch.equal(binding.bof4_gemm(packed, rows, cols, cb, x, tab, k), y)
    y_wide = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k, ws=ws[: need - min(n // 2, 60 << 20)])
    assert torch.equal(y_wide, y) == (split == wide_split)
    w = binding.bof4_dequantize(codes, scales, n, block, cb, oi, ov).reshape(rows, cols)
    for r0 in range(0, rows, 8192):
        wd = w[r0: r0 + 8192].double()
        ref, mag = x.double() @ wd.T, x.double().abs() @ wd.abs().T
        worst = float(((y[:, r0: r0 + 8192].double() - ref).abs() / mag).max())
        assert worst <= (cols + 64) * U, (r0, worst / U)


@pytest.mark.parametrize("rows,cols,n_tokens,listed,split,wide_split", [
    (12288, 4096, 700, False, 1, 0), (7824, 4736, 1050, False, 1, 0), (6978, 4128, 1197, False, 1, 2),
    (5970, 23808, 1065, True, 2, 1), (12230, 7392, 702, True, 2, 3)])
def test_gemm_decoded_first_rounds_no_more_than_the_kernel_it_replaces(rules, rows, cols, n_tokens, listed, split, wide_split):
    """The root mean square error of products that are decoded first and split otherwise, against binary64, next to that of the kernel
    which the call takes in a workspace one byte too small for it; half a per cent is several times what the sample of more
    than 10^6 results leaves open."""
    plan = rules(rows, cols, n_tokens, listed)
    assert (plan.way, plan.decoded_split, plan.wide_split) == (2, split, wide_split)
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    block, n = 32, rows * cols
    codes = torch.randint(0, 256, (n // 2,), generator=g, device=DEV, dtype=torch.uint8)
    scales = (torch.rand(n // block, generator=g, device=DEV) * 0.1 + 0.05).to(torch.float16)
    cb = cb_for(64, 1)
    oi = ov = tab = None
    k = 0
    if listed:  # half of the energy in the list
        sigma = float(binding.bof4_dequantize(codes, scales, n, block, cb).float().pow(2).mean().sqrt()) * 150 ** 0.5
        oi = torch.unique(torch.randint(0, n, (n // 150,), generator=g, device=DEV))
        k = oi.numel()
        ov = (torch.randn(k, generator=g, device=DEV) * sigma).to(torch.float16)
        tab = binding.bof4_gemm_outlier_table(codes, scales, rows, cols, block, cb, oi, ov)
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, block)
    x = torch.randn((n_tokens, cols), generator=g, device=DEV).to(torch.bfloat16)
    ref = x.double() @ binding.bof4_dequantize(codes, scales, n, block, cb, oi, ov).reshape(rows, cols)[:2048].double().T
    ws = torch.empty(plan.need, dtype=torch.uint8, device=DEV)
    err = []
    for size in (plan.need, plan.need - 1):
        y = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k, ws=ws[:size])
        err.append(float((y[:, :2048].double() - ref).norm() / ref.norm()))
    print(f"rms error {err[0]:.3e}, of the other kernel {err[1]:.3e}")
    assert err[0] <= 1.005 * err[1]


@pytest.mark.parametrize("listed", [False, True])
@pytest.mark.parametrize("rows,cols,n_tokens,split,carry", [
    (4100, 1056, 2500, 1, 1), (8001, 1056, 2500, 1, 0), (4096, 4096, 1200, 1, 1), (4096, 11008, 900, 2, 1), (8193, 8192, 900, 2, 1)])
def test_gemm_decoded_first_exact_sums_unit_vectors_and_sums_that_are_not_finite(rules, rows, cols, n_tokens, split, carry, listed):
    """The decoded kernels with and without carried sums (`carry`: without a list), one part and two.  Levels k / 8, constants 2^e, x
    small integers, list values multiples of 1 / 8: every product and every sum is a multiple of 2^-9 below 2^15, so that no
    addition rounds and binary64 on the GPU has the same numbers.  Then a unit vector per token, which picks one column of the
    decoded matrix; and infinite and undefined terms early, at the edge of a chunk and late, which leave the other tokens as
    they are."""
    plan = rules(rows, cols, n_tokens, listed)
    assert (plan.way, plan.decoded_split, plan.decoded_carry) == (2, split, 1 if listed else carry)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + cols)
    block, n = 32, rows * cols
    cb = (np.arange(16) - 8) / 8.0
    codes = torch.randint(0, 256, (n // 2,), generator=g, device=DEV, dtype=torch.uint8)
    xmax = 4 if cols <= 2048 else 1  # |product| <= 4 * xmax or xmax, times cols below 2^15
    scales = torch.exp2(torch.randint(-6, 3 if cols <= 2048 else 1, (n // block,), generator=g, device=DEV).float()).to(torch.float16)
    oi = ov = tab = None
    k = 0
    if listed:
        oi = torch.unique(torch.randint(0, n, (n // 300,), generator=g, device=DEV))
        k = oi.numel()
        top = 32 if cols <= 2048 else 8
        ov = (torch.randint(-top, top + 1, (k,), generator=g, device=DEV).float() / 8).to(torch.float16)
        tab = binding.bof4_gemm_outlier_table(codes, scales, rows, cols, block, cb, oi, ov)
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, block)
    w = binding.bof4_dequantize(codes, scales, n, block, cb, oi, ov).reshape(rows, cols).double()
    x = torch.randint(-xmax, xmax + 1, (n_tokens, cols), generator=g, device=DEV).to(torch.bfloat16)
    ref = x.double() @ w.T
    assert float((x.double().abs() @ w.abs().T).max()) < 2 ** 15
    y = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k)
    assert torch.equal(y.double(), ref)
    bad = {3: (0, "inf"), 130: (63, "-inf"), 131: (cols // 2, "nan"), n_tokens - 1: (cols - 1, "inf")}
    for t, (c, v) in bad.items():
        x[t, c] = float(v)
    z = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k)
    rest = torch.ones(n_tokens, dtype=torch.bool, device=DEV)
    rest[list(bad)] = False
    want = x[~rest].double() @ w.T
    assert torch.equal(z[rest], y[rest]) and not bool(want.isfinite().any())
    assert torch.equal(z[~rest].double().nan_to_num(nan=7.0), want.nan_to_num(nan=7.0))
    picks = torch.arange(n_tokens, device=DEV) * 61 % cols
    x.zero_()
    x[torch.arange(n_tokens, device=DEV), picks] = 1.0
    assert torch.equal(binding.bof4_gemm(packed, rows, cols, cb, x, tab, k).double(), w[:, picks].T)


@pytest.mark.parametrize("rows,cols,n_tokens", [(300, 2304, 330), (520, 512, 600)])
def test_gemm_wide_tile_is_exact_where_every_partial_sum_is_a_binary32_number(rows, cols, n_tokens):
    """As for the other kernel: levels k / 8, constants 2^e, x small integers, list values multiples of 1 / 8, so that no
    addition rounds, in any order."""
    block = 32
    rng = np.random.default_rng(rows)
    cb = (np.arange(16) - 8) / 8.0
    codes = rng.integers(0, 256, rows * cols // 2, dtype=np.uint8)
    scales = (2.0 ** rng.integers(-6, 3, rows * cols // block)).astype(np.float16).view(np.uint16)
    x = torch.from_numpy(rng.integers(-4, 5, (n_tokens, cols)).astype(np.float32)).to(torch.bfloat16)
    xb = inputs.bits(x).reshape(x.shape)
    oi = np.sort(rng.choice(rows * cols, rows * cols // 300, replace=False)).astype(np.int64)
    ov = (rng.integers(-32, 33, oi.size) / 8.0).astype(np.float16).view(np.uint16)
    for lst in ((None, None), (oi, ov)):
        st, y_o, _ = oracle.gemm(codes, scales, rows, cols, block, cb, xb, *lst)
        assert st == oracle.OK
        assert np.array_equal(run_gpu(cb, codes, scales, lst[0], lst[1], rows, cols, block, x), y_o)


def test_gemm_wide_tile_unit_vectors_pick_single_decoded_weights():
    """x = a unit vector per token, at every 61st column: one column of the decoded matrix per token, exactly."""
    rows, cols, block, n_tokens = 300, 2304, 64, 330
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, 1, seed=93)
    picks = np.arange(n_tokens) * 61 % cols
    x = torch.zeros((n_tokens, cols), dtype=torch.bfloat16)
    x[torch.arange(n_tokens), torch.from_numpy(picks)] = 1.0
    y = run_gpu(cb, codes, scales, oi, ov, rows, cols, block, x)
    st, deq = oracle.dequantize(codes, scales, rows * cols, block, cb, oi, ov)
    assert st == oracle.OK
    w_hat = (deq.astype(np.uint32) << 16).view(np.float32).reshape(rows, cols).astype(np.float64)
    assert np.array_equal(y, w_hat[:, picks].T)


@pytest.mark.parametrize("rows,cols,n_tokens", [(300, 2304, 330), (16390, 512, 255)])
def test_gemm_wide_tile_is_bit_reproducible_and_respects_out_workspace_and_stream(rows, cols, n_tokens):
    """Columns split over four workgroups, and not split."""
    block = 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, 1, seed=94)
    cd, sd = torch.from_numpy(codes).to(DEV), dev_u16(scales)
    tab = binding.bof4_gemm_outlier_table(cd, sd, rows, cols, block, cb, dev_i64(oi), dev_u16(ov))
    packed = binding.bof4_gemm_pack(cd, sd, rows, cols, block)
    x = rand_x(n_tokens, cols, 5).to(DEV)
    y1 = binding.bof4_gemm(packed, rows, cols, cb, x, tab, oi.size)
    guarded = torch.full((n_tokens + 2, rows), float("nan"), device=DEV)
    out = guarded[1:-1]
    ws = torch.full((binding.bof4_gemm_workspace_bytes(rows, cols, n_tokens),), 0xFF, dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        y2 = binding.bof4_gemm(packed, rows, cols, cb, x, tab, oi.size, out=out, ws=ws)
    side.synchronize()
    torch.cuda.synchronize()
    assert y2 is out and torch.equal(y1, y2)
    assert bool(guarded[0].isnan().all()) and bool(guarded[-1].isnan().all())


@pytest.mark.parametrize("opq", [0, 1])
@pytest.mark.parametrize("rows,cols,n_tokens", [(300, 2304, 330), (6176, 2304, 40), (12320, 2304, 70)])
def test_gemm_cut_chains_with_sums_that_are_not_finite(rows, cols, n_tokens, opq):
    """Infinite and undefined sums come out as binary64 has them, from chains of additions that were cut before, at and
    after the term that makes them so; the other tokens are what they are without.  The wide tile, and gemm_kernel with
    a second set of accumulators and in two runs."""
    block = 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, opq, seed=92)
    lst = (oi, ov) if opq else (None, None)
    x = rand_x(n_tokens, cols, 17)
    y_clean = run_gpu(cb, codes, scales, lst[0], lst[1], rows, cols, block, x)
    bad = {2: [(0, "inf")], 5: [(3, "nan")], 11: [(1151, "-inf")], 17: [(64, "inf")], 20: [(2303, "inf")],
           33: [(10, "inf"), (1300, "inf")], n_tokens - 1: [(700, "inf"), (701, "-inf"), (2000, "inf")]}
    for t, terms in bad.items():
        for c, v in terms:
            x[t, c] = float(v)
    y = run_gpu(cb, codes, scales, lst[0], lst[1], rows, cols, block, x)
    xb = inputs.bits(x).reshape(x.shape)
    st, y_o, _ = oracle.gemm(codes, scales, rows, cols, block, cb, xb, *lst)
    assert st == oracle.OK
    rest = np.ones(n_tokens, dtype=bool)
    rest[list(bad)] = False
    assert np.array_equal(y[rest], y_clean[rest])
    assert np.isinf(y_o[~rest]).any() and np.isnan(y_o[~rest]).any() and not np.isfinite(y_o[~rest]).any()
    assert np.array_equal(y[~rest], y_o[~rest], equal_nan=True)


@pytest.mark.parametrize("rows,cols,n_tokens", [(6176, 2112, 5), (12320, 2112, 100)])
def test_gemm_with_a_list_and_several_chunks_per_wave(rows, cols, n_tokens):
    """33 chunks over eight waves, so that one wave takes five and the others four: cut after two, or into runs of three
    and two."""
    cb, codes, scales, oi, ov = quantized(rows, cols, 64, 1, 1, seed=89)
    check(cb, codes, scales, oi, ov, rows, cols, 64, rand_x(n_tokens, cols, 15))


@pytest.mark.parametrize("opq", [0, 1])
def test_gemm_a_token_that_is_not_finite_stays_on_its_own(opq):
    """One token carries an infinity: its own results are not finite (every row multiplies it), every other token's are
    what they are without it - nothing leaks through padding, clamped list slots or shared registers."""
    rows, cols, block = 70, 2304, 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, opq, seed=91)
    lst = (oi, ov) if opq else (None, None)
    x = rand_x(37, cols, 17)
    y_clean = run_gpu(cb, codes, scales, lst[0], lst[1], rows, cols, block, x)
    x[5, 1000] = float("inf")
    x[33, 3] = float("nan")
    y = run_gpu(cb, codes, scales, lst[0], lst[1], rows, cols, block, x)
    bad = np.zeros(37, dtype=bool)
    bad[[5, 33]] = True
    assert not np.isfinite(y[bad]).any()
    assert np.array_equal(y[~bad], y_clean[~bad])


@pytest.mark.parametrize("rows,cols,n_tokens", [(70, 96, 1), (70, 2336, 5), (33, 32, 8), (300, 1056, 31), (8200, 2080, 6)])
def test_gemm_x_read_in_place_takes_nothing_from_the_next_token(rows, cols, n_tokens):
    """Few tokens and half a chunk at the end of every row of x: what follows there is the next token, not finite here, or
    the end of the buffer.  (Small matrices, and one of 8192 rows and more with few tokens.)"""
    cb, codes, scales, _, _ = quantized(rows, cols, 32, 1, 0, seed=97)
    x = rand_x(n_tokens, cols, 17)
    y_clean, _ = check(cb, codes, scales, None, None, rows, cols, 32, x)
    x[1::2] = float("nan")
    y = run_gpu(cb, codes, scales, None, None, rows, cols, 32, x)
    assert np.array_equal(y[::2], y_clean[::2]) and np.isnan(y[1::2]).all()


def test_gemm_x_read_in_place_with_two_tiles_of_rows_per_wave():
    """No list, few tokens, a matrix of 2^27 weights and more with half a chunk at the end of its rows: the bound of every product
    here, and nothing from the neighbouring tokens."""
    rows, cols, n_tokens = 8224, 16352, 5
    g = torch.Generator(device=DEV)
    g.manual_seed(99)
    codes = torch.randint(0, 256, (rows * cols // 2,), generator=g, device=DEV, dtype=torch.uint8)
    scales = (torch.rand(rows * cols // 32, generator=g, device=DEV) * 0.1 + 0.05).to(torch.float16)
    cb = cb_for(32, 1) + 0.004
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, 32)
    x = torch.randn((n_tokens, cols), generator=g, device=DEV).to(torch.bfloat16)
    y = binding.bof4_gemm(packed, rows, cols, cb, x)
    w = binding.bof4_dequantize(codes, scales, rows * cols, 32, cb).reshape(rows, cols)
    for r0 in range(0, rows, 2048):
        wd = w[r0: r0 + 2048].double()
        ref, mag = x.double() @ wd.T, x.double().abs() @ wd.abs().T
        assert bool(((y[:, r0: r0 + 2048].double() - ref).abs() <= (cols + 64) * U * mag).all())
    x[1::2] = float("nan")
    z = binding.bof4_gemm(packed, rows, cols, cb, x)
    assert torch.equal(z[::2], y[::2]) and bool(z[1::2].isnan().all())


def test_gemm_unit_vectors_pick_single_decoded_weights():
    """x = a unit vector per token: the product returns one column of the decoded matrix, exactly."""
    rows, cols, block = 45, 2304, 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, 1, seed=79)
    picks = [0, 1, 7, 8, 31, 32, 63, 64, 65, 2049, 2303]
    x = torch.zeros((len(picks), cols), dtype=torch.bfloat16)
    for t, c in enumerate(picks):
        x[t, c] = 1.0
    y_g, y_o = check(cb, codes, scales, oi, ov, rows, cols, block, x)
    st, deq = oracle.dequantize(codes, scales, rows * cols, block, cb, oi, ov)
    assert st == oracle.OK
    w_hat = (deq.astype(np.uint32) << 16).view(np.float32).reshape(rows, cols).astype(np.float64)
    assert np.array_equal(y_g, w_hat[:, picks].T)


def test_gemm_on_the_quantisers_output_equals_the_product_over_the_decoders_output():
    rows, cols, block = 257, 4096, 64
    w = inputs.student_t_matrix(rows, cols, 5.0, 0.02, 0.3, seed=5).reshape(-1).to(DEV)
    cb = cb_for(block, 1)
    T = oracle.opq_threshold(0.95, block)
    codes, scales, oi, ov, k = binding.bof4_quantize(w, block, cb, 1, opq_T=T, out_capacity=w.numel() // 20)
    assert k > 0
    tab = binding.bof4_gemm_outlier_table(codes, scales, rows, cols, block, cb, oi, ov, n_outliers=k)
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, block)
    x = rand_x(48, cols, 21).to(DEV)
    y = binding.bof4_gemm(packed, rows, cols, cb, x, tab, k)
    deq = binding.bof4_dequantize(codes, scales, w.numel(), block, cb, oi, ov, n_outliers=k).reshape(rows, cols)
    ref = x.double() @ deq.double().T
    mag = x.double().abs() @ deq.double().abs().T
    assert torch.all((y.double() - ref).abs() <= (cols + 64) * U * 2 * mag)


def test_gemm_is_bit_reproducible_and_respects_out_workspace_and_stream():
    rows, cols, block = 130, 4096, 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, 1, seed=80)
    cd, sd, oid, ovd = torch.from_numpy(codes).to(DEV), dev_u16(scales), dev_i64(oi), dev_u16(ov)
    tab = binding.bof4_gemm_outlier_table(cd, sd, rows, cols, block, cb, oid, ovd)
    packed = binding.bof4_gemm_pack(cd, sd, rows, cols, block)
    x = rand_x(35, cols, 5).to(DEV)
    y1 = binding.bof4_gemm(packed, rows, cols, cb, x, tab, oi.size)
    out = torch.full((35, rows), float("nan"), device=DEV)
    ws = torch.empty(binding.bof4_gemm_workspace_bytes(rows, cols, 35), dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        y2 = binding.bof4_gemm(packed, rows, cols, cb, x, tab, oi.size, out=out, ws=ws)
    side.synchronize()
    torch.cuda.synchronize()
    assert y2 is out and torch.equal(y1, y2)
    # one token alone gives the same numbers as inside a batch
    y3 = binding.bof4_gemm(packed, rows, cols, cb, x[33:34].contiguous(), tab, oi.size)
    assert torch.equal(y3[0], y1[33])


@pytest.mark.parametrize("rows,cols,n_max,n_tokens", [(1024, 1024, 2000, 1030), (1000, 2048, 700, 350)])
def test_gemm_workspace_of_more_tokens_and_of_the_least_size(rows, cols, n_max, n_tokens):
    """A buffer for more tokens gives the same bits as the call's own; one of the least size (x twice, and the partial
    results of gemm_kernel: two or four workgroups per row tile here, at most 128 tokens) is enough, and nothing behind
    it is touched."""
    block = 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, 1, seed=88)
    cd, sd = torch.from_numpy(codes).to(DEV), dev_u16(scales)
    tab = binding.bof4_gemm_outlier_table(cd, sd, rows, cols, block, cb, dev_i64(oi), dev_u16(ov))
    packed = binding.bof4_gemm_pack(cd, sd, rows, cols, block)
    x = rand_x(n_tokens, cols, 6)
    xd = x.to(DEV)

    def run(ws_bytes):
        ws = torch.full((ws_bytes + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
        y = binding.bof4_gemm(packed, rows, cols, cb, xd, tab, int(oi.size), ws=ws[:ws_bytes])
        assert bool((ws[ws_bytes:] == 0x5A).all())
        return y

    y = run(binding.bof4_gemm_workspace_bytes(rows, cols, n_tokens))
    assert torch.equal(run(binding.bof4_gemm_workspace_bytes(rows, cols, n_max)), y)
    split = {1024: 2, 2048: 4}[cols]  # 16 or 32 chunks of 64 columns, at least eight per workgroup; 32 row tiles for 192
    least = 4 * ((n_tokens + 31) // 32 * 32) * cols + split * 128 * rows * 4
    y_least = run(least)
    with pytest.raises(binding.Bof4Error) as e:
        run(least - 256)
    assert e.value.code == binding.BOF4_ERR_WORKSPACE
    st, y_o, a = oracle.gemm(codes, scales, rows, cols, block, cb, inputs.bits(x).reshape(x.shape), oi, ov)
    assert st == oracle.OK
    for got in (y, y_least):
        assert np.all(np.abs(got.cpu().numpy() - y_o) <= (cols + 64) * U * a)
    assert not torch.equal(y, y_least)  # the least size takes the other kernel


@pytest.mark.parametrize("rows,cols,n_tokens,n_max", [(13551, 2240, 566, 2500), (4471, 1568, 1159, 2500), (1594, 3808, 2273, 2500)])
def test_gemm_without_a_list_gives_the_same_bits_in_a_workspace_of_its_own_and_of_more_tokens(rows, cols, n_tokens, n_max):
    """Products that are decoded first, or nearly, without a list and not (or elsewhere) with one."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)
    codes = torch.randint(0, 256, (rows * cols // 2,), generator=g, device=DEV, dtype=torch.uint8)
    scales = (torch.rand(rows * cols // 32, generator=g, device=DEV) * 0.1 + 0.05).to(torch.float16)
    packed = binding.bof4_gemm_pack(codes, scales, rows, cols, 32)
    x = torch.randn((n_tokens, cols), generator=g, device=DEV).to(torch.bfloat16)
    ys = []
    for n in (n_tokens, n_max):
        ws = torch.empty(binding.bof4_gemm_workspace_bytes(rows, cols, n), dtype=torch.uint8, device=DEV)
        ys.append(binding.bof4_gemm(packed, rows, cols, cb_for(32, 1), x, ws=ws))
    assert torch.equal(*ys)


def test_gemm_pack_layout():
    """Per tile of 32 rows and 64 columns: 64 words of 16 bytes (row lane % 32, columns 32 (lane / 32) .. + 31), then
    64 constants; zeros past the last row and the last column."""
    rows, cols, block = 45, 2304 + 32, 32  # a ragged row tile and half a chunk at the end
    cb, codes, scales, _, _ = quantized(rows, cols, block, 1, 0, seed=83)
    packed = binding.bof4_gemm_pack(torch.from_numpy(codes).to(DEV), dev_u16(scales), rows, cols, block).cpu().numpy()
    n_chunks = (cols + 63) // 64
    assert packed.size == binding.bof4_gemm_packed_bytes(rows, cols) == 2 * n_chunks * (1024 + 128)
    tiles = packed.reshape(2, n_chunks, 1152)
    code_rows = codes.reshape(rows, cols // 2)
    scale_rows = scales.reshape(rows, cols // block)
    for rt, ch, lane in [(0, 0, 0), (0, 0, 33), (0, 5, 63), (1, 7, 12), (1, 36, 3), (1, 36, 35), (1, 2, 13), (1, 2, 45)]:
        row, c = rt * 32 + lane % 32, ch * 64 + 32 * (lane // 32)
        got_q = tiles[rt, ch, 16 * lane: 16 * lane + 16]
        got_m = tiles[rt, ch, 1024 + 2 * lane: 1024 + 2 * lane + 2].view(np.uint16)[0]
        if row < rows and c < cols:
            assert np.array_equal(got_q, code_rows[row, c // 2: c // 2 + 16]) and got_m == scale_rows[row, c // block]
        else:
            assert not got_q.any() and got_m == 0


def test_gemm_argument_errors():
    rows, cols, block = 64, 2048, 64
    cb, codes, scales, oi, ov = quantized(rows, cols, block, 1, 1, seed=81)
    cd, sd = torch.from_numpy(codes).to(DEV), dev_u16(scales)
    x = rand_x(3, cols, 1).to(DEV)
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_gemm_pack(cd, sd, rows, 96, 64)
    assert e.value.code == binding.BOF4_ERR_ARG
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_gemm_pack(cd, sd, rows, cols, 48)
    assert e.value.code == binding.BOF4_ERR_ARG
    with pytest.raises(binding.Bof4Error) as e:  # codes not 16-byte aligned
        binding.bof4_gemm_pack(cd[4:], sd, rows - 1, cols, block)
    assert e.value.code == binding.BOF4_ERR_ARG
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_gemm_pack(cd, sd, rows, cols, block, out=torch.empty(1152 * 63, dtype=torch.uint8, device=DEV))
    assert e.value.code == binding.BOF4_ERR_WORKSPACE
    packed = binding.bof4_gemm_pack(cd, sd, rows, cols, block)
    need = binding.bof4_gemm_workspace_bytes(rows, cols, 3)
    # x twice (in product order, and as much again, 32 token slots), then the partial results of four workgroups per row
    # tile (32 chunks of 64 columns, eight waves each)
    assert need == 2 * 32 * cols * 2 + 4 * 32 * rows * 4
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_gemm(packed, rows, cols, cb, x, ws=torch.empty(need - 256, dtype=torch.uint8, device=DEV))
    assert e.value.code == binding.BOF4_ERR_WORKSPACE
    with pytest.raises(ValueError):
        binding.bof4_gemm(packed, rows, cols, cb, x, None, 3)  # outliers without their table
    with pytest.raises(ValueError):
        binding.bof4_gemm(packed, rows, cols, cb, x.float())
    with pytest.raises(ValueError):
        binding.bof4_gemm(packed, rows + 1, cols, cb, x)  # a packed copy of fewer row tiles
    big = 32768 + 2048
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_gemm(torch.zeros(binding.bof4_gemm_packed_bytes(1, big), dtype=torch.uint8, device=DEV), 1, big, cb,
                          torch.zeros((1, big), dtype=torch.bfloat16, device=DEV))
    assert e.value.code == binding.BOF4_ERR_ARG
    bad_cb = cb.copy()
    bad_cb[3] = bad_cb[4]
    with pytest.raises(binding.Bof4Error):
        binding.bof4_gemm(packed, rows, cols, bad_cb, x)


@pytest.mark.parametrize("rows,cols,n_tokens", [(4096, 4096, 32), (4096, 11008, 32), (11008, 4096, 64),
                                                (8192, 28672, 8)])
def test_gemm_llama_matrices_with_opq(rows, cols, n_tokens):
    """The three matrix shapes of workload 1 and the widest one of workload 4 at full size, signed constants, block 64,
    OPQ q = 0.95: every output against the oracle."""
    wm = inputs.student_t_matrix(rows, cols, 5.0, 0.02, 0.3, seed=rows + cols)
    cb = cb_for(64, 1)
    T = oracle.opq_threshold(0.95, 64)
    st, codes, scales, oi, ov, k = oracle.quantize(inputs.bits(wm.reshape(-1)), 64, cb, 1, opq_T=T)
    assert st == oracle.OK and k > 1000
    check(cb, codes, scales, oi, ov, rows, cols, 64, rand_x(n_tokens, cols, 9))
