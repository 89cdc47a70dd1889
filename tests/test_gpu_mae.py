"""GPU parity of the MAE-criterion Lloyd step (weighted medians) against the oracle: medians, counts and masses
bit-exact, the error sum to relative 1e-9."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_06653_amd import binding, codebooks, inputs
from test_gpu_parity import cb_for, make_weights

pytestmark = pytest.mark.gpu
DEV = "cuda"
RTOL = 1e-9


def mae_cb(block, signed):
    return codebooks.array(codebooks.BOF4S_MAE_64 if signed else codebooks.BOF4_MAE_64)


def assert_mae_close(g, o):
    assert np.array_equal(g["cnt"], o["cnt"])
    assert g["n_used"] == o["n_used"] and g["n_outliers"] == o["n_outliers"]
    assert np.array_equal(g["den"], o["den"])
    assert np.array_equal(np.isnan(g["median"]), np.isnan(o["median"]))
    ok = ~np.isnan(o["median"])
    assert np.array_equal(g["median"][ok], o["median"][ok])  # a median is one of the binary32 samples: exact
    assert abs(g["sae"] - o["sae"]) <= RTOL * o["sae"]


@pytest.mark.parametrize("block", [32, 64, 128, 256])
@pytest.mark.parametrize("signed", [0, 1])
@pytest.mark.parametrize("opq", [0, 1])
def test_mae_step_parity(block, signed, opq):
    w = make_weights(29, 1024, seed=500 + block + signed)  # 14.5 wave tiles, ragged tail
    T = oracle.opq_threshold(0.95, block) if opq else 0.0
    cb = mae_cb(block, signed)
    st, o = oracle.lloyd_step_mae(inputs.bits(w), block, cb, signed, opq_T=T)
    assert st == oracle.OK
    g = binding.bof4_lloyd_step_mae(w.to(DEV), block, cb, signed, opq_T=T)
    assert (o["n_outliers"] > 0) == bool(opq)
    assert_mae_close(g, o)


@pytest.mark.parametrize("block", [32, 64, 256])
@pytest.mark.parametrize("signed", [0, 1])
@pytest.mark.parametrize("opq", [0, 1])
def test_mae_step_without_weights_parity(block, signed, opq):
    """Appendix D's objective (weight_by_max = 0): plain medians of the normalised weights, den = counts,
    sae = sum |x - level|.  2^17 weights, so that the search reads its list in the third pass."""
    w = make_weights(128, 1024, seed=540 + block + signed)
    T = oracle.opq_threshold(0.95, block) if opq else 0.0
    cb = mae_cb(block, signed)
    st, o = oracle.lloyd_step_mae(inputs.bits(w), block, cb, signed, opq_T=T, weight_by_max=False)
    st2, ow = oracle.lloyd_step_mae(inputs.bits(w), block, cb, signed, opq_T=T)
    assert st == oracle.OK and np.any(o["median"] != ow["median"])
    pin = codebooks.PIN_BOF4S if signed else codebooks.PIN_BOF4
    for skip in (0, pin):
        g = binding.bof4_lloyd_step_mae(w.to(DEV), block, cb, signed, opq_T=T, weight_by_max=False, skip_mask=skip)
        if skip:
            wanted = np.array([not ((skip >> l) & 1) for l in range(16)])
            assert np.all(np.isnan(g["median"][~wanted]))
            assert np.array_equal(g["median"][wanted], o["median"][wanted])
            assert np.array_equal(g["den"], o["den"]) and np.array_equal(g["cnt"], o["cnt"])
            assert abs(g["sae"] - o["sae"]) <= RTOL * o["sae"]
        else:
            assert_mae_close(g, o)


def test_mae_em_iterations_follow_the_oracle():
    """Twelve EM iterations with the MAE criterion from the quantile start: same codebooks as the oracle at every
    step (the medians are exact), objective never rising."""
    w = inputs.gaussian_blocks(1 << 12, 64, seed=77)
    wb, wd = inputs.bits(w), w.to(DEV)
    cb_g = cb_o = codebooks.gaussian_quantile_init()
    prev = None
    for it in range(12):
        g = binding.bof4_lloyd_step_mae(wd, 64, cb_g, 1)
        st, o = oracle.lloyd_step_mae(wb, 64, cb_o, 1)
        assert_mae_close(g, o)
        mae = g["sae"] / g["n_used"]
        assert prev is None or mae <= prev * (1 + 1e-12)
        prev = mae
        cb_g = binding.bof4_codebook_update_mae(g, codebooks.PIN_BOF4S, cb_g)
        cb_o = oracle.codebook_update_mae(o, codebooks.PIN_BOF4S, cb_o)
        assert np.array_equal(cb_g, cb_o)


def test_mae_degenerate_inputs():
    """All-zero blocks (no weight: NaN medians, counts still right), a constant tensor, many equal values, blocks whose
    maxima differ by 2^20, and a region that stays empty.  The constant tensor and the one of six values put every
    element on the list of candidates, which runs full: the passes after it fall back to scanning the weights."""
    cb = mae_cb(64, 1)
    cases = []
    cases.append(torch.zeros(64 * 70, dtype=torch.bfloat16))
    cases.append(torch.full((64 * 70,), 0.375, dtype=torch.bfloat16))
    g = torch.Generator().manual_seed(5)
    vals = torch.tensor([-1.0, -0.5, 0.0, 0.25, 0.5, 1.0])[torch.randint(0, 6, (64 * 300,), generator=g)]
    cases.append(vals.to(torch.bfloat16))
    big = torch.randn(64 * 200, generator=g).reshape(-1, 64) * torch.exp2(torch.randint(-10, 11, (200, 1), generator=g).float())
    cases.append(big.reshape(-1).to(torch.bfloat16))
    tiny = (torch.randn(64 * 64, generator=g) * 1e-7).to(torch.bfloat16)  # constants in binary16's subnormal range
    cases.append(tiny)
    for w in cases:
        for signed in (0, 1):
            st, o = oracle.lloyd_step_mae(inputs.bits(w), 64, cb, signed)
            assert st == oracle.OK
            assert_mae_close(binding.bof4_lloyd_step_mae(w.to(DEV), 64, cb, signed), o)


def test_mae_results_in_pinned_memory_and_repeatable():
    w = make_weights(64, 1024, seed=93).to(DEV)
    cb = mae_cb(64, 1)
    ref = binding.bof4_lloyd_step_mae(w, 64, cb, 1)
    rec, keep = binding.pinned_mae_stats()
    for _ in range(3):
        got = binding.bof4_lloyd_step_mae(w, 64, cb, 1, out=rec)
        assert np.array_equal(got["median"], ref["median"]) and np.array_equal(got["cnt"], ref["cnt"])
        assert got["sae"] == ref["sae"] and np.array_equal(got["den"], ref["den"])


def test_mae_step_argument_errors():
    w = make_weights(4, 1024, seed=94).to(DEV)
    cb = mae_cb(64, 1)
    small = torch.empty(1024, dtype=torch.uint8, device=DEV)
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_lloyd_step_mae(w, 64, cb, 1, ws=small)
    assert e.value.code == binding.BOF4_ERR_WORKSPACE
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_lloyd_step_mae(w, 48, cb, 1)
    assert e.value.code == binding.BOF4_ERR_ARG


def test_mae_step_refuses_weights_too_large_for_exact_sums():
    """The 64-bit integer weight sums hold sum |block constant| < 2^38 over all weights; 2^26 weights of 65280 exceed
    that and must be reported, not wrapped around."""
    w = torch.full((1 << 26,), 65280.0, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(binding.Bof4Error) as e:
        binding.bof4_lloyd_step_mae(w, 64, mae_cb(64, 1), 1)
    assert e.value.code == binding.BOF4_ERR_ARG
    # a hundredth of that passes
    w = torch.full((1 << 19,), 65280.0, dtype=torch.bfloat16, device=DEV)
    g = binding.bof4_lloyd_step_mae(w, 64, mae_cb(64, 1), 1)
    assert g["cnt"].sum() == w.numel() and g["den"].sum() == 65280.0 * w.numel()


@pytest.mark.parametrize("signed", [0, 1])
@pytest.mark.parametrize("opq", [0, 1])
def test_mae_step_skips_pinned_regions(signed, opq):
    """With the pinned levels skipped (no fourth pass for the region around zero) the other medians, every count
    and every mass are unchanged; the skipped medians come back as NaN.  (With OPQ this is the configuration in which
    the passes after the second read the list of candidates; without the mask and with OPQ they scan the weights.)"""
    w = make_weights(29, 1024, seed=610 + signed)
    cb = mae_cb(64, signed)
    pin = codebooks.PIN_BOF4S if signed else codebooks.PIN_BOF4
    T = oracle.opq_threshold(0.95, 64) if opq else 0.0
    st, o = oracle.lloyd_step_mae(inputs.bits(w), 64, cb, signed, opq_T=T)
    g = binding.bof4_lloyd_step_mae(w.to(DEV), 64, cb, signed, opq_T=T, skip_mask=pin)
    skipped = np.array([(pin >> l) & 1 for l in range(16)], dtype=bool)
    assert np.isnan(g["median"][skipped]).all()
    assert np.array_equal(g["median"][~skipped], o["median"][~skipped])
    assert np.array_equal(g["cnt"], o["cnt"]) and np.array_equal(g["den"], o["den"])
    assert abs(g["sae"] - o["sae"]) <= RTOL * o["sae"]
    new_g = binding.bof4_codebook_update_mae(g, pin, cb)
    assert np.array_equal(new_g, oracle.codebook_update_mae(o, pin, cb))


def _sampled_tiles(n_tiles):
    """Which wave tiles (4096 weights at block 64) the sampling pass of the MAE step looks at: one in 8 to 64, the most for
    which 2000 or more are left, by the multiplicative hash that bof4_mae.h documents."""
    one_in = 8
    while one_in < 64 and n_tiles // (2 * one_in) >= 2000:
        one_in *= 2
    t = np.arange(n_tiles, dtype=np.uint64)
    return (((t * np.uint64(0x9E3779B1)) & np.uint64(0xFFFFFFFF)) >> np.uint64(16)) & np.uint64(one_in - 1) == 0


@pytest.mark.parametrize("misled", [False, True])
def test_mae_one_pass_search_and_its_fallback(misled, capfd, monkeypatch):
    """From 2^26 weights up the step reads the weights once: a sampling pass over one tile in 8 or more places a window of
    first digits per region, the full pass writes the elements inside to the list.  On ordinary data the exact first
    digit falls inside the window and the list serves all later passes; if the sampled tiles are unlike the rest
    (here: cubed, which moves every region's median) the windows miss, the first pass follows and the second one writes the
    list.  Both ways return the oracle's medians bit for bit; the library's trace line says which way was taken."""
    n_tiles = 16384 + 37
    g = torch.Generator().manual_seed(4242)
    w = torch.randn(n_tiles * 4096, generator=g)
    if misled:
        pick = torch.from_numpy(np.repeat(_sampled_tiles(n_tiles), 4096))
        w[pick] = w[pick] ** 3
    w = w.to(torch.bfloat16)
    cb = mae_cb(64, 1)
    pin = codebooks.PIN_BOF4S
    st, o = oracle.lloyd_step_mae(inputs.bits(w), 64, cb, 1)
    assert st == oracle.OK
    monkeypatch.setenv("BOF4_MAE_TRACE", "1")
    capfd.readouterr()
    got = binding.bof4_lloyd_step_mae(w.to(DEV), 64, cb, 1, skip_mask=pin)
    trace = capfd.readouterr().err
    assert "sampling 1" in trace and f"list unusable {1 if misled else 0}" in trace, trace
    assert ("windows missed, written by the second pass" in trace) == misled, trace
    wanted = np.array([not ((pin >> l) & 1) for l in range(16)])
    assert np.array_equal(got["median"][wanted], o["median"][wanted]) and np.all(np.isnan(got["median"][~wanted]))
    assert np.array_equal(got["den"], o["den"]) and np.array_equal(got["cnt"], o["cnt"])
    assert abs(got["sae"] - o["sae"]) <= RTOL * o["sae"]
    monkeypatch.setenv("BOF4_MAE_NO_SAMPLING", "1")
    two = binding.bof4_lloyd_step_mae(w.to(DEV), 64, cb, 1, skip_mask=pin)
    assert np.array_equal(two["median"], got["median"], equal_nan=True) and two["sae"] == got["sae"]


@pytest.mark.parametrize("block,signed,weighted", [(128, 0, True), (32, 1, False), (256, 1, True)])
def test_mae_one_pass_search_with_opq(block, signed, weighted, capfd, monkeypatch):
    """The one-pass search on heavy-tailed weights with the outlier rule on, the pinned levels skipped (with the
    region around zero wanted the zeroed outliers would run through its search and the step keeps off the list), for
    the absolute and the signed normalisation, weighted and plain medians: medians, masses and counts as the
    oracle's, bit for bit, and the trace line says that the list served the later passes."""
    tile = 64 * min(block, 64)
    n = (16384 + 21) * tile + 3 * block  # just above the size from which the search samples, ragged tail
    w = make_weights(1, n, seed=977 + block)
    T = oracle.opq_threshold(0.95, block)
    cb = mae_cb(block, signed)
    pin = codebooks.PIN_BOF4S if signed else codebooks.PIN_BOF4
    st, o = oracle.lloyd_step_mae(inputs.bits(w), block, cb, signed, opq_T=T, weight_by_max=weighted)
    assert st == oracle.OK and o["n_outliers"] > 0
    monkeypatch.setenv("BOF4_MAE_TRACE", "1")
    capfd.readouterr()
    got = binding.bof4_lloyd_step_mae(w.to(DEV), block, cb, signed, opq_T=T, weight_by_max=weighted, skip_mask=pin)
    trace = capfd.readouterr().err
    assert "sampling 1" in trace and "list unusable 0" in trace, trace
    wanted = np.array([not ((pin >> l) & 1) for l in range(16)])
    assert np.array_equal(got["median"][wanted], o["median"][wanted]) and np.all(np.isnan(got["median"][~wanted]))
    assert np.array_equal(got["den"], o["den"]) and np.array_equal(got["cnt"], o["cnt"])
    assert got["n_used"] == o["n_used"] and got["n_outliers"] == o["n_outliers"]
    assert abs(got["sae"] - o["sae"]) <= RTOL * o["sae"]


@pytest.mark.parametrize("block,opq", [(32, 1), (64, 0), (64, 1), (128, 0), (128, 1), (256, 0), (256, 1)])
def test_mae_one_pass_search_without_the_bin_table(block, opq, capfd, monkeypatch):
    """The one-pass search with two levels closer than a bin of the search table (every weight is compared with all thresholds),
    all regions wanted that the list can serve: medians, masses and counts as the oracle's."""
    n = (16384 + 5) * 64 * min(block, 64) + 3 * block
    w = make_weights(1, n, seed=811 + block)
    cb = mae_cb(block, 1).copy()
    cb[10] = cb[9] + 0.004
    T = oracle.opq_threshold(0.95, block) if opq else 0.0
    skip = codebooks.PIN_BOF4S if opq else 0
    st, o = oracle.lloyd_step_mae(inputs.bits(w), block, cb, 1, opq_T=T)
    assert st == oracle.OK
    monkeypatch.setenv("BOF4_MAE_TRACE", "1")
    capfd.readouterr()
    got = binding.bof4_lloyd_step_mae(w.to(DEV), block, cb, 1, opq_T=T, skip_mask=skip)
    assert "sampling 1" in capfd.readouterr().err
    wanted = np.array([not ((skip >> l) & 1) for l in range(16)])
    assert np.array_equal(got["median"][wanted], o["median"][wanted], equal_nan=True)
    assert np.array_equal(got["den"], o["den"]) and np.array_equal(got["cnt"], o["cnt"])
    assert got["n_outliers"] == o["n_outliers"] and abs(got["sae"] - o["sae"]) <= RTOL * o["sae"]


def test_mae_one_pass_search_on_a_large_tensor_with_all_regions_wanted(capfd, monkeypatch):
    """2^29 weights and more, where the list has room for one weight in 32, no region skipped: ordinary weights are served by the
    windows' list, although the region around zero has octaves for digits and the outermost one holds 1 for every block.
    Medians, masses, counts and the error sum as those of the passes over all the weights."""
    n = (1 << 29) + 64 * 64 * 5 + 64
    g = torch.Generator(device=DEV)
    g.manual_seed(77)
    w = torch.empty(n, dtype=torch.bfloat16, device=DEV)
    for a in range(0, n, 1 << 27):
        w[a: a + (1 << 27)] = torch.randn(min(1 << 27, n - a), generator=g, device=DEV).to(torch.bfloat16)
    monkeypatch.setenv("BOF4_MAE_TRACE", "1")
    capfd.readouterr()
    got = binding.bof4_lloyd_step_mae(w, 64, mae_cb(64, 1), 1)
    trace = capfd.readouterr().err
    assert "sampling 1, list unusable 0" in trace, trace
    monkeypatch.setenv("BOF4_MAE_NO_SAMPLING", "1")
    two = binding.bof4_lloyd_step_mae(w, 64, mae_cb(64, 1), 1)
    for k in ("median", "den", "cnt"):
        assert np.array_equal(two[k], got[k], equal_nan=True), k
    assert two["sae"] == got["sae"] and got["cnt"].sum() == n


@pytest.mark.parametrize("case", ["zeros", "clumps", "close levels", "few values", "full stretch"])
@pytest.mark.parametrize("block", [32])
def test_mae_one_pass_search_edges(block, case, capfd, monkeypatch):
    """The one-pass search just above the size from which it samples, ragged tail: the region around zero wanted, its
    median among zeros of both signs (a window's edge may lie between them); tiles in which several hundred elements lie inside a
    window (they are listed in several goes: the trace says how full the fullest wave's stretch of 682 entries is, at most half
    on ordinary weights); a codebook with two levels closer than a bin of the search table; a tensor
    of few values, for which no list is tried; and one tile of equal weights inside a window, which fill more than a wave's stretch
    of the list (the digits stand, and the other passes do without that list).  Medians, masses and counts as the oracle's, and the error sum bit for bit
    that of the passes over all the weights."""
    tile = 64 * block
    n = (16384 + 3) * tile + 3 * block
    g = torch.Generator().manual_seed(300 + block)
    w = torch.randn(n, generator=g)
    cb, skip, usable = mae_cb(block, 1), codebooks.PIN_BOF4S, 1
    if case == "zeros":
        z = torch.randint(0, 64, (n,), generator=g)
        w[z == 0], w[z == 1] = 0.0, -0.0
        skip = 0xffff ^ (1 << 7)
    elif case == "clumps":  # the first tile of 64 waves: seven blocks of weights next to the median of region 11
        tiles = w[: 64 * tile].reshape(64, 64, block)
        tiles[:, 5:40:5, 0], tiles[:, 5:40:5, 1:] = 1.0, 0.337890625
    elif case == "full stretch":
        assert not _sampled_tiles(2)[1]
        blocks = w[tile: 2 * tile].reshape(64, block)
        blocks[:, 0], blocks[:, 1:], usable = 1.0, 0.337890625, 0
    elif case == "close levels":
        cb = cb.copy()
        cb[10] = cb[9] + 0.004
    else:
        w, usable = torch.randint(-6, 7, (n,), generator=g).float(), 0
    w = w.to(torch.bfloat16)
    st, o = oracle.lloyd_step_mae(inputs.bits(w), block, cb, 1)
    assert st == oracle.OK
    monkeypatch.setenv("BOF4_MAE_TRACE", "2")
    capfd.readouterr()
    wd = w.to(DEV)
    got = binding.bof4_lloyd_step_mae(wd, block, cb, 1, skip_mask=skip)
    trace = capfd.readouterr().err
    assert "sampling 1" in trace and f"list unusable {1 - usable}" in trace, trace
    assert ("declined" in trace) == (case == "few values") and ("a stretch ran full" in trace) == (case == "full stretch"), trace
    if case == "clumps":  # (ordinary waves hold 250 to 330 entries here, 64 of them seven times 31 more)
        assert 250 + 217 <= int(trace.split("fullest stretch ")[1].split(" of 682")[0]) <= 682, trace
    assert case != "zeros" or o["median"][7] == 0.0
    wanted = np.array([not ((skip >> l) & 1) for l in range(16)])
    assert np.array_equal(got["median"][wanted], o["median"][wanted], equal_nan=True)
    assert np.array_equal(got["den"], o["den"]) and np.array_equal(got["cnt"], o["cnt"])
    assert abs(got["sae"] - o["sae"]) <= RTOL * o["sae"]
    monkeypatch.setenv("BOF4_MAE_NO_SAMPLING", "1")
    two = binding.bof4_lloyd_step_mae(wd, block, cb, 1, skip_mask=skip)
    assert np.array_equal(two["median"], got["median"], equal_nan=True) and two["sae"] == got["sae"]


@pytest.mark.parametrize("block,signed", [(32, 1), (64, 0), (256, 1)])
def test_mae_step_on_blocks_whose_constant_binary16_stores_with_fewer_bits(block, signed):
    """A block maximum below binary16's normal range loses bits when stored (1.4375 x 2^-24 becomes 2^-24): the
    block's extreme weights normalise to -1.4375 and +1.4375, outside [-1, 1], and belong to the outermost regions
    with that value - also as medians, when such elements make up most of a region."""
    g = torch.Generator().manual_seed(57 + block)
    n_blocks = 3 * 64 * min(block, 64) // block + 5
    tiny = 1.4375 * 2.0 ** -24
    w = torch.randn(n_blocks, block, generator=g) * 0.05 * tiny  # tiny blocks: only the planted extremes lie far out
    w[:, 1], w[:, 5], w[:, 7] = tiny, -tiny, -tiny
    w[::4] = torch.randn((n_blocks + 3) // 4, block, generator=g) * 0.02  # and some ordinary blocks
    w = w.reshape(-1).to(torch.bfloat16)
    cb = mae_cb(block, signed)
    for weighted in (True, False):
        st, o = oracle.lloyd_step_mae(inputs.bits(w), block, cb, signed, weight_by_max=weighted)
        assert st == oracle.OK
        if not weighted:
            assert o["median"][0] == -1.4375  # most elements of the lowest region are the tiny blocks' minima
        assert_mae_close(binding.bof4_lloyd_step_mae(w.to(DEV), block, cb, signed, weight_by_max=weighted), o)
    st, e = oracle.quant_error(inputs.bits(w), block, cb, signed, 0.0)
    ge = binding.bof4_quant_error(w.to(DEV), block, cb, signed)
    assert ge["n"] == e["n"] and ge["max_abs"] == e["max_abs"] and abs(ge["sse"] - e["sse"]) <= RTOL * e["sse"]
    assert abs(ge["sae"] - e["sae"]) <= RTOL * e["sae"]
