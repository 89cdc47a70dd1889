"""The host's rules of bof4_gemm (which kernel takes a product, where its sums are cut, the workspace that follows), on the CPU:
bof4_gemm_plan.h compiled with the host's compiler."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2505_06653_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_06653_amd", "csrc")
NARROW, WIDE, DECODED = 0, 1, 2
ANY_SIZE = (1 << 64) - 1


class Plan(ctypes.Structure):
    _fields_ = [(k, ctypes.c_uint32) for k in ("way", "wide_split", "decoded_split", "decoded_slab_tiles", "kernel_split",
                                               "carry", "flush", "decoded_carry", "decoded_flush", "x_in_place")] + [("need", ctypes.c_uint64)]


@pytest.fixture(scope="session")
def rules(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "gemm_plan.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                    os.path.join(HERE, "csrc", "gemm_plan.cpp")], check=True)
    lib = ctypes.CDLL(so)
    lib.plan.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int, ctypes.c_uint64, ctypes.POINTER(Plan)]
    lib.plan.restype = None
    lib.workspace_bytes.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32]
    lib.workspace_bytes.restype = ctypes.c_uint64

    def plan(rows, cols, n_tokens, listed, ws_bytes=ANY_SIZE):
        p = Plan()
        lib.plan(rows, cols, n_tokens, int(listed), ws_bytes, ctypes.byref(p))
        return p

    plan.workspace_bytes = lib.workspace_bytes
    return plan


def shapes(count, seed):
    """Seeded shapes over the range of products that can be decoded first, every second one of 512 to 2300 columns."""
    rng = np.random.default_rng(seed)
    for i in range(count):
        cols = int(np.exp(rng.uniform(np.log(512), np.log(2300 if i % 2 else 32768)))) // 32 * 32
        yield int(np.exp(rng.uniform(np.log(300), np.log(60000)))), cols, int(np.exp(rng.uniform(np.log(100), np.log(3000))))


NAMED = [(45826, 1152, 581), (1974, 3968, 1559), (29401, 544, 513), (9496, 576, 1214), (31710, 1216, 581), (13551, 2240, 566)]


def test_gemm_workspace_bytes_is_enough_for_the_kernel_that_is_chosen_with_and_without_a_list(rules):
    """Also the size for more tokens: it takes no call another way than the call's own size (the order of additions would be
    another).  The library tells the same sizes."""
    n_decoded = 0
    for rows, cols, n in NAMED + list(shapes(6000, 1)):
        own = rules.workspace_bytes(rows, cols, n)
        for listed in (False, True):
            best = rules(rows, cols, n, listed)
            assert rules(rows, cols, n, listed, own).way == best.way, (rows, cols, n, listed)
            assert rules(rows, cols, n, listed, best.need - 1).way < best.way or best.way == NARROW
            n_decoded += best.way == DECODED
    assert n_decoded > 1000
    for rows, cols, n in NAMED + list(shapes(100, 2)):
        assert binding.bof4_gemm_workspace_bytes(rows, cols, n) == rules.workspace_bytes(rows, cols, n)
        sizes = [rules.workspace_bytes(rows, cols, m) for m in range(1, n, 13)] + [rules.workspace_bytes(rows, cols, n)]
        assert sizes == sorted(sizes)


def test_gemm_decoded_first_adds_uncarried_sums_only_as_the_wide_tile_would(rules):
    """Where the columns are split as the wide tile splits them the chains are that tile's (the results are the same bits); in all
    other products the sums are carried, over chains that are no longer than those of the kernel that would take the product."""
    alike = other = 0
    for rows, cols, n in [(12288, 4096, 700), (16343, 1376, 588), (5970, 23808, 1065)] + list(shapes(6000, 3)):
        for listed in (False, True):
            p = rules(rows, cols, n, listed)
            if p.way != DECODED:
                continue
            if p.decoded_split == p.wide_split:
                alike += 1
                assert (p.decoded_carry, p.decoded_flush) == (p.carry, p.flush)
                continue
            other += 1
            per_wave = -(-(-(-(-(-cols // 64)) // p.kernel_split)) // 8)  # chunks that a wave of gemm_kernel takes, at most
            assert p.decoded_carry == 1 and 1 <= p.decoded_flush <= p.flush
            assert p.wide_split > 0 or listed or p.decoded_flush <= per_wave
            assert p.wide_split == 0 or p.decoded_split <= p.wide_split or p.decoded_flush < max(p.flush, 2)
    assert alike > 1000 and other > 100, (alike, other)


@pytest.mark.parametrize("rows,cols,n_tokens,listed,way", [
    (28672, 8192, 1200, False, WIDE), (40770, 2112, 757, False, WIDE), (27007, 1792, 628, False, WIDE),
    (57344, 8192, 1200, False, DECODED), (16234, 9888, 2383, False, DECODED), (28672, 8192, 1200, True, DECODED),
    (12288, 4096, 420, True, DECODED), (4096, 4096, 2000, False, DECODED)])
def test_gemm_takes_the_kernel_that_was_measured_faster(rules, rows, cols, n_tokens, listed, way):
    """us, the other kernel / decoded first: 743 / 784, 196 / 208, 124 / 131; 1466 / 1349, 1003 / 933, 860 / 816, 102 / 88,
    97 / 88."""
    assert rules(rows, cols, n_tokens, listed).way == way


@pytest.mark.parametrize("rows,cols,n_tokens,listed,in_place", [
    (4096, 4096, 32, True, 1), (4160, 4032, 32, False, 0), (4160, 4032, 16, True, 1), (10000, 1664, 32, True, 0), (10000, 1024, 32, True, 1),
    (3000, 5568, 32, False, 0), (12000, 1376, 32, False, 0), (12000, 1376, 16, False, 1), (6144, 2688, 32, False, 1),
    (8192, 8192, 8, False, 0), (8192, 11008, 1, False, 0), (8192, 4096, 8, False, 1), (9000, 8192, 8, False, 1), (9000, 8192, 9, False, 0),
    (9000, 8192, 8, True, 0), (8192, 16384, 8, False, 1), (28672, 8192, 1, False, 1), (4096, 11008, 8, False, 0)])
def test_gemm_reads_x_in_place_where_that_was_measured_faster(rules, rows, cols, n_tokens, listed, in_place):
    assert rules(rows, cols, n_tokens, listed).x_in_place == in_place


def test_gemm_reads_x_in_place_with_a_list_only_where_a_wave_takes_one_tile_of_rows(rules):
    """(There is no kernel for the other.)  A wave takes two from 2^27 weights up at these token counts."""
    rng = np.random.default_rng(4)
    for _ in range(20000):
        rows, cols = int(np.exp(rng.uniform(0, 13))), int(rng.integers(1, 1025)) * 32
        p = rules(rows, cols, int(rng.integers(1, 33)), True)
        assert not p.x_in_place or rows * cols < 1 << 27
