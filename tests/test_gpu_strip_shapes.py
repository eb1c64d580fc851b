"""GPU tests of the strip kernels on matrices of few columns (the err pass walks them in groups of rows) and of few rows (the
Q+ pass gives a wave all of them), each on both sides of the rule that takes it there, against the oracle through the
checks of the plain step, of two error vectors and of the count sketch."""
import numpy as np
import pytest

from paper_2312_08538_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from oracle import conef_ref as R
    from paper_2312_08538_amd import binding as B
    import parity_util as U

    B.lib()
    return R, B, U, torch


# (with as many columns as the rank nothing but rounding is left of a residual: only where it agrees to the last bit)
# every group height 64 / columns has matrices that end inside a group, at its end and one row on, and runs of several groups
def _narrow(rank, columns, beside=()):
    L = []
    for m in columns:
        k = 64 // m
        L += [(max(rank + (rank > 1), r), m) for r in (1, k, k + 1, 1024 // m + 1, 3 * 1024 // m + k - 1)]
    return L + list(beside)


NARROW = [
    (1, 4, 128, wl.F32, _narrow(1, [1, 2, 3, 7])),
    (2, 2, 16, wl.BF16, _narrow(2, [3, 5, 15, 16])),
    (3, 8, 64, wl.F32, _narrow(3, [4, 9, 31, 32, 33])),                       # 33 columns: not in groups, nor 31 and 32 beside them
    (4, 4, 512, wl.F32, _narrow(4, [5, 8, 15, 16, 27], [(64, 147), (40, 256)])),
    (8, 4, 8, wl.BF16, _narrow(8, [9, 13, 17, 27])),
    (16, 4, 256, wl.F32, _narrow(16, [17, 21, 32])),
    (9, 8, 16, wl.F32, _narrow(9, [10, 11, 14], [(50, 1100)])),
    (32, 2, 64, wl.F32, _narrow(32, [32])),
]


@pytest.mark.parametrize("rank,bits,block,dtype,layout", NARROW)
def test_matrices_of_few_columns(env, rank, bits, block, dtype, layout):
    import test_gpu_parity as G

    R, B, U, torch = env
    w = wl.Workload("narrow", 21, tuple(layout), rank, bits, block, dtype, "normal", 1.0, 0x7A44)
    assert G._run_model((R, B, U), w, layout, 3, f"narrow-r{rank}-b{bits}-B{block}") == 0


@pytest.mark.parametrize("case", range(len(NARROW)))
def test_matrices_of_few_columns_with_two_vectors(env, case, monkeypatch):
    import test_gpu_iconef_lowrank as I

    rank, bits, block, dtype, layout = NARROW[case]
    monkeypatch.setattr(I, "CASES", [(layout, rank, bits, block)])
    I.test_iconef_with_the_rank_r_compressor(env, 0, dtype)


FLAT = [
    (1, 4, 128, wl.F32, [(1, 1), (1, 63), (1, 257), (1, 3000), (2, 100), (9, 40)]),
    (2, 2, 64, wl.BF16, [(2, 64), (2, 255), (3, 1500), (7, 513)]),
    (3, 8, 16, wl.F32, [(3, 130), (4, 256), (8, 259), (9, 259)]),
    (8, 4, 256, wl.F32, [(8, 8), (8, 1025), (9, 1025), (64, 147)]),
]


@pytest.mark.parametrize("rank,bits,block,dtype,layout", FLAT)
def test_matrices_of_few_rows(env, rank, bits, block, dtype, layout):
    import test_gpu_parity as G

    R, B, U, torch = env
    w = wl.Workload("flat", 22, tuple(layout), rank, bits, block, dtype, "normal", 1.0, 0xF1A7)
    assert G._run_model((R, B, U), w, layout, 3, f"flat-r{rank}-b{bits}-B{block}") == 0


@pytest.mark.parametrize("case", range(len(FLAT)))
def test_matrices_of_few_rows_with_two_vectors(env, case, monkeypatch):
    import test_gpu_iconef_lowrank as I

    rank, bits, block, dtype, layout = FLAT[case]
    monkeypatch.setattr(I, "CASES", [(layout, rank, bits, block)])
    I.test_iconef_with_the_rank_r_compressor(env, 0, dtype)


@pytest.mark.parametrize("case", range(len(FLAT)))
@pytest.mark.parametrize("columns", [False, True])
def test_matrices_of_few_rows_with_the_sketch(env, case, columns, monkeypatch):
    import test_gpu_sketch as S
    import test_gpu_sketch_col as SC

    R, B, U, torch = env
    rank, _, _, dtype, layout = FLAT[case]
    buckets = [max(1, (m if columns else n) // 3) for n, m in layout]
    mod = SC if columns else S
    monkeypatch.setattr(mod, "LAYOUTS", [(layout, buckets, rank)])
    mod.test_factor_stages_match_the_oracle((R, B, U, S, torch) if columns else (R, B, U, torch), 0, dtype, True)
