"""GPU tests of the column sketch's P pass by whole rows (ranks up to 4, wide matrices, 1024 rows or more in the model): eight, four, two
and one row per workgroup, short last groups, narrow matrices beside wide ones, fewer columns than a trip's threads and several trips;
through the column sketch's own checks of the factor stages and of whole steps against the oracle."""
import pytest

from paper_2312_08538_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    ([(2100, 1024), (7, 147)], [204, 29], 4),              # eight rows, the last group of four
    ([(1003, 1100), (60, 33), (5, 4608)], [220, 7, 922], 3),     # four
    ([(1030, 1025)], [1], 1),                              # one bucket
    ([(1026, 2300)], [2300], 2),                           # as many buckets as columns
    ([(1025, 6400)], [6000], 4),                           # two rows: the table fills the LDS
    ([(1024, 12100)], [12000], 2),                         # one
]


@pytest.fixture(scope="module")
def env():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from oracle import conef_ref as R
    from paper_2312_08538_amd import binding as B
    import parity_util as U
    import test_gpu_sketch as S

    B.lib()
    return R, B, U, S, torch


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("gdt,fp16", [(wl.F32, False), (wl.BF16, True)])
def test_factor_stages(env, case, gdt, fp16, monkeypatch):
    import test_gpu_sketch_col as C

    monkeypatch.setattr(C, "LAYOUTS", [CASES[case]])
    C.test_factor_stages_match_the_oracle(env, 0, gdt, fp16)


@pytest.mark.parametrize("case", [0, 1])
def test_update_stage(env, case, monkeypatch):
    import test_gpu_sketch_col as C

    monkeypatch.setattr(C, "LAYOUTS", [CASES[case]])
    C.test_update_stage_and_estimate_are_bit_exact(env, 0, wl.F32, True, 0.9)
