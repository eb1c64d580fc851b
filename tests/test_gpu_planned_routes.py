"""GPU tests of kernels that a rule of the planner picks, on models that tests/test_plan_routes.py holds the planner to: the step in
one launch, the err pass with Q+ in LDS, few rows, and the column sketch's P pass by whole rows, each at the edges of what it takes.
The checks are those of the kernel's own test file, whose models may be planned for other kernels."""
import pytest

from paper_2312_08538_amd import workloads as wl
from test_gpu_few_rows import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

SMALL = [
    # (layout, rank, bits, block): the step in one launch, at every dtype
    ([(256, 128)], 2, 8, 64),                                    # most elements
    ([(1024, 16)], 4, 4, 128),                                   # most rows: P in several trips, 16 Gram tiles; blocks across rows
    ([(8, 1024)], 8, 4, 64),                                     # few rows, as many tiles of columns as waves
    ([(4, 1288), (12, 1032)], 2, 8, 64),                         # more of them
    ([(1, 8), (8, 8), (16, 16)], 1, 2, 16),
    ([(5, 8), (17, 24), (63, 40), (65, 8)], 5, 2, 32),
    ([(100, 136), (33, 264), (560, 40), (129, 72)], 3, 8, 512),  # more scale block than row, short last blocks
    ([(31, 520), (240, 104), (7, 56)], 7, 4, 8),
    ([(128, 64)] * 300, 4, 4, 64),                               # more workgroups than CUs
]
SMALL_NEW = [1, 2, 3, 6, 7, 8]          # the others are cases of test_gpu_small_step.py

WALK = [
    # (rank, bits, block, dtype, layout): the err pass with Q+ in LDS
    (2, 2, 16, wl.BF16, [(2, 8), (33, 10), (129, 14), (511, 63), (40, 4906)]),       # the last: all that fits at rank 2
    (8, 8, 8, wl.BF16, [(8, 8), (9, 1437), (150, 97), (1000, 12)]),                  # ... and at rank 8
    (2, 2, 16, wl.BF16, [(33, 10), (40, 4907)]),                                     # a column too many, at rank 2 and 8: on strips
    (8, 8, 8, wl.BF16, [(9, 1438), (150, 97)]),
]
ON_STRIPS = [2, 3]

FEW_ROWS = [
    # (rank, bits, block, dtype, layout), (shared strips of Q+, orthonormalisation in one launch, rows of the err pass's first item,
    # column chunks of P)
    ((4, 4, 128, wl.F32, [(240, 4000), (40, 2048)]), (1, 1, 16, 16)),        # column chunks of P added in the one launch
    ((8, 2, 256, wl.BF16, [(3300, 2048), (33, 256)]), (0, 0, 32, 4)),        # err pass: items of 32 rows
]

COLUMN_ROWS = [
    # (layout, buckets, rank), rows per workgroup of the first matrix
    (([(959, 1100), (60, 33), (5, 4608)], [220, 7, 922], 3), 4),
    (([(2049, 1025)], [1], 1), 8),                                # one bucket
    (([(2050, 2300)], [2300], 2), 8),                             # as many buckets as columns
    (([(1019, 6400), (5, 64)], [6000, 13], 4), 2),                # the table fills the LDS
]


@pytest.mark.parametrize("case", SMALL_NEW)
@pytest.mark.parametrize("gdt", [wl.F32, wl.BF16])
@pytest.mark.parametrize("beta,kind", [(0.0, "normal"), (0.5, "normal"), (0.0, "zero"), (0.0, "not finite"), (0.0, "low rank")])
def test_step_in_one_launch(case, gdt, beta, kind, monkeypatch):
    import test_gpu_small_step as S

    monkeypatch.setattr(S, "CASES", SMALL)
    S.test_small_step_has_the_bits_of_the_stages(case, gdt, beta, kind)


@pytest.mark.parametrize("case", range(len(WALK)))
def test_err_pass_with_q_in_lds(env, case, monkeypatch):  # noqa: F811
    import test_gpu_walk as W

    monkeypatch.setattr(W, "CASES", WALK)
    W.test_err_pass_with_q_in_lds(env, case)
    W.test_err_pass_with_q_in_lds_and_two_vectors(env, case, monkeypatch)


@pytest.mark.parametrize("case", range(len(FEW_ROWS)))
def test_few_rows(env, case, monkeypatch):  # noqa: F811
    import test_gpu_few_rows as F

    monkeypatch.setattr(F, "CASES", [c for c, _ in FEW_ROWS])
    F.test_few_rows(env, case, monkeypatch)
    if case == 0:
        F.test_few_rows_with_two_vectors(env, case, monkeypatch)


@pytest.mark.parametrize("case", range(len(COLUMN_ROWS)))
@pytest.mark.parametrize("gdt,fp16", [(wl.F32, False), (wl.BF16, True)])
def test_column_sketch_by_rows(env, case, gdt, fp16, monkeypatch):  # noqa: F811
    import test_gpu_sketch as S
    import test_gpu_sketch_col as C

    R, B, U, torch = env
    monkeypatch.setattr(C, "LAYOUTS", [COLUMN_ROWS[case][0]])
    C.test_factor_stages_match_the_oracle((R, B, U, S, torch), 0, gdt, fp16)
    if case == 0:
        C.test_update_stage_and_estimate_are_bit_exact((R, B, U, S, torch), 0, wl.F32, True, 0.9)
