"""Which kernels the planner sends a model's passes to, on both sides of its rules: what runs fast (the figures stand beside the
rules in plan.cpp), which no result shows."""
import json
import os
import subprocess

import pytest

from paper_2312_08538_amd import binding as B
from paper_2312_08538_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    """route(kind, layout, rank, bits, block, dtype): what tests/plan_probe.cpp prints for a model"""
    exe = tmp_path_factory.mktemp("probe") / "plan_probe"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(exe), os.path.join(HERE, "plan_probe.cpp"),
                    os.path.join(build.CSRC, "plan.cpp")], check=True)

    def ask(kind, layout, rank, bits=4, block=128, dtype=B.F32):
        args = [str(exe), kind, *(str(v) for v in (rank, bits, block, dtype)), *(str(v) for mat in layout for v in mat)]
        return json.loads(subprocess.run(args, check=True, capture_output=True, text=True).stdout)

    return ask


def test_octet_q_pass_shares_a_strip_where_that_pays(route):
    """A workgroup per strip: no matrix of more than 256 rows, and not in large models of short rows (400 of 256 x 512 took 160
    us a step so, 153 otherwise)."""
    def joined(layout, rank, **k):
        return route("step", layout, rank, **k)["q_joined"]

    assert joined([(256, 512)] * 64, 4) and joined([(256, 2048)] * 64, 4) and joined([(64, 1024)] * 500, 8)
    assert joined([(256, 512)] * 256, 4, bits=8, dtype=B.BF16)
    assert not joined([(256, 512)] * 400, 4) and not joined([(64, 1024)] * 500, 2) and not joined([(256, 512)] * 500, 8)
    assert not joined([(257, 512)], 4)


def test_err_items_are_cut_only_where_they_do_not_all_run_at_once(route):
    assert route("step", [(16384, 1024)], 4)["err_t_items"] == 2048                 # 64 rows of 128 columns each
    assert route("step", [(256, 512)] * 130, 4)["err_t_items"] > 130 * 4 * 4


def test_norm_pass_of_the_scaled_sign_goes_backwards_in_large_models_only(route):
    small, large = (route("step", [(n, 1024)], 4, bits=2, block=256, dtype=B.BF16) for n in (100000, 131072))
    assert (small["norm_back"], large["norm_back"]) == (0, 1)                       # 18 bits an element: 230 and 302 MB
    r = route("step", [(53000, 1024)], 4)
    assert (r["norm_back"], r["norm_back_two"]) == (0, 1)                           # 36 and 40 bits: 244 and 271 MB


def test_column_sketch_takes_whole_rows_where_that_pays(route):
    """Both sides of the figures beside the rule: 1500 x 1024 took 41.6 us a step by rows and 34.0 by strips, 1024 x 2500 40.4 and 42.3."""
    def rows(layout, rank=4):
        return route("columns", [(n, m, max(1, m // 5)) for n, m in layout], rank)["csc_rows_p"]

    assert rows([(1024, 2500)]) and rows([(2200, 1024)]) and rows([(8000, 4998)]) and rows([(2000, 9000)]) and rows([(6000, 2000)])
    for layout in ([(1500, 1024)], [(1135, 4998)], [(1135, 9000)], [(2000, 2500)], [(4500, 1024)], [(16000, 1500)], [(64, 16000)]):
        assert not rows(layout), layout
    gpt = lambda d: [(3000, d)] + [(d, 3 * d), (d, d), (d, 4 * d), (4 * d, d)] * 8
    assert not rows(gpt(512)) and not rows(gpt(768)) and rows(gpt(1024))
    assert not rows([(20000, 1024)] + [(4096, 1024)] * 4) and not rows([(1024, 2500)], 8)
    import test_gpu_planned_routes as gpu

    for (layout, buckets, rank), want in gpu.COLUMN_ROWS:
        assert route("columns", [(n, m, w) for (n, m), w in zip(layout, buckets)], rank)["csc_rows_p"] == want, layout


def test_step_in_one_launch(route):
    """... for every model of its GPU tests (a second column would be noise in that test's rank-one gradients: rank 1 there), and not
    just beyond the kernel's limits."""
    import test_gpu_planned_routes as gpu

    for layout, rank, bits, block in gpu.SMALL:
        for r in {rank, 1}:
            for dtype in (B.F32, B.BF16):
                assert route("step", layout, r, bits, block, dtype)["one_launch"], (layout, r, dtype)
    for layout, rank, bits, block in (([(1025, 16)], 4, 4, 128), ([(8, 2240)], 8, 4, 64), ([(40, 65)], 4, 4, 64), ([(40, 64)] * 300, 4, 4, 64),
                                      ([(64, 64)], 9, 4, 64), ([(64, 64)], 4, 4, 96)):
        assert not route("step", layout, rank, bits, block)["one_launch"], layout


def test_few_rows(route, monkeypatch):
    import test_gpu_planned_routes as gpu

    monkeypatch.setenv("CONEF_PACK", "0")
    for (rank, bits, block, dtype, layout), want in gpu.FEW_ROWS:
        r = route("step", layout, rank, bits, block, dtype)
        assert (r["q_joined"], r["orth_rows"], r["err_rows"], r["p_chunks"]) == want, layout


def test_err_pass_with_q_in_lds(route):
    import test_gpu_planned_routes as gpu

    for i, (rank, bits, block, dtype, layout) in enumerate(gpu.WALK):
        assert (route("step", layout, rank, bits, block, dtype)["walk"] > 0) == (i not in gpu.ON_STRIPS), layout


PLANTED = [
    # (kind, layout, rank, bits, block, dtype): models with the tables, and models just beyond the limits of the kernels behind them
    ("step", [(256, 128), (40, 64)], 2, 8, 64, B.F32),
    ("step", [(1025, 33), (64, 65)], 3, 4, 64, B.F32),
    ("step", [(257, 1100)], 8, 4, 256, B.F32),
    ("step", [(300, 300)], 16, 4, 128, B.F32),
    ("step", [(200, 170)], 4, 4, 128, B.F32),
    ("rows", [(500, 256, 100), (77, 64, 13), (40, 33, 8)], 4, 8, 4, B.F32),
    ("rows", [(500, 256, 100), (70, 40, 9)], 32, 8, 4, B.BF16),
    ("columns", [(64, 147, 29)], 4, 8, 4, B.F32),
]


@pytest.mark.parametrize("case", range(len(PLANTED)))
def test_check_plan_sees_mistakes_in_what_kernels_index_and_stage_by(route, case):
    kind, layout, rank, bits, block, dtype = PLANTED[case]
    r = route(kind, layout, rank, bits=bits, block=block, dtype=dtype)
    assert r["ok"] and r["missed"] == []


def test_row_order_is_made_for_the_matrices_that_read_it(route):
    """The row sketch's octet kernels walk a matrix's rows bucket by bucket; the linear form and the kernels for any shape do not."""
    assert route("rows", [(500, 256, 100), (70, 40, 9), (64, 33, 9)], 4)["row_order"] == 570
    assert route("rows", [(500, 33, 100), (70, 41, 9)], 4)["row_order"] == 0
    assert route("rows", [(500, 256, 100), (70, 128, 9)], 32, dtype=B.BF16)["row_order"] == 0
