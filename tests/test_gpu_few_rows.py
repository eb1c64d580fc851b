"""GPU tests of what models of few rows take: the octet Q+ pass whose workgroups write Q+ themselves (no matrix of more than 256
rows), the orthonormalisation in one launch (1024 rows, 256 above rank 4), the err pass in items of 16 and 32 rows.  At the edges
of waves, tiles and rules, on both sides of each, against the oracle through the checks of the plain step and of two error
vectors."""
import pytest

from paper_2312_08538_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # (rank, bits, block, dtype, layout)
    (4, 4, 128, wl.F32, [(n, 256) for n in (4, 31, 32, 33, 64, 97, 128, 129, 255, 256)]),
    (8, 8, 64, wl.BF16, [(8, 64), (65, 192), (250, 320), (256, 64)]),
    (2, 2, 512, wl.F32, [(2, 512), (130, 1024), (256, 2048)]),
    (4, 4, 128, wl.F32, [(257, 256), (8, 128), (64, 147)]),                  # one row too many: partial sums
    (4, 4, 128, wl.F32, [(256, 384), (200, 147), (31, 576)]),                # beside the strip family
    (3, 4, 64, wl.F32, [(1024, 33), (1000, 130), (64, 65), (63, 64), (3, 20)]),      # one launch, up to all of its threads
    (3, 4, 64, wl.F32, [(1025, 33), (64, 65)]),                              # two launches
    (4, 4, 128, wl.F32, [(300, 5000), (40, 2048)]),                          # column chunks of P added in it
    (8, 4, 256, wl.F32, [(256, 1100), (65, 512)]),
    (8, 4, 256, wl.F32, [(257, 1100), (65, 512)]),
    (8, 4, 128, wl.F32, [(300, 640), (1500, 384)]),                          # err pass: items of 16 rows
    (8, 2, 256, wl.BF16, [(2100, 2048), (33, 256)]),                         # ... of 32
]


@pytest.fixture(scope="module")
def env():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from oracle import conef_ref as R
    from paper_2312_08538_amd import binding as B
    import parity_util as U

    B.lib()
    return R, B, U, torch


@pytest.mark.parametrize("case", range(len(CASES)))
def test_few_rows(env, case, monkeypatch):
    import test_gpu_parity as G

    R, B, U, torch = env
    monkeypatch.setenv("CONEF_PACK", "0")
    rank, bits, block, dtype, layout = CASES[case]
    w = wl.Workload("few-rows", 23, tuple(layout), rank, bits, block, dtype, "normal", 1.0, 0x7A46)
    assert G._run_model((R, B, U), w, layout, 3, f"few-rows-{case}") == 0


@pytest.mark.parametrize("case", [0, 1, 2, 4, 7, 10])
def test_few_rows_with_two_vectors(env, case, monkeypatch):
    import test_gpu_iconef_lowrank as I

    monkeypatch.setenv("CONEF_PACK", "0")
    rank, bits, block, dtype, layout = CASES[case]
    monkeypatch.setattr(I, "CASES", [(layout, rank, bits, block)])
    I.test_iconef_with_the_rank_r_compressor(env, 0, dtype)
