"""GPU tests of the strip family's err pass with Q+ in LDS, at the edges of what it takes: eight columns (every octet in one or two
rows), rows that start at every place of an octet, short last octets and blocks, several runs per wave, the widest matrices whose
Q+ fits and those just beyond, ranks that are padded, and the launch that it shares with the octet family.  Against the oracle
through the checks of the plain step and of two error vectors: codes bit for bit (fp64 sums of the factors, the residual's fp32
chain in the oracle's order)."""
import pytest

from paper_2312_08538_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # (rank, bits, block, dtype, layout)
    (1, 4, 128, wl.F32, [(1, 8), (3, 9), (100, 15), (65, 31), (5000, 8)]),
    (2, 2, 16, wl.BF16, [(2, 8), (33, 10), (129, 14), (511, 63), (40, 5400)]),       # the last: all that fits at rank 2
    (3, 8, 64, wl.F32, [(3, 11), (77, 65), (40, 129), (31, 650)]),                    # padded to four
    (4, 4, 128, wl.F32, [(64, 147), (300, 577), (37, 53), (24, 2722)]),               # 48 KB
    (4, 4, 128, wl.F32, [(64, 147), (24, 2760)]),                                     # more than that: both on strips
    (5, 2, 512, wl.F32, [(5, 8), (50, 333), (200, 71)]),                              # padded to eight; blocks of several rows
    (8, 8, 8, wl.BF16, [(8, 8), (9, 1441), (150, 97), (1000, 12)]),
    (4, 4, 128, wl.F32, [(64, 147), (128, 576), (200, 256)]),                         # beside the octet family
    (8, 2, 256, wl.F32, [(40, 147), (300, 1000), (512, 512)]),
    (4, 4, 64, wl.F32, [(3000, 1501)]),                                               # several runs per wave, rows of three of them
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
def test_err_pass_with_q_in_lds(env, case):
    import test_gpu_parity as G

    R, B, U, torch = env
    rank, bits, block, dtype, layout = CASES[case]
    w = wl.Workload("walk", 22, tuple(layout), rank, bits, block, dtype, "normal", 1.0, 0x7A45)
    assert G._run_model((R, B, U), w, layout, 2 if case == 9 else 3, f"walk-{case}") == 0


@pytest.mark.parametrize("case", range(len(CASES) - 1))
def test_err_pass_with_q_in_lds_and_two_vectors(env, case, monkeypatch):
    import test_gpu_iconef_lowrank as I

    rank, bits, block, dtype, layout = CASES[case]
    monkeypatch.setattr(I, "CASES", [(layout, rank, bits, block)])
    I.test_iconef_with_the_rank_r_compressor(env, 0, dtype)
