"""The step of models of small matrices in one launch against the stages' own launches (which timed stages take), that the other tests
hold to the oracle: the same bits in P, Q, codes and scales, and nothing written beside them.  Sums are fp64 in both; only the
order of P's and Q+'s differs, which a rounding to fp32 shows for about one entry in 10^8."""
import numpy as np
import pytest

from paper_2312_08538_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # (layout, rank, bits, block)
    ([(256, 128)], 2, 8, 64),                                    # all of a CU's LDS
    ([(1024, 24)], 4, 4, 128),                                   # most rows; blocks across rows
    ([(8, 2240)], 8, 4, 64),                                     # few rows, most tiles of columns
    ([(1, 8), (8, 8), (16, 16)], 1, 2, 16),                      # one octet; N no multiple of a code word
    ([(5, 8), (17, 24), (63, 40), (65, 8)], 5, 2, 32),           # remainders of 16 rows, 64 rows, 16 columns; rank 5
    ([(100, 136), (33, 264), (600, 40), (129, 72)], 3, 8, 512),  # more scale block than row, short last blocks
    ([(31, 1000), (240, 104), (7, 56)], 7, 4, 8),
    ([(40, 64)] * 300, 4, 4, 64),                                # more workgroups than CUs
]


def _run(layout, rank, bits, block, gdt, beta, kind, stages):
    import torch

    from paper_2312_08538_amd import binding as B

    model = B.Model(layout, rank, bits, block, gdt, 991)
    B.conef_set_timing(model.ctx, stages)
    if beta:
        B.conef_set_beta(model.ctx, beta)
    buf = model.alloc()
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    buf["Q"].normal_(generator=gen)
    for k in ("P", "codes", "scales"):
        buf[k].fill_(77)                    # (the padding between matrices keeps it)
    for (n, m), o in zip(layout, model.offsets):
        buf["codes"][o["word_off"]:o["word_off"] + -(-n * m * bits // 32)] = 0
        buf["scales"][o["scale_off"]:o["scale_off"] + -(-n * m // block)] = 0
    out = []
    for t in range(3):
        g = torch.randn(buf["grads"].shape, device="cuda:0", generator=gen)
        if kind == "zero":
            g.zero_()                       # every pivot is dead
        elif kind == "low rank":
            for (n, m), o in zip(layout, model.offsets):
                u = torch.randn(n, 1, device="cuda:0", generator=gen)
                v = torch.randn(1, m, device="cuda:0", generator=gen)
                g[o["grad_off"]:o["grad_off"] + n * m] = (u * v).view(-1)
        elif kind == "not finite":
            o = model.offsets[-1]
            g[o["grad_off"] + 3] = float("inf")
        buf["grads"].copy_(g)
        model.step(buf, t)
        torch.cuda.synchronize()
        out.append({k: buf[k].cpu().numpy().copy() for k in ("P", "Q", "codes", "scales")})
    model.close()
    return out


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("gdt", [wl.F32, wl.BF16])
@pytest.mark.parametrize("beta,kind", [(0.0, "normal"), (0.5, "normal"), (0.0, "zero"), (0.0, "not finite"), (0.0, "low rank")])
def test_small_step_has_the_bits_of_the_stages(case, gdt, beta, kind):
    layout, rank, bits, block = CASES[case]
    if kind == "low rank" and rank > 1:
        rank = 1                            # (a second column would be rounding noise, normalised)
    got = _run(layout, rank, bits, block, gdt, beta, kind, stages=False)
    want = _run(layout, rank, bits, block, gdt, beta, kind, stages=True)
    for t, (g, w) in enumerate(zip(got, want)):
        for k in g:
            same = np.array_equal(g[k].view(np.uint32), w[k].view(np.uint32))
            if not same and kind == "not finite":       # the payload of a NaN is nobody's business
                same = np.array_equal(g[k], w[k], equal_nan=g[k].dtype == np.float32)
            assert same, (t, k, int((g[k].view(np.uint32) != w[k].view(np.uint32)).sum()))
