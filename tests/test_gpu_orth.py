"""The orthonormalisation at the ends of its launches' row ranges: one trip of a workgroup, one partial Gram matrix, one
workgroup of the last launch, and the very tall matrix; every padded rank; and a full step, whose first launch adds the column
chunks of P, against the staged calls."""
import numpy as np
import pytest

from paper_2312_08538_amd import workloads as wl
from test_gpu_parity import env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

ROWS = [16, 17, 63, 64, 65, 255, 256, 257, 511, 513, 1025, 8192, 8193, 20000]


def _panels(rows, rank, dead):
    """Random panels of moderate condition; dead: the second column of every other one is a multiple of the first."""
    out = []
    for i, n in enumerate(rows):
        P = np.random.default_rng([n, rank]).standard_normal((n, rank)).astype(np.float32)
        P *= np.float32(10.0) ** (np.arange(rank) % 4 - 2).astype(np.float32)
        if dead and rank > 1 and i % 2:
            P[:, 1] = 2.0 * P[:, 0]
        out.append(P)
    return out


@pytest.mark.parametrize("dead", [False, True])
@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 7, 8, 9, 16, 31, 32])
def test_row_ranges(env, rank, dead):
    """P^ = P R^-1 against QR in float64 with the signs of a positive diagonal: entries to 2e-7 of 1 (one fp32 rounding of an
    entry below 1 is 6e-8; conditions here are at most 1e5 and everything before the rounding is fp64).  A dependent column is
    zero."""
    import torch

    B = env[1]
    rows = [n for n in ROWS if n >= 2 * rank] + ([140000] if rank in (4, 8) else [])
    panels = _panels(rows, rank, dead)
    model = B.Model([(n, 64) for n in rows], rank, 4, 64, wl.F32, 5)
    buf = model.alloc()
    for P, o in zip(panels, model.offsets):
        buf["P"][o["p_off"]:o["p_off"] + P.size] = torch.from_numpy(P.ravel()).cuda()
    B.conef_orthonormalise(model.ctx, buf["P"], buf["ws"], model.stream_handle())
    torch.cuda.synchronize()
    for i, (n, P, o) in enumerate(zip(rows, panels, model.offsets)):
        got = buf["P"][o["p_off"]:o["p_off"] + P.size].cpu().numpy().reshape(n, rank).astype(np.float64)
        cols = [c for c in range(rank) if not (dead and rank > 1 and i % 2 and c == 1)]
        q, r = np.linalg.qr(P[:, cols].astype(np.float64))
        q *= np.sign(np.diag(r))
        assert np.abs(got[:, cols] - q).max() <= 2e-7, (n, rank)
        for c in set(range(rank)) - set(cols):
            assert not got[:, c].any(), (n, rank, c)
    model.close()


@pytest.mark.parametrize("rank", [1, 3, 4, 5, 8])
def test_full_step_adds_the_chunks(env, rank):
    """A step whose P comes in column chunks (strip and octet kernels) and in one piece: the bits of the stage calls."""
    import torch

    B = env[1]
    layout = [(300, 1536), (65, 4100), (640, 512), (1000, 2048), (64, 64), (17, 700)]
    model = B.Model(layout, rank, 4, 64, wl.F32, 5)
    one, two = model.alloc(), model.alloc()
    torch.manual_seed(3)
    one["grads"].normal_()
    one["Q"].normal_()
    for k in ("grads", "Q"):
        two[k].copy_(one[k])
    st = model.stream_handle()
    for t in range(2):
        model.step(one, t)
        a = two
        B.conef_step_p(model.ctx, a["grads"], a["codes"], a["scales"], a["Q"], a["P"], a["ws"], st)
        B.conef_orthonormalise(model.ctx, a["P"], a["ws"], st)
        B.conef_step_q(model.ctx, a["grads"], a["codes"], a["scales"], a["P"], a["Q"], a["ws"], st)
        B.conef_step_err(model.ctx, a["grads"], a["codes"], a["scales"], a["P"], a["Q"], a["ws"], t, st)
    torch.cuda.synchronize()
    for k in ("P", "Q", "codes", "scales"):
        assert torch.equal(one[k], two[k]), k
    model.close()


@pytest.mark.parametrize("rank,layout", [(rank, [(70, cols), (130, 512)]) for rank, step in ((3, 257), (4, 512), (6, 257), (8, 512))
                                         for cols in (8 * step - 1, 8 * step, 9 * step, 16 * step, 17 * step)])
def test_chunks_on_either_side_of_the_rule(env, rank, layout):
    """Column chunks of P up to and beyond what the orthonormalisation adds up itself (8 and 16 of them): the bits of the stage
    calls."""
    import torch

    B = env[1]
    model = B.Model(layout, rank, 4, 64, wl.F32, 5)
    one, two = model.alloc(), model.alloc()
    torch.manual_seed(4)
    one["grads"].normal_()
    one["Q"].normal_()
    for k in ("grads", "Q"):
        two[k].copy_(one[k])
    st = model.stream_handle()
    model.step(one, 0)
    B.conef_step_p(model.ctx, two["grads"], two["codes"], two["scales"], two["Q"], two["P"], two["ws"], st)
    B.conef_orthonormalise(model.ctx, two["P"], two["ws"], st)
    torch.cuda.synchronize()
    assert torch.equal(one["P"], two["P"])
    model.close()


def test_coarse_gram_tiles(env):
    """A model of so many matrices that its partial Gram matrices cover 256 rows and not 64 (they would exceed the static
    workspace), against QR in float64 as above: tiles of one, two and a part of one."""
    import torch

    B = env[1]
    rank, rows = 8, [16, 255, 256, 257, 512] + [512] * 1750
    model = B.Model([(n, 64) for n in rows], rank, 4, 64, wl.F32, 5)
    assert model.sizes["workspace_bytes"] <= B.STATIC_WORKSPACE_BYTES
    buf = model.alloc()
    buf["P"].normal_()
    panels = _panels(rows[:5], rank, False)
    for P, o in zip(panels, model.offsets):
        buf["P"][o["p_off"]:o["p_off"] + P.size] = torch.from_numpy(P.ravel()).cuda()
    B.conef_orthonormalise(model.ctx, buf["P"], buf["ws"], model.stream_handle())
    torch.cuda.synchronize()
    for n, P, o in zip(rows, panels, model.offsets):
        got = buf["P"][o["p_off"]:o["p_off"] + P.size].cpu().numpy().reshape(n, rank).astype(np.float64)
        q, r = np.linalg.qr(P.astype(np.float64))
        assert np.abs(got - q * np.sign(np.diag(r))).max() <= 2e-7, n
    model.close()


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("rank", [1, 2, 4, 7, 8, 12, 16, 32])
def test_an_entry_that_is_not_finite_stays_in_its_row(env, rank, value):
    """One entry of P that is not finite, in the first, a middle or the last column: in every other row P^ is the factor of the
    other columns, its own column zero (QR in float64 as above)."""
    import torch

    B = env[1]
    bad = sorted({0, rank // 2, rank - 1})
    n, row = 300, 130
    panels = _panels([n] * len(bad), rank, False)
    model = B.Model([(n, 64)] * len(bad), rank, 4, 64, wl.F32, 5)
    buf = model.alloc()
    for P, c, o in zip(panels, bad, model.offsets):
        P[row, c] = value
        buf["P"][o["p_off"]:o["p_off"] + P.size] = torch.from_numpy(P.ravel()).cuda()
    B.conef_orthonormalise(model.ctx, buf["P"], buf["ws"], model.stream_handle())
    torch.cuda.synchronize()
    rest = np.arange(n) != row
    for P, c, o in zip(panels, bad, model.offsets):
        got = buf["P"][o["p_off"]:o["p_off"] + P.size].cpu().numpy().reshape(n, rank).astype(np.float64)
        keep = [k for k in range(rank) if k != c]
        assert not got[rest, c].any(), (rank, c)
        if keep:
            q, r = np.linalg.qr(P[:, keep].astype(np.float64))
            q *= np.sign(np.diag(r))
            assert np.abs(got[np.ix_(rest, keep)] - q[rest]).max() <= 2e-7, (rank, c)
    model.close()
