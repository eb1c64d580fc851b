"""GPU tests of the strip kernels (any layout), of the launches that carry octet and strip workgroups together, and of
the update's row tiles, at the sizes where a rule or a tile ends.  All of them reproduce the oracle bit for bit."""
import numpy as np
import pytest

from paper_2312_08538_amd import workloads as wl
from test_gpu_parity import _run_model, env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,bits,block,dtype", [(1, 4, 128, wl.F32), (3, 8, 64, wl.BF16), (4, 2, 512, wl.F32), (6, 4, 8, wl.F32),
                                                   (8, 4, 256, wl.BF16), (12, 4, 24, wl.F32), (16, 8, 128, wl.BF16), (32, 2, 64, wl.F32)])
def test_strip_kernels_at_the_ends_of_their_tiles(env, rank, bits, block, dtype):
    """Columns one below, at and above a strip (64), a P chunk (256) and the limit between runs of the flat index and
    column segments in the err pass (1024); rows one below, at and above a row tile (32).  Blocks of 24 take the err pass
    for any block."""
    layout = [(33, 63), (32, 65), (31, 255), (65, 257), (40, 1023), (33, 1025), (64, 1029), (35, 2560), (70, 2047)]
    layout = [(max(n, rank), m) for n, m in layout]
    w = wl.Workload("strip-edges", 11, tuple(layout), rank, bits, block, dtype, "normal", 1.0, 0x57819)
    _run_model(env, w, layout, 2, f"strip-r{rank}-b{bits}-B{block}-dt{dtype}")


@pytest.mark.parametrize("rank,bits,block,dtype", [(2, 4, 64, wl.F32), (4, 8, 128, wl.BF16), (4, 4, 256, wl.F32), (8, 2, 128, wl.F32),
                                                   (8, 8, 256, wl.BF16)])
@pytest.mark.parametrize("strips", [1, 7, 24])
def test_octet_and_strip_matrices_in_one_launch(env, rank, bits, block, dtype, strips):
    """A few strip matrices (their workgroups lead the launch, padded to eight) among octet matrices, and more of them
    than the joint launch takes (the two families then run in launches of their own)."""
    layout = [(100, 512), (64, 147)] + [(40, 768), (33 + 2 * strips, 163 if strips < 24 else 2049)] * strips
    w = wl.Workload("mixed", 12, tuple(layout), rank, bits, block, dtype, "normal", 1.0, 0x313D)
    assert _run_model(env, w, layout, 2, f"mixed-r{rank}-b{bits}-B{block}-dt{dtype}-{strips}") == 0


@pytest.mark.parametrize("rank,tiles", [(12, 2), (32, 3), (16, 8)])
def test_update_over_several_row_tiles_per_workgroup(env, rank, tiles):
    """The update on the fp32 matrix cores where a workgroup walks several 64-row tiles: the last item ragged in tiles and
    rows, columns not a multiple of its strip.  Sampled rows (the ends of tiles, items and the matrix) bit for bit."""
    R, B, U = env
    import torch

    m = 1000
    n = tiles * 4096 // 8 * 64 + 64 + 37
    print(f"[update rank {rank} tiles {tiles}] {n} x {m}: launching", flush=True)
    model = B.Model([(n, m)], rank, 4, 128, B.F32, 7)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rank)
    P = torch.randn(model.sizes["p_elems"], device="cuda:0", generator=gen)
    Q = torch.randn(model.sizes["q_elems"], device="cuda:0", generator=gen)
    x = torch.randn(model.sizes["grad_elems"], device="cuda:0", generator=gen)
    rows = np.unique(np.concatenate([np.arange(0, 66), np.arange(64 * tiles - 2, 64 * tiles + 3), np.arange(n // 2 - 40, n // 2 + 40),
                                     np.arange(n - 170, n)]))
    pick = torch.from_numpy(rows).cuda()
    x0 = x[:n * m].view(n, m)[pick].cpu().numpy()
    tail = x[n * m:].clone()
    B.conef_apply_update(model.ctx, P, Q, x, model.stream_handle())
    torch.cuda.synchronize()
    want = R.apply_update(x0, P[:n * rank].view(n, rank)[pick].cpu().numpy(), Q[:m * rank].view(m, rank).cpu().numpy())
    got = x[:n * m].view(n, m)[pick].cpu().numpy()
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
    assert torch.equal(x[n * m:], tail)
    model.close()


@pytest.mark.parametrize("rank,layout", [
    (12, [(2100, 4100), (64, 147), (70, 131)]),        # 1089 tiles of rows on 16-byte boundaries: four row tiles per workgroup, two matrices one
    (32, [(4165, 4096), (300, 4100)]),                 # 2277 tiles: four at rank 32; a matrix of five row tiles in shares of three and two
    (20, [(8256, 4100)]),                              # 4290 tiles: eight, 130 row tiles in 17 shares
    (16, [(1000, 1500), (129, 650)]),                  # few tiles: one per workgroup
    (24, [(2100, 4099), (65, 128)])])                  # nearly all rows off 16-byte boundaries: a tile per workgroup
def test_update_and_decompression_on_either_side_of_the_row_tile_rule(env, rank, layout):
    """Whole matrices, bit for bit: one row tile per workgroup (few tiles, or rows that do not start on 16-byte boundaries)
    and several, the last share ragged in tiles and rows."""
    R, B, U = env
    import torch

    print(f"[update rank {rank}] {layout}: launching", flush=True)
    model = B.Model(layout, rank, 4, 128, B.F32, 7)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rank)
    P = torch.randn(model.sizes["p_elems"], device="cuda:0", generator=gen)
    Q = torch.randn(model.sizes["q_elems"], device="cuda:0", generator=gen)
    x = torch.randn(model.sizes["grad_elems"], device="cuda:0", generator=gen)
    x0, delta = x.clone(), torch.full_like(x, 7.0)
    B.conef_apply_update(model.ctx, P, Q, x, model.stream_handle())
    B.conef_decompress(model.ctx, P, Q, delta, model.stream_handle())
    torch.cuda.synchronize()
    inside = torch.zeros_like(x, dtype=torch.bool)
    for (n, m), o in zip(layout, model.offsets):
        s = slice(o["grad_off"], o["grad_off"] + n * m)
        inside[s] = True
        p = P[o["p_off"]:o["p_off"] + n * rank].view(n, rank).cpu().numpy()
        q = Q[o["q_off"]:o["q_off"] + m * rank].view(m, rank).cpu().numpy()
        want = R.apply_update(x0[s].view(n, m).cpu().numpy(), p, q)
        assert np.array_equal(x[s].view(n, m).cpu().numpy().view(np.uint32), want.view(np.uint32)), f"{n} x {m}: update"
        assert np.array_equal(delta[s].view(n, m).cpu().numpy().view(np.uint32), R.decompress(p, q).view(np.uint32)), f"{n} x {m}: delta"
    assert torch.equal(x[~inside], x0[~inside]) and bool((delta[~inside] == 7.0).all())
    model.close()


def test_an_infinite_factor_entry_stays_in_its_products(env):
    """P pass with an infinity in the last row of Q, columns that do not fill the last operand of four: p Q is infinite
    there with the sign of the product, not NaN from the operand's empty places."""
    R, B, U = env
    import torch

    layout, rank = [(64, 147), (33, 129), (40, 126)], 3
    model = B.Model(layout, rank, 4, 128, B.F32, 5)
    buf = model.alloc("cuda:0")
    rng = np.random.default_rng(5)
    g = [rng.standard_normal((n, m)).astype(np.float32) for n, m in layout]
    for x, (n, m), o in zip(g, layout, model.offsets):
        buf["grads"][o["grad_off"]:o["grad_off"] + n * m] = torch.from_numpy(x.ravel()).cuda()
        q = rng.standard_normal((m, rank)).astype(np.float32)
        q[m - 1, 1] = np.inf
        buf["Q"][o["q_off"]:o["q_off"] + m * rank] = torch.from_numpy(q.ravel()).cuda()
    B.conef_step_p(model.ctx, buf["grads"], buf["codes"], buf["scales"], buf["Q"], buf["P"], buf["ws"], model.stream_handle())
    torch.cuda.synchronize()
    for x, (n, m), o in zip(g, layout, model.offsets):
        P = buf["P"][o["p_off"]:o["p_off"] + n * rank].cpu().numpy().reshape(n, rank)
        assert np.array_equal(P[:, 1], np.where(x[:, m - 1] > 0, np.inf, -np.inf).astype(np.float32))
        assert np.all(np.isfinite(P[:, [0, 2]]))
    model.close()


@pytest.mark.parametrize("rank", [3, 4])
@pytest.mark.parametrize("bits,block", [(2, 64), (4, 128), (8, 64)])
def test_blocks_too_small_to_divide_by_keep_their_codes_apart(env, rank, bits, block):
    """Residuals of 1e-41: levels / max-norm is infinite (a fixed-point product would saturate and the draw wrap it).  The field
    of such a value's neighbour (here zero) stays zero.  Strip and octet matrices; enough values for every draw."""
    R, B, U = env
    import torch

    layout = [(1500, 1026), (1500, 1024)]
    model = B.Model(layout, rank, bits, block, B.F32, 5)
    buf = model.alloc("cuda:0")
    for (n, m), o in zip(layout, model.offsets):
        g = torch.full((n, m), 1e-41)
        g[::2] = -1e-41
        g[:, 1::2] = 0.0
        buf["grads"][o["grad_off"]:o["grad_off"] + n * m] = g.view(-1).cuda()
    P, Q = torch.zeros_like(buf["P"]), torch.zeros_like(buf["Q"])
    B.conef_step_err(model.ctx, buf["grads"], buf["codes"], buf["scales"], P, Q, buf["ws"], 3, model.stream_handle())
    torch.cuda.synchronize()
    for (n, m), o in zip(layout, model.offsets):
        words = buf["codes"][o["word_off"]:o["word_off"] + R.n_words(n * m, bits)].cpu().numpy().view(np.uint32)
        assert not U.unpack(words, n * m, bits).reshape(n, m)[:, 1::2].any()
    model.close()


@pytest.mark.parametrize("rank,bits,block,dtype", [(3, 2, 64, wl.F32), (4, 4, 128, wl.F32), (8, 8, 64, wl.F32), (4, 2, 256, wl.BF16),
                                                   (2, 4, 24, wl.F32), (32, 4, 128, wl.BF16)])
def test_blocks_too_small_to_divide_by_have_zero_codes(env, rank, bits, block, dtype):
    """Blocks whose largest value is at most levels * 2^-112, half of them negative: codes zero, scale kept, in the err pass of
    every family and in the streams (random-k, one and two vectors: of the second the first's argument, unchanged).  A million
    values and more, as one in 65536 draws the zero that made a code of such a value.  Just above, the codes are the oracle's."""
    R, B, U = env
    import torch

    s = (1 << (bits - 1)) - 1
    edge = np.float32(s * 2.0 ** -112)
    layout = [(1100, 1032), (1100, 1024)]
    model = B.Model(layout, rank, bits, block, dtype, 5)
    buf = model.alloc("cuda:0")
    B.conef_rk_configure(model.ctx, [10, 10])
    st, P, Q = model.stream_handle(), torch.zeros_like(buf["P"]), torch.zeros_like(buf["Q"])
    delta = torch.zeros(B.conef_rk_sizes(model.ctx)["delta_elems"], device="cuda:0")
    codes2, scales2 = torch.zeros_like(buf["codes"]), torch.zeros_like(buf["scales"])

    def steps():
        yield "err", lambda: B.conef_step_err(model.ctx, buf["grads"], buf["codes"], buf["scales"], P, Q, buf["ws"], 3, st)
        yield "two vectors", lambda: B.conef_i_step_err(model.ctx, buf["grads"], buf["codes"], buf["scales"], codes2, scales2, P, Q,
                                                        buf["ws"], 3, st)
        yield "random-k", lambda: B.conef_i_rk_step(model.ctx, buf["grads"], buf["codes"], buf["scales"], codes2, scales2, delta, 3, st)

    for value in (edge, np.float32(1e-39)):
        for name, step in steps():
            g = torch.full((model.sizes["grad_elems"],), float(value))
            g[::2] *= -1
            buf["grads"].copy_(g.to(buf["grads"].dtype).cuda())
            for x in (buf["codes"], buf["scales"], codes2, scales2):
                x.zero_()
            step()
            torch.cuda.synchronize()
            assert not buf["codes"].any() and not codes2.any(), (name, value)
            for (n, m), o in zip(layout, model.offsets):
                blocks = R.n_blocks(n * m, block)
                want = buf["grads"][0].abs().float()
                if name != "random-k":          # (there the kept coordinates leave)
                    assert bool((buf["scales"][o["scale_off"]:o["scale_off"] + blocks] == want).all()), (name, value)
    if dtype == wl.F32:
        rng = np.random.default_rng(9)
        x = [(rng.uniform(-1, 1, n * m) * float(edge) * 4).astype(np.float32) for n, m in layout]
        for y in x:
            y[::2 * block] = np.nextafter(edge, np.float32(1))
            for b in range(1, block):
                y[b::2 * block] = np.clip(y[b::2 * block], -edge, edge)
        for y, o in zip(x, model.offsets):
            buf["grads"][o["grad_off"]:o["grad_off"] + y.size] = torch.from_numpy(y).cuda()
        B.conef_reset_error(model.ctx, buf["codes"], buf["scales"], st)
        B.conef_step_err(model.ctx, buf["grads"], buf["codes"], buf["scales"], P, Q, buf["ws"], 3, st)
        torch.cuda.synchronize()
        for l, (y, o) in enumerate(zip(x, model.offsets)):
            words, scales = R.quantise(y, bits, block, 5, l, 3)
            got = buf["codes"][o["word_off"]:o["word_off"] + words.size].cpu().numpy().view(np.uint32)
            assert words.any() and np.array_equal(got, words)
            assert np.array_equal(buf["scales"][o["scale_off"]:o["scale_off"] + scales.size].cpu().numpy(), scales)
    model.close()


def test_high_rank_matrix_with_a_coarser_split(env):
    """A matrix whose finely split partial sums would not fit the static workspace: fewer, larger partials of P and Q+."""
    w = wl.Workload("coarse", 13, ((16384, 700),), 32, 4, 128, wl.F32, "normal", 1.0, 0xC0A25E)
    _run_model(env, w, [(16384, 700)], 1, "coarse-split")


def test_scales_near_the_largest_value_decode_finite(env):
    """Residuals up to 3e38 with 4-bit codes: the second vector of Algorithm 3 takes what the first rounding leaves, at most
    one level of it, and stays finite."""
    R, B, U = env
    import torch

    layout = [(64, 147), (100, 512)]
    model = B.Model(layout, 4, 4, 128, B.F32, 5)
    buf = model.alloc("cuda:0")
    buf["grads"].copy_(torch.from_numpy(np.random.default_rng(6).uniform(-3e38, 3e38, buf["grads"].numel()).astype(np.float32)))
    B.conef_rk_configure(model.ctx, [10, 10])
    delta = torch.zeros(B.conef_rk_sizes(model.ctx)["delta_elems"], device="cuda:0")
    codes2, scales2 = torch.zeros_like(buf["codes"]), torch.zeros_like(buf["scales"])
    B.conef_i_rk_step(model.ctx, buf["grads"], buf["codes"], buf["scales"], codes2, scales2, delta, 1, model.stream_handle())
    torch.cuda.synchronize()
    assert 0 < float(scales2.max()) <= float(buf["scales"].max()) / 7 * 1.0001
    model.close()


@pytest.mark.parametrize("tall", [False, True])
@pytest.mark.parametrize("rank,bits,block,dtype", [(4, 4, 64, wl.F32), (8, 2, 16, wl.BF16), (3, 8, 128, wl.F32), (16, 4, 512, wl.BF16),
                                                   (32, 8, 64, wl.F32), (9, 2, 128, wl.BF16), (17, 4, 64, wl.F32)])
def test_rows_that_start_anywhere_in_an_octet(env, rank, bits, block, dtype, tall):
    """The P and Q+ passes on octets: row lengths of every remainder by 8, below, at and above a strip and three strips; rows
    one below, at and above a wave's step (32) and a workgroup's (128), those of twice the rank and more columns (what a full-rank
    factorisation leaves is rounding error, whose codes are not determined; ranks 9 and 17 are padded to 16 and 32 and leave the
    small ones in, and the stages have a test without this limit).  Without the tall matrix the Q+ pass of most of these models goes
    element by element."""
    layout = [(n, m) for i, m in enumerate([57, 58, 59, 60, 61, 62, 63, 64, 65, 71, 193, 198, 1027])
              for n in ((31, 33, 97, 127, 128, 129, 161)[i % 7],)] + [(40, 7), (33, 1), (50, 17)]
    layout = [(max(n, 2 * rank), max(m, 2 * rank + 1)) for n, m in layout] + [(4500, 257)] * tall
    w = wl.Workload("ragged", 13, tuple(layout), rank, bits, block, dtype, "normal", 1.0, 0x8A66)
    _run_model(env, w, layout, 2, f"ragged-r{rank}-b{bits}-B{block}-dt{dtype}")


def _stages(env, layout, rank, bits, block, dtype, two, seed):
    """P and Q+ by stage calls on random gradients, codes and factors against float64 products of p: an fp32 rounding of p for
    each vector and one of the result, 6e-8 of it each at most."""
    R, B, U = env
    import torch

    model = B.Model(layout, rank, bits, block, dtype, 5)
    buf = model.alloc("cuda:0")
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    s, per = (1 << (bits - 1)) - 1, 32 // bits
    for k in ("grads", "Q", "P"):
        buf[k].normal_(generator=gen)

    def vector(size):
        fields = torch.randint(-s, s + 1, (model.sizes["code_words"], per), device="cuda:0", generator=gen)
        codes = ((fields & ((1 << bits) - 1)) << (torch.arange(per, device="cuda:0") * bits)).sum(1)
        codes = torch.where(codes >= 1 << 31, codes - (1 << 32), codes).to(torch.int32)
        scales = torch.rand(model.sizes["n_scales"], device="cuda:0", generator=gen) * size
        e = torch.zeros(model.sizes["grad_elems"], device="cuda:0")
        B.conef_decode_error(model.ctx, codes, scales, e, model.stream_handle())
        return codes, scales, e

    vectors = [vector(2.0)] + ([vector(0.3)] if two else [])
    P, Q, st = torch.zeros_like(buf["P"]), torch.zeros_like(buf["Q"]), model.stream_handle()
    args = [x for v in vectors for x in v[:2]]
    print(f"[stages {layout[:3]} .. rank {rank} {bits} bits, blocks of {block}, two {two}]: launching", flush=True)
    (B.conef_i_step_p if two else B.conef_step_p)(model.ctx, buf["grads"], *args, buf["Q"], P, buf["ws"], st)
    (B.conef_i_step_q if two else B.conef_step_q)(model.ctx, buf["grads"], *args, buf["P"], Q, buf["ws"], st)
    torch.cuda.synchronize()
    for (n, m), o in zip(layout, model.offsets):
        g = slice(o["grad_off"], o["grad_off"] + n * m)
        p = (buf["grads"][g].double() + sum(v[2][g].double() for v in vectors)).view(n, m)
        rows, cols = slice(o["p_off"], o["p_off"] + n * rank), slice(o["q_off"], o["q_off"] + m * rank)
        for got, want in ((P[rows].view(n, rank), p @ buf["Q"][cols].double().view(m, rank)),
                          (Q[cols].view(m, rank), p.T.contiguous() @ buf["P"][rows].double().view(n, rank))):
            assert float((got.double() - want).norm() / want.norm()) <= 3e-7, (n, m, rank)
    model.close()


@pytest.mark.parametrize("rank,bits,block,dtype,two", [
    (16, 4, 64, wl.F32, False), (32, 2, 64, wl.BF16, False), (32, 8, 512, wl.F32, True), (16, 2, 128, wl.BF16, True), (12, 4, 64, wl.F32, True),
    (24, 4, 8, wl.F32, True), (31, 4, 128, wl.F32, False), (8, 2, 16, wl.BF16, True), (3, 8, 64, wl.F32, True), (1, 4, 64, wl.BF16, True)])
@pytest.mark.parametrize("tall", [False, True])
def test_stages_of_strip_matrices(env, rank, bits, block, dtype, two, tall):
    """Every padded rank, one and two vectors: strips of part of 64 columns, whole ones and a few more, rows below, at and above a
    wave's step; the Q+ pass element by element and (with a tall matrix) on octets."""
    layout = [(33, m) for m in (57, 58, 59, 60, 61, 62, 63, 64, 65, 193)] + [(32, 40), (40, 33), (64, 71), (129, 1027), (161, 35)]
    _stages(env, layout + [(4500, 257)] * tall, rank, bits, block, dtype, two, rank)


@pytest.mark.parametrize("rank", [2, 3])
def test_a_very_wide_matrix_beside_others(env, rank):
    """More than 2^24 columns: that matrix goes element by element, the others on octets (at rank 2 beside an octet matrix, in
    the launch for both)."""
    _stages(env, [(3, 2 ** 24 + 72), (64, 147), (500, 77), (100, 512), (2500, 700)], rank, 4, 64, wl.F32, False, 7)
