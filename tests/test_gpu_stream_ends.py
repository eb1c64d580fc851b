"""GPU parity tests of the element-wise gradient compressors on matrices of every length modulo a sign word (32 elements):
the last octet of a matrix may hold one to eight elements, end its code word or not, and end its sign word or not.  Each
step against the oracle on the same seeded inputs, bit for bit and free-running, over three steps (from the second on the
old codes of the last octet are not zero)."""
import numpy as np
import pytest

from paper_2312_08538_amd import workloads as wl

pytestmark = pytest.mark.gpu

STEPS = 3
# N mod 32 = 0 .. 31 in the matrix's third run of 512, and three shapes of layers: N mod 32 = 8, 16 and 24
LAYOUT = [(1, 1056 + j) for j in range(32)] + [(24, 147), (40, 650), (72, 147)]
SIZES = [(2, 16), (2, 256), (4, 8), (4, 128), (4, 512), (8, 8), (8, 16), (8, 64)]


@pytest.fixture(scope="module")
def env():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from oracle import conef_ref as R
    from paper_2312_08538_amd import binding as B
    import test_gpu_sketch as S

    B.lib()
    return R, B, S, torch


def _fresh(R, bits, block, vectors):
    return [[a for _ in range(vectors) for a in (np.zeros(R.n_words(n * m, bits), np.uint32), np.zeros(R.n_blocks(n * m, block), np.float32))]
            for n, m in LAYOUT]


def _compare_vectors(dev, o, want, tag):
    """dev: the library's codes, scales (, second codes, second scales); want: the oracle's."""
    for i, (d, w) in enumerate(zip(dev, want)):
        off = o["word_off"] if w.dtype == np.uint32 else o["scale_off"]
        got = d[off:off + w.size].cpu().numpy().view(np.uint32)
        w = w.view(np.uint32)
        assert np.array_equal(got, w), f"{tag}: array {i} of the error differs at {np.nonzero(got != w)[0][:8]} of {w.size}"


@pytest.mark.parametrize("bits,block", SIZES)
@pytest.mark.parametrize("gdt", [wl.F32, wl.BF16])
@pytest.mark.parametrize("vectors", [1, 2])
def test_scaled_sign_at_the_end_of_a_matrix(env, bits, block, gdt, vectors):
    R, B, S, torch = env
    seed = 4000 + bits + block
    model = B.Model(LAYOUT, 1, bits, block, gdt, seed)
    buf = model.alloc()
    dev = [buf["codes"], buf["scales"]] + ([torch.zeros_like(buf["codes"]), torch.zeros_like(buf["scales"])] if vectors == 2 else [])
    signs = torch.zeros(B.conef_ss_sizes(model.ctx)["sign_words"], dtype=torch.int32, device="cuda:0")
    cs = torch.zeros(len(LAYOUT), dtype=torch.float32, device="cuda:0")
    rng = np.random.default_rng([bits, block, gdt, vectors])
    states = _fresh(R, bits, block, vectors)
    for t in range(STEPS):
        grads = [S._grad(rng, n, m, gdt) for n, m in LAYOUT]
        S._to_dev_grads(torch, model, buf, grads)
        signs.fill_(-1)
        print(f"[scaled sign ends bits {bits} block {block} gdt {gdt} vectors {vectors}] step {t}: launching", flush=True)
        (B.conef_i_ss_step if vectors == 2 else B.conef_ss_step)(model.ctx, buf["grads"], *dev, signs, cs, buf["ws"], t, model.stream_handle())
        torch.cuda.synchronize()
        for l, (n, m) in enumerate(LAYOUT):
            N, o = n * m, model.offsets[l]
            tag = f"{n} x {m} (N mod 32 = {N % 32}) step {t}"
            if vectors == 2:
                words, c = R.i_ss_step_matrix(grads[l], *states[l], bits, block, seed, l, t)
            else:
                words, c = R.ss_step_matrix(grads[l], *states[l], bits, block, 0.0, seed, l, t)
            # fp64 sums of the same terms in another order: at most one unit in the last place of fp32
            assert abs(float(cs[l].item()) - float(c)) <= float(np.spacing(np.float32(c))), f"{tag}: scale"
            if np.float32(cs[l].item()) != np.float32(c):       # changes every argument: go on from the library's state
                for d, w in zip(dev, states[l]):
                    off = o["word_off"] if w.dtype == np.uint32 else o["scale_off"]
                    w[:] = d[off:off + w.size].cpu().numpy().view(w.dtype)
                continue
            so = B.conef_ss_offsets(model.ctx, l)["sign_off"]
            got = signs[so:so + words.size].cpu().numpy().view(np.uint32).copy()
            if N % 32:
                got[-1] &= np.uint32((1 << (N % 32)) - 1)          # bits beyond the last entry are not part of the result
            assert np.array_equal(got, words), f"{tag}: sign words"
            _compare_vectors(dev, o, states[l], tag)
    model.close()


RAGGED = [(2, 16, 3), (2, 256, 10), (4, 8, 10), (4, 128, 2), (4, 512, 33), (8, 8, 7), (8, 64, 10)]      # bits, block, stratum length


@pytest.mark.parametrize("bits,block,group", RAGGED)
@pytest.mark.parametrize("kind", ["block", "strata", "uniform"])
@pytest.mark.parametrize("vectors", [1, 2])
def test_kept_coordinates_at_the_end_of_a_matrix(env, bits, block, group, kind, vectors):
    R, B, S, torch = env
    gdt = wl.BF16 if (bits + group) % 2 else wl.F32
    beta = 0.0 if vectors == 2 else 0.75
    seed = 4100 + bits + block
    keep = [max(1, n * m // group) for n, m in LAYOUT]
    model = B.Model(LAYOUT, 1, bits, block, gdt, seed)
    B.conef_set_beta(model.ctx, beta)
    if kind == "block":
        B.conef_rb_configure(model.ctx, keep)
        n_delta, offsets = B.conef_rb_sizes(model.ctx)["delta_elems"], B.conef_rb_offsets
        arg, plain, two, call = keep, R.rb_step_matrix, R.i_rb_step_matrix, (B.conef_rb_step, B.conef_i_rb_step)
    else:
        if kind == "strata":
            B.conef_rk_configure(model.ctx, [group] * len(LAYOUT))
        else:
            B.conef_rk_configure_uniform(model.ctx, keep)
        n_delta, offsets = B.conef_rk_sizes(model.ctx)["delta_elems"], B.conef_rk_offsets
        arg = [group] * len(LAYOUT) if kind == "strata" else [-k for k in keep]
        plain, two, call = R.rk_step_matrix, R.i_rk_step_matrix, (B.conef_rk_step, B.conef_i_rk_step)
    buf = model.alloc()
    dev = [buf["codes"], buf["scales"]] + ([torch.zeros_like(buf["codes"]), torch.zeros_like(buf["scales"])] if vectors == 2 else [])
    delta = torch.zeros(n_delta, dtype=torch.float32, device="cuda:0")
    rng = np.random.default_rng([bits, block, vectors, 41])
    states = _fresh(R, bits, block, vectors)
    for t in range(STEPS):
        grads = [S._grad(rng, n, m, gdt) for n, m in LAYOUT]
        S._to_dev_grads(torch, model, buf, grads)
        delta.fill_(float("nan"))
        print(f"[{kind} ends bits {bits} block {block} vectors {vectors}] step {t}: launching", flush=True)
        call[vectors - 1](model.ctx, buf["grads"], *dev, delta, t, model.stream_handle())
        torch.cuda.synchronize()
        for l, (n, m) in enumerate(LAYOUT):
            tag = f"{n} x {m} (N mod 32 = {n * m % 32}) step {t}"
            want = (two(grads[l], *states[l], arg[l], bits, block, seed, l, t) if vectors == 2 else
                    plain(grads[l], *states[l], arg[l], bits, block, beta, seed, l, t))
            o = offsets(model.ctx, l)
            got = delta[o["delta_off"]:o["delta_off"] + want.size].cpu().numpy()
            assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), f"{tag}: kept values"
            _compare_vectors(dev, model.offsets[l], states[l], tag)
    model.close()


@pytest.mark.parametrize("bits,block,group", RAGGED)
@pytest.mark.parametrize("strata", [False, True])
def test_the_first_vector_as_a_random_block_at_the_end_of_a_matrix(env, bits, block, group, strata):
    R, B, S, torch = env
    gdt = wl.F32 if (bits + group) % 2 else wl.BF16
    seed = 4200 + bits + block
    keep = [max(1, n * m // group) for n, m in LAYOUT]
    keep_e = [n * m // 3 for n, m in LAYOUT]
    model = B.Model(LAYOUT, 1, bits, block, gdt, seed)
    if strata:
        B.conef_rk_configure(model.ctx, [group] * len(LAYOUT))
    else:
        B.conef_rb_configure(model.ctx, keep)
    B.conef_i2_configure(model.ctx, keep_e)
    buf = model.alloc()
    e_bufs = [torch.zeros(B.conef_i2_sizes(model.ctx)["e_elems"], dtype=torch.float32, device="cuda:0") for _ in range(2)]
    delta = torch.zeros((B.conef_rk_sizes if strata else B.conef_rb_sizes)(model.ctx)["delta_elems"], dtype=torch.float32, device="cuda:0")
    rng = np.random.default_rng([bits, block, int(strata), 42])
    states = [[np.zeros(k, np.float32)] + s for k, s in zip(keep_e, _fresh(R, bits, block, 1))]
    for t in range(STEPS):
        grads = [S._grad(rng, n, m, gdt) for n, m in LAYOUT]
        S._to_dev_grads(torch, model, buf, grads)
        delta.fill_(float("nan"))
        e_in, e_out = e_bufs[t % 2], e_bufs[(t + 1) % 2]
        e_out.fill_(float("nan"))
        print(f"[first vector block ends bits {bits} block {block} strata {strata}] step {t}: launching", flush=True)
        (B.conef_i2_rk_step if strata else B.conef_i2_rb_step)(model.ctx, buf["grads"], e_in, e_out, buf["codes"], buf["scales"], delta, t,
                                                               model.stream_handle())
        torch.cuda.synchronize()
        for l, (n, m) in enumerate(LAYOUT):
            e, codes, scales = states[l]
            tag = f"{n} x {m} (N mod 32 = {n * m % 32}) step {t}"
            want = (R.i2_rk_step_matrix(grads[l], e, codes, scales, group, bits, block, seed, l, t) if strata else
                    R.i2_rb_step_matrix(grads[l], e, codes, scales, keep[l], bits, block, seed, l, t))
            o = (B.conef_rk_offsets if strata else B.conef_rb_offsets)(model.ctx, l)
            got = delta[o["delta_off"]:o["delta_off"] + want.size].cpu().numpy()
            assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), f"{tag}: kept values"
            eo = B.conef_i2_offsets(model.ctx, l)["e_off"]
            assert np.array_equal(e_out[eo:eo + e.size].cpu().numpy().view(np.uint32), e.view(np.uint32)), f"{tag}: first vector"
            _compare_vectors([buf["codes"], buf["scales"]], model.offsets[l], [codes, scales], tag)
    model.close()
