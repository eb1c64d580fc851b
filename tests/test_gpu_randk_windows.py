"""Random-k where a wave walks several runs of 512 elements and draws its strata's coordinates a window of 256 strata at a
time (models of 8.4 M elements and more): strata of the shortest length the windows take, lengths that put a window's end
inside a run, at a run's end and far behind the item, and a stratum longer than an item.  Against the oracle, bit for bit."""
import numpy as np
import pytest

from paper_2312_08538_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [7, 8, 9, 13, 16, 100, 5000])
@pytest.mark.parametrize("two", [False, True])
def test_windows_of_strata(group, two):
    import torch

    import test_gpu_sketch as S
    from oracle import conef_ref as R
    from paper_2312_08538_amd import binding as B

    n, m, bits, block, seed = 4100, 4099, 4, 128, 77            # four runs per wave, a short last one, a short last stratum
    gdt = wl.BF16 if two else wl.F32
    model = B.Model([(n, m)], 4, bits, block, gdt, seed)
    B.conef_rk_configure(model.ctx, [group])
    buf = model.alloc()
    codes2, scales2 = torch.zeros_like(buf["codes"]), torch.zeros_like(buf["scales"])
    delta = torch.zeros(B.conef_rk_sizes(model.ctx)["delta_elems"], dtype=torch.float32, device="cuda:0")
    rng = np.random.default_rng([group, two])
    state = [np.zeros(R.n_words(n * m, bits), np.uint32), np.zeros(R.n_blocks(n * m, block), np.float32)]
    if two:
        state += [s.copy() for s in state]
    for t in range(2):
        grad = S._grad(rng, n, m, gdt)
        S._to_dev_grads(torch, model, buf, [grad])
        delta.fill_(float("nan"))
        print(f"[random-k windows, strata of {group}, two {two}] step {t}: launching", flush=True)
        if two:
            B.conef_i_rk_step(model.ctx, buf["grads"], buf["codes"], buf["scales"], codes2, scales2, delta, t, model.stream_handle())
            want = R.i_rk_step_matrix(grad, *state, group, bits, block, seed, 0, t)
        else:
            B.conef_rk_step(model.ctx, buf["grads"], buf["codes"], buf["scales"], delta, t, model.stream_handle())
            want = R.rk_step_matrix(grad, *state, group, bits, block, 0.0, seed, 0, t)
        torch.cuda.synchronize()
        assert np.array_equal(delta[:want.size].cpu().numpy().view(np.uint32), want.view(np.uint32)), f"step {t}: kept values"
        for got, arr in zip((buf["codes"], buf["scales"], codes2, scales2), state):
            assert np.array_equal(got[:arr.size].cpu().numpy().view(np.uint32), arr.view(np.uint32)), f"step {t}"
    model.close()
