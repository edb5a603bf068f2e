"""A Hadamard block over more edges than the gradients of all its layers are kept for (a buffer each, 2 GiB): forward as a chain, backward layer by
layer with buffers in turn and weight gradients one by one.  Against the same structures in two halves, each of which is below that line."""
import pytest
import torch

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
def test_beyond_the_line_equals_two_halves_below_it(lib):
    from paper_2203_09697_amd.stack import StackD
    ctx = lib.Context(0)
    emb, half = 32, 210
    w = synth.get_workload("cfg2", emb=emb, int_emb=16, n_res_before=4, n_res_after=4)
    pos, gptr = synth.slab_adsorbate_positions(half, 4, 4, 4, 8, seed=1)
    n = len(pos)
    graph = lambda copies: lib.build_graph(ctx, H.to_dev(torch.as_tensor(pos).repeat(copies, 1), torch.float32),
                                           torch.cat([H.to_dev(gptr, torch.int32)] + [H.to_dev(gptr[1:], torch.int32) + k * n for k in range(1, copies)]),
                                           w.dims.cutoff, w.max_neighbors)
    line = 2 ** 31 // (4 * emb * (2 + 2 * 8))   # 2 GiB of buffers beyond the four
    W = [lib.weights_to_device(synth.weights_D(w.dims, seed=5, bias_scale=0.1))]

    def step(copies, m, g):
        e, t = graph(copies)
        st = StackD(ctx, w.dims, W, t, lib.gp_basis_forward(ctx, w.dims, e, t))
        out = st.forward(m)
        gm, gw = st.backward(g)
        return e["n_edges"], out, gm, gw[0]

    E1 = graph(1)[0]["n_edges"]
    assert E1 < line < 2 * E1, (E1, line)
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    # a gradient with a mean: sums over 1e6 edges of one without keep 1e-3 of their terms, and of a rounding that the edges share all
    m, g = (torch.randn((2 * E1, emb), generator=gen, device="cuda:0") + mean for mean in (0.0, 1.0))
    E2, out, gm, gw = step(2, m, g)
    assert E2 == 2 * E1
    low, high = step(1, m[:E1].contiguous(), g[:E1].contiguous()), step(1, m[E1:].contiguous(), g[E1:].contiguous())
    err = lambda a, b: float((a.double() - b.double()).norm() / b.double().norm())
    # forward: the same kernel on the same rows; backward: 17 layers of 1e-7 to 2e-7 each way, on both sides, 2e-6; a weight gradient is that
    # and its sum, whose terms keep a quarter and more of their size
    assert torch.equal(out, torch.cat([low[1], high[1]]))
    assert err(gm, torch.cat([low[2], high[2]])) < 2e-6
    errs = {k: err(v, low[3][k].double() + high[3][k].double()) for k, v in gw.items()}
    print("E %d grad_m %.1e weights %.1e" % (E2, err(gm, torch.cat([low[2], high[2]])), max(errs.values())))
    assert max(errs.values()) < 2e-6, errs
