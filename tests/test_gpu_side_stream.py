"""Wide Hadamard blocks (weight gradients one by one) on graphs of a few hundred to a few thousand edges: the side stream is in use, and what it
computes does not depend on it."""
import time

import pytest
import torch

import synth
from tests import helpers as H
from tests.test_gpu_block_D import _case

pytestmark = pytest.mark.gpu


def _stack(lib, ctx, emb, slab, blocks):
    from paper_2203_09697_amd.stack import StackD
    w = synth.get_workload("cfg2", emb=emb, int_emb=128)
    pos, ref, e, t = _case(lib, ctx, w, 3, synth.slab_adsorbate_positions(*slab, seed=3))
    W = [synth.weights_D(w.dims, seed=5 + b, bias_scale=0.1) for b in range(blocks)]
    m, gup = synth.edge_embeddings(e["n_edges"], emb, seed=6)
    st = StackD(ctx, w.dims, [lib.weights_to_device(q) for q in W], t, lib.gp_basis_forward(ctx, w.dims, e, t))
    return st, w, pos, ref, W, m, gup


# (structures, nx, ny, layers, adsorbates): 200 to 600 edges, about 1000, more than 2048
@pytest.mark.parametrize("emb,slab", [(512, (1, 2, 2, 3, 3)), (512, (1, 3, 3, 4, 2)), (512, (2, 4, 3, 4, 5)), (1024, (1, 2, 2, 3, 3))])
def test_results_do_not_depend_on_the_side_stream(lib, emb, slab):
    ctx = lib.Context(0)
    st, w, pos, ref, W, m, gup = _stack(lib, ctx, emb, slab, 2)
    got = []
    for on in (True, False):
        lib.gp_set_side_stream(ctx, on)
        out = st.forward(H.to_dev(m, torch.float32)).clone()
        gm, gw = st.backward(H.to_dev(gup, torch.float32))
        got.append([out, gm.clone()] + [v.clone() for g in gw for v in g.values()])
    assert all(torch.equal(a, b) for a, b in zip(*got))
    want = H.oracle_stack_D(ref, H.oracle_basis_D(pos, ref, w.dims), w.dims, W, m, gup)
    err = [H.rel_l2(got[0][0].cpu().numpy(), want[0]), H.rel_l2(got[0][1].cpu().numpy(), want[1])]
    print("E %d out %.2e grad_m %.2e" % (len(m), *err))
    assert max(err) < 2e-6   # as in test_gpu_dense_chain.py


def test_the_side_stream_takes_the_weight_gradients(lib):
    """A pass of width 1024 over a few hundred edges, on two streams 0.79 of the time on one; with every product on one the times are equal."""
    ctx = lib.Context(0)
    st, w, pos, ref, W, m, gup = _stack(lib, ctx, 1024, (1, 2, 2, 4, 3), 2)
    dm, dg = H.to_dev(m, torch.float32), H.to_dev(gup, torch.float32)
    times = {True: [], False: []}
    for k in range(8):
        for on in times:
            lib.gp_set_side_stream(ctx, on)
            for n in (2, 10):
                torch.cuda.synchronize()
                start = time.perf_counter()
                for _ in range(n):
                    st.forward(dm)
                    st.backward(dg)
                torch.cuda.synchronize()
            times[on].append(time.perf_counter() - start)
    print({on: "%.3f ms" % (min(t) * 100) for on, t in times.items()})
    assert min(times[True]) < 0.92 * min(times[False])
