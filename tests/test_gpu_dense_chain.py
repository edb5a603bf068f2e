"""Dense layers of the Hadamard block as chains in one launch (csrc/dense_chain.hip), through the block: rows at the edges of a workgroup's 64
and of a wavefront's 16, every width it is compiled for with narrow and equal triplet widths, no and many residual layers."""
import numpy as np
import pytest
import torch

import synth
from tests import helpers as H
from tests.test_gpu_block_D import _case
from tests.test_gpu_no_triplets import _graph, _pairs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _compare(lib, ctx, w, pos, ref, e, t, blocks=1, split=1):
    from paper_2203_09697_amd.stack import StackD
    dims, E = w.dims, len(ref["src"])
    W = [synth.weights_D(dims, seed=5 + b, bias_scale=0.1) for b in range(blocks)]
    m, gup = synth.edge_embeddings(E, dims.emb, seed=6)
    want = H.oracle_stack_D(ref, H.oracle_basis_D(pos, ref, dims), dims, W, m, gup)
    lib.gp_set_f32_gemm(ctx, split)
    try:
        st = StackD(ctx, dims, [lib.weights_to_device(q) for q in W], t, lib.gp_basis_forward(ctx, dims, e, t))
        out = st.forward(H.to_dev(m, torch.float32)).cpu().numpy()
        gm, gw = st.backward(H.to_dev(gup, torch.float32))
    finally:
        lib.gp_set_f32_gemm(ctx, 1)
    worst = max(H.rel_l2(gw[b][k].cpu().numpy(), g) if np.abs(g).max() > 0 else np.abs(gw[b][k].cpu().numpy()).max() for b in range(blocks) for k, g in want[2][b].items())
    return H.rel_l2(out, want[0]), H.rel_l2(gm.cpu().numpy(), want[1]), H.row_err(out, want[0]), H.row_err(gm.cpu().numpy(), want[1]), worst


def _check(err):
    # a product is 1e-7 off (csrc/dense_chain.hip); up to 20 layers in a row and back, a residual layer adding to what came before, 2e-6;
    # single rows and sums over all edges 1e-5, as for the layers one by one
    print("out %.2e grad_m %.2e rows %.2e %.2e weights %.2e" % err)
    assert max(err[:2]) < 2e-6 and max(err[2:]) < 1e-5


@pytest.mark.parametrize("pairs", [1, 8, 31, 32, 33, 40])     # 2 edges each: 2, 16, 62, 64, 66, 80 rows
@pytest.mark.parametrize("emb,int_emb", [(32, 16), (64, 64), (192, 48)])
def test_rows_at_the_edges_of_a_workgroup(lib, ctx, emb, int_emb, pairs):
    w = synth.get_workload("cfg2", emb=emb, int_emb=int_emb)
    pos, gptr = _pairs(pairs, pairs)
    _check(_compare(lib, ctx, w, pos, *_graph(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)))


@pytest.mark.parametrize("emb,int_emb", [(32, 32), (64, 16), (64, 48), (128, 64), (192, 192), (256, 16), (256, 64), (256, 256)])
@pytest.mark.parametrize("before,after", [(0, 0), (1, 2), (4, 4)])
def test_widths_and_residual_layers(lib, ctx, emb, int_emb, before, after):
    w = synth.get_workload("cfg2", emb=emb, int_emb=int_emb, n_res_before=before, n_res_after=after)
    pos, ref, e, t = _case(lib, ctx, w, 3, synth.slab_adsorbate_positions(1, 2, 2, 3, 3, seed=3))
    _check(_compare(lib, ctx, w, pos, ref, e, t, blocks=2 if before == 1 else 1))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("emb,pairs", [(256, 16384), (256, 16385), (192, 16400)])   # the last graph that takes the chain at width 256, and the next
def test_many_rows(lib, ctx, emb, pairs):
    w = synth.get_workload("cfg2", emb=emb, int_emb=16, n_res_before=0, n_res_after=1)
    pos, gptr = _pairs(pairs, 1)
    _check(_compare(lib, ctx, w, pos, *_graph(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)))


@pytest.mark.parametrize("slabs,nx,ny", [(1, 2, 2), (12, 4, 3)])   # the layers one by one: 64 x 64 and 128 x 128 tiles
def test_a_width_without_a_chain(lib, ctx, slabs, nx, ny):
    w = synth.get_workload("cfg2", emb=224, int_emb=64)
    pos, ref, e, t = _case(lib, ctx, w, 3, synth.slab_adsorbate_positions(slabs, nx, ny, 3, 5, seed=3))
    _check(_compare(lib, ctx, w, pos, ref, e, t))


def test_an_infinity_stays_in_its_row(lib, ctx):
    from paper_2203_09697_amd.stack import StackD
    w = synth.get_workload("cfg2", emb=64, int_emb=32)
    pos, gptr = _pairs(40, 2)
    ref, e, t = _graph(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)
    m, gup = synth.edge_embeddings(len(ref["src"]), 64, seed=6)
    st = StackD(ctx, w.dims, [lib.weights_to_device(synth.weights_D(w.dims, seed=5, bias_scale=0.1))], t, lib.gp_basis_forward(ctx, w.dims, e, t))
    clean = st.forward(H.to_dev(m, torch.float32)).clone()
    m[7, 3], m[70, 1] = np.inf, np.nan
    out = st.forward(H.to_dev(m, torch.float32))
    keep = np.setdiff1d(np.arange(80), [7, 70])
    assert torch.equal(out[keep], clean[keep]) and not torch.isfinite(out[[7, 70]]).any(1).all()
