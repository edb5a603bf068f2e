"""Chains of dense layers of the Hadamard block (csrc/dense_chain.hip) on graphs with triplets, so that the steps about the triplet sum meet live
data: rows at the edges of a workgroup's 64 and of a wavefront's 16, several thousand rows on two streams, one pass by the chains and the other
layer by layer, and the bits that a step keeps of its operand."""
import numpy as np
import pytest
import torch

import synth
from tests import helpers as H
from tests.test_gpu_block_D import _case
from tests.test_gpu_dense_chain import _check, _compare
from tests.test_gpu_no_triplets import _graph, _pairs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _molecules(triangles, pairs, seed):
    """Structures of three atoms (6 edges, 6 triplets each) and of two (2 edges), all near the origin."""
    rng = np.random.default_rng(seed)
    pos, gptr = [], [0]
    for n in [3] * triangles + [2] * pairs:
        corner = np.array([[0.0, 0.0, 0.0], [1.5, 0.0, 0.0], [0.4, 1.6, 0.0]])[:n]
        q, _ = np.linalg.qr(rng.standard_normal((3, 3)))
        pos += list((corner + rng.uniform(-0.2, 0.2, (n, 3))) @ q)
        gptr.append(len(pos))
    return np.array(pos, np.float32), np.array(gptr, np.int32)


@pytest.mark.parametrize("triangles,pairs", [(1, 0), (2, 2), (3, 0), (10, 1), (10, 2), (11, 0), (13, 1), (21, 1), (21, 2)])   # 6, 16, 18, 62, 64, 66, 80, 128, 130
@pytest.mark.parametrize("emb,int_emb", [(32, 16), (128, 64), (256, 48)])
def test_rows_at_the_edges_of_a_workgroup(lib, ctx, emb, int_emb, triangles, pairs):
    w = synth.get_workload("cfg2", emb=emb, int_emb=int_emb)
    pos, ref, e, t = _case(lib, ctx, w, 0, _molecules(triangles, pairs, triangles))
    assert e["n_edges"] == 6 * triangles + 2 * pairs and t["n_triplets"] == 6 * triangles
    _check(_compare(lib, ctx, w, pos, ref, e, t))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("emb", [64, 256])
def test_two_streams_with_triplets(lib, emb):
    # from 2048 edges on: grouped weight gradients on the side stream beside the second chain
    from paper_2203_09697_amd.stack import StackD
    ctx = lib.Context(0)
    w = synth.get_workload("cfg2", emb=emb, int_emb=64)
    pos, ref, e, t = _case(lib, ctx, w, 3, synth.slab_adsorbate_positions(4, 4, 4, 3, 5, seed=3))
    E = e["n_edges"]
    assert E > 4000
    W = [synth.weights_D(w.dims, seed=5 + b, bias_scale=0.1) for b in range(2)]
    m, gup = synth.edge_embeddings(E, emb, seed=6)
    st = StackD(ctx, w.dims, [lib.weights_to_device(q) for q in W], t, lib.gp_basis_forward(ctx, w.dims, e, t))
    got = []
    for on in (True, False, True):
        lib.gp_set_side_stream(ctx, on)
        out = st.forward(H.to_dev(m, torch.float32)).clone()
        gm, gw = st.backward(H.to_dev(gup, torch.float32))
        got.append([out, gm.clone()] + [v.clone() for g in gw for v in g.values()])
    assert all(torch.equal(a, b) for a, b in zip(got[0], got[2]))
    assert all(torch.equal(a, b) for a, b in zip(got[0][:2], got[1][:2]))   # the weight gradients form other groups on one stream
    want = H.oracle_stack_D(ref, H.oracle_basis_D(pos, ref, w.dims), w.dims, W, m, gup)
    worst = max(H.rel_l2(gw[b][k].cpu().numpy(), g) for b in range(2) for k, g in want[2][b].items())
    out, gm = (x.cpu().numpy() for x in got[0][:2])
    _check((H.rel_l2(out, want[0]), H.rel_l2(gm, want[1]), H.row_err(out, want[0]), H.row_err(gm, want[1]), worst))


@pytest.mark.parametrize("forward_at,backward_at", [(0, 8), (8, 0), (8, 8)])
@pytest.mark.parametrize("emb", [64, 256])
def test_one_pass_by_the_chains_the_other_by_layers(lib, ctx, emb, forward_at, backward_at):
    # a chain needs scratch that starts on 16 bytes: what one pass has saved serves the other, whichever way either goes
    from paper_2203_09697_amd.stack import StackD
    w = synth.get_workload("cfg2", emb=emb, int_emb=64)
    pos, ref, e, t = _case(lib, ctx, w, 3, synth.slab_adsorbate_positions(1, 3, 3, 3, 4, seed=4))
    W = synth.weights_D(w.dims, seed=5, bias_scale=0.1)
    m, gup = synth.edge_embeddings(e["n_edges"], emb, seed=6)
    st = StackD(ctx, w.dims, [lib.weights_to_device(W)], t, lib.gp_basis_forward(ctx, w.dims, e, t))
    size = st.scratch.numel()
    room = torch.empty(size + 8, dtype=torch.uint8, device="cuda:0")
    st.scratch = room[forward_at:forward_at + size]
    assert st.scratch.data_ptr() % 16 == forward_at
    out = st.forward(H.to_dev(m, torch.float32)).cpu().numpy()
    st.scratch = room[backward_at:backward_at + size]
    gm, gw = st.backward(H.to_dev(gup, torch.float32))
    gm = gm.cpu().numpy()
    want = H.oracle_stack_D(ref, H.oracle_basis_D(pos, ref, w.dims), w.dims, [W], m, gup)
    worst = max(H.rel_l2(gw[0][k].cpu().numpy(), g) for k, g in want[2][0].items())
    _check((H.rel_l2(out, want[0]), H.rel_l2(gm, want[1]), H.row_err(out, want[0]), H.row_err(gm, want[1]), worst))


@pytest.mark.parametrize("emb", [32, 64, 128, 192, 256])
def test_a_step_keeps_all_bits_of_its_operand(lib, ctx, emb):
    """Weights that are permutations times powers of two: a product has one term per value, exact in fp32 where the operand enters with its 24 bits (22
    bits are up to 1.2e-7 off).  Forward silu(z) = z from 2^13 on and 0 for as much below; backward silu'(0) = 1/2.  What is left is the
    rounding of the skip's addition, half an ulp."""
    w = synth.get_workload("cfg2", emb=emb, int_emb=32, n_res_before=0, n_res_after=0)
    pos, gptr = _pairs(40, 3)
    ref, e, t = _graph(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)
    E, rng = e["n_edges"], np.random.default_rng(emb)
    from paper_2203_09697_amd.stack import StackD
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    p, q = rng.permutation(emb), rng.permutation(emb)
    W["W_ji"][p, np.arange(emb)] = 2.0 ** 20       # column j of the product is row p[j] of the operand
    W["W_lin"][q, np.arange(emb)] = 2.0 ** rng.integers(0, 3, emb)
    st = StackD(ctx, w.dims, [lib.weights_to_device(W)], t, lib.gp_basis_forward(ctx, w.dims, e, t))
    m = (np.sign(rng.standard_normal((E, emb))) * rng.uniform(1.0 / 32.0, 1.0, (E, emb))).astype(np.float32)
    g = rng.standard_normal((E, emb)).astype(np.float32)
    Wji, Wlin, half_ulp = W["W_ji"].astype(np.float64), W["W_lin"].astype(np.float64), 2.0 ** -24
    want = np.maximum(m.astype(np.float64) @ Wji, 0) @ Wlin + m
    out = st.forward(H.to_dev(m, torch.float32)).cpu().numpy()
    assert (np.abs(out - want) <= half_ulp * np.abs(want)).all()
    st.forward(torch.zeros((E, emb), device="cuda:0"))
    gm = st.backward(H.to_dev(g, torch.float32))[0].cpu().numpy()
    want = g + 0.25 * (g.astype(np.float64) @ Wlin.T) @ Wji.T
    assert (np.abs(gm - want) <= half_ulp * np.abs(want)).all()


def test_an_infinity_fills_its_row(lib, ctx):
    from paper_2203_09697_amd.stack import StackD
    w = synth.get_workload("cfg2", emb=64, int_emb=32)
    pos, gptr = _pairs(40, 2)
    ref, e, t = _graph(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)
    m, gup = synth.edge_embeddings(80, 64, seed=6)
    st = StackD(ctx, w.dims, [lib.weights_to_device(synth.weights_D(w.dims, seed=5, bias_scale=0.1))], t, lib.gp_basis_forward(ctx, w.dims, e, t))
    m[7, 3], m[70, 1] = np.inf, np.nan
    out = st.forward(H.to_dev(m, torch.float32))
    assert not torch.isfinite(out[[7, 70]]).any()
