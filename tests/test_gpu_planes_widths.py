"""fp32 products with operands as two fp16 parts (csrc/gemm_planes.hip) at widths that no chain of layers takes, so that the block's dense
layers run layer by layer on small graphs too: 64 x 64 tiles of 160 and 224 columns, 128 x 128 tiles of 224.  What test_gpu_planes.py asks at widths 128
and 192, with its bounds."""
import numpy as np
import pytest
import torch

import synth
from tests import helpers as H
from tests.test_gpu_no_triplets import _graph, _pairs
from tests.test_gpu_planes import _block

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _layers(lib, ctx, emb, slab, seed, **nonzero):
    """A block without residual layers whose weights are zero but for those given."""
    w = synth.get_workload("cfg2", emb=emb, int_emb=64, n_res_before=0, n_res_after=0)
    pos, gptr = synth.slab_adsorbate_positions(*slab, seed=4)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    return w, e, t, e["n_edges"], W, torch.Generator().manual_seed(seed)


SMALL = (1, 2, 2, 3, 4)


@pytest.mark.parametrize("emb", [160, 224])
def test_values_of_every_size(lib, ctx, emb):
    # rows 2^-90 to 2^60 of each other's size, a row of zeros, weights over 2^40 in every column
    w, e, t, E, W, rng = _layers(lib, ctx, emb, SMALL, 1)
    W_lin = torch.randn(emb, emb, generator=rng) * torch.exp2(torch.randint(-20, 21, (1, emb), generator=rng).float())
    W_ji = torch.randn(emb, emb, generator=rng)
    W["W_lin"], W["W_ji"] = W_lin.numpy(), W_ji.numpy()
    gup = torch.randn(E, emb, generator=rng) * torch.exp2(torch.randint(-90, 61, (E, 1), generator=rng).float())
    gup *= torch.exp2(-torch.randint(0, 13, (E, emb), generator=rng).float())
    gup[7] = 0
    _, gm, _ = _block(lib, ctx, w, t, e, W, torch.zeros(E, emb).numpy(), gup.numpy(), 1)
    g = gup.double()
    want = g + 0.25 * (g @ W_lin.double().t()) @ W_ji.double().t()      # silu'(0) = 1/2 in both layers
    err = (torch.as_tensor(gm).double() - want).norm(dim=1) / want.norm(dim=1).clamp_min(1e-300)
    err[7] = torch.as_tensor(gm)[7].abs().max()
    assert float(err.max()) < 1e-6, err.max()


@pytest.mark.parametrize("emb,slab", [(160, SMALL), (224, SMALL), (224, (13, 4, 3, 3, 5))])   # the last: 128 x 128 tiles, the second one 96 wide
@pytest.mark.parametrize("far", [22, 40])
def test_features_and_weights_far_below_their_neighbours(lib, ctx, emb, slab, far):
    # features 2^-far to 2^far of each other's size against weights that are as much the other way; a weight of 2^60 against a zero
    w, e, t, E, W, rng = _layers(lib, ctx, emb, slab, far)
    size = torch.exp2(torch.randint(-far, far + 1, (1, emb), generator=rng).float())
    half = emb // 2
    size[:, half:] = 2.0 ** -far        # the columns that are looked at
    W_lin = torch.randn(emb, emb, generator=rng) / size
    gup = torch.randn(E, emb, generator=rng) * size
    gup[:, 3], W_lin[:, 3] = 0.0, 2.0 ** 60
    W["W_lin"], W["W_ji"] = W_lin.numpy(), torch.eye(emb).numpy()
    _, gm, _ = _block(lib, ctx, w, t, e, W, torch.zeros(E, emb).numpy(), gup.numpy(), 1)
    g, lin = gup.double(), W_lin.double()
    want, terms = g + 0.25 * g @ lin.t(), g.abs() + 0.25 * g.abs() @ lin.abs().t()
    err = ((torch.as_tensor(gm).double() - want).abs() / terms)[:, half:]
    print("E = %d: %.2e" % (E, err.max()))
    assert float(err.max()) < 1e-6


@pytest.mark.parametrize("emb", [160, 224])
def test_weights_far_below_their_column(lib, ctx, emb):
    # the forward product (weights [K, N]): in every column one weight of 2^30, which meets a feature that is zero
    w, e, t, E, W, rng = _layers(lib, ctx, emb, SMALL, 8)
    W_ji = torch.randn(emb, emb, generator=rng)
    W_ji[9] = 2.0 ** 30
    m = torch.randn(E, emb, generator=rng)
    m[:, 9] = 0.0
    W["W_ji"], W["W_lin"] = W_ji.numpy(), torch.eye(emb).numpy()
    out, _, _ = _block(lib, ctx, w, t, e, W, m.numpy(), m.numpy(), 1)
    act = lambda v: v * torch.sigmoid(v)
    want = act(act(m.double() @ W_ji.double())) + m.double()
    assert H.rel_l2(out, want.numpy()) < 1e-6


@pytest.mark.parametrize("emb", [160, 224])
def test_an_infinity_stays_in_its_row(lib, ctx, emb):
    w = synth.get_workload("cfg2", emb=emb, int_emb=64, n_res_before=0, n_res_after=0)
    pos, gptr = _pairs(80, 1)      # without triplets no edge sees another
    _, e, t = _graph(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)
    E, rng = e["n_edges"], torch.Generator().manual_seed(9)
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    W["W_ji"], W["W_lin"] = (torch.randn(emb, emb, generator=rng).numpy() for _ in range(2))
    gup = torch.randn(E, emb, generator=rng)
    got = []
    for value in (None, float("inf"), float("nan")):
        g = gup.clone()
        if value is not None:
            g[17, 40] = value
        got.append(torch.as_tensor(_block(lib, ctx, w, t, e, W, torch.zeros(E, emb).numpy(), g.numpy(), 1)[1]))
    keep = torch.arange(E) != 17
    for bad in got[1:]:
        assert not bool(torch.isfinite(bad[17]).any()) and torch.equal(bad[keep], got[0][keep])


def test_values_do_not_depend_on_the_tile(lib, ctx):
    # the same slab by itself (64 x 64 tiles) and as the first of twenty (128 x 128); no triplets: their kernels go by the graph
    from paper_2203_09697_amd.stack import StackD
    emb = 224
    w = synth.get_workload("cfg2", emb=emb, int_emb=64)
    one, _ = synth.slab_adsorbate_positions(1, 4, 3, 3, 5, seed=3)
    W = synth.weights_D(w.dims, seed=5, bias_scale=0.1)
    for k in ("W_down", "W_up", "W_sbf1", "W_sbf2"):
        W[k] = W[k] * 0
    W = lib.weights_to_device(W)
    got = []
    for n in (1, 20):
        pos, gptr = np.tile(one, (n, 1)), np.arange(n + 1, dtype=np.int32) * len(one)
        e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
        E = e["n_edges"] // n
        m, gup = (H.to_dev(np.tile(x, (n, 1)), torch.float32) for x in synth.edge_embeddings(E, emb, seed=6))
        st = StackD(ctx, w.dims, [W], t, lib.gp_basis_forward(ctx, w.dims, e, t))
        out = st.forward(m).cpu()
        got.append((out[:E], st.backward(gup)[0].cpu()[:E]))
        assert all(bool(torch.isfinite(x).all()) for x in got[-1])
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
