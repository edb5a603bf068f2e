"""fp32 products with operands as two fp16 parts (csrc/gemm_planes.hip), through the Hadamard block whose dense layers they are, and
the fp32 weight gradients of both blocks (three bf16 parts)."""
import numpy as np
import pytest
import torch

import synth
from tests import helpers as H
from tests.test_gpu_block_D import _case

pytestmark = pytest.mark.gpu


# (emb, int_emb, slabs, nx, ny): which tile of the forward products, and what is partial in it
SHAPES = [
    (128, 64, 1, 2, 2),      # 64 x 64 tiles, the last rows a part of one; K = 64 of the up-projection stays with the other kernels
    (272, 144, 2, 2, 2),     # K = 272 and 144 end in half a chunk of 32, N = 272 in half a block of 32 columns
    (192, 64, 12, 4, 3),     # 128 x 128 tiles, the second one half empty
    (64, 64, 16, 4, 4),      # K = 64, taken for its many rows
    (512, 64, 16, 5, 4),     # 128 x 256 tiles
]


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _block(lib, ctx, w, t, e, W, m, gup, split):
    from paper_2203_09697_amd.stack import StackD
    lib.gp_set_f32_gemm(ctx, split)
    try:
        st = StackD(ctx, w.dims, [lib.weights_to_device(W)], t, lib.gp_basis_forward(ctx, w.dims, e, t))
        out = st.forward(H.to_dev(m, torch.float32)).cpu().numpy()
        gm, gw = st.backward(H.to_dev(gup, torch.float32))
        return out, gm.cpu().numpy(), {k: v.cpu().numpy() for k, v in gw[0].items()}
    finally:
        lib.gp_set_f32_gemm(ctx, 1)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("emb,int_emb,slabs,nx,ny", SHAPES, ids=["%d_%d_%d" % s[:3] for s in SHAPES])
def test_block_against_the_oracle(lib, ctx, emb, int_emb, slabs, nx, ny):
    # Relative error of a product: 1.6e-7 at K = 2048 and less below; ten layers in a row and back keep it under 2e-6, and the
    # fp32 instruction on the same inputs is no closer (its products are 2 to 5 times further off; 1.5 leaves room for luck in a
    # single norm).  Sums over all edges (weights, biases most of all) collect what the edges' rounding has in common: the square
    # root of edges times width.  2.6e-6 measured at 23453 edges of width 256 makes 4.2e-6 at 30281 of width 512; 1e-5 allows twice.
    w = synth.get_workload("cfg2", emb=emb, int_emb=int_emb)
    pos, ref, e, t = _case(lib, ctx, w, 3, synth.slab_adsorbate_positions(slabs, nx, ny, 3, 5, seed=3))
    E = len(ref["src"])
    W = synth.weights_D(w.dims, seed=5, bias_scale=0.1)
    m, gup = synth.edge_embeddings(E, emb, seed=6)
    want = H.oracle_stack_D(ref, H.oracle_basis_D(pos, ref, w.dims), w.dims, [W], m, gup)
    got, plain = (_block(lib, ctx, w, t, e, W, m, gup, s) for s in (1, 0))
    for i in range(2):
        err = H.rel_l2(got[i], want[i])
        print("E=%d %s: two fp16 parts %.2e, fp32 instruction %.2e" % (E, ("out", "grad_m")[i], err, H.rel_l2(plain[i], want[i])))
        assert err < 2e-6 and err < 1.5 * H.rel_l2(plain[i], want[i])
        assert H.row_err(got[i], want[i]) < 1e-5
    worst = {s: max(H.rel_l2(r[2][k], g) for k, g in want[2][0].items()) for s, r in (("parts", got), ("instruction", plain))}
    print("weight gradients: 16-bit parts %.2e, fp32 instruction %.2e" % (worst["parts"], worst["instruction"]))
    assert worst["parts"] < 1e-5


def test_values_of_every_size(lib, ctx):
    # Gradient rows 2^-90 to 2^60 of each other's size, a row of zeros, values over 2^12 within every row and weights over 2^40
    # within every column: a row keeps its relative error, since the scale is its own.  All weights but two are zero and so is m,
    # which makes the block linear in its gradient: silu'(0) = 1/2 in both layers.
    w = synth.get_workload("cfg2", emb=128, int_emb=64, n_res_before=0, n_res_after=0)
    pos, ref, e, t = _case(lib, ctx, w, 4, synth.slab_adsorbate_positions(1, 2, 2, 3, 4, seed=4))
    E = len(ref["src"])
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    rng = torch.Generator().manual_seed(1)
    W_lin = torch.randn(128, 128, generator=rng) * torch.exp2(torch.randint(-20, 21, (1, 128), generator=rng).float())
    W_ji = torch.randn(128, 128, generator=rng)
    W["W_lin"], W["W_ji"] = W_lin.numpy(), W_ji.numpy()
    m = torch.zeros(E, 128)
    rows = torch.exp2(torch.randint(-90, 61, (E, 1), generator=rng).float())
    gup = torch.randn(E, 128, generator=rng) * rows * torch.exp2(-torch.randint(0, 13, (E, 128), generator=rng).float())
    gup[7] = 0
    _, gm, _ = _block(lib, ctx, w, t, e, W, m.numpy(), gup.numpy(), 1)
    # dm = gup + (gup / 2) W_lin^T / 2 W_ji^T
    g = gup.double()
    want = g + 0.25 * (g @ W_lin.double().t()) @ W_ji.double().t()
    err = (torch.as_tensor(gm).double() - want).norm(dim=1) / want.norm(dim=1).clamp_min(1e-300)
    err[7] = torch.as_tensor(gm)[7].abs().max()
    assert float(err.max()) < 1e-6, err.max()


def test_weight_gradient_columns_of_every_size(lib, ctx):
    # Columns of the activations over 2^16 and rows over 2^20, a column of zeros: with W_ji = 0 the layer's gradient is m^T dz with dz =
    # (gup / 2) W_lin^T / 2 for any m.  A column that is not far below 2^-17 of the largest of its 32 keeps its relative error.
    w = synth.get_workload("cfg2", emb=128, int_emb=64, n_res_before=0, n_res_after=0)
    pos, ref, e, t = _case(lib, ctx, w, 4, synth.slab_adsorbate_positions(1, 2, 2, 3, 4, seed=4))
    E = len(ref["src"])
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    rng = torch.Generator().manual_seed(2)
    W_lin = torch.randn(128, 128, generator=rng)
    W["W_lin"] = W_lin.numpy()
    m = torch.randn(E, 128, generator=rng) * torch.exp2(-torch.randint(0, 17, (1, 128), generator=rng).float())
    m *= torch.exp2(torch.randint(-10, 11, (E, 1), generator=rng).float())
    m[:, 5] = 0
    gup = torch.randn(E, 128, generator=rng)
    _, _, gw = _block(lib, ctx, w, t, e, W, m.numpy(), gup.numpy(), 1)
    want = 0.25 * m.double().t() @ (gup.double() @ W_lin.double().t())
    got = torch.as_tensor(gw["W_ji"]).double()
    err = (got - want).norm(dim=1) / want.norm(dim=1).clamp_min(1e-300)
    err[5] = got[5].abs().max()
    assert float(err.max()) < 1e-6, err.max()
    want_b = 0.25 * (gup.double() @ W_lin.double().t()).sum(0)
    assert H.rel_l2(gw["b_ji"], want_b.numpy()) < 1e-6


def _weight_gradient(lib, ctx, emb, seed, m_scale, gup_scale):
    """W_ji's gradient and m^T dz in 64 bits, column by column of m: with W_ji = 0, dz = (gup / 2) W_lin^T / 2 for any m."""
    w = synth.get_workload("cfg2", emb=emb, int_emb=64, n_res_before=0, n_res_after=0)
    pos, ref, e, t = _case(lib, ctx, w, 4, synth.slab_adsorbate_positions(1, 2, 2, 3, 4, seed=4))
    E = len(ref["src"])
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    rng = torch.Generator().manual_seed(seed)
    W_lin = torch.eye(emb)      # one product per value: dz is gup / 4 to the last bit
    W["W_lin"] = W_lin.numpy()
    m = torch.randn(E, emb, generator=rng) * m_scale(E, emb, rng)
    gup = torch.randn(E, emb, generator=rng) * gup_scale(E, emb, rng)
    _, _, gw = _block(lib, ctx, w, t, e, W, m.numpy(), gup.numpy(), 1)
    want = 0.25 * m.double().t() @ gup.double()
    size = 0.25 * m.double().abs().t() @ gup.double().abs()     # what the terms of a sum add up to
    return torch.as_tensor(gw["W_ji"]).double(), want, size


@pytest.mark.parametrize("emb", [128, 512])      # the two tiles
@pytest.mark.parametrize("far", [24, 32, 40])
def test_weight_gradient_of_a_column_far_below_its_neighbours(lib, ctx, emb, far):
    # Features 2^-far of the size of those next to them: every value has three bf16 parts of its own (24 bits), so a row of the
    # gradient is as exact as any other.  Bound: terms off by 3 2^-24 and 394 additions in fp32, 2^-24 of the running sum each, whose
    # signs are random: 20 2^-24; 2e-6 is some 30 of them.
    def some_small(E, emb, rng):
        return torch.where(torch.arange(emb) % 8 == 5, 2.0 ** -far, 1.0)[None, :]
    got, want, _ = _weight_gradient(lib, ctx, emb, 3, some_small, lambda E, emb, rng: 1.0)
    err = (got - want).norm(dim=1) / want.norm(dim=1)
    assert float(err.max()) < 2e-6, err.max()


def test_weight_gradient_of_rows_of_every_size(lib, ctx):
    # Edges whose messages are 2^-40 to 2^40 of each other's size and whose gradients are as much the other way: all count alike.
    # Bound as above, against the sum of the terms' absolute values.
    rows = torch.exp2(torch.randint(-40, 41, (4096, 1), generator=torch.Generator().manual_seed(6)).float())
    got, want, size = _weight_gradient(lib, ctx, 128, 4, lambda E, emb, rng: rows[:E], lambda E, emb, rng: 1.0 / rows[:E])
    assert float(((got - want).abs() / size).max()) < 2e-6


def test_bilinear_weight_gradients_row_by_row(lib, ctx):
    # The fp32 bilinear block: its Gaussians are 1 to 1e-28 and less of each other's size over the edges of a graph, and the gradients of the
    # weights that meet them lie in rows of such sizes.  The sum over the edges of W_rbfS's and W_c's gradients is exact to fp32 in every
    # row (the block's own rounding, some 1e-6, comes on top: 1e-5).
    from paper_2203_09697_amd.binding_g import StackG
    w = synth.get_workload("cfg3", emb=64, int_emb=32, num_radial=128, dtype="f32")
    pos, gptr = synth.slab_adsorbate_positions(1, 2, 2, 3, 4, seed=4)
    ref = H.oracle_graph(pos, gptr, w.dims.cutoff, w.max_neighbors)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
    W = synth.weights_G(w.dims, seed=5)
    m, gup = synth.edge_embeddings(len(ref["src"]), 64, seed=6)
    basis = lib.gp_basis_forward(ctx, w.dims, e, t)
    st = StackG(ctx, w.dims, [lib.weights_to_device(W)], t, basis)
    st.forward(H.to_dev(m, torch.float32))
    _, gw = st.backward(H.to_dev(gup, torch.float32))
    ob = H.oracle_basis_G(pos, ref, w.dims)
    ob["rbf"] = basis["rbf"].cpu().double()       # the same Gaussians, however small
    want = H.oracle_stack_G(ref, ob, w.dims, [W], m, gup)[2][0]
    for name, rows in (("W_rbfS", (128,)), ("W_c", (w.dims.num_spherical, 128))):
        got, ref_rows = (np.asarray(x, np.float64).reshape(-1, want[name].shape[-1]) for x in (gw[0][name].cpu(), want[name]))
        size = np.linalg.norm(ref_rows, axis=1)
        seen = size > 1e-26                         # below: parts of the values are no normal numbers any more
        err = np.linalg.norm(got - ref_rows, axis=1)[seen] / size[seen]
        print("%s: rows of size %.1e to %.1e, worst %.1e" % (name, size[seen].min(), size.max(), err.max()))
        assert size[seen].min() < 1e-9 * size.max() and err.max() < 1e-5


# (emb, slabs, nx, ny): the three tiles of the products with planes; 272: the last 32 k are half past the end
@pytest.mark.parametrize("emb,slabs,nx,ny", [(128, 1, 2, 2), (272, 1, 2, 2), (192, 12, 4, 3), (512, 16, 5, 4)])
@pytest.mark.parametrize("far", [22, 40])
def test_features_and_weights_far_below_their_neighbours(lib, ctx, emb, slabs, nx, ny, far):
    # Features of a row 2^-far to 2^far of each other's size meet weights that are as much the other way, so that all terms of a sum count
    # alike; a weight of 2^60 meets a feature that is zero.  A value keeps 21 bits at least whatever stands beside it, the dropped products
    # are below 2^-22 of theirs: terms 2^-21 + 2^-21 + 2^-22 off at most, 1.2e-6, mostly a quarter of it, and of random sign; the additions
    # of some 20 partial sums in fp32 add 2^-24 each.  1e-6 of the sum of the terms' sizes: half of the largest sum.
    w = synth.get_workload("cfg2", emb=emb, int_emb=64, n_res_before=0, n_res_after=0)
    pos, gptr = synth.slab_adsorbate_positions(slabs, nx, ny, 3, 4, seed=4)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
    E = e["n_edges"]
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    rng = torch.Generator().manual_seed(far)
    size = torch.exp2(torch.randint(-far, far + 1, (1, emb), generator=rng).float())
    half = emb // 2
    size[:, half:] = 2.0 ** -far        # the columns that are looked at: the gradient that goes past the block is nothing there
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


def test_weights_far_below_their_column(lib, ctx):
    # The forward product (weights [K, N]): in every column one weight of 2^30, which meets a feature that is zero.
    w = synth.get_workload("cfg2", emb=128, int_emb=64, n_res_before=0, n_res_after=0)
    pos, gptr = synth.slab_adsorbate_positions(1, 2, 2, 3, 4, seed=4)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
    E = e["n_edges"]
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    rng = torch.Generator().manual_seed(8)
    W_ji = torch.randn(128, 128, generator=rng)
    W_ji[9] = 2.0 ** 30
    m = torch.randn(E, 128, generator=rng)
    m[:, 9] = 0.0
    W["W_ji"], W["W_lin"] = W_ji.numpy(), torch.eye(128).numpy()
    out, _, _ = _block(lib, ctx, w, t, e, W, m.numpy(), m.numpy(), 1)
    act = lambda v: v * torch.sigmoid(v)
    want = act(act(m.double() @ W_ji.double())) + m.double()
    assert H.rel_l2(out, want.numpy()) < 1e-6


def test_an_infinity_stays_in_its_row(lib, ctx):
    # pairs of atoms by themselves: without triplets no edge sees another
    w = synth.get_workload("cfg2", emb=128, int_emb=64, n_res_before=0, n_res_after=0)
    pos = np.arange(80, dtype=np.float32)[:, None] * np.float32([100.0, 0.0, 0.0])
    pos = np.stack([pos, pos + np.float32([1.5, 0.0, 0.0])], 1).reshape(-1, 3)
    gptr = np.asarray([0, len(pos)], np.int32)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
    E = e["n_edges"]
    W = {k: v * 0 for k, v in synth.weights_D(w.dims, seed=5, bias_scale=0.0).items()}
    rng = torch.Generator().manual_seed(9)
    W["W_ji"], W["W_lin"] = torch.randn(128, 128, generator=rng).numpy(), torch.randn(128, 128, generator=rng).numpy()
    gup = torch.randn(E, 128, generator=rng)
    got = []
    for value in (None, float("inf"), float("nan")):
        g = gup.clone()
        if value is not None:
            g[17, 40] = value
        got.append(torch.as_tensor(_block(lib, ctx, w, t, e, W, torch.zeros(E, 128).numpy(), g.numpy(), 1)[1]))
    keep = torch.arange(E) != 17
    for bad in got[1:]:
        assert not bool(torch.isfinite(bad[17]).any()) and torch.equal(bad[keep], got[0][keep])


@pytest.mark.timeout(300)
@pytest.mark.parametrize("emb,slabs", [(256, 12), (1024, 3)])
def test_bias_gradients_collect_no_rounding_of_one_sign(lib, ctx, emb, slabs):
    # A bias gradient sums a value of every edge: what the products' rounding has in common on all of them adds up, what has none grows
    # as the root of their number.  The fp32 instruction's own sums come out low; the products in two fp16 parts are no further off.
    w = synth.get_workload("cfg2", emb=emb, int_emb=64)
    pos, ref, e, t = _case(lib, ctx, w, 3, synth.slab_adsorbate_positions(slabs, 4, 4, 3, 5, seed=3))
    W = synth.weights_D(w.dims, seed=5, bias_scale=0.1)
    m, gup = synth.edge_embeddings(len(ref["src"]), emb, seed=6)
    want = H.oracle_stack_D(ref, H.oracle_basis_D(pos, ref, w.dims), w.dims, [W], m, gup)[2][0]
    err = {}
    for split in (1, 0):
        got = _block(lib, ctx, w, t, e, W, m, gup, split)[2]
        err[split] = max(H.rel_l2(got[k], want[k]) for k in want if k[0] == "b")
    print("E=%d: two fp16 parts %.2e, fp32 instruction %.2e" % (len(ref["src"]), err[1], err[0]))
    assert err[1] < err[0]


@pytest.mark.parametrize("saved_at,scratch_at", [(8, 0), (0, 8), (8, 8)])
def test_buffers_that_do_not_start_on_16_bytes(lib, ctx, saved_at, scratch_at):
    # saved and scratch may start anywhere: the same results by the kernels that do not need more
    from paper_2203_09697_amd.stack import StackD
    w = synth.get_workload("cfg2", emb=128, int_emb=128)
    pos, gptr = synth.slab_adsorbate_positions(1, 2, 2, 3, 4, seed=4)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
    W = lib.weights_to_device(synth.weights_D(w.dims, seed=5, bias_scale=0.1))
    m, gup = (H.to_dev(x, torch.float32) for x in synth.edge_embeddings(e["n_edges"], 128, seed=6))
    basis = lib.gp_basis_forward(ctx, w.dims, e, t)
    got = []
    for at in ((0, 0), (saved_at, scratch_at)):
        st = StackD(ctx, w.dims, [W], t, basis)
        room = [torch.empty(b.numel() + 8, dtype=torch.uint8, device="cuda:0") for b in (st.saved[0], st.scratch)]
        st.saved[0], st.scratch = room[0][at[0]:at[0] + st.saved[0].numel()], room[1][at[1]:at[1] + st.scratch.numel()]
        assert st.saved[0].data_ptr() % 16 == at[0] and st.scratch.data_ptr() % 16 == at[1]
        out = st.forward(m).cpu().numpy()
        gm, gw = st.backward(gup)
        got.append([out, gm.cpu().numpy()] + [gw[0][k].cpu().numpy() for k in sorted(gw[0])])
    for a, b in zip(*got):
        assert H.rel_l2(b, a) < 5e-6      # fp32 sums in another order, and those of two forms against each other


@pytest.mark.parametrize("emb,many", [(128, 20), (512, 20)])     # 64 x 64 tiles of one slab; 128 x 128 and 128 x 256 of many
def test_values_do_not_depend_on_the_tile(lib, ctx, emb, many):
    # the same slab by itself and as the first of many: other tiles, the same values.  No triplets: their kernels go by the graph.
    from paper_2203_09697_amd.stack import StackD
    w = synth.get_workload("cfg2", emb=emb, int_emb=64)
    one, _ = synth.slab_adsorbate_positions(1, 4, 3, 3, 5, seed=3)
    W = synth.weights_D(w.dims, seed=5, bias_scale=0.1)
    for k in ("W_down", "W_up", "W_sbf1", "W_sbf2"):
        W[k] = W[k] * 0
    W = lib.weights_to_device(W)
    got = []
    for n in (1, many):
        pos, gptr = np.tile(one, (n, 1)), np.arange(n + 1, dtype=np.int32) * len(one)
        e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), w.dims.cutoff, w.max_neighbors)
        E = e["n_edges"] // n
        m, gup = (H.to_dev(np.tile(x, (n, 1)), torch.float32) for x in synth.edge_embeddings(E, emb, seed=6))
        st = StackD(ctx, w.dims, [W], t, lib.gp_basis_forward(ctx, w.dims, e, t))
        out = st.forward(m).cpu()
        got.append((out[:E], st.backward(gup)[0].cpu()[:E]))
        for first in got[-1]:
            assert bool(torch.isfinite(first).all())
    print("E = %d and %d" % (E, E * many))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
