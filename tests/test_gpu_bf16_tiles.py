"""bf16 products of the bilinear block at the row counts where the tile of the global->LDS kernel changes: the bf16 block against
the fp32 block of the same inputs (which the other tests hold against the oracle)."""
from dataclasses import replace

import pytest
import torch

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

# emb, emb_trip, slabs, nx, ny, symmetric -> rows; wide tiles / narrow tiles
SHAPES = [
    (256, 64, 9, 4, 3, False),     # 8 to 16 thousand rows: 128x128 / 64x64
    (512, 64, 10, 4, 3, True),     # ... of 512 columns: 128x256 in one round / 64x64
    (320, 64, 15, 4, 4, False),    # 16 to 32 thousand rows, N no multiple of the tile: 256x256 / 128x64
    (1024, 128, 15, 4, 4, False),  # a last round of tiles mostly empty: 128x128 / 128x128
]


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("emb,trip,slabs,nx,ny,symmetric", SHAPES, ids=["%d_%d_%d" % s[:3] for s in SHAPES])
def test_bf16_block_near_fp32_block(lib, ctx, emb, trip, slabs, nx, ny, symmetric):
    _near_fp32(lib, ctx, slabs, nx, ny, dict(emb=emb, int_emb=trip, symmetric=symmetric))


@pytest.mark.parametrize("num_radial,num_spherical,emb_cbf", [(8, 3, 5), (40, 7, 16), (136, 8, 16), (128, 7, 16)])
def test_radial_table_widths(lib, ctx, num_radial, num_spherical, emb_cbf):
    # contractions that end inside a step of 16 and inside the second pass of 128, 15 to 128 rows of the table
    _near_fp32(lib, ctx, 1, 2, 2, dict(emb=64, int_emb=32, num_radial=num_radial, num_spherical=num_spherical, emb_cbf=emb_cbf))


def _near_fp32(lib, ctx, slabs, nx, ny, widths):
    from paper_2203_09697_amd.binding_g import StackG
    w = synth.get_workload("cfg3", **widths)
    dims, emb = w.dims, widths["emb"]
    pos, gptr = synth.slab_adsorbate_positions(slabs, nx, ny, 3, 5, seed=3)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), dims.cutoff, w.max_neighbors)
    basis = lib.gp_basis_forward(ctx, dims, e, t)
    W = synth.weights_G(dims, seed=5)
    m, gup = synth.edge_embeddings(e["n_edges"], emb, seed=6)
    res = {}
    for dtype in ("bf16", "f32"):
        st = StackG(ctx, replace(dims, dtype=dtype), [lib.weights_to_device(W)], t, basis)
        out = st.forward(H.to_dev(m, torch.float32)).cpu().numpy()
        gm, gw = st.backward(H.to_dev(gup, torch.float32))
        res[dtype] = dict({k: v.cpu().numpy() for k, v in gw[0].items()}, out=out, grad_m=gm.cpu().numpy())
    print("E = %d" % e["n_edges"])
    for k, ref in res["f32"].items():      # bf16 operands, fp32 sums: 4e-3 to 9e-3 of the norm, a row 4 times that
        assert H.rel_l2(res["bf16"][k], ref) < 2e-2, k
    for k in ("out", "grad_m"):
        assert H.row_err(res["bf16"][k], res["f32"][k]) < 8e-2, k
