"""Scratch of the Hadamard block and of the output block, by the calls that return it (host functions; no GPU is used)."""
from types import SimpleNamespace

import pytest

from paper_2203_09697_amd.binding import gp_block_workspace
from paper_2203_09697_amd.binding_o import gp_output_workspace


def _dims(emb, before, after):
    return SimpleNamespace(variant="D", dtype="f32", emb=emb, int_emb=64, num_radial=6, num_spherical=7, cutoff=6.0, envelope_p=5, basis_emb=8,
                           emb_rbf=0, emb_cbf=0, emb_bil=0, n_res_before=before, n_res_after=after, radial_at_target=False, symmetric=False)


@pytest.mark.parametrize("emb", [32, 64, 192, 256, 384, 512, 2048])
@pytest.mark.parametrize("before,after", [(0, 0), (1, 2), (4, 4)])
def test_block_scratch(emb, before, after):
    d = _dims(emb, before, after)
    # on both sides of the size where the gradients of all layers no longer have a buffer each, and far beyond
    turn = 2 ** 31 // (4 * emb * max(2 * (before + after) + 2, 1))
    sizes = [0, 1, 1000, 40000, turn - 1, turn, turn + 1, 2 * turn, 10 ** 7, 4 * 10 ** 7]
    got = {E: gp_block_workspace(d, E, 14 * E)[1] for E in sorted(sizes)}
    sizes = sorted(got)
    assert all(got[a] <= got[b] for a, b in zip(sizes, sizes[1:]))
    for E in sizes:
        # seven arrays over edges and columns, the narrow ones; 2 GiB in all for what groups of weight gradients add, and partial sums and weights
        rows = 4 * E * (7 * emb + 2 * 64 + 7 * 8 + 7 * 64)
        assert got[E] <= rows + 2 ** 31 + 2 ** 29, (E, got[E] - rows)


def test_output_scratch():
    narrow, wide = (gp_output_workspace(256, 256, R, 3, 1000, 10 ** 6)[1] for R in (16, 17))
    assert narrow < 10 ** 8 and wide > 4 * 256 * 10 ** 6   # an array over edges and columns only where the gate is a product
