"""Bases and cosines of a Hadamard graph in one launch (few triplets) against the general path over index arrays: both sizes of either
half of the launch, edges that end inside a workgroup's share, and graphs without a triplet."""
from types import SimpleNamespace

import pytest
import torch

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


# (atoms, atoms per A^3, cutoff): 16 and 64 lanes per edge change over at 128 triplets per edge, 4 and 32 edges a workgroup at 12288 edges
@pytest.mark.parametrize("n,density,cutoff,long_lists,many", [(2, 0.5, 5.0, False, False), (67, 0.1, 4.0, False, False),
                                                             (700, 0.1, 4.6, False, True), (131, 0.5, 20.0, True, True),
                                                             (111, 0.5, 30.0, False, False), (112, 0.5, 30.0, False, True)])
def test_one_launch_equals_the_general_path(lib, n, density, cutoff, long_lists, many):
    ctx = lib.Context(0)
    pos, gptr = synth.cube_positions(n, (n / density) ** (1 / 3), 0.3, seed=n)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), cutoff, 0)
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg2").dims), cutoff=cutoff))
    E, T = e["n_edges"], t["n_triplets"]
    assert T < 4 * 1000 * 1000 and (T >= 128 * E) == long_lists and (E >= 12288) == many
    one = lib.gp_basis_forward(ctx, dims, e, t)
    general = lib.gp_basis_forward(ctx, dims, e, {k: v for k, v in t.items() if k != "id_swap"})   # without the lists by centre atom
    torch.cuda.synchronize()
    for k in ("rbf", "rad"):
        assert torch.equal(one[k], general[k]), k
    if T == 0:
        return
    # three products and two sums of numbers below one in fp32, in either order of the sums: within 5 half ulps of one each
    u, kj, ji = e["unit"].double(), t["idx_kj"].long(), t["idx_ji"].long()
    want = -(u[ji] * u[kj]).sum(1).clamp(-1, 1)
    for b in (one, general):
        assert (b["cos_alpha"].double() - want).abs().max() < 3e-7
        assert torch.equal(b["cos_alpha_kj"], b["cos_alpha"][t["perm_kj"].long()])


@pytest.mark.parametrize("n,cutoff", [(300, 10.0), (360, 11.0)])   # long lists, some 7 and 11 million triplets
def test_one_launch_of_many_triplets_equals_the_general_path(lib, n, cutoff):
    ctx = lib.Context(0)
    pos, gptr = synth.cube_positions(n, (n / 0.08) ** (1 / 3), 0.3, seed=n)
    e, t = lib.build_graph(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), cutoff, 0)
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg2").dims), cutoff=cutoff))
    assert 4 * 1000 * 1000 < t["n_triplets"] < 16 * 1000 * 1000 and t["n_triplets"] >= 128 * e["n_edges"]
    one = lib.gp_basis_forward(ctx, dims, e, t)
    general = lib.gp_basis_forward(ctx, dims, e, {k: v for k, v in t.items() if k != "id_swap"})
    for k in ("rbf", "rad"):
        assert torch.equal(one[k], general[k]), k
    # as above
    u, kj, ji = e["unit"].double(), t["idx_kj"].long(), t["idx_ji"].long()
    want = -(u[ji] * u[kj]).sum(1).clamp(-1, 1)
    for b in (one, general):
        assert (b["cos_alpha"].double() - want).abs().max() < 3e-7
        assert torch.equal(b["cos_alpha_kj"], b["cos_alpha"][t["perm_kj"].long()])
