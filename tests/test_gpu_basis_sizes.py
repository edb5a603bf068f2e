"""GPU parity of the per-edge basis kernels at the edges of their launch shapes: few and many edges, remainders, unaligned
and long runs of Gaussian functions."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import synth
from oracle import basis as obasis
from tests import helpers as H

pytestmark = pytest.mark.gpu

# lengths enter as fp32 and the values are rounded to fp32 once: half an ulp of the result
TOL = 6e-8


def _basis(lib, dims, dist):
    n = len(dist)
    ctx = lib.Context(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda:0")
    e = dict(n_edges=n, dist=H.to_dev(dist, torch.float32), unit=torch.zeros((n, 3), device="cuda:0"))
    b = lib.gp_basis_forward(ctx, dims, e, dict(n_triplets=0, idx_kj=none, idx_ji=none))
    torch.cuda.synchronize()
    return b


@pytest.mark.parametrize("n", [1, 3, 5, 16383, 16384, 16400 + 7])
@pytest.mark.parametrize("S,R", [(7, 6), (8, 16), (1, 1)])
def test_bessel_bases(lib, n, S, R):
    rng = np.random.default_rng(n)
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg2").dims), num_spherical=S, num_radial=R))
    dist = rng.uniform(0.05, dims.cutoff, n).astype(np.float32)
    b = _basis(lib, dims, dist)
    d64 = torch.tensor(dist.astype(np.float64))
    rbf = obasis.rbf_bessel(d64, dims.cutoff, R, dims.envelope_p).numpy()
    rad = obasis.sbf_radial(d64, dims.cutoff, S, R, dims.envelope_p).reshape(n, -1).numpy()
    for got, want in ((b["rbf"], rbf), (b["rad"], rad)):
        got = got.cpu().numpy()
        assert np.all(np.abs(got - want) <= TOL * np.abs(want) + 1e-12), np.abs(got - want).max()


@pytest.mark.parametrize("R", [2, 8, 9, 128, 1024])
@pytest.mark.parametrize("n", [1, 257])
def test_gaussian_basis(lib, n, R):
    rng = np.random.default_rng(R)
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg4").dims), num_radial=R))
    dist = rng.uniform(0.05, dims.cutoff, n).astype(np.float32)
    got = _basis(lib, dims, dist)["rbf"].cpu().numpy()
    want = obasis.rbf_gauss(torch.tensor(dist.astype(np.float64)), dims.cutoff, R, dims.envelope_p).numpy()
    assert np.all(np.abs(got - want) <= TOL * np.abs(want) + 1e-38)


@pytest.mark.parametrize("n", [5, 16384 + 3])
@pytest.mark.parametrize("S,R", [(7, 6), (1, 1)])
def test_bessel_bases_one_at_a_time(lib, n, S, R):
    # either output may be left out; the other one is the same to the bit and nothing else is written
    import ctypes as C
    from paper_2203_09697_amd import binding as B
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg2").dims), num_spherical=S, num_radial=R))
    dist = np.random.default_rng(n).uniform(0.05, dims.cutoff, n).astype(np.float32)
    want, d, ctx = _basis(lib, dims, dist), B.Dims(dims), lib.Context(0)
    x = H.to_dev(dist, torch.float32)
    for name in ("rbf", "rad"):
        got = torch.full((want[name].numel() + 64,), -7.0, device="cuda:0")
        ctx.check(lib.load().gp_basis_forward(ctx._h, C.byref(d), B._ptr(x), None, None, None, None, C.c_int64(n), C.c_int64(0),
                                              *(B._ptr(got) if k == name else None for k in ("rbf", "rad")), None, None, None))
        torch.cuda.synchronize()
        assert torch.equal(got[:-64], want[name].reshape(-1)) and bool((got[-64:] == -7.0).all())


@pytest.mark.parametrize("n", [1, 2047, 2048, 16383, 16384, 16400 + 7])   # pairs of atoms: two edges each, no triplets
@pytest.mark.parametrize("S,R", [(1, 1), (1, 7), (1, 8), (2, 5), (7, 6), (8, 16)])   # 2, 14, 16, 15, 48, 144 functions
def test_length_gradients_of_bessel_bases(lib, n, S, R):
    # the chain from the basis gradients to the edge lengths, at the edges of its launch shapes, through the forces of a pair:
    # minus the sum of both edges' derivatives along the bond
    import ctypes as C
    from paper_2203_09697_amd import binding as B
    from paper_2203_09697_amd.binding_e import gp_edges_by_source, gp_forces_from_basis_grad_D
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg2").dims), num_spherical=S, num_radial=R))
    rng = np.random.default_rng(n)
    ctx = lib.Context(0)
    pos = np.zeros((n, 2, 3))
    way = rng.normal(size=(n, 3))
    pos[:, 1] = way / np.linalg.norm(way, axis=1)[:, None] * rng.uniform(0.3, 0.99 * dims.cutoff, (n, 1))
    e, t = lib.build_graph(ctx, H.to_dev(pos.reshape(-1, 3), torch.float32), H.to_dev(2 * np.arange(n + 1), torch.int32), dims.cutoff)
    E = e["n_edges"]
    assert E == 2 * n and t["n_triplets"] == 0
    g_rbf, g_rad = rng.normal(size=(E, R)).astype(np.float32), rng.normal(size=(E, S * R)).astype(np.float32)
    forces, nb = torch.empty((2 * n, 3), device="cuda:0"), C.c_size_t()
    ctx.check(lib.load().gp_forces_workspace(C.c_int64(E), C.c_int64(0), C.byref(nb)))
    gp_forces_from_basis_grad_D(ctx, dims, e, t, *gp_edges_by_source(ctx, e), H.to_dev(g_rbf, torch.float32), H.to_dev(g_rad, torch.float32),
                                torch.empty(1, device="cuda:0"), forces, torch.empty(max(nb.value, 8), dtype=torch.uint8, device="cuda:0"))
    torch.cuda.synchronize()
    d = e["dist"].cpu().double().requires_grad_(True)
    b = (obasis.rbf_bessel(d, dims.cutoff, R, dims.envelope_p) * torch.tensor(g_rbf.astype(np.float64))).sum()
    b = b + (obasis.sbf_radial(d, dims.cutoff, S, R, dims.envelope_p).reshape(E, -1) * torch.tensor(g_rad.astype(np.float64))).sum()
    gd = torch.autograd.grad(b, d)[0].reshape(n, 2)     # the edges of atom 2k come before those of atom 2k + 1
    unit = e["unit"].cpu().double()
    want = -(gd.sum(1)[:, None, None] * unit.reshape(n, 2, 3)).reshape(2 * n, 3)
    # both derivatives are rounded to fp32 once, then a product and a sum: at most 4 half ulps of their size
    room = 2.4e-7 * gd.abs().sum(1).repeat_interleave(2)[:, None] + 1e-12
    assert bool(((forces.cpu().double() - want).abs() <= room).all())
