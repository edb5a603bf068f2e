"""The edges' passes of the output block with few radial functions (kernels of their own up to 16, products above): both sizes of the kernels
and the first count without one, features that end inside a wavefront's 64, atoms without edges, runs of edges that end early."""
import numpy as np
import pytest
import torch

import synth
from tests import helpers as H
from tests.test_gpu_output import _oracle_out

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 8, 9, 16, 17])
@pytest.mark.parametrize("emb,edges", [(40, 1), (65, 33), (256, 1030), (64, 33000)])   # 33000: runs of more than 32
def test_output_block(lib, R, emb, edges):
    from paper_2203_09697_amd import binding_o as O
    ctx, rng, N, L = lib.Context(0), np.random.default_rng(R + emb), 37, 2
    dst = np.sort(rng.choice(np.setdiff1d(np.arange(N), [0, 5, 36]), edges))
    row_ptr, gptr = np.searchsorted(dst, np.arange(N + 1)), np.array([0, 20, N])
    m, rbf = rng.standard_normal((edges, emb)).astype(np.float32), rng.standard_normal((edges, R)).astype(np.float32)
    coef = rng.standard_normal(2).astype(np.float32)
    W = synth.weights_out(emb, 48, R, L, seed=3, bias_scale=0.2)
    want_E, want_gm, want_W = _oracle_out(m, rbf, dst, gptr, N, W, coef)
    Wd = lib.weights_to_device(W)
    gW = {k: torch.empty_like(v) for k, v in Wd.items()}
    sb, cb = O.gp_output_workspace(emb, 48, R, L, N, edges)
    saved, scratch = (torch.empty(max(b, 8), dtype=torch.uint8, device="cuda:0") for b in (sb, cb))
    dm, drbf, dptr = H.to_dev(m, torch.float32), H.to_dev(rbf, torch.float32), H.to_dev(gptr, torch.int32)
    energy, gm = torch.empty(2, device="cuda:0"), torch.empty_like(dm)
    O.gp_output_forward(ctx, Wd, dm, drbf, H.to_dev(row_ptr, torch.int32), dptr, False, energy, saved, scratch)
    back = lambda acc, out, w: O.gp_output_backward(ctx, Wd, dm, drbf, H.to_dev(dst, torch.int32), dptr, N, H.to_dev(coef, torch.float32), saved, acc, out, w, scratch)
    back(False, gm, gW)
    base = torch.randn_like(gm)
    twice = base.clone()
    back(True, twice, None)
    torch.cuda.synchronize()
    # sums of at most 33000 products in fp32 by runs of a few dozen, and five small products of 1e-7 each
    err = {"energy": H.rel_l2(energy.cpu().numpy(), want_E), "grad_m": H.rel_l2(gm.cpu().numpy(), want_gm)}
    err.update({k: H.rel_l2(gW[k].cpu().numpy(), g) for k, g in want_W.items()})
    print({k: "%.1e" % v for k, v in err.items()})
    assert max(err.values()) < 3e-6
    # on top of another gradient the sum is rounded once, to half an ulp of it (6e-8); norms, as above: triangle inequality
    want = base.cpu().numpy().astype(np.float64) + want_gm
    assert np.linalg.norm(twice.cpu().numpy() - want) <= 6e-8 * np.linalg.norm(want) + 3e-6 * np.linalg.norm(want_gm)


@pytest.mark.parametrize("R", [1, 6, 12, 16])
def test_the_gate_of_the_backward_pass_is_rounded_once(lib, R):
    """No layers, W_up = I, w_final = 1 and dL/dE = 1: grad_m is the gate itself, one rounding to fp32 (at most 6e-8, 2e-8 to 3e-8 in the norm); a sum
    of 6 to 16 products in fp32 is 4e-8 to 7e-8 off."""
    from paper_2203_09697_amd import binding_o as O
    ctx, rng, N, emb, edges = lib.Context(0), np.random.default_rng(R), 50, 64, 5000
    dst = np.sort(rng.integers(0, N, edges))
    row_ptr, gptr = np.searchsorted(dst, np.arange(N + 1)), np.array([0, N])
    m, rbf = rng.standard_normal((edges, emb)).astype(np.float32), rng.standard_normal((edges, R)).astype(np.float32)
    W = dict(synth.weights_out(emb, emb, R, 0, seed=3), W_up=np.eye(emb, dtype=np.float32), w_final=np.ones(emb, np.float32))
    Wd = lib.weights_to_device(W)
    sb, cb = O.gp_output_workspace(emb, emb, R, 0, N, edges)
    saved, scratch = (torch.empty(max(b, 8), dtype=torch.uint8, device="cuda:0") for b in (sb, cb))
    dm, drbf, dptr = H.to_dev(m, torch.float32), H.to_dev(rbf, torch.float32), H.to_dev(gptr, torch.int32)
    gm = torch.empty_like(dm)
    O.gp_output_forward(ctx, Wd, dm, drbf, H.to_dev(row_ptr, torch.int32), dptr, False, torch.empty(1, device="cuda:0"), saved, scratch)
    O.gp_output_backward(ctx, Wd, dm, drbf, H.to_dev(dst, torch.int32), dptr, N, torch.ones(1, device="cuda:0"), saved, False, gm, None, scratch)
    err = H.rel_l2(gm.cpu().numpy(), rbf.astype(np.float64) @ W["W_rbf"].astype(np.float64))
    print("R %d %.2e" % (R, err))
    assert err < 3.2e-8


@pytest.mark.parametrize("R", [6, 12, 16])
def test_the_gate_of_the_forward_pass_is_rounded_once(lib, R):
    """One edge an atom, an atom a structure, no layers, W_up = I and one value in w_final: the energy is m times the gate, two roundings to fp32 of 2e-8
    to 3e-8 each, 4e-8 together; with a gate summed in fp32 5e-8 (6 functions) to 8e-8 (16)."""
    from paper_2203_09697_amd import binding_o as O
    ctx, rng, N, emb = lib.Context(0), np.random.default_rng(R), 4000, 64
    m, rbf = rng.standard_normal((N, emb)).astype(np.float32), rng.standard_normal((N, R)).astype(np.float32)
    W = dict(synth.weights_out(emb, emb, R, 0, seed=3), W_up=np.eye(emb, dtype=np.float32), w_final=np.eye(emb, dtype=np.float32)[5])
    saved, scratch = (torch.empty(max(b, 8), dtype=torch.uint8, device="cuda:0") for b in O.gp_output_workspace(emb, emb, R, 0, N, N))
    energy, ptr = torch.empty(N, device="cuda:0"), H.to_dev(np.arange(N + 1), torch.int32)
    O.gp_output_forward(ctx, lib.weights_to_device(W), H.to_dev(m, torch.float32), H.to_dev(rbf, torch.float32), ptr, ptr, False, energy, saved, scratch)
    err = H.rel_l2(energy.cpu().numpy(), m[:, 5].astype(np.float64) * (rbf.astype(np.float64) @ W["W_rbf"][:, 5].astype(np.float64)))
    print("R %d %.2e" % (R, err))
    assert err < 4.5e-8
