"""Weight gradients of a block that share a launch (gp_gemm_tn_group): the error of the sums alone.  With W_ji = 2^20 I and every other weight
zero, dW_lin = max(m, 0)^T g 2^19 and db_lin = (sum of g) / 2 hold exactly, and no other rounding enters.  Residual layers behind it, without effect
on either, fill the launch with products."""
import numpy as np
import pytest
import torch

import synth
from tests import helpers as H
from tests.test_gpu_no_triplets import _graph, _pairs

pytestmark = pytest.mark.gpu


# The error of one product by itself, in sums of one sign over its runs of 32 to 340 rows, is 1.1, 1.5, 1.7, 2.4, 3.3 and 2.4e-7; sums of 16
# chunks in runs of thousands of rows have 1.2, 1.9, 2.4, 2.6, 2.9 and 2.9e-7.  As they are: 0.9, 1.3, 1.4, 1.9, 2.0 and 1.6e-7.
@pytest.mark.parametrize("emb,pairs,bound", [(256, 217, 1.3e-7), (256, 750, 1.6e-7), (256, 3797, 1.8e-7), (256, 11365, 2.1e-7), (256, 21690, 2.1e-7), (64, 21690, 2.1e-7)])
def test_sums_over_the_edges(lib, emb, pairs, bound):
    from paper_2203_09697_amd.stack import StackD
    ctx = lib.Context(0)
    w = synth.get_workload("cfg2", emb=emb, int_emb=64, n_res_before=0, n_res_after=4)
    pos, gptr = _pairs(pairs, pairs)
    ref, e, t = _graph(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)
    E, err_W, err_b = e["n_edges"], 0.0, 0.0
    W = {k: torch.zeros_like(v) for k, v in lib.weights_to_device(synth.weights_D(w.dims, seed=5)).items()}
    W["W_ji"] = torch.eye(emb, device="cuda:0") * 2.0 ** 20
    st = StackD(ctx, w.dims, [W], t, lib.gp_basis_forward(ctx, w.dims, e, t))
    for seed in range(3):
        rng = np.random.default_rng(seed)
        # max(m, 0) is 1/32 or more where it is not zero: silu(2^20 m) is then 2^20 m to the last bit, and 0 for the others
        m = (np.sign(rng.standard_normal((E, emb))) * rng.uniform(1.0 / 32.0, 1.0, (E, emb))).astype(np.float32)
        g = rng.standard_normal((E, emb)).astype(np.float32)
        st.forward(H.to_dev(m, torch.float32))
        _, gw = st.backward(H.to_dev(g, torch.float32))
        want = np.maximum(m, 0).astype(np.float64).T @ g.astype(np.float64) * 2.0 ** 19
        err_W += H.rel_l2(gw[0]["W_lin"].cpu().numpy(), want) / 3
        err_b += H.rel_l2(gw[0]["b_lin"].cpu().numpy(), g.astype(np.float64).sum(0) / 2) / 3
    print("E %d W %.2e b %.2e" % (E, err_W, err_b))
    assert err_W < bound
    # columns of zero mean: fp32 sums of eight values and of each run's result, 6e-8; summed in fp32 throughout 0.9e-7 to 1.4e-7
    assert err_b < 7.5e-8
