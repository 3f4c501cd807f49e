"""Parity of single kernels and of the branches of their dispatch, at the sizes where they can go wrong: edges of
tiles, remainders, the smallest and the largest of their ranges.  Workspaces start as NaN patterns, so a kernel that
reads what no kernel of its own call wrote shows."""
import numpy as np
import pytest
import torch

import csat_inputs as gen
import paper_2507_02957_amd as csat
from oracle import csat_oracle as orc
from tests.gpu_harness import DEV, TOL, DeviceProblem, assert_close, to_dev, to_np
from tests.test_gpu_parity import _mu, _small, _support_check, options  # noqa: F401  (options: fixture)

pytestmark = pytest.mark.gpu


def _problem(w, Q, K, V, Phi):
    p = DeviceProblem(w, Q, K, V, Phi)
    p.ws.fill_(0xFF)
    return p


@pytest.mark.parametrize("iters", [0, 3])
@pytest.mark.parametrize("d", [64, 128])
def test_separate_matrices_read_only_what_the_call_wrote(d, iters):
    """V~ for a separate value matrix needs V transposed in this call, also where the synthesis reads V as it is."""
    w = _small("kv_fresh", B=1, H=2, n_q=70, n=200, d=d, m=48, dtype="bf16", iters=iters)
    Q, K, V = gen.make_qkv(w)
    PhiV = gen.make_workload_phi(w)
    PhiK = gen.quantize(gen.make_phi("rademacher", w.m, w.n, seed=7), w.dtype)
    mu = _mu(PhiV)
    ref = orc.forward(Q, K, V, PhiV, w.lam, mu, iters, Phi_K=PhiK)
    p = _problem(w, Q, K, V, PhiV)
    C, Z = p.empty(p.BH, w.n_q, w.d), p.empty(p.BH, w.n_q, w.d)
    csat.csat_forward_kv(p.dims, p.Q, p.K, p.V, to_dev(PhiK, w.dtype), p.Phi, w.lam, mu, iters, C, Z, None, p.ws)
    torch.cuda.synchronize()
    assert_close("Z", to_np(Z), ref["Z"], TOL[w.dtype])
    assert_close("C", to_np(C), ref["C"] if iters else ref["Z"], TOL[w.dtype])
