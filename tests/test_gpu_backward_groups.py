"""The backward kernel at p = 1 in groups of 64 elements (meshes just above half of what
they take in one round of the chip, and in FP32 large ones with a small batch)
against the oracle's autograd, and with the same coefficient gradients as in smaller
groups, which the same mesh takes with a larger batch; p = 3 on both sides of the line
between groups of one and of two elements."""
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from oracle import lor_oracle as orc
from tests.test_gpu_backward import DEV, _gpu_grads, _rel, _rowwise, oracle_loss_grads

pytestmark = pytest.mark.gpu


def _terms(m, cot, rp, ci):
    """Per element sum |G_uv| * max |K_uv|, the size of the 64 terms of dL/dkappa: at
    p = 1 this is one number per element, whose own size says nothing about its error
    (the terms have both signs, and of 10^5 elements some cancel to 10^-5)."""
    X = torch.from_numpy(m["coords"])
    sv = orc.h1_subelement_vertices(torch.from_numpy(m["elem_dofs"]), 1).reshape(-1, 8)
    K = orc.h1_subelement_matrices(X[sv], torch.ones(len(sv), dtype=torch.float64), 0.0)
    n = rp.numel() - 1
    key = torch.repeat_interleave(torch.arange(n), rp[1:] - rp[:-1]) * n + ci
    pos = torch.searchsorted(key, (sv[:, :, None] * n + sv[:, None, :]).reshape(-1))
    return cot[0][pos].reshape(-1, 64).abs().sum(1) * K.abs().amax((1, 2))


@pytest.mark.parametrize("n,more", [((33, 33, 33), 5), ((35, 35, 35), 5), ((56, 55, 55), 3)])
def test_groups_of_64(n, more):
    m = meshgen.box_mesh(*n, 1, 0.1)
    kap = meshgen.kappa_field(m["nel"], 1, 1.0, seed=3, batch=more)
    rp, ci, _ = orc.h1_matrix(m["coords"], m["elem_dofs"], 1, kap[0].detach(), 0.7)
    cot = meshgen.cotangent(more, rp[-1].item(), seed=1)
    gk_ref, gx_ref = oracle_loss_grads(m, 1, kap[:1], 0.7, cot[:1], rp, ci)
    size = _terms(m, cot, rp, ci)
    pat = lor.lor_pattern(lor.LOR_H1, 1, torch.from_numpy(m["elem_dofs"]).to(DEV), m["ndofs"])
    # entries of K to 1e-12 and 1e-6 of a row's largest, as everywhere; in FP32 the sum
    # of 64 terms adds up to 64 roundings of 6e-8
    for dt, tol, err, tolx in ((torch.float64, 1e-12, _rowwise, 1e-10), (torch.float32, 5e-6, _rel, 1e-5)):
        gk, gx = _gpu_grads(pat, m, kap[:1], 0.7, cot[:1], dt)
        assert bool(((gk - gk_ref).reshape(-1).abs() <= tol * size).all())
        assert err(gx, gx_ref) <= tolx
        all_gk, _ = _gpu_grads(pat, m, kap, 0.7, cot, dt)
        assert torch.equal(all_gk[:1], gk)


@pytest.mark.parametrize("n", [(32, 6, 4), (769, 1, 1), (11, 11, 11)])     # 768 (at most), 769 and 1,331 elements
def test_groups_at_p3(n):
    m = meshgen.box_mesh(*n, 3, 0.1)
    kap = meshgen.kappa_field(m["nel"], 3, 1.0, seed=3, batch=2)
    rp, ci, _ = orc.h1_matrix(m["coords"], m["elem_dofs"], 3, kap[0].detach(), 0.7)
    cot = meshgen.cotangent(2, rp[-1].item(), seed=1)
    gk_ref, gx_ref = oracle_loss_grads(m, 3, kap, 0.7, cot, rp, ci)
    pat = lor.lor_pattern(lor.LOR_H1, 3, torch.from_numpy(m["elem_dofs"]).to(DEV), m["ndofs"])
    gk, gx = _gpu_grads(pat, m, kap, 0.7, cot, torch.float32)
    assert _rel(gk, gk_ref) <= 1e-5 and _rel(gx, gx_ref) <= 1e-5
