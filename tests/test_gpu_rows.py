"""The row-by-row kernels (small meshes that are no lattice) against the oracle
and the coloured kernels: every degree, vertices of 1 to 12 elements (more than
the lanes of a row), renumbered vertices, rotated elements, batches, row counts
that do not fill a workgroup, and the FP32 fallback counters."""
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from oracle import lor_oracle as orc
from tests.gpu_helpers import check_whole_matrix, row_rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _mesh(kind, p):
    if kind == "prism5":
        m = meshgen.prism_mesh(p, 5, 2, 0.1)
    elif kind == "tri":
        m = meshgen.tri_split_mesh(2, 3, p, 0.1)
    else:
        m = meshgen.box_mesh(3, 2, 2, p, 0.1)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1)
    if kind == "renumbered":
        m, _ = meshgen.renumber_vertices(m, seed=3)
    if kind == "rotated":
        m, kap, _ = meshgen.reorient_elements(m, seed=5, kappa=kap)
    return m, kap


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("kind", ["prism5", "tri", "renumbered", "rotated"])
def test_h1_rows(kind, p):
    m, kap = _mesh(kind, p)
    X = m["coords"].copy()
    ed, x = torch.from_numpy(m["elem_dofs"]).to(DEV), torch.from_numpy(X).to(DEV)
    pat = lor.lor_pattern(lor.LOR_H1, p, ed, m["ndofs"])
    assert not pat.owner
    rp, ci, v = orc.h1_matrix(X, m["elem_dofs"], p, kap, 0.7)
    v64 = lor.lor_assemble_h1(pat, ed, x, kap, 0.7)
    assert row_rel_err(rp, ci, v64.cpu(), ci, v) <= 1e-12
    v32 = lor.lor_assemble_h1(pat, ed, x, kap.float(), 0.7, dtype=torch.float32)
    assert row_rel_err(rp, ci, v32.cpu(), ci, v) <= 1e-6
    check_whole_matrix(pat, v64, v32)
    vb = lor.lor_assemble_h1(pat, ed, x, torch.stack([kap, 0.5 * kap, kap]), 0.7)
    assert torch.equal(vb[0], v64) and torch.equal(vb[2], v64)
    counts = []
    for kernel in ("auto", "colored"):     # a threshold that about half of the curved cells pass
        diag = torch.zeros(2, dtype=torch.int32, device=DEV)
        lor.lor_assemble_h1(pat, ed, x, kap.float(), 0.7, dtype=torch.float32, fp64_fallback=True,
                            det_ratio_thresh=1.02, diag=diag, kernel=kernel)
        counts.append(diag.cpu().tolist())
    assert counts[0] == counts[1]


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("space", ["nd", "rt"])
@pytest.mark.parametrize("kind", ["prism5", "tri", "rotated"])
def test_vector_rows(kind, space, p):
    m, kap = _mesh(kind, p)
    make = meshgen.edge_map_from_vertices if space == "nd" else meshgen.face_map_from_vertices
    dm, n = make(m["elem_dofs"], p)
    dm, _ = meshgen.flip_edge_signs(dm, n, seed=7)
    ed, x, dmap = (torch.from_numpy(a).to(DEV) for a in (m["elem_dofs"], m["coords"], dm))
    pat = lor.lor_pattern(lor.LOR_ND if space == "nd" else lor.LOR_RT, p, dmap, n)
    assert not pat.owner
    assert pat.sched.max_row_nnz == int((pat.row_ptr[1:] - pat.row_ptr[:-1]).max())
    ref = orc.nd_matrix if space == "nd" else orc.rt_matrix
    call = lor.lor_assemble_nd if space == "nd" else lor.lor_assemble_rt
    rp, ci, v = ref(m["coords"], m["elem_dofs"], dm, p, kap, 0.7, n)
    v64 = call(pat, ed, dmap, x, kap, 0.7, m["ndofs"])
    assert row_rel_err(rp, ci, v64.cpu(), ci, v) <= 1e-12
    v32 = call(pat, ed, dmap, x, kap.float(), 0.7, m["ndofs"], dtype=torch.float32)
    assert row_rel_err(rp, ci, v32.cpu(), ci, v) <= 1e-6
    check_whole_matrix(pat, v64, v32)
    vb = call(pat, ed, dmap, x, torch.stack([kap, 0.5 * kap]), 0.7, m["ndofs"])
    assert torch.equal(vb[0], v64)
    counts = []
    for kernel in ("auto", "colored"):
        diag = torch.zeros(2, dtype=torch.int32, device=DEV)
        call(pat, ed, dmap, x, kap.float(), 0.7, m["ndofs"], dtype=torch.float32, fp64_fallback=True,
             det_ratio_thresh=1.02, diag=diag, kernel=kernel)
        counts.append(diag.cpu().tolist())
    assert counts[0] == counts[1]
