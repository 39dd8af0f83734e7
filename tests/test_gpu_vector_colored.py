"""The coloured H(curl) and H(div) kernels where a workgroup walks several groups
of elements (more elements per colour than the resident workgroups take, with a
remainder in the last group and the last workgroup), against the owner-computes
kernels on the same box, and batches against single calls."""
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from tests.gpu_helpers import row_rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# about 1.1 times 8 colours x the elements resident at once
@pytest.mark.parametrize("p,n", [(1, (61, 61, 60)), (2, (33, 33, 33)), (3, (21, 21, 21)), (4, (13, 13, 14)),
                                 (5, (13, 13, 13)), (3, (3, 1, 2)), (4, (1, 1, 1)), (5, (2, 1, 1))])
def test_groups(p, n):
    m = meshgen.box_mesh(*n, p, 0.1)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1)
    dm, nedges = meshgen.nd_edge_map_box(*n, p)
    dm, _ = meshgen.flip_edge_signs(dm, nedges, seed=7)
    ed, x, ee = (torch.from_numpy(a).to(DEV) for a in (m["elem_dofs"], m["coords"], dm))
    pat = lor.lor_pattern(lor.LOR_ND, p, ee, nedges)
    assert pat.owner
    rp, ci = pat.row_ptr.cpu().numpy(), pat.col_idx.cpu().numpy()
    own = lor.lor_assemble_nd(pat, ed, ee, x, kap, 0.7, m["ndofs"])
    col = lor.lor_assemble_nd(pat, ed, ee, x, kap, 0.7, m["ndofs"], kernel="colored")
    assert row_rel_err(rp, ci, col.cpu(), ci, own.cpu().numpy()) <= 1e-12
    c32 = lor.lor_assemble_nd(pat, ed, ee, x, kap.float(), 0.7, m["ndofs"], dtype=torch.float32, kernel="colored")
    assert row_rel_err(rp, ci, c32.cpu(), ci, own.cpu().numpy()) <= 1e-6
    vb = lor.lor_assemble_nd(pat, ed, ee, x, torch.stack([kap, 0.5 * kap]), 0.7, m["ndofs"], kernel="colored")
    assert torch.equal(vb[0], col)


def test_rt_groups():
    """H(div) at p = 6, one element per workgroup of eight waves: about 600
    elements per colour on 512 resident workgroups."""
    n, p = (11, 11, 10), 6
    m = meshgen.box_mesh(*n, p, 0.1)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1)
    fm, nfaces = meshgen.face_map_box(*n, p)
    fm, _ = meshgen.flip_edge_signs(fm, nfaces, seed=7)
    ed, x, ff = (torch.from_numpy(a).to(DEV) for a in (m["elem_dofs"], m["coords"], fm))
    pat = lor.lor_pattern(lor.LOR_RT, p, ff, nfaces)
    assert pat.owner
    rp, ci = pat.row_ptr.cpu().numpy(), pat.col_idx.cpu().numpy()
    own = lor.lor_assemble_rt(pat, ed, ff, x, kap, 0.7, m["ndofs"])
    col = lor.lor_assemble_rt(pat, ed, ff, x, kap, 0.7, m["ndofs"], kernel="colored")
    assert row_rel_err(rp, ci, col.cpu(), ci, own.cpu().numpy()) <= 1e-12
    c32 = lor.lor_assemble_rt(pat, ed, ff, x, kap.float(), 0.7, m["ndofs"], dtype=torch.float32, kernel="colored")
    assert row_rel_err(rp, ci, c32.cpu(), ci, own.cpu().numpy()) <= 1e-6
