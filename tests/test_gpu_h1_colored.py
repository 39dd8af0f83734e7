"""The coloured H1 kernel with more elements of a colour than its workgroups take
in one group: several groups per workgroup, a ragged last group, and (p = 1)
more elements per workgroup than it has lanes."""
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from oracle import lor_oracle as orc
from tests.gpu_helpers import check_whole_matrix, row_rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("p,n,layers", [(1, 45, 40), (2, 13, 11), (3, 9, 7), (4, 9, 10), (5, 8, 9), (6, 6, 7)])
def test_many_groups_match_the_oracle(p, n, layers):
    m = meshgen.tri_split_mesh(n, layers, p, 0.1)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1)
    rp, ci, v = orc.h1_matrix(m["coords"], m["elem_dofs"], p, kap, 0.7)
    ed, x = torch.from_numpy(m["elem_dofs"]).to(DEV), torch.from_numpy(m["coords"]).to(DEV)
    pat = lor.lor_pattern(lor.LOR_H1, p, ed, m["ndofs"])
    assert not pat.owner
    v64 = lor.lor_assemble_h1(pat, ed, x, kap, 0.7)
    assert row_rel_err(rp, ci, v64.cpu(), ci, v) <= 1e-12
    v32 = lor.lor_assemble_h1(pat, ed, x, kap.float(), 0.7, dtype=torch.float32)
    assert row_rel_err(rp, ci, v32.cpu(), ci, v) <= 1e-6
    check_whole_matrix(pat, v64, v32)


def test_more_elements_per_workgroup_than_lanes():
    """p = 1 on a box large enough for more than 64 elements per workgroup of 64 lanes."""
    m = meshgen.box_mesh(160, 160, 128, 1, 0.1)
    kap = meshgen.kappa_field(m["nel"], 1, 1.0, seed=1)
    ed, x = torch.from_numpy(m["elem_dofs"]).to(DEV), torch.from_numpy(m["coords"]).to(DEV)
    pat = lor.lor_pattern(lor.LOR_H1, 1, ed, m["ndofs"])
    a = lor.lor_assemble_h1(pat, ed, x, kap, 0.7, kernel="colored")
    b = lor.lor_assemble_h1(pat, ed, x, kap, 0.7, kernel="owner")
    rows = torch.repeat_interleave(torch.arange(pat.nrows, device=DEV),
                                   (pat.row_ptr[1:] - pat.row_ptr[:-1]).long())
    den = torch.zeros(pat.nrows, dtype=torch.float64, device=DEV).scatter_reduce(0, rows, b.abs(), "amax")
    num = torch.zeros(pat.nrows, dtype=torch.float64, device=DEV).scatter_reduce(0, rows, (a - b).abs(), "amax")
    assert float((num / den).max()) <= 1e-12
