"""A batch large enough that the default kernel of a general mesh is another one than
for one of its entries alone (coloured instead of row by row): every entry against
the oracle, and the same bits in a batch and alone where the kernel is named."""
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from oracle import lor_oracle as orc
from tests.gpu_helpers import check_whole_matrix, row_rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("space,p,n,layers,batch,cells_per_color", [
    ("h1", 6, 2, 4, 16, 26000), ("nd", 3, 3, 3, 30, 8500), ("rt", 4, 3, 3, 20, 35000)])
def test_batch_across_the_line(space, p, n, layers, batch, cells_per_color):
    m = meshgen.tri_split_mesh(n, layers, p, 0.1)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1)
    scale = [1.0 + 0.25 * b for b in range(batch)]
    ed, x = torch.from_numpy(m["elem_dofs"]).to(DEV), torch.from_numpy(m["coords"]).to(DEV)
    if space == "h1":
        pat = lor.lor_pattern(lor.LOR_H1, p, ed, m["ndofs"])
        ref = lambda k: orc.h1_matrix(m["coords"], m["elem_dofs"], p, k, 0.7)
        call = lambda k, **kw: lor.lor_assemble_h1(pat, ed, x, k, 0.7, dtype=k.dtype, **kw)
    else:
        make = meshgen.edge_map_from_vertices if space == "nd" else meshgen.face_map_from_vertices
        dm, nrows = make(m["elem_dofs"], p)
        dmap = torch.from_numpy(dm).to(DEV)
        pat = lor.lor_pattern(lor.LOR_ND if space == "nd" else lor.LOR_RT, p, dmap, nrows)
        f, g = (orc.nd_matrix, lor.lor_assemble_nd) if space == "nd" else (orc.rt_matrix, lor.lor_assemble_rt)
        ref = lambda k: f(m["coords"], m["elem_dofs"], dm, p, k, 0.7, nrows)
        call = lambda k, **kw: g(pat, ed, dmap, x, k, 0.7, m["ndofs"], dtype=k.dtype, **kw)
    cells, line = m["nel"] * p ** 3, cells_per_color * pat.ncolors
    assert not pat.owner and cells <= line < cells * batch
    for dt, tol in ((torch.float64, 1e-12), (torch.float32, 1e-6)):
        k = torch.stack([s * kap for s in scale]).to(dt)
        vb, colored = call(k), call(k, kernel="colored")
        for b in (0, batch - 1):
            rp, ci, v = ref(scale[b] * kap)
            assert row_rel_err(rp, ci, call(k[b]).cpu(), ci, v) <= tol
            assert row_rel_err(rp, ci, vb[b].cpu(), ci, v) <= tol
            assert torch.equal(call(k[b], kernel="colored"), colored[b])
        check_whole_matrix(pat, vb, colored)
