"""The two tile shapes of the owner-computes H1 kernel (8 x 8 and 16 x 16 cells)
at their edges: cell counts at, just below and just above a multiple of the
16 x 16 tile's stride of 15, on meshes wide enough that it is chosen (49 of its
tiles, ten layers), and one on which the 8 x 8 tile is."""
import numpy as np
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from oracle import lor_oracle as orc
from tests.gpu_helpers import check_whole_matrix, row_rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("nx,ny,nz,p", [
    (105, 105, 10, 1),   # 7 x 7 full tiles
    (104, 91, 10, 1),    # the last tile one cell short; one cell wide
    (21, 20, 2, 5),      # 105 x 100 cells
    (15, 16, 5, 1),      # one wave per tile; one column over
])
def test_tiles_match_the_oracle(nx, ny, nz, p):
    m = meshgen.box_mesh(nx, ny, nz, p, 0.1)
    m, order = meshgen.permute_elements(m, seed=2)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1)
    c = (nx * p // 2) + (nx * p + 1) * (ny * p // 2 + (ny * p + 1) * (nz * p // 2))
    X = m["coords"].copy()
    X[c, 0] += 0.9 * (X[c + 1, 0] - X[c, 0])      # a pinched vertex: cells past the fallback threshold
    rp, ci, v = orc.h1_matrix(X, m["elem_dofs"], p, kap, 0.7)
    ed, x = torch.from_numpy(m["elem_dofs"]).to(DEV), torch.from_numpy(X).to(DEV)
    pat = lor.lor_pattern(lor.LOR_H1, p, ed, m["ndofs"])
    assert pat.owner
    v64 = lor.lor_assemble_h1(pat, ed, x, kap, 0.7)
    counts = []
    for kernel in ("owner", "colored"):
        diag = torch.zeros(2, dtype=torch.int32, device=DEV)
        v32 = lor.lor_assemble_h1(pat, ed, x, kap.float(), 0.7, dtype=torch.float32, fp64_fallback=True, diag=diag,
                                  kernel=kernel)
        counts.append(diag.cpu().tolist())
        assert row_rel_err(rp, ci, v32.cpu(), ci, v) <= 1e-6
        check_whole_matrix(pat, v32)
    assert counts[0] == counts[1] and counts[0][0] > 0
    assert row_rel_err(rp, ci, v64.cpu(), ci, v) <= 1e-12
    check_whole_matrix(pat, v64)
    batch = torch.stack([kap, 2.0 * kap])
    vb = lor.lor_assemble_h1(pat, ed, x, batch, 0.7)
    assert torch.equal(vb[0], v64) or row_rel_err(rp, ci, vb[0].cpu(), ci, v) <= 1e-12
    assert np.isfinite(vb.cpu().numpy()).all()
