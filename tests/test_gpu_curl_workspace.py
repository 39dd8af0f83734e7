"""What the discrete curl leaves in its workspace: the first incidence of every face,
INT32_MAX for a face that no element names, whatever was there before."""
import numpy as np
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("p", [1, 3])
def test_first_incidences(p):
    ee, ned = meshgen.nd_edge_map(2, p)
    fm, nf = meshgen.face_map(2, p)
    n = nf + 5
    ids = np.where(fm < 0, -1 - fm, fm).reshape(-1)
    want = np.full(n, 2 ** 31 - 1, dtype=np.int32)
    np.minimum.at(want, ids, np.arange(ids.size, dtype=np.int32))
    for before in (0, 7, -1, ids.size, 2 ** 31 - 1):
        w = torch.full((n,), before, dtype=torch.int32, device=DEV)
        lor.lor_discrete_curl(p, ee, fm, ned, n, workspace=w, device=DEV)
        assert np.array_equal(w.cpu().numpy(), want)
    w = torch.zeros(4, dtype=torch.int32, device=DEV)       # no element at all
    none = np.zeros((0, fm.shape[1]), np.int32), np.zeros((0, ee.shape[1]), np.int32)
    lor.lor_discrete_curl(p, none[1], none[0], 1, 4, workspace=w, device=DEV)
    assert w.cpu().tolist() == [2 ** 31 - 1] * 4
