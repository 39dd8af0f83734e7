"""The discrete curl's choice of a face's element (the lowest that names it):
faces named by many elements and by none, names out of range, and a scratch
array that already holds anything, against the oracle's first incidence."""
import numpy as np
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from oracle import lor_oracle as orc

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6])
def test_any_face_map(p, dtype):
    n = 3
    ee, ned = meshgen.nd_edge_map(n, p)
    fm, nf = meshgen.face_map(n, p)
    ee, _ = meshgen.flip_edge_signs(ee, ned, seed=p)
    fm, _ = meshgen.flip_edge_signs(fm, nf, seed=p + 1)
    ids = np.where(fm < 0, -1 - fm, fm)
    keep = np.unique(ids)
    rng = np.random.default_rng(p)
    # a few faces named all over the mesh; the faces that this leaves without a name drop out of the oracle's
    many = rng.random(ids.shape) < 0.2
    ids = np.where(many, rng.integers(0, 5, ids.shape), ids)
    fm2 = np.where(fm < 0, -1 - ids, ids).astype(np.int32)
    named, dense = np.unique(ids, return_inverse=True)
    dense = dense.reshape(ids.shape)
    rp, ci, v = orc.discrete_curl(ee, np.where(fm < 0, -1 - dense, dense), p, len(named))
    extra = 4                                      # named by no element
    none = np.setdiff1d(np.arange(nf + extra), named)
    assert len(keep) == nf and len(none) >= extra
    want_c = np.zeros((nf + extra, 4), np.int64)
    want_v = np.zeros((nf + extra, 4))
    want_c[named], want_v[named] = ci.numpy().reshape(-1, 4), v.numpy().reshape(-1, 4)
    total = fm2.size
    scratch = [torch.full((nf + extra,), x, dtype=torch.int32) for x in (0, -1, 2 ** 31 - 1, -2 ** 31, total, total - 1)]
    scratch.append(torch.from_numpy(rng.integers(0, total, nf + extra).astype(np.int32)))
    for w in scratch:
        diag = torch.zeros(2, dtype=torch.int32, device=DEV)
        grp, gci, gv = lor.lor_discrete_curl(p, ee, fm2, ned, nf + extra, dtype=dtype, diag=diag, workspace=w.to(DEV),
                                             device=DEV)
        assert torch.equal(grp.cpu().long(), torch.arange(0, 4 * (nf + extra) + 1, 4))
        assert torch.equal(gci.cpu().long(), torch.from_numpy(want_c).reshape(-1))
        assert torch.equal(gv.cpu(), torch.from_numpy(want_v).reshape(-1).to(dtype))
        assert diag.cpu().tolist() == [len(none), 0]
    # a name out of range is counted and left out
    bad = fm2.copy()
    bad[-1, -1] = nf + extra
    diag = torch.zeros(2, dtype=torch.int32, device=DEV)
    lor.lor_discrete_curl(p, ee, bad, ned, nf + extra, dtype=dtype, diag=diag, device=DEV)
    assert diag.cpu().tolist()[1] == 1
