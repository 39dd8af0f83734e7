"""The element colouring of the general pattern path is the sequential greedy
colouring in element order, for chains inside one wave, across waves and across
workgroups, and with more representatives than lanes per element (H(curl))."""
import numpy as np
import pytest
import torch

import meshgen

pytestmark = pytest.mark.gpu
lor = pytest.importorskip("paper_2210_12253_amd")
DEV = "cuda:0"


def _greedy(m):
    """Sequential greedy colours of a signed or unsigned element map [nel, nloc]."""
    ids = np.where(m < 0, -1 - m, m)
    used = [0] * (int(ids.max()) + 1)      # colours around each dof, as a bit mask
    out = np.empty(len(ids), dtype=np.int32)
    for e, row in enumerate(ids):
        mask = 0
        for g in row:
            mask |= used[g]
        c = 0
        while mask >> c & 1:
            c += 1
        out[e] = c
        for g in row:
            used[g] |= 1 << c
    return out


@pytest.mark.parametrize("space,mesh", [
    ("h1", "one"), ("h1", "prism"), ("h1", "tri_small"), ("h1", "tri_large"), ("h1", "tri_permuted"),
    ("nd", "prism"), ("nd", "tri_small"), ("nd", "box"), ("rt", "tri_small"), ("2d", "tri2d")])
def test_colours_are_sequential_greedy(space, mesh):
    p = 2
    if mesh == "one":
        m = meshgen.tri_split_mesh(1, 1, p)
        m["elem_dofs"] = np.unique(m["elem_dofs"][:1], return_inverse=True)[1].reshape(1, -1).astype(np.int32)
        m["elem_dofs"] = m["elem_dofs"][:, ::-1].copy()    # not a box lattice: the general path
    elif mesh == "prism":
        m = meshgen.prism_mesh(p, 5, 3)
    elif mesh == "box":
        m = meshgen.box_mesh(7, 5, 6, p)
    elif mesh == "tri2d":
        m = meshgen.tri_split_mesh_2d(9, p)
    else:
        m = meshgen.tri_split_mesh(3, 2, p) if mesh == "tri_small" else meshgen.tri_split_mesh(7, 9, p)
        if mesh == "tri_permuted":
            m, _ = meshgen.permute_elements(m, 3)
    em, n = m["elem_dofs"], int(m["elem_dofs"].max()) + 1
    if space == "nd":
        em, n = meshgen.edge_map_from_vertices(em, p)
    elif space == "rt":
        em, n = meshgen.face_map_from_vertices(em, p)
    sp = {"h1": lor.LOR_H1, "nd": lor.LOR_ND, "rt": lor.LOR_RT, "2d": lor.LOR_H1_2D}[space]
    pat = lor.lor_pattern(sp, p, torch.from_numpy(em).to(DEV), n)
    s = pat.sched
    raw = pat.sched_dev[s.off_color:s.off_color + 4 * len(em)].cpu().numpy()
    ref = _greedy(em)
    assert np.array_equal(np.frombuffer(raw.tobytes(), dtype=np.int32), ref)
    assert pat.ncolors == ref.max() + 1


def test_refused_under_capture():
    """The pattern calls read counts back: on a stream under capture they fail
    before they queue anything, and work as before afterwards."""
    m = meshgen.tri_split_mesh(2, 3, 2, 0.1)
    ed = torch.from_numpy(m["elem_dofs"]).to(DEV)
    want = lor.lor_pattern(lor.LOR_H1, 2, ed, m["ndofs"])
    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        g.capture_begin()
        try:
            with pytest.raises(lor.LorError):
                lor.lor_pattern(lor.LOR_H1, 2, ed, m["ndofs"])
        finally:
            g.capture_end()
    torch.cuda.synchronize()
    again = lor.lor_pattern(lor.LOR_H1, 2, ed, m["ndofs"])
    assert torch.equal(want.row_ptr, again.row_ptr) and torch.equal(want.col_idx, again.col_idx)
