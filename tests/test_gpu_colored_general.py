"""The coloured kernels by name on meshes that are no lattice (9 to 12 colours, vertices
of 3 to 12 elements, rotated elements), where the default takes the row-by-row
kernels while a mesh is small: values against the oracle in both types, batches
against single calls, with several elements per workgroup and ragged last groups."""
import pytest
import torch

import meshgen
import paper_2210_12253_amd as lor
from oracle import lor_oracle as orc
from tests.gpu_helpers import check_whole_matrix, row_rel_err
from tests.test_gpu_rows import DEV, _mesh

pytestmark = pytest.mark.gpu


def _check(m, kap, p, space):
    ed, x = torch.from_numpy(m["elem_dofs"]).to(DEV), torch.from_numpy(m["coords"]).to(DEV)
    if space == "h1":
        pat = lor.lor_pattern(lor.LOR_H1, p, ed, m["ndofs"])
        rp, ci, v = orc.h1_matrix(m["coords"], m["elem_dofs"], p, kap, 0.7)
        call = lambda k, **kw: lor.lor_assemble_h1(pat, ed, x, k, 0.7, dtype=k.dtype, kernel="colored", **kw)
    else:
        make = meshgen.edge_map_from_vertices if space == "nd" else meshgen.face_map_from_vertices
        dm, n = make(m["elem_dofs"], p)
        dm, _ = meshgen.flip_edge_signs(dm, n, seed=7)
        dmap = torch.from_numpy(dm).to(DEV)
        pat = lor.lor_pattern(lor.LOR_ND if space == "nd" else lor.LOR_RT, p, dmap, n)
        ref, asm = (orc.nd_matrix, lor.lor_assemble_nd) if space == "nd" else (orc.rt_matrix, lor.lor_assemble_rt)
        rp, ci, v = ref(m["coords"], m["elem_dofs"], dm, p, kap, 0.7, n)
        call = lambda k, **kw: asm(pat, ed, dmap, x, k, 0.7, m["ndofs"], dtype=k.dtype, kernel="colored", **kw)
    assert not pat.owner
    v64 = call(kap)
    assert row_rel_err(rp, ci, v64.cpu(), ci, v) <= 1e-12
    k32 = kap.float()
    v32 = call(k32)
    assert row_rel_err(rp, ci, v32.cpu(), ci, v) <= 1e-6
    # a threshold that about half of the curved cells pass: those in FP64
    f32 = call(k32, fp64_fallback=True, det_ratio_thresh=1.02)
    assert row_rel_err(rp, ci, f32.cpu(), ci, v) <= 1e-6
    check_whole_matrix(pat, v64, v32, f32)
    for k, one in ((kap, v64), (k32, v32)):
        vb = call(torch.stack([k, 0.5 * k, k]))
        assert torch.equal(vb[0], one) and torch.equal(vb[2], one)


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("space", ["h1", "nd", "rt"])
@pytest.mark.parametrize("kind", ["prism5", "tri", "rotated"])
def test_small(kind, space, p):
    if space == "nd" and p == 6:
        return   # H(curl) of degree 6 is assembled on edge lattices only
    m, kap = _mesh(kind, p)
    _check(m, kap, p, space)


@pytest.mark.parametrize("space,p,n,layers", [
    ("h1", 1, 20, 9), ("h1", 2, 13, 11), ("h1", 3, 9, 7), ("h1", 4, 6, 5), ("h1", 5, 4, 5), ("h1", 6, 3, 4),
    ("nd", 1, 9, 10), ("nd", 2, 5, 7), ("nd", 3, 4, 5), ("nd", 4, 3, 3), ("nd", 5, 2, 3),
    ("rt", 1, 9, 10), ("rt", 2, 6, 7), ("rt", 3, 5, 5), ("rt", 4, 3, 4), ("rt", 5, 3, 2), ("rt", 6, 2, 3)])
def test_many_elements(space, p, n, layers):
    m = meshgen.tri_split_mesh(n, layers, p, 0.1)
    _check(m, meshgen.kappa_field(m["nel"], p, 1.0, seed=1), p, space)


@pytest.mark.parametrize("p,n,layers", [(2, 28, 22), (3, 16, 17), (4, 16, 17), (5, 12, 15), (6, 9, 13)])
def test_h1_several_groups_per_workgroup(p, n, layers):
    """More elements of a colour than the resident workgroups take in one group (2,048
    of four elements at p = 2, of one at p = 3 and 4; 1,024 at p = 5, 512 at p = 6), against
    the generic comparator, which goes through the explicit refined mesh."""
    m = meshgen.tri_split_mesh(n, layers, p, 0.1)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1).to(DEV)
    ed, x = torch.from_numpy(m["elem_dofs"]).to(DEV), torch.from_numpy(m["coords"]).to(DEV)
    pat = lor.lor_pattern(lor.LOR_H1, p, ed, m["ndofs"])
    resident = {2: 8192, 3: 2048, 4: 2048, 5: 1024, 6: 512}[p]
    ptr = list(pat.sched.color_ptr)[:pat.ncolors + 1]
    assert max(b - a for a, b in zip(ptr, ptr[1:])) > resident
    ref = lor.lor_assemble_h1_unstructured(pat, lor.lor_refine_map(p, ed), x, kap, 0.7)
    rows = torch.repeat_interleave(torch.arange(pat.nrows, device=DEV), (pat.row_ptr[1:] - pat.row_ptr[:-1]).long())
    largest = torch.zeros(pat.nrows, dtype=torch.float64, device=DEV).scatter_reduce(0, rows, ref.abs(), "amax")
    for dt, tol in ((torch.float64, 1e-12), (torch.float32, 1e-6)):
        v = lor.lor_assemble_h1(pat, ed, x, kap.to(dt), 0.7, dtype=dt, kernel="colored")
        assert float(((v.double() - ref).abs() / largest[rows]).max()) <= tol


@pytest.mark.parametrize("space,p,n,layers", [("nd", 4, 9, 9), ("nd", 5, 8, 9), ("rt", 5, 14, 10), ("rt", 6, 10, 8)])
def test_vector_several_groups_per_workgroup(space, p, n, layers):
    """The same for H(curl) and H(div) (256 to 1,024 resident workgroups): random rows
    against the oracle, and symmetry."""
    m = meshgen.tri_split_mesh(n, layers, p, 0.1)
    kap = meshgen.kappa_field(m["nel"], p, 1.0, seed=1)
    dm, nrows = (meshgen.edge_map_from_vertices if space == "nd" else meshgen.face_map_from_vertices)(m["elem_dofs"], p)
    dm, _ = meshgen.flip_edge_signs(dm, nrows, seed=7)
    ed, x, dmap = (torch.from_numpy(a).to(DEV) for a in (m["elem_dofs"], m["coords"], dm))
    pat = lor.lor_pattern(lor.LOR_ND if space == "nd" else lor.LOR_RT, p, dmap, nrows)
    ptr = list(pat.sched.color_ptr)[:pat.ncolors + 1]
    assert max(b - a for a, b in zip(ptr, ptr[1:])) > {"nd": 256, "rt": 1024 if p == 5 else 512}[space]
    pick = torch.randperm(nrows, generator=torch.Generator().manual_seed(p))[:300].sort().values
    rows, rp, ci, v = (orc.nd_rows if space == "nd" else orc.rt_rows)(m["coords"], m["elem_dofs"], dm, p, kap, 0.7, pick)
    asm = lor.lor_assemble_nd if space == "nd" else lor.lor_assemble_rt
    full_rp = pat.row_ptr.cpu().long()
    at = torch.cat([torch.arange(int(full_rp[r]), int(full_rp[r + 1])) for r in rows.tolist()])
    for dt, tol in ((torch.float64, 1e-12), (torch.float32, 1e-6)):
        got = asm(pat, ed, dmap, x, kap.to(dt), 0.7, m["ndofs"], dtype=dt, kernel="colored")
        assert row_rel_err(rp, pat.col_idx.cpu()[at], got.cpu()[at], ci, v) <= tol
        check_whole_matrix(pat, got)
