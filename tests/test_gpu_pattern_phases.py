"""The two phases of the pattern call: an element map that is not the one phase 1
saw is refused also where its rows have the same lengths, and on a box lattice the
temporaries are back when the call returns."""
import ctypes

import pytest
import torch

import meshgen
from paper_2210_12253_amd import lor as L

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _phases(first, second, p, n):
    """Return codes of phase 1 on one map and phase 2 on another, and the message."""
    lib, s, nnz = L.load_library(), L.LorSched(), ctypes.c_int64(0)
    a, b = torch.from_numpy(first).to(DEV), torch.from_numpy(second).to(DEV)
    rp = torch.empty(n + 1, dtype=torch.int32, device=DEV)
    st = torch.cuda.current_stream().cuda_stream
    args = (L.LOR_H1, p, len(first), n)
    rc1 = lib.lor_pattern(*args, a.data_ptr(), rp.data_ptr(), ctypes.byref(nnz), None, ctypes.byref(s), st)
    ci = torch.empty(nnz.value, dtype=torch.int32, device=DEV)
    buf = torch.empty(s.dev_bytes, dtype=torch.uint8, device=DEV)
    s.dev = buf.data_ptr()
    rc2 = lib.lor_pattern(*args, b.data_ptr(), rp.data_ptr(), ctypes.byref(nnz), ci.data_ptr(), ctypes.byref(s), st)
    return rc1, rc2, lib.lor_last_error().decode()


def test_other_map_is_refused():
    p = 2
    m = meshgen.box_mesh(3, 4, 2, p)
    turned, _, _ = meshgen.reorient_elements(m, seed=5, kappa=meshgen.kappa_field(m["nel"], p, 1.0))
    box, other = m["elem_dofs"], turned["elem_dofs"]     # the same vertices, rows and columns
    for first, second in ((other, box), (box, other)):
        rc1, rc2, msg = _phases(first, second, p, m["ndofs"])
        assert rc1 == L.LOR_OK and rc2 == L.LOR_EINVAL and "phase 1" in msg
    for both in (box, other):
        assert _phases(both, both, p, m["ndofs"])[:2] == (L.LOR_OK, L.LOR_OK)
    moved, _ = meshgen.permute_elements(m, seed=2)       # a lattice with its elements in any order stays one
    assert _phases(box, moved["elem_dofs"], p, m["ndofs"])[:2] == (L.LOR_OK, L.LOR_OK)


def test_lattice_temporaries_are_back_at_return():
    hip = ctypes.CDLL("libamdhip64.so")

    def free():
        a, b = ctypes.c_size_t(), ctypes.c_size_t()
        assert hip.hipMemGetInfo(ctypes.byref(a), ctypes.byref(b)) == 0
        return a.value
    m = meshgen.box_mesh(48, 48, 48, 2)      # about 900,000 vertices: scratch of 10 MB
    ed = torch.from_numpy(m["elem_dofs"]).to(DEV)
    for _ in range(2):                       # torch's own blocks are there from the second time on
        torch.cuda.synchronize()
        before = free()
        pat = L.lor_pattern(L.LOR_H1, 2, ed, m["ndofs"])
        after = free()
        del pat
    assert before - after < 2 << 20          # (what the runtime itself may take)
