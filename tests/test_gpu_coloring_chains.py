"""Meshes numbered along their length, whose greedy colouring is one long chain of
dependencies: a launch of the colouring ends with elements that still wait for
uncoloured neighbours, and the next launches take them (one channel of elements
for H(curl) and H(div), a narrow 2D strip, a long irregular extrusion for H1)."""
import time

import numpy as np
import pytest
import torch

import meshgen
from tests.test_gpu_coloring import DEV, _greedy, lor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("space", ["nd", "rt", "2d", "h1"])
def test_long_chain(space):
    if space == "nd":
        sp, (em, n) = lor.LOR_ND, meshgen.nd_edge_map_box(60000, 1, 1, 1)
    elif space == "rt":
        sp, (em, n) = lor.LOR_RT, meshgen.face_map_box(60000, 1, 1, 1)
    else:
        sp = lor.LOR_H1_2D if space == "2d" else lor.LOR_H1
        m = meshgen.box_mesh_2d(4, 15000, 1) if space == "2d" else meshgen.tri_split_mesh(1, 12000, 1)
        em, n = m["elem_dofs"], m["ndofs"]
    pat = lor.lor_pattern(sp, 1, torch.from_numpy(em).to(DEV), n)
    s = pat.sched
    raw = pat.sched_dev[s.off_color:s.off_color + 4 * len(em)].cpu().numpy()
    ref = _greedy(em)
    assert np.array_equal(np.frombuffer(raw.tobytes(), dtype=np.int32), ref)
    assert pat.ncolors == ref.max() + 1


def test_time_grows_with_the_chain():
    """Waves that cannot finish leave early instead of each waiting its full time:
    a chain 6.7 times as long takes 6.7 times as long (24 times if they all wait)."""
    def seconds(nel):
        em, n = meshgen.nd_edge_map_box(nel, 1, 1, 1)
        em = torch.from_numpy(em).to(DEV)
        best = float("inf")
        for _ in range(3):
            torch.cuda.synchronize()
            t = time.perf_counter()
            lor.lor_pattern(lor.LOR_ND, 1, em, n)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best
    assert seconds(400000) < 12 * seconds(60000)
