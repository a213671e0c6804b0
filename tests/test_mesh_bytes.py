"""Device memory of a mesh (host only): a buffer that held these meshes before
several steps shared a launch holds them still."""
import ctypes as C

import numpy as np
import pytest

from paper_2208_12795_amd import etpic as E
from paper_2208_12795_amd import synth


@pytest.mark.parametrize("cells,most", [((1, 1, 1), 8_064), ((5, 5, 5), 644_736), ((10, 12, 14), 8_587_776)])
def test_mesh_buffer_has_not_grown(cells, most):
    xyz, tv = synth.kuhn_mesh(cells, (1.0, 1.0, 1.0), 0.1, np.random.default_rng(20))
    xyz, tv = np.ascontiguousarray(xyz), np.ascontiguousarray(tv, np.int32)
    cnt, b = np.zeros(4, np.int64), C.c_size_t(0)
    ptr = lambda a, t: a.ctypes.data_as(C.POINTER(t))
    assert E.lib().etpic_mesh_sizes(xyz.shape[0], ptr(xyz, C.c_double), tv.shape[0], ptr(tv, C.c_int32),
                                    ptr(cnt, C.c_int64), C.byref(b)) == E.OK
    assert b.value <= most
