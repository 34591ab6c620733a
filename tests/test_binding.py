"""The ctypes binding without a GPU: what it hands back to a caller."""
import numpy as np
import pytest


class _Lib:
    """Stands in for libhs.so: 1000 cells, fields of increasing numbers."""

    def hs_num_cells(self, h, c):
        return 1000

    def hs_sample_moments(self, h, c, mode, n, u, T, q, ns):
        k = 0
        for p, m in ((n, 1000), (u, 3000), (T, 1000), (q, 3000)):
            np.ctypeslib.as_array(p, (m,))[:] = np.arange(k, k + m)
            k += m
        return 0


@pytest.mark.parametrize("mode", [0, 1])
def test_fields_are_independent_arrays(mode):
    """Each field owns its memory: keeping one does not keep the others'."""
    from paper_2506_23917_amd.hs import Sim
    sim = Sim.__new__(Sim)
    sim.L, sim.h = _Lib(), None
    out = sim.sample_moments(0, mode)
    k = 0
    for f, shape in (("n", (1000,)), ("u", (1000, 3)), ("T", (1000,)), ("q", (1000, 3))):
        a = out[f]
        assert a.shape == shape and a.dtype == np.float64 and a.flags.c_contiguous
        assert a.flags.owndata and a.base is None
        assert np.array_equal(a.ravel(), np.arange(k, k + a.size))
        k += a.size
