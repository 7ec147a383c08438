"""The worklist of the h iteration starts empty whatever the solve before left:
a launch that fails between the listing and the end of a solve leaves its
length behind, and entries appended after it would run past the list."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_1905_03344_amd import inputs

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _workspace_pointer(sim, field):
    """Address of a pointer member of the bound workspace (the members before
    it are all pointers)."""
    from paper_1905_03344_amd import ffi
    with open(os.path.join(ROOT, "paper_1905_03344_amd", "csrc", "sph_internal.h")) as f:
        body = re.search(r"struct Workspace \{(.*?)\n\};", f.read(), re.S).group(1)
    body = re.sub(r"//[^\n]*", "", body)
    k = 0
    for decl in body.split(";"):
        for name in re.findall(r"\*+\s*(\w+)", decl):
            if name == field:
                layout = ffi.lib()._Z10sph_layoutPK10sph_paramsPvP9Workspace
                layout.restype = ctypes.c_size_t
                out = (ctypes.c_void_p * 128)()
                base = (sim.ws.data_ptr() + 255) & ~255
                layout(ctypes.byref(sim.params), ctypes.c_void_p(base), out)
                return out[k]
            k += 1
    raise KeyError(field)


@pytest.mark.parametrize("n_side", [17, 47])
def test_stale_worklist_length(n_side):
    import torch
    from paper_1905_03344_amd.state import Simulation
    ic = inputs.square_patch(n_side, 3)
    sim = Simulation(ic, extra_per_particle=256)
    sim.evaluate()
    sim.sync()
    h, nc, rows = sim.numpy("h").copy(), sim.numpy("nc").copy(), sim.nl_idx.clone()
    at = _workspace_pointer(sim, "wl_count") - sim.ws.data_ptr()
    assert 0 <= at < sim.ws_bytes
    # a solve at the kept h lists no particle; the length of one that broke off
    # (its entries are particles: they are what the solve above listed)
    sim.ws[at:at + 8].view(torch.int64).fill_(64)
    sim.find_neighbors()
    _, st = sim.sync()
    assert st.h_counts == ic.n
    np.testing.assert_array_equal(sim.numpy("h"), h)
    np.testing.assert_array_equal(sim.numpy("nc"), nc)
    valid = torch.arange(sim.params.list_stride, device=sim.device) < sim.field("nc")[:, None]
    a, b = (r.view(sim.stride, -1)[:ic.n][valid] for r in (rows, sim.nl_idx))
    assert torch.equal(a, b)
