"""Bytes of the build's workspace: the buffers that only graphs of more than two
node types use are sized for those alone."""
import ctypes as C
import os

import pytest

from paper_2608_02168_amd import api


@pytest.mark.skipif(not os.path.exists(api.LIB_PATH), reason="libhg.so not built")
def test_build_workspace_follows_the_node_types():
    n, e = 1_000_000, 20_000_000
    fake = C.c_void_p(0x1000)  # sizes only: never dereferenced

    def size(n_ntype):
        g = api.GraphDesc(n, e, 4, n_ntype, fake, fake, fake, fake, fake, 0, None, None, 0, 0)
        o = api.OverlapDesc(n // 10, 0, 0, api.HG_THETA_NONE, 0, 1, None)
        return api.lib().hg_build_csr_workspace_size(C.byref(g), C.byref(o))

    assert size(1) == size(2) and size(3) == size(4)
    # 14 bytes a node and a word per edge for more than two types, a bit per edge for two
    saved = 14 * n + 4 * e - e // 8
    assert abs((size(3) - size(2)) - saved) < 0.02 * saved
