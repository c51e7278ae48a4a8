"""What the entry points that spread a chain over workgroups refuse."""
from __future__ import annotations

import ctypes


def test_refusals():
    import paper_1006_2566_amd as hsg
    from paper_1006_2566_amd import batch as hb
    hb._bind()
    lib = hsg.lib()
    assert lib.hsg_batch_parts(258) == 0 == lib.hsg_batch_parts(0)
    d = hb._Batch(1, 0, 1, 1, 1, 1, 1, 1, None, 1, 256, 0)
    assert lib.hsg_batch_init_parts(ctypes.byref(d), 258, 1, None) == -1
    assert lib.hsg_batch_init_parts(ctypes.byref(d), 8, None, None) == -1
    assert lib.hsg_batch_overlap_parts(ctypes.byref(d), 1, 65536, 8, 1, 1, None) == -1
    assert lib.hsg_batch_overlap_parts(ctypes.byref(d), 1, 1, 8, None, 1, None) == -1
