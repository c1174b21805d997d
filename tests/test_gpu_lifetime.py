"""Handles given back in either order: a garbage collector may finalise a layer
before the banks created from it (both unreachable in one cycle), and a bank
counts itself out of its layer when it is destroyed."""
import gc
import weakref
from dataclasses import replace

import numpy as np
import pytest

from test_gpu_edge import SMALL, _session
from workloads import make_weights

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_layer_destroyed_before_its_banks():
    import paper_2608_22526_amd as rs3
    cfg = replace(SMALL, n_obj=3, union_objects=False)
    sess = _session(cfg, make_weights(cfg))
    layer, banks = sess.layer, sess.banks
    rs3.lib().rs3_layer_destroy(layer.h)
    layer.h = None
    assert banks[0].info()["n_keys"] == 0      # its banks' memory is still there
    for b in banks:
        rs3.lib().rs3_bank_destroy(b.h)
        b.h = None


def test_session_is_freed_without_the_collector():
    cfg = SMALL
    gc.disable()
    try:
        sess = _session(cfg, make_weights(cfg))
        gone = weakref.ref(sess)
        del sess
        assert gone() is None
    finally:
        gc.enable()
