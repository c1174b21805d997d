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


def _free_bytes():
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _wide(n_banks):
    """A layer of 1,024 channels (10 MB of weights) and small banks."""
    from types import SimpleNamespace
    import paper_2608_22526_amd as rs3
    rng = np.random.default_rng(0)
    W = [rng.standard_normal((r, 1024), dtype=np.float32) for r in (1024, 256, 256, 1024)]
    layer = rs3.Layer(1024, 4, 256, rs3.RS3_F32, *W)
    return SimpleNamespace(layer=layer, banks=[rs3.Bank(layer, 64, 2, 1) for _ in range(n_banks)])


def test_weights_live_as_long_as_the_last_bank():
    import paper_2608_22526_amd as rs3
    _wide(1)                                    # what the library allocates once
    before = _free_bytes()
    h = _wide(2)
    rs3.lib().rs3_layer_destroy(h.layer.h)
    h.layer.h = None
    g = rs3.Grid(8, 8, 1)
    K, V = (torch.randn((1, 64, 256), device="cuda") for _ in range(2))
    mask, n = torch.ones((1, 8, 8), dtype=torch.uint8, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    for i, b in enumerate(h.banks):             # a commit reads W_k and W_v
        rs3.commit([b], g, K, V, 64 * 256, mask, 0, 0, 0, 64, n)
        torch.cuda.synchronize()
        assert b.error() == 0 and np.array_equal(b.export()["K"].reshape(-1), K.cpu().numpy().reshape(-1))
        assert before - _free_bytes() >= 8 << 20   # the weights are held
        rs3.lib().rs3_bank_destroy(b.h)
        b.h = None
    del K, V, mask, n
    assert before - _free_bytes() < 4 << 20        # and given back with the last bank


def test_handles_given_back_from_several_threads():
    """Layers and banks destroyed in parallel: each layer is freed once."""
    from concurrent.futures import ThreadPoolExecutor
    import paper_2608_22526_amd as rs3
    lib = rs3.lib()
    _wide(1)
    before = _free_bytes()
    with ThreadPoolExecutor(6) as pool:
        for _ in range(20):
            h = _wide(5)
            calls = [(lib.rs3_layer_destroy, h.layer.h)] + [(lib.rs3_bank_destroy, b.h) for b in h.banks]
            for x in [h.layer] + h.banks:
                x.h = None
            list(pool.map(lambda c: c[0](c[1]), calls))
    assert before - _free_bytes() < 12 << 20       # less than one layer of the twenty
