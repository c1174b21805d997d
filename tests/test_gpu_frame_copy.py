"""Out-of-place frames: the copy of the token grid that rides in the energy
launch (or beside the query projection) against separate in-place calls on a
copy made here, bit for bit."""
from dataclasses import replace

import numpy as np
import pytest

from test_gpu_edge import SMALL, _dev, _host, _session
from workloads import make_weights, to_storage

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,n,C,n_obj,shared,dtype,rope", [
    (24, 20, 64, 1, True, "bf16", False),     # short last energy block
    (24, 20, 64, 3, True, "bf16", True),      # one grid to three objects (rotary: projection launch)
    (40, 40, 64, 6, True, "bf16", False),     # more outputs than one copy work-group writes, short last group
    (33, 31, 128, 64, True, "bf16", True),
    (64, 64, 64, 16, False, "bf16", False),   # the wide energy form, a grid each
    (100, 41, 72, 64, False, "f32", False),   # wide form, short last column slice and row block
    (70, 9, 256, 2, False, "bf16", False),    # mask rows beside, a grid each
])
def test_out_of_place_frame(m, n, C, n_obj, shared, dtype, rope):
    cfg = replace(SMALL, m=m, n=n, C=C, H=1, d_h=C, n_obj=n_obj, shared_x=shared, union_objects=n_obj == 1,
                  dtype=dtype, cap_frames=2, f_max=3)
    W = make_weights(cfg)
    rng = np.random.default_rng(m * n + C)
    n_x = 1 if shared else n_obj

    def tokens(*shape):
        return _dev(to_storage(rng.standard_normal(shape).astype(np.float32), dtype))

    X = tokens(n_x, cfg.mn, C)
    K, V = tokens(n_obj, cfg.mn, cfg.d_kv), tokens(n_obj, cfg.mn, cfg.d_kv)
    masks = _dev((rng.random((n_obj, m, n)) < 0.1).astype(np.uint8))
    k = [max(1, cfg.mn // 5)] * (1 if cfg.union_objects else n_obj)
    outs = []
    for way in ("frame", "separate", "readout"):
        sess = _session(cfg, W, rope_theta=50.0 if rope else None)
        sess.commit(K, V, masks, 0, True)
        Y = torch.full((n_obj, cfg.mn, C), 3.0, dtype=X.dtype, device="cuda")
        if way == "frame":
            sess.frame(masks, X, k, Y, K, V, masks, 1)
        else:
            sess.select(masks, X, k)
            if way == "readout":
                sess.readout(X, Y)
            elif n_obj == 1 or not shared:      # in place on a copy
                Y.copy_(X)
                sess.readout(Y, Y)
            else:                               # one object at a time, in place
                Y.copy_(X.expand_as(Y))
                import paper_2608_22526_amd as rs3
                ws = torch.zeros(rs3.readout_workspace_size(sess.layer, 1, cfg.mn), dtype=torch.uint8, device="cuda")
                S = 0
                for o in range(n_obj):
                    rs3.readout(sess.layer, sess.grid, 1, Y[o], 0, [sess.banks[o]], sess.sel_idx[o], sess.sel_count[o:],
                                0, cfg.mn, S, Y[o], 0, 0, ws)
        torch.cuda.synchronize()
        assert all(b.error() == 0 for b in sess.banks)
        outs.append((_host(Y), _host(sess.sel_idx), _host(sess.sel_count)))
    sel, cnt = outs[0][1], outs[0][2]
    for y, s, c in outs[1:]:
        assert np.array_equal(c, cnt)
        for o in range(n_obj):
            g = 0 if cfg.union_objects else o
            rows = sel[g][:cnt[g]]
            assert np.array_equal(s[g][:cnt[g]], rows)
            rest = np.setdiff1d(np.arange(cfg.mn), rows)
            xo = _host(X)[0 if shared else o]
            for a in (outs[0][0][o], y[o]):
                assert np.array_equal(a[rest].view(np.uint8), xo[rest].view(np.uint8))
            a, b = outs[0][0][o][rows], y[o][rows]
            if n_obj == 1 or not shared or y is outs[2][0]:
                assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
            else:   # other key splits: the same rows up to rounding
                f = [(v.astype(np.uint32) << 16).view(np.float32) for v in (a, b)]
                assert np.abs(f[0] - f[1]).max() <= 4e-2
