"""fp32 readout and commit against the oracle."""
from dataclasses import replace

import numpy as np
import pytest

from harness import OraclePipeline, compare_bank, max_abs
from test_gpu_edge import _dev, _host, _session
from workloads import CONFIGS, make_weights

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# fp32 sums of the sizes here stay within this of the oracle (the repository's
# tolerance for fp32 outputs)
TOL = 1e-4


def _commit(sess, orc, rng, mask, t, pin):
    cfg = orc.cfg
    K, V = (rng.standard_normal((cfg.n_obj, cfg.mn, cfg.d_kv)).astype(np.float32) for _ in range(2))
    masks = np.broadcast_to(mask, (cfg.n_obj, cfg.m, cfg.n)).astype(np.uint8)
    sess.commit(_dev(K), _dev(V), _dev(masks), t, pin)
    orc.commit(K, V, masks, t, pin)


def _first(cfg, count):
    m = np.zeros(cfg.mn, np.uint8)
    m[:count] = 1
    return m.reshape(cfg.m, cfg.n)


def _read(sess, orc, rng, k):
    cfg = orc.cfg
    X = rng.standard_normal((1, cfg.mn, cfg.C)).astype(np.float32)
    full = np.ones((cfg.n_obj, cfg.m, cfg.n), np.uint8)
    Xd = _dev(X)
    sess.select(_dev(full), Xd, [k] * sess.n_groups)
    sel, _ = orc.select(full, X, [k] * sess.n_groups)
    Y = torch.zeros((cfg.n_obj, cfg.mn, cfg.C), device="cuda")
    sess.readout(Xd, Y)
    torch.cuda.synchronize()
    Yh = _host(Y)
    for o in range(cfg.n_obj):
        rows = sel[0 if cfg.union_objects else o]
        assert max_abs(Yh[o][rows], orc.readout_rows(X, o, rows)) <= TOL
        rest = np.setdiff1d(np.arange(cfg.mn), rows)
        assert np.array_equal(Yh[o][rest].view(np.uint32), X[0][rest].view(np.uint32))


@pytest.mark.parametrize("kept", [31, 32, 33, 40, 63])
def test_stale_rows_of_a_partly_resident_tile(kept):
    """A tile whose resident rows end past its 32nd key, with rows of an
    evicted frame behind them: the stale rows take no part."""
    cfg = replace(CONFIGS["tiny_f32"], f_max=2, n_pin=1, cap_frames=1)
    W = make_weights(cfg, logit_scale=3.0)
    sess, orc = _session(cfg, W), OraclePipeline(cfg, W)
    rng = np.random.default_rng(kept)
    _commit(sess, orc, rng, _first(cfg, 0), 0, True)
    _commit(sess, orc, rng, _first(cfg, 128), 1, False)
    _commit(sess, orc, rng, _first(cfg, kept), 2, False)   # evicts frame 1, whose rows stay behind
    compare_bank(sess.banks[0].export(), orc.banks[0])
    _read(sess, orc, rng, 20)


@pytest.mark.parametrize("H,d_h,d_kv,n_obj,absorb,rope,k,kept", [
    (1, 32, 16, 1, False, False, 33, (70, 90, 10)),     # a second query tile of one row, partial tiles
    (4, 64, 64, 2, False, True, 64, (256, 256, 256)),   # rotary, several heads and objects
    (2, 128, 80, 1, False, False, 1, (1, 64, 65)),      # one query, contraction of ten units
    (1, 256, 256, 1, False, False, 100, (130, 0, 31)),  # widest head, an empty frame
    (1, 64, 64, 1, True, False, 40, (33, 95, 200)),     # the attention on the raw rows
    (3, 16, 48, 1, False, False, 20, (50, 60, 70)),     # a head width the tiled form does not know
])
def test_tiled_readout_and_commit(H, d_h, d_kv, n_obj, absorb, rope, k, kept):
    """The matrix-core form against the oracle, and bit for bit the same rows
    from rs3_frame as from the separate calls."""
    C = 64 if absorb else H * d_h
    cfg = replace(CONFIGS["tiny_f32"], C=C, H=H, d_h=C // H, d_kv=d_kv, n_obj=n_obj, union_objects=n_obj == 1,
                  f_max=3, n_pin=1, cap_frames=4)
    W = make_weights(cfg, logit_scale=2.0)
    kw = dict(absorb=absorb, rope_theta=100.0 if rope else None)
    sess, orc = _session(cfg, W, **kw), OraclePipeline(cfg, W)
    if rope:
        import oracle
        orc.rope = oracle.axial_table(cfg.m, cfg.n, cfg.d_h, 100.0)
    rng = np.random.default_rng(H * d_h + d_kv)
    _read(sess, orc, rng, k)                            # empty bank: y = x bit for bit
    for t, n in enumerate(kept):
        _commit(sess, orc, rng, _first(cfg, n), t, t == 0)
    for o in range(n_obj):
        compare_bank(sess.banks[o].export(), orc.banks[o])
    _read(sess, orc, rng, k)
    # one more frame, once as three calls and once as rs3_frame, on two sessions
    ys = []
    for one_call in (False, True):
        s2, rng2 = _session(cfg, W, **kw), np.random.default_rng(7)
        o2 = OraclePipeline(cfg, W)
        for t, n in enumerate(kept):
            _commit(s2, o2, rng2, _first(cfg, n), t, t == 0)
        X, K, V = (_dev(rng2.standard_normal(s).astype(np.float32))
                   for s in ((1, cfg.mn, C), (n_obj, cfg.mn, d_kv), (n_obj, cfg.mn, d_kv)))
        full = torch.ones((n_obj, cfg.m, cfg.n), dtype=torch.uint8, device="cuda")
        Y = torch.zeros((n_obj, cfg.mn, C), device="cuda")
        if one_call:
            s2.frame(full, X, [k] * s2.n_groups, Y, K, V, full, 9)
        else:
            s2.select(full, X, [k] * s2.n_groups)
            s2.readout(X, Y)
            s2.commit(K, V, full, 9, False)
        Y2 = torch.zeros_like(Y)
        s2.readout(X, Y2)                               # reads the frame just written
        torch.cuda.synchronize()
        ys.append((_host(Y), _host(Y2), s2.banks[0].export()["K"]))
    for a, b in zip(*ys):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("H,all_keys", [(1, False), (2, False), (1, True), (2, True)])
def test_overflowing_logits(H, all_keys):
    """Logits that overflow to -inf over the first half tile, or over every key
    of head 0: a query reads the keys that it has, and the other heads whatever
    head 0 holds.  The workspace form and the direct form agree."""
    import paper_2608_22526_amd as rs3
    from types import SimpleNamespace
    d_h = 64 // H
    cfg = replace(CONFIGS["tiny_f32"], C=64, H=H, d_h=d_h, d_kv=64, f_max=3, n_pin=1, cap_frames=2)
    eye = np.eye(64, dtype=np.float32)
    sess = _session(cfg, SimpleNamespace(Wq=eye, Wk=eye, Wv=eye, Wo=eye))
    rng = np.random.default_rng(H)
    K, V, X = (rng.standard_normal((1, cfg.mn, 64)).astype(np.float32) for _ in range(3))
    K[..., 0] = 0.0
    K[0, :cfg.mn if all_keys else 40, 0] = -3e38
    X[..., 0] = 0.0
    X[0, ::3, 0] = 100.0
    sess.commit(_dev(K), _dev(V), _dev(_first(cfg, 100)[None]), 0, True)
    Xd, full = _dev(X), _dev(np.ones((1, cfg.m, cfg.n), np.uint8))
    sess.select(full, Xd, [cfg.mn])
    ys = []
    for ws in (sess.ws_read, None):
        Y = torch.zeros((1, cfg.mn, 64), device="cuda")
        rs3.readout(sess.layer, sess.grid, 1, Xd, 0, sess.banks, sess.sel_idx, sess.sel_count, 0, cfg.mn, 0, Y, 0, ws=ws)
        torch.cuda.synchronize()
        ys.append(_host(Y)[0])
    rows = np.arange(cfg.mn)
    exp = X[0].astype(np.float64)
    for h in range(H):
        c = slice(h * d_h, (h + 1) * d_h)
        s = X[0, rows, c].astype(np.float64) @ K[0, :100, c].astype(np.float64).T / np.sqrt(d_h)
        s[s < -3e38] = -np.inf
        m = s.max(axis=1, keepdims=True)
        p = np.exp(s - np.where(np.isfinite(m), m, 0.0))
        l = p.sum(axis=1, keepdims=True)
        exp[rows, c] += np.where(l > 0, p / np.where(l > 0, l, 1.0), 0.0) @ V[0, :100, c].astype(np.float64)
    for y in ys:
        assert np.abs(y - exp).max() <= TOL
