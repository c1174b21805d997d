"""The attention of launches with many work-groups, through rs3_attend, against
fp64: every head width, sizes at the edges of its tiles (32 queries, 64 keys, a
window of 64 tiles per split), logits that outgrow the first tile's reference,
and infinities."""
from dataclasses import replace

import numpy as np
import pytest

from workloads import make_weights, storage_to_f64, to_storage

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _attend(Q, K, V, n_splits=0):
    """bf16 storage [rows][H][d_h] -> (O, fp64 reference), each [n_q][H][d_h]."""
    import paper_2608_22526_amd as rs3
    from paper_2608_22526_amd.session import to_device, to_host
    n_q, H, d_h = Q.shape
    n_kv = K.shape[0]
    ws = torch.zeros(max(rs3.attend_workspace_size(n_q, n_kv, H, d_h, rs3.RS3_BF16, n_splits), 256),
                     dtype=torch.uint8, device="cuda")
    O = torch.full((n_q, H, d_h), 7.0, dtype=torch.float32, device="cuda")
    rs3.attend(to_device(Q), to_device(K), to_device(V), n_q, n_kv, H, d_h, rs3.RS3_BF16, O, ws, n_splits)
    torch.cuda.synchronize()
    q, k, v = (storage_to_f64(a, "bf16") for a in (Q, K, V))
    ref = np.empty((n_q, H, d_h))
    with np.errstate(invalid="ignore", over="ignore"):
        for h in range(H):
            s = q[:, h] @ k[:, h].T / np.sqrt(d_h)
            p = np.exp(s - s.max(axis=1, keepdims=True))
            ref[:, h] = (p / p.sum(axis=1, keepdims=True)) @ v[:, h]
    return to_host(O).astype(np.float64), ref


def _rand(rng, *shape, scale=1.0):
    return to_storage((scale * rng.standard_normal(shape)).astype(np.float32), "bf16")


@pytest.mark.parametrize("d_h,H", [(32, 8), (64, 3), (128, 2), (256, 1)])
@pytest.mark.parametrize("n_q,n_kv,n_splits", [(1, 1, 0), (33, 63, 0), (129, 65, 2), (300, 4200, 1), (257, 4097, 5),
                                              (100, 9000, 0)])   # waves without rows at heads of 128
def test_tile_edges(d_h, H, n_q, n_kv, n_splits):
    rng = np.random.default_rng(d_h + n_q + n_kv)
    got, ref = _attend(_rand(rng, n_q, H, d_h, scale=2.0), _rand(rng, n_kv, H, d_h), _rand(rng, n_kv, H, d_h), n_splits)
    # the queries are rounded to bf16 once more after scaling (2^-9 of a logit
    # whose deviation is 2, so under 2 % of a weight at 5 deviations), the
    # weights and the partials once each; |V| stays below 5
    assert np.abs(got - ref).max() <= 5e-2
    assert np.linalg.norm(got - ref) <= 1e-2 * np.linalg.norm(ref)


@pytest.mark.parametrize("d_h", [32, 64, 128, 256])
@pytest.mark.parametrize("rise", [40.0, 100.0, 160.0, 3000.0])
def test_logits_far_above_the_first_tile(d_h, rise):
    """Keys whose logits climb by `rise` (base 2) over the split, with gaps that
    leave one key all the weight: within the range of the weights kept against
    the first tile's maximum, and past it, where the split is run again."""
    rng = np.random.default_rng(int(rise) + d_h)
    n_q, n_kv = 40, 64 * 5
    K = np.zeros((n_kv, 1, d_h), np.float32)
    K[::64, 0, 0] = np.arange(5) / 4.0           # one climbing key per tile
    K[1::64, 0, 0] = -1.0
    Q = np.zeros((n_q, 1, d_h), np.float32)
    Q[:, 0, 0] = rise * np.sqrt(d_h) / 1.4426950408889634
    Q[1, 0, 0] *= -1.0                           # falls instead: every tile's keys at -1 share the weight
    V = _rand(rng, n_kv, 1, d_h)
    for n_splits in (1, 2):
        got, ref = _attend(to_storage(Q, "bf16"), to_storage(K, "bf16"), V, n_splits)
        assert np.abs(got - ref).max() <= 2e-2 * max(1.0, np.abs(ref).max())


def test_infinite_keys():
    """A key with an infinite channel: queries whose logit with it is -inf leave
    the key out; where it is +inf the weights are undefined, and so is the row
    (which has no positive weight sum and comes back 0)."""
    rng = np.random.default_rng(3)
    n_q, n_kv, d_h = 70, 200, 64
    K = rng.standard_normal((n_kv, 1, d_h)).astype(np.float32)
    K[150] = 0.0
    K[150, 0, 0] = np.inf
    Q = np.abs(rng.standard_normal((n_q, 1, d_h))).astype(np.float32) + 0.1
    Q[::2, 0, 0] *= -1.0
    got, ref = _attend(to_storage(Q, "bf16"), to_storage(K, "bf16"), _rand(rng, n_kv, 1, d_h), 1)
    assert np.isnan(ref[1::2]).all() and (got[1::2] == 0.0).all()
    assert np.abs(got[::2] - ref[::2]).max() <= 5e-2


@pytest.mark.parametrize("H,rope", [(1, False), (2, False), (4, True), (8, True)])
def test_result_does_not_depend_on_the_workspace(H, rope):
    """Rows of the last query tile past the selected count are never written:
    whatever the workspace holds there, the selected rows are the same bits."""
    import paper_2608_22526_amd as rs3
    from test_gpu_edge import SMALL, _dev, _host, _session
    cfg = replace(SMALL, C=256, H=H, d_h=256 // H, d_kv=64, f_max=3, cap_frames=3)
    sess = _session(cfg, make_weights(cfg, logit_scale=3.0), rope_theta=100.0 if rope else None)
    rng = np.random.default_rng(H)
    K, V, X = (_rand(rng, 1, cfg.mn, w) for w in (64, 64, 256))
    full = _dev(np.ones((1, cfg.m, cfg.n), np.uint8))
    for t in range(3):
        sess.commit(_dev(np.roll(K, t, axis=1)), _dev(np.roll(V, t, axis=1)), full, t, t == 0)
    Xd = _dev(X)
    sess.select(full, Xd, [37])
    n = rs3.readout_workspace_size(sess.layer, 1, cfg.mn)
    out = []
    for byte in (0, 0xFF, 0x7F, 0xFF):     # zeros, NaN, about 3e38
        ws = torch.full((n,), byte, dtype=torch.uint8, device="cuda")
        Y = torch.empty_like(Xd)
        rs3.readout(sess.layer, sess.grid, 1, Xd, 0, sess.banks, sess.sel_idx, sess.sel_count, 0, cfg.mn, 0, Y, 0, ws=ws)
        torch.cuda.synchronize()
        out.append(_host(Y))
    for y in out[1:]:
        assert np.array_equal(y, out[0])


@pytest.mark.parametrize("d_h", [32, 64, 128, 256])
def test_error_against_64_bits(d_h):
    """No further from fp64 than weights against the maximum of half tiles (moved
    in steps of at least 2^8) and partials in bf16 are, whose rounding is
    modelled here; the queries count as the kernel has them, rounded once."""
    n_q, n_kv = 256, 64 * 40
    rng = np.random.default_rng(d_h)
    bf = lambda x: storage_to_f64(to_storage(np.asarray(x, np.float32), "bf16"), "bf16")
    Q, K, V = _rand(rng, n_q, 1, d_h, scale=3.0), _rand(rng, n_kv, 1, d_h), _rand(rng, n_kv, 1, d_h)
    got, _ = _attend(Q, K, V, 2)
    q = bf(storage_to_f64(Q, "bf16").astype(np.float32)[:, 0] * np.float32(1.4426950408889634 / np.sqrt(d_h)))
    v = storage_to_f64(V, "bf16")[:, 0]
    s = q @ storage_to_f64(K, "bf16")[:, 0].T
    w = np.exp2(s - s.max(axis=1, keepdims=True))
    exact = (w / w.sum(axis=1, keepdims=True)) @ v
    ms, ls, os_ = [], [], []
    for half in (s[:, :n_kv // 2], s[:, n_kv // 2:]):
        ref = np.empty_like(half)
        m = np.full(n_q, -np.inf)
        for t in range(0, half.shape[1], 32):
            mx = half[:, t:t + 32].max(axis=1)
            m = np.where(mx > m + 8, mx, m)
            ref[:, t:t + 32] = m[:, None]
        p = bf(np.exp2(half - ref)) * np.exp2(ref - m[:, None])
        ms.append(m)
        ls.append(p.sum(axis=1))
        os_.append(bf(p @ v[len(os_) * (n_kv // 2):][:n_kv // 2] / ls[-1][:, None]))
    e = [np.exp2(m - np.maximum(*ms)) * l for m, l in zip(ms, ls)]
    model = (e[0][:, None] * os_[0] + e[1][:, None] * os_[1]) / (e[0] + e[1])[:, None]
    assert np.linalg.norm(got[:, 0] - exact) <= np.linalg.norm(model - exact)


@pytest.mark.parametrize("d_h", [32, 64, 128, 256])
def test_values_of_any_size(d_h):
    """Values scaled by a power of two give the result scaled by it, bit for bit:
    the partials keep their precision at any size.  A channel that is not finite
    leaves the others as they are."""
    rng = np.random.default_rng(d_h)
    n_q, n_kv = 40, 500
    Q, K = _rand(rng, n_q, 1, d_h, scale=2.0), _rand(rng, n_kv, 1, d_h)
    V = storage_to_f64(_rand(rng, n_kv, 1, d_h), "bf16")
    V[:, 0, 3] *= 2.0 ** -12
    base, ref = _attend(Q, K, to_storage(V.astype(np.float32), "bf16"), 3)
    assert np.linalg.norm(base - ref) <= 1e-2 * np.linalg.norm(ref)
    assert np.linalg.norm((base - ref)[..., 3]) <= 1e-2 * np.linalg.norm(ref[..., 3])
    for k in (-90, -30, -12, 14, 30, 100):
        got, _ = _attend(Q, K, to_storage((V * 2.0 ** k).astype(np.float32), "bf16"), 3)
        assert np.array_equal(got, base * 2.0 ** k), k
    V[77, 0, 5] = np.inf
    got, _ = _attend(Q, K, to_storage(V.astype(np.float32), "bf16"), 3)
    rest = np.setdiff1d(np.arange(d_h), [5])
    assert (got[:, 0, 5] == np.inf).all() and np.array_equal(got[..., rest], base[..., rest])
    got, _ = _attend(Q, K, to_storage(np.zeros_like(V, dtype=np.float32), "bf16"), 3)
    assert (got == 0.0).all()


@pytest.mark.parametrize("d_h", [32, 64, 128, 256])
def test_first_tile_at_minus_infinity(d_h):
    """Products that overflow to -inf over the whole first tile (and, for some
    queries, the first two), beside queries for which they do not: every query
    reads the keys that it has."""
    rng = np.random.default_rng(d_h)
    n_q, n_kv = 70, 64 * 6 + 10
    Q, K = rng.standard_normal((n_q, 1, d_h)).astype(np.float32), rng.standard_normal((n_kv, 1, d_h)).astype(np.float32)
    K[:, 0, :3] = 0.0
    K[:64, 0, 0] = K[64:128, 0, 1] = -3e38
    K[128:, 0, 2] = -1.0
    Q[:, 0, :3] = 0.0
    Q[::2, 0, 0] = 1e3                     # -inf on the first tile
    Q[::4, 0, 1] = 1e3                     # and on the second
    Q[::8, 0, 2] = 300.0 * np.sqrt(d_h)    # the keys left are far below 0
    V = _rand(rng, n_kv, 1, d_h)
    for n_splits in (1, 2, 4):   # four: the first split holds the first two tiles alone
        got, ref = _attend(to_storage(Q, "bf16"), to_storage(K, "bf16"), V, n_splits)
        assert np.abs(got - ref).max() <= 5e-2


@pytest.mark.parametrize("H", [1, 2, 4, 8])
@pytest.mark.parametrize("kept", [20, 32, 84])
def test_dead_half_of_a_tile(H, kept):
    """Rows of an evicted frame that are not finite, in the half of a tile that
    no resident row shares: they take no part."""
    from harness import TOL, OraclePipeline
    from test_gpu_edge import SMALL, _dev, _host, _session
    import oracle
    cfg = replace(SMALL, C=256, H=H, d_h=256 // H, d_kv=64, f_max=2, n_pin=1, cap_frames=1)
    W = make_weights(cfg)
    sess, orc = _session(cfg, W, rope_theta=100.0), OraclePipeline(cfg, W)
    orc.rope = oracle.axial_table(cfg.m, cfg.n, cfg.d_h, 100.0)
    rng = np.random.default_rng(kept + H)
    for t, n in enumerate((0, 470, kept)):     # the third wraps to the start and evicts the second
        K, V = (rng.standard_normal((1, cfg.mn, cfg.d_kv)).astype(np.float32) for _ in range(2))
        if n == 470:
            V[0, (kept + 31) // 32 * 32:] = np.inf
            V[0, 200:300] = np.nan
        mask = np.zeros((1, cfg.mn), np.uint8)
        mask[0, :n] = 1
        mask = mask.reshape(1, cfg.m, cfg.n)
        K, V = to_storage(K, "bf16"), to_storage(V, "bf16")
        sess.commit(_dev(K), _dev(V), _dev(mask), t, t == 0)
        orc.commit(K, V, mask, t, t == 0)
    X = _rand(rng, 1, cfg.mn, cfg.C)
    Xd, full = _dev(X), np.ones((1, cfg.m, cfg.n), np.uint8)
    sess.select(_dev(full), Xd, [50])
    rows = orc.select(full, X, [50])[0][0]
    Y = torch.zeros((1, cfg.mn, cfg.C), dtype=torch.bfloat16, device="cuda")
    sess.readout(Xd, Y)
    got = storage_to_f64(_host(Y)[0][rows], "bf16")
    assert np.abs(got - orc.readout_rows(X, 0, rows)).max() <= TOL["bf16"]
