"""GPU parity of the budget front-ends: adaptive per-head budgets (exact
integers from the GPU's pooled scores) and ragged per-unit compression (every
unit against the float64 oracle with its own budget, to the parity bar of the
uniform path)."""
import numpy as np
import pytest

import workloads as W
from oracle import grkv_frontend_oracle as FO
from oracle import grkv_oracle as O
from tests.parity import D_TOL, V_TOL, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _pooled(cfg, qd, Kd, Vd):
    import paper_2605_31105_amd as G
    res = G.compress(qd, Kd, Vd, cfg.window, cfg.budget, cfg.pool_kernel, cfg.lam)
    return G.intermediates(res)["pooled"].contiguous()


@pytest.mark.parametrize("cfg_id", [2, 4])
def test_adaptive_budgets(cfg_id):
    import paper_2605_31105_amd as G
    cfg = W.config(cfg_id)
    q, K, V = W.make_batch(cfg)
    qd, Kd, Vd = (to_device(a, cfg.dtype) for a in (q, K, V))
    pooled = _pooled(cfg, qd, Kd, Vd)
    got = G.adaptive_budgets(pooled, cfg.layers, cfg.kv_heads, cfg.budget, cfg.window)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    want = FO.adaptive_budgets(pooled.cpu().numpy().astype(np.float64), cfg.layers,
                               cfg.kv_heads, cfg.budget, cfg.window)
    print("budgets", got[:16], flush=True)
    assert np.array_equal(got, want)
    assert np.all(got.reshape(cfg.layers, cfg.kv_heads).sum(axis=1) == cfg.kv_heads * cfg.budget)


def _ragged_check(cfg, q, K, V, budgets, units=None, **opts):
    """Every unit (or the sampled ``units``) against the oracle with its own
    budget; every unit's retained set checked for the properties that hold at
    any size."""
    import paper_2605_31105_amd as G
    qd, Kd, Vd = (to_device(a, cfg.dtype) for a in (q, K, V))
    idx, k_out, v_out, stats, off = G.compress_ragged(qd, Kd, Vd, cfg.window, budgets,
                                                      cfg.pool_kernel, cfg.lam, **opts)
    torch.cuda.synchronize()
    idx, v_out, stats = idx.cpu().numpy(), v_out.cpu().numpy(), stats.cpu().numpy()
    kc = k_out.cpu()
    kb = kc.view(torch.int16).numpy().view(np.uint16) if cfg.dtype == "bf16" else kc.numpy()
    oo = {k: v for k, v in opts.items() if k in ("n_sink", "beta", "fix_window", "causal_window")}
    opt = O.Options(**oo) if oo else None
    assert np.array_equal(off, FO.packed_offsets(budgets))
    for u, b in enumerate(budgets):
        ids = idx[int(off[u]):int(off[u]) + int(b)]
        assert np.all(np.diff(ids) > 0)
        assert np.array_equal(ids[-cfg.window:], np.arange(cfg.n - cfg.window, cfg.n))
    assert np.all(stats[:, 3] == 0)
    for u in (range(len(budgets)) if units is None else units):
        b = int(budgets[u])
        s = slice(int(off[u]), int(off[u]) + b)
        r = O.compress_unit(*(W.decode(a[u], cfg.dtype) for a in (q, K, V)), cfg.window, b,
                            cfg.pool_kernel, cfg.lam, opt)
        assert np.array_equal(idx[s], r["idx"]), "unit %d: retained set" % u
        assert np.array_equal(kb[s], K[u][r["idx"]])
        verr = np.abs(v_out[s] - r["Vstar"]).max() / np.abs(r["Vstar"]).max()
        print(dict(unit=u, budget=b, v_err=float(verr), d=float(stats[u, 2]),
                   d_oracle=float(r["D_after"])), flush=True)
        assert verr <= V_TOL and stats[u, 3] == r["status"]
        if r["D_after"] > 1e-12:
            assert abs(stats[u, 2] - r["D_after"]) / r["D_after"] <= D_TOL
        else:   # budget = n: nothing evicted, the merge is exact
            assert stats[u, 2] <= 1e-6


def test_ragged_pyramid():
    import paper_2605_31105_amd as G
    cfg = W.config(2, layers=4, kv_heads=2, n=2048, budget=256)
    q, K, V = W.make_batch(cfg)
    budgets = G.pyramid_budgets(cfg.layers, cfg.kv_heads, cfg.budget, cfg.window, cfg.n)
    assert len(set(budgets.tolist())) == cfg.layers
    _ragged_check(cfg, q, K, V, budgets)


def test_ragged_adaptive():
    import paper_2605_31105_amd as G
    cfg = W.config(2)
    q, K, V = W.make_batch(cfg)
    qd, Kd, Vd = (to_device(a, cfg.dtype) for a in (q, K, V))
    budgets = G.adaptive_budgets(_pooled(cfg, qd, Kd, Vd), cfg.layers, cfg.kv_heads, cfg.budget,
                                 cfg.window).cpu().numpy()
    _ragged_check(cfg, q, K, V, budgets)


def test_ragged_token_based_and_mixed_budgets():
    # pool width 1 (token-based scoring), budgets differing unit to unit
    cfg = W.config(2, layers=1, kv_heads=4, n=1000, budget=200, pool_kernel=1)
    q, K, V = W.make_batch(cfg)
    _ragged_check(cfg, q, K, V, [200, 32, 1000, 137])


def test_ragged_uniform_equals_compress():
    import paper_2605_31105_amd as G
    cfg = W.config(2)
    q, K, V = W.make_batch(cfg)
    qd, Kd, Vd = (to_device(a, cfg.dtype) for a in (q, K, V))
    a = G.compress(qd, Kd, Vd, cfg.window, cfg.budget, cfg.pool_kernel, cfg.lam)
    idx, k_out, v_out, stats, _ = G.compress_ragged(qd, Kd, Vd, cfg.window,
                                                    [cfg.budget] * cfg.units, cfg.pool_kernel,
                                                    cfg.lam)
    torch.cuda.synchronize()
    assert torch.equal(a.idx.reshape(-1), idx) and torch.equal(a.k_out.reshape(-1, cfg.head_dim), k_out)
    assert torch.equal(a.v_out.reshape(-1, cfg.head_dim), v_out) and torch.equal(a.stats, stats)


def test_ragged_full_workload_pyramid_and_adaptive_sampled():
    # the 32-layer n=32k workload in one ragged call per front-end, sampled
    # units against the oracle (the adaptive sample holds the smallest and
    # the largest budget)
    import paper_2605_31105_amd as G
    cfg = W.config(4)
    q, K, V = W.make_batch(cfg)
    b = G.pyramid_budgets(cfg.layers, cfg.kv_heads, cfg.budget, cfg.window, cfg.n)
    _ragged_check(cfg, q, K, V, b, units=(0, 37, 128, 255))
    qd, Kd, Vd = (to_device(a, cfg.dtype) for a in (q, K, V))
    b = G.adaptive_budgets(_pooled(cfg, qd, Kd, Vd), cfg.layers, cfg.kv_heads, cfg.budget,
                           cfg.window).cpu().numpy()
    del qd, Kd, Vd
    _ragged_check(cfg, q, K, V, b, units=(int(np.argmin(b)), int(np.argmax(b)), 101, 200))


@pytest.mark.parametrize("label,cfg_id,over,budgets", [
    ("fp32", 1, {}, [16, 300]),
    ("bf16-m256", 2, dict(layers=1, kv_heads=2, n=2048, window=64, budget=512), [512, 300]),
], ids=["fp32", "bf16-m256"])
def test_ragged_generic_path(label, cfg_id, over, budgets):
    # shapes outside the bf16 fast path run one call per run of equal budgets
    cfg = W.config(cfg_id, **over)
    q, K, V = W.make_batch(cfg)
    _ragged_check(cfg, q, K, V, budgets)


def _shift_sampled_ranks(flat, kk, above):
    """Exchanges sampled and other keys so that the search's samples place the
    kk-th largest key one and a half bracket half-widths off: above (or below) its
    bracket of sampled ranks."""
    N = flat.shape[1]
    stride = -(-N // 8192)
    ns = -(-N // stride)
    i = np.arange(ns)
    pos = (i >> 2) * 4 * stride + 8 * (i & 3) if N >= 65536 else i * stride
    pos = pos[pos < N]
    r = kk // stride
    delta = min((5 if N >= 65536 else 4) * int(np.sqrt(r * (1 - min(r / ns, 1)))) + 8,
                18432 // (2 * stride))
    want = r - 3 * delta // 2 if above else r + 3 * delta // 2
    assert 0 < want < ns
    free = np.setdiff1d(np.arange(N), pos)
    for x in flat:
        T = np.partition(x, N - kk)[N - kk]
        have = np.count_nonzero(x[pos] >= T)
        if above:     # fewer samples at or above T
            a, b = pos[x[pos] >= T], free[x[free] < T]
        else:
            a, b = pos[x[pos] < T], free[x[free] >= T]
        k = abs(have - want)
        assert (have > want) == above and k <= min(a.size, b.size)
        a, b = a[:k].copy(), b[:k].copy()
        x[a], x[b] = x[b], x[a]
        assert np.count_nonzero(x[pos] >= T) == want


@pytest.mark.parametrize("layers,heads,P,budget,dist", [
    (3, 1, 500, 60, "normal"),          # every key fits the candidate area
    (2, 3, 4096, 300, "normal"),        # 12288 keys: the most that fit
    (2, 3, 4097, 300, "normal"),        # more than fit: three heads take the radix
    (2, 4, 3073, 300, "normal"),        # and four are sampled
    (4, 8, 20011, 1500, "normal"),
    (2, 8, 9000, 700, "two-values"),    # ties too many for the bracket: full radix
    (2, 5, 8000, 700, "sampled-low"),   # samples miss the top: the bracket fails its check
    (2, 8, 20000, 1500, "sampled-low"),  # the same with four samples per cache line
    (2, 4, 6000, 6032, "normal"),       # every token of the layer taken
    (2, 4, 6000, 32, "normal"),         # none taken
    (2, 1, 20000, 900, "normal"),       # few heads, one batch of loads: radix
    (2, 1, 40000, 900, "normal"),       # and two batches
    (2, 1, 66000, 900, "normal"),       # one head, sampled four per cache line
    (2, 2, 40000, 900, "normal"),
    (3, 17, 997, 90, "normal"),         # more heads than waves, short segments
    (2, 128, 130, 40, "normal"),
    (1, 3, 70001, 30000, "normal"),     # a high rank
    (1, 8, 80000, 6352, "normal"),      # the bracket's width is capped
    (1, 8, 65537, 4096, "normal"),
    (1, 8, 131000, 8192, "normal"),     # too many keys per sample: radix
    (1, 16, 131000, 8192, "normal"),
    (2, 8, 20000, 1500, "rank-above"),  # T just above the bracket: full radix
    (2, 8, 20000, 1500, "rank-below"),  # and just below
    (2, 5, 8000, 700, "rank-above"),    # the same with one sample per cache line
    (2, 5, 8000, 700, "rank-below"),
    (2, 8, 40000, 3000, "runs"),        # neighbouring scores alike
    (2, 8, 40000, 20000, "zeros"),      # ties at zero
    (2, 8, 4000, 3900, "zeros"),
    (2, 8, 40000, 3000, "narrow"),      # scores within a percent of each other
    (2, 4, 6000, 700, "narrow"),
])
def test_adaptive_budgets_search_paths(layers, heads, P, budget, dist):
    import paper_2605_31105_amd as G
    rng = np.random.default_rng(layers * 1000 + P)
    U = layers * heads
    if dist == "two-values":
        p = np.where(rng.random((U, P)) < 0.3, 1.0, 0.5).astype(np.float32)
    else:
        p = np.exp(1.5 * rng.standard_normal((U, P))).astype(np.float32)
    if dist == "sampled-low":
        flat = p.reshape(layers, -1)
        stride = -(-flat.shape[1] // 8192)
        assert stride > 1
        flat += 1.0
        flat[:, ::stride] *= np.float32(1e-3)
        if flat.shape[1] >= 65536:
            for k in range(4):
                flat[:, 8 * k::4 * stride] *= np.float32(1e-3)
    if dist == "runs":
        p = (np.repeat(p[:, ::32], 32, axis=1)[:, :P]
             * np.exp(0.1 * rng.standard_normal((U, P)))).astype(np.float32)
    if dist == "narrow":
        p = np.exp(0.005 * rng.standard_normal((U, P))).astype(np.float32)
    if dist == "zeros":
        p = np.maximum(p - 3.0, 0.0).astype(np.float32)
    if dist.startswith("rank-"):
        _shift_sampled_ranks(p.reshape(layers, -1), heads * (budget - 32), dist == "rank-above")
    print("case", layers, heads, P, budget, dist, flush=True)
    got = G.adaptive_budgets(torch.from_numpy(p).cuda(), layers, heads, budget, 32)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), FO.adaptive_budgets(p, layers, heads, budget, 32))
