"""GPU parity of the carrier-concentration diagnostics (grkv_carrier_stats)
against the float64 oracle.

The assignment is an argmax of fp32 cosine similarities on the GPU and of
fp64 ones in the oracle, so where the two differ the GPU's choice must be a
near-tie: its fp64 cosine within 1e-5 of the best.  The metrics are compared
with the oracle's metrics of the GPU's own assignment (exact integer loads),
and L_common with the same sum taken from the stats in float64.
"""
import numpy as np
import pytest

import workloads as W
from oracle import grkv_carrier_oracle as CO
from oracle import grkv_oracle as O
from tests.parity import to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(cfg, q, K, V):
    import paper_2605_31105_amd as G
    qd, Kd, Vd = (to_device(a, cfg.dtype) for a in (q, K, V))
    res = G.compress(qd, Kd, Vd, cfg.window, cfg.budget, cfg.pool_kernel, cfg.lam)
    assign, counts, metrics, lc = G.carrier_stats(Kd, res.idx, cfg.group, res.stats)
    torch.cuda.synchronize()
    return dict(idx=res.idx.cpu().numpy().astype(np.int64), stats=res.stats.cpu().numpy(),
                assign=assign.cpu().numpy(), counts=counts.cpu().numpy(),
                metrics=metrics.cpu().numpy(), l_common=float(lc.cpu()[0]))


def _check_unit(cfg, K, gpu, u):
    Kd = W.decode(K[u], cfg.dtype)
    idx = gpu["idx"][u]
    ga = gpu["assign"][u].astype(np.int64)
    oa = CO.carrier_assignment(Kd, idx)
    assert np.array_equal(ga < 0, oa < 0)
    ev = np.flatnonzero(oa >= 0)
    diff = ev[ga[ev] != oa[ev]]
    if diff.size:
        Cm = CO.cosine_matrix(Kd[diff], Kd[idx])
        best = Cm.max(axis=1)
        chosen = Cm[np.arange(diff.size), ga[diff]]
        assert np.all(chosen >= best - 1e-5), "unit %d: a non-tie assignment differs" % u
    # metrics of the GPU's assignment, loads exact
    m = CO.carrier_metrics(ga, idx)
    assert np.array_equal(gpu["counts"][u], m["counts"])
    want = [m[k] for k in ("b", "b_eff", "a_max", "gini", "boundary_fraction", "boundary_share",
                           "enrichment", "boundary_interior_load")]
    np.testing.assert_allclose(gpu["metrics"][u], np.array(want, dtype=np.float64), rtol=2e-6,
                               equal_nan=True)
    return dict(unit=u, evicted=int(ev.size), differ=int(diff.size),
                b_over_c=m["b"] / idx.size, beff_over_c=m["b_eff"] / idx.size,
                a_max=m["a_max"], enrichment=m["enrichment"])


def _lcommon_check(gpu):
    st = gpu["stats"].astype(np.float64)
    want = float(np.sum(st[:, 2] * st[:, 0]) / np.sum(st[:, 0]))
    assert abs(gpu["l_common"] - want) <= 1e-6 * max(want, 1e-30)


def test_carrier_config2():
    cfg = W.config(2)
    q, K, V = W.make_batch(cfg)
    gpu = _run(cfg, q, K, V)
    for u in range(cfg.units):
        print(_check_unit(cfg, K, gpu, u), flush=True)
    _lcommon_check(gpu)
    # L_common against the oracle's own value step on these units
    yf, yc = [], []
    for u in range(cfg.units):
        r = O.compress_unit(*(W.decode(a[u], cfg.dtype) for a in (q, K, V)), cfg.window,
                            cfg.budget, cfg.pool_kernel, cfg.lam)
        yf.append(r["Y"])
        yc.append(r["X"] @ r["Vstar"])
    want = CO.l_common(yf, yc)
    assert abs(gpu["l_common"] - want) <= 2e-3 * want, (gpu["l_common"], want)


@pytest.mark.parametrize("label,over", [
    ("head-dim-64", dict(head_dim=64)),
    ("ragged-n", dict(n=1000, budget=200)),
    ("budget-eq-n", dict(n=640, budget=640)),
    ("budget-eq-window", dict(budget=32)),
], ids=["head-dim-64", "ragged-n", "budget-eq-n", "budget-eq-window"])
def test_carrier_edges(label, over):
    base = dict(layers=1, kv_heads=2, n=2048, budget=256)
    base.update(over)
    cfg = W.config(2, **base)
    q, K, V = W.make_batch(cfg)
    gpu = _run(cfg, q, K, V)
    for u in range(cfg.units):
        print(label, _check_unit(cfg, K, gpu, u), flush=True)
    if label == "budget-eq-n":
        assert np.all(gpu["assign"] == -1) and np.all(gpu["metrics"][:, 0] == 0)


def test_carrier_config4_sampled():
    cfg = W.config(4)
    q, K, V = W.make_batch(cfg)
    gpu = _run(cfg, q, K, V)
    for u in (0, 255):
        print(_check_unit(cfg, K, gpu, u), flush=True)
    _lcommon_check(gpu)
    # every unit: loads sum to the evicted count, b <= c, b_eff <= b
    c = cfg.budget
    assert np.all(gpu["counts"].sum(axis=1) == cfg.n - c)
    met = gpu["metrics"]
    assert np.all(met[:, 0] <= c) and np.all(met[:, 1] <= met[:, 0] + 1e-3)


@pytest.mark.parametrize("units,n,c,d,kind", [
    (256, 1000, 200, 128, "normal"),    # one row tile per wave, a part-filled last key tile
    (128, 1030, 64, 64, "normal"),      # the same at head dim 64, one whole key tile
    (256, 1000, 512, 128, "normal"),    # two row tiles per wave
    (205, 1111, 525, 64, "normal"),     # the same at head dim 64, a part-filled last key tile
    (100, 1000, 100, 128, "normal"),    # two row tiles, since one would take a second round
    (3, 2048, 300, 128, "normal"),      # the assignments counted two at a time
    (3, 2049, 300, 128, "normal"),      # and sixteen
    (4, 900, 256, 128, "normal"),       # the most slots whose pairs are summed directly
    (4, 900, 257, 64, "normal"),        # the fewest that go through the histogram
    (2, 20000, 130, 64, "one-carrier"), # one load of all tokens, pairs directly
    (2, 20000, 300, 64, "one-carrier"), # a load past the histogram of loads
    (2, 3000, 100, 128, "duplicates"),  # equal cosines go to the lower slot
])
def test_carrier_tiles_and_loads(units, n, c, d, kind):
    import paper_2605_31105_amd as G
    rng = np.random.default_rng(units + n)
    K = rng.standard_normal((units, n, d)).astype(np.float32)
    idx = np.sort(np.stack([rng.choice(n, c, replace=False) for _ in range(units)]), axis=1)
    for u in range(units):
        if kind == "one-carrier":
            x = rng.standard_normal(d).astype(np.float32)
            K[u] = x + 0.01 * K[u]
            K[u, idx[u, 1:]] *= -1.0
        elif kind == "duplicates":
            K[u] = K[u][rng.integers(0, 7, n)]
            K[u, idx[u, 50:60]] = 0.0
    bits = W.f32_to_bf16_bits(K)
    print("case", units, n, c, d, kind, flush=True)
    a, cnt, met, _ = G.carrier_stats(to_device(bits, "bf16"),
                                     torch.from_numpy(idx.astype(np.int32)).cuda(), 4)
    torch.cuda.synchronize()
    gpu = dict(idx=idx, assign=a.cpu().numpy(), counts=cnt.cpu().numpy(), metrics=met.cpu().numpy())
    cfg = W.config(2, head_dim=d)
    for u in (0, 1, units - 1):
        print(_check_unit(cfg, bits, gpu, u), flush=True)
        if kind == "duplicates":   # products of equal keys are equal bit for bit
            keep = gpu["assign"][u] >= 0
            assert np.array_equal(gpu["assign"][u][keep], CO.carrier_assignment(
                W.decode(bits[u], "bf16"), idx[u])[keep])
        if kind == "one-carrier":
            assert gpu["counts"][u].max() >= 8192
