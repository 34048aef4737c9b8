"""TUNER_ALGO_AUTO's fp32 networks (factored first layer, two-plane f16 second layer) at the sizes
where they can go wrong, against the CPU oracle and against the fp32 matrix instructions
(TUNER_ALGO_MFMA).  Run with -m gpu on an MI355X."""
import os

import numpy as np
import pytest

import oracle
import parity
import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

THREADS = min(16, os.cpu_count() or 1)


def space_with_tail(lead, tail, n_rules=1):
    radices = list(lead) + list(tail)
    values = [[float(j + 1) for j in range(r)] for r in radices]
    scales = [wl.SCALE_LOG2 if p % 3 == 0 else wl.SCALE_LINEAR for p in range(len(radices))]
    st = wl.Stream(len(radices) * 1009 + sum(radices))
    terms = (st.integers(n_rules * sum(radices), 5).astype(np.int64) - 2).astype(np.int32).reshape(n_rules, sum(radices))
    terms[:, np.repeat(np.array(radices) > 64, radices)] = 0        # (the rule tables hold 192 entries)
    return wl.Space("tail-" + "x".join(map(str, radices)), values, scales, terms, np.full(n_rules, 2, np.int64))


def predict(sp, m, begin, count, **kw):
    from paper_1506_00842_amd.api import Sweep
    pred, mask = Sweep(sp, m, 0, **kw).predict_all(begin, count)
    torch.cuda.synchronize()
    return pred.cpu().numpy(), mask.cpu().numpy()


# spans (configurations of the trailing parameters) at and beyond both ends of the rule, divisors of
# 32 and none, rows that end inside a tile; widths at the edges of the 32-unit tiles
@pytest.mark.parametrize("lead,tail", [
    ((8, 7, 6, 5, 4), (11,)), ((8, 7, 6, 5, 4), (10,)), ((9, 8, 7, 6), (128,)), ((9, 8, 7, 6), (129,)),
    ((16, 8, 4, 4), (2, 2, 2, 2, 2)), ((6, 5, 4, 3, 3), (5, 7)), ((12, 8, 6), (3, 16)), ((5, 8, 8), (2, 1, 37)),
    ((200, 9), (13,)), ((4, 4, 4, 4, 4, 4, 4, 4), (2, 2)),
])
@pytest.mark.parametrize("hidden", [[1, 1], [33, 31], [64, 65], [128, 17], [96, 97], [20, 128], [128, 128]])
def test_spans_and_widths(lead, tail, hidden):
    sp = space_with_tail(lead, tail)
    n = sp.n_configs
    m = wl.make_model([sp.n_params, *hidden, 1], 3, 7)
    for begin, count in ((0, min(n, 5000)), (n // 3 + 1, min(n - n // 3 - 1, 3001)), (n - 37, 37)):
        oy, ov, _ = oracle.predict_range(sp, m, begin, count, threads=THREADS)
        gp, gm = predict(sp, m, begin, count)
        assert np.array_equal(gm, ov)
        parity.check_predictions(gp, oy, ov)
    # the same configurations, whatever range they are swept in
    whole, _ = predict(sp, m, 0, n)
    part, _ = predict(sp, m, n // 3 + 1, min(n - n // 3 - 1, 3001))
    assert np.array_equal(part.view(np.int32), whole[n // 3 + 1:n // 3 + 1 + len(part)].view(np.int32))


@pytest.mark.parametrize("hidden", [16, 30, 64, 80, 100])
def test_one_hidden_layer(hidden):
    sp = space_with_tail((8, 8, 8, 8, 5), (2, 2, 3, 3))          # 737,280 configurations: factored
    m = wl.make_model([sp.n_params, hidden, 1], 11, hidden)
    begin, count = 100_003, 200_001
    oy, ov, _ = oracle.predict_range(sp, m, begin, count, threads=THREADS)
    gp, gm = predict(sp, m, begin, count)
    assert np.array_equal(gm, ov)
    parity.check_predictions(gp, oy, ov)


def layers(m, e):
    """Views of member e's arrays: W1, b1, W2, b2, wo."""
    (w1, b1), (w2, b2), (wo, _) = m.member_layers(e)
    return w1, b1, w2, b2, wo


def scale_weights(m, kind):
    for e in range(m.n_members):
        w1, b1, w2, b2, wo = layers(m, e)
        if kind == "large-w2":
            w2 *= np.float32(1e6)                       # beyond 64
        elif kind == "small-w2":
            w2 *= np.float32(1e-6)                      # below f16's normal range
        elif kind == "mixed-rows":
            w2 *= (10.0 ** np.linspace(-30, 30, w2.shape[0]))[:, None].astype(np.float32)
        elif kind == "large-bias":
            w2 *= np.float32(1e-8)
            b2 += np.float32(3.0)
        elif kind == "zero-rows":
            w2[::2] = 0
        elif kind == "large-w1":
            w1 *= np.float32(300.0)                     # exponents beyond the factored range
        elif kind == "huge":
            w1 *= np.float32(1e30)
            w2 *= np.float32(1e37)


@pytest.mark.parametrize("kind", ["large-w2", "small-w2", "mixed-rows", "large-bias", "zero-rows", "large-w1", "huge"])
@pytest.mark.parametrize("lead,tail,hidden", [((8, 7, 6, 5), (2, 2, 2, 2, 2), [48, 40]), ((64, 8), (5,), [48, 40]),
                                              ((8, 7, 6, 5), (2, 2, 2, 2, 2), [128, 120])])
def test_magnitudes_of_weights(kind, lead, tail, hidden):
    """Weights of unusual magnitude: the error against the oracle, in the 2-norm over the
    configurations, stays within twice that of the fp32 instructions (weights beyond 64 use them)
    plus the fp32 rounding of the result, 1e-6 of the predictions' scale."""
    sp = space_with_tail(lead, tail, n_rules=0)
    m = wl.make_model([sp.n_params, *hidden, 1], 2, 5)
    scale_weights(m, kind)
    import paper_1506_00842_amd as T
    n = sp.n_configs
    oy, ov, _ = oracle.predict_range(sp, m, 0, n, threads=THREADS)
    auto, _ = predict(sp, m, 0, n)
    mfma, _ = predict(sp, m, 0, n, algo=T.TUNER_ALGO_MFMA)
    err, ref = np.linalg.norm(auto - oy), np.linalg.norm(mfma - oy)
    print(kind, sp.name, "error", err, "fp32 instructions", ref)
    assert err <= 2 * ref + 1e-6 * parity.scale_of(oy) * np.sqrt(n), (err, ref)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("where", ["w1", "b1", "w2", "b2", "wo"])
def test_non_finite_weights(value, where):
    """One weight that is not finite: the same results as the fp32 instructions, NaN for NaN."""
    sp = space_with_tail((8, 7, 6, 5), (2, 2, 2, 2, 2), n_rules=0)
    m = wl.make_model([sp.n_params, 40, 33, 1], 2, 9)
    a = dict(zip(("w1", "b1", "w2", "b2", "wo"), layers(m, 1)))[where]
    a.reshape(-1)[5] = value
    import paper_1506_00842_amd as T
    auto, _ = predict(sp, m, 0, 3000)
    mfma, _ = predict(sp, m, 0, 3000, algo=T.TUNER_ALGO_MFMA)
    assert np.array_equal(np.isnan(auto), np.isnan(mfma))
    fine = np.isfinite(mfma)
    assert np.array_equal(auto[~fine & ~np.isnan(auto)], mfma[~fine & ~np.isnan(mfma)])
    if fine.any():
        np.testing.assert_allclose(auto[fine], mfma[fine], rtol=0, atol=2e-5 * max(1.0, np.abs(mfma[fine]).max()))


def test_list_evaluation():
    sp = space_with_tail((8, 7, 6, 5), (2, 2, 2, 2, 2))
    m = wl.make_model([sp.n_params, 100, 40, 1], 3, 3)
    from paper_1506_00842_amd.api import Sweep
    idx = np.random.default_rng(1).integers(0, sp.n_configs, 5003).astype(np.uint64)
    sw = Sweep(sp, m, 0)
    pi, mi = sw.predict_indices(torch.from_numpy(idx.astype(np.uint32).view(np.int32)).to("cuda:0"))
    torch.cuda.synchronize()
    ry, rv = oracle.predict_indices(sp, m, idx, threads=THREADS)
    assert np.array_equal(mi.cpu().numpy(), rv)
    parity.check_predictions(pi.cpu().numpy(), ry, rv)


@pytest.mark.parametrize("members,hidden", [(64, [128, 128]), (512, [64, 64]), (2000, [30])])
def test_static_scratch_keeps_ensembles_whose_tables_outgrow_it(members, hidden):
    """Their workspace exceeds the static array, the fp32 matrix network's does not: the call
    runs on that one, bit for bit."""
    import paper_1506_00842_amd as T
    from paper_1506_00842_amd.api import Sweep
    sp = space_with_tail((3,) * 16, (3,) * 4)
    m = wl.make_model([sp.n_params, *hidden, 1], members, 3)
    k, begin, count = 10, 1000003, 700
    auto = Sweep(sp, m, k)
    ref = Sweep(sp, m, k, algo=T.TUNER_ALGO_MFMA)
    assert T.tuner_workspace_bytes(auto.space, auto.model, k) > T.TUNER_STATIC_SCRATCH_BYTES
    assert T.tuner_workspace_bytes(ref.space, ref.model, k) <= T.TUNER_STATIC_SCRATCH_BYTES
    T.tuner_predict_topk_static(auto.space, auto.model, begin, count, k, 0, auto.values, auto.indices, auto.n_found)
    ref.topk(begin, count)
    torch.cuda.synchronize()
    assert int(ref.n_found.item()) == k and torch.equal(auto.n_found, ref.n_found)
    assert torch.equal(auto.values, ref.values) and torch.equal(auto.indices, ref.indices)
