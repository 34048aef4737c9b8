"""Edges of the single-workgroup sampler and of the accuracy metric.  Run with -m gpu."""
import numpy as np
import pytest

import oracle
import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def tuner_for(sp):
    from paper_1506_00842_amd.api import Tuner
    return Tuner(sp)


# both sides of the table sizes and of the switch to the table in memory (8192 samples), batches
# that end inside the draws, draws that run out, spaces smaller than the sample
@pytest.mark.parametrize("maker,n,max_draws", [
    (wl.paper_stereo, 1, 1), (wl.paper_stereo, 2048, 4096), (wl.paper_stereo, 2049, 4097),
    (wl.paper_stereo, 8192, 8192), (wl.paper_stereo, 8192, 200_000), (wl.paper_stereo, 8193, 200_000),
    (wl.paper_convolution, 3000, 3100), (wl.tiny, 256, 20_000), (wl.tiny, 1000, 64_000), (wl.large, 5000, 12_000),
])
def test_sampler_edges(maker, n, max_draws):
    sp = maker().space
    idx, found = tuner_for(sp).sample_valid(11, n, max_draws)
    torch.cuda.synchronize()
    expect = oracle.sample_valid(sp, 11, n, max_draws)
    got = idx.cpu().numpy().view(np.uint32)
    assert int(found.item()) == len(expect)
    assert np.array_equal(got[:len(expect)].astype(np.uint64), expect)
    assert np.all(got[len(expect):] == 0xFFFFFFFF)


def test_sampler_without_valid_configurations():
    sp = wl.paper_convolution().space
    none = wl.Space("none", sp.values, sp.scales, sp.constraint_terms, np.full(1, -1, np.int64))
    idx, found = tuner_for(none).sample_valid(1, 50, 9000)
    torch.cuda.synchronize()
    assert int(found.item()) == 0 and bool((idx == -1).all())


# per term 2 ulp of e^y / t <= 1.5 (4e-7, absolute: e^y and t nearly cancel), and the sum's rounding
# (partial sums of up to 100 terms, then a tree: 1e-6 of the sum)
@pytest.mark.parametrize("offset_pred,offset_time", [(0, 0), (1, 0), (0, 3), (2, 2)])
@pytest.mark.parametrize("n", [1, 3, 4, 4095, 4096, 16_387, 100_003])
def test_mean_relative_error_alignment(n, offset_pred, offset_time):
    rng = np.random.default_rng(n)
    pred = rng.normal(-5.0, 1.0, n + 4).astype(np.float32)
    times = (np.exp(pred) * rng.uniform(0.7, 1.4, n + 4)).astype(np.float32)
    p, t = pred[offset_pred:offset_pred + n], times[offset_time:offset_time + n]
    dp, dt = torch.from_numpy(pred).cuda()[offset_pred:offset_pred + n], torch.from_numpy(times).cuda()[offset_time:offset_time + n]
    mean, used = tuner_for(wl.tiny().space).mean_relative_error(dp, dt)
    want = np.mean(np.abs(np.exp(p.astype(np.float64)) - t) / t.astype(np.float64))
    assert int(used.item()) == n
    assert abs(float(mean.item()) - want) <= 4e-7 + 1e-6 * want


@pytest.mark.parametrize("y,t", [(0.5, 1e-40), (-85.0, 1e-37), (-100.0, 3e-39), (0.5, 3e38), (88.0, 1.0), (88.0, 2e38),
                                 (89.0, 1.0), (-200.0, 1.0), (79.0, 1e34), (-79.0, 1e-34), (0.0, 1.0)])
@pytest.mark.parametrize("n", [1, 16_383, 16_384])        # alone, or among failed runs in the short and the long form
def test_mean_relative_error_range(n, y, t):
    y, t = np.float32(y), np.float32(t)
    pred, times = torch.zeros(n), torch.full((n,), -1.0)
    pred[n // 3], times[n // 3] = float(y), float(t)
    mean, used = tuner_for(wl.tiny().space).mean_relative_error(pred.cuda(), times.cuda())
    with np.errstate(over="ignore"):
        want = float(np.float32(np.abs(np.float64(np.float32(np.exp(np.float64(y)))) - np.float64(t)) / np.float64(t)))
    assert int(used.item()) == 1
    got = float(mean.item())
    assert got == want or abs(got - want) <= 3e-7 * max(want, 1.0), (got, want)
