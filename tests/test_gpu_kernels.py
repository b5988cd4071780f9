"""The event kernels over the dimensions they are compiled for, with and
without histograms and at every replica count, against the FP64 oracle on the
same points.  Tolerances are the paths' own: 1e-12 for FP64 sums and bins;
FP32-mixed 1e-6 up to d = 8, growing like d / 8 beyond."""
import numpy as np
import pytest

import oracle
from paper_2002_12921_amd import Vegas

pytestmark = pytest.mark.gpu

KINDS = {"gauss": oracle.GAUSS, "bimodal": oracle.BIMODAL, "genz_disc": oracle.GENZ_DISC, "genz_peak": oracle.GENZ_PEAK}


def _params(kind, d):
    r = np.random.default_rng(100 + d)
    if kind == "gauss":
        return [0.2] + list(r.uniform(0.3, 0.7, d))
    if kind == "bimodal":
        return [0.25] + list(r.uniform(0.3, 0.4, d)) + list(r.uniform(0.6, 0.7, d))
    if kind == "genz_disc":
        return list(r.uniform(0.5, 1.5, d)) + list(r.uniform(0.01, 0.1, d))
    return list(r.uniform(0.7, 1.4, d)) + list(r.uniform(0.3, 0.7, d))


def _check(kind, prec, d, N, M, replicas=(0,), params=None):
    params = params or _params(kind, d)
    pr = oracle.Problem(d, N, KINDS[kind], params, seed=11)
    # a grid away from uniform, its own in every dimension
    r = np.random.default_rng(d)
    E = np.zeros((d, N + 1))
    E[:, 1:] = np.cumsum(r.uniform(0.5, 1.5, (d, N)), axis=1)
    E /= E[:, -1:]
    E[:, -1] = 1.0
    o1, o2, Ho = oracle.accumulate(pr, E, 0, M)
    if kind == "genz_disc":
        # the oracle's normalisation has e^c - e^(c a), of which c (1 - a) remain:
        # a relative 2^-53 / c, 1e-10 at c = 1e-6
        c, a = np.array(params[:d]), np.array(params[d:])
        r = np.prod((np.exp(c) - np.exp(c * a)) / (np.expm1(c * (1.0 - a)) * np.exp(c * a)))
        o1, o2, Ho = o1 * r, o2 * r * r, Ho * (r * r)
    tol = 1e-12 if prec == "fp64" else 1e-6 * max(1.0, d / 8)
    sums = set()
    for rep in replicas:
        v = Vegas(d, N, kind, params, prec, seed=11)
        v.set_edges(E)
        if rep:
            v.set_hist_replicas(rep)
        v.iterate(M)
        S1, S2, H = v.last_iteration()
        assert abs(S1 - o1) <= tol * abs(o1) and abs(S2 - o2) <= tol * abs(o2), (d, rep)
        assert np.all(np.abs(H - Ho) <= tol * Ho.sum(axis=1, keepdims=True)), (d, rep)
        sums.add((S1, S2))
    w = Vegas(d, N, kind, params, prec, seed=11)
    w.set_edges(E)
    w.iterate(M, hist=False)
    S1, S2, H = w.last_iteration()
    sums.add((S1, S2))
    assert len(sums) == 1, (d, sums)  # the same bits with and without histograms, whatever the replicas
    assert not H.any()


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_every_dimension(kind, prec):
    """d = 1..21, 24, 25 and 32: the kernels without guards, the guarded ones
    on either side of a bucket's edge, and odd and even bin counts."""
    for d in list(range(1, 22)) + [24, 25, 32]:
        _check(kind, prec, d, 11 if d % 2 else 12, 6007)


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("kind,d,N", [("gauss", 1, 2), ("gauss", 6, 255), ("bimodal", 7, 65), ("genz_peak", 13, 64),
                                      ("genz_disc", 18, 50), ("bimodal", 20, 100), ("gauss", 9, 255),
                                      ("genz_disc", 19, 119), ("gauss", 32, 60), ("genz_peak", 3, 40)])
def test_replica_counts(kind, d, N, prec):
    """Every histogram replica count that fits gives the same sums and bins: one
    dimension after another, and in sets of two (8 replicas) and four (4), the
    last set whole, partial or padded past the LDS."""
    entry = 8 if prec == "fp32_mixed" and kind != "bimodal" else 16
    fits = [r for r in (1, 2, 4, 8, 16) if d * N * (entry + 8 * r) + 512 <= 160 * 1024]
    _check(kind, prec, d, N, 9001, [0] + fits)


def test_largest_blocks_lds():
    """The largest grids that fit the LDS (d * n_bins = 6816 in FP64, 10224 in
    FP32-mixed) still run, and one more bin is still refused."""
    from paper_2002_12921_amd import VegasError
    for prec, d, N in (("fp64", 48, 142), ("fp32_mixed", 48, 213)):
        _check("gauss", prec, d, N, 3001)
        with pytest.raises(VegasError):
            Vegas(d, N + 1, "gauss", _params("gauss", d), prec)


@pytest.mark.parametrize("N,a", [(2, 0.0), (3, 0.5), (50, 0.123456), (64, 0.999), (65, 0.25), (255, 0.7)])
def test_disc_threshold_search(N, a):
    """The discontinuity's position at every bin count the refinement has a
    variant for, at and beside the first and last positions of a bin: events
    counted inside are the oracle's, after a refinement (one wave or the block
    rebuilds the thresholds) and with new parameters from the device."""
    import torch
    d, M = 2, 30_011
    params = [0.7, 1.3, a, 0.2]
    v = Vegas(d, N, "genz_disc", params, "fp64", seed=3)
    for step in range(3):
        E = v.edges()
        if step == 2:  # an edge of the current grid as the threshold
            params = [0.7, 1.3, float(E[0, N // 2]), float(np.nextafter(E[1, 1], 0))]
            v.set_params_device(torch.tensor(params, dtype=torch.float64, device="cuda"))
        pr = oracle.Problem(d, N, oracle.GENZ_DISC, params, seed=3)
        v.iterate(M, refine=True)
        S1, S2, H = v.last_iteration()
        o1, o2, Ho = oracle.accumulate(pr, E, step, M)
        assert abs(S1 - o1) <= 1e-12 * o1 and abs(S2 - o2) <= 1e-12 * o2, step
        assert np.all(np.abs(H - Ho) <= 1e-12 * Ho.sum(axis=1, keepdims=True)), step
        assert np.max(np.abs(v.edges() - oracle.refine(H, E, 1.5))) <= 1e-12, step


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 200])
def test_combination_over_many_records(n):
    """The combination reads its records 64 at a time: every n around that, with
    iterations left out, equals the sums taken one after another."""
    v = Vegas(1, 10, "gauss", [0.3, 0.4], "fp64", seed=5)
    I, var = [], []
    for k in range(n):
        use = k % 3 != 1 or n == 1
        v.iterate(257, combine=use)
        S1, S2, _ = v.last_iteration()
        if use:
            i, s = oracle.iteration_stats(S1, S2, 257)
            I.append(i)
            var.append(s)
    r = v.result()
    m, s, c = oracle.combine(np.array(I), np.array(var))
    assert r["n_iter"] == n and r["n_combined"] == len(I)
    assert abs(r["integral"] - m) <= 1e-13 * abs(m) and abs(r["sigma"] - s) <= 1e-13 * s
    assert (np.isnan(c) and np.isnan(r["chi2_dof"])) or abs(r["chi2_dof"] - c) <= 1e-11 * max(c, 1.0)


@pytest.mark.parametrize("d,N", [(1, 2), (1, 255), (2, 255), (3, 255), (9, 50), (18, 50), (19, 50), (16, 255), (25, 255)])
def test_edges_there_and_back(d, N):
    """Edges carried by one launch, by two and as a copy, and read back by a
    kernel (up to 4096 values) or a copy: the same bits, and the tables built
    from them give the oracle's sums; results waited for through work of more
    than a millisecond are those of that work."""
    _check("genz_disc" if d < 4 else "gauss", "fp64", d, N, 3001)
    params = _params("gauss", d)
    v = Vegas(d, N, "gauss", params, "fp64", seed=3)
    r = np.random.default_rng(N)
    E = np.zeros((d, N + 1))
    E[:, 1:] = np.cumsum(r.uniform(0.5, 1.5, (d, N)), axis=1)
    E /= E[:, -1:]
    E[:, -1] = 1.0
    v.set_edges(E)
    assert np.array_equal(v.edges(), E)
    v.iterate(30_000_000, hist=False)
    first = v.result()
    S1, S2, _ = v.last_iteration()
    assert first["n_iter"] == 1 and abs(first["integral"] - S1 / 3e7) <= 1e-13 * abs(first["integral"])
    v.iterate(1000, hist=False)
    assert v.result()["n_iter"] == 2


@pytest.mark.parametrize("kind,d,params", [
    ("gauss", 1, [1e-150, 0.5]), ("gauss", 1, [50.0, 0.5]), ("gauss", 4, [0.02] + [0.4] * 4), ("gauss", 13, [3.0] + [0.9] * 13),
    ("bimodal", 2, [0.02, 0.3, 0.3, 0.7, 0.7]), ("bimodal", 28, [0.5] + [0.2] * 28 + [0.9] * 28),
    ("genz_disc", 2, [200.0, 150.0, 0.1, 0.2]), ("genz_disc", 5, [1e-6] * 5 + [0.05] * 5)])
def test_exponential_range(kind, d, params):
    """Exponents from 0 past where the exponential is cut (2^-4000), normalisations
    from 1e-9 to 1e150, and the width product's two forms (d up to 24 and beyond)."""
    _check(kind, "fp64", d, 12, 6007, params=params)


@pytest.mark.parametrize("kind", ["gauss", "bimodal", "genz_disc"])
def test_nan_parameter_is_not_hidden(kind):
    """A parameter set on the device that is not a number gives results that are
    not numbers, although the FP64 exponential's argument goes through a minimum."""
    import torch
    d = 3
    q = _params(kind, d)
    v = Vegas(d, 20, kind, q, "fp64")
    for k in range(len(q)):
        p = torch.tensor(q, dtype=torch.float64, device="cuda")
        p[k] = float("nan")
        v.set_params_device(p)
        v.iterate(1000, refine=False, hist=False)
        assert np.isnan(v.last_iteration()[0]), k
