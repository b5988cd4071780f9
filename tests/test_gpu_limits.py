"""Calls at the ends of what the entry points take."""
import numpy as np
import pytest
import torch

import oracle
from paper_2002_12921_amd import Vegas, VegasError
from paper_2002_12921_amd.batch import VegasBatch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 20, 23, 25, 26, 27, 28])
def test_user_values_near_the_largest_double(d):
    """f = 1e300 on the uniform grid (w = 1): S1 = 1e300 M, within the rounding of
    M = 1000 sums, in every remainder of d by four, below and beyond d = 24."""
    v = Vegas(d, 2, source="__device__ vegas_real vegas_integrand(const vegas_real* x, int dim, const double* p)\n"
                           "{ return 1e300; }", precision="fp64")
    for hist in (True, False):
        v.iterate(1000, hist=hist)
        S1 = v.last_iteration()[0]
        assert abs(S1 / 1000 - 1e300) <= 1e-12 * 1e300, (d, hist, S1)


@pytest.mark.parametrize("kind,d,a,x", [("gauss", 1, 3.0, 690), ("gauss", 2, 3.0, 690), ("gauss", 3, 2.0, 700), ("gauss", 4, 2.0, 700),
                                        ("gauss", 5, 3.0, 690), ("bimodal", 5, 3.0, 690), ("gauss", 22, 0.6, 760),
                                        ("gauss", 25, 0.6, 760), ("bimodal", 25, 0.6, 760), ("gauss", 27, 0.6, 770)])
def test_values_near_the_smallest_double(kind, d, a, x):
    """A Gaussian centred far outside, about e^-x in the middle: the values that
    count are beyond 2^-1010 and keep their digits. An exponent near 700 has its
    own rounding in the value: some 2^-53 700 (d + 5) of it, 3e-12 at d = 30; 4e-12."""
    N, M = 2, 6007
    mu = 0.5 + a * np.sqrt(x / d)
    params = [a] + [mu] * d * (2 if kind == "bimodal" else 1)
    pr = oracle.Problem(d, N, oracle.GAUSS if kind == "gauss" else oracle.BIMODAL, params, seed=11)
    E = np.tile([0.0, 0.5, 1.0], (d, 1))
    o1 = oracle.accumulate(pr, E, 0, M)[0]
    v = Vegas(d, N, kind, params, "fp64", seed=11)
    v.iterate(M, hist=False)
    S1 = v.last_iteration()[0]
    assert 2.0 ** -1000 < o1 < 2.0 ** -940
    assert abs(S1 - o1) <= 4e-12 * o1, (S1, o1)


@pytest.mark.parametrize("d", [24, 25, 26, 27, 28, 33])
def test_narrow_bins_in_all_dimensions(d):
    """Widths whose product is near 2^-1020: an event's weight keeps its digits,
    also while the product is formed. Gaussian against the oracle (about 100
    roundings of each value: 1e-13), and a constant as source on the same bins."""
    N, M = 10, 60007
    a, E = 2.0 ** (-930.0 / d), np.tile(np.append(np.arange(N) * 2.0 ** (-1020.0 / d), 1.0), (d, 1))
    pr = oracle.Problem(d, N, oracle.GAUSS, [a] + [0.0] * d, seed=11)
    o1, o2, _ = oracle.accumulate(pr, E, 0, M)
    v = Vegas(d, N, "gauss", [a] + [0.0] * d, "fp64", seed=11)
    v.set_edges(E)
    v.iterate(M, hist=False)
    S1, S2, _ = v.last_iteration()
    assert o1 > 0 and abs(S1 - o1) <= 1e-13 * o1 and abs(S2 - o2) <= 2e-13 * o2
    # every event inside counts 2^930 (N 2^(-1020/d))^d: S1^2 / S2 of them
    u = Vegas(d, N, source="__device__ vegas_real vegas_integrand(const vegas_real* x, int dim, const double* p)\n"
                           "{ for (int i = 0; i < dim; ++i) if (x[i] >= %s) return 0; return 0x1p930; }" % E[0, N - 1].hex(),
              precision="fp64", seed=11)
    u.set_edges(E)
    u.iterate(M, hist=False)
    S1, S2, _ = u.last_iteration()
    b = v.dump_events(0, M, iteration=0)[:, :d].cpu().numpy()
    inside = int((b < N - 1).all(axis=1).sum())
    value = 2.0 ** 930 * np.prod(N * (E[:, 1] - E[:, 0]))
    assert inside > 100 and abs(S1 - inside * value) <= 1e-13 * S1 and abs(S2 - inside * value * value) <= 2e-13 * S2


def test_constant_near_the_largest_double():
    """The bimodal integrand's normalisation times N^d between 2^1023 and 2^1024,
    both peaks in one place: f w is of order one and so are the sums."""
    d, N, M = 2, 3, 6007
    a = 2.0 ** -511.6
    params = [a] + [0.0] * (2 * d)
    assert 1023 < np.log2(0.5 * N * N / np.pi) - 2 * np.log2(a) < 1024
    E = np.tile([0.0, 2.0 ** -511, 0.5, 1.0], (d, 1))
    v = Vegas(d, N, "bimodal", params, "fp64", seed=11)
    v.set_edges(E)
    ev = v.dump_events(0, M).cpu().numpy()
    b, delta = ev[:, :d], ev[:, d:2 * d]
    # f w = prod of (a sqrt(pi))^-1 e^{-(x/a)^2} N W over the events with both bins at the peak
    peak = (b == 0).all(axis=1)
    x = delta[peak] * 2.0 ** -511
    val = np.exp(-((x / a) ** 2)) / np.sqrt(np.pi) * (N * (2.0 ** -511 / a))
    o1 = val.prod(axis=1).sum()
    v.iterate(M, hist=False)
    S1 = v.last_iteration()[0]
    assert np.isfinite(o1) and abs(S1 - o1) <= 1e-12 * o1, (S1, o1)


@pytest.mark.parametrize("kind,at,more", [("bimodal", 1, {}), ("bimodal", 2, {}), ("bimodal", 5, {0: np.inf}), ("gauss", 1, {0: np.inf})])
@pytest.mark.parametrize("N", [20, 21])
def test_infinite_parameter_is_not_hidden(kind, at, more, N):
    """Infinite parameters set on the device whose exponent is not a number give
    results that are not numbers."""
    d = 3
    q = [0.3] + [0.4] * d + ([0.6] * d if kind == "bimodal" else [])
    v = Vegas(d, N, kind, q, "fp64")
    p = torch.tensor(q, dtype=torch.float64, device="cuda")
    p[at] = float("inf")
    for k, x in more.items():
        p[k] = x
    v.set_params_device(p)
    v.iterate(1000)
    S1, S2, H = v.last_iteration()
    assert np.isnan(S1) and np.isnan(S2) and np.isnan(H).any()
    assert np.isnan(v.dump_events(0, 10)[:, -1].cpu().numpy()).all()


@pytest.mark.parametrize("kind,at", [("gauss", 1), ("bimodal", 3), ("bimodal", 4), ("genz_disc", 0)])
def test_nan_parameter_in_event_records(kind, at):
    """A parameter that is not a number shows in the records of f as in the sums."""
    d = 3
    q = {"gauss": [0.3] + [0.4] * d, "bimodal": [0.3] + [0.4] * d + [0.6] * d, "genz_disc": [1.0] * d + [0.0] * d}[kind]
    v = Vegas(d, 20, kind, q, "fp64")
    p = torch.tensor(q, dtype=torch.float64, device="cuda")
    p[at] = float("nan")
    v.set_params_device(p)
    assert np.isnan(v.dump_events(0, 10)[:, -1].cpu().numpy()).all()


@pytest.mark.parametrize("c", [-3.0, -2e3, -1e10, -1e300])
def test_negative_genz_constant(c):
    """c is not checked where it comes from the device: f = nu e^{c x} falls then,
    down to 0, and never grows."""
    N, M, a = 20, 6007, 0.25
    v = Vegas(1, N, "genz_disc", [1.0, a], "fp64", seed=11)
    v.set_params_device(torch.tensor([c, a], dtype=torch.float64, device="cuda"))
    v.iterate(M)
    S1, S2, H = v.last_iteration()
    x = v.dump_events(0, M, iteration=0)[:, 2].cpu().numpy()
    with np.errstate(under="ignore", over="ignore"):
        f = np.where(x > a, c / np.expm1(c * (1.0 - a)) * np.exp(c * (x - a)), 0.0)
    # (x - a is rounded: c 2^-53 of f each)
    tol = max(1e-12, 4 * abs(c) * 2.0 ** -53) if abs(c) < 1e9 else 0.0
    assert abs(S1 - f.sum()) <= tol * f.sum() and abs(S2 - (f * f).sum()) <= 2 * tol * (f * f).sum()
    assert np.all(np.abs(H.sum() - (f * f).sum()) <= 2 * tol * (f * f).sum())


@pytest.mark.parametrize("c", [1e3, 1e7, 1e10, 1e300])
def test_genz_constant_beyond_the_range(c):
    """Where e^(c (1 - a)) overflows, the normalisation is 0 and the sums are not numbers."""
    v = Vegas(2, 20, "genz_disc", [1.0, 1.0, 0.25, 0.0], "fp64", seed=11)
    v.set_params_device(torch.tensor([1.0, c, 0.25, 0.0], dtype=torch.float64, device="cuda"))
    v.iterate(6007, hist=False)
    assert np.isnan(v.last_iteration()[0])


def _largest(prec, kind):
    """(d, N, replicas) whose table, histogram copies and 128 bytes of partial
    sums fit 160 KiB with less than another 128 bytes to spare."""
    entry = 8 if prec == "fp32_mixed" and kind not in ("bimodal",) else 16
    out = []
    for d in range(1, 65):
        for N in range(2, 256):
            for rep in (1, 2, 4, 8, 16):
                need = (d * N * entry + 127) // 128 * 128 + d * N * 8 * rep + 128
                if 160 * 1024 - 128 < need <= 160 * 1024:
                    out.append((d, N, rep))
    return out


@pytest.mark.parametrize("prec,kind", [("fp64", "gauss"), ("fp32_mixed", "gauss"), ("fp32_mixed", "bimodal"), ("fp64", "genz_disc")])
def test_replicas_that_just_fit(prec, kind):
    """Replica counts whose LDS fits by less than 128 bytes are accepted, and the
    launch gives the oracle's sums and bins, and without histograms the same bits."""
    sizes = _largest(prec, kind)
    assert len(sizes) >= 2
    tol = 1e-12 if prec == "fp64" else 1e-6
    for d, N, rep in sizes:
        if kind.startswith("genz"):
            params = [1.0] * d + [0.01] * d
        else:
            params = [0.4] + [0.5] * d * (2 if kind == "bimodal" else 1)
        v = Vegas(d, N, kind, params, prec, seed=11)
        v.set_hist_replicas(rep)
        v.iterate(9001)
        S1, S2, H = v.last_iteration()
        k = {"gauss": oracle.GAUSS, "bimodal": oracle.BIMODAL, "genz_disc": oracle.GENZ_DISC}[kind]
        pr = oracle.Problem(d, N, k, params, seed=11)
        o1, o2, Ho = oracle.accumulate(pr, np.tile(np.arange(N + 1) / N, (d, 1)), 0, 9001)
        t = tol * max(1.0, d / 8) if prec != "fp64" else tol
        assert abs(S1 - o1) <= t * o1 and abs(S2 - o2) <= t * o2, (d, N, rep)
        assert np.all(np.abs(H - Ho) <= t * Ho.sum(axis=1, keepdims=True)), (d, N, rep)
        w = Vegas(d, N, kind, params, prec, seed=11)
        w.set_hist_replicas(rep)
        w.iterate(9001, hist=False)
        assert w.last_iteration()[:2] == (S1, S2), (d, N, rep)


@pytest.mark.parametrize("d,N,prec,rep", [(11, 186, "fp64", 8), (62, 33, "fp64", 8), (22, 186, "fp32_mixed", 4)])
def test_user_replicas_that_just_fit(d, N, prec, rep):
    """The same for a runtime-compiled integrand (f = 1 on the uniform grid): S1 = M
    and every bin's S2 counts its events; one replica count more is refused."""
    v = Vegas(d, N, source="__device__ vegas_real vegas_integrand(const vegas_real* x, int dim, const double* p)\n"
                           "{ return 1; }", precision=prec)
    v.set_hist_replicas(rep)
    v.iterate(9001)
    S1, S2, H = v.last_iteration()
    assert abs(S1 - 9001) <= 1e-6 * 9001 and np.all(np.abs(H.sum(axis=1) - S2) <= 1e-9 * S2)
    with pytest.raises(VegasError):
        v.set_hist_replicas(2 * rep)


@pytest.mark.parametrize("d,N", [(2, 10), (16, 100)])
def test_captured_edges_follow_the_host_array(d, N):
    """vegas_set_edges recorded into a graph reads the caller's edges at each
    replay, whether they are few or many."""
    def grid(seed):
        r = np.random.default_rng(seed)
        E = np.zeros((d, N + 1))
        E[:, 1:] = np.cumsum(r.uniform(0.5, 1.5, (d, N)), axis=1)
        E /= E[:, -1:]
        E[:, -1] = 1.0
        return E
    params = [0.3] + [0.5] * d
    v = Vegas(d, N, "gauss", params, "fp64", seed=7)
    other = Vegas(d, N, "gauss", params, "fp64", seed=7)
    s = torch.cuda.Stream()
    v.stream = s
    host = grid(0)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        v.set_edges(host)
        v.iterate(5003)
    for rep in range(3):
        E = grid(rep)
        host[:] = E
        with torch.cuda.stream(s):
            g.replay()
        assert np.array_equal(v.edges(), E), rep
        S1 = v.last_iteration()[0]
        pr = oracle.Problem(d, N, oracle.GAUSS, params, seed=7)
        o1 = oracle.accumulate(pr, E, 0, 5003)[0]
        assert abs(S1 - o1) <= 1e-12 * o1, rep
        # eager work between replays
        other.set_edges(E)
        other.iterate(1000)
        torch.cuda.synchronize()


def test_captured_edges_made_by_the_call_are_kept():
    """A list of edges captured: the array made of it lives as long as the Vegas
    object, so the replays read its values."""
    v = Vegas(1, 4, "gauss", [0.3, 0.5], "fp64", seed=7)
    s = torch.cuda.Stream()
    v.stream = s
    E = [[0.0, 0.1, 0.4, 0.7, 1.0]]
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        v.set_edges(E)
    for _ in range(3):
        v.set_edges([[0.0, 0.2, 0.3, 0.9, 1.0]])
        with torch.cuda.stream(s):
            g.replay()
        assert v.edges().tolist() == E
    assert len(v._captured_edges) == 1


def test_tuning_cache_of_an_earlier_schedule(monkeypatch, tmp_path):
    """A stored choice under the tag of an earlier kind of schedule (fixed tiles)
    is not taken: the plan tunes and stores its own."""
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("VEGAS_BATCH_TUNE_CACHE", str(path))
    probs = [{"dim": d, "n_bins": 20, "params": [0.2] + [0.5] * d, "n_events": 20_000, "precision": "fp64"} for d in (2, 3, 6)]
    assert not VegasBatch(probs, 3, 2).schedule()["from_cache"]
    line = path.read_text()
    tag = line.split()[0]
    assert tag.startswith("vegas-batch-v")
    path.write_text(line.replace(tag, "vegas-batch-v1"))
    assert not VegasBatch(probs, 3, 2).schedule()["from_cache"]
    assert len(path.read_text().splitlines()) == 2
    assert VegasBatch(probs, 3, 2).schedule()["from_cache"]


def test_reads_behind_long_runs():
    """Results, edges and sums asked for while more than the millisecond for which
    the host looks for the mark is still queued are those of the queued work,
    and so are the next reads, which find the mark."""
    d, N = 8, 50
    params = [0.2] + [0.45] * d
    v = Vegas(d, N, "gauss", params, "fp64", seed=3)
    M = 1_000_000_000
    v.timing_enable()
    reads = []
    for k, read in enumerate((v.result, v.edges, v.last_iteration)):
        v.iterate(M, refine=True)
        reads.append(read())
        v.iterate(1000, hist=False)
        assert v.result()["n_iter"] == 2 * k + 2
    ms = v.timing_read()[0] / 3
    assert ms > 2.0, ms
    w = Vegas(d, N, "gauss", params, "fp64", seed=3)
    for k in range(3):
        w.iterate(M, refine=True)
        torch.cuda.synchronize()
        got = (w.result, w.edges, w.last_iteration)[k]()
        if k == 0:
            assert abs(got["integral"] - reads[0]["integral"]) <= 1e-12 * abs(got["integral"])
            assert got["n_events"] == reads[0]["n_events"] == M
        elif k == 1:
            assert np.max(np.abs(got - reads[1])) <= 1e-9
        else:
            assert abs(got[0] - reads[2][0]) <= 1e-9 * got[0]
        w.iterate(1000, hist=False)


def test_device_buffers_are_final_after_a_read():
    """After result(), edges() or last_iteration() returns, work on another stream,
    ordered behind nothing, sees what the call's stream has done."""
    d, N, M = 4, 50, 200_003
    s, other = torch.cuda.Stream(), torch.cuda.Stream()
    v = Vegas(d, N, "gauss", [0.2] + [0.45] * d, "fp64", seed=3)
    torch.cuda.synchronize()
    v.stream = s
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for k in range(50):
        v.iterate(M, refine=True)
        E = S = None
        if k % 3 == 0:
            r = v.result()
        elif k % 3 == 1:
            E = v.edges()
        else:
            S = v.last_iteration()
        v.stream = other
        v.last_iteration_device(out)
        other.synchronize()
        got = out.cpu().numpy()
        again = v.last_iteration()
        assert got[0] == again[0] / M, k
        if E is not None:
            assert np.array_equal(E, v.edges()), k
        elif S is not None:
            assert S[0] == again[0] and np.array_equal(S[2], again[2]), k
        else:
            assert r["last_integral"] == got[0], k
        other.synchronize()
        v.stream = s


def test_dear_user_integrands_keep_their_waves():
    """A runtime-compiled integrand is not held to one block of 512 threads a compute
    unit for the sake of histogram replicas where its registers admit two."""
    dear = """__device__ vegas_real vegas_integrand(const vegas_real* x, int dim, const double* p)
{ vegas_real s = 0, q = 1;
  for (int i = 0; i < VEGAS_DIM; ++i) { s += sin(x[i] * vegas_real(3)); q *= vegas_real(1) + x[i] * x[i]; }
  return exp(-s * s) / q; }"""
    for d, N in ((16, 50), (20, 100), (10, 200)):
        v = Vegas(d, N, source=dear, precision="fp32_mixed")
        info = v.launch_info()
        assert info["blocks_per_cu"] * info["threads"] >= 1024, info
        v.iterate(3000)
        assert np.isfinite(v.last_iteration()[0])


@pytest.mark.parametrize("kind,d,N,prec", [("genz_peak", 16, 37, "fp32_mixed"), ("genz_peak", 9, 50, "fp64"), ("gauss", 12, 37, "fp64"),
                                           ("bimodal", 9, 50, "fp32_mixed")])
def test_one_large_block_beyond_eight_dimensions(kind, d, N, prec):
    """The histogram kernels beyond d = 8 are compiled for one block of 1024 threads
    a compute unit and are not launched as two of 768."""
    q = {"gauss": [0.2] + [0.5] * d, "bimodal": [0.2] + [0.4] * d + [0.6] * d, "genz_peak": [1.0] * d + [0.1] * d}[kind]
    info = Vegas(d, N, kind, q, prec).launch_info()
    assert info["threads"] != 768, info
