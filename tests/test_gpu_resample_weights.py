"""GPU parity of the one-shot resampling entry point (smc_resample_weights:
caller-held log-weights in, normalisation summary and sorted ancestors out)
against the oracle's normalisation and resampling (Section 2.1; Eq.
resample), for every scheme, ragged sizes, zero weights, the decision rule
and the error path."""
import numpy as np
import pytest

from gpu_helpers import assert_ancestors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SCHEMES = {"multinomial": 0, "systematic": 1, "stratified": 2}


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_5583_amd import _lib
    _lib.load()
    return _lib


def _weights(n, seed, zeros=0.0):
    rng = np.random.default_rng(seed)
    lw = rng.normal(0.0, 3.0, n) - 700.0          # far from 0: the max shift matters
    if zeros:
        lw[rng.random(n) < zeros] = -np.inf
    return lw


def _run(L, lw, scheme, threshold=0.5, force=0, seed=17, step=5, problem=0, anc_init=None):
    n = lw.size
    d_lw = torch.as_tensor(lw, device="cuda")
    anc = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    if anc_init is not None:
        anc.copy_(torch.as_tensor(anc_init, dtype=torch.int32))
    summary = torch.zeros(5, dtype=torch.float64, device="cuda")
    nb = L.smc_resample_weights_workspace(n, SCHEMES[scheme])
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    L.smc_resample_weights(d_lw.data_ptr(), n, SCHEMES[scheme], threshold, force, seed, step,
                           problem, anc.data_ptr(), summary.data_ptr(), ws.data_ptr(), nb,
                           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return anc.cpu().numpy().astype(np.int64), summary.cpu().numpy()


@pytest.mark.parametrize("scheme", list(SCHEMES))
@pytest.mark.parametrize("n", [1, 1000, 70001, 1 << 20])
def test_matches_oracle(L, orc, scheme, n):
    lw = _weights(n, n + len(scheme), zeros=0.2 if n > 1 else 0.0)
    anc, sm = _run(L, lw, scheme, force=1, seed=17, step=5, problem=3)
    Lo, L2o, esso = orc.normalise(lw)
    assert abs(sm[0] - Lo) <= 1e-12 * max(1.0, abs(Lo))
    assert abs(sm[1] - L2o) <= 1e-12 * max(1.0, abs(L2o))
    assert abs(sm[2] - esso) <= 1e-12 * esso
    assert sm[3] == 1.0 and sm[4] == 0.0
    anc_o, S_o, u_o = orc.resample(scheme, 17, 5, lw, p=3)
    assert_ancestors(anc, anc_o, S_o, u_o, what="%s n=%d" % (scheme, n))
    assert np.all(np.isfinite(lw[anc]))           # zero weights are never chosen


def test_decision_rule(L, orc):
    n = 5000
    lw = _weights(n, 3)
    _, _, ess = orc.normalise(lw)
    assert ess < 0.5 * n
    # ESS below threshold N: resample; above: ancestors untouched
    anc, sm = _run(L, lw, "systematic", threshold=1.2 * ess / n)
    assert sm[3] == 1.0
    keep = np.arange(n)
    anc, sm = _run(L, lw, "systematic", threshold=0.5 * ess / n, anc_init=keep)
    assert sm[3] == 0.0 and np.array_equal(anc, keep)
    anc, sm = _run(L, lw, "systematic", threshold=0.0, anc_init=keep)   # never
    assert sm[3] == 0.0 and np.array_equal(anc, keep)
    anc, sm = _run(L, lw, "systematic", threshold=1.0)                  # always
    assert sm[3] == 1.0
    anc_o, S_o, u_o = orc.resample("systematic", 17, 5, lw)
    assert_ancestors(anc, anc_o, S_o, u_o)


def test_all_zero_weights_report_an_error(L):
    lw = np.full(3000, -np.inf)
    keep = np.arange(3000)
    anc, sm = _run(L, lw, "systematic", force=1, anc_init=keep)
    assert sm[3] == 0.0 and sm[4] != 0.0
    assert np.array_equal(anc, keep)


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 5000, 262144, 262145])
@pytest.mark.parametrize("case", ["plain", "zeros", "all zero", "nan", "inf", "kept"])
def test_launch_forms_agree(L, orc, n, case):
    # systematic resampling in one launch (one tile), two (up to 256 tiles) and
    # by the general path: the summary is that of the stratified scheme, which
    # always takes the general path, bit for bit; the ancestors the oracle's
    lw = _weights(n, n, zeros=0.3 if case == "zeros" and n > 1 else 0.0)
    if case == "all zero":
        lw[:] = -np.inf
    if case in ("nan", "inf"):
        lw[n // 2] = np.nan if case == "nan" else np.inf
    force = 0 if case == "kept" else 1
    keep = np.full(n, 7)
    anc, sm = _run(L, lw, "systematic", threshold=0.0, force=force, anc_init=keep)
    _, ref = _run(L, lw, "stratified", threshold=0.0, force=force, anc_init=keep)
    assert np.array_equal(sm, ref, equal_nan=True)
    if sm[3] == 0.0:
        assert np.array_equal(anc, keep)
    elif case in ("plain", "zeros"):
        anc_o, S_o, u_o = orc.resample("systematic", 17, 5, lw)
        assert_ancestors(anc, anc_o, S_o, u_o)


@pytest.mark.parametrize("scheme", ["stratified", "multinomial"])
@pytest.mark.parametrize("n,case", [(300000, "one"), (4097, "one"), (5121, "last"),
                                    (100003, "block"), (262144, "few"), (70001, "wide")])
def test_concentrated_weights(L, orc, n, scheme, case):
    # tiles that own many times their share of the slots: more than a round of
    # chunk ends (255 chunks of 1024), one particle, a tile or a few particles
    # with all the weight, log-weights far apart
    rng = np.random.default_rng(n)
    lw = rng.normal(0.0, 1.0, n)
    if case == "wide":
        lw *= 10.0
    else:
        heavy = {"one": [n // 2], "last": [n - 1], "block": np.arange(n // 3, n // 3 + 900),
                 "few": rng.integers(0, n, 7)}[case]
        lw -= 45.0
        lw[heavy] += 45.0
    anc, sm = _run(L, lw, scheme, threshold=0.0, force=1)
    anc_o, S_o, u_o = orc.resample(scheme, 17, 5, lw)
    assert sm[3] == 1.0
    assert_ancestors(anc, anc_o, S_o, u_o)


@pytest.mark.parametrize("scheme", ["stratified", "multinomial"])
def test_concentrated_weights_cost_their_stores(L, scheme):
    # one particle with all the weight of a million: one workgroup writes every
    # slot, without drawing or searching for each (ten times the call with even
    # weights at most; with them sixty to eighty times)
    n, code = 1 << 20, L.SCHEMES[scheme]
    nb = L.smc_resample_weights_workspace(n, code)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    anc = torch.zeros(n, dtype=torch.int32, device="cuda")
    summary = torch.zeros(5, dtype=torch.float64, device="cuda")
    even = torch.zeros(n, dtype=torch.float64, device="cuda")
    one = even.clone()
    one[n // 2] = 100.0
    stream = torch.cuda.current_stream().cuda_stream
    ms = [[], []]
    for r in range(12):
        for q, lw in enumerate((even, one)):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                L.smc_resample_weights(lw.data_ptr(), n, code, 0.0, 1, 1, 3, 0, anc.data_ptr(),
                                       summary.data_ptr(), ws.data_ptr(), nb, stream)
            b.record()
            b.synchronize()
            if r >= 2:
                ms[q].append(a.elapsed_time(b))
    t = [float(np.median(v)) for v in ms]
    assert t[1] < 10.0 * t[0], t


@pytest.mark.parametrize("scheme", ["stratified", "multinomial"])
@pytest.mark.parametrize("part", [9, 16, 33, 64, 250])
def test_weights_on_a_part_of_the_population(L, orc, scheme, part):
    # a stretch of the particles with all the weight, equal: every chunk of the
    # slots has many owners and each slot is searched, in the last tile of the
    # stretch up to the tile's end
    n = 70001
    for first in (n // 5, n - n // part):
        lw = np.full(n, -800.0)
        lw[first:first + n // part] = 0.0
        anc, sm = _run(L, lw, scheme, threshold=0.0, force=1)
        anc_o, S_o, u_o = orc.resample(scheme, 17, 5, lw)
        assert_ancestors(anc, anc_o, S_o, u_o)


def test_invalid_arguments(L):
    from paper_1306_5583_amd import SmcError
    lw = torch.zeros(100, dtype=torch.float64, device="cuda")
    anc = torch.zeros(100, dtype=torch.int32, device="cuda")
    sm = torch.zeros(5, dtype=torch.float64, device="cuda")
    nb = L.smc_resample_weights_workspace(100, 1)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    with pytest.raises(SmcError):      # workspace too small
        L.smc_resample_weights(lw.data_ptr(), 100, 1, 0.5, 1, 1, 1, 0, anc.data_ptr(),
                               sm.data_ptr(), ws.data_ptr(), nb - 1, s)
    with pytest.raises(SmcError):      # unknown scheme
        L.smc_resample_weights(lw.data_ptr(), 100, 9, 0.5, 1, 1, 1, 0, anc.data_ptr(),
                               sm.data_ptr(), ws.data_ptr(), nb, s)
    with pytest.raises(SmcError):      # misaligned log-weights
        L.smc_resample_weights(lw.data_ptr() + 8, 99, 1, 0.5, 1, 1, 1, 0, anc.data_ptr(),
                               sm.data_ptr(), ws.data_ptr(), nb, s)
