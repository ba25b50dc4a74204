"""GPU parity of LAMA-PD and LAMA-FD (Algorithm 1; Section IV with the
normalisation of the proof of Lemma 2) against the FP64 oracle, element by
element on the same seeded inputs: max over systems of
||z - z_ref||_inf / ||z_ref||_inf <= 1e-4 and sigma2 within 0.05 dB, for
QPSK, 16-QAM and 64-QAM and T_max = 1, 2, 3, both one-pass forms, across
several row blocks, ragged rows and uneven clusters."""
import numpy as np
import pytest

import oracle
from paper_1808_04473_amd import synth
from gpu_util import TOL_DB, TOL_Z, dev, host, max_db_err, max_rel_err, need_gpu, torch

pytestmark = pytest.mark.gpu

MODS = {4: "qpsk", 16: "16qam", 64: "64qam"}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def run(mode, b, t_max, qam, prec, nu=None, info=False):
    from paper_1808_04473_amd import api
    H, y = dev(b.H), dev(b.y)
    if mode == "pd":
        out = api.eq_pd_lama(H, y, b.n0, b.cluster_off, t_max=t_max, qam=qam, precision=prec, return_info=info)
    else:
        out = api.eq_fd_lama(H, y, b.n0, b.cluster_off, t_max=t_max, qam=qam, precision=prec, return_info=info,
                             nu=None if nu is None else dev(nu.astype(np.float32)))
    torch.cuda.synchronize()
    return [host(t) for t in out]


def ref(mode, b, t_max, qam, nu=None):
    if mode == "pd":
        return oracle.eq_pd_lama(b.H, b.y, b.n0, b.cluster_off, t_max, qam)
    return oracle.eq_fd_lama(b.H, b.y, b.n0, b.cluster_off, t_max, qam, nu=nu)


SHAPES = [(64, 32, 4, 2), (200, 256, 16, 8), (24, 1024, 32, 16), (13, 37, 5, [0, 5, 20, 37]),
          (9, 100, 24, [0, 40, 100])]


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("qam", [4, 16, 64])
@pytest.mark.parametrize("t_max", [1, 2, 3])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"W{s[0]}B{s[1]}U{s[2]}")
def test_lama_matches_oracle(mode, prec, qam, t_max, shape):
    W, B, U, C = shape
    off = C if isinstance(C, list) else None
    nc = len(C) - 1 if isinstance(C, list) else C
    b = synth.make_batch(W, B, U, nc, 10.0, MODS[qam], seed=W + B + qam, cluster_off=off)
    z, s2, info = run(mode, b, t_max, qam, prec, info=True)
    zr, sr = ref(mode, b, t_max, qam)
    ez, es = max_rel_err(z, zr), max_db_err(s2, sr)
    print(f"lama {mode} {prec} qam{qam} T={t_max} W={W} B={B} U={U}: z err {ez:.2e}, sigma2 {es:.5f} dB", flush=True)
    assert ez <= TOL_Z[prec], ez
    assert es <= TOL_DB, es
    assert (info == 0).all()


def test_lama_fd_given_weights():
    b = synth.make_batch(21, 96, 8, 3, 10.0, "16qam", seed=31)
    nu = np.random.default_rng(2).uniform(0.1, 1.0, size=(21, 3, 8))
    z, s2 = run("fd", b, 3, 16, "fp32", nu=nu)
    zr, sr = ref("fd", b, 3, 16, nu=nu)
    assert max_rel_err(z, zr) <= TOL_Z["fp32"]
    assert max_db_err(s2, sr) <= TOL_DB


@pytest.mark.filterwarnings("ignore:invalid value:RuntimeWarning")  # the oracle on the NaN input
@pytest.mark.parametrize("mode", ["pd", "fd"])
def test_lama_non_finite_input(mode):
    b = synth.make_batch(8, 64, 8, 2, 10.0, "16qam", seed=32)
    b.y[5, 3] = np.complex64(complex(np.inf, 0))
    z, s2, info = run(mode, b, 2, 16, "fp32", info=True)
    assert np.isnan(z[5]).all()
    bad = info[5] if mode == "pd" else info[5, 0]
    assert bad == -1
    keep = np.arange(8) != 5
    zr, sr = ref(mode, b, 2, 16)
    assert max_rel_err(z[keep], zr[keep]) <= TOL_Z["fp32"]


def test_lama_beats_lmmse_on_qpsk():
    """At B = 256, U = 64 (beta = 1/4), QPSK, SNR 6 dB, LAMA-PD after a few
    iterations has a lower empirical MSE than L-MMSE (Section III-C: LAMA
    approaches the individually optimal detector where L-MMSE does not)."""
    from paper_1808_04473_amd import api
    b = synth.make_batch(400, 256, 32, 8, 6.0, "qpsk", seed=33)
    H, y = dev(b.H), dev(b.y)
    zl, _ = api.eq_pd_lama(H, y, b.n0, b.cluster_off, t_max=6, qam=4)
    zm, _ = api.eq_pd(H, y, b.n0, b.cluster_off)
    torch.cuda.synchronize()
    zl, zm = host(zl), host(zm)
    # L-MMSE is biased: compare after removing its common gain
    g = np.vdot(b.s.ravel(), zm.ravel()) / np.vdot(b.s.ravel(), b.s.ravel())
    mse_l = np.mean(np.abs(zl - b.s) ** 2)
    mse_m = np.mean(np.abs(zm / g - b.s) ** 2)
    assert mse_l < mse_m, (mse_l, mse_m)


# ---------------------------------------------------------------- several receive vectors
SYM_SHAPES = [(30, 256, 16, 8, 14), (6, 130, 24, [0, 60, 130], 40), (9, 37, 5, [0, 5, 20, 37], 3)]


def _sym_batch(shape, qam, seed):
    W, B, U, C, S = shape
    off = C if isinstance(C, list) else None
    nc = len(C) - 1 if isinstance(C, list) else C
    return synth.make_symbol_batch(W, B, U, nc, S, 10.0, MODS[qam], seed=seed, cluster_off=off)


def _check_sym(mode, b, t_max, qam, prec, nu=None):
    from paper_1808_04473_amd import api
    fn = api.eq_pd_lama_sym if mode == "pd" else api.eq_fd_lama_sym
    kw = {} if mode == "pd" else {"nu": None if nu is None else dev(nu.astype(np.float32))}
    z, s2, info = fn(dev(b.H), dev(b.Y), b.n0, b.cluster_off, t_max=t_max, qam=qam, precision=prec,
                     return_info=True, **kw)
    torch.cuda.synchronize()
    z, s2, info = host(z), host(s2), host(info)
    assert (info == 0).all()
    rf = oracle.eq_pd_lama if mode == "pd" else oracle.eq_fd_lama
    worst = 0.0
    for s in range(b.Y.shape[1]):
        if mode == "pd":
            zr, sr = rf(b.H, b.Y[:, s], b.n0, b.cluster_off, t_max, qam)
        else:
            zr, sr = rf(b.H, b.Y[:, s], b.n0, b.cluster_off, t_max, qam, nu=nu)
        ez = max_rel_err(z[:, s], zr)
        worst = max(worst, ez)
        assert ez <= TOL_Z[prec], (s, ez)
        assert max_db_err(s2[:, s], sr) <= TOL_DB
    return worst


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("qam", [4, 16])
@pytest.mark.parametrize("t_max", [1, 3])
@pytest.mark.parametrize("shape", SYM_SHAPES, ids=lambda s: f"W{s[0]}B{s[1]}U{s[2]}S{s[4]}")
def test_lama_symbols_match_oracle(mode, prec, qam, t_max, shape):
    """eq_pd_lama_sym / eq_fd_lama_sym: every vector against the oracle's
    LAMA on that vector alone (z and its own sigma2)."""
    b = _sym_batch(shape, qam, seed=shape[0] + qam + t_max)
    worst = _check_sym(mode, b, t_max, qam, prec)
    print(f"lama sym {mode} {prec} qam{qam} T={t_max} {shape}: z err {worst:.2e}", flush=True)


def test_lama_symbols_fd_given_weights():
    b = _sym_batch((11, 96, 8, 3, 9), 16, seed=51)
    nu = np.random.default_rng(6).uniform(0.1, 1.0, size=(11, 3, 8))
    _check_sym("fd", b, 2, 16, "fp32", nu=nu)


@pytest.mark.parametrize("mode", ["pd", "fd"])
def test_lama_symbols_non_finite_vector(mode):
    """A NaN in one receive vector gives NaN for that vector only."""
    from paper_1808_04473_amd import api
    b = _sym_batch((6, 64, 8, 2, 5), 16, seed=52)
    b.Y[2, 3, 17] = np.complex64(complex(np.nan, 0.0))
    fn = api.eq_pd_lama_sym if mode == "pd" else api.eq_fd_lama_sym
    z, s2 = fn(dev(b.H), dev(b.Y), b.n0, b.cluster_off, t_max=2, qam=16)
    torch.cuda.synchronize()
    z = host(z)
    assert np.isnan(z[2, 3]).all()
    keep = np.ones(z.shape[:2], bool)
    keep[2, 3] = False
    assert np.isfinite(z[keep]).all()


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("shape,t_max", [
    ((7, 40, 8, [0, 13, 25, 40], 2), 2), ((7, 40, 8, [0, 13, 25, 40], 2), 3),
    ((5, 67, 16, [0, 17, 33, 50, 67], 3), 4), ((5, 67, 16, [0, 17, 33, 50, 67], 4), 4),
    ((4, 96, 17, 2, 2), 4), ((4, 96, 17, 2, 2), 5), ((3, 100, 32, [0, 34, 66, 100], 3), 7)])
def test_lama_symbols_few_vectors(mode, prec, shape, t_max):
    """Vector and iteration counts on both sides of the line between a kernel
    run per vector and the 16-vector tiles."""
    _check_sym(mode, _sym_batch(shape, 16, seed=61), t_max, 16, prec)


@pytest.mark.parametrize("mode", ["pd", "fd"])
def test_lama_symbols_few_vectors_non_finite(mode):
    """As for the tiles: NaN for that vector only, and no system code."""
    from paper_1808_04473_amd import api
    b = _sym_batch((6, 64, 8, 2, 2), 16, seed=62)
    b.Y[2, 1, 17] = np.complex64(complex(np.nan, 0.0))
    fn = api.eq_pd_lama_sym if mode == "pd" else api.eq_fd_lama_sym
    z, s2, info = fn(dev(b.H), dev(b.Y), b.n0, b.cluster_off, t_max=3, qam=16, return_info=True)
    torch.cuda.synchronize()
    z = host(z)
    assert np.isnan(z[2, 1]).all() and (host(info) == 0).all()
    z[2, 1] = 0
    assert np.isfinite(z).all()


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("S", [1, 2, 3, 4, 5, 8, 9, 10, 11])
@pytest.mark.parametrize("shape", [(5, 80, 5, [0, 20, 41, 60, 80]), (3, 260, 16, [0, 64, 129, 193, 260]), (3, 150, 17, 2),
                                   (3, 260, 32, [0, 130, 260])], ids=lambda s: f"B{s[1]}U{s[2]}")
def test_lama_symbols_many_iterations(mode, prec, S, shape):
    """Vector after vector in the lane groups, at the vector counts where its
    stream changes form, and the tiles on the other side of the line."""
    _check_sym(mode, _sym_batch(shape + (S,), 4, seed=63 + S), 12, 4, prec)


@pytest.mark.parametrize("S,t_max", [(2, 6), (3, 6), (5, 8)])
def test_lama_symbols_systems_per_wave(S, t_max):
    """As many PD systems as fill the lane groups of a wave."""
    _check_sym("pd", _sym_batch((6200, 24, 5, 1, S), 4, seed=64), t_max, 4, "fp32")


def test_lama_symbols_many_iterations_given_weights():
    b = _sym_batch((7, 120, 8, 3, 6), 4, seed=65)
    nu = np.random.default_rng(7).uniform(0.1, 1.0, size=(7, 3, 8))
    _check_sym("fd", b, 16, 4, "fp32", nu=nu)


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("U", [8, 32])
def test_lama_symbols_of_an_interval_share_one_pass(mode, U):
    """14 vectors are equalised from one Gram whatever the iteration count: in
    the tile, where a vector's result does not depend on the others'."""
    from paper_1808_04473_amd import api
    fn = api.eq_pd_lama_sym if mode == "pd" else api.eq_fd_lama_sym
    b = _sym_batch((6, 4 * U, U, 2, 16), 4, seed=66)
    H, Y = dev(b.H), dev(b.Y)
    for t_max in (16, 40):
        z, s2 = fn(H, Y, b.n0, b.cluster_off, t_max=t_max, qam=4)
        z14, s14 = fn(H, Y[:, :14].contiguous(), b.n0, b.cluster_off, t_max=t_max, qam=4)
        assert torch.equal(z14, z[:, :14]) and torch.equal(s14, s2[:, :14])


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("U", [5, 16, 20])
@pytest.mark.parametrize("t_max", [1, 3])
def test_lama_symbols_of_one_vector_is_the_single_call(mode, U, t_max):
    from paper_1808_04473_amd import api
    b = _sym_batch((9, 3 * U + 6, U, 3 if mode == "fd" else 1, 1), 16, seed=67)
    args = (b.n0, b.cluster_off, t_max, 16)
    one, sym = (api.eq_pd_lama, api.eq_pd_lama_sym) if mode == "pd" else (api.eq_fd_lama, api.eq_fd_lama_sym)
    z, s2 = one(dev(b.H), dev(b.Y[:, 0]), *args)
    zs, ss = sym(dev(b.H), dev(b.Y), *args)
    assert torch.equal(zs[:, 0], z) and torch.equal(ss[:, 0], s2)


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("S", [1, 3, 6])
def test_lama_symbols_non_finite_vector_by_vector(mode, S):
    """As for the tiles: NaN for that vector only, and no system code."""
    from paper_1808_04473_amd import api
    b = _sym_batch((6, 64, 8, 4, S), 4, seed=68)
    b.Y[2, S - 1, 17] = np.complex64(complex(np.nan, 0.0))
    fn = api.eq_pd_lama_sym if mode == "pd" else api.eq_fd_lama_sym
    z, s2, info = fn(dev(b.H), dev(b.Y), b.n0, b.cluster_off, t_max=30, qam=4, return_info=True)
    torch.cuda.synchronize()
    z = host(z)
    assert np.isnan(z[2, S - 1]).all() and (host(info) == 0).all()
    z[2, S - 1] = 0
    assert np.isfinite(z).all()


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("mode,shape", [
    ("pd", (8300, 16, 3, 1, 4)), ("pd", (8300, 16, 3, 1, 5)), ("pd", (2500, 48, 20, 1, 2)), ("pd", (2500, 48, 20, 1, 5)),
    ("fd", (1100, 105, 5, 5, 2)), ("fd", (1100, 105, 5, 7, 4)), ("fd", (700, 104, 5, 13, 5)), ("fd", (700, 120, 20, 3, 2)),
    ("fd", (700, 160, 20, 4, 5)), ("fd", (300, 245, 17, 7, 8)), ("fd", (20, 104, 5, 13, 3)), ("fd", (20, 245, 17, 7, 3)),
], ids=lambda v: v if isinstance(v, str) else f"W{v[0]}U{v[2]}C{v[3]}S{v[4]}")
def test_lama_symbols_waves_and_vectors(mode, shape, prec):
    """Vector after vector: each number of vectors per wave, and of waves per
    FD subcarrier, whose rounds do not divide among them.  Up to 4 vectors (2
    above 16 users) the sums are the single call's, bit for bit; more come from
    the tiles.  Among thousands of systems of 3 users the iterations amplify
    rounding by up to 1e4, in the single call too: each system's bound is
    scaled by what the oracle makes of a relative change of H and y by 1e-6."""
    from paper_1808_04473_amd import api
    b = _sym_batch(shape, 4, seed=69)
    args = (b.n0, b.cluster_off, 4, 4)
    one, sym = (api.eq_pd_lama, api.eq_pd_lama_sym) if mode == "pd" else (api.eq_fd_lama, api.eq_fd_lama_sym)
    rf = oracle.eq_pd_lama if mode == "pd" else oracle.eq_fd_lama
    z, s2 = sym(dev(b.H), dev(b.Y), *args, precision=prec)
    H, Y = b.H.astype(np.complex128), b.Y.astype(np.complex128)
    rng = np.random.default_rng(70)
    pert = [[x * (1 + 1e-6 * rng.standard_normal(x.shape)) for x in (H, Y)] for _ in range(2)]
    for s in range(b.Y.shape[1]):
        if shape[4] <= (4 if shape[2] <= 16 else 2) or shape[0] == 20:
            z1, s21 = one(dev(b.H), dev(b.Y[:, s]), *args, precision=prec)
            assert torch.equal(z[:, s], z1) and torch.equal(s2[:, s], s21)
        zr, sr = rf(H, Y[:, s], *args)
        ref = np.abs(zr).max(1)
        err = np.abs(host(z[:, s]) - zr).max(1) / ref
        db = np.abs(10 * np.log10(host(s2[:, s]) / sr)).max(1)
        kz, ks = np.ones(len(zr)), np.ones(len(zr))
        for Hp, Yp in pert:
            zp, sp = rf(Hp, Yp[:, s], *args)
            kz = np.maximum(kz, np.abs(zp - zr).max(1) / ref / 1e-6)
            ks = np.maximum(ks, np.abs(np.log(sp / sr)).max(1) / 1e-6)
        assert (err <= TOL_Z[prec] * kz).all(), (s, (err / kz).max())
        assert (db <= TOL_DB * ks).all(), (s, (db / ks).max())


@pytest.mark.parametrize("U", [4, 20])
@pytest.mark.parametrize("S", [2, 17])
def test_lama_symbols_fd_info_is_of_the_gram_itself(U, S):
    """A Gram that is finite, and not so divided by w_c = 1/2, is no bad input:
    the single call's code, of the vector-by-vector calls and of the tiles."""
    from paper_1808_04473_amd import api
    b = _sym_batch((6, 64, U, 2, S), 4, seed=71)
    H = b.H.copy()
    H[2] *= 2.8e18 / np.abs(H[2])  # 32 |h|^2 = 2.5e38
    H[4, 5, 1] = np.inf
    args = (b.n0, b.cluster_off, 2, 4)
    _, _, one = api.eq_fd_lama(dev(H), dev(b.Y[:, 0]), *args, return_info=True)
    _, _, sym = api.eq_fd_lama_sym(dev(H), dev(b.Y), *args, return_info=True)
    want = np.zeros((6, 2), np.int32)
    want[4, 0] = -1
    assert (host(one) == want).all() and (host(sym) == want).all()
