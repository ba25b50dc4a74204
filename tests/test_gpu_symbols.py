"""GPU parity of eq_pd_sym / eq_fd_sym (several receive vectors per channel
matrix, Section VI-B) against the FP64 oracle, element by element on the
same seeded inputs, per receive vector: max over (w, s) of
||z_ws - z_ref_ws||_inf / ||z_ref_ws||_inf <= 1e-4, sigma2 within 0.05 dB.

Cases span several row blocks and a ragged tail (B not a multiple of the
block rows, uneven clusters), symbol counts below, at and above one tile
(16 vectors for U <= 16, 32 above), one vector, FD with given weights, a
non-finite receive vector, the FP64 re-solve queue, and the launch size the
benchmark times (sampled outputs plus properties of the whole batch)."""
import numpy as np
import pytest

import oracle
from paper_1808_04473_amd import synth
from gpu_util import TOL_DB, TOL_Z, dev, host, max_db_err, max_rel_err, need_gpu, torch

pytestmark = pytest.mark.gpu

PRECS = ["fp32", "bf16x3"]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def run(mode, b, prec, nu=None, info=False):
    from paper_1808_04473_amd import api
    H, Y = dev(b.H), dev(b.Y)
    if mode == "pd":
        out = api.eq_pd_sym(H, Y, b.n0, b.cluster_off, precision=prec, return_info=info)
    else:
        out = api.eq_fd_sym(H, Y, b.n0, b.cluster_off, precision=prec, return_info=info,
                            nu=None if nu is None else dev(nu.astype(np.float32)))
    torch.cuda.synchronize()
    return [host(t) for t in out]


def ref(mode, b, nu=None):
    if mode == "pd":
        return oracle.eq_pd_symbols(b.H, b.Y, b.n0, b.cluster_off)
    return oracle.eq_fd_symbols(b.H, b.Y, b.n0, b.cluster_off, nu=nu)


def check(mode, b, prec, nu=None):
    z, s2 = run(mode, b, prec, nu)
    zr, sr = ref(mode, b, nu)
    assert z.shape == zr.shape
    ez, es = max_rel_err(z, zr), max_db_err(s2, sr)
    print(f"{mode} {prec} W={b.H.shape[0]} B={b.H.shape[1]} U={b.H.shape[2]} S={b.Y.shape[1]} "
          f"C={len(b.cluster_off) - 1}: z err {ez:.2e}, sigma2 {es:.4f} dB", flush=True)
    assert ez <= TOL_Z[prec], ez
    assert es <= TOL_DB, es


# (W, B, U, C or offsets, S)
SHAPES = [
    (64, 32, 4, 2, 14),                      # the small workload, 14 symbols
    (40, 256, 16, 8, 14),                    # the paper's B=256, C=8, U=16
    (8, 1024, 32, 16, 14),                   # B=1024, C=16, U=32
    (13, 37, 5, [0, 5, 20, 37], 3),          # ragged rows and clusters
    (9, 100, 16, [0, 33, 34, 100], 16),      # exactly one tile, a one-row cluster
    (7, 96, 12, 4, 17),                      # two tiles, ragged symbol tail
    (5, 130, 24, [0, 60, 130], 40),          # U > 16: tiles of 32, tail of 8
    (6, 48, 8, 3, 1),                        # one vector
    (5, 64, 32, 2, 33),                      # full 32-user tile, two tiles
]


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"W{s[0]}B{s[1]}U{s[2]}S{s[4]}")
def test_symbols_match_oracle(mode, prec, shape):
    W, B, U, C, S = shape
    off = C if isinstance(C, list) else None
    nc = len(C) - 1 if isinstance(C, list) else C
    b = synth.make_symbol_batch(W, B, U, nc, S, 10.0, "16qam", seed=W * 1000 + B + S, cluster_off=off)
    check(mode, b, prec)


@pytest.mark.parametrize("prec", PRECS)
def test_fd_symbols_given_weights(prec):
    b = synth.make_symbol_batch(11, 96, 8, 3, 9, 5.0, "qpsk", seed=77)
    nu = np.random.default_rng(5).uniform(0.1, 1.0, size=(11, 3, 8))
    check("fd", b, prec, nu=nu)


@pytest.mark.parametrize("mode", ["pd", "fd"])
def test_one_vector_equals_single_vector_call(mode):
    """nsym = 1 gives what eq_pd / eq_fd give for the same y (both within
    the gate of the oracle, and close to each other)."""
    from paper_1808_04473_amd import api
    b = synth.make_symbol_batch(50, 256, 16, 8, 1, 10.0, "16qam", seed=8)
    z1, s1 = run(mode, b, "fp32")
    H, y = dev(b.H), dev(b.Y[:, 0, :])
    fn = api.eq_pd if mode == "pd" else api.eq_fd
    z0, s0 = fn(H, y, b.n0, b.cluster_off)
    torch.cuda.synchronize()
    assert max_rel_err(z1[:, 0], host(z0)) <= 2e-5
    assert max_db_err(s1, host(s0)) <= 1e-3


@pytest.mark.parametrize("mode", ["pd", "fd"])
def test_non_finite_vector_stays_in_its_symbol(mode):
    """A NaN in one receive vector gives NaN for that vector only: the
    other vectors of the subcarrier, sigma2 and info are unaffected."""
    b = synth.make_symbol_batch(6, 64, 8, 2, 5, 10.0, "qpsk", seed=9)
    b.Y[2, 3, 17] = np.complex64(complex(np.nan, 0.0))
    z, s2, info = run(mode, b, "fp32", info=True)
    assert np.isnan(z[2, 3]).all()
    keep = np.ones(z.shape[:2], bool)
    keep[2, 3] = False
    zr, sr = ref(mode, b)
    assert max_rel_err(z[keep], zr[keep]) <= TOL_Z["fp32"]
    assert max_db_err(s2, sr) <= TOL_DB
    assert (info == 0).all()


@pytest.mark.parametrize("mode", ["pd", "fd"])
def test_symbols_fp64_queue(mode):
    """Nearly collinear users and a tiny N0: every subcarrier is routed to
    the FP64 re-solve, which recomputes all vectors of every tile."""
    rng = np.random.default_rng(12)
    W, B, U, C, S = 40, 48, 4, 2, 20
    b = synth.make_symbol_batch(W, B, U, C, S, 10.0, "qpsk", seed=13)
    H = b.H.astype(np.complex128)
    H[:, :, 1] = H[:, :, 0] + 1e-4 * (rng.standard_normal((W, B)) + 1j * rng.standard_normal((W, B)))
    b.H = H.astype(np.complex64)
    b.Y = np.matmul(b.x.astype(np.complex128), np.swapaxes(b.H.astype(np.complex128), 1, 2)).astype(np.complex64)
    b.n0 = float(np.float32(1e-9))
    z, s2, info = run(mode, b, "fp32", info=True)
    flags = (info & (1 << 30)) != 0
    routed = flags if mode == "pd" else flags.any(axis=1)
    assert routed.all(), int(routed.sum())
    zr, sr = ref(mode, b)
    assert max_rel_err(z, zr) <= TOL_Z["fp32"]
    assert max_db_err(s2, sr) <= TOL_DB


def test_symbols_bench_launch_size():
    """B=256, C=8, U=16 with 14 symbols at 38,400 subcarriers (32 frames of
    1200), as timed: every output finite, info clear, sampled subcarriers
    against the oracle."""
    from paper_1808_04473_amd import api
    frames = [synth.config_symbol_batch(2, 14, 10.0, frame=f) for f in range(32)]
    Hn = np.concatenate([f.H for f in frames])
    Yn = np.concatenate([f.Y for f in frames])
    n0, off = frames[0].n0, frames[0].cluster_off
    del frames
    H, Y = dev(Hn), dev(Yn)
    idx = np.unique(np.concatenate([[0, Hn.shape[0] - 1],
                                    np.random.default_rng(4).choice(Hn.shape[0], 256, replace=False)]))
    sel = torch.from_numpy(idx).to(H.device)
    for mode in ("pd", "fd"):
        for prec in PRECS:
            fn = api.eq_pd_sym if mode == "pd" else api.eq_fd_sym
            z, s2, info = fn(H, Y, n0, off, precision=prec, return_info=True)
            torch.cuda.synchronize()
            assert int(info.ne(0).sum().item()) == 0
            assert bool(torch.isfinite(torch.view_as_real(z)).all().item())
            assert bool((s2 > 0).all().item())
            rf = oracle.eq_pd_symbols if mode == "pd" else oracle.eq_fd_symbols
            zr, sr = rf(Hn[idx], Yn[idx], n0, off)
            ez, es = max_rel_err(host(z[sel]), zr), max_db_err(host(s2[sel]), sr)
            print(f"{mode} {prec} 38400 x 14: {len(idx)} sampled, z err {ez:.2e}, sigma2 {es:.4f} dB", flush=True)
            assert ez <= TOL_Z[prec] and es <= TOL_DB


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("kind", ["zf", "mrc", "lmmse_unbiased"])
@pytest.mark.parametrize("shape", [(30, 256, 16, 8, 14), (6, 130, 24, [0, 60, 130], 40), (9, 37, 5, [0, 5, 20, 37], 3)],
                         ids=lambda s: f"W{s[0]}B{s[1]}U{s[2]}S{s[4]}")
def test_linear_symbols_match_oracle(mode, prec, kind, shape):
    """equalizer="zf" / "mrc" / "lmmse_unbiased" through the multi-vector calls: each vector
    against the oracle's equaliser on that vector alone."""
    from paper_1808_04473_amd import api
    W, B, U, C, S = shape
    off = C if isinstance(C, list) else None
    nc = len(C) - 1 if isinstance(C, list) else C
    b = synth.make_symbol_batch(W, B, U, nc, S, 10.0, "16qam", seed=41 + S, cluster_off=off)
    fn = api.eq_pd_sym if mode == "pd" else api.eq_fd_sym
    z, s2, info = fn(dev(b.H), dev(b.Y), b.n0, b.cluster_off, precision=prec, equalizer=kind, return_info=True)
    torch.cuda.synchronize()
    z, s2, info = host(z), host(s2), host(info)
    # ZF on a square local Gram (B_c = U) may be routed to FP64; no failures
    assert ((info & ~(1 << 30)) == 0).all()
    if kind != "zf" or B >= 4 * U:
        assert (info == 0).all(), np.unique(info)
    rf = oracle.eq_pd_linear if mode == "pd" else oracle.eq_fd_linear
    for s in range(b.Y.shape[1]):
        zr, sr = rf(b.H, b.Y[:, s], b.n0, b.cluster_off, kind)
        assert max_rel_err(z[:, s], zr) <= TOL_Z[prec]
        assert max_db_err(s2, sr) <= TOL_DB


def test_mrc_symbols_user_without_channel():
    """MRC through the multi-vector call: a zero column of H gives info =
    u + 1 and NaN for every vector of that subcarrier only."""
    from paper_1808_04473_amd import api
    b = synth.make_symbol_batch(5, 64, 8, 2, 6, 10.0, "qpsk", seed=43)
    b.H[2, :, 4] = 0
    z, s2, info = api.eq_pd_sym(dev(b.H), dev(b.Y), b.n0, b.cluster_off, equalizer="mrc", return_info=True)
    torch.cuda.synchronize()
    z, info = host(z), host(info)
    assert info[2] == 5 and np.isnan(z[2]).all()
    assert (info[np.arange(5) != 2] == 0).all() and np.isfinite(z[np.arange(5) != 2]).all()


@pytest.mark.parametrize("mode", ["pd", "fd"])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("S", [1, 2, 15, 16, 17, 32, 33])
@pytest.mark.parametrize("shape", [(5, 33, 3, 2), (4, 63, 16, 5), (3, 77, 17, 2), (3, 160, 32, 5)],
                         ids=lambda s: f"B{s[1]}U{s[2]}C{s[3]}")
def test_symbol_tile_edges(mode, prec, S, shape):
    """Vector counts at the edges of the 16-vector tiles, row blocks that end
    inside a block of 16 or 32 rows, full and partial user tiles, and cluster
    counts that leave a wave of a subcarrier a partial round."""
    W, B, U, C = shape
    cuts = [c * (B // C) + (c % 2 if 0 < c < C else 0) for c in range(C)] + [B]
    b = synth.make_symbol_batch(W, B, U, C, S, 10.0, "16qam", seed=B + 7 * S, cluster_off=cuts)
    check(mode, b, prec)


@pytest.mark.parametrize("W", [512, 513])
@pytest.mark.parametrize("S", [17, 31, 32, 33])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("eqz", ["lmmse", "mrc", "lama"])
def test_pd_symbols_above_16_vectors(W, S, prec, eqz):
    """Either side of the batch size up to which every 16 vectors of a
    subcarrier have a wave; some of the systems routed to FP64."""
    from paper_1808_04473_amd import api
    B, U = 40, 18
    b = synth.make_symbol_batch(W, B, U, 1, S, 10.0, "16qam", seed=S)
    H = b.H.copy()
    ill = [3, W - 1]
    if eqz == "lmmse":
        rng = np.random.default_rng(14)
        H[ill, :, 1] = H[ill, :, 0] + 1e-4 * (rng.standard_normal((2, B)) + 1j * rng.standard_normal((2, B)))
        b.Y = np.matmul(b.x.astype(np.complex128), np.swapaxes(H.astype(np.complex128), 1, 2)).astype(np.complex64)
        b.n0 = float(np.float32(1e-9))
    some = np.array([0, 3, 4, W // 2, W - 2, W - 1])
    args = (b.n0, b.cluster_off)
    for rep in range(2):  # the FP64 queue starts empty each time
        if eqz == "lama":
            z, s2, info = api.eq_pd_lama_sym(dev(H), dev(b.Y), *args, t_max=2, qam=16, precision=prec, return_info=True)
        else:
            z, s2, info = api.eq_pd_sym(dev(H), dev(b.Y), *args, precision=prec, equalizer=eqz, return_info=True)
        z, s2, info = host(z)[some], host(s2)[some], host(info)
        for s in range(S):
            y = b.Y[some][:, s]
            if eqz == "lama":
                zr, sr = oracle.eq_pd_lama(H[some], y, *args, 2, 16)
            elif eqz == "mrc":
                zr, sr = oracle.eq_pd_linear(H[some], y, *args, "mrc")
            else:
                zr, sr = oracle.eq_pd(H[some], y, *args)
            assert max_rel_err(z[:, s], zr) <= TOL_Z[prec], s
            assert max_db_err(s2[:, s] if eqz == "lama" else s2, sr) <= TOL_DB
        flags = (info & (1 << 30)) != 0
        assert flags[ill].all() if eqz == "lmmse" else not info.any()


def test_pd_symbols_of_two_tiles_side_by_side():
    """24 vectors of a batch that leaves SIMDs idle take about as long as 14
    (1.0 of it, 1.3 with both tiles in one wave)."""
    from paper_1808_04473_amd import api
    W, B, U = 256, 2048, 32
    g = torch.Generator(device="cuda").manual_seed(1)
    H = torch.randn(W, B, U, generator=g, device="cuda", dtype=torch.complex64) / 32
    Y = torch.randn(W, 24, B, generator=g, device="cuda", dtype=torch.complex64)

    def ms(Y):
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                api.eq_pd_sym(H, Y, 0.1, [0, B], precision="bf16x3", equalizer="mrc")
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 20)
        return best

    Y14 = Y[:, :14].contiguous()
    ms(Y)
    t14, t24 = ms(Y14), ms(Y)
    print(f"MRC of 14 vectors {t14:.3f} ms, of 24 {t24:.3f} ms", flush=True)
    assert t24 <= 1.15 * t14
