"""Batches whose waves, at several per subcarrier, would be more than a launch
takes (2^32 work-items): they run with fewer, and the first and last subcarriers
come out as in a batch of their own."""
import pytest
import torch

pytestmark = pytest.mark.gpu
N0 = 0.1


def _api():
    from paper_1808_04473_amd import api
    return api


def _batch(W, B, S=None):
    """W a multiple of 1024: random rows, repeated."""
    g = torch.Generator(device="cuda").manual_seed(W % 1000 + B)
    def rep(*shape):
        out = torch.empty(W, *shape, device="cuda", dtype=torch.complex64)
        out.view(W // 1024, 1024, *shape).copy_(torch.randn(1024, *shape, generator=g, device="cuda", dtype=torch.complex64))
        return out
    return rep(B, 1), rep(B) if S is None else rep(S, B)


def _same(got, want):
    # sums of up to 13 terms in another order: 13 roundings of the largest
    want = torch.view_as_real(want) if want.is_complex() else want
    got = torch.view_as_real(got) if got.is_complex() else got
    assert (got - want).abs().max() <= 1e-5 * want.abs().max()


def _ends(f, *batch):
    """f(batch) at both ends against f of those subcarriers alone."""
    full = f(*batch)
    torch.cuda.synchronize()
    for part in (slice(0, 1024), slice(-1024, None)):
        for a, b in zip(full, f(*(x[part].contiguous() for x in batch))):
            _same(a[part], b)


def test_fd_forward_and_adjoint():
    api = _api()
    W, C = (1 << 24) + 1024, 13  # four waves a subcarrier
    off = list(range(C + 1))
    H, y = _batch(W, C)
    _ends(lambda H, y: api.eq_fd(H, y, N0, off), H, y)
    _ends(lambda H, y: api.eq_fd_backward(H, y, N0, off, gz=y[:, :1].contiguous())[:2], H, y)


def test_fd_symbols():
    api = _api()
    W, C = (1 << 25) + 1024, 5  # two waves a subcarrier
    off = list(range(C + 1))
    H, Y = _batch(W, C, 2)
    _ends(lambda H, Y: api.eq_fd_sym(H, Y, N0, off)[:1], H, Y)
    _ends(lambda H, Y: api.eq_fd_sym(H, Y, N0, off, equalizer="mrc")[:1], H, Y)


def test_fd_lama_tile():
    api = _api()
    H, Y = _batch((1 << 25) + 1024, 2, 17)
    _ends(lambda H, Y: api.eq_fd_lama_sym(H, Y, N0, [0, 1, 2], t_max=1, qam=4)[:1], H, Y)
