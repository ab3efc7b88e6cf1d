"""GPU: how far the fp32 kernels are from a 64-bit evaluation, in the 2-norm.

The bound of the state.  One step rounds the contraction (V products and sums), the outer product's
FMA, tanh (0.3 ulp rms) and the update H + (1 - f) (Z - H) (two roundings); with gates around 0.85
the state remembers some ten steps of it, and W has gain below one.  An emulation of one chain of
products with the outer product added last, every rounding in fp32, gives 0.9e-7 relative to the state
at all V; the outer product at the head of one of four chains gives 1.18e-7 (V = 32) and 1.40e-7
(V = 64)."""
import numpy as np
import pytest

from paper_2603_14360_amd import binding as mb
import oracle

pytestmark = pytest.mark.gpu


def _problem(B, T, N, K, V, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q, k, v = r(B, T, N, K) * K ** -0.5, r(B, T, N, K) * K ** -0.5, r(B, T, N, V) * K ** -0.5
    f = torch.sigmoid(r(B, T, N) + 2)
    W = r(N, V, V) * (0.25 * V ** -0.5) + 0.5 * torch.eye(V, device="cuda")
    return q, k, v, f, W, r(B, N, K, V) * 0.1


@pytest.mark.parametrize("K,V", [(16, 16), (64, 16), (32, 32), (64, 32), (32, 64), (64, 64), (128, 64)])
def test_state_error(K, V):
    print("case", K, V, flush=True)
    B, T, N = 4, 512, 4
    args = _problem(B, T, N, K, V, 7)
    scan = mb.Scan(B, T, N, K, V, "f32", backward=False)
    _, HT = scan.fwd(*args)
    ref = oracle.fwd(*[x.double().cpu().numpy() for x in args])[1]
    err = np.linalg.norm(HT.double().cpu().numpy() - ref) / np.linalg.norm(ref)
    print("state error %.3e" % err, flush=True)
    assert err < 1.05e-7


# bounds, in ulp of the result.  Its own rounding: 0.5.  Below 1, x^3 p(x^2) is at most a quarter of the
# result and its two factors and their product are rounded: another 0.5, and 0.1 for the fit.  From 1 on
# 2 / (1 + e) has a relative error of half an ulp of the exponent's argument times ln 2 (1.7e-7 up to 4, 3.3e-7 up
# to 8) and an ulp (1.2e-7) each of the exponential, the sum and the reciprocal, 4.5e-7 in all, and is 0.24 of an
# ulp of 6e-8 at 1: 1.8; 0.095 at 1.5 with 6.1e-7: 1.0; nothing beyond 3
TANH = [(1e-6, 1e-3, 0.6), (1e-3, 0.3, 0.75), (0.3, 0.55, 1.0), (0.55, 0.7, 1.1), (0.7, 1, 1.1), (1, 1.5, 2.3),
        (1.5, 3, 1.5), (3, 12, 0.6), (12, 3e38, 0.6)]


@pytest.mark.parametrize("lo,hi,bound", TANH)
@pytest.mark.parametrize("K,V", [(128, 16), (128, 32), (128, 64)])
def test_tanh(K, V, lo, hi, bound):
    """One step with W = 0, f = 0 and v = 1: the state is tanh(k), k in [lo, hi] in both signs; in
    one head all of a wave's values are of the range, in the other a few among small ones."""
    import torch
    print("case", K, V, lo, hi, flush=True)
    B = 512
    g = torch.Generator(device="cuda").manual_seed(11)
    u = torch.rand(B, 1, 2, K, generator=g, device="cuda", dtype=torch.float64)
    k = (lo + (hi - lo) * u).float().clamp(lo, hi)
    k[:, :, :, ::3] *= -1
    k[:, :, 1, 1::2] = 0.25
    z = lambda *s: torch.zeros(*s, device="cuda")
    scan = mb.Scan(B, 1, 2, K, V, "f32", backward=False)
    _, HT = scan.fwd(k, k, z(B, 1, 2, V) + 1, z(B, 1, 2), z(2, V, V))
    assert torch.equal(HT, HT[..., :1].expand_as(HT))
    ref = torch.tanh(k[:, 0].double())
    ulp = torch.exp2(torch.floor(torch.log2(ref.abs())) - 23)
    err = float(((HT[..., 0].double() - ref) / ulp).abs().max())
    print("tanh error %.2f ulp" % err, flush=True)
    assert err <= bound


def test_tanh_of_no_number():
    import torch
    k = torch.full((1, 1, 1, 16), 0.5, device="cuda")
    k[0, 0, 0, :4] = torch.tensor([float("inf"), -float("inf"), float("nan"), 1e38], device="cuda")
    z = lambda *s: torch.zeros(*s, device="cuda")
    _, HT = mb.Scan(1, 1, 1, 16, 16, "f32", backward=False).fwd(k, k, z(1, 1, 1, 16) + 1, z(1, 1, 1), z(1, 16, 16))
    col = HT[0, 0, :, 0]
    assert col[0] == 1 and col[1] == -1 and col[2].isnan() and col[3] == 1
    assert (col[4:] - 0.46211716).abs().max() < 1e-7 and torch.equal(HT[0, 0, :2, :], col[:2, None].expand(2, 16))
