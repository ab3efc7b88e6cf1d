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
