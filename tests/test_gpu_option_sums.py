"""Sums over (b, t) of the options' gradients (dw_r, dalpha, dbeta) and the gate's chain rule:
column counts below, at and beyond a workgroup's, rows with and without a remainder of the
unrolled walk, against float64 sums of the very tensors that the call saw or returned."""
import pytest

from paper_2603_14360_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("B,T,N,V", [(1, 1, 1, 16), (1, 2, 3, 16), (2, 131, 17, 16), (1, 700, 65, 16), (3, 1367, 2, 32),
                                     (2, 37, 130, 64), (1, 5, 84, 16), (1, 4500, 1, 16)])
def test_sums_over_batch_and_time(io, B, T, N, V):
    import torch
    print("case", io, B, T, N, V, flush=True)
    K = 16
    g = torch.Generator(device="cuda").manual_seed(B + T + N + V)
    dt = torch.bfloat16 if io == "bf16" else torch.float32
    r = lambda *s, d=dt: torch.randn(*s, generator=g, device="cuda").to(d)
    q, k, v, dy = r(B, T, 1, K) / 4, r(B, T, 1, K) / 4, r(B, T, N, V), r(B, T, N, V)
    x, w_r = r(B, T, N, d=torch.float32), r(N, V)
    W = (r(N, V, V, d=torch.float32) * 0.2 * V ** -0.5).to(dt)
    al, be = torch.rand(N, generator=g, device="cuda") + 0.5, r(N, d=torch.float32) * 0.3
    scan = mb.Scan(B, T, N, K, V, io, Nqk=1)
    scan.fwd(q, k, v, x, W, w_r=w_r, gate=(al, be))
    out = [o.clone() for o in scan.bwd(q, k, v, x, W, None, dy, w_r=w_r, gate=(al, be))]
    df, dw_r, da, db = out[3].double(), out[6].double(), out[7].double(), out[8].double()
    # terms of a running sum and of the two sums behind it: fewer than 64 + 256 + 32 additions of
    # at most half an ulp of the sum of magnitudes (the bound is met with a wide margin)
    eps = 352 * 2.0 ** -24
    term = dy.double() * v.double()
    assert ((dw_r - term.sum((0, 1))).abs() <= eps * term.abs().sum((0, 1))).all()
    assert ((db - df.sum((0, 1))).abs() <= eps * df.abs().sum((0, 1))).all()
    u = x.double() + be.double()
    term = df * torch.nn.functional.softplus(u) / (al.double() * torch.sigmoid(u))
    assert ((da - term.sum((0, 1))).abs() <= (eps + 1e-5) * term.abs().sum((0, 1))).all()
    # every row went through the chain rule once: the plain backward on psi(x)
    psi = torch.exp(-al.double() * torch.nn.functional.softplus(u)).float()
    scan.fwd(q, k, v, psi, W, w_r=w_r)
    g0 = scan.bwd(q, k, v, psi, W, None, dy, w_r=w_r)[3].double()
    ref = -g0 * al.double() * torch.exp(-al.double() * torch.nn.functional.softplus(u)) * torch.sigmoid(u)
    assert (df - ref).abs().max() <= (1e-5 if io == "f32" else 2e-2) * ref.abs().max()
