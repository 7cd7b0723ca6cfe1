"""GELU and its derivative in the epilogues of the bf16 FFN, element by element against 64 bits: one group whose weights are unit
matrices, so that the forward pass returns the rounded activation of its input and the backward pass the rounded derivative."""
import math

import pytest
import torch

import gpu_util as G
from paper_2411_10003_amd import binding

pytestmark = pytest.mark.gpu
N = 64
HALF_STEP = 2.0 ** -8                                         # of bf16 (8 significant bits), relative to the number rounded


def _layer(rows, saved=True):
    hd = binding.Handle(T=rows, d=N, h=N, E=8, k=1, P=1, self_dest=0, G=8, dtype="bf16", act="gelu", renorm=0, device=G.DEV)
    hd.set_act_saved(saved)
    i32 = dict(dtype=torch.int32, device=G.DEV)
    counts, lay, x = torch.zeros(8, **i32), hd.new_layout(), torch.zeros(rows, N, dtype=torch.bfloat16, device=G.DEV)
    idx = torch.zeros(rows, 1, **i32)
    hd.expert_counts(idx, counts)
    hd.dispatch(torch.zeros(8, **i32), x, idx, counts, lay, torch.zeros_like(x))
    return hd, lay


def _weights(m):
    return m.to(torch.bfloat16).to(G.DEV).expand(8, N, N).contiguous()


def _forward(X, W1, W2):
    hd, lay = _layer(X.shape[0])
    Yp, Z = torch.zeros_like(X), torch.zeros_like(X)
    hd.expert_ffn_fwd(X, lay, W1, W2, None, Yp, Z, None)
    return Yp, Z


def _derivative(Z, saved):
    hd, lay = _layer(Z.shape[0], saved)
    eye, ones, dXp = _weights(torch.eye(N)), torch.ones_like(Z), torch.zeros_like(Z)
    if saved:
        hd.expert_ffn_fwd(Z, lay, eye, eye, None, torch.zeros_like(Z), torch.zeros_like(Z), None)
    dW = [torch.zeros(8, N, N, device=G.DEV) for _ in range(2)]
    hd.expert_ffn_bwd(ones, Z, Z, None, lay, eye, eye, None, dXp, *dW, None)
    return dXp


def _every_bf16():
    """Every bf16 number of magnitude 2^-20 to 10, either sign, in rows of 64."""
    bits = torch.arange(0x3580, 0x4120 + 1, dtype=torch.int32)
    z = (torch.cat([bits, bits | 0x8000]) << 16).view(torch.float32)
    z = torch.cat([z, z.new_ones(-z.numel() % N)]).view(-1, N)
    return z.to(torch.bfloat16).to(G.DEV)


def test_every_pre_activation():
    z = _every_bf16()
    eye = _weights(torch.eye(N))
    Yp, Z = _forward(z, eye, eye)
    assert torch.equal(Z, z)
    zd = z.double()
    want = 0.5 * zd * torch.special.erfc(-zd * math.sqrt(0.5))
    # half a bf16 step, and the relative error that the rational approximation of erf has in the tail (0.35 % at -6, 2.0 % at -10)
    bound = (HALF_STEP + torch.where(zd < 0, 2.2e-4 * zd * zd, 0.0) + 1e-6) * want.abs()
    off = ((Yp.double() - want).abs() / bound).flatten()
    worst = int(off.argmax())
    assert float(off[worst]) <= 1.0, (float(zd.flatten()[worst]), float(Yp.flatten()[worst]), float(want.flatten()[worst]))


@pytest.mark.parametrize("saved", [True, False])
def test_every_derivative(saved):
    z = _every_bf16()
    zd = z.double()
    want = 0.5 * torch.special.erfc(-zd * math.sqrt(0.5)) + zd * torch.exp(-0.5 * zd * zd) / math.sqrt(2 * math.pi)
    # half a bf16 step, and the absolute error near the zero at -0.75, the relative one in the tail (2e-4 at -10)
    bound = HALF_STEP * want.abs() + torch.where(zd < -1.5, 2.0 ** -11 * want.abs(), 4e-7)
    off = ((_derivative(z, saved).double() - want).abs() / bound).flatten()
    worst = int(off.argmax())
    assert float(off[worst]) <= 1.0, (float(zd.flatten()[worst]), float(want.flatten()[worst]))


def _same(got, want):
    torch.testing.assert_close(got, torch.tensor(want), rtol=0, atol=0, equal_nan=True)


def test_past_the_range():
    """Infinities, NaN and numbers whose square is infinite, as z Phi(z) and its derivative have them."""
    inf, nan = math.inf, math.nan
    first = torch.tensor([3e38, -3e38, nan, 5e19, -5e19, 20.0, -20.0])              # times 2: the pre-activations
    X = torch.zeros(first.numel(), N)
    X[:, 0] = first
    W1 = torch.zeros(N, N)
    W1[0] = 2.0
    Yp, Z = _forward(X.to(torch.bfloat16).to(G.DEV), _weights(W1), _weights(torch.full((N, N), 1.0 / N)))
    z = Z[:, 0].float().cpu()
    _same(z[:3], [inf, -inf, nan])
    y = Yp.float().cpu()
    for row, want in zip(y, [inf, nan, nan, float(z[3]), 0.0, 40.0, 0.0]):
        _same(row, [want] * N)
    D = _derivative(Z, False).float().cpu()
    for row, want in zip(D, [nan, nan, nan, 1.0, 0.0, 1.0, 0.0]):
        _same(row, [want] * N)
