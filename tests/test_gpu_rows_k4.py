"""Combine and its gradient with four experts per token in bf16, at row lengths around the pieces a wave requests at a time
(64 lanes x 8 elements, two pieces): against plain fp32 sums of the same rows."""
import numpy as np
import pytest
import torch

import gpu_util as G
from paper_2411_10003_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d", [(1, 64), (5, 512), (7, 576), (9, 1024), (6, 1088), (13, 4160)])
def test_combine_of_four(T, d):
    k = 4
    cfg = wl.scaled(wl.CONFIGS[1], T=T, d=d, h=64, E=8, k=k, P=4, n_replicas=0, self_dest=0)
    hd = G.make_handle(cfg, G=1)
    rng = np.random.default_rng(T * d)
    A = T * k
    Yp = wl.round_to_bf16(rng.standard_normal((A, d)).astype(np.float32))
    dOut = wl.round_to_bf16(rng.standard_normal((T, d)).astype(np.float32))
    w = rng.random((T, k), dtype=np.float32)
    pos = rng.permutation(A).astype(np.int32)
    rows = Yp[pos].reshape(T, k, d).astype(np.float64)
    out = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda")
    dYp = torch.zeros(A, d, dtype=torch.bfloat16, device="cuda")
    dw = torch.zeros(T, k, device="cuda")
    hd.combine(G.dev(Yp, "bf16"), G.dev(pos), G.dev(w), out)
    hd.combine_bwd(G.dev(dOut, "bf16"), G.dev(Yp, "bf16"), G.dev(pos), G.dev(w), dYp, dw)
    torch.cuda.synchronize()
    # one rounding to bf16 (2^-9 relative) of an fp32 sum of four products
    want = (w[:, :, None] * rows).sum(1)
    terms = (np.abs(w[:, :, None] * rows)).sum(1)
    assert np.all(np.abs(out.float().cpu().numpy() - want) <= 2.0 ** -8 * np.abs(want) + 2.0 ** -21 * terms)
    # one product, one rounding: bit for bit
    grad = np.zeros((A, d), np.float32)
    grad[pos] = (w[:, :, None] * dOut[:, None, :]).reshape(A, d)
    assert np.array_equal(dYp.float().cpu().numpy(), wl.round_to_bf16(grad))
    # an fp32 dot product: d additions of terms in any order
    dots = (rows * dOut[:, None, :]).sum(2)
    assert np.all(np.abs(dw.cpu().numpy() - dots) <= d * 2.0 ** -24 * np.abs(rows * dOut[:, None, :]).sum(2))
