"""Gradient of the gate weights against the oracle at the edges of its 16 lanes per token: expert counts below, at and past a
multiple of 16, every number of selected experts the handle allows, token counts that leave a block partly empty."""
import numpy as np
import pytest
import torch

import gpu_util as G
from oracle import moe_oracle as orc
from paper_2411_10003_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("renorm", [0, 1])
@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (15, 5, 5), (16, 16, 1), (33, 17, 8), (257, 64, 2), (100, 100, 3), (40, 1024, 8)])
def test_gate_bwd(T, E, k, renorm):
    cfg = wl.scaled(wl.CONFIGS[1], T=T, d=64, h=64, E=E, k=k, P=1, renorm=renorm, n_replicas=0)
    rng = np.random.default_rng(T + E + k)
    logits = (3.0 * rng.standard_normal((T, E))).astype(np.float32)
    idx = np.argsort(-logits, axis=1, kind="stable")[:, :k].astype(np.int32)
    dw = rng.standard_normal((T, k)).astype(np.float32)
    hd = G.make_handle(cfg, G=1)
    dl = torch.full((T, E), 7.0, dtype=torch.float32, device=G.DEV)
    hd.gate_bwd(G.dev(dw), G.dev(logits), G.dev(idx), dl)
    torch.cuda.synchronize()
    G.assert_rows_close(G.host(dl), orc.gate_bwd(dw, logits, idx, renorm), 1e-5, "dlogits", floor=1.0)


def test_masked_experts_get_no_gradient():
    """An expert whose logit is -inf has probability zero and takes no part."""
    T, E, k = 50, 40, 2
    cfg = wl.scaled(wl.CONFIGS[1], T=T, d=64, h=64, E=E, k=k, P=1, renorm=0, n_replicas=0)
    rng = np.random.default_rng(1)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    logits[:, 7] = -np.inf
    idx = np.argsort(-logits, axis=1, kind="stable")[:, :k].astype(np.int32)
    dw = rng.standard_normal((T, k)).astype(np.float32)
    dl = torch.full((T, E), 7.0, dtype=torch.float32, device=G.DEV)
    G.make_handle(cfg, G=1).gate_bwd(G.dev(dw), G.dev(logits), G.dev(idx), dl)
    torch.cuda.synchronize()
    got = G.host(dl)
    assert (got[:, 7] == 0).all() and np.isfinite(got).all()
    G.assert_rows_close(got, orc.gate_bwd(dw, logits, idx, 0), 1e-5, "dlogits", floor=1.0)
