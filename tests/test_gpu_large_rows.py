"""Expert computation (Section 4.2, Eq. 2-3) on a row space whose hidden activations exceed 2^31 elements
and whose largest group exceeds 2^32 bytes per hidden matrix: element offsets must be 64-bit and the
32-bit offsets of the buffer loads of the weight-gradient contraction must be re-based on the way.
Sampled rows and hidden units against the oracle; the rows sit at the start, around the 2^31-element
and 2^32-byte marks, at the group boundary and at the end."""
import numpy as np
import pytest
import torch

import gpu_util as G
from paper_2411_10003_amd import binding, workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(600)
def test_rows_beyond_32_bit_offsets():
    d, h, act, dt = 64, 14336, "swiglu", "bf16"
    rows = [160000, 3840]
    A = sum(rows)
    assert A * h > 2 ** 31 and rows[0] * h * 2 > 2 ** 32
    tol = G.TOL[dt]
    rng = np.random.default_rng(4242)

    def draw(*shape, scale=1.0):
        a = (rng.standard_normal(shape) * scale).astype(np.float32)
        wl.round_to_bf16(a)
        return a
    X, dY = draw(A, d), draw(A, d)
    W1, W3, W2 = draw(2, d, h, scale=d ** -0.5), draw(2, d, h, scale=d ** -0.5), draw(2, h, d, scale=h ** -0.5)
    idx = np.repeat(np.arange(2, dtype=np.int32), rows)          # expert of every row; k = 1, rows in group order
    goe = np.arange(2, dtype=np.int32)

    hd = binding.Handle(T=A, d=d, h=h, E=2, k=1, P=1, self_dest=0, G=2, dtype=dt, act=act, renorm=0, device=G.DEV)
    L = hd.new_layout()
    L.slot_offsets.copy_(torch.tensor([0, rows[0], A], dtype=torch.int32))
    L.dest_slots.copy_(torch.tensor([0, 2], dtype=torch.int32))
    bf = dict(dtype=torch.bfloat16, device=G.DEV)
    dXp_in, ddY = G.dev(X, dt), G.dev(dY, dt)
    dW = [G.dev(w, dt) for w in (W1, W2, W3)]
    Yp, Z, U = torch.zeros(A, d, **bf), torch.empty(A, h, **bf), torch.empty(A, h, **bf)
    dXp = torch.zeros(A, d, **bf)
    g1 = torch.empty(2, d, h, dtype=torch.float32, device=G.DEV)
    g3 = torch.empty_like(g1)
    g2 = torch.empty(2, h, d, dtype=torch.float32, device=G.DEV)
    print("[large rows] device pass", flush=True)
    hd.expert_ffn_fwd(dXp_in, L, dW[0], dW[1], dW[2], Yp, Z, U)
    hd.expert_ffn_bwd(ddY, dXp_in, Z, U, L, dW[0], dW[1], dW[2], dXp, g1, g2, g3)
    torch.cuda.synchronize()

    m31 = 2 ** 31 // h                                           # first row whose elements lie past 2^31
    m32 = 2 ** 32 // (2 * h)                                     # first row past 2^32 bytes
    sample = sorted(set([0, 1, 255, 256, m31 - 1, m31, m31 + 1, m32 - 1, m32, m32 + 1, rows[0] - 1, rows[0], rows[0] + 1, A - 1]
                        + [int(x) for x in rng.integers(0, A, 12)]))
    a_s = np.array(sample, dtype=np.int32)
    print("[large rows] sampled rows", flush=True)
    Yo, Zo, Uo, _ = G.orc.ffn_fwd(X, idx, goe, W1, W2, W3, 1, act, a_s, True)
    r = torch.from_numpy(a_s.astype(np.int64)).to(G.DEV)
    assert G.rel_l2(G.host(Yp[r]), Yo) <= tol
    assert G.rel_l2(G.host(Z[r]), Zo) <= tol
    assert G.rel_l2(G.host(U[r]), Uo) <= tol
    dXo = G.orc.ffn_bwd_rows(X, idx, goe, W1, W2, W3, 1, act, a_s, dY[a_s].astype(np.float64))
    assert G.rel_l2(G.host(dXp[r]), dXo) <= tol
    print("[large rows] sampled hidden units", flush=True)
    for g in range(2):
        for j in (0, 4097, h - 1):
            r2, c1, c3 = G.orc.ffn_bwd_hidden(X, idx, goe, W1, W2, W3, 1, act, dY, g, j)
            assert G.rel_l2(G.host(g2[g, j, :]), r2) <= tol, (g, j)
            assert G.rel_l2(G.host(g1[g, :, j]), c1) <= tol, (g, j)
            assert G.rel_l2(G.host(g3[g, :, j]), c3) <= tol, (g, j)


def _check_ranges(T):
    """Tokens at the start, around the boundaries between launches and at the end."""
    step = 1 << 26
    return [(0, 40)] + [(t - 24, t + 40) for t in (step, 3 * step, T // step * step) if t + 40 <= T] + [(T - 33, T)]


def test_gate_gradient_of_more_tokens_than_a_launch_takes():
    """16 threads per token: 2^28 tokens are more threads than a launch may have."""
    T, E = (1 << 28) + 101, 2
    assert 16 * T > 1 << 32
    big = binding.Handle(T=T, d=64, h=64, E=E, k=1, P=1, self_dest=0, G=1, dtype="bf16", act="gelu", renorm=0, device=G.DEV, alloc_workspace=False)
    g = torch.Generator(device=G.DEV).manual_seed(1)
    logits = torch.randn(T, E, device=G.DEV, generator=g)
    dw = torch.randn(T, 1, device=G.DEV, generator=g)
    idx = (logits[:, 1:] > logits[:, :1]).to(torch.int32)
    dl = torch.full((T, E), 7.0, device=G.DEV)
    big.gate_bwd(dw, logits, idx, dl)
    torch.cuda.synchronize()
    for a, b in _check_ranges(T):
        want = G.orc.gate_bwd(G.host(dw[a:b]), G.host(logits[a:b]), G.host(idx[a:b]), 0)
        G.assert_rows_close(G.host(dl[a:b]), want, 1e-5, f"dlogits {a}", floor=1.0)
    assert not bool((dl[:, 0] == 7.0).any())
    del logits, dw, idx, dl
    torch.cuda.empty_cache()


@pytest.mark.timeout(300)
def test_gate_of_more_tokens_than_a_launch_takes():
    """Eight threads per token: 2^29 tokens are more threads than a launch may have (69 GB of them at d = 64)."""
    T, d, E = (1 << 29) + 101, 64, 4
    assert 8 * T > 1 << 32
    big = binding.Handle(T=T, d=d, h=64, E=E, k=1, P=1, self_dest=0, G=1, dtype="bf16", act="gelu", renorm=0, device=G.DEV, alloc_workspace=False)
    rng = np.random.default_rng(5)
    X = torch.zeros(T, d, dtype=torch.bfloat16, device=G.DEV)
    Wg = (rng.standard_normal((d, E)) * d ** -0.5).astype(np.float32)
    bg = rng.standard_normal(E).astype(np.float32)
    rows = {}
    for a, b in _check_ranges(T):
        rows[a, b] = wl.round_to_bf16(rng.standard_normal((b - a, d)).astype(np.float32))
        X[a:b] = G.dev(rows[a, b], "bf16")
    logits = torch.full((T, E), 7.0, device=G.DEV)
    idx = torch.full((T, 1), -1, dtype=torch.int32, device=G.DEV)
    w = torch.zeros(T, 1, device=G.DEV)
    big.gate_topk(X, G.dev(Wg), G.dev(bg), logits, idx, w)
    torch.cuda.synchronize()
    for (a, b), x in rows.items():
        ref = G.orc.route(x, Wg, bg, 1, 0)
        assert np.array_equal(G.host(logits[a:b]).view(np.uint32), ref["logits"].view(np.uint32))
        assert np.array_equal(G.host(idx[a:b]), ref["idx"])
        assert np.allclose(G.host(w[a:b]), ref["w"], rtol=1e-5, atol=1e-7)
    assert not bool((idx < 0).any())
    del X, logits, idx, w
    torch.cuda.empty_cache()


@pytest.mark.timeout(300)
def test_row_movers_of_more_tokens_than_a_launch_takes():
    """64 threads per token: 2^26 tokens are more threads than a launch may have.  Weights of one and zero logit gradients, so
    that every result is a copy."""
    T, d, E = (1 << 26) + 101, 64, 2
    hd = binding.Handle(T=T, d=d, h=64, E=E, k=1, P=1, self_dest=0, G=2, dtype="bf16", act="gelu", renorm=0, device=G.DEV)
    g = torch.Generator(device=G.DEV).manual_seed(3)
    X = torch.randint(0x3e00, 0x4000, (T, d), dtype=torch.int16, device=G.DEV, generator=g).view(torch.bfloat16)     # 0.125 to 2
    idx = torch.randint(0, E, (T, 1), dtype=torch.int32, device=G.DEV, generator=g)
    counts, lay = torch.zeros(E, dtype=torch.int32, device=G.DEV), hd.new_layout()
    Xp = torch.zeros(T, d, dtype=torch.bfloat16, device=G.DEV)
    bits = lambda t: t.view(torch.int16)                          # noqa: E731
    hd.expert_counts(idx, counts)
    hd.dispatch(torch.zeros(E, dtype=torch.int32, device=G.DEV), X, idx, counts, lay, Xp)
    torch.cuda.synchronize()
    assert counts.tolist() == torch.bincount(idx.view(-1), minlength=E).tolist()
    assert torch.equal(lay.perm.long(), torch.argsort(idx.view(-1), stable=True))
    assert torch.equal(bits(Xp), bits(X)[lay.perm.long()])
    del hd.ws
    ones, out = torch.ones(T, 1, device=G.DEV), torch.zeros(T, d, dtype=torch.bfloat16, device=G.DEV)
    hd.combine(Xp, lay.pos, ones, out)
    assert torch.equal(out, X)
    hd.dispatch_bwd(Xp, lay.pos, out.zero_())
    assert torch.equal(out, X)
    hd.input_grad(Xp, lay.pos, torch.zeros(T, E, device=G.DEV), torch.ones(d, E, device=G.DEV), out.zero_())
    assert torch.equal(out, X)
    dw = torch.full((T, 1), 7.0, device=G.DEV)
    hd.combine_bwd(X, Xp, lay.pos, ones, out.zero_(), dw)
    assert torch.equal(out, Xp)
    for a, b in [(0, 40)] + [(t - 24, t + 40) for t in (1 << 25, 1 << 26)] + [(T - 33, T)]:
        want = (X[a:b].double() ** 2).sum(1)
        assert torch.allclose(dw[a:b, 0].double(), want, rtol=1e-5, atol=0)
    assert not bool((dw == 7.0).any())
    del X, Xp, idx, lay, ones, out, dw
    torch.cuda.empty_cache()
