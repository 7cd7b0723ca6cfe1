"""The fp32 grouped FFN on the fp32 matrix cores against the oracle, at the sizes where its tiles can go wrong: the tile
sizes (32 x 32 and 64 x 32 with a shared contraction, 64 x 64), widths that are no multiple of a tile, a slice or four floats, ragged
and empty groups, more groups than lanes, and operands that are not 16-byte aligned.  Checks and tolerance (1e-5, row by
row) are those of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from paper_2411_10003_amd import workload as wl
import test_gpu_parity as P

pytestmark = pytest.mark.gpu

G = P.G          # module-scoped fixtures of the parity tests
orc = P.orc


def _cfg(**kw):
    kw = dict(dict(dtype="f32", act="gelu", k=2, E=8, P=4, alpha=1.2, n_replicas=1, backward=True), **kw)
    return wl.scaled(wl.CONFIGS[0], **kw)


CASES = [
    _cfg(T=70, d=64, h=32),                                     # one tile across, contractions of one slice and less
    _cfg(T=97, d=68, h=33, act="swiglu"),                       # widths one past a tile; h odd: 4-byte requests
    _cfg(T=200, d=60, h=127),
    _cfg(T=333, d=132, h=260, act="swiglu", alpha=2.5),         # h a multiple of four only, very uneven groups
    _cfg(T=640, d=256, h=64, k=1, E=80, P=1, n_replicas=0),     # 80 hosted groups, some of them empty
    _cfg(T=2500, d=516, h=1092),                                # 64 x 64 tiles, 64 x 32 where 516 wide, remainders in all
    _cfg(T=1100, d=292, h=612, act="swiglu"),                   # 32 x 32 tiles of two weight matrices, last slices of 36 steps
    _cfg(T=2500, d=260, h=1092, act="swiglu", alpha=2.0),       # 64 x 64 tiles of two weight matrices, last slices of 4 steps
    _cfg(T=2500, d=516, h=1090, act="swiglu", alpha=2.0),       # the same with 4-byte requests
    _cfg(T=2500, d=292, h=612, act="swiglu", alpha=0.5),        # 64 x 64 tiles where 612 wide, else 32 x 32
    _cfg(T=1100, d=1004, h=804, act="swiglu"),                  # 64 x 32 tiles, also of two weight matrices, last slices of 44 and 36 steps
    _cfg(T=250, d=160, h=517),                                  # 32 x 32 tiles, a few more than run at once with four buffers
]
_ids = lambda c: f"{c.act}-T{c.T}-d{c.d}-h{c.h}-E{c.E}-k{c.k}"   # noqa: E731


@pytest.mark.parametrize("cfg", CASES, ids=_ids)
def test_forward(G, orc, cfg):
    P.test_ffn_forward_and_combine(G, orc, cfg)


@pytest.mark.parametrize("cfg", CASES, ids=_ids)
def test_backward(G, orc, cfg):
    P.test_backward_calls(G, orc, cfg)


def _shifted(t):
    """The same tensor four bytes past a 16-byte boundary."""
    if t is None:
        return None
    flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:]
    flat.copy_(t.reshape(-1))
    return flat.view(t.shape)


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_unaligned_operands_give_the_same_bits(G, act):
    """4-byte requests feed the same order of multiply-adds as 16-byte requests."""
    cfg = _cfg(T=300, d=128, h=192, act=act)
    case = G.Case(cfg)
    hd = G.make_handle(cfg)
    res = []
    for f in (lambda t: t, _shifted):
        b = G.binding.LayerBuffers(hd, True)
        G.gpu_route(hd, case, b)
        hd.dispatch(case.ddest, case.dX, b.idx, b.counts, b.layout, b.Xp)
        b.Yp.zero_(); b.dXp.zero_()
        W1, W2, W3 = f(case.dW1), f(case.dW2), f(case.dW3)
        dYp = f(torch.randn(cfg.A, cfg.d, device=G.DEV, generator=torch.Generator(device=G.DEV).manual_seed(3)))
        Z, U, Yp, dXp = f(b.Z.zero_()), f(b.U.zero_()) if act == "swiglu" else None, f(b.Yp), f(b.dXp)
        hd.expert_ffn_fwd(f(b.Xp), b.layout, W1, W2, W3, Yp, Z, U)
        dW = [f(torch.zeros_like(b.dW1)), f(torch.zeros_like(b.dW2)), f(torch.zeros_like(b.dW1)) if act == "swiglu" else None]
        hd.expert_ffn_bwd(dYp, f(b.Xp), Z, U, b.layout, W1, W2, W3, dXp, *dW)
        torch.cuda.synchronize()
        res.append([Yp, Z, U, dXp, *dW])
    for a, c in zip(*res):
        assert (a is None) == (c is None)
        if a is not None:
            assert np.array_equal(G.host(a).view(np.uint32), G.host(c).view(np.uint32))


@pytest.mark.timeout(300)
def test_more_tiles_than_the_threads_of_one_axis(G):
    """The most groups, the narrowest rows and a wide hidden layer: 2^24 blocks of 256 threads and more, of which a few have
    rows.  Against a float64 product; tolerance as above for the weight gradients.  Yp and dXp are sums of K = h terms taken one
    after the other: partial sum i is about i^0.5 terms large and rounded by 2^-24 / 3^0.5 of itself (rms), together
    (K / 2)^0.5 2^-24 / 3^0.5 = 2.5e-5 of the whole sum, of which four times is allowed."""
    E, d, h = 1024, 4, (1 << 20) + 64
    assert 1024 * (h // 64) * 256 > 1 << 32
    used = {0: 3, 1: 1, 700: 40, 1023: 20}
    A = sum(used.values())
    hd = G.binding.Handle(T=A, d=d, h=h, E=E, k=1, P=1, self_dest=0, G=E, dtype="f32", act="gelu", renorm=0, device=G.DEV)
    g = torch.Generator(device=G.DEV).manual_seed(9)
    idx = torch.tensor([e for e, n in used.items() for _ in range(n)], dtype=torch.int32, device=G.DEV)
    counts, lay = torch.zeros(E, dtype=torch.int32, device=G.DEV), hd.new_layout()
    X, dYp = torch.randn(A, d, device=G.DEV, generator=g), torch.randn(A, d, device=G.DEV, generator=g)
    Xp, Z = torch.empty(A, d, device=G.DEV), torch.zeros(A, h, device=G.DEV)
    hd.expert_counts(idx, counts)
    hd.dispatch(torch.zeros(E, dtype=torch.int32, device=G.DEV), X, idx, counts, lay, Xp)
    W1, W2 = torch.zeros(E, d, h, device=G.DEV), torch.zeros(E, h, d, device=G.DEV)
    for e in used:
        W1[e] = torch.randn(d, h, device=G.DEV, generator=g) * d ** -0.5
        W2[e] = torch.randn(h, d, device=G.DEV, generator=g) * h ** -0.5
    Yp, dXp = torch.full((A, d), 7.0, device=G.DEV), torch.full((A, d), 7.0, device=G.DEV)
    dW1, dW2 = torch.full((E, d, h), 7.0, device=G.DEV), torch.full((E, h, d), 7.0, device=G.DEV)
    hd.expert_ffn_fwd(Xp, lay, W1, W2, None, Yp, Z, None)
    hd.expert_ffn_bwd(dYp, Xp, Z, None, lay, W1, W2, None, dXp, dW1, dW2, None)
    torch.cuda.synchronize()
    chain = 4 * (h / 2 / 3) ** 0.5 * 2.0 ** -24
    o = 0
    for e, n in used.items():
        x, dy, w1, w2 = Xp[o:o + n].double(), dYp[o:o + n].double(), W1[e].double(), W2[e].double()
        z = x @ w1
        cdf = 0.5 * (1 + torch.erf(z * 0.5 ** 0.5))
        dz = (dy @ w2.t()) * (cdf + z * torch.exp(-0.5 * z * z) * (2 * np.pi) ** -0.5)
        for got, want, what in ((Yp[o:o + n], (z * cdf) @ w2, "Yp"), (dXp[o:o + n], dz @ w1.t(), "dXp"),
                                (dW1[e], x.t() @ dz, "dW1"), (dW2[e].t(), dy.t() @ (z * cdf), "dW2")):
            G.assert_rows_close(G.host(got), want.cpu().numpy(), 1e-5 if what[:2] == "dW" else chain, f"{what} {e}")
        o += n
    for e in (2, 512, 1022):
        assert not bool(dW1[e].any()) and not bool(dW2[e].any())
    del W1, W2, dW1, dW2
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T,h,parts", [(60, 128, 4), (1100, 320, 4), (3000, 512, 4), (2500, 1092, 1)])
@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_precision_of_a_contraction(G, T, h, parts, act):
    """Against 64 bits, in the tiles that T k rows and h columns take: chains of d / parts products (32 x 32 tiles: a wave each for a
    quarter of them; 64 x 32: two waves with two sums each).  Each rounds by 0.425 x 2^-24 of a partial sum that grows like the
    root of the chain (test_gpu_gate_grad.py): (n / 2)^0.5 of that, and the parts' sums."""
    cfg = _cfg(T=T, d=3000, h=h, act=act, n_replicas=0, P=1)
    d, A, E = cfg.d, cfg.A, cfg.E
    hd = G.make_handle(cfg, G=E)
    g = torch.Generator(device=G.DEV).manual_seed(T + h)
    idx = torch.arange(A, device=G.DEV, dtype=torch.int32) % E
    counts, lay = torch.zeros(E, dtype=torch.int32, device=G.DEV), hd.new_layout()
    X, Xp = torch.randn(T, d, device=G.DEV, generator=g), torch.empty(A, d, device=G.DEV)
    hd.expert_counts(idx, counts)
    hd.dispatch(torch.zeros(E, dtype=torch.int32, device=G.DEV), X, idx, counts, lay, Xp)
    W1, W2 = torch.randn(E, d, h, device=G.DEV, generator=g), torch.randn(E, h, d, device=G.DEV, generator=g)
    W3 = torch.randn(E, d, h, device=G.DEV, generator=g) if act == "swiglu" else None
    Yp, Z = torch.zeros(A, d, device=G.DEV), torch.zeros(A, h, device=G.DEV)
    U = torch.zeros_like(Z) if act == "swiglu" else None
    hd.expert_ffn_fwd(Xp, lay, W1, W2, W3, Yp, Z, U)
    bound = 0.425 * 2.0 ** -24 * ((d / parts + parts) / 2) ** 0.5
    for got, W in ((Z, W1), (U, W3)) if act == "swiglu" else ((Z, W1),):
        want = torch.cat([x.double() @ w.double() for x, w in zip(Xp.split(counts.tolist()), W)])
        assert float((got.double() - want).norm() / want.norm()) < 1.15 * bound


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_rows_too_far_apart_for_an_offset(G, act):
    """A hidden layer of 2^24: 64 rows of it are 2^32 bytes.  Against a float64 product; tolerance as for the many tiles above."""
    d, h, rows = 4, 1 << 24, [3, 0, 2]
    hd = G.binding.Handle(T=5, d=d, h=h, E=3, k=1, P=1, self_dest=0, G=3, dtype="f32", act=act, renorm=0, device=G.DEV)
    g = torch.Generator(device=G.DEV).manual_seed(11)
    idx = torch.repeat_interleave(torch.arange(3, dtype=torch.int32), torch.tensor(rows)).to(G.DEV)
    counts, lay = torch.zeros(3, dtype=torch.int32, device=G.DEV), hd.new_layout()
    X, dYp = torch.randn(5, d, device=G.DEV, generator=g), torch.randn(5, d, device=G.DEV, generator=g)
    Xp, Z = torch.empty(5, d, device=G.DEV), torch.zeros(5, h, device=G.DEV)
    U = torch.zeros_like(Z) if act == "swiglu" else None
    hd.expert_counts(idx, counts)
    hd.dispatch(torch.zeros(3, dtype=torch.int32, device=G.DEV), X, idx, counts, lay, Xp)
    W1 = torch.randn(3, d, h, device=G.DEV, generator=g) * d ** -0.5
    W2 = torch.randn(3, h, d, device=G.DEV, generator=g) * h ** -0.5
    W3 = torch.randn(3, d, h, device=G.DEV, generator=g) * d ** -0.5 if act == "swiglu" else None
    Yp, dXp, dW1, dW2 = torch.zeros(5, d, device=G.DEV), torch.zeros(5, d, device=G.DEV), torch.full_like(W1, 7.0), torch.full_like(W2, 7.0)
    dW3 = torch.full_like(W1, 7.0) if act == "swiglu" else None
    hd.expert_ffn_fwd(Xp, lay, W1, W2, W3, Yp, Z, U)
    hd.expert_ffn_bwd(dYp, Xp, Z, U, lay, W1, W2, W3, dXp, dW1, dW2, dW3)
    torch.cuda.synchronize()
    assert not bool(dW1[1].any()) and not bool(dW2[1].any()) and (dW3 is None or not bool(dW3[1].any()))
    chain = 4 * (h / 2 / 3) ** 0.5 * 2.0 ** -24
    rel = lambda a, b: float((a.double() - b).norm() / b.norm())   # noqa: E731
    for e, o in ((0, 0), (2, 3)):
        n = rows[e]
        x, dy, w1, w2 = Xp[o:o + n].double(), dYp[o:o + n].double(), W1[e].double(), W2[e].double()
        z, dA = x @ w1, dy @ w2.t()
        if act == "swiglu":
            w3 = W3[e].double()
            u, sg = x @ w3, torch.sigmoid(z)
            a, dz, du = z * sg * u, dA * u * (sg * (1 + z * (1 - sg))), dA * z * sg
            dx = dz @ w1.t() + du @ w3.t()
            assert rel(dW3[e], x.t() @ du) < 1e-5 and rel(U[o:o + n], u) < 1e-5
        else:
            cdf = 0.5 * (1 + torch.erf(z * 0.5 ** 0.5))
            a, dz = z * cdf, dA * (cdf + z * torch.exp(-0.5 * z * z) * (2 * np.pi) ** -0.5)
            dx = dz @ w1.t()
        assert rel(Yp[o:o + n], a @ w2) < chain and rel(dXp[o:o + n], dx) < chain
        assert rel(dW1[e], x.t() @ dz) < 1e-5 and rel(dW2[e], a.t() @ dy) < 1e-5


def test_rows_too_far_apart_for_four_of_them(G):
    """A hidden layer of 2^28: 4 rows of it are 2^32 bytes.  The forward pass, its matrices in one array, two slices of steps."""
    d, h, n = 68, 1 << 28, 2
    hd = G.binding.Handle(T=n, d=d, h=h, E=1, k=1, P=1, self_dest=0, G=1, dtype="f32", act="swiglu", renorm=0, device=G.DEV)
    g = torch.Generator(device=G.DEV).manual_seed(12)
    W = torch.empty(d * h + 8, device=G.DEV)
    for i in range(0, W.numel(), 1 << 28):
        W[i:i + (1 << 28)].normal_(std=d ** -0.5, generator=g)
    W1, W2, W3 = W[:d * h].view(1, d, h), W[4:4 + d * h].view(1, h, d), W[8:].view(1, d, h)
    idx, counts, lay = torch.zeros(n, dtype=torch.int32, device=G.DEV), torch.zeros(1, dtype=torch.int32, device=G.DEV), hd.new_layout()
    Xp, Yp = torch.empty(n, d, device=G.DEV), torch.zeros(n, d, device=G.DEV)
    Z, U = torch.zeros(n, h, device=G.DEV), torch.zeros(n, h, device=G.DEV)
    hd.expert_counts(idx, counts)
    hd.dispatch(torch.zeros(1, dtype=torch.int32, device=G.DEV), torch.randn(n, d, device=G.DEV, generator=g), idx, counts, lay, Xp)
    hd.expert_ffn_fwd(Xp, lay, W1, W2, W3, Yp, Z, U)
    torch.cuda.synchronize()
    y, x = torch.zeros(n, d, dtype=torch.float64, device=G.DEV), Xp.double()
    rel = lambda a, b: float((a.double() - b).norm() / b.norm())   # noqa: E731
    for c in range(0, h, 1 << 23):
        cols = slice(c, c + (1 << 23))
        z, u = x @ W1[0, :, cols].double(), x @ W3[0, :, cols].double()
        assert rel(Z[:, cols], z) < 1e-5 and rel(U[:, cols], u) < 1e-5
        y += (z * torch.sigmoid(z) * u) @ W2[0, cols].double()
    assert rel(Yp, y) < 4 * (h / 2 / 3) ** 0.5 * 2.0 ** -24
    del W, W1, W2, W3, Z, U, hd
    torch.cuda.empty_cache()
