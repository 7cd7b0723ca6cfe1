"""Gate selection, counts, layout and positions where the number of experts or chunks changes the path: expert counts that
are no power of two, up to the largest; every number of chunks at which a launch is fused or split; several experts per
token; ties, NaN and infinities.  All of it exact against the oracle."""
import numpy as np
import pytest
import torch

import gpu_util as G
from oracle import moe_oracle as orc
from paper_2411_10003_amd import workload as wl

pytestmark = pytest.mark.gpu


def _cfg(**kw):
    return wl.scaled(wl.CONFIGS[1], **dict(dict(d=64, h=64, k=2, n_replicas=0, self_dest=0), **kw))


CASES = [
    _cfg(T=1, E=1, k=1, P=1),
    _cfg(T=127, E=5, P=5, k=3),                       # one chunk, not full
    _cfg(T=128, E=16, P=4),                           # exactly one chunk
    _cfg(T=129, E=63, P=7, k=1),
    _cfg(T=513, E=64, P=64),                          # P as many as experts
    _cfg(T=700, E=65, P=13, k=8),                     # a second row of lanes with one expert
    _cfg(T=4096, E=256, P=16, k=1),                   # the most chunks and experts dispatched in one launch
    _cfg(T=4097, E=256, P=16, k=1),                   # a chunk past that
    _cfg(T=60, d=4160, E=12, P=3, k=3),               # rows of three pieces, the last one short
    _cfg(T=50, d=36, E=7, P=7, dtype="f32"),          # fp32 rows of nine 16-byte vectors
    _cfg(T=8192, E=24, P=4),                          # the last number of chunks counted in one block
    _cfg(T=8193, E=24, P=4),                          # the first past it
    _cfg(T=300, E=257, P=257, k=8),                   # past the experts of the one-block counts
    _cfg(T=4000, E=1024, P=512, k=8),                 # the most experts, 125 chunks
    _cfg(T=40000, E=1000, P=10, k=2),                 # more chunks than are added up: the scan
    _cfg(T=140000, E=64, P=8, k=2),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: f"{c.dtype}-T{c.T}-d{c.d}-E{c.E}-k{c.k}-P{c.P}")
def test_counts_layout_positions(cfg):
    rng = np.random.default_rng(cfg.T + cfg.E)
    p = rng.gamma(0.3, size=cfg.E) + 1e-4             # uneven, with experts that get next to nothing
    noise = rng.gumbel(size=(cfg.T, cfg.E)).astype(np.float32) + np.log(p).astype(np.float32)
    idx = np.argpartition(-noise, min(cfg.k, cfg.E) - 1, axis=1)[:, :cfg.k].astype(np.int32)
    dest = rng.integers(0, cfg.P, size=cfg.E).astype(np.int32)
    cnt = orc.counts(idx, cfg.E)
    lay = orc.place(idx, cnt, dest, cfg.P)
    X = rng.standard_normal((cfg.T, cfg.d)).astype(np.float32)
    if cfg.dtype == "bf16":
        wl.round_to_bf16(X)
    hd = G.make_handle(cfg, G=min(cfg.E, 64))
    for after in (False, True):
        b = G.binding.LayerBuffers(hd, False)
        d_idx = G.dev(idx)
        b.counts.fill_(-1)
        hd.expert_counts(d_idx, b.counts)
        assert np.array_equal(G.host(b.counts), cnt)
        hd.dispatch(G.dev(dest), G.dev(X, cfg.dtype), d_idx, b.counts, b.layout, b.Xp, after_counts=after)
        torch.cuda.synchronize()
        G.assert_layout_equal(b, lay)
        assert np.array_equal(G.host(b.Xp), orc.dispatch(X, lay["perm"], cfg.k))
        hosted = int((dest == cfg.self_dest).sum())
        assert hd.read_status() == (0 if hosted <= min(cfg.E, 64) else -3)


@pytest.mark.parametrize("E,k", [(72, 1), (128, 8), (129, 3), (300, 8), (1024, 8)])
def test_routing_of_many_experts(E, k):
    """Selection and weights for more than 64 experts, with ties, NaN and infinities among the biases."""
    cfg = _cfg(T=203, E=E, k=k, P=1, renorm=1)
    rng = np.random.default_rng(E + k)
    X = wl.round_to_bf16(rng.standard_normal((cfg.T, cfg.d)).astype(np.float32))
    Wg = (rng.standard_normal((cfg.d, E)) * 0.1).astype(np.float32)
    Wg[:, 40:60] = Wg[:, 40:41]                       # twenty experts that always tie
    bg = rng.standard_normal(E).astype(np.float32)
    bg[40:60] = 2.0
    bg[3] = -np.inf
    bg[7] = np.nan
    ref = orc.route(X, Wg, bg, k, 1)
    hd = G.make_handle(cfg, G=1)
    b = G.binding.LayerBuffers(hd, False)
    hd.gate_topk(G.dev(X, "bf16"), G.dev(Wg), G.dev(bg), b.logits, b.idx, b.w)
    torch.cuda.synchronize()
    got = G.host(b.logits)
    assert np.array_equal(np.isnan(got), np.isnan(ref["logits"]))
    ok = ~np.isnan(got)
    assert np.array_equal(got.view(np.uint32)[ok], ref["logits"].view(np.uint32)[ok])
    assert np.array_equal(G.host(b.idx), ref["idx"])
    assert np.allclose(G.host(b.w), ref["w"], rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("T,d,E", [
    (1, 64, 4), (17, 128, 8), (16, 192, 12),                     # one wave per partial sum, one block of columns and more
    (33, 4160, 16), (100, 320, 20), (50, 256, 132),              # experts in blocks of 16, the last one partly empty
    (8200, 64, 16), (8193, 192, 16),                             # the last number of tokens with a block per 16, the first past it
    (4100, 320, 36), (5000, 128, 64), (3000, 192, 68),           # 64 tokens per block: three and four tiles of experts, two passes
    (5000, 320, 20), (16384, 192, 24), (16385, 448, 32),         # two tiles of experts: rings of three steps, the last T with them, of two
    (90, 128, 18),                                               # no multiple of four: the general kernel
    (33, 4096, 32), (49, 4160, 32), (20, 1024, 48), (65, 64, 36), (2000, 1024, 64), (30, 1088, 64), (17, 512, 52),   # experts of a
    (30, 512, 48), (30, 576, 48), (1025, 320, 64), (1024, 320, 64), (30, 256, 64),
    # block of 16 tokens in two, three and four units that route them, up to the longest rows, and past those
], ids=str)
def test_gate_logits_bit_for_bit(T, d, E):
    cfg = _cfg(T=T, d=d, E=E, k=min(2, E), P=1, renorm=1)
    rng = np.random.default_rng(T + d + E)
    X = wl.round_to_bf16(rng.standard_normal((T, d)).astype(np.float32))
    Wg = (rng.standard_normal((d, E)) * d ** -0.5).astype(np.float32)
    bg = rng.standard_normal(E).astype(np.float32)
    ref = orc.route(X, Wg, bg, cfg.k, 1)
    hd = G.make_handle(cfg, G=1)
    b = G.binding.LayerBuffers(hd, False)
    hd.gate_topk(G.dev(X, "bf16"), G.dev(Wg), G.dev(bg), b.logits, b.idx, b.w)
    torch.cuda.synchronize()
    assert np.array_equal(G.host(b.logits).view(np.uint32), ref["logits"].view(np.uint32))
    assert np.array_equal(G.host(b.idx), ref["idx"])
    assert np.allclose(G.host(b.w), ref["w"], rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("T,d,E,off", [
    (1, 4, 4, 0), (17, 68, 8, 0), (16, 192, 12, 1),              # one wave per partial sum; rows that end inside a block of columns
    (33, 4100, 16, 0), (100, 316, 20, 3), (50, 132, 132, 0),     # experts in blocks of 16, the last one partly empty
    (8200, 36, 16, 0), (8193, 100, 16, 0), (5000, 324, 20, 2),   # 64 tokens per block, one and two tiles of experts
    (4100, 260, 36, 0), (5000, 72, 64, 0), (3000, 132, 68, 0),   # four tiles of experts, two passes
    (40, 2048, 32, 0), (40, 2052, 32, 0), (31, 512, 48, 0), (700, 500, 64, 1), (15, 516, 64, 0), (64, 4, 20, 0),
    (16384, 60, 24, 0), (16385, 60, 24, 0), (16385, 64, 32, 3), (16400, 256, 20, 0), (16400, 260, 20, 0),    # one round of blocks, short rows past it
    (31, 516, 48, 0), (1500, 500, 64, 1), (30, 256, 64, 0), (30, 260, 64, 2),   # units, as above
    (90, 100, 18, 0),                                            # no multiple of four: the general kernel
], ids=str)
def test_fp32_gate_logits_bit_for_bit(T, d, E, off):
    """off: floats by which the tokens begin past a 16-byte boundary."""
    cfg = _cfg(T=T, d=d, E=E, k=min(2, E), P=1, renorm=1, dtype="f32")
    rng = np.random.default_rng(T + d + E)
    X = rng.standard_normal((T, d)).astype(np.float32)
    Wg = (rng.standard_normal((d, E)) * d ** -0.5).astype(np.float32)
    bg = rng.standard_normal(E).astype(np.float32)
    ref = orc.route(X, Wg, bg, cfg.k, 1)
    hd = G.make_handle(cfg, G=1)
    b = G.binding.LayerBuffers(hd, False)
    dX = torch.zeros(T * d + off, device=G.DEV)[off:]
    dX.copy_(G.dev(X, "f32").reshape(-1))
    hd.gate_topk(dX.view(T, d), G.dev(Wg), G.dev(bg), b.logits, b.idx, b.w)
    torch.cuda.synchronize()
    assert np.array_equal(G.host(b.logits).view(np.uint32), ref["logits"].view(np.uint32))
    assert np.array_equal(G.host(b.idx), ref["idx"])
    assert np.allclose(G.host(b.w), ref["w"], rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("x_off,w_off", [(1, 0), (2, 0), (6, 0), (0, 1), (3, 3)], ids=str)
@pytest.mark.parametrize("T,d,E", [(40, 128, 8), (8200, 64, 16), (700, 192, 48), (50, 256, 132)], ids=str)
def test_gate_of_operands_at_any_address(T, d, E, x_off, w_off):
    """Tokens that begin at any bf16, a gate matrix that begins at any float: the same bits."""
    cfg = _cfg(T=T, d=d, E=E, k=2, P=1, renorm=1)
    rng = np.random.default_rng(T + E)
    X = wl.round_to_bf16(rng.standard_normal((T, d)).astype(np.float32))
    Wg = (rng.standard_normal((d, E)) * d ** -0.5).astype(np.float32)
    bg = rng.standard_normal(E).astype(np.float32)
    ref = orc.route(X, Wg, bg, cfg.k, 1)

    def at(a, off, dtype):                            # the same values, `off` elements past a 16-byte boundary
        t = G.dev(a, dtype)
        flat = torch.zeros(t.numel() + off, dtype=t.dtype, device=G.DEV)[off:]
        assert flat.data_ptr() % 16 == off * t.element_size() % 16
        flat.copy_(t.reshape(-1))
        return flat.view(t.shape)

    hd = G.make_handle(cfg, G=1)
    b = G.binding.LayerBuffers(hd, False)
    hd.gate_topk(at(X, x_off, "bf16"), at(Wg, w_off, "f32"), G.dev(bg), b.logits, b.idx, b.w)
    torch.cuda.synchronize()
    assert np.array_equal(G.host(b.logits).view(np.uint32), ref["logits"].view(np.uint32))
    assert np.array_equal(G.host(b.idx), ref["idx"])
    assert np.allclose(G.host(b.w), ref["w"], rtol=1e-5, atol=1e-7)
