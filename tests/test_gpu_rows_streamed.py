"""Rows of 64 MB and more, which go out by nontemporal stores: every token bit for bit as calls of so few tokens that all their rows are
under the line (plain stores) leave it, the scatter against the rows it copies, the gate's parameter gradients against float64."""
import pytest
import torch

import gpu_util as G
from paper_2411_10003_amd import binding

pytestmark = pytest.mark.gpu
E = 8
LINE = 64 << 20


def _handle(T, d, k, dtype):
    return binding.Handle(T=T, d=d, h=64, E=E, k=k, P=4, self_dest=0, G=2, dtype=dtype, act="gelu", renorm=0, device=G.DEV)


@pytest.mark.parametrize("T,d,k,dtype", [
    (8192, 4096, 1, "bf16"),                                   # all calls exactly at the line
    (8191, 4096, 2, "bf16"),                                   # just under it for T x d, over it for T k x d
    (8193, 4160, 2, "bf16"),
    (8199, 4096, 3, "bf16"),                                   # any number of experts per token
    (8200, 4096, 4, "bf16"),
    (4097, 4096, 2, "f32"),
])
def test_streamed_rows(T, d, k, dtype):
    g = torch.Generator(device=G.DEV).manual_seed(T + d + k)
    hd = _handle(T, d, k, dtype)
    e, A, dev = hd.elt, T * k, dict(device=G.DEV)
    rand = lambda *s: torch.randn(*s, generator=g, **dev)      # noqa: E731
    X, Yp, dOut, dXp = rand(T, d).to(e), rand(A, d).to(e), rand(T, d).to(e), rand(A, d).to(e)
    w, dl, Wg = rand(T, k), rand(T, E), rand(d, E)
    idx = rand(T, E).topk(k, dim=1).indices.int()
    counts, lay = torch.zeros(E, dtype=torch.int32, **dev), hd.new_layout()
    Xp = torch.zeros(A, d, dtype=e, **dev)
    hd.expert_counts(idx, counts)
    hd.dispatch((torch.arange(E, **dev) // 2).int(), X, idx, counts, lay, Xp)
    assert torch.equal(Xp, X[(lay.perm // k).long()])

    def run(hd, t0, t1, out, dYp, dw, dX, dXs):
        pos = lay.pos[t0 * k:t1 * k]
        hd.combine(Yp, pos, w[t0:t1], out[t0:t1])
        hd.combine_bwd(dOut[t0:t1], Yp, pos, w[t0:t1], dYp, dw[t0:t1])
        hd.input_grad(dXp, pos, dl[t0:t1], Wg, dX[t0:t1])
        hd.dispatch_bwd(dXp, pos, dXs[t0:t1])

    row = k * d * X.element_size()                             # of a token, in the widest of the calls (gradient of the combine)
    n = next(n for n in range(2, 99) if -(-T // n) * row < LINE)
    assert T * row >= LINE
    outs = []
    for parts in (1, n):
        bufs = [torch.full((T, d), 3.0, dtype=e, **dev), torch.full((A, d), 3.0, dtype=e, **dev), torch.full((T, k), 3.0, **dev),
                torch.full((T, d), 3.0, dtype=e, **dev), torch.full((T, d), 3.0, dtype=e, **dev)]
        cuts = [T * i // parts for i in range(parts + 1)]
        for t0, t1 in zip(cuts, cuts[1:]):
            assert parts == 1 or (t1 - t0) * row < LINE
            run(hd if parts == 1 else _handle(t1 - t0, d, k, dtype), t0, t1, *bufs)
        torch.cuda.synchronize()
        outs.append(bufs)
    for name, a, b in zip(("out", "dYp", "dw", "dX", "backward of the send"), *outs):
        assert torch.equal(a, b), name

    dWg, dbg = torch.zeros(d, E, **dev), torch.zeros(E, **dev)
    hd.gate_bwd_params(X, dl, dWg, dbg)
    want, terms = X.double().t() @ dl.double(), X.double().abs().t() @ dl.double().abs()
    # chains of at most 256 additions, 64 partials in four sums: 2^-24 relative to the terms each
    assert bool(((dWg.double() - want).abs() <= 512 * 2.0 ** -24 * terms).all())
    assert bool(((dbg.double() - dl.double().sum(0)).abs() <= 512 * 2.0 ** -24 * dl.double().abs().sum(0)).all())
