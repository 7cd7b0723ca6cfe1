"""Forward passes of a batch that fits one row tile (a decoding step), whose weights are requested past the caches: against a
float64 product, and bit for bit against a batch with more rows of other destinations, which is tiled alike and reads its weights the
other way.  Rows on both sides of the line for either geometry (128, 256)."""
import pytest
import torch

import gpu_util as G
from paper_2411_10003_amd import binding

pytestmark = pytest.mark.gpu


def _forward(rows, other, X, W, d, h, act):
    Gn, A = len(rows), sum(rows) + other
    hd = binding.Handle(T=A, d=d, h=h, E=Gn + 1, k=1, P=2, self_dest=0, G=Gn, dtype="bf16", act=act, renorm=0, device=G.DEV)
    idx = torch.tensor([e for e, n in enumerate([*rows, other]) for _ in range(n)], dtype=torch.int32, device=G.DEV).view(A, 1)
    counts, lay = torch.zeros(Gn + 1, dtype=torch.int32, device=G.DEV), hd.new_layout()
    x = torch.zeros(A, d, dtype=torch.bfloat16, device=G.DEV)
    x[:sum(rows)] = X
    Xp, Yp = torch.zeros_like(x), torch.zeros_like(x)
    hd.expert_counts(idx, counts)
    hd.dispatch(torch.tensor([0] * Gn + [1], dtype=torch.int32, device=G.DEV), x, idx, counts, lay, Xp)
    hd.expert_ffn_fwd(Xp, lay, *W, Yp, None, None)
    torch.cuda.synchronize()
    t = G.ffn_tiling(hd, rows)
    return Yp[:sum(rows)], [(t[c]["side"], t[c]["parts"], t[c].get("first")) for c in ("fwd1", "fwd2")]


@pytest.mark.parametrize("rows,d,h,act", [
    ([1], 64, 64, "gelu"),
    ([100, 28], 320, 1088, "swiglu"),                          # 128 rows
    ([100, 29], 320, 1088, "swiglu"),
    ([128, 0, 128], 1088, 192, "gelu"),                        # 256 rows
    ([129, 128], 1088, 192, "gelu"),
    ([40, 3, 21], 1024, 4160, "swiglu"),                       # contractions that are cut
    ([90, 60, 50, 56], 2112, 3136, "gelu"),
])
def test_few_rows(rows, d, h, act):
    Gn, M = len(rows), sum(rows)
    g = torch.Generator(device=G.DEV).manual_seed(d + h + M)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=g, device=G.DEV) * std).to(torch.bfloat16)   # noqa: E731
    X, W1, W2 = rnd(M, d), rnd(Gn, d, h, std=d ** -0.5), rnd(Gn, h, d, std=h ** -0.5)
    W3 = rnd(Gn, d, h, std=d ** -0.5) if act == "swiglu" else None
    Y, tiling = _forward(rows, 0, X, (W1, W2, W3), d, h, act)
    r0 = 0
    for e, n in enumerate(rows):
        x = X[r0:r0 + n].double()
        z = x @ W1[e].double()
        a = torch.nn.functional.silu(z) * (x @ W3[e].double()) if W3 is not None else torch.nn.functional.gelu(z)
        if n:
            # two roundings to bf16 (2^-9 each), with room for their spread over a row
            G.assert_rows_close(G.host(Y[r0:r0 + n]), (a @ W2[e].double()).cpu().numpy(), 1e-2, f"group {e}")
        r0 += n
    for other in (257, 300, 400):
        Z, same = _forward(rows, other, X, (W1, W2, W3), d, h, act)
        if same == tiling:
            assert torch.equal(Y, Z)
