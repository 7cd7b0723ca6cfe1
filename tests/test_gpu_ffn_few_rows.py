"""Forward passes of a batch that fits one row tile (a decoding step).  Where their weights are more than the caches keep these are
requested past the caches: against a float64 product, and bit for bit against a batch of a few more rows, of other destinations, that
is tiled alike and reads its weights the other way.  Each entry says how the library lays out either contraction (side of a tile, parts
of a tile that is cut, whether it is cut unevenly) and which of them reads past the caches."""
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
    t = G.ffn_tiling(hd, rows, 256)
    return (Yp[:sum(rows)], [(t[c]["side"], t[c]["parts"], t[c]["first"] > 0) for c in ("fwd1", "fwd2")],
            tuple(hd.lib.moe_ffn_reads_once(hd._h, c) for c in (0, 1)))


SMALL = [                                                      # layers whose weights may stay in the caches
    ([1], 64, 64, "gelu"),
    ([100, 28], 320, 1088, "swiglu"),                          # 128 rows
    ([100, 29], 320, 1088, "swiglu"),
    ([128, 0, 128], 1088, 192, "gelu"),                        # 256 rows
    ([129, 128], 1088, 192, "gelu"),
    ([40, 3, 21], 1024, 4160, "swiglu"),                       # contractions that are cut
    ([90, 60, 50, 56], 2112, 3136, "gelu"),
]
WHOLE, CUT = [(128, 1, False)], [(128, 8, False)]
PAST = [
    # rows, rows of other destinations in the batch it is compared with, d, h, activation, layout, which are read past the caches
    ([17, 11, 11, 8, 8, 9], 130, 3392, 3328, "gelu", [(128, 3, False)] * 2, (1, 1)),
    ([29, 20, 25, 26, 28], 1, 576, 23872, "gelu", WHOLE + CUT, (1, 1)),                             # 128 rows
    ([15, 23, 24, 22, 19, 24], 2, 5696, 1984, "gelu", [(128, 5, False)] + WHOLE, (1, 1)),
    ([2, 3, 6, 1, 1, 3, 2, 2], 130, 4352, 4416, "gelu", WHOLE + [(128, 1, True)], (1, 1)),
    ([31, 27, 27, 23, 20], 1, 1024, 8832, "swiglu", [(128, 2, False)] + CUT, (1, 1)),
    ([8, 11, 10, 7, 12, 4, 6, 6], 130, 2304, 2432, "swiglu", WHOLE + [(128, 3, False)], (1, 1)),
    # both weight matrices of SwiGLU in 256 x 256 tiles: up to 256 rows
    ([62, 59, 64, 71], 1, 4352, 3328, "swiglu", [(256, 2, False), (128, 3, False)], (1, 0)),        # 256 rows
    ([51, 59, 59, 39, 48], 1, 1600, 6208, "swiglu", [(256, 1, False), (128, 7, False)], (1, 0)),
    ([55, 74], 130, 1728, 15040, "swiglu", [(256, 1, False)] + CUT, (1, 0)),
    ([7, 24, 15, 8, 15, 19, 17, 0], 30, 6400, 1024, "swiglu", [(256, 4, False)] + WHOLE, (1, 1)),   # fwd1 reads past the caches on both sides
]


@pytest.mark.parametrize("rows,other,d,h,act,layout,past", [(r, 0, d, h, a, None, (0, 0)) for r, d, h, a in SMALL] + PAST)
def test_few_rows(rows, other, d, h, act, layout, past):
    Gn, M = len(rows), sum(rows)
    g = torch.Generator(device=G.DEV).manual_seed(d + h + M)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=g, device=G.DEV) * std).to(torch.bfloat16)   # noqa: E731
    X, W1, W2 = rnd(M, d), rnd(Gn, d, h, std=d ** -0.5), rnd(Gn, h, d, std=h ** -0.5)
    W3 = rnd(Gn, d, h, std=d ** -0.5) if act == "swiglu" else None
    Y, tiling, once = _forward(rows, 0, X, (W1, W2, W3), d, h, act)
    assert once == past and layout in (None, tiling)
    r0 = 0
    for e, n in enumerate(rows):
        x = X[r0:r0 + n].double()
        z = x @ W1[e].double()
        a = torch.nn.functional.silu(z) * (x @ W3[e].double()) if W3 is not None else torch.nn.functional.gelu(z)
        if n:
            # two roundings to bf16 (2^-9 each), with room for their spread over a row
            G.assert_rows_close(G.host(Y[r0:r0 + n]), (a @ W2[e].double()).cpu().numpy(), 1e-2, f"group {e}")
        r0 += n
    if not other:
        return
    Z, same, plain = _forward(rows, other, X, (W1, W2, W3), d, h, act)
    assert same == tiling and sum(plain) < sum(once)
    assert torch.equal(Y, Z)
