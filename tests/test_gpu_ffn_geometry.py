"""The two tile geometries of the bf16 grouped FFN against a plain float64 product on the GPU, forward and backward, at the
sizes where a tile, a part of a split contraction or the choice between the two can go wrong: row counts around 128 and
256, widths that are odd multiples of 64, contractions of one pair of slices up to ones cut into eight parts, empty groups,
many groups, and shapes on both sides of the rule that picks the geometry; what the second list covers is asserted.
Tolerance as in test_gpu_parity.py: 1e-2 row by row, four roundings to bf16 (2^-9 each) with room for their spread."""
import numpy as np
import pytest
import torch

import gpu_util as G
from paper_2411_10003_amd import binding

pytestmark = pytest.mark.gpu

CASES = [
    # rows per hosted group, rows of other destinations behind them, d, h, activation
    ([1], 0, 64, 64, "gelu"),
    ([127, 0, 129], 5, 64, 192, "swiglu"),
    ([128, 1, 255, 257], 0, 320, 64, "gelu"),
    ([33], 10, 64, 4096, "swiglu"),                        # eight parts of 16 slices each
    ([200, 3], 0, 4160, 64, "gelu"),                       # parts that end at uneven slices
    ([40, 300], 7, 1088, 1600, "swiglu"),
    ([5] * 40, 0, 128, 192, "gelu"),                       # many groups, one ragged tile each
    ([0, 0, 0], 64, 64, 128, "swiglu"),                    # nothing to do
    ([700, 513, 90], 0, 448, 2112, "gelu"),
    ([14000, 3000], 0, 2112, 320, "swiglu"),               # many rows, contractions of ten slices
    ([30000], 0, 64, 1600, "gelu"),                        # and of one pair
    # few tiles of long contractions in the weight gradients: cut into parts, beside groups that are not
    ([9000, 200, 0, 33], 0, 320, 192, "swiglu"),
    ([4000], 100, 2944, 128, "gelu"),
    ([7000, 6500, 100, 6000, 31], 0, 1088, 448, "gelu"),
    ([300] * 20 + [8000], 0, 64, 320, "swiglu"),
]

# The same with what is covered: contraction -> side of its tiles and parts of a cut tile (weight gradients: of the group cut
# into most), as the library says it will run them.  (Many rows of other destinations make it expect more here than there are.)
PLANNED = [
    # row contractions in 256 x 256 tiles cut into two, three and four parts, at odd slices and over two segments (bwd2, swiglu)
    ([300, 3], 20000, 1856, 704, "gelu", dict(fwd1=(256, 2), bwd1=(256, 2))),
    ([300, 1, 257], 20000, 384, 2624, "gelu", dict(fwd2=(256, 3), bwd2=(256, 3))),
    ([400, 300, 257, 100], 20000, 704, 2624, "swiglu", dict(fwd2=(256, 3), bwd2=(256, 4))),
    ([300, 40], 20000, 192, 3136, "gelu", dict(fwd2=(256, 4), bwd2=(256, 4))),
    ([257], 20000, 1600, 640, "swiglu", dict(fwd1=(256, 2), fwd2=(256, 1), bwd1=(128, 3), bwd2=(256, 1))),
    # and left whole
    ([9000, 4000, 130], 64, 192, 2752, "swiglu", dict(fwd1=(256, 1), bwd1=(256, 1))),
    ([12000, 511, 7000], 0, 320, 3136, "gelu", dict(fwd1=(256, 1), fwd2=(256, 1), bwd1=(256, 1), bwd2=(256, 1))),
    # weight gradients in 256 x 256 tiles
    ([1500, 10], 30000, 1600, 1088, "swiglu", dict(bwd1=(256, 2), dW1=(256, 1), dW2=(256, 1))),
    ([15, 1657, 22, 3, 67], 20000, 448, 2816, "gelu", dict(dW1=(256, 2), dW2=(256, 2))),
    ([4, 3074, 20, 2, 8, 0, 26], 20000, 448, 2816, "gelu", dict(dW1=(256, 3), dW2=(256, 3))),
    ([9, 107, 1, 5603], 20000, 448, 2496, "swiglu", dict(dW1=(256, 4), dW2=(256, 4))),
    # what the workspace holds: two parts instead of three (two long groups of 60 tiles), seven instead of eight
    ([4, 193, 3886, 18, 2672], 20000, 1088, 2880, "swiglu", dict(dW1=(256, 2), dW2=(256, 2))),
    ([8471, 2907, 2273], 64, 704, 1152, "swiglu", dict(dW1=(128, 7), dW2=(128, 7))),
    # all parts of the weight gradients together are one per lane: fewer parts than a group alone would be cut into
    ([44000] + [20] * 59, 0, 64, 192, "gelu", dict(dW1=(128, 5), dW2=(128, 5))),
    ([40000, 40000] + [30] * 58, 0, 64, 64, "swiglu", dict(dW1=(128, 3), dW2=(128, 3))),
]


def _id(v):
    if isinstance(v, list):
        return f"{len(v)}g{sum(v)}r"
    return "-".join(f"{n}:{a}/{b}" for n, (a, b) in v.items()) if isinstance(v, dict) else str(v)


@pytest.mark.parametrize("rows,other,d,h,act,plan", [(*c, {}) for c in CASES] + PLANNED, ids=_id)
def test_forward_backward(rows, other, d, h, act, plan):
    Gn, M, A = len(rows), sum(rows), sum(rows) + other
    E = Gn + 1                                             # the last expert belongs to another destination
    g = torch.Generator(device=G.DEV).manual_seed(d + h + M)

    def rnd(*shape, std=1.0):
        return (torch.randn(*shape, generator=g, device=G.DEV) * std).to(torch.bfloat16)

    hd = binding.Handle(T=A, d=d, h=h, E=E, k=1, P=2, self_dest=0, G=Gn, dtype="bf16", act=act, renorm=0, device=G.DEV)
    tiling = G.ffn_tiling(hd, rows)
    for name, want in plan.items():
        t = tiling[name]
        assert (t["side"], max(t["parts"]) if name[0] == "d" else t["parts"]) == want, (name, t)
    idx = torch.repeat_interleave(torch.arange(E, dtype=torch.int32), torch.tensor(rows + [other])).to(G.DEV)
    dest = torch.tensor([0] * Gn + [1], dtype=torch.int32, device=G.DEV)
    counts, lay = torch.zeros(E, dtype=torch.int32, device=G.DEV), hd.new_layout()
    Xp, dYp = torch.empty(A, d, dtype=torch.bfloat16, device=G.DEV), rnd(A, d)
    hd.expert_counts(idx, counts)
    hd.dispatch(dest, rnd(A, d), idx, counts, lay, Xp)     # idx is sorted: rows stay where they are
    W1, W2 = rnd(Gn, d, h, std=d ** -0.5), rnd(Gn, h, d, std=h ** -0.5)
    W3 = rnd(Gn, d, h, std=d ** -0.5) if act == "swiglu" else None
    fill = rnd(A, max(d, h))
    Yp, dXp, Z = (fill[:, :w].contiguous().clone() for w in (d, d, h))
    U = Z.clone() if act == "swiglu" else None
    dW = [torch.full((Gn, d, h), 7.0, device=G.DEV), torch.full((Gn, h, d), 7.0, device=G.DEV),
          torch.full((Gn, d, h), 7.0, device=G.DEV) if act == "swiglu" else None]
    hd.expert_ffn_fwd(Xp, lay, W1, W2, W3, Yp, Z, U)
    hd.expert_ffn_bwd(dYp, Xp, Z, U, lay, W1, W2, W3, dXp, *dW)
    # added to what the buffers hold: doubling is exact in fp32
    acc = [t.clone() if t is not None else None for t in dW]
    hd.expert_ffn_bwd_acc(dYp, Xp, Z, U, lay, W1, W2, W3, dXp, *acc)
    torch.cuda.synchronize()
    assert all(t is None or torch.equal(a, 2 * t) for t, a in zip(dW, acc))
    for t, w in ((Yp, d), (dXp, d), (Z, h)) + (((U, h),) if act == "swiglu" else ()):
        assert torch.equal(t[M:], fill[M:, :w]), "rows of other destinations were touched"

    # A hidden unit's gradient in a group of a few rows is one activation, or a few, times dYp: act(z) from a z rounded to
    # bf16 is off by up to |z act'(z) / act(z)| 2^-9 of itself, which grows like z^2 in the negative tail (0.014 at z = -2.5),
    # while the whole gradient stays within 2^-9 of its norm.  So weight gradients are measured against the typical row.
    def close(got, want, what):
        G.assert_rows_close(G.host(got), want.cpu().numpy(), 1e-2, what, floor=1.0 if what.startswith("dW") else 0.02)

    o = 0
    for i, n in enumerate(rows):
        if n == 0:
            assert all(t is None or not bool(t[i].any()) for t in dW)
            continue
        x, dy = Xp[o:o + n].double(), dYp[o:o + n].double()
        w1, w2 = W1[i].double(), W2[i].double()
        z = x @ w1
        dA = dy @ w2.t()
        if act == "swiglu":
            w3 = W3[i].double()
            u, sg = x @ w3, torch.sigmoid(z)
            a, du, dz = z * sg * u, dA * z * sg, dA * u * (sg * (1 + z * (1 - sg)))
            dx = dz @ w1.t() + du @ w3.t()
            close(U[o:o + n], u, "U")
            close(dW[2][i], x.t() @ du, "dW3")
        else:
            cdf = 0.5 * (1 + torch.erf(z * 0.5 ** 0.5))
            a, dz = z * cdf, dA * (cdf + z * torch.exp(-0.5 * z * z) * (2 * np.pi) ** -0.5)
            dx = dz @ w1.t()
        close(Z[o:o + n], z, "Z")
        close(Yp[o:o + n], a @ w2, "Yp")
        close(dXp[o:o + n], dx, "dXp")
        close(dW[0][i], x.t() @ dz, "dW1")
        close(dW[1][i], a.t() @ dy, "dW2")
        o += n


# Tiles left over by the full rounds that are more than half of the blocks: each cut in two unevenly, two to four remainders per
# block.  Contraction -> side of the tiles and slices of the first part.  (No group of a few rows, for the sake of the weight
# gradients: of two rows a hidden unit's gradient is one activation times dYp, and one three times the typical, off by its three
# roundings, 3 x 3^0.5 x 2^-9 = 1.0e-2 of the typical row, is no error.)
UNEVEN = [
    ([7230, 7370, 2263, 590, 2238], 0, 320, 3584, "gelu", dict(fwd2=(256, 84), bwd2=(256, 84))),
    ([5254, 86, 272, 495, 4572], 20000, 576, 1792, "swiglu", dict(bwd2=(256, 84))),        # the remainder in the second segment
    ([4108, 3421, 7092], 0, 576, 2560, "swiglu", dict(bwd2=(256, 132))),                   # three remainders
    ([2859, 6751], 20000, 1088, 3136, "swiglu", dict(bwd2=(256, 168))),                    # four, the last block has three
    ([1662, 5275, 1374, 1478, 1981], 0, 320, 3840, "gelu", dict(fwd2=(128, 90), bwd2=(128, 90))),
    ([74, 7199, 7190], 0, 320, 2496, "swiglu", dict(bwd2=(128, 128))),
    ([1375, 7446], 0, 1344, 1984, "swiglu", dict(bwd2=(128, 92))),                         # after a full round
]


def _uneven(hd, rows, plan, cus=None):
    tiling = G.ffn_tiling(hd, rows, cus)
    for name, want in plan.items():
        assert (tiling[name]["side"], tiling[name]["first"]) == want and tiling[name]["parts"] == 1, (name, tiling[name])


@pytest.mark.parametrize("rows,other,d,h,act,plan", UNEVEN, ids=_id)
def test_uneven_cuts(rows, other, d, h, act, plan):
    """Right, and the same bits whatever the workspace held and whichever part of a tile came last."""
    test_forward_backward(rows, other, d, h, act, {})
    Gn, A = len(rows), sum(rows) + other
    hd = binding.Handle(T=A, d=d, h=h, E=Gn + 1, k=1, P=2, self_dest=0, G=Gn, dtype="bf16", act=act, renorm=0, device=G.DEV)
    _uneven(hd, rows, plan)
    g = torch.Generator(device=G.DEV).manual_seed(1)
    rnd = lambda *s: torch.randn(*s, generator=g, device=G.DEV).to(torch.bfloat16)   # noqa: E731
    counts, lay = torch.tensor(rows + [other], dtype=torch.int32, device=G.DEV), hd.new_layout()
    idx = torch.repeat_interleave(torch.arange(Gn + 1, dtype=torch.int32, device=G.DEV), counts)
    Xp, dYp = torch.empty(A, d, dtype=torch.bfloat16, device=G.DEV), rnd(A, d)
    hd.dispatch(torch.tensor([0] * Gn + [1], dtype=torch.int32, device=G.DEV), rnd(A, d), idx, counts, lay, Xp)
    W = [rnd(Gn, d, h), rnd(Gn, h, d), rnd(Gn, d, h) if act == "swiglu" else None]
    dW = [torch.empty_like(w, dtype=torch.float32) if w is not None else None for w in W]
    seen = None
    for i in range(4):
        Yp, dXp, Z = torch.zeros_like(Xp), torch.zeros_like(Xp), torch.zeros(A, h, dtype=torch.bfloat16, device=G.DEV)
        U = torch.zeros_like(Z) if act == "swiglu" else None
        if i % 2 == 0:
            hd.ws.fill_(255)
        hd.expert_ffn_fwd(Xp, lay, *W, Yp, Z, U)
        if i % 2 == 0:
            hd.ws.fill_(1)
        hd.expert_ffn_bwd(dYp, Xp, Z, U, lay, *W, dXp, *dW)
        torch.cuda.synchronize()
        if seen is None:
            seen = (Yp, dXp)
        assert torch.equal(Yp.view(torch.int16), seen[0].view(torch.int16)) and torch.equal(dXp.view(torch.int16), seen[1].view(torch.int16))
