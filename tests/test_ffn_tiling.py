"""How the bf16 FFN says it lays out a contraction, without a GPU: arguments, and that every cut stays inside the workspace
and the lanes it is made for."""
import ctypes
import random

import pytest

import gpu_util as G
from paper_2411_10003_amd import binding


def _handle(rows, other, d, h, act="gelu", dtype="bf16", G_cap=None, E=None):
    n = len(rows) if G_cap is None else G_cap
    return binding.Handle(T=sum(rows) + other, d=d, h=h, E=n + 1 if E is None else E, k=1, P=1, self_dest=0, G=n, dtype=dtype, act=act,
                          renorm=0, alloc_workspace=False)


def test_arguments():
    lib, hd = binding.load(), _handle([100, 200], 0, 128, 256)
    r, out = (ctypes.c_int32 * 2)(100, 200), (ctypes.c_int32 * 80)()
    assert lib.moe_ffn_tiling(hd._h, 0, 256, 2, r, out) == 0
    assert lib.moe_ffn_tiling(None, 0, 256, 2, r, out) == -1 and lib.moe_ffn_tiling(hd._h, 0, 256, 2, None, out) == -1
    assert lib.moe_ffn_tiling(hd._h, 6, 256, 2, r, out) == -2 and lib.moe_ffn_tiling(hd._h, 0, 256, 3, r, out) == -2
    f32 = _handle([100, 200], 0, 128, 256, dtype="f32")
    assert lib.moe_ffn_tiling(f32._h, 0, 256, 2, r, out) == -5


@pytest.mark.parametrize("seed", range(4))
def test_cuts_fit(seed):
    rng = random.Random(seed)
    cut = {k: 0 for k in ((128, "row"), (256, "row"), (128, "wgrad"), (256, "wgrad"))}
    for _ in range(400):
        n = rng.choice([1, 2, 4, 7, 17, 30, 64])
        rows = [int(10 ** rng.uniform(0, 4)) for _ in range(n)]
        d, h = 64 * rng.randint(1, 40), 64 * rng.randint(1, 80)
        hd = _handle(rows, rng.choice([0, 20000]), d, h, rng.choice(["gelu", "swiglu"]))
        for name, t in G.ffn_tiling(hd, rows, 256).items():
            side, units = t["side"], 320 * (256 // t["side"]) ** 2
            assert side in (128, 256) and t["blocks"] == (512 if side == 128 else 256)
            tiles = t["row_tiles"] * t["col_tiles"]
            if name[0] == "d":
                assert all(1 <= p <= (8 if side == 128 else 4) for p in t["parts"])
                assert sum(t["parts"]) <= 64 and sum(p for p in t["parts"] if p > 1) * tiles <= units
                cut[side, "wgrad"] += max(t["parts"]) > 1
                assert t["finish"] or max(t["parts"]) == 1
            else:
                assert t["row_tiles"] == len(G.ffn_row_tiles([(0, x) for x in rows], side))
                rest = tiles - t["n_full"]
                assert t["n_full"] % t["blocks"] == 0 and 0 <= rest < t["blocks"]
                assert t["parts"] == 1 or (t["finish"] and rest > 0 and rest * t["parts"] <= min(units, t["blocks"]) and t["slices"] >= 16 * t["parts"])
                assert len(G.ffn_split_tiles(t)) == (rest if t["parts"] > 1 else 0)
                cut[side, "row"] += t["parts"] > 1
    assert all(cut.values()), cut


@pytest.mark.parametrize("n,rows,d,h", [(8, 3276, 256, 512), (16, 5000, 64, 64), (8, 1866, 384, 512), (24, 2000, 128, 448), (17, 3276, 256, 512)])
def test_groups_that_fill_the_xcds_stay_whole(n, rows, d, h):
    """Eight equal groups, or more, keep the eight XCDs busy whole: cutting them adds a finishing launch and shortens nothing."""
    t = G.ffn_tiling(_handle([rows] * n, 0, d, h), [rows] * n, 256)
    for name in ("dW1", "dW2"):
        assert t[name]["parts"] == [1] * n, name


@pytest.mark.parametrize("n,rows,d,h,E", [(3, 1982, 1280, 1792, 12), (6, 2128, 1728, 64, 24), (6, 1286, 64, 2112, 24)])
def test_cuts_that_would_not_pay_are_not_made(n, rows, d, h, E):
    """Fewer groups than XCDs, but as many rounds or nearly: parts of them would take the XCDs as long as the whole groups."""
    t = G.ffn_tiling(_handle([rows] * n, rows * n, d, h, E=E), [rows] * n, 256)
    for name in ("dW1", "dW2"):
        assert t[name]["parts"] == [1] * n, name


def test_long_groups_are_cut():
    rows = [9000, 200, 0, 33]
    t = G.ffn_tiling(_handle(rows, 0, 320, 192), rows, 256)
    for name in ("dW1", "dW2"):
        assert t[name]["parts"] == [8, 1, 1, 1] and t[name]["finish"] == 1, name


@pytest.mark.parametrize("rows,d,h", [([9000] + [1000] * 30, 256, 512), ([30000] + [400] * 23, 512, 256), ([44000] + [20] * 30, 64, 64)], ids=lambda v: str(len(v)) if isinstance(v, list) else str(v))
def test_long_groups_among_many_are_cut(rows, d, h):
    t = G.ffn_tiling(_handle(rows, 0, d, h), rows, 256)
    for name in ("dW1", "dW2"):
        assert t[name]["finish"] == 1, name
        if rows[0] > 20 * rows[1]:
            assert t[name]["parts"][0] > 1 and t[name]["parts"][1:] == [1] * (len(rows) - 1), name


@pytest.mark.parametrize("rows,d,h,want", [
    ([44000] + [20] * 59, 64, 192, 5),                         # 60 groups leave four lanes: five parts instead of eight
    ([40000, 40000] + [30] * 58, 64, 64, 3),                   # shared by two
    ([44000] + [20] * 63, 64, 64, 1),                          # a lane for each group and none left
    ([44000] + [20] * 56, 64, 64, 8),                          # just enough
], ids=lambda v: str(len(v)) if isinstance(v, list) else str(v))
def test_more_parts_than_lanes(rows, d, h, want):
    """All parts together are at most 64: long groups are cut into fewer parts, not left whole."""
    t = G.ffn_tiling(_handle(rows, 0, d, h), rows, 256)
    for name in ("dW1", "dW2"):
        parts = t[name]["parts"]
        n = sum(r > 1000 for r in rows)
        assert parts[:n] == [want] * n and parts[n:] == [1] * (len(rows) - n) and sum(parts) <= 64, (name, parts)


def test_uneven_cuts_fit():
    """Two units per tile in the workspace, both parts whole pairs of slices, and a remainder worth its way."""
    rng, seen = random.Random(5), set()
    for _ in range(3000):
        rows = [int(10 ** rng.uniform(0, 4)) for _ in range(rng.choice([1, 3, 8]))]
        d, h = 64 * rng.randint(1, 40), 64 * rng.randint(20, 120)
        hd = _handle(rows, rng.choice([0, 20000]), d, h, rng.choice(["gelu", "swiglu"]))
        for name, t in G.ffn_tiling(hd, rows, 256).items():
            if name[0] == "d" or not t["first"]:
                continue
            rem, rest = t["row_tiles"] * t["col_tiles"] - t["n_full"], t["slices"] - t["first"]
            assert name in ("fwd2", "bwd2") and t["parts"] == 1
            assert t["blocks"] // 2 < rem < t["blocks"] and 2 * rem * t["side"] ** 2 <= 512 * 256 ** 2
            assert t["first"] % 2 == 0 and rest % 2 == 0 and rest >= 28 and t["first"] >= rest
            seen.add((t["side"], -(-rem // (t["blocks"] - rem))))
    assert {(256, 2), (256, 3), (128, 2), (128, 3)} <= seen


@pytest.mark.parametrize("act,longest", [("gelu", 3584), ("swiglu", 1792)])
def test_workspace_for_uneven_cuts_only_where_they_are_made(act, longest):
    """320 partial tiles of 256 x 256 floats, 512 from the shortest contraction over h that may be cut unevenly."""
    def rest(h):                                               # beside the T x h intermediates
        return _handle([128], 0, 64, h, act).workspace_bytes - (3 if act == "swiglu" else 2) * 128 * h * 2
    tile = 256 * 256 * 4
    assert 320 * tile < rest(64) < 321 * tile
    assert rest(longest - 64) == rest(64) and rest(longest) == rest(64) + 192 * tile == rest(2 * longest)
    rng, seen = random.Random(6), 0
    for _ in range(600):                                       # every cut that is made finds its place
        rows, h = [int(10 ** rng.uniform(2, 4)) for _ in range(rng.choice([1, 3, 8]))], 64 * rng.randint(20, 80)
        hd = _handle(rows, 0, 64 * rng.randint(1, 40), h, act)
        for t in G.ffn_tiling(hd, rows, 256).values():
            if t.get("first"):
                assert 2 * (t["row_tiles"] * t["col_tiles"] - t["n_full"]) * t["side"] ** 2 * 4 <= 512 * tile and h >= longest
                seen += 1
    assert seen


def test_what_is_read_past_the_caches():
    """Weights of more than 256 MB (2^28 bytes) altogether, of batches of one row tile."""
    lib = binding.load()

    def once(T, d, h, act, groups=4):
        hd = binding.Handle(T=T, d=d, h=h, E=16, k=1, P=2, self_dest=0, G=groups, dtype="bf16", act=act, renorm=0, alloc_workspace=False)
        sides = [G.ffn_tiling(hd, [T], 256)[c]["side"] for c in ("fwd1", "fwd2")]
        return sides, [lib.moe_ffn_reads_once(hd._h, c) for c in (0, 1)]
    assert once(64, 2048, 8192, "gelu") == ([128, 128], [0, 0])                     # 2^28 bytes
    assert once(64, 2048, 8256, "gelu") == ([128, 128], [1, 1])
    assert once(64, 512, 2048, "swiglu") == ([128, 128], [0, 0])                    # 25 MB
    assert once(128, 4096, 14336, "swiglu") == ([256, 128], [1, 1]) and once(129, 4096, 14336, "swiglu") == ([256, 128], [1, 0])
    assert once(256, 4096, 14336, "swiglu")[1] == [1, 0] and once(257, 4096, 14336, "swiglu")[1] == [0, 0]
    assert once(128, 4096, 14336, "gelu") == ([128, 128], [1, 1]) and once(129, 4096, 14336, "gelu")[1] == [0, 0]
    assert lib.moe_ffn_reads_once(None, 0) == -1
