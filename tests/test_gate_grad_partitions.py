"""Token partitions of the gate's parameter gradients, read from the workspace of fp32 handles (no GPU)."""
import random

import pytest

from paper_2411_10003_amd import binding


def _partitions(T, d, E):
    hd = binding.Handle(T=T, d=d, h=64, E=E, k=1, P=1, self_dest=0, G=1, dtype="f32", act="gelu", renorm=0, alloc_workspace=False)
    align = lambda n: -(-n // 256) * 256                       # noqa: E731
    rest = 256 + 2 * align(-(-T // 256) * E * 4) + 2 * align(T * 64 * 4)
    return (hd.workspace_bytes - rest) // ((d * E + E) * 4)


@pytest.mark.parametrize("T,d,E,n", [(64, 64, 8, 1), (65, 64, 8, 2), (4096, 64, 8, 64), (4097, 64, 8, 33), (4894, 1180, 16, 39), (8192, 64, 8, 64), (4894, 64, 40, 40)])
def test_whole_trips(T, d, E, n):
    assert _partitions(T, d, E) == n


def test_partials_are_worth_their_traffic_and_chains_stay_short():
    rng = random.Random(3)
    for _ in range(400):
        T, d, E = int(10 ** rng.uniform(0, 4.8)), 4 * rng.randint(1, 1024), rng.choice([1, 8, 16, 33, 128, 129, 256, 1024])
        n, least, trips = _partitions(T, d, E), min(32, -(-T // 256)), -(-T // 64)
        assert least <= n <= min(64, trips)                    # chains of 256 tokens, or a thirty-second of all, at most
        if n > least:
            fewest = -(-trips // -(-trips // n))               # no partition whose trips the others could take,
            assert n == fewest or (E > 32 and n % 8 == 0 and n <= max(fewest, least) * 9 / 8)    # but for eights of them
            assert E <= 128 or n * d * E * 4 <= 9 << 20
