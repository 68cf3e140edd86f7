"""The rules that choose among paths with the same results (csrc/routes.hpp), compiled for the host: the sizes that a rule was
placed by fall on the side they were measured for."""
from routes_rules import rules  # noqa: F401


# group, k_max, pool, scores given, managed -> 0 head by head, 1 by groups, 2 by groups with the rows kept
ORDER = [
    # 64 sequences of 2 K to 16 K tokens, a tenth of each pool listed: lists of 1405 to 1433 for a pool of 14 336, 39.2 to 40 %
    ((4, 1405, 14336, 0, 0), 2), ((4, 1433, 14336, 0, 0), 2), ((4, 1433, 14336, 1, 0), 1), ((4, 1405, 14336, 1, 0), 1),
    ((4, 2048, 28672, 0, 0), 0), ((4, 2048, 28672, 1, 0), 0),                  # 28.6 %, lists of a selection
    ((8, 1434, 28672, 0, 0), 1), ((8, 2048, 28672, 1, 0), 1), ((8, 2150, 28672, 0, 0), 2), ((8, 1720, 28672, 0, 0), 1), ((8, 4096, 122880, 0, 0), 0),
    ((2, 1146, 14336, 0, 0), 0), ((2, 1147, 14336, 0, 0), 1), ((2, 14336, 14336, 0, 0), 1), ((2, 2000, 14336, 1, 0), 0),
    # managed loops: room for a seventh of the pool, for 2480 entries, for a twentieth
    ((4, 4096, 28704, 0, 1), 2), ((8, 8576, 60064, 0, 1), 2), ((2, 4096, 28704, 0, 1), 2), ((4, 2480, 29168, 0, 1), 2),
    ((4, 1434, 28672, 0, 1), 2), ((4, 1433, 28672, 0, 1), 0), ((8, 700, 28672, 0, 1), 0), ((2, 700, 28672, 0, 1), 0),
    ((1, 14336, 14336, 0, 0), 0), ((4, 100, 0, 0, 0), 0), ((4, 0, 14336, 0, 0), 0), ((8, 2147483647, 2147483647, 0, 0), 2),
]


def test_order_of_the_gather(rules):
    got = rules(*("order %d %d %d %d %d" % a for a, _ in ORDER))
    assert got == [want for _, want in ORDER]


# fp32, group, window, k_max, scores given -> the window's workgroups start first
FIRST = [((0, 4, 4096, 2048, 0), 0), ((0, 4, 4096, 2048, 1), 1), ((0, 1, 8192, 16, 0), 0), ((1, 4, 512, 60, 0), 1), ((1, 8, 1024, 1900, 0), 1),
         ((1, 1, 4096, 600, 0), 1), ((1, 1, 1024, 585, 0), 0), ((1, 1, 256, 1800, 0), 0), ((1, 1, 256, 1800, 1), 1)]


def test_which_part_of_a_shared_launch_starts_first(rules):
    got = rules(*("first %d %d %d %d %d" % a for a, _ in FIRST))
    assert got == [want for _, want in FIRST]


# fp32, head_dim, sequences * KV heads, group, window, pool, k_max -> the step takes two launches
SHORT = [
    ((1, 64, 4, 1, 256, 2048, 64), 1), ((0, 128, 8, 4, 256, 2048, 512), 1), ((0, 128, 8, 4, 256, 2048, 513), 0),
    ((1, 128, 8, 4, 256, 2048, 768), 1), ((1, 128, 8, 4, 256, 2048, 769), 0), ((1, 64, 8, 4, 256, 4096, 1536), 1), ((1, 64, 8, 4, 256, 4096, 1537), 0),
    ((0, 64, 64, 4, 256, 2048, 64), 1), ((0, 64, 65, 4, 256, 2048, 64), 0), ((0, 64, 32, 8, 256, 2048, 64), 1), ((0, 64, 33, 8, 256, 2048, 64), 0),
    ((0, 128, 8, 4, 256, 98304, 64), 1), ((0, 128, 8, 4, 256, 98305, 64), 0), ((0, 128, 8, 2, 256, 98305, 64), 0),
    ((0, 128, 8, 1, 256, 131072, 64), 1), ((0, 128, 8, 1, 256, 131073, 64), 0), ((0, 64, 8, 4, 256, 262144, 64), 1), ((0, 64, 8, 4, 256, 262145, 64), 0),
    ((0, 128, 8, 8, 256, 16384, 64), 1), ((0, 128, 8, 8, 256, 16385, 64), 0),
    # fp32 heads of 64 in groups of 8: the pool's keys and the list together
    ((1, 64, 8, 8, 1024, 16384, 1536), 1), ((1, 64, 8, 8, 1024, 32768, 1536), 0), ((1, 64, 32, 8, 1024, 12800, 64), 1), ((1, 64, 29, 8, 374, 17015, 141), 1),
    ((1, 64, 32, 8, 300, 32768, 64), 1), ((1, 64, 32, 8, 300, 32769, 64), 0), ((1, 64, 32, 8, 1024, 12800, 640), 0),
    ((1, 128, 32, 8, 1024, 64000, 768), 1), ((1, 64, 64, 4, 1024, 64000, 1536), 1),
    # more workgroups than a flat grid has numbers for
    ((1, 64, 256, 1, 256, 2000000, 64), 1), ((1, 64, 256, 1, 256, 2200000, 64), 0),
    ((1, 64, 4, 1, 0, 2048, 64), 0), ((1, 64, 4, 1, 256, 0, 64), 0), ((1, 64, 4, 1, 256, 2048, 0), 0),
]


def test_short_steps(rules):
    got = rules(*("short %d %d %d %d %d %d %d" % a for a, _ in SHORT))
    assert got == [want for _, want in SHORT]
