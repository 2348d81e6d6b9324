"""rn_stats keeps the size it had before it told the route (the field lies in what
was padding), and the binding's bits are the header's."""
import ctypes as C
import os
import re

from paper_1607_07696_amd import rn

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "rn.h")


def test_stats_size():
    assert C.sizeof(rn.Stats) == 64 and rn.Stats.route.offset == 60


def test_route_bits():
    bits = re.findall(r"#define\s+(RN_ROUTE_\w+)\s+(\d+)", open(HEADER).read())
    assert len(bits) == 9
    for name, value in bits:
        assert getattr(rn, name) == int(value), name
