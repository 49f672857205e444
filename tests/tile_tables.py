"""The tile tables of the GEMM sources and the choice they lead to, read from
the sources, so that the shapes of the tile tests can be held to them."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2205_02491_amd", "csrc")
NCU = 256
# (n, k), odd and ragged, so that every entry of every table below is taken
SHAPES = [(65, 17), (371, 171), (515, 241), (629, 297), (707, 339), (713, 353), (803, 381),
          (821, 395), (1025, 493), (1121, 549), (1283, 577), (1475, 675), (1745, 871),
          (2435, 773), (3329, 899)]
# FP32 products of the staged kernel: real and complex, with the FP32 copy of H
# (columns off the cache lines, large blocks) and without
STAGED_SHAPES = [(4001, 1001), (5003, 1201), (8001, 401), (9601, 801)]
# the same for the INT8 products' column widths, 14 moduli
INT8_SHAPES = [(33, 5), (257, 97), (393, 193), (521, 257), (769, 193), (769, 257), (1025, 385),
               (1161, 577), (1537, 513)]


def table(function):
    src = open(os.path.join(CSRC, "gemm.hip")).read()
    body = src[src.index(f"void {function}("):]
    rows = re.search(r"Tile t\[\] = \{(.*?)\};", body, re.S).group(1)
    return [tuple(int(x) for x in e) for e in re.findall(r"\{\s*(\d+),\s*(\d+),\s*(\d+)\}", rows)]


def tiles(m, n, tm, tn):
    return -(-m // tm) * -(-n // tn)


def choose(t, m, n):
    """Tile of an m x n result: least rounds of 256 tiles, times area over rate,
    the earlier one on a tie."""
    return min(t, key=lambda e: -(-tiles(m, n, e[0], e[1]) // NCU) * e[0] * e[1] / e[2])[:2]


def int8_widths():
    src = open(os.path.join(CSRC, "crt.hip")).read()
    body = src[src.index("void crt_gemm("):]
    rows = re.search(r"tiles\[\] = \{(.*?)\};", body, re.S).group(1)
    return [tuple(int(x) for x in e) for e in re.findall(r"\{\s*(\d+),\s*(\d+)\}", rows)]


def int8_width(t, n, k, planes):
    return min(t, key=lambda e: -(-tiles(n, k, 256, 32 * e[0]) * planes // NCU) * e[0] / e[1])[0]
