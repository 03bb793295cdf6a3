"""The lazy-reduction masks of the whole-row kernels (csrc/ntt_block.h), the digit ModUp (csrc/modup.hip) and the fused
row passes (csrc/fused_row.hip) against the bounds of the fp64 butterflies, in units of q: a reducing stage maps a
bound b to 1 + 0.375 b, a lazy one to 0.5 + 1.375 b, and every value must stay below 8 q.  Also the byte forms of the
balanced base-256 digits that the matrix-core projection multiplies, against their definition.
"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2609_12378_amd", "csrc")


def source(name):
    return open(os.path.join(CSRC, name)).read()


def run(b, mask, stages):
    peak = b
    for s in range(stages):
        b = (1 + 0.375 * b if (mask >> s) & 1 else 1.375 * b + 0.5) * (1 + 2.0 ** -40)
        peak = max(peak, b)
    return b, peak


def chain(text, fn):
    """{log2 points: mask} of a constexpr chain `s == 4 ? 0x0c : s == 5 ? ... : last`; the last under None."""
    body = re.search(r"constexpr unsigned %s\(int \w+\)\s*\{\s*return (.*?);\s*\}" % fn, text, re.S).group(1)
    out = {int(k): int(v, 16) for k, v in re.findall(r"== (\d) \? (0x[0-9a-f]+)", body)}
    out[None] = int(re.search(r"(0x[0-9a-f]+)\s*$", body).group(1), 16)
    return out


@pytest.mark.parametrize("logs", [4, 5, 6, 7, 8])
def test_digit_modup_passes(logs):
    text = source("modup.hip")
    cols = chain(text, "up_col_mask")
    row = int(re.search(r"constexpr unsigned kUpRowMask = (0x[0-9a-f]+);", text).group(1), 16)
    out, peak = run(1.0, cols.get(logs, cols[None]), logs)     # canonical residues of the conversion
    assert peak < 8 and out < 2
    out_r, peak_r = run(4.3, row, 8)                           # k_conv_col8's rows are below 4.3 q
    assert peak_r < 7 and out_r < 8


@pytest.mark.parametrize("logs", [4, 5, 6])
def test_whole_row_kernels(logs):
    text = source("ntt_block.h")
    cols = chain(text, "col_mask")
    row = int(re.search(r"constexpr unsigned kRowMask = (0x[0-9a-f]+);", text).group(1), 16)
    out, peak = run(1.0, cols.get(logs, cols[None]), logs)
    assert peak < 8 and out < 2
    out_r, peak_r = run(out, row, 8)
    assert peak_r < 8 and out_r < 8


def test_fused_row_passes():
    row = int(re.search(r"constexpr unsigned kRowMask = (0x[0-9a-f]+);", source("fused_row.hip")).group(1), 16)
    out, peak = run(4.3, row, 8)
    assert peak < 7 and out < 8


def test_balanced_digits_by_one_addition():
    k80 = 0x0080808080808080
    for v in [0, 1, 127, 128, 129, 255, 256, 0x7f7f, 0x8080, 0x7f80, 2 ** 50 - 1, 2 ** 50 - 129, 2 ** 49 + 0x80,
              0x2807f80ff017f]:
        digits, w = [], v
        for _ in range(7):                       # the definition: digits in [-128, 127], carry upwards
            t = w & 255
            w >>= 8
            if t >= 128:
                t, w = t - 256, w + 1
            digits.append(t & 255)
        assert w == 0
        x = (v + k80) ^ k80
        assert [(x >> (8 * a)) & 255 for a in range(7)] == digits
