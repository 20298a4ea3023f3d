"""Stored Wigner-d tables end in zeros, because the contraction kernels read
past a pair's degrees: on the last node of the last blocks that is past the
table.  The pair list of every plan is laid out here as the library does it and
the furthest element that any kernel reads is compared with the padding."""
import os
import re

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
INTERNAL = os.path.join(HERE, "..", "paper_2605_23923_amd", "csrc", "su2fft_internal.h")
PT = 16
BANDLIMITS = [B for B in range(1, 129) if any(2 * B == 2 ** a * 3 ** b for a in range(1, 9) for b in range(6))]


def _padding():
    with open(INTERNAL) as fh:
        m = re.search(r"constexpr int TABLE_PAD = (\d+);", fh.read())
    assert m, "TABLE_PAD"
    return int(m.group(1))


def _degrees(B, so3, symmetric):
    """Degrees per position of the pair list (0: padding)."""
    pairs = [(m, n) for m in range(-(B - 1), B) for n in range(-(B - 1), B)
             if (m - n) % 2 == 0 and not (so3 and m % 2)]
    L = [(B - 1 - max(abs(m), abs(n))) // 2 + 1 for m, n in pairs]
    if not symmetric:
        return L + [0] * (-len(L) % PT)
    low = [d for (m, _), d in zip(pairs, L) if m < 0]
    mid = [d for (m, _), d in zip(pairs, L) if m == 0]
    high = [d for (m, _), d in zip(pairs, L) if m > 0]
    pad = -len(low) % PT
    width = len(mid) + 1
    while width % PT:
        width += 2
    ends = (width - len(mid) - 1) // 2
    h = len(mid) // 2 + 1
    out = low + [0] * (pad + ends) + mid[:h] + [0] + mid[h:] + [0] * (ends + pad) + high
    assert len(out) % PT == 0
    return out


def _furthest(B, so3, symmetric):
    """Elements past the table's last value that the kernels read."""
    N, L = 2 * B, _degrees(B, so3, symmetric)
    tiles = [L[i:i + PT] for i in range(0, len(L), PT)]
    owners = (len(tiles) + 1) // 2 if symmetric else len(tiles)
    size, reads = 0, 0
    for tile in tiles[:owners]:
        lsum = sum(tile)
        rows = (max(tile) + 15) // 16  # row tiles that every pair of the tile reads through LDS
        column = size + (N - 1) * lsum
        for d in tile:
            if d:
                # adjacent values per row tile (three may be loaded as four); 32 degrees at a time in split BF16
                reads = max(reads, column + 15 * rows + (4 if rows == 3 else rows), column + 32 * ((d + 31) // 32))
            column += d
        size += N * lsum
    return reads - size


@pytest.mark.parametrize("so3", [False, True])
def test_padding_covers_the_furthest_read(so3):
    pad = _padding()
    worst = {(B, sym): _furthest(B, so3, sym) for B in BANDLIMITS for sym in (False, True)}
    assert all(v <= pad for v in worst.values()), {k: v for k, v in worst.items() if v > pad}
    if not so3:
        # 16 elements do not cover it: a pair of 29 degrees in a tile of 36
        assert worst[72, True] > 16
