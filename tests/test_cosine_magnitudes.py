"""The block decoder shares products between outputs of the inverse DCT: every
table entry fp32(C(k)/2 cos((2n + 1) k pi / 16)) is, bit for bit, one of the
eight fp32(C(k)/2 cos(k pi / 16)) it holds, up to the sign."""
import math

import numpy as np


def _c(k, n):
    return np.float32((math.sqrt(0.5) if k == 0 else 1.0) / 2.0 *
                      math.cos((2.0 * n + 1.0) * k * math.pi / 16.0))


# (index into c, sign) of entry (k, n), n = 0..3, as the kernel pairs them
PAIRS = {0: [(0, 1), (0, 1), (0, 1), (0, 1)], 1: [(1, 1), (3, 1), (5, 1), (7, 1)],
         2: [(2, 1), (6, 1), (6, -1), (2, -1)], 3: [(3, 1), (7, -1), (1, -1), (5, -1)],
         4: [(4, 1), (4, -1), (4, -1), (4, 1)], 5: [(5, 1), (1, -1), (7, 1), (3, 1)],
         6: [(6, 1), (2, -1), (2, 1), (6, -1)], 7: [(7, 1), (5, -1), (3, 1), (1, -1)]}


def test_every_entry_is_a_held_magnitude():
    held = [_c(k, 0) for k in range(8)]
    # the library's host code evaluates the angle as k pi / 16
    assert held == [np.float32((math.sqrt(0.5) if k == 0 else 1.0) / 2.0 *
                               math.cos(k * math.pi / 16.0)) for k in range(8)]
    for k, row in PAIRS.items():
        for n, (i, sign) in enumerate(row):
            assert _c(k, n) == np.float32(sign) * held[i], (k, n)
