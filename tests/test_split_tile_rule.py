"""The tile of a BF16-split product against what was measured (256 compute
units): 64- over 128-tile time of the products of a refinement, at sizes where
one of them is at least 6% faster."""

import pytest

# (name, transpose A, transpose B, symmetric output)
KINDS = {"nn": (0, 0, 0), "tn": (1, 0, 1), "nt": (0, 1, 1)}

MEASURED = [
    # kind, n, batch, time with 64-tiles / time with 128-tiles
    ("nn", 1536, 1, 0.58), ("nn", 2016, 1, 0.68), ("nn", 2496, 1, 0.83), ("nn", 2784, 1, 1.06),
    ("nn", 2880, 1, 0.83), ("nn", 3264, 1, 1.10), ("nn", 3360, 1, 1.14), ("nn", 3456, 1, 1.21),
    ("nn", 3552, 1, 0.91), ("nn", 3648, 1, 0.90), ("nn", 3936, 1, 1.09), ("nn", 4096, 1, 1.07),
    ("nn", 4224, 1, 1.06), ("nn", 2501, 1, 0.57), ("nn", 3650, 1, 0.60), ("nn", 3999, 1, 0.68),
    ("nn", 2048, 3, 1.15), ("nn", 1536, 5, 1.13), ("nn", 3400, 2, 1.17), ("nn", 1024, 12, 1.13),
    ("nn", 1000, 33, 1.16), ("nn", 700, 30, 0.90), ("nn", 256, 150, 0.65), ("nn", 256, 300, 0.61),
    ("nn", 300, 64, 0.59),
    ("tn", 1536, 1, 0.37), ("tn", 2208, 1, 0.65), ("tn", 2784, 1, 0.73), ("tn", 3072, 1, 0.92),
    ("tn", 3552, 1, 1.23), ("tn", 3744, 1, 1.24), ("tn", 3936, 1, 1.29), ("tn", 4096, 1, 1.20),
    ("tn", 4224, 1, 1.18), ("tn", 3333, 1, 0.37), ("tn", 3650, 1, 0.44), ("tn", 3999, 1, 0.32),
    ("tn", 2048, 3, 1.13), ("tn", 1536, 5, 0.92), ("tn", 2600, 2, 1.08), ("tn", 3400, 2, 1.21),
    ("tn", 700, 30, 0.90), ("tn", 512, 64, 0.67), ("tn", 512, 100, 0.74), ("tn", 256, 300, 0.62),
    ("tn", 1024, 20, 0.79), ("tn", 1000, 33, 0.92),
    ("nt", 1536, 1, 0.32), ("nt", 2784, 1, 0.63), ("nt", 3456, 1, 0.74), ("nt", 3840, 1, 0.93),
    ("nt", 4096, 1, 0.85), ("nt", 3001, 1, 0.66), ("nt", 512, 64, 0.57), ("nt", 3400, 2, 1.08),
    ("nt", 1000, 33, 0.81),
]


@pytest.mark.parametrize("kind,n,batch,ratio", MEASURED)
def test_the_faster_tile_is_taken(kind, n, batch, ratio):
    from paper_2607_12430_amd import _lib
    ta, tb, sym = KINDS[kind]
    assert _lib.lib().msqrt_test_split_tile(ta, tb, sym, n, n, n, batch, 256) == (64 if ratio < 1 else 128)
