"""Host logic of bench.py's tile options (no GPU)."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_no_tile_given_leaves_the_choice_to_the_library():
    """set_tile_ex(op, 0, 0, 0) restores the library's own choice: what --no-tune times."""
    assert bench.given_tile("") == (0, 0, 0)
    assert bench.given_tile("8,64") == (8, 64, 4) and bench.given_tile("4,32,4") == (4, 32, 4)
