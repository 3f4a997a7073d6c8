"""Column-wise centres where the column-sum pass changes: first output slots
found on the way or by a pass of their own (255 and 256 tensors), slices of
256 to 4,096 sent entries (2^16, 2^18 and 2^20 of them), columns summed on chip (one,
a few, up to a quarter of a slice) or directly, many tensors in a slice,
nothing sent, and calls of one context in turn (the sums start from zero)."""
import numpy as np
import pytest

from paper_1704_05021_amd import gd
from parity import check_case

pytestmark = pytest.mark.gpu


def _run(sizes, cols, drops, seed, pers=(False, True)):
    rng = np.random.default_rng(seed)
    off = [0] + np.cumsum(sizes).tolist()
    g = (rng.standard_t(3, off[-1]) * 1e-3).astype(np.float32)
    r = rng.normal(0, 1e-3, off[-1]).astype(np.float32)
    comp = gd.Compressor(off)
    comp.set_columns(cols)
    for drop in drops:
        for per in pers:
            for debug in (0, 5):  # the direct form's list, and the candidate form's
                check_case(g, r, off, drop, per, gd.GD_QUANT_COLUMN_MEAN, comp=comp, columns=cols, debug_bracket=debug,
                           what=f"T={len(sizes)} drop={drop} per={per} debug={debug}")


@pytest.mark.parametrize("tensors", [1, 2, 254, 255, 256, 1100])
def test_tensor_counts(tensors):
    rng = np.random.default_rng(tensors)
    cols = rng.choice([1, 2, 7, 64, 500], tensors)
    sizes = cols * rng.integers(0, max(2, 200_000 // tensors // 60), tensors)
    sizes[0] = cols[0] * 4
    _run(sizes, cols.tolist(), (0.5, 0.99, 1.0), tensors)


@pytest.mark.parametrize("columns", [1, 3, 255, 256, 257, 1023, 1024, 1025, 8192])
@pytest.mark.parametrize("rows,drop", [(7, 0.0), (900, 0.9)])
def test_columns(columns, rows, drop):
    n = columns * rows
    _run([n, 2 * columns, n], [columns, 2 * columns, columns], (drop,), columns)


@pytest.mark.parametrize("n,drop", [(1 << 16, 0.0), ((1 << 16) + 1024, 0.0), (1 << 18, 0.0), ((1 << 18) + 1024, 0.0),
                                    (1 << 20, 0.0), ((1 << 20) + 1024, 0.0), (7_000_064, 0.7)])
def test_many_entries(n, drop):
    # up to and past 2^20 entries, in the direct and the candidate form
    _run([n - 1024, 1024], [64, 1024], (drop,), 1, pers=(False,))


@pytest.mark.parametrize("tensors", [200, 3000])
@pytest.mark.parametrize("drop", [0.0, 0.5])
def test_many_tensors_in_a_slice(tensors, drop):
    # slices that span many tensors: of as many entries as columns and one less, of
    # twice as many (what slices of 4,096 sum on chip), none, and one large
    # tensor among them; up to and past 2^16, 2^18 and 2^20 entries in all
    rng = np.random.default_rng(tensors)
    for scale in (1, 4, 20) if tensors == 200 else (1, 3):
        cols = rng.choice([1, 2, 3, 8, 100], tensors)
        sizes = cols * rng.choice([0, 1, 2, 3, 40], tensors) * scale
        sizes[5], cols[5] = 100_000 * scale, 400
        _run(sizes, cols.tolist(), (drop,), tensors + scale, pers=(False,))
