"""Matrices whose leaf level takes the default groups of four column blocks."""
import numpy as np


def uneven_arrow(widths, b, seed=0):
    """Dense blocks of the given widths, each coupled to the same b last
    columns: supernodes of w columns and w + b rows in one level, and one of b
    columns above them.  Lower CSC with values that make it diagonally
    dominant, and the identity order."""
    starts = np.concatenate([[0], np.cumsum(widths)])
    n = int(starts[-1]) + b
    end = np.concatenate([np.repeat(starts[1:], widths), np.full(b, n)])  # of each column's dense part
    border = np.concatenate([np.full(n - b, b), np.zeros(b, dtype=np.int64)])
    col = np.arange(n)
    count = end - col + border
    colptr = np.concatenate([[0], np.cumsum(count)]).astype(np.int64)
    cols = np.repeat(col, count)
    k = np.arange(colptr[-1]) - colptr[cols]  # place in the column
    dense = (end - col)[cols]
    rows = np.where(k < dense, cols + k, n - b + k - dense)
    values = -np.random.default_rng(seed).uniform(0.5, 1.5, rows.size)
    values[colptr[:-1]] = 0.0
    values[colptr[:-1]] = 1.0 - np.bincount(rows, values, n) - np.bincount(cols, values, n)
    return colptr, rows.astype(np.int32), values, col.astype(np.int32)


# Two wide supernodes hold the level above the limit of 3500 tiles beyond the
# first and the fifth block (4144 and 3609; 3138 beyond the ninth), so that two
# groups of four follow each other; the narrow ones end raggedly inside the
# second group, in its second block and in its last, and inside the first.
# Either half alone stays below the limit (2160, 1984).
WIDTHS = ([4200, 350], [4000, 500, 150])
BORDER = 8
