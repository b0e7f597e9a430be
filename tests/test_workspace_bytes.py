"""Workspace sizes of the shapes whose streaming fills take more memory than
the tile fill (CPU only).  The tile fill's workspace is, to within a percent
for large shapes, its direction blocks, its face planes and 16 bytes a tile
beside the pairwise tables of the pruned mode."""
import numpy as np
import pytest

import paper_2311_17530_amd as msa

GB = 1 << 30


def tile_bytes(lens):
    k, T = len(lens), msa.tile_edge(len(lens))
    P = [1 + (n + T - 1) // T for n in lens]
    tiles = int(np.prod(P, dtype=np.int64))
    cells = [n + 1 for n in lens]
    faces = sum((P[i] - 1) * int(np.prod([c for j, c in enumerate(cells) if j != i],
                                         dtype=np.int64)) for i in range(k))
    tables = sum(2 * cells[i] * cells[j] for i in range(k) for j in range(i))
    return tiles * (T ** k + 16) + 4 * faces + 4 * tables


# thin shapes, most of whose exchange words belong to no cell
@pytest.mark.parametrize("lens", [[2032, 1932, 2288, 23], [509, 1506, 1153, 34],
                                  [762, 2005, 367, 69], [1936, 1508, 668, 89], [1000, 1000, 1000, 17]],
                         ids=lambda s: "x".join(map(str, s)))
def test_large_workspaces_are_the_tile_fills(lens):
    assert tile_bytes(lens) > 64 * GB
    assert msa.workspace_bytes(lens) <= 1.01 * tile_bytes(lens)


@pytest.mark.parametrize("lens", [[3, 3, 3, 3], [40, 4, 4, 200], [2, 72, 71, 1], [128] * 4,
                                  [1, 1, 1, 1, 100], [40] * 5, [12, 12, 12, 12, 12]],
                         ids=lambda s: "x".join(map(str, s)))
def test_other_workspaces_grow_to_a_bound(lens):
    assert msa.workspace_bytes(lens) <= 2.02 * tile_bytes(lens) + (64 << 20) + (1 << 20)
