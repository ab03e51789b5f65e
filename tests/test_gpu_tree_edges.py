"""The node table at the edges of its launches, against the oracle's direct
definition: snapshot counts around the sixteen nodes that the first, one-block
launch still splits, empty snapshots among them, levels of more blocks than a
group of block totals holds, node tables of more than one group of point
totals, ranges of nine and of eighty-one particles and around (the octant
search reads nine at a time)."""
import numpy as np
import pytest

from gpu_util import compare_tree, to_dev
from oracle import lod as olod
from paper_0811_2055_amd import lib
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_snap", [2, 3, 15, 16, 17, 129, 1030])
@pytest.mark.parametrize("D", [0, 1, 4])
def test_snapshots(n_snap, D):
    import torch
    rng = np.random.default_rng(n_snap)
    # sizes 0, 1, 7..10, 80..83 and larger, in every order
    sizes = rng.choice([0, 0, 1, 7, 8, 9, 10, 80, 81, 82, 83, 200], n_snap)
    sizes[-1] = 0
    sizes[0] = 500
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    s = synth.small_clustered(int(off[-1]), 100 + n_snap)
    ref = olod.lod_build(s.x, s.y, s.z, s.m, n=6, D=D, seed=4, snap_offsets=off)
    offs = torch.from_numpy(off).cuda().view(torch.uint64)
    tree = lib.build(*to_dev(s), lib.BuildParams(n=6, max_depth=D, seed=4), snap_offsets=offs)
    compare_tree(tree.host(), ref, f"{n_snap} snapshots D={D}")


@pytest.mark.parametrize("N", [1, 2, 8, 9, 10, 80, 81, 82, 728, 729, 730])
def test_small_ranges(N):
    s = synth.uniform(N, N)
    ref = olod.lod_build(s.x, s.y, s.z, s.m, n=1, D=3, seed=4)
    compare_tree(lib.build(*to_dev(s), lib.BuildParams(n=1, max_depth=3, seed=4)).host(), ref, f"N={N}")


@pytest.mark.parametrize("N,n", [(70000, 1), (20000, 2)])
def test_many_nodes(N, n):
    s = synth.uniform(N, 6)
    ref = olod.lod_build(s.x, s.y, s.z, s.m, n=n, D=6, seed=4)
    compare_tree(lib.build(*to_dev(s), lib.BuildParams(n=n, max_depth=6, seed=4)).host(), ref, f"N={N} n={n}")
