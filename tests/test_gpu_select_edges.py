"""The node selection at the edges of its forms, against the oracle's direct
definition: list histograms kept or not (n around 2048), candidates that
overflow the flag bytes (above 131072) or the threshold bin's queue (above
2048), lists whose chunks start at every alignment, nodes of lists, of ranges
and of both."""
import numpy as np
import pytest

from gpu_util import compare_tree, to_dev
from oracle import lod as olod
from paper_0811_2055_amd import lib
import synth

pytestmark = pytest.mark.gpu


def _clump(n, seed, cells):
    """n particles in `cells` equal cells of a depth-2 grid (overfull leaves at depth 2)."""
    rng = np.random.default_rng(seed)
    c = rng.integers(0, cells, n)
    x = ((c & 3) + 0.98 * rng.random(n)) / 4
    y = ((c >> 2 & 3) + 0.98 * rng.random(n)) / 4
    z = (c >> 4 & 3) / 4 + 0.2 * rng.random(n)
    s = synth.uniform(n, seed)
    s.x[:], s.y[:], s.z[:] = x, y, z
    s.m[:] = (0.5 + rng.random(n)).astype(np.float32) / n
    return s


CASES = {
    "hist-off": (lambda: synth.plummer_mix(120000, 1), 2047, 4, 1),
    "hist-on": (lambda: synth.plummer_mix(120000, 1), 2048, 4, 1),
    "hist-on-alpha0": (lambda: synth.plummer_mix(90001, 2), 2049, 4, 0),
    "hist-on-inverse": (lambda: synth.plummer_mix(90001, 3), 3001, 5, -1),
    "flags-full": (lambda: _clump(131072 + 9, 4, 1), 2048, 2, 1),
    "flags-over": (lambda: _clump(2 * 131072 + 77, 5, 2), 5000, 2, 1),
    "queue-over": (lambda: _clump(300000, 6, 1), 100000, 2, 0),
    "mixed": (lambda: _clump(260001, 7, 23), 2500, 4, 1),
    "small-lists": (lambda: synth.small_clustered(30011, 8), 5, 8, 1),
}


@pytest.mark.parametrize("mode,threads", [(1, 0), (1, 64), (1, 512), (2, 256), (2, 1024)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_selection_edges(name, mode, threads):
    make, n, D, alpha = CASES[name]
    s = make()
    ref = olod.lod_build(s.x, s.y, s.z, s.m, n=n, D=D, alpha=alpha, seed=3)
    tree = lib.build(*to_dev(s), lib.BuildParams(n=n, max_depth=D, alpha=alpha, seed=3, mode=mode,
                                                 select_threads=threads))
    compare_tree(tree.host(), ref, name)
