"""GPU parity of the pruned insertion descents: every number of wavefronts per restart that the launches choose, on both sides of the
sizes and restart counts where it changes; the matrix in LDS, as a triangle and in memory; ties, zones of equal costs (more
candidates than one round scores), entries beyond 2^16."""
import numpy as np
import pytest

from gen import hierarchical_matrix, random_matrix
from gpu_util import say
from test_gpu_local_pruned import BOTH, INSERTION, check

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


def zones(n, k):
    z = np.random.default_rng(n + k).integers(0, k, n)
    c = np.where(z[:, None] == z[None, :], 100, 1000)
    np.fill_diagonal(c, 0)
    return c.astype(np.int32)


@pytest.mark.parametrize("n,restarts", [(32, 40), (33, 40), (48, 512), (48, 513), (65, 3), (65, 257), (100, 1024), (100, 1025), (128, 256), (128, 512),
                                        (129, 3), (150, 257), (161, 300), (192, 300), (193, 3), (255, 300), (256, 3), (256, 300),
                                        (257, 3), (257, 257), (512, 257), (513, 2), (513, 257), (1000, 1)])
def test_every_number_of_wavefronts(n, restarts):
    for c, tag in ((hierarchical_matrix(n, (4, 8), ((50, 100), (200, 400), (800, 2000)), 0.3, True, n), "racks"),
                   (random_matrix(n, n, symmetric=True, lo=0, hi=4), "ties"), (zones(n, 2), "two zones"), (zones(n, 9), "nine zones"),
                   (random_matrix(n, n, symmetric=True, lo=1, hi=1 << 20), "beyond 2^16")):
        if n > 512 and tag != "racks":
            continue
        for classes in (BOTH, INSERTION) if n < 512 else (BOTH,):
            say(f"pruned insertion groups N={n} R={restarts} {tag} classes={classes}")
            check(c, classes, restarts, 21, sorted({0, restarts - 1}))


@pytest.mark.parametrize("n,k", [(257, 8), (700, 12)])
def test_candidates_of_several_rooms(n, k):
    """Nodes whose candidates find no room beside those of their wavefront's other nodes: laid out after them."""
    for classes in (BOTH, INSERTION) if n < 512 else (BOTH,):
        say(f"pruned insertion, several rooms N={n} zones={k} classes={classes}")
        check(zones(n, k), classes, 2, 23, [1])


@pytest.mark.parametrize("n,restarts", [(128, 256), (128, 257), (192, 257), (256, 256), (256, 257)])
def test_levels_of_equal_costs(n, restarts):
    """Hosts in racks without noise: more and fewer partners at the racks' cost than the line between the pruned and the exhaustive kernel,
    and entries that the latter does not take."""
    node = np.arange(n)
    for rack in (n // 4, n // 2):
        c = np.where(node[:, None] // rack == node[None, :] // rack, 300, 1000)
        c = np.where(node[:, None] // 4 == node[None, :] // 4, 100, c)
        np.fill_diagonal(c, 0)
        for factor in (1, 100):
            for classes in (BOTH, INSERTION):
                say(f"pruned insertion, levels N={n} R={restarts} racks of {rack} times {factor} classes={classes}")
                check((c * factor).astype(np.int32), classes, restarts, 25, [0, restarts - 1])
