"""What the host side plans before it launches, without a GPU: workspace
sizes."""
import numpy as np
import pytest

from paper_1606_08281_amd import lik


def _network(U):
    orders, stoich = np.zeros((1, U), np.int32), np.zeros((1, U), np.int32)
    stoich[0, 0] = 1
    return lik.Network(orders, stoich)


# (species, particles) -> filters that fit the no-allocation entry point's 64 MiB
SCRATCH_FITS = {(1, 200): 8729, (4, 1000): 1232, (4, 200): 4859, (9, 65): 5526, (20, 64): 5670,
                (32, 64): 3734, (32, 4096): 59}


@pytest.mark.parametrize("shape", sorted(SCRATCH_FITS))
def test_workspace_size_never_shrinks_with_the_batch(shape):
    """A workspace made for a batch holds every smaller one, and the largest
    batch of the no-allocation entry point stays what it was."""
    U, H = shape
    net, size = _network(U), lik.lib().lik_workspace_size
    need = [size(net.handle, n, 1, H) for n in range(9000)]
    shrinks = [n for n in range(1, 9000) if need[n] < need[n - 1]]
    assert not shrinks
    assert sum(b <= 64 << 20 for b in need) - 1 == SCRATCH_FITS[shape]
