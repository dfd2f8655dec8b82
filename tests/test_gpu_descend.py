"""The descent loop's two ways of running its iterations."""
import numpy as np
import pytest

from paper_1706_07413_amd import adscl
from test_gpu_adjoint import coeffs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ns,T", [([65, 129, 33, 65], 0.2), ([257], 0.1), ([1001, 901], 0.02)])
def test_replayed_iterations_equal_enqueued_ones_in_one_class(Ns, T):
    """All instances in one kernel configuration: an iteration is captured once and replayed.
    Two calls in a row, with the context's own work between them; every history and
    coefficient is that of directly enqueued iterations, bit for bit."""
    n = len(Ns)
    eps, c0 = np.linspace(0.3, 0.6, n), coeffs(31, n, 6)
    print("descend, one class", Ns, flush=True)
    b = adscl.Batch(Ns, a_collapse=0.0, n_modes=6)
    assert len(b.kernel_stats()[0]) == 1
    want = b.descend(eps, c0, 4, T, 5, step0=0.05, ckpt_every=16, eager=True)
    for _ in range(2):
        got = b.descend(eps, c0, 4, T, 5, step0=0.05, ckpt_every=16)
        for x, y in zip(got, want):
            assert np.array_equal(x, y)
        b.init_modes(eps, c0)
        b.step(7, 1e9)
    assert np.all(np.isfinite(want[1]))
