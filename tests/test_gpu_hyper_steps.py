"""GPU parity of the hypernetwork's recurrences and heads at the edges of their blocking: layer counts around the
four-step blocks of the recurrences, input widths around the eight-column blocks of the input projection, and layers
of rows around the eight row steps of a head block."""
import pytest

import workloads
from gpu_support import say
from test_gpu_hyper import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [32, 64, 128])
@pytest.mark.parametrize("L,D", [(1, 1), (2, 9), (4, 7), (5, 8), (8, 3), (9, 33)])
def test_hyper_blocking(H, L, D):
    sizes = [(1, 33, 255, 257, 64, 5, 2049, 31, 129)[l] for l in range(L)]
    say(f"hypernetwork blocking: L={L} D={D} H={H}")
    _check(workloads.make_hyper_case((295, H, L, D), sizes, D, H), step=3)
