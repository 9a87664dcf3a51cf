"""The transform kernel where its build, its row layout or its dispatch
changes, beyond the sets of test_gpu_fft.py.  Tolerance 0 against the oracle:
the results are integers."""
import pytest

import test_gpu_fft as F

pytestmark = pytest.mark.gpu

# run-time digit counts: two rows a turn at the rings that lacked one, and the
# workgroup that takes all 160 KB of LDS
RUNTIME = [F.case(33, 512, 6, 4), F.case(9, 512, 9, 1), F.case(6, 2048, 7, 4),
           F.case(67, 256, 3, 8), F.case(5, 1024, 5, 6)]


@pytest.mark.parametrize("p", RUNTIME, ids=[p.name for p in RUNTIME])
def test_run_time_digit_counts(O, p):
    assert F.bound(p) <= 0.25
    F.check(O, p, ("ntt",), 9500 + RUNTIME.index(p), 5, False)
    F.check(O, p, ("ntt",), 9520 + RUNTIME.index(p), 3, True)
