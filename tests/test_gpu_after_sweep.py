"""GPU: swap round, counters and measurement in one launch against the CPU
FP64 oracle: one bath and two, full and ragged groups of baths, the most baths
it takes and one more, one to five replicas, swap rounds and measurements at
different sweeps, a recomputation between the two."""
import pytest

from paper_2511_13508_amd import rlpt
from tests.test_gpu_ahead import run_both
from tests.test_gpu_parity import compare_fp64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ns,T,reps,cfg", [
    ([8], 1, 3, {}), ([8], 2, 4, {}), ([6, 70], 8, 2, {}), ([9], 9, 5, {}), ([6, 7, 8], 17, 1, dict(swap_interval=3)),
    ([8], 64, 2, {}), ([8], 65, 2, {}), ([66], 5, 3, dict(measure_interval=2, swap_interval=3)),
    ([8], 64, 24, {}), ([8], 64, 25, {})])
def test_swap_and_measure_fp64(oracle, Ns, T, reps, cfg):
    kw = dict(dict(measure_interval=1, resync_interval=6), **cfg)
    compare_fp64(*run_both(oracle, Ns, 0, T, reps, 18, precision=rlpt.FP64, **kw))
