"""Checkpoint and resume: a run saved after n1 sweeps and continued for n2
sweeps in a fresh context gives bit for bit the state, energies,
temperature permutation and accumulators of the uninterrupted n1 + n2 run."""
import numpy as np
import pytest

from paper_2511_13508_amd import rlpt
from tests.gpu_util import make_ctx
from tests.test_gpu_parity import SEED0, temps_geo

pytestmark = pytest.mark.gpu


def snapshot(ctx):
    E, temp_of = ctx.energies()
    return ctx.get_state(), E, temp_of, ctx.observables(), ctx.counters()


@pytest.mark.parametrize("precision,field_mode", [(rlpt.FP32, rlpt.FIELDS_STREAM), (rlpt.FP64, rlpt.FIELDS_STREAM),
                                                  (rlpt.FP32, rlpt.FIELDS_CACHED)])
def test_resume_is_bitwise(tmp_path, precision, field_mode):
    graphs = [rlpt.Graph(48, SEED0 + 700), rlpt.Graph(32, SEED0 + 701)]
    temps = temps_geo(0.3, 1.5, 6)
    kw = dict(n_temps=6, n_reps=2, precision=precision, field_mode=field_mode, swap_interval=2,
              resync_interval=25, measure_start=10, measure_interval=2, n_bins=20, series_len=64)
    a = make_ctx(graphs, temps, **kw)
    a.init(9)
    a.sweep(70)
    path = str(tmp_path / "run.ckpt")
    a.checkpoint_save(path)
    a.sweep(80)
    ref = snapshot(a)
    b = make_ctx(graphs, temps, **kw)
    b.checkpoint_load(path)
    b.sweep(80)
    got = snapshot(b)
    assert np.array_equal(got[0], ref[0])
    assert np.array_equal(got[1], ref[1])
    assert np.array_equal(got[2], ref[2])
    for k in ref[3]:
        assert np.array_equal(got[3][k], ref[3][k]), k
    assert got[4] == ref[4]


def test_checkpoint_of_another_context_is_rejected(tmp_path):
    g = [rlpt.Graph(24, SEED0 + 702)]
    a = make_ctx(g, temps_geo(0.5, 1.0, 3), n_temps=3, n_reps=2)
    a.init(1)
    a.sweep(5)
    path = str(tmp_path / "a.ckpt")
    a.checkpoint_save(path)
    b = make_ctx(g, temps_geo(0.5, 1.0, 4), n_temps=4, n_reps=2)
    with pytest.raises(rlpt.RlptError) as e:
        b.checkpoint_load(path)
    assert e.value.code == rlpt.RLPT_E_ARG
    c = make_ctx([rlpt.Graph(24, SEED0 + 703)], temps_geo(0.5, 1.0, 3), n_temps=3, n_reps=2)
    with pytest.raises(rlpt.RlptError):
        c.checkpoint_load(path)
    with open(path, "rb") as f:
        head = f.read(200)
    bad = str(tmp_path / "bad.ckpt")
    with open(bad, "wb") as f:
        f.write(head)
    with pytest.raises(rlpt.RlptError):
        a.checkpoint_load(bad)


@pytest.mark.parametrize("Ns,field_mode", [([48, 32], rlpt.FIELDS_CACHED), ([90], rlpt.FIELDS_CACHED),
                                           ([48, 32], rlpt.FIELDS_STREAM), ([90], rlpt.FIELDS_STREAM)])
def test_saving_leaves_the_run_alone(tmp_path, Ns, field_mode):
    """A run that writes checkpoints has the bits of one that does not: the
    cached fields that a sweep carries on are not formed anew by the save."""
    graphs = [rlpt.Graph(N, SEED0 + 710 + i) for i, N in enumerate(Ns)]
    temps = temps_geo(0.3, 1.5, 6)
    kw = dict(n_temps=6, n_reps=2, field_mode=field_mode, resync_interval=0, n_bins=20)
    a, b = (make_ctx(graphs, temps, **kw) for _ in range(2))
    for c in (a, b):
        c.init(9)
    for _ in range(4):
        a.sweep(7)
        b.sweep(7)
        a.checkpoint_save(str(tmp_path / "run.ckpt"))
    got, ref = snapshot(a), snapshot(b)
    assert np.array_equal(got[0], ref[0])
    assert np.array_equal(got[1], ref[1])
    assert np.array_equal(got[2], ref[2])
    for k in ref[3]:
        assert np.array_equal(got[3][k], ref[3][k]), k
