"""GPU: sweeps of short lists, several steps of a copy decided at a time,
against the CPU FP64 oracle: fewer steps than a window, windows that do not
divide the steps, lists of exactly the longest length that takes this sweep,
more copies than it serves, one and two chunks per lane."""
import numpy as np
import pytest

from paper_2511_13508_amd import rlpt
from tests import synth
from tests.gpu_util import make_ctx, oracle_pt
from tests.test_gpu_parity import compare_fp64
from tests.test_gpu_pairs import compare_fp32

pytestmark = pytest.mark.gpu

SEED = 2511135080 + 1300


def run_both(oracle, Ns, z, T, reps, sweeps, **cfg):
    temps = synth.geometric_temps(0.3, 1.5, T)
    graphs = [rlpt.Graph(N, SEED + i, mean_degree=z) for i, N in enumerate(Ns)]
    ctx = make_ctx(graphs, temps, n_temps=T, n_reps=reps, n_bins=10, **cfg)
    ctx.init(4)
    ctx.sweep(sweeps)
    ctx.check()
    ors = []
    for mu, N in enumerate(Ns):
        pt = oracle_pt(oracle, oracle.Graph(N, SEED + mu, mean_degree=z), temps, mu, ctx.cfg, 4)
        pt.run(sweeps)
        ors.append(pt)
    return ctx, ors


@pytest.mark.parametrize("Ns,z,T,reps,cfg", [
    ([6, 9, 5], 0, 4, 2, {}), ([17], 0, 3, 1, dict(swap_interval=4)), ([15], 0, 3, 2, dict(rho=2)),
    ([16], 0, 40, 20, {}),  # more copies than the chip has room for several waves each
    ([300, 33, 1023], 9, 3, 2, dict(shared_pairs=1)), ([1024], 32, 2, 1, dict(swap_interval=3)),
    ([32], 0, 3, 2, {}), ([40, 33], 0, 3, 1, dict(swap_interval=2))])
def test_ahead_trajectory_fp64(oracle, Ns, z, T, reps, cfg):
    compare_fp64(*run_both(oracle, Ns, z, T, reps, 24, precision=rlpt.FP64, resync_interval=12, **cfg))


@pytest.mark.parametrize("Ns,z,T,reps", [([14], 0, 5, 2), ([24], 0, 4, 2), ([32, 38], 0, 6, 2), ([700, 1001], 20, 5, 1)])
def test_ahead_fp32(oracle, Ns, z, T, reps):
    compare_fp32(*run_both(oracle, Ns, z, T, reps, 4, precision=rlpt.FP32))


def test_longest_list_of_the_short_sweep():
    """128 entries per list take the short sweep, one more does not; both
    agree with the streaming kernel on the same FP64 chain."""
    temps = synth.geometric_temps(0.4, 1.5, 3)
    for z in (92, 96, 100, 108, 116):  # the longest list of these samples crosses 128
        g = [rlpt.Graph(64, SEED + 30, mean_degree=z)]
        ctxs = [make_ctx(g, temps, n_temps=3, n_reps=2, precision=rlpt.FP64, n_bins=4, **kw)
                for kw in (dict(list_layout=rlpt.LAYOUT_PACKED),
                           dict(list_layout=rlpt.LAYOUT_CHUNKED, block_threads=64, copies_per_block=1))]
        for c in ctxs:
            c.init(9)
            c.sweep(12)
        # the same decisions; energies differ by the order of FP64 sums of ~100 terms
        assert np.allclose(ctxs[0].get_state(), ctxs[1].get_state(), rtol=0, atol=1e-12), z
        assert np.allclose(ctxs[0].energies()[0], ctxs[1].energies()[0], rtol=1e-11, atol=1e-11), z


@pytest.mark.parametrize("N,T,reps,precision", [(40, 3, 1, rlpt.FP64), (48, 4, 2, rlpt.FP64), (56, 3, 1, rlpt.FP64),
                                                (40, 6, 2, rlpt.FP32), (48, 5, 1, rlpt.FP32), (56, 4, 2, rlpt.FP32)])
def test_ahead_three_to_six_chunks(oracle, N, T, reps, precision):
    if precision == rlpt.FP64:
        compare_fp64(*run_both(oracle, [N], 0, T, reps, 24, precision=precision, resync_interval=12))
    else:
        compare_fp32(*run_both(oracle, [N, N - 3], 0, T, reps, 4, precision=precision))


@pytest.mark.parametrize("Ns,precision", [([19], rlpt.FP64), ([24, 21], rlpt.FP64), ([28], rlpt.FP64), ([31], rlpt.FP64),
                                          ([20, 30], rlpt.FP32), ([26], rlpt.FP32)])
def test_ahead_five_to_sixteen_entries(oracle, Ns, precision):
    if precision == rlpt.FP64:
        compare_fp64(*run_both(oracle, Ns, 0, 5, 2, 24, precision=precision, resync_interval=12))
    else:
        compare_fp32(*run_both(oracle, Ns, 0, 5, 2, 4, precision=precision))


@pytest.mark.parametrize("Ns,z", [([995], 128), ([994], 128), ([1024], 128), ([1024, 24], 128)])
def test_lists_past_the_short_sweep_at_the_largest_sizes_fp64(oracle, Ns, z):
    """Lists of 129 to 512 entries have 512-thread instances only, whose LDS
    holds 994 FP64 modes; larger samples keep the sweep of one step at a time."""
    temps = synth.geometric_temps(0.3, 1.5, 2)
    degree = [z if N > 100 else 0 for N in Ns]
    graphs = [rlpt.Graph(N, SEED + i, mean_degree=d) for i, (N, d) in enumerate(zip(Ns, degree))]
    ctx = make_ctx(graphs, temps, n_temps=2, n_reps=1, n_bins=10, precision=rlpt.FP64, resync_interval=4)
    ctx.init(4)
    ctx.sweep(6)
    ctx.check()
    ors = []
    for mu, (N, d) in enumerate(zip(Ns, degree)):
        pt = oracle_pt(oracle, oracle.Graph(N, SEED + mu, mean_degree=d), temps, mu, ctx.cfg, 4)
        pt.run(6)
        ors.append(pt)
    compare_fp64(ctx, ors)


@pytest.mark.parametrize("N,z,precision", [(256, 24, rlpt.FP64), (48, 0, rlpt.FP64), (256, 24, rlpt.FP32)])
def test_hot_ladders_take_one_step_at_a_time(oracle, N, z, precision):
    """Where most updates are accepted a step at a time is swept: the bits of a
    context that names the same launch tile, and the oracle's chain."""
    temps = synth.geometric_temps(20.0, 100.0, 3)
    kw = dict(n_temps=3, n_reps=2, n_bins=10, precision=precision)
    g = [rlpt.Graph(N, SEED, mean_degree=z)]
    a = make_ctx(g, temps, **kw)
    block, copies = a.tile()
    b = make_ctx(g, temps, block_threads=int(block), copies_per_block=int(copies[0]), **kw)
    for c in (a, b):
        c.init(4)
        c.sweep(6)
    assert np.array_equal(a.get_state(), b.get_state()) and np.array_equal(a.energies()[0], b.energies()[0])
    pt = oracle_pt(oracle, oracle.Graph(N, SEED, mean_degree=z), temps, 0, a.cfg, 4)
    pt.run(6)
    (compare_fp64 if precision == rlpt.FP64 else compare_fp32)(a, [pt])
