"""GPU: autotuned launch tiles and the batched uneven-N configuration
(N in {32, 48, 64, 96, 128} x 32 samples x 32 temperatures x 2 replicas in one
launch, HIP-graph replay), checked against the CPU oracle on sampled disorder
samples (one per N) whose 64 copies the oracle runs in full."""
import numpy as np
import pytest

from paper_2511_13508_amd import rlpt
from tests import synth
from tests.gpu_util import make_ctx, oracle_pt
from tests.test_gpu_parity import compare_fp64

pytestmark = pytest.mark.gpu

SEED2 = 2511135080 + 200


def test_autotune_then_tuned_tiles_keep_parity(oracle):
    Ns = [16, 40, 24, 40]
    seeds = [SEED2 + 900 + i for i in range(len(Ns))]
    graphs = [rlpt.Graph(N, s) for N, s in zip(Ns, seeds)]
    temps = synth.geometric_temps(0.4, 1.5, 6)
    rlpt.tune_clear()
    n = rlpt.autotune(graphs, temps, n_temps=6, n_reps=2, precision=rlpt.FP64, sweeps_per_trial=2)
    assert n >= 2 * 15 - 2  # every tile for both N classes (minus any over the LDS limit)
    ent = rlpt.tune_entries()
    assert {e["n_modes"] for e in ent} == {16, 24, 40}
    ctx = make_ctx(graphs, temps, n_temps=6, n_reps=2, precision=rlpt.FP64, swap_interval=1, resync_interval=20,
                   measure_start=10, measure_interval=2, n_bins=16)
    block, copies = ctx.tile()
    # the chosen workgroup size minimises the summed best times; copies are best at that size
    best = {}
    for N in (16, 24, 40):
        cands = [e for e in ent if e["n_modes"] == N and e["block_threads"] == block]
        best[N] = min(cands, key=lambda e: e["ms_per_sweep"])["copies_per_block"]
    assert [int(c) for c in copies] == [best[N] for N in Ns]
    ctx.init(3)
    ctx.sweep(60)
    ors = []
    for mu, (N, s) in enumerate(zip(Ns, seeds)):
        pt = oracle_pt(oracle, oracle.Graph(N, s), temps, mu, ctx.cfg, 3)
        pt.run(60)
        ors.append(pt)
    compare_fp64(ctx, ors)
    rlpt.tune_clear()


def test_batched_uneven_full_size_sampled(oracle):
    """The batched configuration at full size (10,240 copies), FP32, graph
    replay; for one sample of each N the oracle runs all 64 copies over the
    same 2 sweeps.  FP32 states agree within 2e-5; at most one copy per
    sample may separate at an FP32 acceptance-boundary flip."""
    Ns = [32, 48, 64, 96, 128]
    per_N = 32
    temps = synth.geometric_temps(0.3, 1.5, 32)
    graphs, seeds, Nlist = [], [], []
    for i, N in enumerate(Ns):
        for m in range(per_N):
            s = SEED2 + 1000 * i + m
            graphs.append(rlpt.Graph(N, s))
            seeds.append(s)
            Nlist.append(N)
    ctx = make_ctx(graphs, temps, n_temps=32, n_reps=2, precision=rlpt.FP32, swap_interval=1, resync_interval=0,
                   measure_start=0, measure_interval=1, n_bins=50)
    assert ctx.n_copies == 10240
    ctx.init(5)
    ctx.run_graph(1, 2)
    ctx.check()
    a = ctx.get_state()
    E, temp_of = ctx.energies()
    offs = np.concatenate([[0], np.cumsum([ctx.R * N for N in Nlist])])
    for i, N in enumerate(Ns):
        mu = i * per_N + (7 * i) % per_N  # one sampled disorder sample per N
        pt = oracle_pt(oracle, oracle.Graph(N, seeds[mu]), temps, mu, ctx.cfg, 5)
        pt.run(2)
        ga = a[offs[mu]:offs[mu + 1]].reshape(ctx.R, N)
        bad = 0
        for c in range(ctx.R):
            ok = np.allclose(ga[c], pt.a[c], rtol=0, atol=2e-5) and temp_of[mu * ctx.R + c] == pt.temp_of[c]
            ok = ok and abs(E[mu * ctx.R + c] - pt.E[c]) <= 1e-4 * max(1.0, abs(pt.E[c]))
            bad += 0 if ok else 1
        assert bad <= 1, (N, bad)
    obs = ctx.observables()
    assert np.all(obs["e_n"] == 2 * 2)  # two measurements x two replicas per (sample, T)


def test_autotune_times_the_launches_that_run():
    """Samples swept in pair space are no part of the trials of the others: a
    tile of N = 32 (4 samples of 12 copies) is timed in a small part of the
    milliseconds that streaming the lists of N = 256 takes; every N has its
    entries, and an explicit ladder's context still takes the tuned tiles."""
    graphs = [rlpt.Graph(N, SEED2 + 950 + i) for i, N in enumerate([256, 256, 32, 32, 32, 32])]
    temps = synth.geometric_temps(0.4, 1.5, 6)
    rlpt.tune_clear()
    try:
        rlpt.autotune(graphs, temps, n_temps=6, n_reps=2, sweeps_per_trial=4)
        ms = {N: [e["ms_per_sweep"] for e in rlpt.tune_entries() if e["n_modes"] == N] for N in (32, 256)}
        assert len(ms[32]) >= 13 and len(ms[256]) >= 13
        assert np.median(ms[32]) < 0.5 * min(ms[256])
        hot = make_ctx(graphs, synth.geometric_temps(5.0, 20.0, 6), n_temps=6, n_reps=2)
        block, copies = hot.tile()
        best = {N: min((e for e in rlpt.tune_entries() if e["n_modes"] == N and e["block_threads"] == block),
                       key=lambda e: e["ms_per_sweep"])["copies_per_block"] for N in (32, 256)}
        assert [int(c) for c in copies] == [best[g.N] for g in graphs]
    finally:
        rlpt.tune_clear()
