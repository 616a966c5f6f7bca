"""GPU: the pair-space sweep (all fields of a sweep from one banded product,
corrected where an update is accepted) against the CPU FP64 oracle, at the
sizes where its tables and tiles change: the smallest N it serves, odd N, the
largest N whose product fits a workgroup's LDS and the next, N = 256; copies
that do not fill a matrix-core tile; both constraints and pair schedules;
degenerate frequency sums, single splits and a wider linewidth; several sweeps
per launch; mixed N in one context."""
import numpy as np
import pytest

from paper_2511_13508_amd import rlpt
from tests import synth
from tests.gpu_util import make_ctx, oracle_pt

pytestmark = pytest.mark.gpu

SEED = 2511135080 + 1200


def run_both(oracle, Ns, T, reps, sweeps, graph={}, **cfg):
    temps = synth.geometric_temps(0.3, 1.5, T)
    graphs = [rlpt.Graph(N, SEED + i, **graph) for i, N in enumerate(Ns)]
    ctx = make_ctx(graphs, temps, n_temps=T, n_reps=reps, precision=rlpt.FP32, n_bins=20, **cfg)
    ctx.init(6)
    ctx.sweep(sweeps)
    ctx.check()
    ors = []
    for mu, N in enumerate(Ns):
        pt = oracle_pt(oracle, oracle.Graph(N, SEED + mu, **graph), temps, mu, ctx.cfg, 6)
        pt.run(sweeps)
        ors.append(pt)
    return ctx, ors


def compare_fp32(ctx, ors):
    """FP32 states and energies of the same chain: proposals are FP32 (a few
    units of 6e-8 relative to amplitudes of order one per update of a mode,
    within 2e-5), energies sums of ~N updates (1e-4); a copy may separate at an
    acceptance decided within the FP32 rounding of dE, at most one per sample."""
    a = ctx.get_state() if len(set(ctx.Ns)) == 1 else None
    E, temp_of = ctx.energies()
    at = 0
    for mu, pt in enumerate(ors):
        N = ctx.Ns[mu]
        g = (a[at:at + ctx.R * N] if a is not None else ctx.get_state(mu * ctx.R, ctx.R)).reshape(ctx.R, N)
        at += ctx.R * N
        bad = 0
        for c in range(ctx.R):
            ok = np.allclose(g[c], pt.a[c], rtol=0, atol=2e-5) and temp_of[mu * ctx.R + c] == pt.temp_of[c]
            bad += not (ok and abs(E[mu * ctx.R + c] - pt.E[c]) <= 1e-4 * max(1.0, abs(pt.E[c])))
        assert bad <= 1, (N, bad)


@pytest.mark.parametrize("N,T,reps,samples", [(88, 5, 1, 2), (97, 7, 3, 1), (136, 4, 2, 2), (137, 5, 1, 3),
                                              (181, 17, 1, 1), (255, 3, 1, 1), (256, 8, 2, 1)])
def test_pair_sweep_sizes(oracle, N, T, reps, samples):
    compare_fp32(*run_both(oracle, [N] * samples, T, reps, 3, resync_interval=2))


@pytest.mark.parametrize("N,cfg", [(96, dict(rho=2)), (150, dict(rho=2)), (96, dict(shared_pairs=1)),
                                   (150, dict(shared_pairs=1)), (120, dict(swap_interval=3, resync_interval=0)),
                                   (160, dict(swap_interval=3, resync_interval=0)),
                                   (96, dict(list_layout=rlpt.LAYOUT_PACKED)),
                                   (144, dict(list_layout=rlpt.LAYOUT_PACKED))])
def test_pair_sweep_options(oracle, N, cfg):
    compare_fp32(*run_both(oracle, [N], 6, 2, 3, **cfg))


@pytest.mark.parametrize("N,graph", [(96, dict(omega_kind=rlpt.OMEGA_COMB)), (140, dict(omega_kind=rlpt.OMEGA_COMB)),
                                     (96, dict(split_mask=rlpt.SPLIT_A)), (140, dict(split_mask=rlpt.SPLIT_B)),
                                     (96, dict(gamma=0.02))])
def test_pair_sweep_graphs(oracle, N, graph):
    compare_fp32(*run_both(oracle, [N], 4, 1, 2, graph=graph))


def test_pair_sweep_mixed_sizes(oracle):
    """Classes the pair-space sweep serves beside classes swept from their lists."""
    compare_fp32(*run_both(oracle, [32, 128, 64, 200, 128, 90], 4, 2, 2))


@pytest.mark.parametrize("Ns", [[100], [176], [48, 112]])
def test_pair_sweep_replays(Ns):
    """Eager sweeps, one launch of several sweeps and HIP-graph replay give the same bits."""
    temps = synth.geometric_temps(0.4, 1.5, 4)
    graphs = [rlpt.Graph(N, SEED + 40 + i) for i, N in enumerate(Ns)]
    kw = dict(n_temps=4, n_reps=2, precision=rlpt.FP32, swap_interval=3, resync_interval=6, measure_interval=3, n_bins=8)
    ctxs = [make_ctx(graphs, temps, **kw) for _ in range(3)]
    for c in ctxs:
        c.init(2)
    for _ in range(12):
        ctxs[0].sweep(1)
    ctxs[1].sweep(12)
    ctxs[2].run_graph(6, 2)
    a, E = [np.concatenate([c.get_state(i * c.R, c.R) for i in range(c.S)]) for c in ctxs], [c.energies() for c in ctxs]
    for i in (1, 2):
        assert np.array_equal(a[0], a[i])
        assert np.array_equal(E[0][0], E[i][0]) and np.array_equal(E[0][1], E[i][1])


@pytest.mark.parametrize("Ns,cfg", [([88, 88], {}), ([97], dict(rho=2)), ([201], dict(list_layout=rlpt.LAYOUT_PACKED)),
                                    ([256], dict(shared_pairs=1)), ([96, 40], {})])
def test_cached_field_mode(oracle, Ns, cfg):
    """The cached-field mode follows the same chain, served by the pair-space
    sweep or, with a sample below its smallest N, by its own."""
    compare_fp32(*run_both(oracle, Ns, 5, 2, 3, field_mode=rlpt.FIELDS_CACHED, resync_interval=2, **cfg))


@pytest.mark.parametrize("first", [0, 1])
def test_cached_checkpoint_across_sweeps(oracle, tmp_path, first):
    """A checkpoint holds the fields of its amplitudes whichever sweep wrote it:
    the other one (an explicit launch tile belongs to the cached-field sweep)
    continues the oracle's chain from it."""
    N, T, reps = 96, 5, 2
    temps = synth.geometric_temps(0.3, 1.5, T)
    g = rlpt.Graph(N, SEED)
    kw = dict(n_temps=T, n_reps=reps, n_bins=20, field_mode=rlpt.FIELDS_CACHED, resync_interval=0)
    ctxs = [make_ctx([g], temps, **kw), make_ctx([g], temps, block_threads=128, copies_per_block=1, **kw)]
    a, b = ctxs[first], ctxs[1 - first]
    a.init(6)
    a.sweep(2)
    a.checkpoint_save(str(tmp_path / "c"))
    b.checkpoint_load(str(tmp_path / "c"))
    b.sweep(2)
    b.check()
    pt = oracle_pt(oracle, oracle.Graph(N, SEED), temps, 0, b.cfg, 6)
    pt.run(4)
    compare_fp32(b, [pt])


@pytest.mark.parametrize("Ns,T,reps", [([137, 96, 30, 88, 40, 160], 4, 2), ([88, 20], 32, 32)])
def test_mixed_sizes_side_by_side(oracle, Ns, T, reps):
    """Samples of several N: one launch for N <= 136, one above, the smaller
    ones swept from their lists on a second stream; and enough copies for the
    smaller workgroups."""
    compare_fp32(*run_both(oracle, Ns, T, reps, 2))


def test_mixed_sizes_replay_bitwise_in_graphs():
    """Captured segments (the second stream forked and joined inside) give the
    eager run's bits, replay after replay, with eager sweeps between."""
    temps = synth.geometric_temps(0.3, 1.5, 5)
    graphs = [rlpt.Graph(N, SEED + i) for i, N in enumerate([96, 40, 140])]
    kw = dict(n_temps=5, n_reps=2, n_bins=20, swap_interval=2, resync_interval=6, measure_interval=2)
    a, b = (make_ctx(graphs, temps, **kw) for _ in range(2))
    for c in (a, b):
        c.init(3)
    for n, segments in ((6, 2), (6, 1), (12, 2)):
        a.run_graph(n, segments)
        a.sweep(6)
        b.sweep(n * segments + 6)
        for mu in range(3):
            assert np.array_equal(a.get_state(mu * a.R, a.R), b.get_state(mu * b.R, b.R)), (n, segments, mu)
        assert np.array_equal(a.energies()[0], b.energies()[0])
        assert np.array_equal(a.energies()[1], b.energies()[1])
        assert a.counters() == b.counters()


@pytest.mark.parametrize("Ns,cfg", [([96], {}), ([160, 40], {}), ([128], dict(shared_pairs=1))])
def test_hot_ladders_are_swept_from_their_lists(oracle, Ns, cfg):
    """Where most updates are accepted the lists are streamed: the bits of a
    context that names the same launch tile, and the oracle's chain."""
    temps = synth.geometric_temps(5.0, 20.0, 4)
    graphs = [rlpt.Graph(N, SEED + i) for i, N in enumerate(Ns)]
    kw = dict(n_temps=4, n_reps=2, n_bins=20, **cfg)
    a = make_ctx(graphs, temps, **kw)
    block, copies = a.tile()
    b = make_ctx(graphs, temps, block_threads=int(block), copies_per_block=int(copies[0]), **kw)
    assert len(set(copies)) == 1
    for c in (a, b):
        c.init(6)
        c.sweep(3)
    for mu in range(len(Ns)):
        assert np.array_equal(a.get_state(mu * a.R, a.R), b.get_state(mu * b.R, b.R))
    assert np.array_equal(a.energies()[0], b.energies()[0])
    ors = []
    for mu, N in enumerate(Ns):
        pt = oracle_pt(oracle, oracle.Graph(N, SEED + mu), temps, mu, a.cfg, 6)
        pt.run(3)
        ors.append(pt)
    compare_fp32(a, ors)


@pytest.mark.parametrize("Ns", [[96], [140, 40]])
def test_smaller_workspaces_take_the_lists(oracle, monkeypatch, Ns):
    """A workspace without room for the tables in pair space (the size of a
    context that names a launch tile), or for those of the energies either, is
    taken, and gives the same chain; one without room for the lists is not."""
    size_of, want = rlpt.lib().rlpt_workspace_size, {}

    def workspace_size(cfg, graphs, n, out):
        rc = size_of(cfg, graphs, n, out)
        want["size"] = out._obj.value
        out._obj.value = want.get("give", out._obj.value)
        return rc

    monkeypatch.setattr(rlpt.lib(), "rlpt_workspace_size", workspace_size)
    kw = dict(resync_interval=2)
    full, ors = run_both(oracle, Ns, 4, 2, 3, **kw)
    most = want["size"]
    tile, _ = run_both(oracle, Ns, 4, 2, 1, block_threads=256, copies_per_block=1, **kw)
    least = want["size"]
    assert least < most
    for give in (most, most - 256, least, least - 256):
        want["give"] = give
        ctx, _ = run_both(oracle, Ns, 4, 2, 3, **kw)
        compare_fp32(ctx, ors)
        if give < most:  # the lists' bits, whatever the size
            ref = ref if give < most - 256 else ctx.get_state(0, ctx.R)
            assert np.array_equal(ctx.get_state(0, ctx.R), ref)
        E, E64 = ctx.energies()[0], ctx.energy_fp64()
        assert np.all(np.abs(E - E64) <= 1e-4 * np.maximum(1.0, np.abs(E64)))
    want["give"] = least // 4
    with pytest.raises(rlpt.RlptError) as e:
        run_both(oracle, Ns, 4, 2, 1, **kw)
    assert e.value.code == rlpt.RLPT_E_NOMEM
