"""GPU: FP32 sweeps against the CPU FP64 oracle, every copy accounted for: a
copy may part from the oracle only where one of its acceptance tests is decided
within the FP32 rounding of dE (found by replaying the copy's updates one by
one), so a wrong tail of a tile of copies or targets cannot pass as a boundary
flip.  19 and 33 copies leave 3 copies and 1 in the last tile of 16."""
import numpy as np
import pytest

from paper_2511_13508_amd import rlpt
from tests import synth
from tests.gpu_util import make_ctx, oracle_pt

pytestmark = pytest.mark.gpu

SEED = 2511135080 + 1500
TAG_PAIR, TAG_MOVE = 0x50414952, 0x4D4F5645


def replay(oracle, og, copy, beta, run_seed, sweeps):
    """The copy's chain without swaps, one update at a time (rho = 4, own pairs).
    Returns its state and the smallest |dE + log(u) / beta|, in units of
    2 (|d_j| |F_j| + |d_k| |F_k|), the size of dE's terms before they cancel."""
    N = og.N
    a = oracle.init_copy(N, run_seed, copy)
    closest = np.inf
    unit = lambda w: float(int(w) >> 11) * 2.0 ** -53  # noqa: E731
    below = lambda w, n: ((int(w) >> 32) * n) >> 32  # noqa: E731
    for s in range(sweeps):
        for t in range(N // 2):
            wp = oracle.philox([t, s, copy, 0], [run_seed, TAG_PAIR])
            wm = oracle.philox([t, s, copy, 0], [run_seed, TAG_MOVE])
            j, k = below(wp[0], N), below(wp[1], N - 1)
            k += k >= j
            u0, u1, u2, u = (unit(w) for w in wm)
            K, th = (abs(a[j]) ** 4 + abs(a[k]) ** 4) ** 0.25, 0.5 * np.pi * u2
            nj = K * np.sqrt(max(np.cos(th), 0.0)) * np.exp(2j * np.pi * u0)
            nk = K * np.sqrt(max(np.sin(th), 0.0)) * np.exp(2j * np.pi * u1)
            snap = a.copy()
            snap[j] = nj
            F = oracle.fields(og, snap)
            dj, dk = nj - a[j], nk - a[k]
            dE = -2.0 * (np.conj(dj) * F[j]).real - 2.0 * (np.conj(dk) * F[k]).real
            size = 2.0 * (abs(dj) * abs(F[j]) + abs(dk) * abs(F[k]))
            closest = min(closest, abs(dE + np.log(max(u, 1e-300)) / beta) / size)
            if dE <= 0 or u < np.exp(-beta * dE):
                a[j], a[k] = nj, nk
    return a, closest


def check_every_copy(oracle, Ns, z, T, reps, sweeps, t_max=1.5, **cfg):
    temps = synth.geometric_temps(0.3, t_max, T)
    graphs = [rlpt.Graph(N, SEED + i, mean_degree=z) for i, N in enumerate(Ns)]
    ctx = make_ctx(graphs, temps, n_temps=T, n_reps=reps, precision=rlpt.FP32, swap_interval=100, resync_interval=0,
                   n_bins=10, **cfg)
    ctx.init(8)
    ctx.sweep(sweeps)
    ctx.check()
    E = ctx.energies()[0]
    for mu, N in enumerate(Ns):
        og = oracle.Graph(N, SEED + mu, mean_degree=z)
        pt = oracle_pt(oracle, og, temps, mu, ctx.cfg, 8)
        pt.run(sweeps)
        a = ctx.get_state(mu * ctx.R, ctx.R).reshape(ctx.R, N)
        for c in range(ctx.R):
            at = mu * ctx.R + c
            if np.allclose(a[c], pt.a[c], rtol=0, atol=2e-5) and abs(E[at] - pt.E[c]) <= 1e-4 * max(1.0, abs(pt.E[c])):
                continue
            ref, closest = replay(oracle, og, at, 1.0 / temps[c % T], 8, sweeps)
            assert np.allclose(ref, pt.a[c], rtol=0, atol=1e-9), (N, c)
            assert closest <= 1e-5, (N, c, closest, float(np.abs(a[c] - pt.a[c]).max()))
    # the replay is the oracle's chain
    ref, _ = replay(oracle, og, ctx.S * ctx.R - 1, 1.0 / temps[T - 1], 8, sweeps)
    assert np.allclose(ref, pt.a[ctx.R - 1], rtol=0, atol=1e-9)


@pytest.mark.parametrize("Ns,T,reps", [([96], 19, 1), ([88, 91], 33, 1), ([136], 11, 3), ([137], 19, 1), ([181], 33, 1),
                                       ([255, 201], 19, 1), ([256], 33, 1), ([40, 128, 170], 19, 1)])
def test_pair_space_every_copy(oracle, Ns, T, reps):
    check_every_copy(oracle, Ns, 0, T, reps, 2)


@pytest.mark.parametrize("Ns,z,T,reps", [([14], 0, 19, 1), ([24, 17], 0, 11, 3), ([33], 0, 19, 1), ([48], 0, 33, 1),
                                         ([500], 20, 19, 1), ([300], 60, 11, 3)])
def test_several_steps_every_copy(oracle, Ns, z, T, reps):
    check_every_copy(oracle, Ns, z, T, reps, 2)
