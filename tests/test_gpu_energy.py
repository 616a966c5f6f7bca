"""GPU: FP64 energies as a banded product on the matrix cores against the CPU
oracle's sum over terms: fewer pairs than a tile of 16 rows, sizes around whole
tiles, the largest N, copies that do not fill a tile of 16, several samples of
different N, more copies than many ranges' partial energies have room for, and
graphs whose frequency sums coincide."""
import numpy as np
import pytest

from paper_2511_13508_amd import rlpt
from tests import synth
from tests.gpu_util import make_ctx

pytestmark = pytest.mark.gpu

SEED = 2511135080 + 1400


@pytest.mark.parametrize("Ns,T,reps,precision,graph", [
    ([4], 1, 1, rlpt.FP64, dict(omega_kind=rlpt.OMEGA_COMB)), ([6, 5], 3, 5, rlpt.FP32, {}), ([17], 4, 4, rlpt.FP32, {}),
    ([33, 16, 57], 17, 1, rlpt.FP64, {}), ([64], 33, 1, rlpt.FP32, dict(omega_kind=rlpt.OMEGA_COMB)),
    ([91], 3, 2, rlpt.FP64, dict(split_mask=rlpt.SPLIT_B)), ([129], 2, 1, rlpt.FP32, dict(gamma=0.01)),
    ([256, 40], 5, 1, rlpt.FP64, {}), ([255], 2, 2, rlpt.FP32, {}), ([12], 4, 5000, rlpt.FP32, {})])
def test_banded_energies(oracle, Ns, T, reps, precision, graph):
    """A sum of n products in FP64, each of a few roundings, in two orders:
    within n * 2^-52 of the terms' absolute sum at worst, sqrt(n) of it as a
    rule; 1e-13 of the absolute sum covers both for n up to a million terms."""
    temps = synth.geometric_temps(0.5, 1.5, T)
    graphs = [rlpt.Graph(N, SEED + i, **graph) for i, N in enumerate(Ns)]
    ctx = make_ctx(graphs, temps, n_temps=T, n_reps=reps, precision=precision)
    ctx.init(3)
    E = ctx.energy_fp64()
    for mu, N in enumerate(Ns):
        og = oracle.Graph(N, SEED + mu, **graph)
        a = ctx.get_state(mu * ctx.R, ctx.R).reshape(ctx.R, N)
        q = np.asarray(og.quads).reshape(-1, 4)
        for c in {0, 1 % ctx.R, 15 % ctx.R, 16 % ctx.R, ctx.R - 1}:
            size = 2 * np.sum(np.abs(og.J) * np.prod(np.abs(a[c])[q], axis=1))
            assert abs(E[mu * ctx.R + c] - oracle.energy(og, a[c])) <= 1e-13 * max(size, 1.0), (N, c)


@pytest.mark.parametrize("N,precision", [(256, rlpt.FP64), (230, rlpt.FP64), (256, rlpt.FP32)])
def test_banded_energies_of_more_copies_than_the_scratch_has_room_for(oracle, N, precision):
    """131074 copies: one range per copy would be all that the static scratch
    holds, but a range's pairs have to fit a workgroup's LDS too."""
    reps = 65537
    ctx = make_ctx([rlpt.Graph(N, SEED)], [0.5, 1.0], n_temps=2, n_reps=reps, precision=precision, measure_interval=0)
    ctx.init(3)
    E = ctx.energy_fp64()
    og = oracle.Graph(N, SEED)
    q = np.asarray(og.quads).reshape(-1, 4)
    for c in (0, 15, 16, 65537, ctx.R - 2, ctx.R - 1):
        a = ctx.get_state(c, 1)
        size = 2 * np.sum(np.abs(og.J) * np.prod(np.abs(a)[q], axis=1))
        assert abs(E[c] - oracle.energy(og, a)) <= 1e-13 * max(size, 1.0), c
