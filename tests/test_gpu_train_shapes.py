"""GPU: the learned proposal's layers, their gradients and the mixture head at
the shapes where the products' tiles and loads change, against the FP64 oracle
on the same bfloat16 operands: extents that are no multiple of 4 (narrow
loads), of a tile or of a K stage; enough tiles for the larger tile; more
components than the head has waves; more coordinates than it keeps."""
import numpy as np
import pytest

from oracle import mlp as M
from tests import synth
from tests.test_gpu_mlp import _store_pairs, mlp_ctx, unflatten

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,K,B,nets", [(5, 33, 1, 7, 1), (9, 50, 5, 70, 2), (20, 64, 8, 129, 1), (40, 100, 2, 600, 2),
                                          (150, 64, 3, 40, 1), (64, 256, 8, 512, 5), (63, 130, 7, 900, 3)])
def test_layers_and_gradients(N, H, K, B, nets):
    """The loss, which every output enters, to 1e-4; gradients per tensor within
    1e-2 of their norm and cosine >= 0.999: FP32 sums against FP64 ones,
    activations and gradients rounded to bfloat16 (2^-9) between the layers."""
    ctx = mlp_ctx(N, 1, max(nets, 2), 1, H, K, B, nets=nets, cap=B)
    ctx.init(1)
    ctx.mlp_setup(list(range(nets)), seed=3)
    NP, Out = ctx.mlp_sizes()
    pairs = []
    for net in range(nets):
        ctx.mlp_set_params(net, synth.random_mlp_params(2 * N, H, Out, seed=210 + net, out_scale=0.5))
        pairs.append(_store_pairs(ctx, net, synth.random_constrained_state(N, 220 + net, B),
                                  synth.random_constrained_state(N, 230 + net, B)))
    net = nets - 1
    b, a = pairs[net]
    params = M.rounded(unflatten(synth.random_mlp_params(2 * N, H, Out, seed=210 + net, out_scale=0.5), N, H, K))
    L_ref, g_ref = M.loss_and_grads(params, b, a, N, K)
    L, g = ctx.mlp_loss_grad(net)
    assert abs(L - L_ref) <= 1e-4 * abs(L_ref)
    for k, x in unflatten(g, N, H, K).items():
        x, y = x.ravel(), g_ref[k].ravel()
        assert np.linalg.norm(x - y) <= 1e-2 * np.linalg.norm(y), k
        assert np.dot(x, y) >= 0.999 * np.linalg.norm(x) * np.linalg.norm(y), k
