"""The projection step, whose wavefronts take quarters of a K tile (64 columns): K that ends inside a block group, a quarter or
a tile, fewer quarters than wavefronts and several rounds of them, token rows that do not fill 16, each rank-group count it has
an instance for, every source (fp32, codes) and layout (cells, code cells, rows), against the oracle."""
import numpy as np
import pytest

from oracle import mxint
from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload

pytestmark = pytest.mark.gpu


# cells (M <= 32), code cells (16 < .. of single workgroups per column block), rows (M > 32), the last one with as
# many wavefronts as tiles, four quarters each
@pytest.mark.parametrize("M", [1, 5, 17, 33, 47, 1043])
@pytest.mark.parametrize("K,N,k,w_bits", [(16, 40, 8, 4), (80, 100, 0, 4), (272, 64, 24, 4), (1040, 96, 40, 4), (4176, 70, 64, 4),
                                          (11056, 48, 16, 4), (4112, 64, 256, 2), (33040, 32, 33, 2)])
def test_forward_and_codes(M, K, N, k, w_bits):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = oracle_layer_big(K, N, k if k <= min(K, N) else min(K, N), seed=K + M, w_bits=w_bits)
    X = synth.gen_activations(np.random.default_rng(M + K), M, K, ch, 50.0)
    h = upload(layer)
    Xd = torch.from_numpy(X).cuda()
    out = lambda: torch.full((M, (N + 3) // 4 * 4), 7.0, device="cuda")[:, :N]
    ws = torch.full((binding.lqer_linear_workspace_bytes(h, M),), 255, dtype=torch.uint8, device="cuda")
    Y = binding.lqer_linear_forward(h, Xd, Y=out(), workspace=ws)
    assert_forward_matches(Y.cpu().numpy(), X, layer)
    codes, exps = binding.lqer_quantize_mx(Xd, 8)
    oc, oe = mxint.mx_quantize(X, 8, axis=-1)
    assert np.array_equal(codes.cpu().numpy(), oc) and np.array_equal(exps.cpu().numpy(), oe)
    ws.fill_(255)
    assert torch.equal(binding.lqer_linear_forward_q(h, codes, exps, Y=out(), workspace=ws), Y)
    h.free()
