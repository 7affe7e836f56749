"""Layers that share their activations: the projection of a layer that finds them stored adds up T = X_q A_k in the order of the
layer's own call, whatever its rank, so Y has the same bits.  Activations whose blocks are many binades apart, so that T's sums
round."""
import numpy as np
import pytest

from helpers import oracle_layer_big, upload

pytestmark = pytest.mark.gpu


def _wide(seed, M, K):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((M, K)) * np.exp(2.5 * rng.standard_normal((M, K)))).astype(np.float32)


# eight K slices of two tiles; 8, 16, 19 and 25 blocks of 16 rows: below and above 256 workgroups by row blocks, slices and planes of
# rank groups
@pytest.mark.parametrize("w_bits", [2, 4])
@pytest.mark.parametrize("M", [128, 256, 300, 400])
def test_large_ranks_behind_another_layer(M, w_bits):
    import torch
    from paper_2402_02446_amd import binding
    K, hs = 4096, []
    for i, k in enumerate((16, 128, 256)):
        hs.append(upload(oracle_layer_big(K, 256, k, seed=40 + i, w_bits=w_bits)[0]))
    X = torch.from_numpy(_wide(M, M, K)).cuda()
    for g, h in zip(binding.lqer_linear_forward_shared(hs, X), hs):
        assert torch.equal(g, binding.lqer_linear_forward(h, X))
        h.free()


# 2048 blocks of 16 rows and more, where fp32 rows are read by the row-wise form, codes and stored activations by the other one;
# 4-bit layers of these sizes take other operands, and the same form whatever the source
@pytest.mark.parametrize("w_bits", [2, 4])
@pytest.mark.parametrize("M,K,ranks", [(33000, 1040, (16, 33)), (32768, 2304, (64, 256))])
def test_many_tokens_from_every_source(M, K, ranks, w_bits):
    import torch
    from paper_2402_02446_amd import binding
    hs = [upload(oracle_layer_big(K, 256, k, seed=50 + i, w_bits=w_bits)[0]) for i, k in enumerate(ranks)]
    X = torch.from_numpy(_wide(K, M, K)).cuda()
    codes, exps = binding.lqer_quantize_mx(X, 8)
    for g, h in zip(binding.lqer_linear_forward_shared(hs, X), hs):
        Y = binding.lqer_linear_forward(h, X)
        assert torch.equal(g, Y)
        assert torch.equal(binding.lqer_linear_forward_q(h, codes, exps), Y)
        h.free()
