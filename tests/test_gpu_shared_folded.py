"""Layers of one few-token call that together fit a round of four column groups a workgroup: wavefronts that keep two K slices each.  K of
one to several steps, odd and even, with a last step that is not full; 1, 5 and 16 tokens; ranks 0 to 64; layers whose last workgroup has
columns past their end; beside groups beyond that round.  And the wide layers' shape on both sides of its line."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 5, 16])
@pytest.mark.parametrize("K,specs", [(256, ((10304, 32), (10400, 0))), (1024, ((10252, 8), (10240, 64))), (1296, ((10304, 33), (10272, 16))),
                                     (2304, ((10240, 16), (11008, 48))), (528, ((11008, 16), (11008, 16), (11040, 16))),
                                     (1536, ((10240, 64), (10300, 16))), (1552, ((10240, 64), (10300, 16)))])
def test_bits_are_the_layers_own(M, K, specs):
    import torch
    from paper_2402_02446_amd import binding
    layers, hs, ch = [], [], None
    for i, (N, k) in enumerate(specs):
        layer, c = oracle_layer_big(K, N, k, seed=70 + i)
        ch = c if ch is None else ch
        layers.append(layer)
        hs.append(upload(layer))
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    cols = np.r_[0:40, 127:130, 10200:10240]
    for layer, h, g in zip(layers, hs, binding.lqer_linear_forward_shared(hs, Xd)):
        assert torch.equal(g, binding.lqer_linear_forward(h, Xd))
        assert_forward_matches(g.cpu().numpy()[:, cols], X, layer, cols=cols)
        h.free()


@pytest.mark.parametrize("M", [1, 16, 32])
@pytest.mark.parametrize("N,k,w_bits", [(16384, 32, 4), (16416, 32, 4), (16420, 128, 2)])
def test_wide_layers(M, N, k, w_bits):
    import torch
    from paper_2402_02446_amd import binding
    K = 784
    layer, ch = oracle_layer_big(K, N, k, seed=N, w_bits=w_bits)
    h = upload(layer)
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Y = binding.lqer_linear_forward(h, torch.from_numpy(X).cuda()).cpu().numpy()
    cols = np.r_[0:40, 8191:8200, N - 40:N]
    assert_forward_matches(Y[:, cols], X, layer, cols=cols)
    h.free()


# Ranks above 64 on wide layers: eight K slices at up to 4 tokens from five K tiles on, else four; they add in another order.
@pytest.mark.parametrize("M,K,N,k,w_bits,shape", [(1, 1024, 10272, 128, 4, 12141), (4, 1040, 10272, 80, 4, 12181), (2, 2320, 16384, 256, 2, 12181), (4, 4096, 10240, 256, 4, 12181),
                                                  (5, 1040, 10272, 128, 2, 12141), (1, 1296, 16416, 128, 4, 12241)])
def test_slices_of_wide_layers_of_a_large_rank(M, K, N, k, w_bits, shape):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = oracle_layer_big(K, N, k, seed=K, w_bits=w_bits)
    h = upload(layer)
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    Y = binding.lqer_linear_forward(h, Xd)
    assert torch.equal(binding.lqer_linear_forward_ex(h, Xd, path=1, variant=shape), Y)
    if M <= 4:                                       # (beyond, eight slices do not fit)
        assert torch.equal(binding.lqer_linear_forward_ex(h, Xd, path=1, variant=12181), Y) == (shape == 12181)
    cols = np.r_[0:40, 5000:5040, N - 40:N]
    assert_forward_matches(Y.cpu().numpy()[:, cols], X, layer, cols=cols)
    h.free()
