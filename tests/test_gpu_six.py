"""The tiled kernel's fp6 form (8-bit activation codes in two halves against 4-bit weights, on block-scaled matrix
instructions): edges of its 128-row tiles in M, of column groups and tiles in N, one and few K tiles, both exponent forms of the
layer, whole tiles and tiles cut along K, 6-bit activations, layers that share their activations, against the oracle."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload
from test_gpu_planes import _run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [121, 122])
@pytest.mark.parametrize("M,K,N,k,wide", [(1, 16, 32, 8, False), (127, 256, 48, 16, True), (128, 240, 520, 130, False), (129, 512, 96, 40, False),
                                          (255, 768, 272, 256, True), (300, 1296, 1042, 64, False)])
def test_whole_tiles(variant, M, K, N, k, wide):
    layer, ch = oracle_layer_big(K, N, min(k, N), seed=M + K)
    if wide:
        layer.We[0, 0], layer.We[N - 1, -1] = 90, 140             # more than 16 values apart
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()


@pytest.mark.parametrize("variant", [221, 222, 321, 322])
@pytest.mark.parametrize("M,K,N,k", [(130, 4112, 1040, 32), (513, 1296, 272, 128)])
def test_cut_tiles(variant, M, K, N, k):
    layer, ch = oracle_layer_big(K, N, k, seed=M)
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()


def test_codes_and_exponents_of_every_size():
    """Every code on both sides, rows and columns whose exponents are far apart, zero rows, subnormal blocks: with one
    non-zero product per output the result is that product."""
    import torch
    from paper_2402_02446_amd import binding
    K, N, M = 256, 64, 255
    layer, _ = oracle_layer_big(K, N, 16, seed=3)
    from oracle import mxint
    W = np.zeros((K, N), np.float32)
    W[0] = np.where(np.arange(N) % 8 < 1, 7, np.arange(N) % 8) * 2.0 ** (np.arange(N) // 4 - 8.0) * np.where(np.arange(N) % 3, 1, -1)
    c, e = mxint.mx_quantize(W, 4, axis=0)
    layer.Wc[:] = mxint.pack_codes(np.ascontiguousarray(c.T), 4)
    layer.We[:] = e.T
    layer.Bc[:] = 0
    X = np.zeros((M, K), np.float32)
    X[:, 0] = (np.arange(M) - 127) * 2.0 ** (np.arange(M) % 60 - 30.0)
    X[:, 1] = 64 * 2.0 ** (np.arange(M) % 60 - 30.0)               # keeps the block's exponent where the code of column 0 is small
    X[7] = 0
    h = upload(layer)
    Y = binding.lqer_linear_forward_ex(h, torch.from_numpy(X).cuda(), path=2, variant=121).cpu().numpy()
    want = mxint.mx_dequantize(*mxint.mx_quantize(X, 8, axis=-1), 8, axis=-1)[:, :1] * mxint.mx_dequantize(c, e, 4, axis=0)[:1]
    assert np.array_equal(Y, want.astype(np.float32))
    h.free()


@pytest.mark.parametrize("act_bits", [8, 6])
def test_shared_activations_and_narrow_ones(act_bits):
    """The automatic choice above its line, alone and as a group (T of the second layer from the stored operands): same bits."""
    import torch
    from paper_2402_02446_amd import binding
    M, K, shapes = 4500, 4112, ((4160, 32), (4128, 80))
    rng = np.random.default_rng(5)
    layers, hs, ch = [], [], None
    for i, (N, k) in enumerate(shapes):
        layer, c = oracle_layer_big(K, N, k, seed=20 + i)
        ch = c if ch is None else ch
        h = upload(layer)
        h.set_activation_bits(act_bits)
        layers.append(layer)
        hs.append(h)
    X = synth.gen_activations(rng, M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    alone = [binding.lqer_linear_forward(h, Xd) for h in hs]
    group = binding.lqer_linear_forward_shared(hs, Xd)
    rows, cols = np.array([0, 127, 128, 2049, M - 1]), np.array([0, 31, 32, 515, 4111, 4127])
    for layer, y, g in zip(layers, alone, group):
        assert torch.equal(y, g)
        assert_forward_matches(y.cpu().numpy()[np.ix_(rows, cols)], X[rows], layer, cols=cols, act_bits=act_bits)
    for h in hs:
        h.free()
