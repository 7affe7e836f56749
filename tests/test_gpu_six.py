"""The fp6 form of the tiled and the staged kernel (8-bit activation codes in two halves against 4-bit weights, on block-scaled matrix
instructions): edges of their 128- and 64-row tiles in M, of column groups and tiles in N, one and few K tiles, both exponent forms of the
layer, whole tiles, tiles cut along K and planes, 6-bit activations, layers that share their activations, against the oracle."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload
from test_gpu_planes import _run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [121, 122, 141, 142, 143])
@pytest.mark.parametrize("M,K,N,k,wide", [(1, 16, 32, 8, False), (65, 512, 144, 24, False), (127, 256, 48, 16, True), (128, 240, 520, 130, False), (129, 512, 96, 40, False),
                                          (255, 768, 272, 256, True), (300, 1296, 1042, 64, False)])
def test_whole_tiles(variant, M, K, N, k, wide):
    layer, ch = oracle_layer_big(K, N, min(k, N), seed=M + K)
    if wide:
        layer.We[0, 0], layer.We[N - 1, -1] = 90, 140             # more than 16 values apart
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()


@pytest.mark.parametrize("variant", [221, 222, 321, 322, 241, 242, 243])
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
def test_codes_as_input(act_bits):
    """Codes of every size, -128 among them, and exponent bytes to 255 at a size the fp6 form takes: the oracle's values; a
    row with a block whose values are beyond fp32 is NaN."""
    import torch
    from oracle import forward
    from paper_2402_02446_amd import binding
    M, K, N = 4500, 2064, 4160
    layer, _ = oracle_layer_big(K, N, 16, seed=4)
    h = upload(layer)
    h.set_activation_bits(act_bits)
    rng = np.random.default_rng(8)
    top = 128 if act_bits == 8 else 32
    Xc = rng.integers(-top, top, (M, K)).astype(np.int8)
    Xe = rng.integers(120, 130, (M, K // 16)).astype(np.uint8)
    Xc[5], Xe[5] = 0, 0
    for row, e in ((0, 253), (1, 254), (2, 255), (127, 255)):      # one block each: the first with room for its exponent, the last without
        Xc[row, 32:48] = 3
        Xe[row, 2] = e
    Xc[127, 40] = top - 1
    rows = np.array([0, 1, 2, 5, 127, 128, 300, M - 1])
    Y = binding.lqer_linear_forward_q(h, torch.from_numpy(Xc).cuda(), torch.from_numpy(Xe).cuda()).cpu().numpy()[rows]
    want = forward.forward_q(Xc[rows], Xe[rows], layer, act_bits) if act_bits != 8 else forward.forward_q(Xc[rows], Xe[rows], layer)
    assert np.isnan(Y[4]).all()
    keep = [0, 1, 2, 3, 5, 6, 7]
    err = np.linalg.norm(Y[keep] - want[keep], axis=1) / np.maximum(np.linalg.norm(want[keep], axis=1), 1e-300)
    assert (err <= 2e-5).all(), err
    h.free()


def test_shared_layers_of_two_forms():
    """A group with a layer of rank 0, which keeps bf16 operands: everybody's bits are those of its own call."""
    import torch
    from paper_2402_02446_amd import binding
    M, K = 4500, 2064
    hs = []
    for i, (N, k) in enumerate(((4160, 0), (4128, 32), (96, 16), (4160, 16))):
        hs.append(upload(oracle_layer_big(K, N, k, seed=30 + i)[0]))
    X = torch.from_numpy(np.random.default_rng(6).standard_normal((M, K)).astype(np.float32)).cuda()
    for g, h in zip(binding.lqer_linear_forward_shared(hs, X), hs):
        assert torch.equal(g, binding.lqer_linear_forward(h, X))
    for h in hs:
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
