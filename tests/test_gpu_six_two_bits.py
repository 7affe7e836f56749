"""2-bit weights as fp4 operands against fp6 ones: every tile shape whole and cut at the edges of rows, columns and K, ranks of one and
several rounds; every code at every place of a block; layers whose exponents keep them in the bf16 form; groups of both widths."""
import numpy as np
import pytest

from oracle import mxint
from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload
from test_gpu_planes import _run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [121, 122, 221, 222, 141, 142, 143, 144, 241, 242, 243, 244])
@pytest.mark.parametrize("M,K,N,k", [(65, 1040, 144, 24), (255, 2064, 1042, 256), (129, 1296, 544, 100)])
def test_every_shape(variant, M, K, N, k):
    layer, ch = oracle_layer_big(K, N, k, seed=M, w_bits=2)
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()


@pytest.mark.parametrize("variant", [121, 122, 143])
def test_codes_at_every_place(variant):
    """With one non-zero weight per column the result is its product, exactly."""
    import torch
    from paper_2402_02446_amd import binding
    K, N, M = 512, 1024, 128
    layer, _ = oracle_layer_big(K, N, 16, seed=3, w_bits=2)
    W = np.zeros((K, N), np.float32)
    W[np.arange(N) % K, np.arange(N)] = np.where(np.arange(N) < K, 1.0, -1.0) * 2.0 ** (np.arange(N) % 5)
    c, e = mxint.mx_quantize(W, 2, axis=0)
    e = np.where(np.abs(c).reshape(K // 16, 16, N).max(1) > 0, e, 127)           # zero blocks: an exponent near the others'
    layer.Wc[:] = mxint.pack_codes(np.ascontiguousarray(c.T), 2)
    layer.We[:] = e.T
    layer.Bc[:] = 0
    h = upload(layer)
    X = np.random.default_rng(1).standard_normal((M, K)).astype(np.float32)
    Y = binding.lqer_linear_forward_ex(h, torch.from_numpy(X).cuda(), path=2, variant=variant).cpu().numpy()
    Xq = mxint.mx_dequantize(*mxint.mx_quantize(X, 8, axis=-1), 8, axis=-1)
    assert np.array_equal(Y, (Xq @ mxint.mx_dequantize(c, e, 2, axis=0)).astype(np.float32))
    h.free()


@pytest.mark.parametrize("low", [1, 90, "0..", "1.."])
def test_exponents_the_form_does_not_take(low):
    """Exponent bytes of more than 16 values, and of at most 16 from 0 or 1 on (a nibble and a bias below 2): bf16 operands, also at sizes
    the others take fp6 ones."""
    import torch
    from paper_2402_02446_amd import binding
    M, K, N = 700, 2048, 528
    layer, ch = oracle_layer_big(K, N, 64, seed=5, w_bits=2)
    X = synth.gen_activations(np.random.default_rng(2), M, K, ch, 50.0)
    if isinstance(low, str):
        layer.We -= layer.We.min() - np.uint8(low[0])
        assert layer.We.max() < 16
        layer.Bc[:] = 0                               # (a correction of X's size, not of W's)
        X *= np.float32(2.0 ** 100)                   # results of normal size
    else:
        layer.We[0, 0] = low
    h = upload(layer)
    Xd = torch.from_numpy(X).cuda()
    assert_forward_matches(binding.lqer_linear_forward(h, Xd).cpu().numpy(), X, layer)
    with pytest.raises(binding.LqerError, match="LQER_ERR_SHAPE"):
        binding.lqer_linear_forward_ex(h, Xd, path=2, variant=121)
    h.free()


@pytest.mark.parametrize("act_bits", [8, 6])
@pytest.mark.parametrize("variant", [0, 121, 143, 244])
def test_activations_of_both_widths_and_as_codes(act_bits, variant):
    """fp32 input against the oracle, the same bits from its codes; codes of every size, -128 among them, and exponent bytes to 255: the oracle's
    values, and NaN in a row with a block whose values are beyond fp32."""
    import torch
    from oracle import forward
    from paper_2402_02446_amd import binding
    M, K, N = 270, 2064, 544
    layer, ch = oracle_layer_big(K, N, 128, seed=4, w_bits=2)
    h = upload(layer)
    h.set_activation_bits(act_bits)
    X = synth.gen_activations(np.random.default_rng(act_bits), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    Y = binding.lqer_linear_forward_ex(h, Xd, path=2, variant=variant)
    assert_forward_matches(Y.cpu().numpy(), X, layer, act_bits=act_bits)
    codes, exps = binding.lqer_quantize_mx(Xd, act_bits)
    if variant == 0:
        assert torch.equal(binding.lqer_linear_forward_q(h, codes, exps), Y)
        rng = np.random.default_rng(8)
        top = 128 if act_bits == 8 else 32
        Xc = rng.integers(-top, top, (M, K)).astype(np.int8)
        Xe = rng.integers(120, 130, (M, K // 16)).astype(np.uint8)
        Xc[5], Xe[5] = 0, 0
        for row, e in ((0, 253), (1, 254), (2, 255), (127, 255)):  # one block each: the first with room for its exponent, the last without
            Xc[row, 32:48] = 3
            Xe[row, 2] = e
        Xc[127, 40] = top - 1
        Y = binding.lqer_linear_forward_q(h, torch.from_numpy(Xc).cuda(), torch.from_numpy(Xe).cuda()).cpu().numpy()
        assert np.isnan(Y[127]).all()
        keep = np.r_[0:127, 128:M]
        want = forward.forward_q(Xc[keep], Xe[keep], layer, act_bits)
        err = np.linalg.norm(Y[keep] - want, axis=1) / np.maximum(np.linalg.norm(want, axis=1), 1e-300)
        assert (err <= 2e-5).all(), err
    h.free()


def test_groups_of_both_widths():
    import torch
    from paper_2402_02446_amd import binding
    M, K = 600, 2048
    hs = [upload(oracle_layer_big(K, N, k, seed=40 + i, w_bits=b)[0]) for i, (N, k, b) in enumerate(((1024, 64, 2), (528, 64, 4), (1040, 256, 2), (96, 0, 2)))]
    X = torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    for g, h in zip(binding.lqer_linear_forward_shared(hs, X), hs):
        assert torch.equal(g, binding.lqer_linear_forward(h, X))
    for h in hs:
        h.free()
