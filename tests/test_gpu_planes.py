"""The staged kernel (64-row tiles, whole or as K planes), which calls of 33 to about a thousand tokens take: edges of
tiles in M and N, K ranges that the planes do not divide, ranks 0 to 256, both weight widths, both exponent forms, fp32 and
MXINT8 output, against the oracle; the same bits on a second run with other contents in the workspace.  The automatic choice
at these sizes is nearly always the 64 x 128 tile; every shape, whole and in planes, is forced below."""
import numpy as np
import pytest

from oracle import mxint
from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload

pytestmark = pytest.mark.gpu


def _run_and_check(layer, h, X, path, variant):
    """fp32 on two contents of the workspace (255: every float in it is a NaN), the same bits and nothing behind the N
    columns touched, against the oracle; MXINT8 output = the quantizer applied to that Y."""
    import torch
    from paper_2402_02446_amd import binding
    M, N = X.shape[0], layer.N
    Xd = torch.from_numpy(X).cuda()
    ws = torch.empty(binding.lqer_linear_workspace_bytes(h, M, path), dtype=torch.uint8, device="cuda")
    first = None
    for fill in (0, 255):
        ws.fill_(fill)
        buf = torch.full((M, (N + 7) // 4 * 4), 7.0, dtype=torch.float32, device="cuda")
        binding.lqer_linear_forward_ex(h, Xd, Y=buf[:, :N], workspace=ws, path=path, variant=variant)
        torch.cuda.synchronize()
        assert (buf[:, N:] == 7.0).all()
        first = buf[:, :N].clone() if first is None else first
        assert torch.equal(buf[:, :N], first)
    Y = first.cpu().numpy()
    assert_forward_matches(Y, X, layer)
    if N % 16 == 0:
        ws.fill_(255)
        codes, exps = binding.lqer_linear_forward_requant(h, Xd, workspace=ws, path=path, variant=variant)
        oc, oe = mxint.mx_quantize(Y, 8, axis=-1)
        assert np.array_equal(exps.cpu().numpy(), oe) and np.array_equal(codes.cpu().numpy(), oc)


# 131 .. 133 whole tiles, 231 .. 233 planes of 64 x 256, 64 x 512, 64 x 128.  N just past one column group, a wavefront's two,
# and each tile width; K of 2, 5, 9, 17 tiles; the second size of each kind with a byte per exponent instead of a nibble
@pytest.mark.parametrize("variant", [131, 132, 133, 231, 232, 233])
@pytest.mark.parametrize("w_bits", [4, 2])
@pytest.mark.parametrize("M,K,N,k,wide", [(33, 272, 48, 8, False), (65, 2304, 97, 33, True), (70, 1040, 144, 0, False), (100, 2304, 272, 128, True),
                                          (64, 4112, 272, 24, False), (129, 1296, 560, 256, False), (190, 1040, 1042, 64, True)])
def test_every_shape(variant, w_bits, M, K, N, k, wide):
    layer, ch = oracle_layer_big(K, N, k, seed=M + K + w_bits, w_bits=w_bits)
    if wide:
        layer.We[0, 0], layer.We[N - 1, -1] = 90, 140             # more than 16 values apart
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()


def test_shapes_that_are_not_to_be_had():
    from paper_2402_02446_amd import binding
    import torch
    layer, _ = oracle_layer_big(256, 64, 8, seed=1)
    h = upload(layer)
    X = torch.zeros((40, 256), device="cuda")
    for variant in (231, 331, 30, 34, 134):                      # planes of a single K tile; equal shares; no such shape
        with pytest.raises(binding.LqerError):
            binding.lqer_linear_forward_ex(h, X, path=2, variant=variant)
    h.free()


# K tiles of 256: 1 (nothing to cut), 5, 9, 17, 43 (ragged last planes)
@pytest.mark.parametrize("M,K,N,k,w_bits", [
    (33, 256, 100, 8, 4), (64, 1040, 128, 0, 4), (65, 4112, 1001, 24, 4), (127, 2304, 272, 64, 4), (128, 11008, 512, 32, 4),
    (203, 4112, 1104, 24, 4), (257, 4096, 2064, 33, 4), (700, 1280, 3072, 16, 4), (90, 2048, 272, 256, 4),
    (33, 272, 100, 100, 2), (64, 2304, 1040, 256, 2), (300, 4096, 528, 65, 2), (1100, 1040, 2064, 200, 2)])
def test_planes_and_narrow_tiles(M, K, N, k, w_bits):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = oracle_layer_big(K, N, k, seed=M + K, w_bits=w_bits)
    h = upload(layer)
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    assert binding.lqer_linear_path(h, M) == 2
    ws = h.workspace(M)
    first = None
    for fill in (0, 255):                                     # 255: every float of the workspace is a NaN
        ws.fill_(fill)
        buf = torch.full((M, (N + 7) // 4 * 4), 7.0, dtype=torch.float32, device="cuda")
        binding.lqer_linear_forward(h, Xd, Y=buf[:, :N])
        torch.cuda.synchronize()
        assert (buf[:, N:] == 7.0).all()                      # nothing behind the N columns is touched
        first = buf[:, :N].clone() if first is None else first
        assert torch.equal(buf[:, :N], first)
    Y = first.cpu().numpy()
    assert_forward_matches(Y, X, layer)
    if N % 16 == 0:
        ws.fill_(255)
        codes, exps = binding.lqer_linear_forward_requant(h, Xd)
        oc, oe = mxint.mx_quantize(Y, 8, axis=-1)
        assert np.array_equal(exps.cpu().numpy(), oe) and np.array_equal(codes.cpu().numpy(), oc)
    h.free()


# fp32 rounds once per MFMA step at the size the sum has reached.  As the kernel sums - the correction, then half of K; the
# other half - these are 2.7e-7 (both widths) from the oracle; one chain over K with the correction last is 3.4e-7.
@pytest.mark.parametrize("w_bits", [4, 2])
def test_large_rank_is_summed_in_short_chains(w_bits):
    import torch
    from paper_2402_02446_amd import binding
    M, K, N, k = 512, 4096, 4096, 256
    layer, ch = oracle_layer_big(K, N, k, seed=5, w_bits=w_bits)
    h = upload(layer)
    X = synth.gen_activations(np.random.default_rng(5), M, K, ch, 50.0)
    cols = np.arange(0, N, 8)
    Y = binding.lqer_linear_forward(h, torch.from_numpy(X).cuda()).cpu().numpy()[:, cols]
    assert_forward_matches(Y, X, layer, cols=cols, tol=3.0e-7)
    h.free()


# Many tokens on a small layer: tiles of 128 rows are the faster ones there, also with a rank above 64 and with 2-bit weights
# (384 x 2816 with rank 256 at 20710 tokens 147 us against 169, 2-bit 592 x 912 at 63752 tokens 142 against 168).  The two
# kernels add the correction at different ends, which tells their results apart.
@pytest.mark.parametrize("M,K,N,k,w_bits", [(20710, 384, 2816, 256, 4), (63752, 592, 912, 64, 2)])
def test_many_tokens_take_tiles_of_128_rows(M, K, N, k, w_bits):
    import torch
    from paper_2402_02446_amd import binding
    layer, _ = oracle_layer_big(K, N, k, seed=M, w_bits=w_bits)
    h = upload(layer)
    X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda")
    Y = binding.lqer_linear_forward(h, X)
    same = {v for v in (111, 112, 211, 131, 132, 133) if torch.equal(Y, binding.lqer_linear_forward_ex(h, X, path=2, variant=v))}
    assert same & {111, 112, 211} and not same & {131, 132, 133}, same
    h.free()
