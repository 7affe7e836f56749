"""The staged kernel (64-row tiles, whole or as K planes), which calls of 33 to about a thousand tokens take: edges of
tiles in M and N, K ranges that the planes do not divide, ranks 0 to 256, both weight widths, fp32 and MXINT8 output,
against the oracle; the same bits on a second run with other contents in the workspace."""
import numpy as np
import pytest

from oracle import mxint
from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload

pytestmark = pytest.mark.gpu


# K tiles of 256: 1 (nothing to cut), 5, 9, 17, 43 (ragged last planes); N around the 128 / 256 / 512 column tiles
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
