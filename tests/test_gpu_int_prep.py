"""The INT variant's quantizer and projection in one launch (ranks 1 to 64): K groups below, at and past a wavefront count, past what stays in
registers; token counts that 8 does not divide (of up to 128: test_which_launches_with_a_small_rank); both sides of the size from which the separate launches are the faster.  Results against the
oracle; codes and scales in the workspace bit for bit the stand-alone quantizer's, for scales of zero, infinity and all between."""
import numpy as np
import pytest

from test_gpu_int import _standin_layer, _upload
from test_gpu_int_few import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,k", [(129, 128, 40, 8), (131, 640, 64, 32), (136, 1024, 64, 33), (255, 1152, 64, 64), (130, 2048, 36, 16),
                                     (142, 2176, 64, 48), (201, 4096, 64, 32), (133, 8320, 64, 64), (2180, 11008, 32, 32), (2181, 11008, 32, 32)])
def test_against_the_oracle(M, K, N, k):
    _run(M, K, N, k)


@pytest.mark.parametrize("M,K,k", [(131, 256, 16), (139, 1536, 40), (150, 4224, 8), (137, 11008, 64)])
def test_codes_and_scales_are_the_quantizers(M, K, k):
    import torch
    from paper_2402_02446_amd import binding
    layer, _ = _standin_layer(K, 128, k, seed=K, n_outlier=4)
    h = _upload(layer)
    rng = np.random.default_rng(K)
    X = np.zeros((M, K + 8), np.float32)
    X[:, :K] = rng.standard_normal((M, K))
    X[:, :K] *= (127.0 * 2.0 ** np.linspace(-28, 17, M) / np.abs(X).max(1))[:, None].astype(np.float32)
    X[7] = 0.0
    Xd = torch.from_numpy(X).cuda()[:, :K]
    codes, scales = binding.lqer_quantize_int8_token(Xd.contiguous())
    ws = h.workspace(M)
    ws.fill_(0x5A)
    binding.lqer_linear_forward(h, Xd, workspace=ws)
    torch.cuda.synchronize()
    mp = (M + 127) // 128 * 128
    got = ws[:M * K].view(torch.int8).view(M, K // 32, 2, 16).transpose(2, 3).reshape(M, K)      # runs of 32: even elements, odd ones
    assert torch.equal(got, codes)
    at = (mp * K + 255) // 256 * 256
    assert torch.equal(ws[at:at + 4 * M].view(torch.float32), scales.float())
    h.free()
