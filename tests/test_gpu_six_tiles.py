"""Tiles of the kernel on fp6 operands at the edges of its dispatch: the 128 x 128 shape whole and in planes; T final, as two and as more
partial sums, one and several rounds of 64 ranks of the correction; rows and columns that end inside and at the end of a tile; the same bits
whatever the workspace held before."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from helpers import oracle_layer_big, upload
from test_gpu_planes import _run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [144, 244])
@pytest.mark.parametrize("M,K,N,k", [(33, 512, 32, 8), (128, 528, 128, 33), (129, 1296, 144, 130), (257, 768, 1042, 256)])
def test_128_x_128(variant, M, K, N, k):
    layer, ch = oracle_layer_big(K, N, min(k, N), seed=M + K)
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()


# three K tiles: T final; six, nine and seventeen: two, four and eight partial sums
@pytest.mark.parametrize("variant", [121, 122, 142, 143, 144])
@pytest.mark.parametrize("M,K,N,k", [(300, 704, 512, 64), (256, 1536, 1042, 65), (128, 2064, 256, 32), (65, 4112, 544, 200)])
def test_partial_sums_of_t(variant, M, K, N, k):
    layer, ch = oracle_layer_big(K, N, k, seed=M)
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()


@pytest.mark.parametrize("variant", [121, 122, 221, 222])
def test_bits_do_not_depend_on_the_workspace(variant):
    import torch
    from paper_2402_02446_amd import binding
    M, K, N, k = 1000, 2064, 1200, 72
    layer, _ = oracle_layer_big(K, N, k, seed=9)
    h = upload(layer)
    X = torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    ws = h.workspace(M, 2)
    first = None
    for fill in (0, 255, 127):
        ws.fill_(fill)
        Y = binding.lqer_linear_forward_ex(h, X, workspace=ws, path=2, variant=variant)
        first = Y if first is None else first
        assert torch.equal(first, Y)
    h.free()
