"""The staged kernel spells out a K tile's four chunks and its last tile apart: one K tile, two, and few, whole and as planes of
one or two tiles each, with and without a correction, both weight widths and exponent forms, against the oracle."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from helpers import oracle_layer_big, upload
from test_gpu_planes import _run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [131, 132, 133, 231, 232, 233])
@pytest.mark.parametrize("w_bits", [4, 2])
@pytest.mark.parametrize("M,K,N,k,wide", [(33, 16, 32, 0, False), (64, 256, 144, 16, True), (65, 240, 520, 130, False), (70, 512, 96, 40, False),
                                          (129, 768, 272, 0, True), (47, 1280, 130, 65, False)])
def test_few_k_tiles(variant, w_bits, M, K, N, k, wide):
    if variant > 200 and K <= 256:
        pytest.skip("one K tile: no planes")
    layer, ch = oracle_layer_big(K, N, min(k, N), seed=M + K + w_bits, w_bits=w_bits)
    if wide:
        layer.We[0, 0], layer.We[N - 1, -1] = 90, 140             # more than 16 values apart
    h = upload(layer)
    _run_and_check(layer, h, synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0), path=2, variant=variant)
    h.free()
