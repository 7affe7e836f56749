"""The projection step, whose wavefronts take quarters of a K tile (64 columns): K that ends inside a block group, a quarter or
a tile, fewer quarters than wavefronts and several rounds of them, token rows that do not fill 16, each rank-group count it has
an instance for, every source (fp32, codes) and layout (cells, code cells, rows), against the oracle."""
import numpy as np
import pytest

from oracle import mxint
from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload

pytestmark = pytest.mark.gpu


# cells (M <= 32), code cells (16 < .. of single workgroups per column block), rows (M > 32), the last one with as
# many wavefronts as tiles, four quarters each
@pytest.mark.parametrize("M", [1, 5, 17, 33, 47, 1043])
@pytest.mark.parametrize("K,N,k,w_bits", [(16, 40, 8, 4), (80, 100, 0, 4), (272, 64, 24, 4), (1040, 96, 40, 4), (4176, 70, 64, 4),
                                          (11056, 48, 16, 4), (4112, 64, 256, 2), (33040, 32, 33, 2)])
def test_forward_and_codes(M, K, N, k, w_bits):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = oracle_layer_big(K, N, k if k <= min(K, N) else min(K, N), seed=K + M, w_bits=w_bits)
    X = synth.gen_activations(np.random.default_rng(M + K), M, K, ch, 50.0)
    h = upload(layer)
    Xd = torch.from_numpy(X).cuda()
    out = lambda: torch.full((M, (N + 3) // 4 * 4), 7.0, device="cuda")[:, :N]
    ws = torch.full((binding.lqer_linear_workspace_bytes(h, M),), 255, dtype=torch.uint8, device="cuda")
    Y = binding.lqer_linear_forward(h, Xd, Y=out(), workspace=ws)
    assert_forward_matches(Y.cpu().numpy(), X, layer)
    codes, exps = binding.lqer_quantize_mx(Xd, 8)
    oc, oe = mxint.mx_quantize(X, 8, axis=-1)
    assert np.array_equal(codes.cpu().numpy(), oc) and np.array_equal(exps.cpu().numpy(), oe)
    ws.fill_(255)
    assert torch.equal(binding.lqer_linear_forward_q(h, codes, exps, Y=out(), workspace=ws), Y)
    h.free()


# Ranks above 64 where project_kernel takes the groups beyond the fourth (M K (kp - 64) above 1.3e9, four K tiles a slice): planes of six, five
# and four groups, the last one short; 64 and 32 rows a wavefront; T final and in slices; fp6 and (rank 0 first, so that they share) bf16 operands
@pytest.mark.parametrize("M,K,k,w_bits,wide", [(2050, 4096, 256, 2, False), (4100, 2064, 192, 4, False), (8200, 2048, 140, 2, True), (1100, 8192, 256, 4, False)])
def test_ranks_above_64_of_large_calls(M, K, k, w_bits, wide):
    import torch
    from paper_2402_02446_amd import binding
    N = 288
    layer, ch = oracle_layer_big(K, N, k, seed=M, w_bits=w_bits)
    if wide:
        layer.We[0, 0] = 90                                       # bf16 operands for a 2-bit layer
    h = upload(layer)
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    Y = binding.lqer_linear_forward(h, Xd)
    rows, cols = np.array([0, 15, 16, 31, 32, 63, 64, M // 2, M - 1]), np.arange(0, N, 3)
    assert_forward_matches(Y.cpu().numpy()[np.ix_(rows, cols)], X[rows], layer, cols=cols)
    other = upload(oracle_layer_big(K, 96, 32, seed=1, w_bits=w_bits)[0])
    for first, second in ((other, h), (h, h)):
        assert torch.equal(binding.lqer_linear_forward_shared([first, second], Xd)[1], Y)      # from the stored activations: the same bits
    other.free()
    h.free()


# Slices of K: as many as make one workgroup to a compute unit of at least three quarters of them, else 384 workgroups.  The partial sums of
# T are in the workspace: two layers of ranks 16 and 32, whose rows are equally long, differ by them alone.
@pytest.mark.parametrize("M,K,slices", [(1024, 4096, 4), (1040, 4096, 8), (1536, 4096, 2), (2048, 4096, 2), (2049, 4096, 4), (3056, 4096, 4), (3057, 4096, 1),
                                        (4096, 10704, 1), (4097, 10704, 2), (4133, 1008, 2), (4133, 768, 1), (6128, 4096, 2), (6129, 4096, 1), (8177, 4096, 1)])
def test_slices_of_the_contraction(M, K, slices):
    import torch
    from paper_2402_02446_amd import binding
    layers = [oracle_layer_big(K, 64, k, seed=k) for k in (16, 32)]
    hs = [upload(layer) for layer, _ in layers]
    need = [binding.lqer_linear_workspace_bytes(h, M) for h in hs]
    rows = (M + 95 + 255) // 256 * 256
    assert need[1] - need[0] == (rows * 16 * 4 * slices if slices > 1 else 0)
    X = synth.gen_activations(np.random.default_rng(M), M, K, layers[1][1], 50.0)
    Y = binding.lqer_linear_forward(hs[1], torch.from_numpy(X).cuda())
    at = np.array([0, 15, 16, 127, 128, M // 2, M - 1])
    assert_forward_matches(Y.cpu().numpy()[at], X[at], layers[1][0])
    for h in hs:
        h.free()
