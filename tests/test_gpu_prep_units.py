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
# and four groups, even ones and a last one that is short; 64 and 32 rows a wavefront; T final and in slices; fp6 operands, and bf16 ones (2-bit
# layers whose exponents are far apart); 8- and 6-bit activations, as fp32, as codes and as another layer has stored them.
@pytest.mark.parametrize("M,K,k,w_bits,wide,act_bits,rows", [
    (2050, 4096, 256, 2, False, 8, 64), (4000, 2576, 192, 4, False, 8, 32), (4100, 2576, 192, 4, False, 6, 64), (8200, 2048, 140, 2, True, 8, 32),
    (1100, 8192, 256, 4, False, 8, 64), (8200, 1296, 192, 4, False, 8, 64), (8200, 1040, 256, 2, True, 8, 64), (4100, 2064, 256, 4, False, 8, 64),
    (8200, 1296, 240, 4, False, 6, 64), (3900, 2576, 208, 4, False, 8, 32), (8200, 3344, 112, 4, False, 8, 32)])
def test_ranks_above_64_of_large_calls(M, K, k, w_bits, wide, act_bits, rows):
    import torch
    from paper_2402_02446_amd import binding
    N = 288
    layer, ch = oracle_layer_big(K, N, k, seed=M, w_bits=w_bits)
    others = [oracle_layer_big(K, 96, r, seed=1, w_bits=w_bits)[0] for r in (32, 16)]
    if wide:
        for l in [layer] + others:
            l.We[0, 0] = 90
    h, other, small = upload(layer), upload(others[0]), upload(others[1])
    # the kernel, and its rows: what launch_prep and launch_project go by
    tp_rows, KT, kp = (M + 95 + 255) // 256 * 256, (K + 255) // 256, (k + 15) // 16 * 16
    slices = max(1, (binding.lqer_linear_workspace_bytes(other, M) - binding.lqer_linear_workspace_bytes(small, M)) // (tp_rows * 16 * 4))
    planes = (kp // 16 - 4 + 5) // 6
    assert M * K * (kp - 64) > 1.3e9 and -(-KT // slices) >= 4
    assert rows == (64 if -(-M // 64) * slices * planes >= 256 else 32)
    for x in (h, other):
        x.set_activation_bits(act_bits)
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    Y = binding.lqer_linear_forward(h, Xd)
    at, cols = np.array([0, 15, 16, 31, 32, 63, 64, M // 2, M - 1]), np.arange(0, N, 3)
    assert_forward_matches(Y.cpu().numpy()[np.ix_(at, cols)], X[at], layer, cols=cols, act_bits=act_bits)
    codes, exps = binding.lqer_quantize_mx(Xd, act_bits)
    assert torch.equal(binding.lqer_linear_forward_q(h, codes, exps), Y)
    for first in (other, h):                                        # from the stored activations: the same bits
        assert torch.equal(binding.lqer_linear_forward_shared([first, h], Xd)[1], Y)
    for x in (h, other, small):
        x.free()


# Slices of K: as many as make one workgroup to a compute unit of at least three quarters of them, else 384 workgroups if a slice keeps three tiles.  The partial sums of
# T are in the workspace: two layers of ranks 16 and 32, whose rows are equally long, differ by them alone.
@pytest.mark.parametrize("M,K,slices", [(1024, 4096, 4), (1040, 4096, 4), (1040, 6144, 8), (1536, 4096, 2), (2048, 4096, 2), (2049, 4096, 4), (3056, 4096, 4), (3057, 4096, 1),
                                        (4096, 10704, 1), (4097, 10704, 2), (4133, 1536, 2), (4133, 1280, 1), (4133, 768, 1), (2049, 3072, 4), (2049, 2816, 2), (6128, 4096, 2), (6129, 4096, 1), (8177, 4096, 1)])
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


# 188 blocks of 16 tokens take four slices of K; on the static scratch, which holds T in two but not in four, two; so in a workspace of that size.
def test_fewer_slices_where_the_scratch_is_full():
    import torch
    from paper_2402_02446_amd import binding
    M, K, N, k = 3000, 3072, 288, 256
    layer, ch = oracle_layer_big(K, N, k, seed=9)
    h = upload(layer)
    rows, part = (M + 95 + 255) // 256 * 256, (M + 95 + 255) // 256 * 256 * k * 4
    plan = rows * (K + 2 * k) * 2
    assert plan + 2 * part < (32 << 20) < plan + 4 * part
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    at = np.array([0, 15, 16, 127, 128, M // 2, M - 1])
    need = binding.lqer_linear_workspace_bytes(h, M)
    few = torch.full((need - 2 * part,), 255, dtype=torch.uint8, device="cuda")
    Y = binding.lqer_linear_forward_static(h, Xd)
    for y in (Y, binding.lqer_linear_forward(h, Xd, workspace=few), binding.lqer_linear_forward_shared([h, h], Xd, workspace=few)[1]):
        assert_forward_matches(y.cpu().numpy()[at], X[at], layer)
    with pytest.raises(binding.LqerError, match="LQER_ERR_WORKSPACE"):
        binding.lqer_linear_forward(h, Xd, workspace=few[:-256])
    with pytest.raises(binding.LqerError, match="LQER_ERR_WORKSPACE"):
        binding.lqer_linear_forward_shared([h, h], Xd, workspace=few[:-256])
    with pytest.raises(binding.LqerError, match="LQER_ERR_WORKSPACE"):
        binding.lqer_linear_forward_static(h, torch.zeros(4700, K, device="cuda"))
    h.free()
