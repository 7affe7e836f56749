"""Which layers and calls take fp6 operands, and what they give: layers without such a copy at sizes that would take it, exponents far
apart inside one matrix instruction, tiles of the staged kernel above 1.5e11 operations, groups of layers of unequal widths and ranks."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload

pytestmark = pytest.mark.gpu


def _rows_and_cols(M, N):
    return np.unique([0, 63, 64, 127, 128, M // 2, M - 2, M - 1]), np.unique([0, 31, 32, 127, 128, 511 % N, N // 2, N - 1])


def _forward(layer, X):
    import torch
    from paper_2402_02446_amd import binding
    h = upload(layer)
    Y = binding.lqer_linear_forward(h, torch.from_numpy(X).cuda())
    h.free()
    rows, cols = _rows_and_cols(*Y.shape)
    return rows, cols, Y[torch.from_numpy(rows).cuda()][:, torch.from_numpy(cols).cuda()].cpu().numpy()


@pytest.mark.parametrize("byte", [0, 1])
def test_layer_whose_exponents_the_scales_cannot_hold(byte):
    """A block with codes and an exponent byte below 2: the layer keeps bf16 operands, at a size the others take fp6 ones."""
    M, K, N = 2500, 4096, 8192
    layer, ch = oracle_layer_big(K, N, 32, seed=1)
    layer.We[N - 1, 3] = byte
    X = synth.gen_activations(np.random.default_rng(2), M, K, ch, 50.0)
    rows, cols, Y = _forward(layer, X)
    assert_forward_matches(Y, X[rows], layer, cols=cols)


@pytest.mark.parametrize("M,K,N,k", [(300, 2048, 640, 32), (2100, 4096, 9000, 64)])
def test_exponents_far_apart_inside_an_instruction(M, K, N, k):
    """Blocks of both operands over some forty binades, side by side along K: sums that round at every step."""
    rng = np.random.default_rng(M)
    layer, _ = oracle_layer_big(K, N, k, seed=2)
    layer.We[:] = np.clip(layer.We.astype(int) + rng.integers(-20, 21, layer.We.shape), 2, 245)
    X = (rng.standard_normal((M, K)) * 2.0 ** np.repeat(rng.integers(-20, 21, (M, K // 16)), 16, axis=1)).astype(np.float32)
    rows, cols, Y = _forward(layer, X)
    assert_forward_matches(Y, X[rows], layer, cols=cols)


# short K, a large rank, few columns: shapes of the staged kernel where tiled_kernel's used to be the only ones
@pytest.mark.parametrize("M,K,N,k", [(20000, 256, 16400, 128), (3640, 816, 25700, 256), (65500, 7300 // 16 * 16, 160, 32)])
def test_large_calls_in_staged_tiles(M, K, N, k):
    layer, ch = oracle_layer_big(K, N, k, seed=3)
    X = synth.gen_activations(np.random.default_rng(4), M, K, ch, 50.0)
    rows, cols, Y = _forward(layer, X)
    assert_forward_matches(Y, X[rows], layer, cols=cols)


@pytest.mark.parametrize("M,K,specs", [
    (256, 4096, ((4096, 32), (1024, 32), (1024, 32))), (2048, 4096, ((4096, 32), (1024, 32), (1024, 32))),
    (4500, 2048, ((8192, 256), (512, 256), (512, 16))), (8000, 512, ((20000, 128), (1024, 128), (96, 0))), (40, 1024, ((1024, 64), (96, 16)))])
def test_groups_of_unequal_layers(M, K, specs):
    import torch
    from paper_2402_02446_amd import binding
    hs = [upload(oracle_layer_big(K, N, k, seed=60 + i)[0]) for i, (N, k) in enumerate(specs)]
    rng = np.random.default_rng(M)
    X = torch.from_numpy((rng.standard_normal((M, K)) * np.exp(2.0 * rng.standard_normal((M, K)))).astype(np.float32)).cuda()
    for g, h in zip(binding.lqer_linear_forward_shared(hs, X), hs):
        assert torch.equal(g, binding.lqer_linear_forward(h, X))
        h.free()


# Both sides of the lines: few K tiles and a rank up to 32, one tile at any rank, eight tiles and more on few activations.  A call on bf16
# operands has the bits it has without the fp6 copy of the weights; one on fp6 operands sums in another order.
@pytest.mark.parametrize("M,K,N,k,six", [(700, 512, 400, 32, False), (3125, 512, 400, 32, False), (3126, 512, 400, 32, True), (700, 512, 400, 33, True),
                                         (12500, 256, 300, 64, False), (12501, 256, 300, 64, True), (500, 1024, 400, 8, False), (501, 1024, 400, 8, True),
                                         (69, 4096, 640, 32, False), (74, 4096, 640, 32, True), (69, 4096, 640, 64, True), (150, 1040, 400, 32, True)])
def test_which_calls_take_fp6_operands(M, K, N, k, six):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = oracle_layer_big(K, N, k, seed=5)
    h = upload(layer)
    X = synth.gen_activations(np.random.default_rng(4), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    Y = binding.lqer_linear_forward(h, Xd)
    h.drop_fp6()
    assert torch.equal(binding.lqer_linear_forward(h, Xd), Y) != six
    h.free()
    rows, cols = _rows_and_cols(M, N)
    rows = rows[rows < M]
    assert_forward_matches(Y.cpu().numpy()[np.ix_(rows, cols)], X[rows], layer, cols=cols)


def test_tiles_of_a_large_ragged_y():
    """Two K tiles and a Y beyond the caches whose rows share cache lines: tiles of 64 rows, which sum two chains, not those of 128 x 512, which
    sum one.  (Half of the time of the large ones is such lines' way to memory and back.)"""
    import torch
    from paper_2402_02446_amd import binding
    M, K, N = 8192, 512, 16244
    h = upload(oracle_layer_big(K, N, 32, seed=6)[0])
    X = torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    Y = binding.lqer_linear_forward(h, X)
    assert torch.equal(Y, binding.lqer_linear_forward_ex(h, X, path=2, variant=143))
    assert not torch.equal(Y, binding.lqer_linear_forward_ex(h, X, path=2, variant=121))
    h.free()
