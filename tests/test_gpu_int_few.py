"""The INT variant's few-token launches: edges of the blocks of 32 tokens, column counts around a workgroup's 32, K groups
that slices, wavefronts and register sets do not divide, ranks to 128, all-zero tokens; its general launches on the fewest
tokens that take them - K planes of both products, a plane of its own for the correction, ragged row tiles; against the
oracle, and the same bits on a second run with other contents in the workspace."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from test_gpu_int import _check, _standin_layer, _upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,k", [(1, 128, 33, 16), (4, 1152, 64, 128), (5, 7296, 65, 33), (17, 4224, 100, 8), (31, 11008, 96, 32),
                                     (32, 2304, 31, 0), (33, 4096, 1040, 64), (128, 1024, 528, 100)])
def test_few_tokens(M, K, N, k):
    _run(M, K, N, k)


# more than 128 tokens, or more work than the few-token launches take; 7 ranks blocks of 16, an odd number, and 8
@pytest.mark.parametrize("M,K,N,k", [(129, 2304, 528, 33), (200, 4096, 1100, 64), (100, 11008, 4096, 32), (130, 512, 300, 128),
                                     (257, 1024, 2080, 112), (70, 8192, 11008, 16)])
def test_general_launches(M, K, N, k):
    _run(M, K, N, k)


def _run(M, K, N, k):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = _standin_layer(K, N, min(k, N), seed=K + M, n_outlier=4)
    h = _upload(layer)
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 30.0)
    if M > 2:
        X[M // 2] = 0.0
    ws = h.workspace(M)
    first = None
    for fill in (0, 255):
        ws.fill_(fill)
        buf = torch.full((M, (N + 7) // 4 * 4), 7.0, dtype=torch.float32, device="cuda")
        binding.lqer_linear_forward(h, torch.from_numpy(X).cuda(), Y=buf[:, :N])
        torch.cuda.synchronize()
        assert (buf[:, N:] == 7.0).all()
        first = buf[:, :N].clone() if first is None else first
        assert torch.equal(buf[:, :N], first)
    _check(first.cpu().numpy(), X, layer)
    h.free()


# Without a correction Y is a sum of K / 128 scaled group sums times one token scale.  One fp32 rounding of it is 2.5e-8 rms
# (2^-24 / sqrt(3), over a factor of 2 of values); the few additions before are small beside it.  With the scale applied to
# each of two planes it is 3.7e-8.
def test_token_scale_is_applied_once():
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = _standin_layer(512, 11008, 0, seed=1)
    h = _upload(layer)
    X = synth.gen_activations(np.random.default_rng(1), 200, 512, ch, 50.0)
    cols = np.arange(0, 11008, 7)
    Y = binding.lqer_linear_forward(h, torch.from_numpy(X).cuda()).cpu().numpy()[:, cols]
    err, _ = _check(Y, X, layer, cols)
    assert err <= 3.0e-8, err
    h.free()


# Which launches a call takes shows in the workspace it asks for: the general ones keep 128 rows of codes and planes of Y, the
# few-token ones whole blocks of 32 rows.  Either form's workspace is enough for the call, and both give the oracle's result.
@pytest.mark.parametrize("M,K,N,general", [(32, 512, 11008, False), (128, 512, 11008, True), (96, 4096, 2048, False), (32, 28672, 1024, True),
                                           (1, 28672, 1024, False), (70, 1024, 16384, True)])
def test_which_launches_and_either_workspace(M, K, N, general):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = _standin_layer(K, N, 0, seed=M)
    h = _upload(layer)
    need = binding.lqer_linear_workspace_bytes(h, M)
    few = (M + 31) // 32 * 32 * K + 512                          # rank 0: codes and token scales
    assert need > few if general else need == few
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    cols = np.arange(0, N, 5)
    for nbytes in (need, few):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
        Y = binding.lqer_linear_forward(h, torch.from_numpy(X).cuda(), workspace=ws)
        _check(Y.cpu().numpy()[:, cols], X, layer, cols)
    with pytest.raises(binding.LqerError):
        binding.lqer_linear_forward(h, torch.from_numpy(X).cuda(), workspace=ws[:few - 256])
    h.free()


# The same at ranks whose general launches quantize and project in one: the planes of T are reserved whatever its form.
@pytest.mark.parametrize("M,K,N,k,general", [(9, 1024, 4288, 48, False), (55, 256, 11168, 8, True), (32, 128, 15168, 32, True), (16, 4096, 4096, 32, False),
                                             (64, 11264, 544, 16, True), (24, 11264, 544, 16, False), (40, 2048, 2048, 33, False), (7, 640, 15808, 32, False)])
def test_which_launches_with_a_small_rank(M, K, N, k, general):
    import torch
    from paper_2402_02446_amd import binding
    layer, ch = _standin_layer(K, N, k, seed=M)
    h = _upload(layer)
    need = binding.lqer_linear_workspace_bytes(h, M)
    at = lambda n: (n + 255) // 256 * 256
    per = min((K // 128 + 7) // 8, 7)
    few = at((M + 31) // 32 * 32 * K) + at(512) + at((K // 128 + per - 1) // per * M * ((k + 31) // 32 * 32) * 4)
    assert need > few if general else need == few
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    cols = np.arange(0, N, 5)
    for nbytes in (need, few):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
        Y = binding.lqer_linear_forward(h, torch.from_numpy(X).cuda(), workspace=ws)
        _check(Y.cpu().numpy()[:, cols], X, layer, cols)
    h.free()
