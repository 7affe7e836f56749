"""lqer_linear_forward_shared on few tokens: layers that take the same shape of the streaming kernel run as one launch pair.
Every Y holds the bits of the layer's own forward pass - pairs of workgroups, single ones, ragged widths, different ranks
including none, both exponent forms, more layers than one launch takes, layers of other formats in between - also with only
the workspace that the widest layer needs alone, on a second run, and in a replayed graph."""
import numpy as np
import pytest

from paper_2402_02446_amd import synth
from helpers import assert_forward_matches, oracle_layer_big, upload

pytestmark = pytest.mark.gpu


def _layers(K, specs):
    from oracle import factors
    out = []
    for i, (N, k, w_bits) in enumerate(specs):
        if w_bits == 4 and i % 2 == 1:
            d = synth.random_packed_layer(np.random.default_rng(100 * K + i), K, N, k)
            d["We"][0, 0] = 90                                   # spans more than 16 values: exponent bytes, not nibbles
            out.append(factors.PackedLayer(**d))
        else:
            out.append(oracle_layer_big(K, N, k, seed=i, w_bits=w_bits)[0])
    return out


@pytest.mark.parametrize("K,specs", [
    (4096, [(1040, 32, 4), (1040, 16, 4), (528, 0, 4)]),                                 # pairs of workgroups
    (2304, [(100, 0, 4), (272, 33, 4), (1001, 64, 4), (33, 8, 4), (64, 24, 4), (272, 16, 2), (272, 40, 4)]),
    (1040, [(11008, 8, 4), (10300, 24, 4)]),                                             # two column groups per wavefront
    (4624, [(10272, 0, 4), (10300, 64, 4)]),                                             # and two slices of K each
])
@pytest.mark.parametrize("M", [1, 4, 5, 16, 17, 32])
def test_shared_few_tokens(K, specs, M):
    _run(K, specs, M)


# The shapes that those layers, pairs of workgroups nearly all, do not take: one workgroup per column group or two, K in one
# step (272, 1552: one tile, seven) or several (2304: nine) - 11181 / 11241 - and two wavefronts of two column groups - 12241 -
# in one step and in several.
@pytest.mark.parametrize("K,specs", [
    (272, [(100, 8, 4), (272, 33, 4), (1001, 0, 4)]),
    (1552, [(2080, 24, 4), (65, 64, 4)]),
    (2304, [(5200, 32, 4), (5281, 16, 4)]),
    (272, [(25504, 16, 4), (25600, 64, 4)]),
    (2576, [(25504, 0, 4), (25540, 32, 4)]),
])
@pytest.mark.parametrize("M", [4, 16, 32])
def test_shared_few_tokens_other_shapes(K, specs, M):
    _run(K, specs, M)


def _run(K, specs, M):
    import torch
    from paper_2402_02446_amd import binding
    layers = _layers(K, specs)
    hs = [upload(l) for l in layers]
    ch = synth.gen_outlier_channels(np.random.default_rng(1), K, 8)
    X = synth.gen_activations(np.random.default_rng(M), M, K, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    out = lambda: [torch.full((M, (l.N + 3) // 4 * 4), 7.0, dtype=torch.float32, device="cuda")[:, :l.N] for l in layers]
    alone = out()
    for h, Y in zip(hs, alone):
        binding.lqer_linear_forward(h, Xd, Y=Y)
    least = max(binding.lqer_linear_workspace_bytes(h, M) for h in hs)
    full = binding.lqer_linear_shared_workspace_bytes(hs, M)
    assert full >= least
    for nbytes, fill in ((full, 0), (full, 255), (least, 255)):
        ws = torch.full((nbytes,), fill, dtype=torch.uint8, device="cuda")
        Ys = out()
        binding.lqer_linear_forward_shared(hs, Xd, Ys=Ys, workspace=ws)
        torch.cuda.synchronize()
        for i, (Y, w) in enumerate(zip(Ys, alone)):
            assert torch.equal(Y, w), (i, nbytes, fill)
            assert (Y._base[:, layers[i].N:] == 7.0).all()
    for l, Y in zip(layers, alone):
        if l.N < 2000:
            assert_forward_matches(Y.cpu().numpy(), X, l)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    Ys = out()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        binding.lqer_linear_forward_shared(hs, Xd, Ys=Ys, workspace=ws)
    for rep in range(3):
        for Y in Ys:
            Y.fill_(float("nan"))
        binding.lqer_linear_forward(hs[0], Xd)                  # eager work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(Y, w) for Y, w in zip(Ys, alone)), rep
    for h in hs:
        h.free()
