"""Device memory that a layer takes beside its records: the fp6 copy of 4-bit weights."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

K, N = 8192, 4096
RECORDS = K // 256 * (N // 32) * 4608               # bytes of one form of the weights, at most


def _import(k):
    """A layer of zero codes, and the device memory its import took."""
    import torch
    from paper_2402_02446_amd import binding
    kp = (k + 15) // 16 * 16
    fac = () if k == 0 else (np.zeros((kp, K), np.int8), np.full((kp, K // 16), 127, np.uint8),
                             np.zeros((N, kp), np.int8), np.full((N, kp // 16), 127, np.uint8))
    We = np.full((N, K // 16), 120, np.uint8)
    We[0, 0] = 100                                  # the wider form of the records
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    h = binding.lqer_layer_import(K, N, k, np.zeros((N, K // 2), np.uint8), We, *fac)
    return h, free - torch.cuda.mem_get_info()[0]


def test_rank_zero_has_one_form_of_the_weights():
    _import(0)[0].free()                            # (what a process's first import takes for good)
    h, taken = _import(0)
    h.free()
    assert taken < 1.5 * RECORDS


def test_the_copy_gives_way_on_a_fuller_card():
    import torch
    _import(16)[0].free()
    h, taken = _import(16)
    h.free()
    assert 1.5 * RECORDS < taken < 2.5 * RECORDS
    total = torch.cuda.mem_get_info()[1]
    held = torch.empty(total // 2, dtype=torch.uint8, device="cuda")
    h, taken = _import(16)
    Y = h_forward(h)
    h.free()
    del held
    torch.cuda.empty_cache()
    assert taken < 1.5 * RECORDS
    assert not Y.any()                              # (zero codes)


def h_forward(h):
    import torch
    from paper_2402_02446_amd import binding
    return binding.lqer_linear_forward(h, torch.randn(300, K, device="cuda")).cpu()


def test_the_copy_can_be_seen_and_given_back():
    import torch
    from helpers import assert_forward_matches, oracle_layer_big, upload
    from paper_2402_02446_amd import binding, synth
    layer, ch = oracle_layer_big(1024, 416, 32, seed=5)
    X = synth.gen_activations(np.random.default_rng(5), 700, 1024, ch, 50.0)
    Xd = torch.from_numpy(X).cuda()
    h = upload(layer)
    assert h.fp6_bytes() == 4 * 13 * 4608
    first = binding.lqer_linear_forward(h, Xd)
    h.drop_fp6()
    assert h.fp6_bytes() == 0
    h.drop_fp6()                                    # (nothing left)
    assert_forward_matches(binding.lqer_linear_forward(h, Xd).cpu().numpy(), X, layer)
    assert_forward_matches(first.cpu().numpy(), X, layer)
    with pytest.raises(binding.LqerError, match="LQER_ERR_SHAPE"):
        binding.lqer_linear_forward_ex(h, Xd, path=2, variant=121)      # an fp6 shape by force
    h.free()
    for other in (upload(oracle_layer_big(1024, 416, 0, seed=6)[0]), upload(oracle_layer_big(1024, 416, 32, seed=7, w_bits=2)[0])):
        assert other.fp6_bytes() == 0
        other.drop_fp6()
        other.free()
    assert binding.lib().lqer_layer_fp6_bytes(None) == 0 and binding.lib().lqer_layer_drop_fp6(None) == 1
