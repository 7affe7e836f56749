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
