"""Per-token INT8 codes without a division per value: bit for bit what dividing in fp32 gives, at the ties between two codes and
the fp32 values beside them, for scales over the whole fp16 range, for scales that round to zero or infinity, and for rows longer
and shorter than what the kernel keeps in registers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _expected(X):
    with np.errstate(all="ignore"):
        m = np.abs(X).max(1)
        s = np.where(m == 0, np.float16(1), (m / np.float32(127)).astype(np.float16))
        q = np.rint(X / s.astype(np.float32)[:, None])
        return np.clip(np.where(np.isnan(q), -127, q), -127, 127).astype(np.int8), s


def _check(X):
    import torch
    from paper_2402_02446_amd import binding
    codes, scales = binding.lqer_quantize_int8_token(torch.from_numpy(X).cuda())
    want, s = _expected(X)
    assert np.array_equal(scales.cpu().numpy().view(np.uint16), s.view(np.uint16))
    assert np.array_equal(codes.cpu().numpy(), want)


def test_ties_and_their_neighbours():
    rng = np.random.default_rng(0)
    bits = np.unique(np.r_[1:64, 1000:1100, 0x3C00, 0x3BFF, 0x7BFF, rng.integers(1, 0x7C00, 800)]).astype(np.uint16)
    s = bits.view(np.float16).astype(np.float32)[:, None]
    mid = (s * (np.arange(-127, 127, dtype=np.float32) + np.float32(0.5))[None, :]).astype(np.float32)        # exact: 11 + 8 bits
    X = np.concatenate([s * np.float32(127), mid, np.nextafter(mid, np.float32(np.inf)), np.nextafter(mid, np.float32(-np.inf))], 1)
    X = np.concatenate([X, np.zeros((X.shape[0], -X.shape[1] % 4), np.float32)], 1).astype(np.float32)
    _check(X)


# maxima from 127 2^-26 (a scale of zero) to 127 2^16 (an infinite one); rows around 1024, 4 x 1024 and 12 x 1024 values
@pytest.mark.parametrize("K", [4, 252, 1024, 1028, 4092, 4100, 11008, 12288, 12292, 28672])
def test_scales_and_lengths(K):
    rng = np.random.default_rng(K)
    X = rng.standard_normal((48, K)).astype(np.float32)
    X *= (127.0 * 2.0 ** np.linspace(-28, 17, 48) / np.abs(X).max(1))[:, None].astype(np.float32)
    X[7] = 0.0
    _check(X)
