"""The statistics epilogue on logits near the lowest bf16 value."""

import numpy as np
import pytest
import torch

from oracle import accept as oa
from tests.gpu_util import dev_f32, dev_u8, host, host_bf16_bits, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,V,K,lda", [
    (8, 1024, 128, 0), (33, 28672, 256, 0), (320, 4096, 256, 0), (33, 2048, 256, 140_000_000),
])
def test_statistics_of_logits_near_the_lowest_value(M, V, K, lda):
    """Logits so low that z * c2 overflows to -inf count as absent, also where
    they fill all of a lane's or a group's columns."""
    p = need_gpu()
    say(f"lowest logits M={M} V={V} K={K} lda={lda}")
    T = 0.7
    a = torch.full((M, K), 0x38, dtype=torch.uint8, device="cuda")         # 1.0
    if lda:
        v = torch.empty(((M - 1) * lda + K,), dtype=torch.uint8, device="cuda").as_strided((M, K), (lda, 1))
        v.copy_(a)
        a = v
    w = np.full((V, K), 0x38, np.uint8)
    sw = np.random.default_rng(3).uniform(0.5, 1.5, V).astype(np.float32) * np.float32(4.0 / K)
    low = np.arange(V) // 512 % 2 == 0
    low[: V // 4] = True
    w[low] = 0xB8
    sw[low] = np.float32(3.2e38 / K)
    z, st = p.gemm_logit_stats(a, dev_f32(np.ones(M)), dev_u8(w), dev_f32(sw), T)
    bits = host_bf16_bits(z)
    zf = (bits.astype(np.uint32) << 16).view(np.float32)
    assert np.all(np.isfinite(zf)) and np.all(zf[:, low] < -3e38)
    st = host(st)
    assert not np.any(np.isnan(st))
    m, s = st[..., 0].astype(np.float64), st[..., 1].astype(np.float64)
    Mg = m.max(axis=1)
    Z = np.sum(s * np.exp2(np.where(np.isfinite(m), m, -np.inf) - Mg[:, None]), axis=1)
    zmax, Zr = oa.softmax_normalizer(bits, T)
    c2 = np.float32(1.4426950408889634 / float(np.float32(T)))
    np.testing.assert_array_equal(Mg.astype(np.float32), (zmax * np.float64(c2)).astype(np.float32))
    np.testing.assert_allclose(Z, Zr, rtol=2e-5)
