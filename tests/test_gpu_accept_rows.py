"""Logit rows that start on any 2-byte boundary and vocabularies that are no
multiple of 8, against the same logits in aligned rows padded with -inf to a
multiple of 8: padding adds exact zeros to every sum and wins no maximum, so
chains and trees, greedy and sampled, must give the same tokens.  The logits
around the tensor are larger than any in it."""

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import accept as oa
from tests.gpu_util import dev_f32, dev_i32, host, need_gpu, say

pytestmark = pytest.mark.gpu

HIGH, NEG_INF = 0x7f00, 0xff80           # bf16 bits: 1.7e38 and -inf


def _dev(bits, off):
    """The bits as a bf16 tensor that starts `off` elements into its buffer."""
    buf = np.full(bits.size + off + 8, HIGH, np.uint16)
    buf[off:off + bits.size] = bits.reshape(-1)
    t = torch.from_numpy(buf.view(np.int16)).cuda().view(torch.bfloat16)
    return t[off:off + bits.size].view(bits.shape)


def _padded(bits):
    V = bits.shape[-1]
    out = np.full(bits.shape[:-1] + ((V + 7) // 8 * 8,), NEG_INF, np.uint16)
    out[..., :V] = bits
    return out


@pytest.mark.parametrize("V", [1, 2, 7, 8, 9, 15, 63, 4095, 4096, 4097, 4103, 8191, 16383, 16384, 16389, 32001])
@pytest.mark.parametrize("off", [0, 1, 4, 7])
def test_rows_on_any_boundary(V, off):
    p = need_gpu()
    say(f"accept rows V={V} offset={off}")
    B, k = 5, 3
    zt, zd = wl.accept_logits(B, k, V, V, 0.9, scale=2.0)
    zt[1, :, V - 1] = 0x4200             # 32: the last logit of these rows is their maximum
    x = wl.draft_tokens_sampled(zd, 0.7, seed=3)
    u = wl.philox_uniforms((B, k + 1), seed=4)
    u[2] = np.float32(1 - 2.0 ** -24)    # the last element with mass
    par = np.tile(np.array([-1, -1, 0], np.int32), (B, 1))
    a = (_dev(zt, off), _dev(zd, off))
    b = (_dev(_padded(zt), 0), _dev(_padded(zd), 0))
    dx, du = dev_i32(x), dev_f32(u)

    def runs(t, d):
        yield p.verify_accept(t, None, dx, None, 0.0)
        yield p.verify_accept(t, d, dx, du, 0.7)
        yield p.verify_accept(t, None, dx, du, 0.7)
        yield p.verify_accept_tree(t, dev_i32(par), dx, None, 0.0)
        yield p.verify_accept_tree(t, dev_i32(par), dx, du, 0.7)

    got, want = list(runs(*a)), list(runs(*b))
    for g, w in zip(got, want):
        for x1, x2 in zip(g, w):
            np.testing.assert_array_equal(host(x1), host(x2))
    out, num = oa.accept_greedy(zt, x)
    np.testing.assert_array_equal(host(got[0][0]), out)
    np.testing.assert_array_equal(host(got[0][1]), num)


@pytest.mark.parametrize("V", [16384 * 16, 16384 * 16 + 5, 16384 * 33 + 64])   # one batch of chunks, the next, a third
def test_sampling_positions_over_batches_of_chunks(V):
    """Uniform logits of weight 2^-60 but for a few tokens of equal weight, spread
    over the vocabulary: u picks the tokens in order, at every place of the
    search (first and last chunk, chunk and wave edges, both sides of a batch).
    The u lie in the middle of the tokens' intervals, so rounding cannot matter."""
    p = need_gpu()
    say(f"search V={V}")
    toks = sorted({0, 63, 64, 4095, 4096, 16383, 16384, V // 2, 262143 % V, V - 65, V - 1})
    n = len(toks)
    z = np.full((n, 1 + 1, V), -60 * 0.6931, np.float32)
    z[:, :, toks] = 0.0
    zt = wl.bf16_bits_from_f32(z)
    x = np.full((n, 1), V + 1, np.int32)                     # rejected: the sample comes from row 0
    u = np.stack([np.full(n, 0.5), (np.arange(n) + 0.5) / n], 1).astype(np.float32)
    t = _dev(zt, 0)
    out, num = p.verify_accept(t, None, dev_i32(x), dev_f32(u), 1.0)
    assert np.all(host(num) == 0)
    np.testing.assert_array_equal(host(out)[:, 0], toks)
    par = np.full((n, 1), -1, np.int32)
    out, _, num = p.verify_accept_tree(t, dev_i32(par), dev_i32(x), dev_f32(u), 1.0)
    assert np.all(host(num) == 0)
    np.testing.assert_array_equal(host(out)[:, 0], toks)
