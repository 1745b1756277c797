"""The inverse-CDF search where rounding decides: the token it emits has mass."""

import numpy as np
import pytest

import workloads as wl
from tests.gpu_util import dev_bf16, dev_f32, dev_i32, host, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("toks,z", [
    ((5, 4096, 8192, 12388), (0, -53, -53, 0)),      # one in each 4096-logit part of a chunk: the scan of part totals
    ((5, 70, 130, 12388), (-53, -53, 0, 0)),         # in three of a part's 64-logit ranges: the scan within a part
    ((0, 1, 2, 12388), (-53, -53, 0, 0)),            # three elements of one range: the scan within a range
])
@pytest.mark.parametrize("V", [16384, 16384 * 17])   # one batch of chunks, two
def test_target_in_a_rounding_gap(V, toks, z):
    """Four tokens have mass: 1/2 twice and 2^-54 twice, the total 1.  With
    u = 1/2 the target is 1/2.  Adding 1/2 and then the two small masses, one
    by one, loses both (ties, to even); adding the small ones to each other
    first does not.  So sums of the same masses in different orders differ in
    the last bit, and the target lies between them.  No token without mass may
    be taken for it."""
    p = need_gpu()
    say(f"search gap V={V} {toks}")
    T = float(np.float32(1.4426950408889634))               # log2(e) / T rounds to 1: p = 2^z / Z, exactly
    logits = np.full((1, 2, V), -np.inf, np.float32)
    logits[:, :, list(toks)] = z
    zt = dev_bf16(wl.bf16_bits_from_f32(logits))
    top = toks[z.index(0)]
    out, num = p.verify_accept(zt, None, dev_i32([[top]]), dev_f32([[0.0, 0.5]]), T)
    say(f"  chain {host(out)} {host(num)}")
    assert host(num)[0] == 1 and host(out)[0, 1] in toks     # the draft accepted, then the bonus token
    out, _, num = p.verify_accept_tree(zt, dev_i32([[-1]]), dev_i32([[V + 1]]), dev_f32([[0.0, 0.5]]), T)
    say(f"  tree {host(out)} {host(num)}")
    assert host(num)[0] == 0 and host(out)[0, 0] in toks
