"""The GEMM's tile kinds at their edges: K loops shorter than, as long as and
longer than the pipeline (both parities of the alternating schedule), ragged
last tiles, K splits, operand rows too far apart for 32-bit offsets.

Against the oracle on sampled outputs, with the tolerance and the accumulation
bound of test_gpu_gemm.py; the bf16 output must be the RNE of the fp32 one."""

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import accept as oa, gemm as og, quantize as oq
from tests import gemm_shapes
from tests.gpu_util import dev_f32, dev_u8, host, host_bf16_bits, need_gpu, say
from tests.test_gpu_gemm import TOL, _check_bound, _f32_to_bf16_bits, _sample

pytestmark = pytest.mark.gpu

SHAPES = (
    [(250, 60000, 128 * k) for k in (1, 2, 3, 6)]        # 256x256, 2 stages
    + [(1990, 6100, 128 * k) for k in (1, 3, 4)]         # 160x384, 2 stages
    + [(319, 28000, 128 * k) for k in (1, 2, 3, 4, 7)]   # 160x224, 3 stages
    + [(127, 60000, 128 * k) for k in (2, 4, 5)]         # 128x256, 3 stages
    + [(2000, 4090, 128 * k) for k in (1, 5, 9)]         # 256x128, 3 stages, grouped M-tiles
    + [(159, 28000, 640), (310, 14300, 640)]             # 160x128, 4 stages
    + [(127, 28000, 128 * k) for k in (2, 4, 5)]         # 128x128, 4 stages
    + [(630, 4000, 1280), (159, 14300, 512)]             # 160x64
    + [(200, 6100, 640), (33, 28000, 768)]               # 64x128
    + [(75, 28000, 1152), (7, 60000, 256)]               # 80x128, 3 stages
    + [(79, 8200, 768), (79, 28000, 128)]                # 80x64
    + [(33, 8200, 256), (61, 8200, 640)]                 # 64x64
    + [(5, 5000, 256), (1, 9, 128)]                      # 32x64
    + [(640, 4090, 14336), (1000, 4090, 14336), (320, 4090, 14336), (512, 4090, 14336),     # K split: 160x128 in 2,
       (300, 4096, 8192), (1000, 500, 8192), (7, 100, 2560), (80, 6144, 4096)]              # 256x128, 160x128 in 4 ...
)


def _codes(M, N, K):
    return (wl.fp8_code_bytes(M, K, seed=M + K), wl.fp8_code_bytes(N, K, seed=N + K + 1),
            wl.uniform_scales(M, seed=M), wl.uniform_scales(N, seed=N + 1))


def _check(y32, y16_bits, a, sa, w, sw):
    rows, cols = _sample(a.shape[0], 24, 3), _sample(w.shape[0], 48, 4)
    y_ref = og.gemm(a[rows], sa[rows], w[cols], sw[cols])
    assert np.max(np.abs(y32[np.ix_(rows, cols)] - y_ref)) <= TOL * np.max(np.abs(y_ref))
    _check_bound(y32, y_ref, a, sa, w, sw, rows, cols)
    np.testing.assert_array_equal(y16_bits, _f32_to_bf16_bits(y32))


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_tile_edges(M, N, K):
    p = need_gpu()
    say(f"gemm tile M={M} N={N} K={K} ws={p.gemm_workspace_bytes(M, N, K)}")
    a, w, sa, sw = _codes(M, N, K)
    ws = torch.zeros((max(16, p.gemm_workspace_bytes(M, N, K)),), dtype=torch.uint8, device="cuda")
    args = (dev_u8(a), dev_f32(sa), dev_u8(w), dev_f32(sw))
    ld = (N + 7) // 8 * 8 + 8
    outs = []
    for dt in (torch.float32, torch.bfloat16):
        out = torch.full((M, ld), -7.0, dtype=dt, device="cuda")
        p.gemm(*args, out=out[:, :N], workspace=ws)
        assert torch.all(out[:, N:] == -7.0)
        assert torch.all(ws[:16384] == 0)
        outs.append(out[:, :N])
    _check(host(outs[0]), host_bf16_bits(outs[1]), a, sa, w, sw)


def test_split_shape_without_a_workspace_runs_unsplit():
    """Where the workspace is optional, a call without one gives the same sums
    in another order: within the fp32 rounding of K accumulations."""
    p = need_gpu()
    M, N, K = 640, 4096, 14336
    assert p.gemm_workspace_bytes(M, N, K) > 0
    a, w, sa, sw = _codes(M, N, K)
    args = (dev_u8(a), dev_f32(sa), dev_u8(w), dev_f32(sw))
    ws = torch.zeros((p.gemm_workspace_bytes(M, N, K),), dtype=torch.uint8, device="cuda")
    y_split = host(p.gemm(*args, out_dtype=torch.float32, workspace=ws)).astype(np.float64)
    y_plain = host(p.gemm(*args, out_dtype=torch.float32)).astype(np.float64)
    assert np.max(np.abs(y_split - y_plain)) <= TOL * np.max(np.abs(y_plain))


@pytest.mark.parametrize("sa_mul,sw_mul", [(2.0 ** -66, 2.0 ** -58), (2.0 ** 66, 2.0 ** 64)])
def test_bf16_rounding_at_the_ends_of_the_range(sa_mul, sw_mul):
    """Subnormal and overflowing outputs: the hardware conversion to bf16 is
    the RNE of the fp32 output there too."""
    p = need_gpu()
    M, N, K = 64, 512, 256
    a, w, sa, sw = _codes(M, N, K)
    args = (dev_u8(a), dev_f32(sa * np.float32(sa_mul)), dev_u8(w), dev_f32(sw * np.float32(sw_mul)))
    y32 = host(p.gemm(*args, out_dtype=torch.float32))
    y16 = host_bf16_bits(p.gemm(*args))
    special = np.isinf(y32) | ((np.abs(y32) < 2.0 ** -126) & (y32 != 0))
    assert special.any() and not special.all()
    np.testing.assert_array_equal(y16, _f32_to_bf16_bits(y32))


def _far(t, ld):
    """The rows of t at a stride of ld bytes."""
    big = torch.empty(((t.shape[0] - 1) * ld + t.shape[1],), dtype=torch.uint8, device="cuda")
    v = big.as_strided(t.shape, (ld, 1))
    v.copy_(t)
    return v


@pytest.mark.parametrize("lda,ldw", [(140_000_000, 0), (0, 70_000_000)])
def test_rows_of_a_tile_past_4gib(lda, ldw):
    """Every epilogue on operands whose rows of one tile span more than 4 GiB,
    against the same call on packed operands (the kernels walk K alike)."""
    p = need_gpu()
    M, N, K = 33, 128, 512
    say(f"far rows lda={lda} ldw={ldw}")
    a, w, sa, sw = _codes(M, N, K)
    da, dw, dsa, dsw = dev_u8(a), dev_u8(w), dev_f32(sa), dev_f32(sw)
    fa = _far(da, lda) if lda else da
    fw = _far(dw, ldw) if ldw else dw
    y = p.gemm(fa, dsa, fw, dsw, out_dtype=torch.float32)
    _check(host(y), host_bf16_bits(p.gemm(fa, dsa, fw, dsw)), a, sa, w, sw)
    assert torch.equal(p.gemm_silu_mul(fa, dsa, fw, dsw), p.gemm_silu_mul(da, dsa, dw, dsw))
    for T in (0.7, 0.0):
        lf, sf = p.gemm_logit_stats(fa, dsa, fw, dsw, T)
        lp, sp = p.gemm_logit_stats(da, dsa, dw, dsw, T)
        assert torch.equal(lf.contiguous().view(torch.int16), lp.contiguous().view(torch.int16))
        if T == 0.0:
            assert torch.equal(sf.contiguous().view(torch.int32), sp.contiguous().view(torch.int32))
        else:
            assert torch.equal(sf[..., 0], sp[..., 0])
            torch.testing.assert_close(sf[..., 1], sp[..., 1], rtol=2e-5, atol=0)


@pytest.mark.parametrize("M,V,K,T", [
    (250, 30000, 384, 0.7), (159, 60000, 768, 0.7), (79, 60000, 384, 0.0), (79, 28000, 768, 0.7), (7, 100, 384, 0.0),
])
def test_statistics_of_the_stored_logits(M, V, K, T):
    """The statistics epilogue of each tile kind that has one describes the
    logits it stores, which are the unsplit plain GEMM's."""
    p = need_gpu()
    say(f"logit stats M={M} V={V} K={K} T={T}")
    a, w, sa, sw = _codes(M, V, K)
    args = (dev_u8(a), dev_f32(sa * np.float32(0.02)), dev_u8(w), dev_f32(sw))
    z, st = p.gemm_logit_stats(*args, T)
    assert torch.equal(z.contiguous().view(torch.int16), p.gemm(*args).contiguous().view(torch.int16))
    st = host(st)
    zf = oq.bf16_to_f32(host_bf16_bits(z))
    if T == 0.0:
        best = np.max(st[..., 0], axis=1)
        idx = np.where(st[..., 0] == best[:, None], st[..., 1].copy().view(np.int32), np.iinfo(np.int32).max).min(axis=1)
        np.testing.assert_array_equal(best, zf.max(axis=1))
        np.testing.assert_array_equal(idx, zf.argmax(axis=1))
        return
    zmax, Z = oa.softmax_normalizer(host_bf16_bits(z), T)
    Mg = st[..., 0].max(axis=1)
    Zg = np.sum(st[..., 1].astype(np.float64) * np.exp2(st[..., 0].astype(np.float64) - Mg[:, None]), axis=1)
    c2 = np.float32(1.4426950408889634 / T)
    np.testing.assert_array_equal(Mg, (zmax * np.float64(c2)).astype(np.float32))
    np.testing.assert_allclose(Zg, Z, rtol=2e-5)


@pytest.mark.parametrize("M,V,K", [(33, 32896, 8192), (59, 38296, 6656)])
def test_stored_logits_are_the_unsplit_plain_ones_where_the_tiles_differ(M, V, K):
    """Wide shapes whose plain GEMM may split K: a call without a workspace
    does not, and sums K in the order of the statistics GEMM, whatever tile
    each takes."""
    p = need_gpu()
    say(f"logits M={M} V={V} K={K}")
    a, w, sa, sw = _codes(M, V, K)
    args = (dev_u8(a), dev_f32(sa * np.float32(0.02)), dev_u8(w), dev_f32(sw))
    z, _ = p.gemm_logit_stats(*args, 0.7)
    assert torch.equal(z.contiguous().view(torch.int16), p.gemm(*args).contiguous().view(torch.int16))


@pytest.mark.parametrize("M,N,K", [(33, 28672, 512), (33, 12352, 1024)])
def test_far_rows_of_staggered_shapes(M, N, K):
    """Wide shapes that start K at staggered steps: rows of one tile more than
    4 GiB apart give the bits that packed rows give."""
    p = need_gpu()
    say(f"far rows staggered M={M} N={N} K={K}")
    a, w, sa, sw = _codes(M, N, K)
    da, dw, dsa, dsw = dev_u8(a), dev_u8(w), dev_f32(sa * np.float32(0.02)), dev_f32(sw)
    fa = _far(da, 140_000_000)
    assert torch.equal(p.gemm(fa, dsa, dw, dsw, out_dtype=torch.float32), p.gemm(da, dsa, dw, dsw, out_dtype=torch.float32))
    lf, sf = p.gemm_logit_stats(fa, dsa, dw, dsw, 0.0)
    lp, sp = p.gemm_logit_stats(da, dsa, dw, dsw, 0.0)
    assert torch.equal(lf.contiguous().view(torch.int16), lp.contiguous().view(torch.int16))
    assert torch.equal(sf.contiguous().view(torch.int32), sp.contiguous().view(torch.int32))


@pytest.mark.parametrize("T", [0.7, 0.0])
def test_far_rows_of_the_wide_lm_head_tile(T):
    """A shape on the 160x384 tile whose interface does not limit the strides:
    activation rows further apart than that tile addresses."""
    p = need_gpu()
    M, V, K, lda = 71, 66200, 512, 28_000_000
    say(f"far LM head M={M} V={V} K={K} T={T}")
    a, w, sa, sw = _codes(M, V, K)
    da, dw, dsa, dsw = dev_u8(a), dev_u8(w), dev_f32(sa * np.float32(0.02)), dev_f32(sw)
    lf, sf = p.gemm_logit_stats(_far(da, lda), dsa, dw, dsw, T)
    lp, sp = p.gemm_logit_stats(da, dsa, dw, dsw, T)
    assert torch.equal(lf.contiguous().view(torch.int16), lp.contiguous().view(torch.int16))
    assert torch.equal(sf[..., 0], sp[..., 0])
    if T == 0.0:
        assert torch.equal(sf.contiguous().view(torch.int32), sp.contiguous().view(torch.int32))
    else:
        torch.testing.assert_close(sf[..., 1], sp[..., 1], rtol=2e-5, atol=0)


@pytest.mark.parametrize("M,V,K", [shape for shape, _ in gemm_shapes.STATS])
@pytest.mark.parametrize("T", [0.7, 0.0])
def test_statistics_of_every_tile(M, V, K, T):
    test_statistics_of_the_stored_logits(M, V, K, T)


@pytest.mark.parametrize("M,N,K", [shape for shape, _ in gemm_shapes.SPLIT])
def test_split_tile_edges(M, N, K):
    test_tile_edges(M, N, K)
