"""The native argument marshalling: what it refuses, and that outputs the
caller gives come back as the same objects."""

import fractions

import pytest
import torch

import paper_2606_18502_amd as p
from tests.gpu_util import need_gpu


def test_cpu_tensors_and_non_tensors_are_refused():
    x = torch.zeros((8, 512), dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="x must be a CUDA"):
        p.quantize(x)
    with pytest.raises(ValueError, match="x must be a CUDA"):
        p.quantize([1.0])
    with pytest.raises(ValueError, match="parents must be a CUDA"):
        p.tree_attention_mask(torch.zeros((2, 4), dtype=torch.int32))
    with pytest.raises(TypeError):
        p.quantize()


@pytest.mark.gpu
def test_refused_arguments():
    need_gpu()
    d = dict(device="cuda")
    x = torch.zeros((8, 512), dtype=torch.bfloat16, **d)
    q, s = p.quantize(x)
    w, sw = p.quantize(torch.ones((64, 512), dtype=torch.bfloat16, **d))
    bad = [
        (lambda: p.quantize(x.float()), "x must have dtype torch.bfloat16, got torch.float32"),
        (lambda: p.quantize(x.t()), "x must be a 2-D row-major view"),
        (lambda: p.quantize(x, out=torch.zeros((8, 512), dtype=torch.int8, **d)), "out must have dtype torch.uint8"),
        (lambda: p.calibrate(x, torch.zeros(2, **d)), "one fp32 value"),
        (lambda: p.gemm(q, s, w[:, :256], sw), "disagree on K"),
        (lambda: p.gemm(q, s[:4], w, sw), "sa must hold M"),
        (lambda: p.gemm(q, s, w, sw, out_dtype=torch.float16), "out must be bf16 or fp32"),
        (lambda: p.gemm_silu_mul(q, s, w[:63], sw), "w must be"),
        (lambda: p.gemm_logit_stats(q, s, w, sw, 0.7, stats=torch.zeros((8, 1), **d)), "stats must be"),
        (lambda: p.verify_accept(x.view(2, 4, 512), None, torch.zeros((2, 2), dtype=torch.int32, **d), None, 0.0),
         "draft_tokens must be contiguous"),
        (lambda: p.verify_accept_tree(x.view(2, 4, 512), torch.zeros((2, 3), dtype=torch.int32, **d),
                                      torch.zeros((3, 2), dtype=torch.int32, **d).t(), None, 0.0), "tokens must be"),
    ]
    for call, message in bad:
        with pytest.raises(ValueError, match=message):
            call()
    with pytest.raises(p.SpecError) as e:
        p.quantize(torch.zeros((8, 12), dtype=torch.bfloat16, **d))
    assert e.value.status == 3
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_given_outputs_come_back_and_streams_are_followed():
    need_gpu()
    x = torch.randn((8, 4096), device="cuda").to(torch.bfloat16)
    w, sw = p.quantize(torch.randn((1024, 4096), device="cuda").to(torch.bfloat16))
    out, scales = torch.empty((8, 4096), dtype=torch.uint8, device="cuda"), torch.empty(8, device="cuda")
    q, s = p.quantize(x, out=out, scales=scales)
    assert q is out and s is scales
    y = torch.empty((8, 1024), dtype=torch.bfloat16, device="cuda")
    assert p.gemm(q, s, w, sw, out=y) is y                       # (a workspace is made for the call)
    assert p.gemm(q, s, w, sw, workspace=torch.zeros(16, dtype=torch.uint8, device="cuda")).shape == (8, 1024)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):                   # a launch on any other stream would not be captured
            p.quantize(x, out=out, scales=scales)
    ref_q, ref_s = out.clone(), scales.clone()
    out.zero_()
    scales.zero_()
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref_q) and torch.equal(scales, ref_s)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(320, 4096, 4096), (80, 6144, 4096)])
def test_an_unsplit_gemm_allocates_nothing_but_its_output(M, N, K):
    """Decode-sized projections whose K is not split: no workspace is made."""
    need_gpu()
    q, s = p.quantize(torch.randn((M, K), device="cuda").to(torch.bfloat16))
    w, sw = p.quantize(torch.randn((N, K), device="cuda").to(torch.bfloat16))
    out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    made = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]
    before = made()
    p.gemm(q, s, w, sw, out=out)
    assert made() == before
    y = p.gemm(q, s, w, sw)
    assert made() == before + 1 and torch.equal(y, out)


@pytest.mark.gpu
def test_a_temperature_is_whatever_float_takes():
    need_gpu()
    d = dict(device="cuda")
    z = torch.randn((2, 3, 512), **d).to(torch.bfloat16)
    x, u = torch.zeros((2, 2), dtype=torch.int32, **d), torch.rand((2, 3), **d)
    want = p.verify_accept(z, None, x, u, 0.75)
    for T in ("0.75", fractions.Fraction(3, 4), torch.tensor(0.75), torch.full((1,), 0.75, **d)):
        got = p.verify_accept(z, None, x, u, T)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    with pytest.raises(ValueError):
        p.verify_accept(z, None, x, u, "warm")
    with pytest.raises(TypeError):
        p.verify_accept(z, None, x, u, None)
