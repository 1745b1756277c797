"""Torch-facing wrappers of the C ABI.

Signatures only: the arguments are checked and marshalled by the native module
built from csrc/torch_bind.cpp, and every step of the verify path runs in the
HIP kernels of libspecfp8.so; torch provides device memory and the current
stream.  There is no CPU or torch fallback: without the built library every
call raises.
"""

from __future__ import annotations

from typing import Optional, Tuple

import torch

from . import _lib

_bind = None      # the native marshalling module, once loaded


def _load_bind():
    """Load the native marshalling module (and with it libspecfp8.so); raises if it has not been built."""
    global _bind
    _lib.load()
    from . import _torch_bind
    _torch_bind.init(_lib.SpecError)
    _bind = _torch_bind
    return _bind


def quantize(x: torch.Tensor, per_tensor_scale: Optional[torch.Tensor] = None, silu_mul: bool = False,
             out: Optional[torch.Tensor] = None, scales: Optional[torch.Tensor] = None
             ) -> Tuple[torch.Tensor, torch.Tensor]:
    """E4M3 row quantization of bf16 rows (spec_fp8_quantize).

    x: bf16 [rows, cols] (or [rows, 2*cols] with silu_mul).  Dynamic per-row
    scales unless `per_tensor_scale` (fp32 [1]) is given.
    Returns (codes uint8 [rows, cols], scales fp32 [rows] or the given [1]).
    """
    return (_bind or _load_bind()).quantize(x, per_tensor_scale, silu_mul, out, scales)


def calibrate(x: torch.Tensor, running_scale: torch.Tensor, silu_mul: bool = False) -> torch.Tensor:
    """Static min-max calibration step (spec_fp8_quantize, SPEC_SCALE_CALIBRATE).

    running_scale: fp32 [1], updated in place to max(running_scale, scale of
    the largest |x|); start it at 0 and pass every calibration batch.
    """
    return (_bind or _load_bind()).calibrate(x, running_scale, silu_mul)


def silu_mul(x: torch.Tensor, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """h = bf16(silu(gate) * up) for x = [gate | up] bf16 [rows, 2*cols] (spec_silu_mul_bf16)."""
    return (_bind or _load_bind()).silu_mul(x, out)


def clip_count(x: torch.Tensor, scale: torch.Tensor, count: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Values of bf16 rows x that the static per-tensor scale clips (spec_fp8_clip_count):
    |fl32(x * fl32(1/scale))| > 448.  Accumulates into `count` (int64 [1]
    holding the uint64 count; a new zeroed counter if None) and returns it."""
    return (_bind or _load_bind()).clip_count(x, scale, count)


def kv_cache_write(k: torch.Tensor, v: torch.Tensor, slot_mapping: torch.Tensor, k_cache: torch.Tensor,
                   v_cache: torch.Tensor, k_scale: torch.Tensor, v_scale: torch.Tensor,
                   per_tensor: bool = False) -> None:
    """Quantize new keys and values to E4M3 into the FP8 KV cache (spec_fp8_kv_cache_write).

    k, v: bf16 [T, H, D] views (unit stride over D and heads packed side by
    side, e.g. column blocks of the QKV output viewed as [T, H, D]);
    slot_mapping: int64 [T] (negative = skip); k_cache, v_cache: uint8
    [num_slots, H, D] contiguous (a paged [blocks, block_size, H, D] cache
    viewed flat).  Per-row scales: k_scale, v_scale fp32 [num_slots, H],
    written at the stored slots; per_tensor=True: fp32 [1], read.
    """
    (_bind or _load_bind()).kv_cache_write(k, v, slot_mapping, k_cache, v_cache, k_scale, v_scale, per_tensor)


def gemm_workspace_bytes(M: int, N: int, K: int) -> int:
    return int(_lib.load().spec_fp8_gemm_workspace_bytes(M, N, K))


def gemm(a: torch.Tensor, sa: torch.Tensor, w: torch.Tensor, sw: torch.Tensor,
         out_dtype: torch.dtype = torch.bfloat16, out: Optional[torch.Tensor] = None,
         workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Y = dec(A) dec(W)^T * sa * sw (spec_fp8_gemm).

    a: uint8 E4M3 [M,K]; sa: fp32 [M] (per token) or [1] (per tensor);
    w: uint8 E4M3 [N,K]; sw: fp32 [N] (per channel) or [1].
    workspace: gemm_workspace_bytes(M, N, K) bytes on the GPU, 16-byte aligned,
    zero-filled once and then kept for all calls of a stream.  Bring one: without it
    (or with one too small) a decode-sized projection that splits K gets a new
    zero-filled one in every call, and any other shape runs with K unsplit, which is
    slower and sums in another order.
    """
    f32 = True if out_dtype is torch.float32 else (False if out_dtype is torch.bfloat16 else None)
    return (_bind or _load_bind()).gemm(a, sa, w, sw, f32, out, workspace)


def gemm_silu_mul(a: torch.Tensor, sa: torch.Tensor, w: torch.Tensor, sw: torch.Tensor,
                  out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """h = bf16(silu(gate) * up) of the fused gate|up projection (spec_fp8_gemm_silu_mul).

    a: uint8 E4M3 [M,K]; w: uint8 E4M3 [2I,K] (gate rows, then up rows);
    sa, sw as for gemm.  Returns h bf16 [M,I].
    """
    return (_bind or _load_bind()).gemm_silu_mul(a, sa, w, sw, out)


def logit_stats_count(M: int, V: int, K: int) -> int:
    return int(_lib.load().spec_logit_stats_count(M, V, K))


def gemm_logit_stats(a: torch.Tensor, sa: torch.Tensor, w: torch.Tensor, sw: torch.Tensor, temperature: float,
                     out: Optional[torch.Tensor] = None, stats: Optional[torch.Tensor] = None
                     ) -> Tuple[torch.Tensor, torch.Tensor]:
    """LM-head GEMM with the acceptance statistics in its epilogue (spec_fp8_gemm_logit_stats).

    a: uint8 E4M3 [M,K] (final hidden states of the verify rows); w: uint8 E4M3 [V,K];
    sa, sw as for gemm.  Returns (logits bf16 [M,V], stats fp32 [M,G,2]) with
    G = logit_stats_count(M, V, K) column groups per row.
    """
    return (_bind or _load_bind()).gemm_logit_stats(a, sa, w, sw, temperature, out, stats)


def accept_workspace_bytes(B: int, k: int, V: int) -> int:
    return int(_lib.load().spec_verify_accept_workspace_bytes(B, k, V))


def verify_accept(target_logits: torch.Tensor, draft_logits: Optional[torch.Tensor], draft_tokens: torch.Tensor,
                  uniforms: Optional[torch.Tensor], temperature: float,
                  workspace: Optional[torch.Tensor] = None,
                  out_tokens: Optional[torch.Tensor] = None, num_accepted: Optional[torch.Tensor] = None,
                  target_stats: Optional[torch.Tensor] = None) -> Tuple[torch.Tensor, torch.Tensor]:
    """Greedy (T=0) or speculative-sampling (T>0) acceptance (spec_verify_accept, or
    spec_verify_accept_stats when target_stats from gemm_logit_stats are given).

    target_logits bf16 [B,k+1,V]; draft_logits bf16 [B,k,V] or None;
    draft_tokens int32 [B,k]; uniforms fp32 [B,k+1] (T>0);
    target_stats fp32 [B*(k+1), G, 2] (pairs) or None.
    Returns (out_tokens int32 [B,k+1] (-1 padded), num_accepted int32 [B]).
    """
    return (_bind or _load_bind()).verify_accept(target_logits, draft_logits, draft_tokens, uniforms, temperature,
                                                 workspace, out_tokens, num_accepted, target_stats)


def verify_accept_noalloc(target_logits: torch.Tensor, draft_logits: Optional[torch.Tensor],
                          draft_tokens: torch.Tensor, uniforms: Optional[torch.Tensor], temperature: float,
                          out_tokens: torch.Tensor, num_accepted: torch.Tensor) -> Tuple[torch.Tensor, torch.Tensor]:
    """verify_accept through spec_verify_accept_noalloc: no workspace, the
    library's fixed device scratch instead, and no allocation here either (the
    outputs are the caller's).  Same arguments and results as verify_accept."""
    return (_bind or _load_bind()).verify_accept_noalloc(target_logits, draft_logits, draft_tokens, uniforms,
                                                         temperature, out_tokens, num_accepted)


def accept_tree_workspace_bytes(B: int, N: int, V: int) -> int:
    return int(_lib.load().spec_verify_accept_tree_workspace_bytes(B, N, V))


def verify_accept_tree(target_logits: torch.Tensor, parents: torch.Tensor, tokens: torch.Tensor,
                       uniforms: Optional[torch.Tensor], temperature: float,
                       workspace: Optional[torch.Tensor] = None, out_tokens: Optional[torch.Tensor] = None,
                       accepted_nodes: Optional[torch.Tensor] = None, num_accepted: Optional[torch.Tensor] = None
                       ) -> Tuple[torch.Tensor, torch.Tensor, torch.Tensor]:
    """Token-tree acceptance (spec_verify_accept_tree).

    target_logits bf16 [B,N+1,V]; parents, tokens int32 [B,N]; uniforms fp32 [B,N+1] (T>0).
    Returns (out_tokens int32 [B,N+1], accepted_nodes int32 [B,N], num_accepted int32 [B]).
    """
    return (_bind or _load_bind()).verify_accept_tree(target_logits, parents, tokens, uniforms, temperature, workspace,
                                                      out_tokens, accepted_nodes, num_accepted)


def tree_attention_mask(parents: torch.Tensor, mask: Optional[torch.Tensor] = None,
                        depth: Optional[torch.Tensor] = None) -> Tuple[torch.Tensor, torch.Tensor]:
    """Ancestor-or-self masks and depths of B drafted trees (spec_tree_attention_mask).

    parents: int32 [B, N] (N <= 64).  Returns (mask int64 [B, N] holding the
    uint64 bit patterns, bit j = node j; depth int32 [B, N]).
    """
    return (_bind or _load_bind()).tree_attention_mask(parents, mask, depth)
