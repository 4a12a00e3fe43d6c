"""The native binding's own checks (CPU only): a caller's result tensor that cannot hold the result, or has a type the
library does not write, is refused before any address is taken.  The tensors here live on the CPU, so a call that gets
past the check in question ends at the next one, which wants device tensors."""
import os

import pytest
import torch

BF16, F32, I8 = torch.bfloat16, torch.float32, torch.int8
B, H, S, D = 2, 4, 6, 64


@pytest.fixture(scope="module")
def sa():
    from paper_2407_07304_amd import build, slimattn
    if not (os.path.exists(slimattn.LIB_PATH) and os.path.exists(slimattn.BINDING_PATH)):
        build.build()
    return slimattn


def z(*shape, dtype=BF16):
    return torch.zeros(shape, dtype=dtype)


def prefill_calls(sa):
    q, k = z(B, H, S, D), z(B, H, S, D)
    return [lambda f=f, **kw: f(q, k, k, 0.1, **kw)
            for f in (sa.slim_attn_prefill, sa.slim_attn_prefill_emit_int8, sa.slim_attn_prefill_two_sweep, sa.slim_attn_prefill_strip)]


@pytest.mark.parametrize("which", range(4))
def test_prefill_results_that_are_refused(sa, which):
    call = prefill_calls(sa)[which]
    for kw in ({"out_dtype": torch.float16}, {"out_dtype": torch.float64}, {"out": z(B, H, S, D, dtype=torch.float16)},
               {"out": z(B, H, S, D, dtype=torch.int16)}):
        with pytest.raises(AssertionError, match="bf16 or fp32"):
            call(**kw)
    default = torch.get_default_dtype()
    try:
        torch.set_default_dtype(torch.float64)
        with pytest.raises(AssertionError, match="bf16 or fp32"):
            call(out_dtype=None)
    finally:
        torch.set_default_dtype(default)
    with pytest.raises(AssertionError, match="too small"):
        call(out=z(B, H, S - 1, D))
    for out in (z(B, H, S, D), z(B, H, S, D, dtype=F32)):
        with pytest.raises(AssertionError, match="device tensors"):
            call(out=out)


@pytest.mark.parametrize("which", range(1, 4))
def test_prefill_results_of_another_shape_are_taken(sa, which):
    for out in (z(B * H * S * D), z(B, H, S + 3, D, dtype=F32), z(B * H, S, D)):
        with pytest.raises(AssertionError, match="device tensors"):
            prefill_calls(sa)[which](out=out)


def test_decode_results_that_are_refused(sa):
    q, c, s = z(B, H, 1, D), z(B, H, S, D, dtype=I8), z(B, H, S, dtype=F32)
    lens = z(B, dtype=torch.int32)
    for call in (lambda out: sa.slim_attn_decode_int8(q, c, s, c, s, 0.1, out=out, workspace=z(16)),
                 lambda out: sa.slim_attn_decode_int8_varlen(q, c, s, c, s, lens, 0.1, out=out, workspace=z(16))):
        with pytest.raises(AssertionError, match="too small"):
            call(z(B, H, D - 1))
        for out in (z(B, H, 1, D), z(B, H, D), z(B * H * D + 5)):
            with pytest.raises(AssertionError, match="device tensors"):
                call(out)


def test_quantiser_results_that_are_refused(sa):
    x = z(B, H, S, D)
    good_c, good_s = z(B, H, S, D, dtype=I8), z(B, H, S, dtype=F32)
    with pytest.raises(AssertionError, match="codes is too small"):
        sa.kv_quant_int8(x, z(B, H, S - 1, D, dtype=I8), good_s)
    with pytest.raises(AssertionError, match="scales is too small"):
        sa.kv_quant_int8(x, good_c, z(B, H, S - 1, dtype=F32))
    for c, s in ((good_c, good_s), (good_c.view(-1), good_s.view(-1))):
        with pytest.raises(AssertionError, match="device tensors"):
            sa.kv_quant_int8(x, c, s)
