"""Python face of the C-ABI library (``include/slimattn.h``): signatures and defaults.

Tensors are torch tensors on the GPU (PyTorch supplies device memory and the HIP stream);
every step of the path runs in the library's kernels.  The tensors are checked, the results a
caller leaves out allocated and the library called by the native binding ``_slimbind``
(``csrc/binding.cpp``); ``load()`` gives the plain C ABI through ctypes.  There is no CPU
fallback: if a built library is missing, the first call raises.
"""
import ctypes
import importlib
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libslimattn.so")
BINDING_PATH = os.path.join(_HERE, "_slimbind.so")

SLIM_OK = 0
SLIM_BF16, SLIM_F32, SLIM_I8 = 0, 1, 2

_lib = None
_native = None


class SlimError(RuntimeError):
    def __init__(self, status, text):
        super().__init__("slimattn status %d: %s" % (status, text))
        self.status = status


def load():
    """Loads ``libslimattn.so`` and returns its C ABI; raises if it has not been built (``build.build()``)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError("%s is missing: run `python -m paper_2407_07304_amd.build` (hipcc, gfx950) first; "
                              "there is no fallback path" % LIB_PATH)
        lib = ctypes.CDLL(LIB_PATH)
        p, i, f = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
        lib.kv_quant_int8.argtypes = [p, p, p, i, i, i, i, i, i, f, p]
        lib.kv_quant_int8.restype = i
        lib.kv_quant_int8_pair.argtypes = [p, p, p, p, p, p, i, i, i, i, i, i, f, p]
        lib.kv_quant_int8_pair.restype = i
        lib.kv_quant_int8_append.argtypes = [p, p, p, p, i, i, i, i, i, i, f, p]
        lib.kv_quant_int8_append.restype = i
        lib.slim_attn_prefill.argtypes = [p, p, p, p, p, p, i, i, i, i, i, i, f, i, i, p]
        lib.slim_attn_prefill.restype = i
        lib.slim_attn_prefill_block_rows.argtypes = [i, i, i, i, i, i, i, i]
        lib.slim_attn_prefill_block_rows.restype = i
        lib.slim_attn_prefill_emit_int8.argtypes = [p, p, p, p, p, p, p, p, i, i, i, i, i, i, f, i, p]
        lib.slim_attn_prefill_emit_int8.restype = i
        lib.slim_attn_prefill_two_sweep_workspace_bytes.argtypes = [i, i, i, i, i]
        lib.slim_attn_prefill_two_sweep_workspace_bytes.restype = ctypes.c_size_t
        lib.slim_attn_prefill_two_sweep.argtypes = [p, p, p, p, p, ctypes.c_size_t, i, i, i, i, i, i, f, i, p]
        lib.slim_attn_prefill_two_sweep.restype = i
        lib.slim_attn_prefill_strip_max_seq_len.argtypes = []
        lib.slim_attn_prefill_strip_max_seq_len.restype = i
        lib.slim_attn_prefill_strip.argtypes = [p, p, p, p, i, i, i, i, i, i, f, i, p]
        lib.slim_attn_prefill_strip.restype = i
        lib.slim_attn_decode_int8_workspace_bytes.argtypes = [i, i, i, i, i]
        lib.slim_attn_decode_int8_workspace_bytes.restype = ctypes.c_size_t
        lib.slim_attn_decode_int8.argtypes = [p, p, p, p, p, p, p, ctypes.c_size_t, i, i, i, i, i, i, f, p]
        lib.slim_attn_decode_int8.restype = i
        lib.slim_attn_decode_int8_static_max_bytes.argtypes = []
        lib.slim_attn_decode_int8_static_max_bytes.restype = ctypes.c_size_t
        lib.slim_attn_decode_int8_static.argtypes = [p, p, p, p, p, p, i, i, i, i, i, i, f, p]
        lib.slim_attn_decode_int8_static.restype = i
        lib.slim_attn_decode_int8_varlen.argtypes = [p, p, p, p, p, p, p, p, ctypes.c_size_t, i, i, i, i, i, i, f, p]
        lib.slim_attn_decode_int8_varlen.restype = i
        lib.slim_attn_decode_int8_plan.argtypes = [i, i, i, i, i, i, ctypes.POINTER(i), ctypes.POINTER(i)]
        lib.slim_attn_decode_int8_plan.restype = i
        lib.slim_attn_decode_int8_plan_options.argtypes = [i, i, i, i, i, i, ctypes.POINTER(i), ctypes.POINTER(i)]
        lib.slim_attn_decode_int8_plan_options.restype = i
        lib.slim_status_string.argtypes = [i]
        lib.slim_status_string.restype = ctypes.c_char_p
        _lib = lib
    return _lib


def status_string(status: int) -> str:
    return load().slim_status_string(int(status)).decode()


def _check(status):
    if status != SLIM_OK:
        raise SlimError(status, status_string(status))


def _load_native():
    """The native binding; raises like ``load()`` if it has not been built."""
    global _native
    if _native is None:
        load()
        if not os.path.exists(BINDING_PATH):
            raise ImportError("%s is missing: run `python -m paper_2407_07304_amd.build` (hipcc, gfx950) first; "
                              "there is no fallback path" % BINDING_PATH)
        native = importlib.import_module(__package__ + "._slimbind")
        native.set_raise_status(_check)
        _native = native
    return _native


def kv_quant_int8(x, codes=None, scales=None):
    """x [B,Hkv,S,D] bf16 -> (codes int8 [B,Hkv,S,D], scales fp32 [B,Hkv,S])."""
    return (_native or _load_native()).kv_quant(x, codes, scales)


def kv_quant_int8_pair(k, v, k_codes=None, k_scale=None, v_codes=None, v_scale=None):
    """kv_quant_int8 on k and v [B,Hkv,S,D] bf16 in one launch -> (k_codes, k_scale, v_codes, v_scale)."""
    return (_native or _load_native()).kv_quant_pair(k, v, k_codes, k_scale, v_codes, v_scale)


def slim_attn_prefill(q, k, v, softmax_scale, causal=True, k_scale=None, v_scale=None, out=None,
                      out_dtype=torch.bfloat16):
    """q [B,Hq,S,D] bf16; k, v [B,Hkv,S,D] bf16, or int8 with k_scale/v_scale [B,Hkv,S] fp32."""
    return (_native or _load_native()).prefill(q, k, v, softmax_scale, causal, k_scale, v_scale, out, out_dtype)


def slim_attn_decode_int8_workspace_bytes(batch, q_heads, kv_heads, kv_len, head_dim) -> int:
    return int(load().slim_attn_decode_int8_workspace_bytes(batch, q_heads, kv_heads, kv_len, head_dim))


def slim_attn_decode_int8(q, k_codes, k_scale, v_codes, v_scale, softmax_scale, causal=False, out=None,
                          workspace=None):
    """q [B,Hq,1,D] bf16; codes [B,Hkv,T,D] int8; scales [B,Hkv,T] fp32 -> out [B,Hq,1,D] bf16."""
    return (_native or _load_native()).decode(q, k_codes, k_scale, v_codes, v_scale, softmax_scale, causal, out, workspace)


def slim_attn_decode_int8_static_max_bytes() -> int:
    return int(load().slim_attn_decode_int8_static_max_bytes())


def slim_attn_decode_int8_static(q, k_codes, k_scale, v_codes, v_scale, softmax_scale, out, causal=False):
    """slim_attn_decode_int8 with the library's own static scratch array: no workspace argument, and nothing is
    allocated here either, so the caller passes ``out`` [B,Hq,1,D] bf16."""
    return (_native or _load_native()).decode_static(q, k_codes, k_scale, v_codes, v_scale, softmax_scale, out, causal)


def slim_attn_decode_int8_varlen(q, k_codes, k_scale, v_codes, v_scale, kv_lens, softmax_scale, causal=False, out=None,
                                 workspace=None):
    """As slim_attn_decode_int8, sequence b attending to its first kv_lens[b] cached tokens (kv_lens [B] int32,
    on the device)."""
    return (_native or _load_native()).decode_varlen(q, k_codes, k_scale, v_codes, v_scale, softmax_scale, causal, out,
                                                     workspace, kv_lens)


def kv_quant_int8_append(x_new, codes, scales, positions):
    """Quantises x_new [B,Hkv,1,D] bf16 into token positions[b] of the cache (codes [B,Hkv,T,D] int8, scales
    [B,Hkv,T] fp32, both updated in place); positions [B] int32 on the device."""
    return (_native or _load_native()).kv_quant_append(x_new, codes, scales, positions)


def slim_attn_prefill_emit_int8(q, k, v, softmax_scale, causal=True, out=None, out_dtype=torch.bfloat16):
    """Prefill on bf16 K/V that also writes their INT8 cache: returns (out, k_codes, k_scale, v_codes, v_scale)."""
    return (_native or _load_native()).prefill_emit(q, k, v, softmax_scale, causal, out, out_dtype)


def slim_attn_prefill_two_sweep(q, k, v, softmax_scale, causal=True, out=None, out_dtype=torch.bfloat16, workspace=None):
    """The two-sweep comparison variant of the bf16 prefill (row maxima first, then everything else)."""
    return (_native or _load_native()).prefill_two_sweep(q, k, v, softmax_scale, causal, out, out_dtype, workspace)


def slim_attn_prefill_strip_max_seq_len() -> int:
    return int(load().slim_attn_prefill_strip_max_seq_len())


def slim_attn_prefill_strip(q, k, v, softmax_scale, causal=True, out=None, out_dtype=torch.bfloat16):
    """The comparison variant of the bf16 prefill that keeps a row block's whole score strip on chip."""
    return (_native or _load_native()).prefill_strip(q, k, v, softmax_scale, causal, out, out_dtype)
