"""Helpers shared by the GPU parity tests: host bits <-> device tensors, error metrics."""
import ctypes

import numpy as np
import torch

MAX_ABS = 2e-2    # bf16 attention output against the fp64 oracle
MEAN_ABS = 2e-3


def dev_bf16(bits: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)


def dev(a: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host_f64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float64).cpu().numpy()


def assert_form(sa, rows, B, Hq, Hkv, S, D, causal, kv_int8, out_f32):
    """The call takes the prefill's form with row blocks of `rows` rows: a test of one form must not end up in another."""
    got = sa.load().slim_attn_prefill_block_rows(B, Hq, Hkv, S, D, int(causal), sa.SLIM_I8 if kv_int8 else sa.SLIM_BF16,
                                                 sa.SLIM_F32 if out_f32 else sa.SLIM_BF16)
    assert got == rows, "row blocks of %d rows, the test is of those of %d" % (got, rows)


def assert_plan(sa, plan, B, Hq, Hkv, T, D, by_length=None):
    """A decode with lengths of its own takes this plan: (waves per workgroup, workgroups per row), and deals its rows by length or not."""
    w, n = ctypes.c_int(), ctypes.c_int()
    assert sa.load().slim_attn_decode_int8_plan(B, Hq, Hkv, T, D, 1, ctypes.byref(w), ctypes.byref(n)) == 0
    assert (w.value, n.value) == plan, "plan %s, the test is of %s" % ((w.value, n.value), plan)
    if by_length is not None:
        assert sa.load().slim_attn_decode_int8_plan_options(B, Hq, Hkv, T, D, 1, ctypes.byref(w), ctypes.byref(n)) == 0
        assert w.value == by_length, "rows dealt by length: %d" % w.value


def check_close(got: np.ndarray, want: np.ndarray, what=""):
    err = np.abs(got - want)
    assert np.isfinite(got).all(), "%s: non-finite output" % what
    mx, mean = float(err.max()), float(err.mean())
    assert mx <= MAX_ABS and mean <= MEAN_ABS, "%s: max-abs %.3e (limit %.0e), mean-abs %.3e (limit %.0e)" % (
        what, mx, MAX_ABS, mean, MEAN_ABS)
    return mx, mean
