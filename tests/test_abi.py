"""CPU-only checks of the C ABI: the library loads, exports every declared symbol, and
rejects bad arguments before anything is launched (no GPU is touched)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "slimattn.h")


@pytest.fixture(scope="module")
def lib():
    from paper_2407_07304_amd import slimattn, build
    if not os.path.exists(slimattn.LIB_PATH):
        build.build()
    return slimattn.load()


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b([a-z_0-9]+)\s*\(", text)) - {"defined"})


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert {"kv_quant_int8", "slim_attn_prefill", "slim_attn_decode_int8", "slim_attn_decode_int8_varlen",
            "kv_quant_int8_append", "kv_quant_int8_pair", "slim_attn_prefill_emit_int8", "slim_attn_decode_int8_workspace_bytes", "slim_status_string",
            "slim_attn_prefill_two_sweep", "slim_attn_prefill_two_sweep_workspace_bytes", "slim_attn_prefill_strip",
            "slim_attn_prefill_strip_max_seq_len", "slim_attn_decode_int8_static", "slim_attn_decode_int8_static_max_bytes"} <= set(names)
    for n in names:
        assert getattr(lib, n) is not None


def test_status_strings(lib):
    seen = set()
    for code in range(7):
        s = lib.slim_status_string(code).decode()
        assert s and s not in seen
        seen.add(s)
    assert lib.slim_status_string(99).decode() == "unknown status"


P = ctypes.c_void_p
A = 0x1000   # a fake, aligned, never dereferenced address: every case below fails validation first


def prefill(lib, q=A, k=A, v=A, ks=None, vs=None, out=A, B=1, Hq=2, Hkv=2, S=16, D=128, causal=1, scale=0.1,
            kvd=0, od=0):
    return lib.slim_attn_prefill(P(q), P(k), P(v), P(ks), P(vs), P(out), B, Hq, Hkv, S, D, causal, scale, kvd, od, None)


def test_prefill_rejects_bad_arguments(lib):
    NULL, SHAPE, UNSUP, ALIGN = 1, 2, 3, 4
    assert prefill(lib, q=None) == NULL
    assert prefill(lib, out=None) == NULL
    assert prefill(lib, kvd=2) == NULL                 # INT8 without scales
    assert prefill(lib, ks=A, vs=A) == NULL            # bf16 with scales
    assert prefill(lib, kvd=1) == UNSUP and prefill(lib, od=2) == UNSUP
    assert prefill(lib, D=96) == UNSUP
    assert prefill(lib, S=0) == SHAPE and prefill(lib, B=-1) == SHAPE
    assert prefill(lib, Hq=3, Hkv=2) == SHAPE
    assert prefill(lib, causal=2) == SHAPE
    assert prefill(lib, scale=0.0) == SHAPE and prefill(lib, scale=float("nan")) == SHAPE
    assert prefill(lib, scale=float("inf")) == SHAPE
    assert prefill(lib, k=A + 8) == ALIGN
    assert prefill(lib, kvd=2, ks=A + 4, vs=A) == ALIGN
    assert prefill(lib, B=65536, Hq=65536, Hkv=65536, S=4096) == SHAPE   # not indexable


def test_quant_rejects_bad_arguments(lib):
    f = lib.kv_quant_int8
    assert f(P(None), P(A), P(A), 1, 1, 1, 4, 128, 0, 1.0, None) == 1
    assert f(P(A), P(A), P(A), 1, 1, 1, 0, 128, 0, 1.0, None) == 2
    assert f(P(A), P(A), P(A), 1, 1, 1, 4, 100, 0, 1.0, None) == 3
    assert f(P(A), P(A + 1), P(A), 1, 1, 1, 4, 128, 0, 1.0, None) == 4
    # the scalars of the common tail that the quantiser does not use are still checked for range
    assert f(P(A), P(A), P(A), 1, 0, 1, 4, 128, 0, 1.0, None) == 2
    assert f(P(A), P(A), P(A), 1, 3, 2, 4, 128, 0, 1.0, None) == 2
    assert f(P(A), P(A), P(A), 1, 1, 1, 4, 128, 2, 1.0, None) == 2
    assert f(P(A), P(A), P(A), 1, 1, 1, 4, 128, 0, 0.0, None) == 2
    assert f(P(A), P(A), P(A), 1, 1, 1, 4, 128, 0, float("nan"), None) == 2


def test_decode_rejects_bad_arguments_and_reports_workspace(lib):
    ws = lib.slim_attn_decode_int8_workspace_bytes
    per_row = lambda D: (D + 2) * 4   # one (max, sum, accumulator[D]) record per split
    assert ws(16, 32, 32, 8192, 128) % (16 * 32 * per_row(128)) == 0 and ws(16, 32, 32, 8192, 128) > 0
    assert ws(1, 1, 1, 1, 64) == per_row(64)
    assert ws(2, 4, 4, 100000, 64) >= ws(2, 4, 4, 1000, 64) > 0
    assert ws(1, 3, 2, 10, 128) == 0 and ws(1, 1, 1, 10, 96) == 0
    f = lib.slim_attn_decode_int8

    def call(q=A, kc=A, ks=A, vc=A, vs=A, out=A, wsp=A, wsb=1 << 30, B=1, Hq=2, Hkv=2, T=100, D=128, causal=0, scale=0.1):
        return f(P(q), P(kc), P(ks), P(vc), P(vs), P(out), P(wsp), wsb, B, Hq, Hkv, T, D, causal, scale, None)

    assert call(vs=None) == 1 and call(wsp=None) == 1
    assert call(T=0) == 2 and call(Hq=4, Hkv=3) == 2 and call(scale=-1.0) == 2
    assert call(D=32) == 3
    assert call(out=A + 2) == 4
    assert call(wsb=ws(1, 2, 2, 100, 128) - 1) == 5


def test_decode_workspace_is_a_whole_number_of_split_records_for_every_geometry(lib):
    """Host logic only: whatever split geometry the library picks (per-head or grouped-query kernel), the workspace
    is n_split records of (max, sum, accumulator[D]) per (batch, query head), with at least one split and never
    more splits than the cache has 32-token tiles (plus the one a two-wave workgroup may leave empty)."""
    ws = lib.slim_attn_decode_int8_workspace_bytes
    for D in (64, 128):
        for (B, Hq, Hkv) in ((1, 1, 1), (1, 32, 32), (16, 32, 32), (16, 64, 8), (3, 40, 1), (64, 8, 8), (2, 64, 2), (1, 8, 4)):
            for T in (1, 31, 32, 33, 100, 2048, 8191, 8192, 32768, 100000):
                n, rec = ws(B, Hq, Hkv, T, D), B * Hq * (D + 2) * 4
                assert n > 0 and n % rec == 0, (B, Hq, Hkv, T, D, n)
                splits = n // rec
                assert 1 <= splits <= (T + 31) // 32 + 1, (B, Hq, Hkv, T, D, splits)


def test_rows_that_fit_the_static_scratch_fit_it_at_every_length(lib):
    """The static entry point refuses a call for its rows, never for how many splits the plan would like: up to two
    records a row within the scratch array, every cache length is taken (one record is enough for the per-head kernel)."""
    limit = lib.slim_attn_decode_int8_static_max_bytes()
    for D in (64, 128):
        rec = (D + 2) * 4
        for (B, Hq, Hkv) in ((200, 16, 2), (26, 120, 3), (127, 200, 5), (467, 32, 1), (375, 4, 4), (425, 16, 16), (1000, 16, 16), (1, 64, 8)):
            for T in (64, 500, 1761, 4061, 8066, 16384, 65464):
                n = lib.slim_attn_decode_int8_workspace_bytes(B, Hq, Hkv, T, D)
                assert 0 < n <= max(limit, B * Hq * rec * (1 if Hq == Hkv else 2)), (B, Hq, Hkv, T, D, n)


def test_decode_leaves_no_long_sequence_to_a_few_workgroups(lib):
    """Sequences of different lengths: one of full length among short ones still makes enough workgroups, or its
    workgroups get few enough tokens, or the whole batch makes many, or the records fill the library's own scratch.
    (The entry point cannot know the lengths: the plan has to hold for every mix of them.)"""
    limit = lib.slim_attn_decode_int8_static_max_bytes()
    for D in (64, 128):
        for (B, Hq, Hkv) in ((8, 32, 32), (16, 32, 32), (32, 8, 8), (8, 8, 8), (100, 8, 8), (128, 4, 4), (6, 40, 1), (300, 32, 32),
                             (16, 32, 8), (4, 64, 8), (32, 32, 8), (10, 32, 8), (3, 64, 2), (200, 16, 2)):
            grouped = 2 <= Hq // Hkv <= 32
            heads = Hkv if grouped else Hq
            for T in (1000, 2300, 5000, 8192, 16384, 33000, 65536):
                record = B * Hq * (D + 2) * 4
                n = lib.slim_attn_decode_int8_workspace_bytes(B, Hq, Hkv, T, D) // record
                few_tokens = T < (n + 1) * (32 * D if grouped else 2048)
                many = B * heads * (n + 1) > 768 if grouped else B * heads * n >= 1536
                assert few_tokens or many or heads * n >= 128 or (n + 1) * record > limit, (B, Hq, Hkv, T, D, n)


def test_decode_of_wide_groups_splits_short_caches(lib):
    """17 to 32 query heads on a KV head: a few rows of some hundred tokens are cut, not left to a workgroup each."""
    for D, Hq, T in ((128, 20, 777), (128, 32, 777), (64, 32, 1500), (128, 32, 1500)):
        for B in (1, 2, 8, 16):
            assert lib.slim_attn_decode_int8_workspace_bytes(B, Hq, 1, T, D) // (B * Hq * (D + 2) * 4) >= 4, (B, Hq, T, D)


def test_varlen_decode_rejects_bad_arguments(lib):
    f = lib.slim_attn_decode_int8_varlen

    def call(lens=A, q=A, wsp=A, wsb=1 << 30, T=100, D=128):
        return f(P(q), P(A), P(A), P(A), P(A), P(lens), P(A), P(wsp), wsb, 1, 2, 2, T, D, 0, 0.1, None)

    assert call(lens=None) == 1 and call(q=None) == 1
    assert call(lens=A + 2) == 4 and call(q=A + 4) == 4
    assert call(T=0) == 2 and call(D=96) == 3
    assert call(wsb=8) == 5


def test_quant_pair_rejects_bad_arguments(lib):
    f = lib.kv_quant_int8_pair

    def call(k=A, v=A, kc=A, ks=A, vc=A, vs=A, B=2, Hq=2, Hkv=2, S=100, D=128, causal=0, scale=1.0):
        return f(P(k), P(v), P(kc), P(ks), P(vc), P(vs), B, Hq, Hkv, S, D, causal, scale, None)

    assert call(k=None) == 1 and call(v=None) == 1 and call(vs=None) == 1 and call(kc=None) == 1
    assert call(S=0) == 2 and call(B=-1) == 2
    assert call(D=96) == 3
    assert call(v=A + 8) == 4 and call(vc=A + 4) == 4
    assert call(Hq=3) == 2 and call(causal=2) == 2 and call(scale=0.0) == 2


def test_append_rejects_bad_arguments(lib):
    f = lib.kv_quant_int8_append

    def call(x=A, codes=A, scales=A, pos=A, B=2, Hq=2, Hkv=2, T=100, D=128, causal=0, scale=1.0):
        return f(P(x), P(codes), P(scales), P(pos), B, Hq, Hkv, T, D, causal, scale, None)

    assert call(x=None) == 1 and call(pos=None) == 1 and call(scales=None) == 1
    assert call(T=0) == 2 and call(B=0) == 2
    assert call(D=100) == 3
    assert call(codes=A + 8) == 4 and call(pos=A + 1) == 4
    assert call(Hq=3) == 2 and call(causal=-1) == 2 and call(scale=float("inf")) == 2


def test_prefill_two_sweep_rejects_bad_arguments(lib):
    f = lib.slim_attn_prefill_two_sweep
    need = lib.slim_attn_prefill_two_sweep_workspace_bytes(1, 4, 2, 100, 128)
    assert need == 1 * 4 * 100 * 2 * 4
    assert lib.slim_attn_prefill_two_sweep_workspace_bytes(1, 4, 3, 100, 128) == 0

    def call(q=A, k=A, v=A, out=A, ws=A, wb=need, S=100, D=128, od=0):
        return f(P(q), P(k), P(v), P(out), P(ws), wb, 1, 4, 2, S, D, 1, 0.1, od, None)

    assert call(ws=None) == 1 and call(v=None) == 1
    assert call(S=0) == 2
    assert call(D=96) == 3 and call(od=7) == 3
    assert call(ws=A + 4) == 4
    assert call(wb=need - 1) == 5


def test_prefill_strip_rejects_bad_arguments(lib):
    f = lib.slim_attn_prefill_strip
    assert lib.slim_attn_prefill_strip_max_seq_len() == 2048

    def call(q=A, k=A, v=A, out=A, S=100, D=128, od=0, Hq=4, Hkv=2, causal=1, scale=0.1):
        return f(P(q), P(k), P(v), P(out), 1, Hq, Hkv, S, D, causal, scale, od, None)

    assert call(q=None) == 1 and call(out=None) == 1
    assert call(S=0) == 2 and call(Hq=3) == 2 and call(causal=3) == 2 and call(scale=-1.0) == 2
    assert call(D=96) == 3 and call(od=7) == 3
    assert call(v=A + 4) == 4


def test_probe_library_exports_what_its_header_declares():
    from paper_2407_07304_amd import probes
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "slimprobe.h")).read(), flags=re.S)
    names = sorted(set(re.findall(r"\b(slim_probe_[a-z_0-9]+)\s*\(", text)))
    assert names == ["slim_probe_gqa_decode_traffic", "slim_probe_mfma_bf16", "slim_probe_quant_traffic", "slim_probe_stream_read"]
    lib = probes.load()
    for n in names:
        assert getattr(lib, n) is not None
    # bad arguments are refused before anything is enqueued (no GPU is touched)
    assert lib.slim_probe_stream_read(P(None), 1024, P(A), None) == 1
    assert lib.slim_probe_stream_read(P(A), 1000, P(A), None) == 1
    assert lib.slim_probe_quant_traffic(P(A), P(A), P(A), 10, 96, None) == 1
    assert lib.slim_probe_mfma_bf16(P(A), P(A), 0, P(A), 1, 1, None) == 1
    assert lib.slim_probe_gqa_decode_traffic(P(A), P(A), P(A), P(A), P(A), P(A), 16, 2, 64, 8, 8192, 128, None) == 1   # workspace too small
    assert lib.slim_probe_gqa_decode_traffic(P(A), P(A), P(A), P(A), P(A), P(A), 1 << 30, 1, 4, 4, 100, 128, None) == 1     # not a grouped shape


def test_prefill_form_of_a_call(lib):
    f = lib.slim_attn_prefill_block_rows
    assert f(1, 4, 3, 100, 128, 1, 0, 0) == 0 and f(1, 2, 2, 100, 96, 1, 0, 0) == 0 and f(1, 2, 2, 0, 128, 1, 0, 0) == 0
    assert f(1, 2, 2, 100, 128, 2, 0, 0) == 0 and f(1, 2, 2, 100, 128, 1, 1, 0) == 0 and f(1, 2, 2, 100, 128, 1, 0, 2) == 0
    # bf16 K and V of many heads are more than the L2s hold: the form that reads them once per 32 rows is not taken
    for B, H in ((40, 32), (40, 40), (64, 32)):
        assert f(B, H, H, 300, 64, 0, 0, 0) == 128
    # short sequences, not causal, bf16 results of 128 values: 256 rows, where 32 take a sixth to a third longer
    for shape in ((8, 24, 8, 134), (4, 40, 8, 152), (44, 4, 4, 155), (6, 32, 8, 199)):
        assert f(*shape, 128, 0, 0, 0) == 256, shape
    # few rows in all, not causal: 32, where 128 are slower
    assert f(4, 32, 8, 100, 128, 0, 0, 0) == f(4, 40, 8, 67, 128, 0, 0, 1) == f(10, 16, 2, 93, 128, 0, 0, 1) == 32
    # long INT8 sequences of few heads, which that form would widen once per 32 rows
    for Hkv in (8, 2):
        assert f(1, 8, Hkv, 5000, 128, 1, 2, 0) == f(1, 8, Hkv, 5000, 128, 1, 2, 1) == 128
    # the form with a workgroup of 256 threads per 32 rows and head is taken only where a launch can hold them (less than
    # 2^32 threads); the item lists of the others need no more workgroups than the chip has compute units
    short, at_limit = f(170, 30000, 30000, 96, 64, 1, 0, 0), f(200, 30000, 30000, 96, 64, 1, 0, 0)
    assert 170 * 30000 * 3 * 256 < 2 ** 32 <= 200 * 30000 * 3 * 256 and short == 32 and at_limit == 128
    for B, H, S in ((600, 30000, 1), (300, 60000, 32), (280, 30000, 64), (200, 30000, 96), (150, 60000, 128)):
        for D in (64, 128):
            for kv in (0, 2):
                for od in (0, 1):
                    assert f(B, H, H, S, D, 1, kv, od) in (128, 256), (B, H, S, D, kv, od)


def test_decode_plan_of_a_call(lib):
    w, n = ctypes.c_int(), ctypes.c_int()
    f = lib.slim_attn_decode_int8_plan
    assert f(1, 4, 2, 100, 128, 0, None, ctypes.byref(n)) == 1 and f(1, 4, 3, 100, 128, 0, ctypes.byref(w), ctypes.byref(n)) == 2
    assert f(1, 4, 2, 100, 96, 0, ctypes.byref(w), ctypes.byref(n)) == 3 and f(1, 4, 2, 100, 128, 2, ctypes.byref(w), ctypes.byref(n)) == 2

    def plan(*shape, ragged=1):
        assert f(*shape, ragged, ctypes.byref(w), ctypes.byref(n)) == 0
        assert n.value * shape[0] * shape[1] * (shape[4] + 2) * 4 <= lib.slim_attn_decode_int8_workspace_bytes(*shape)
        return w.value, n.value

    # grouped heads, 128 codes a token: a batch that fills the chip keeps workgroups of four waves, of which three fit a
    # compute unit, for lengths of their own too (the allocated length says nothing about how long the contexts are)
    for shape, splits in (((48, 32, 8, 3001, 128), 1), ((100, 32, 8, 4000, 128), 1), ((32, 32, 8, 3000, 128), 1),
                          ((16, 64, 8, 8192, 128), 2)):
        assert plan(*shape) == plan(*shape, ragged=0) == (4, splits), shape
    for shape, splits in (((16, 32, 8, 32768, 128), 6), ((32, 32, 8, 8192, 128), 2), ((32, 32, 8, 32768, 128), 3), ((100, 16, 2, 6000, 64), 2)):   # cut finer than equal lengths
        assert plan(*shape) == (4, splits), shape
    # 64 codes a token: eight waves up to one workgroup a compute unit
    assert plan(32, 32, 8, 3000, 64) == (8, 1) and plan(33, 32, 8, 300, 64) == (4, 1) and plan(32, 32, 8, 3000, 64, ragged=0) == (4, 1)
    # fewer workgroups than compute units, and more than sixteen heads a KV head: always eight
    assert plan(20, 16, 4, 700, 128)[0] == plan(64, 40, 2, 3000, 128)[0] == 8


def test_decode_short_steps_keep_whole_rows(lib):
    w, n = ctypes.c_int(), ctypes.c_int()

    def splits(*shape, ragged):
        assert lib.slim_attn_decode_int8_plan(*shape, ragged, ctypes.byref(w), ctypes.byref(n)) == 0
        # (the workspace that the library asks for is enough for both entry points, whichever plan has more splits)
        assert n.value * shape[0] * shape[1] * (shape[4] + 2) * 4 <= lib.slim_attn_decode_int8_workspace_bytes(*shape)
        return n.value

    # a second launch would outlast the step: 3 to 21 % longer from the host
    for shape in ((21, 4, 4, 1590, 64), (9, 8, 8, 1483, 64), (3, 32, 32, 1437, 128), (16, 4, 4, 1172, 128)):
        assert splits(*shape, ragged=1) == 1, shape
    for shape in ((2, 32, 32, 1210, 128), (20, 4, 4, 1186, 128), (2, 32, 32, 1400, 64)):
        assert splits(*shape, ragged=0) == 1, shape
    # longer ones gain by it; three lengths of up to 1437 tokens are shorter than three of 1437
    for shape in ((20, 4, 4, 1300, 128), (3, 32, 32, 1600, 128), (16, 8, 8, 2000, 64), (30, 4, 4, 2229, 128)):
        assert splits(*shape, ragged=0) > 1 and splits(*shape, ragged=1) > 1, shape
    assert splits(3, 32, 32, 1437, 128, ragged=0) == 2


def test_decode_records_of_a_call(lib):
    r, t = ctypes.c_int(), ctypes.c_int()
    f = lib.slim_attn_decode_int8_plan_options
    assert f(1, 4, 2, 100, 128, 0, None, ctypes.byref(t)) == 1 and f(1, 4, 3, 100, 128, 0, ctypes.byref(r), ctypes.byref(t)) == 2
    assert f(1, 4, 2, 100, 96, 0, ctypes.byref(r), ctypes.byref(t)) == 3 and f(1, 4, 2, 100, 128, 2, ctypes.byref(r), ctypes.byref(t)) == 2

    def through(*shape, ragged=1):
        assert f(*shape, ragged, ctypes.byref(r), ctypes.byref(t)) == 0
        return t.value

    # splits of different lengths: plain stores where the caches are long (through the L2 these took 2 to 4 % longer), not where they
    # are short; equal lengths, and a sequence alone, end together
    for shape in ((41, 16, 2, 23692, 64), (30, 16, 2, 41089, 64), (15, 64, 8, 26557, 64), (8, 64, 8, 40000, 128), (32, 16, 2, 8000, 64)):
        assert through(*shape) == 0 and through(*shape, ragged=0) == 1, shape
    for shape in ((24, 16, 2, 2525, 128), (2, 64, 8, 4734, 128), (3, 32, 32, 2450, 64), (1, 64, 8, 100000, 128)):
        assert through(*shape) == 1, shape
    assert through(48, 32, 8, 3001, 128) == through(16, 32, 32, 8192, 128, ragged=0) == 0   # (no records)


def test_prefill_emit_rejects_bad_arguments(lib):
    f = lib.slim_attn_prefill_emit_int8

    def call(q=A, k=A, v=A, out=A, kc=A, ks=A, vc=A, vs=A, S=100, D=128, od=0):
        return f(P(q), P(k), P(v), P(out), P(kc), P(ks), P(vc), P(vs), 1, 4, 2, S, D, 1, 0.1, od, None)

    assert call(kc=None) == 1 and call(vs=None) == 1 and call(q=None) == 1
    assert call(S=0) == 2
    assert call(D=96) == 3 and call(od=7) == 3
    assert call(vc=A + 4) == 4 and call(k=A + 2) == 4


def test_binding_fails_loudly_without_the_library(tmp_path, monkeypatch):
    # no CPU fallback: a missing library is an error, not a slower path
    from paper_2407_07304_amd import slimattn
    monkeypatch.setattr(slimattn, "LIB_PATH", str(tmp_path / "libslimattn.so"))
    monkeypatch.setattr(slimattn, "_lib", None, raising=False)
    with pytest.raises(ImportError, match="no fallback"):
        slimattn.load()


def test_product_code_does_not_touch_the_oracle():
    # the oracle is test infrastructure: nothing under the package imports or loads it
    pkg = os.path.join(os.path.dirname(HEADER), "..", "paper_2407_07304_amd")
    for root, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h")):
                text = open(os.path.join(root, f)).read()
                assert not re.search(r"import\s+oracle|from\s+oracle|oracle[/.]|libslim_oracle|slim_oracle\.", text), f
