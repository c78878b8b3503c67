"""The rule that splits a batch's private pages into chunks (kvprm::private_chunk_rule), called in the
library on the host: every form it picks is reached by the GPU cases of test_gpu_chunks.py, a
batch with enough pages makes a wave for most compute units whatever its kv-heads, and a table of
unknown lengths is not cut longer than a full one would be."""
import ctypes

import numpy as np
import pytest

import paper_2607_09153_amd as kv

from test_gpu_chunks import CASES


class Dims(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("layers", "H", "nq", "nkv", "d", "F", "g")] + \
        [("theta", ctypes.c_float), ("eps", ctypes.c_float), ("wdt", ctypes.c_int), ("kvdt", ctypes.c_int)]


class Chunks(ctypes.Structure):
    _fields_ = [("shift", ctypes.c_int), ("heads", ctypes.c_int)]


_rule = kv.lib._ZN5kvprm18private_chunk_ruleERKNS_4DimsEiPKiS4_b
_rule.restype = Chunks
_rule.argtypes = [ctypes.POINTER(Dims), ctypes.c_int, ctypes.POINTER(ctypes.c_int),
                  ctypes.POINTER(ctypes.c_int), ctypes.c_bool]
_long = kv.lib._ZN5kvprm16long_chunk_shiftEx
_long.argtypes = [ctypes.c_longlong]

COMPUTE_UNITS = 256
KVDT = {"f32": 0, "bf16": 1, "fp8": 2}


def _pick(nkv, d, dtype, lengths, known=True):
    """(pages per chunk, heads per block, pages) of a batch, with slots for 16-page chunks (fp32: 32)
    and for 128 shorter ones."""
    pages = [(n + 15) // 16 for n in lengths]
    if not known:
        pages = [max(1, *pages)] * len(pages)
    base = 32 if dtype == "f32" else 16
    slots = [max(-(-max(pages) // base) + 1, 129)] * len(pages)
    ints = ctypes.c_int * len(pages)
    r = _rule(Dims(1, 64, nkv, nkv, d, 64, 1, 1.0, 0.0, 0, KVDT[dtype]), len(pages), ints(*pages),
              ints(*slots), known)
    return 1 << r.shift, r.heads, pages


def test_gpu_cases_reach_every_form():
    forms = set()
    for nq, nkv, d, dtype, lengths in CASES:
        if dtype == "f32":
            continue
        for known in (True, False):
            chunk, heads, pages = _pick(nkv, d, dtype, lengths, known)
            if max(pages) > 32 or len(pages) * nkv > 256:  # (else the one-launch kernel)
                assert heads in (1, nkv)
                forms.add((chunk, "one" if heads == 1 else "all"))
    assert forms == {(c, "one") for c in (4, 8, 16, 32, 64)} | {(64, "all")}


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("nkv", range(1, 9))
def test_enough_pages_make_enough_waves(nkv, dtype):
    rng = np.random.default_rng(91)
    for d in (64, 128):
        for B in (1, 2, 3, 4, 7, 8, 16, 32, 64):
            for longest in (600, 2100, 4100, 8200, 16000, 32000):
                lengths = rng.integers(longest // 2, longest + 1, B).tolist()
                chunk, heads, pages = _pick(nkv, d, dtype, lengths)
                waves = sum(-(-n // chunk) for n in pages) * nkv
                in_16 = sum(-(-n // 16) for n in pages) * nkv
                assert waves >= min(160, in_16), (d, B, longest, chunk, waves)
                assert heads == 1 or sum(-(-n // 64) for n in pages) >= 160


def test_unknown_lengths_take_no_longer_chunks_than_a_full_table():
    for nkv in (1, 2, 4, 8):
        for B in (1, 2, 4, 8, 16, 32, 64):
            for longest in (300, 2000, 9600, 32768):
                chunk, heads, pages = _pick(nkv, 128, "bf16", [longest] * B, known=False)
                assert chunk <= 1 << _long(sum(pages)) and heads == 1
