"""Host tests of the launch rules, read off the workspace a call asks for (no GPU).

A tail prefill's workspace holds the rotated queries, the V^T tiles of the long kernel (none
for a short tail) and, per split of the key range, the partial outputs (f16 or fp32) with
two floats a row; each region is a multiple of 256 bytes.
"""
import ctypes

import pytest

import paper_2609_18935_amd as tu


def _up(n):
    return (n + 255) // 256 * 256


def _size(hq, hkv, d, T, rows, splits=0):
    p = tu.attn_params(hq, hkv, d, kv_splits=splits)
    return tu.lib().tail_prefill_attention_workspace_size(ctypes.byref(p), T, rows)


def _splits(hq, hkv, d, T, rows):
    """(split count, bytes of a partial output value) of the library's own choice."""
    extra = _size(hq, hkv, d, T, rows) - _size(hq, hkv, d, T, rows, 1)
    if extra == 0:
        return 1, 4
    for size in (2, 4):
        for s in range(2, 129):
            if _up(s * T * hq * d * size) + _up(s * T * hq * 8) == extra:
                return s, size
    raise AssertionError(f"{extra} bytes of partial outputs")


# Launches that equal query tiles would run whole: split for their uneven tiles, or because the
# short kernel's units are smaller, with fp32 partials; the others in f16.
@pytest.mark.parametrize("hq,hkv,d,T,rows,split,size", [
    (16, 2, 256, 2048, 0, True, 2),       # one workgroup on half the CUs: split to fill them
    (16, 2, 256, 2721, 0, True, 4),
    (16, 2, 256, 4096, 0, True, 4),
    (16, 2, 256, 3500, 8000, True, 4),
    (16, 2, 256, 8191, 0, False, 4),
    (16, 2, 256, 512, 8192, True, 2),
    (16, 4, 64, 3000, 0, True, 4),
    (16, 4, 64, 4096, 0, True, 4),
    (32, 8, 128, 1600, 0, False, 4),
    (16, 2, 256, 1, 300, True, 4),        # short tails
    (16, 2, 256, 1, 32768, True, 2),
    (16, 4, 64, 16, 600, True, 4),
    (32, 8, 128, 1, 400, False, 4),
])
def test_partial_outputs_keep_fp32_where_a_launch_would_run_whole(hq, hkv, d, T, rows, split, size):
    n, b = _splits(hq, hkv, d, T, rows)
    assert (n > 1, b) == (split, size), (n, b)


# A short tail packs no V^T tiles. One row tile of 32 packed rows: always; two: up to 32,768 units
# of 32 rows and 32 keys; up to eight: up to 8,192.
@pytest.mark.parametrize("hq,hkv,d,T,keys,short", [
    (16, 2, 256, 1, 1 << 20, True),
    (16, 2, 256, 4, 1 << 20, True),
    (32, 8, 128, 8, 1 << 20, True),
    (32, 8, 128, 9, 65536, True),
    (32, 8, 128, 9, 65537, False),
    (32, 8, 128, 16, 65536, True),
    (32, 8, 128, 16, 65537, False),
    (16, 2, 256, 8, 262144, True),
    (16, 2, 256, 8, 262145, False),
    (32, 8, 128, 17, 10912, True),       # three row tiles: 341 units of keys
    (32, 8, 128, 17, 10913, False),
    (16, 4, 64, 64, 8192, True),         # eight
    (16, 4, 64, 64, 8193, False),
    (16, 4, 64, 65, 1000, False),
])
def test_short_tail_limits(hq, hkv, d, T, keys, short):
    tiles = 0 if short else _up(2 * hkv * ((keys + 63) // 64) * d * 72)
    assert _size(hq, hkv, d, T, keys - T, 1) == 256 + _up(2 * T * hq * d) + tiles
