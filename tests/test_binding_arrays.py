"""The binding's bulk conversions give the C arrays that field-by-field
conversion gives, and leave to it what only it converts or refuses."""
import ctypes as C
import struct
from itertools import chain

import numpy as np
import pytest

from paper_2609_27193_amd import layercheck as LC


def one_by_one(segments):
    arr = (LC.lc_segment * len(segments))()
    for i, s in enumerate(segments):
        arr[i] = LC.lc_segment(s.layer, 0, s.numel, s.weight, s.shadow or None, None, None, None)
    return bytes(arr)


@pytest.mark.parametrize("n", [1, 3, 219])
def test_segments_packed_at_once(n):
    segs = [LC.Segment(i // 2, (1 << 40) + i, (1 << 63) + 2 * i, 4096 * (i + 1), 8, 16, 24) for i in range(n)]
    arr = (LC.lc_segment * n)()
    assert struct.calcsize(LC._STATIC_FIELDS) == C.sizeof(LC.lc_segment)
    struct.pack_into(LC._STATIC_FIELDS * n, arr, 0, *chain.from_iterable(map(LC._static_fields, segs)))
    assert bytes(arr) == one_by_one(segs)


@pytest.mark.parametrize("layer,shadow", [(0, None), (-1, 4096), ((1 << 33) + 7, 4096)])
def test_values_outside_the_format_are_left_to_ctypes(layer, shadow):
    seg = LC.Segment(layer, 5, 4096, shadow, None, None, None)
    with pytest.raises((struct.error, TypeError)):
        struct.pack(LC._STATIC_FIELDS, *LC._static_fields(seg))
    with pytest.raises(LC.LCError) as e:  # refused by the library, before any GPU work
        LC.lc_score_layers_static([seg], 1, LC.LC_DT_BF16, 1e-8, 8)
    assert e.value.code == LC.LC_ERR_INVALID_ARG


@pytest.mark.parametrize("ptrs", [[], [4096], list(range(8, 8 * 300, 8)), [np.int64(16), np.uint64(1 << 63)], [(1 << 64) - 2]])
def test_addresses(ptrs):
    got = LC._addresses(ptrs)
    assert bytes(got) == bytes((C.c_void_p * len(ptrs))(*[int(x) for x in ptrs]))
    assert bytes(LC._addresses([3.0, np.float64(8)])) == bytes((C.c_void_p * 2)(3, 8))  # what int() takes
