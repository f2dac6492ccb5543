"""Who merges a (sequence, kv head) of a decode launch: every order in which its workgroups can reach their counter, in a host build of
the header that the kernel includes."""
import ctypes

import pytest

from tests.decode_model import build_model


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    return build_model(tmp_path_factory)


@pytest.mark.parametrize("awaited", [False, True])
@pytest.mark.parametrize("parts", [0, 1, 2, 4])  # (no correction; the kernel has 4)
@pytest.mark.parametrize("splits", [1, 2, 3, 5])
def test_every_order_ends_in_one_merge(model, splits, parts, awaited):
    for looks in (0, 1, 2, 5):
        most, by_correction = ctypes.c_int(), ctypes.c_int()
        assert model.every_order_merges_once(splits, parts, int(awaited), looks, ctypes.byref(most), ctypes.byref(by_correction)), (splits, parts, looks)
        # one look before the partial results are combined, then a bounded wait, once
        first = 1 if splits == 1 and parts > 0 else 0
        assert most.value <= first + (looks if awaited and parts > 0 else 0), (splits, looks)
        assert by_correction.value == (parts > 0)  # reached: it arrived last, or the wait had run out
