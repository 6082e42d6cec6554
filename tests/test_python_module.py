"""What the Python module over libtw (csrc/tw_python.cpp) takes and refuses, as far as that can be seen
without a GPU: tensors in host memory stand where a check ahead of the tensors' own has to speak first."""
import ctypes

import pytest
import torch

import paper_2505_11329_amd as tw
from paper_2505_11329_amd.binding import FusedArgs, LayerArgs

HOST = torch.zeros((4, 64), dtype=torch.bfloat16)
WEIGHT = torch.zeros((64,), dtype=torch.bfloat16)


class LongerThanItSays(list):
    """Three items, and a length of one."""

    def __len__(self):
        return 1


class ShorterThanItSays(list):
    def __len__(self):
        return 7


def fill(kind, partials, room=1):
    """fill_fused / fill_layer with an array for `room` pointers."""
    arr = (ctypes.c_void_p * room)()
    if kind == "fused":
        return tw.binding.native().fill_fused(FusedArgs(), arr, partials, HOST, WEIGHT, 1e-5, 0, HOST, HOST)
    return tw.binding.native().fill_layer(LayerArgs(), arr, HOST, HOST, partials, HOST, WEIGHT, 1e-5, HOST, 0, 0, HOST,
                                          HOST, HOST, 0)


@pytest.mark.parametrize("kind", ["fused", "layer"])
def test_pointer_arrays_are_never_filled_past_their_end(kind):
    """The array is made by the partials' length and filled by iterating over them: where the two differ,
    or the array is too small for either, nothing is written."""
    for partials in (LongerThanItSays([HOST] * 3), ShorterThanItSays([HOST] * 3)):
        with pytest.raises(ValueError, match="has a length of . and iterates over 3"):
            fill(kind, partials)
    with pytest.raises(ValueError, match="room for 1 of 2"):
        fill(kind, [HOST, HOST])
    with pytest.raises(TypeError, match=r"partials\[0\] must be a GPU tensor"):     # room enough: on to the tensors
        fill(kind, [HOST])


def test_sequences_without_a_length_are_refused_and_cuts_may_be_any_iterable():
    streams = (None, None)
    for partials in ((t for t in [HOST]), iter([HOST]), LongerThanItSays([HOST] * 3)):
        with pytest.raises((TypeError, ValueError), match="len"):
            tw.reduce_add_rmsnorm(partials, HOST, WEIGHT, 1e-5, out=HOST, residual_out=HOST)
    with pytest.raises(TypeError, match="len"):
        tw.weave_train((b for b in []), 0, *streams)
    with pytest.raises(ValueError, match="length"):
        tw.weave_train(LongerThanItSays([{}, {}]), 0, *streams)
    with pytest.raises(TypeError, match="len"):
        tw.overlap_launch(dict(partials=iter([HOST]), residual=HOST, weight=WEIGHT, eps=1e-5, out=HOST, residual_out=HOST),
                          None, *streams)
