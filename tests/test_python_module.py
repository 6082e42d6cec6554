"""What the Python module over libtw (csrc/tw_python.cpp) takes and refuses, as far as that can be seen
without a GPU: tensors in host memory stand where a check ahead of the tensors' own has to speak first."""
import collections
import ctypes
import types

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


class MissingIsHost(dict):
    """Every key that is not there stands for a tensor in host memory."""

    def __missing__(self, key):
        return HOST


class Lookup(dict):
    """A dict whose items are made when they are asked for."""

    def __getitem__(self, key):
        return HOST


FUSED = dict(partials=[HOST], residual=HOST, weight=WEIGHT, eps=1e-5, out=HOST, residual_out=HOST)


@pytest.mark.parametrize("make", [dict, collections.OrderedDict, types.MappingProxyType, collections.UserDict,
                                  collections.ChainMap], ids=lambda m: m.__name__)
def test_argument_groups_may_be_any_mapping(make):
    """... and get as far as the tensors, which are refused for lying in host memory."""
    with pytest.raises(TypeError, match=r"partials\[0\] must be a GPU tensor"):
        tw.overlap_launch(make(FUSED), None, None, None)
    with pytest.raises(TypeError, match="B must be a GPU tensor"):
        tw.overlap_launch(None, make(dict(A=HOST, B=HOST, C=None, b_layout=tw.B_NK)), None, None)
    with pytest.raises(TypeError, match=r"partials\[0\] must be a GPU tensor"):
        tw.weave_train([make(dict(FUSED, X1=HOST, W1=HOST, W2=HOST, Y=HOST))], 0, None, None)
    with pytest.raises(KeyError, match="weight"):
        tw.overlap_launch(make({k: v for k, v in FUSED.items() if k != "weight"}), None, None, None)


def test_argument_groups_are_asked_the_way_python_asks():
    with pytest.raises(TypeError, match="B must be a GPU tensor"):
        tw.overlap_launch(None, MissingIsHost(A=HOST), None, None)
    with pytest.raises(TypeError, match="B must be a GPU tensor"):
        tw.overlap_launch(None, Lookup(A=None, B=None), None, None)
    with pytest.raises(TypeError):
        tw.overlap_launch([HOST], None, None, None)
    # optional ones through get(): __missing__ does not stand in for them
    with pytest.raises(TypeError, match="B must be a GPU tensor"):
        tw.overlap_launch(None, MissingIsHost(A=HOST, B=HOST), None, None)


@pytest.mark.parametrize("name", ["out", "residual_out", "Y"])
def test_a_train_makes_no_outputs_of_its_own(name):
    """It returns none, so one made for it would be freed with kernels still to write it."""
    with pytest.raises(TypeError, match="%s must be a GPU tensor" % name):
        tw.weave_train([dict(FUSED, X1=HOST, W1=HOST, W2=HOST, Y=HOST) | {name: None}], 0, None, None)


def test_numbers_are_read_as_int_and_float_read_them():
    """b_layout is compared with the two layouts, not rounded to one."""
    for bad in (0.5, "0", 2, -1, None, 1.25):
        with pytest.raises(ValueError, match="b_layout must be B_NK or B_KN"):
            tw.gemm_bf16(HOST, HOST, b_layout=bad)
    for good in (0, 1.0, False, True):
        with pytest.raises((TypeError, ValueError), match="B must be a GPU tensor"):
            tw.gemm_bf16(HOST, HOST, b_layout=good)


@pytest.mark.gpu
def test_eps_is_whatever_float_takes():
    x, w = torch.randn((3, 64), device="cuda:0").bfloat16(), torch.ones((64,), dtype=torch.bfloat16, device="cuda:0")
    want = tw.reduce_add_rmsnorm([x], x, w, 1e-5)[0]
    for eps in ("1e-5", torch.tensor(1e-5, dtype=torch.float64)):
        assert torch.equal(tw.reduce_add_rmsnorm([x], x, w, eps)[0], want)
    assert torch.equal(tw.reduce_add_rmsnorm([x], x, w, True)[0], tw.reduce_add_rmsnorm([x], x, w, 1.0)[0])
