"""What the compiled marshalling module takes as a problem or a decode shape: what a ctypes call of the same C function
takes, read when the call is made.  Every call here is refused on the host: no GPU."""
import copy
import ctypes as C

import pytest

import paper_2503_17922_amd as W


def _problem(**kw):
    base = dict(n_q_heads=8, n_kv_heads=2, head_dim=128, w_obs=16, seq_len=[700], win=[8], top_p=[8], k_windows=[10], dtype=W.WKV_BF16)
    base.update(kw)
    return W.Problem(**base)


def _shape(**kw):
    base = dict(batch=1, n_q_heads=8, n_kv_heads=2, head_dim=128, dtype=W.WKV_BF16, capacity=100)
    base.update(kw)
    return W.DecodeShape(**base)


PROBLEM_CALLS = {
    "score": lambda p: W.wkv_score(p, None, None, None, None, None, stream=0),
    "window_pool": lambda p: W.wkv_window_pool(p, None, None, stream=0),
    "topk_windows": lambda p: W.wkv_topk_windows(p, None, None, None, None, stream=0),
    "gather_group": lambda p: W.wkv_gather_group(p, [None], [None], None, None, [None], [None], stream=0),
    "compress_group": lambda p: W.wkv_compress_group(p, 1, None, None, [None], [None], [None], [None], None, None, None, None, stream=0),
    "compress_groups": lambda p: W.wkv_compress_groups(p, 1, 1, [None], None, [None], [None], [None], [None], None, None, None, None, stream=0),
}
SHAPE_CALLS = {
    "decode_step": lambda s: W.wkv_decode_step(s, None, None, None, None, None, None, None, None, stream=0),
    "decode_step_static": lambda s: W.wkv_decode_step_static(s, None, None, None, None, None, None, None, stream=0),
}
CALLS = [pytest.param(f, _problem, _shape, id=n) for n, f in PROBLEM_CALLS.items()] + \
        [pytest.param(f, _shape, _problem, id=n) for n, f in SHAPE_CALLS.items()]


@pytest.mark.parametrize("call,right,wrong", CALLS)
def test_the_other_structure_is_refused(call, right, wrong):
    with pytest.raises(W.WkvError, match="NULL"):
        call(right())
    with pytest.raises(C.ArgumentError):
        call(wrong())

    class HasAddress:
        def __init__(self, o):
            self.o = o
            self._addr = C.addressof(o.c)

        def ref(self):
            return self.o.ref()

    with pytest.raises(C.ArgumentError):
        call(HasAddress(wrong()))
    with pytest.raises(W.WkvError, match="NULL"):         # its ref() is what a ctypes call asks for
        call(HasAddress(right()))
    for o in (None, 0, object(), right().c):
        with pytest.raises(AttributeError):
            call(o)
    changed = right()
    changed.c = wrong().c
    with pytest.raises(C.ArgumentError):
        call(changed)
    changed.c = 4096
    with pytest.raises((C.ArgumentError, TypeError)):     # (ctypes.byref raises TypeError itself)
        call(changed)


@pytest.mark.parametrize("call,right,wrong", CALLS)
def test_the_structure_is_read_when_the_call_is_made(call, right, wrong):
    o = right()
    o.c.head_dim = 96
    with pytest.raises(W.WkvError, match="head_dim 96"):
        call(o)
    o.c = type(o.c).from_buffer_copy(o.c)                # another structure in its place
    o.c.head_dim = 80
    with pytest.raises(W.WkvError, match="head_dim 80"):
        call(o)
    other = copy.copy(o)
    other.c = type(o.c).from_buffer_copy(o.c)
    other.c.head_dim = 72
    with pytest.raises(W.WkvError, match="head_dim 72"):
        call(other)
    with pytest.raises(W.WkvError, match="head_dim 80"):
        call(o)


def test_a_deep_copy_has_a_structure_of_its_own():
    original = _shape()
    shape = copy.deepcopy(original)
    shape.c.batch = 0
    with pytest.raises(W.WkvError, match="batch must be >= 1"):
        W.wkv_decode_step(shape, *[None] * 8, stream=0)


@pytest.mark.parametrize("reference", [C.byref, C.pointer])
def test_a_subclass_may_make_its_own_reference(reference):
    class Other(W.DecodeShape):
        def ref(self):
            c = type(self.c).from_buffer_copy(self.c)
            c.capacity = 0
            return reference(c)

    with pytest.raises(W.WkvError, match="capacity"):
        W.wkv_decode_step(Other(batch=1, n_q_heads=8, n_kv_heads=2, head_dim=128, dtype=W.WKV_BF16, capacity=100), *[None] * 8, stream=0)
