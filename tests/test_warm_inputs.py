"""The record of the layers' inputs in the warm-start network's cache: a decoder layer
whose concatenation was read in place holds its two parts until the tensor is asked for,
and whichever way a dictionary is read or copied gives the tensor."""
import copy
import pickle

import pytest

from paper_1203_3583_amd.warmstart import _LayerInputs


class _Net:
    """Upsampling and concatenation of strings."""

    def __init__(self):
        self.formed = 0

    def _up(self, a):
        return a + a

    def _cat(self, a, b):
        self.formed += 1
        return a + b


PLAIN = {0: "x", 8: "llss", 9: "y", 10: "mmtt", 11: "z"}


def _inputs():
    net = _Net()
    return net, _LayerInputs(net, {0: "x", 8: ("l", "ss"), 9: "y", 10: ("m", "tt"), 11: "z"})


def _merged(d):
    d |= {0: "w"}
    return dict(d)


def _updated(d):
    e = {}
    e.update(d)
    return e


READS = {
    "dict": dict, "unpacked": lambda d: {**d}, "copy": lambda d: d.copy(), "copy.copy": copy.copy,
    "deepcopy": copy.deepcopy, "pickle": lambda d: pickle.loads(pickle.dumps(d)), "update": _updated,
    "items": lambda d: dict(d.items()), "values": lambda d: dict(zip(d.keys(), d.values())),
    "get": lambda d: {i: d.get(i) for i in d}, "subscript": lambda d: {i: d[i] for i in d},
    "pop": lambda d: {i: d.pop(i) for i in list(d)},
    "popitem": lambda d: dict(reversed([d.popitem() for _ in range(len(d))])),
    "setdefault": lambda d: {i: d.setdefault(i, None) for i in d},
    "or": lambda d: d | {}, "ror": lambda d: {} | d, "repr": lambda d: eval(repr(d)),
    "reversed": lambda d: {i: d[i] for i in reversed(list(reversed(d)))},
}


@pytest.mark.parametrize("how", list(READS))
def test_reads_as_a_dictionary_of_tensors(how):
    _, d = _inputs()
    got = READS[how](d)
    assert type(got) is dict and got == PLAIN and list(got) == list(PLAIN)


def test_is_a_dictionary():
    net, d = _inputs()
    assert isinstance(d, dict) and len(d) == 5 and list(d) == list(PLAIN) and 8 in d and 7 not in d
    assert d.parts(8) == ("l", "ss") and d.parts(0) == "x" and net.formed == 0
    assert d == PLAIN and PLAIN == dict(d) and net.formed == 2
    assert d.parts(8) == "llss" and d[8] == "llss" and net.formed == 2   # formed once
    assert d.get(7) is None and d.get(7, "d") == "d" and d.pop(7, "d") == "d"
    with pytest.raises(KeyError):
        d[7]
    with pytest.raises(KeyError):
        d.pop(7)
    d[9] = "new"
    del d[0]
    assert d.parts(9) == "new" and list(d) == [8, 9, 10, 11]
    assert _merged(_inputs()[1]) == {**PLAIN, 0: "w"}
    net, d = _inputs()
    d.clear()
    assert len(d) == 0 and net.formed == 0
