"""The quick way to the chunks' addresses gives what .ctypes.data gives, and
steps aside for every array that it does not take."""
import ctypes as C

import numpy as np
import pytest

import paper_2608_19273_amd as pb


def test_addresses_equal_the_general_way():
    big = np.zeros((5, 4, 4, 4, 5))
    chunks = list(big) + [np.zeros(7), np.zeros((3, 1, 2))[:, 0, 0][:1], big[2, 1:3], np.frombuffer(bytearray(64))]
    got = pb._addresses(chunks)
    assert list(got) == [a.ctypes.data for a in chunks]
    assert len(pb._addresses([])) == 1 and C.sizeof(pb._addresses([])) == C.sizeof(C.c_void_p)
    big.resize((6, 4, 4, 4, 5), refcheck=False)   # no buffer is left exported


@pytest.mark.parametrize("a", [np.zeros((4, 4)).T, np.zeros(8)[::2], np.zeros(4, np.float32), np.zeros(4, ">f8"),
                               np.zeros(4, np.int64), np.zeros(0), np.ma.zeros(4), memoryview(bytearray(32)),
                               np.frombuffer(bytes(32))], ids=lambda a: type(a).__name__)
def test_steps_aside(a):
    assert pb._addresses([np.zeros(4), a]) is None
