"""The dynamic mask's scratch fits for every frame size that the calls accept,
by the library's own host functions (no GPU)."""
import ctypes

import numpy as np
import pytest

import paper_1905_02082_amd as rf


class FrameDev(ctypes.Structure):
    _fields_ = [("depth", ctypes.c_void_p), ("rgb", ctypes.c_void_p), ("W", ctypes.c_int), ("H", ctypes.c_int),
                ("rest", ctypes.c_float * 7)]


@pytest.fixture(scope="module")
def sizes():
    """(bytes of the rule's bits, bytes of the members, room(tiles))"""
    L = rf.lib()
    edge, member = L["_ZN2rf16flood_edge_bytesERKNS_8FrameDevE"], L["_ZN2rf18flood_member_bytesERKNS_8FrameDevE"]
    room = L["_ZN2rf15flood_edge_roomEj"]
    for fn in (edge, member, room):
        fn.restype = ctypes.c_size_t
    room.argtypes = [ctypes.c_uint32]

    def of(W, H):
        f = FrameDev(None, None, W, H)
        return edge(ctypes.byref(f)), member(ctypes.byref(f))

    return of, room


def shapes():
    edges = sorted({1, 2, 3, 7, 8, 9, 15, 63, 64, 65, 127, 128, 129, 255, 256, 257, 319, 320, 321, 511, 513, 1023, 1025,
                    4097, 65537, 1 << 20, 1 << 22})
    out = [(a, b) for a in range(1, 70) for b in range(1, 70)]
    return out + [(a, b) for a in edges for b in edges if a * b <= 1 << 26]


def up(x):
    return (x + 255) // 256 * 256


def test_bits_fit_the_maps_scratch(sizes):
    """A map for exactly the frame: its last cache level has a tile of 8192
    bytes for each 256 pixels and 64 spare ones, its member scratch a byte a
    pixel, rounded up to 256."""
    of, room = sizes
    for W, H in shapes():
        edge, member = of(W, H)
        assert up(edge) <= room((W * H + 255) // 256 + 64), (W, H)
        assert member <= up(W * H), (W, H)


def test_bits_fit_the_static_array(sizes):
    """Every frame within the static variant's limit (4 MiB for a byte a pixel
    and the tile flags) fits its 6 MiB array, so none of them is refused."""
    of, _ = sizes
    rng = np.random.default_rng(0)
    tried = 0
    longest = {w: (4 << 20) // w for w in list(range(1, 2200)) + [4097, 65537, 1 << 20, 1 << 22]}
    for w, h in list(longest.items()) + [(h, w) for w, h in longest.items()]:
        for W, H in ((w, h), (w, max(1, h - int(rng.integers(0, 64))))):
            flags = 8 * ((W + 31) // 32) * ((H + 31) // 32)
            while H > 1 and up(W * H) + flags > 4 << 20:
                H -= 1
                flags = 8 * ((W + 31) // 32) * ((H + 31) // 32)
            if up(W * H) + flags > 4 << 20:
                continue
            edge, member = of(W, H)
            assert up(up(member) + flags) + edge <= 6 << 20, (W, H)
            tried += 1
    assert tried > 4000
