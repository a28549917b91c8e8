"""The pieces a walk batch's box is cut into (csrc/vr_walk_pieces.h, compiled
here for the CPU) against the definition in exact integers: over the whole range
of boxes, moves and workgroups the split is the smallest whose pieces fit a
window, and windows are taken only where 16 moves a piece allow it, up to boxes
of 32,768 cells, where 16 x 16,384 x 16,384 does not fit 32 bits."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1805_08893_amd", "csrc")
SIDE = 64


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    src, lib = d / "p.cpp", d / "p.so"
    src.write_text('#include "vr_walk_pieces.h"\n'
                   'extern "C" unsigned long long pieces(uint32_t bw, uint32_t bh, uint32_t r, uint32_t p, uint32_t m) {\n'
                   '    const vr::WalkPieces w = vr::walk_pieces(bw, bh, r, p, m);\n'
                   '    return (unsigned long long)w.windowed << 32 | w.split;\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    f = C.CDLL(str(lib)).pieces
    f.restype = C.c_ulonglong
    f.argtypes = [C.c_uint32] * 5
    return lambda *a: ((r := f(*a)) & 0xFFFFFFFF, bool(r >> 32))


def test_pieces(pieces):
    boxes = [(0, 0), (1, 1), (2, 64), (63, 5), (64, 64), (65, 1), (127, 200), (256, 256), (4096, 4096), (20000, 3),
             (32766, 1), (32767, 32767), (32768, 32768), (1, 32768)]
    for bw, bh in boxes:
        for longest in (0, 1, 3, 4, 16, 24, 25, 30, 31, 32, 33, 64, 128):
            for parts, least in ((1, 1), (4, 2), (16, 4)):
                room = SIDE - 2 * longest
                split = least if room <= 0 else max(least, -(-bw // room), -(-bh // room))
                for moves in (1, 15, 16, 17, 63, 64, 796, 1023, 1024, 65535):
                    got, windowed = pieces(bw, bh, longest, parts, moves)
                    assert got == split, (bw, bh, longest, parts, moves)
                    assert windowed == (room > 0 and 16 * split * split <= moves), (bw, bh, longest, parts, moves)
                    if windowed:
                        assert max(-(-bw // split), -(-bh // split)) + 2 * longest <= SIDE
