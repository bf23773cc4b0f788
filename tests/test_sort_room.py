"""CPU: the scratch of the node sorts, sized for 2n nodes before their number is
known, holds a sort of every smaller count (the size of a sort's tiles changes
at 2^18 elements, so the words of a count do not grow with it everywhere)."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def words():
    import paper_2602_05804_amd as P

    out = []
    for name in ("sort_words", "sort_room"):
        f = getattr(P.lib(), f"_ZN4sfmm{len(name)}{name}Eli")  # sfmm::name(int64_t, int)
        f.restype, f.argtypes = C.c_size_t, [C.c_int64, C.c_int]
        out.append(f)
    return out


@pytest.mark.parametrize("passes", [1, 3])
def test_room_covers_every_smaller_count(words, passes):
    need, room = words
    most = 0  # the words of the most demanding count so far
    for k in range(1, 1 << 20):
        most = max(most, need(k, passes))
        assert room(k, passes) >= most, k
    assert room((1 << 20) + 4096, passes) == need((1 << 20) + 4096, passes)  # and no more than that
