"""The decode split rule on the host: a call never takes more partials than the
memory sized for it holds, and never fewer splits than that size stands for."""
import itertools

import pytest

from paper_2608_04771_amd import binding as B


@pytest.mark.parametrize("cus", [1, 32, 64, 256, 304])
@pytest.mark.parametrize("dim", [64, 128])
def test_partials_fit_and_splits_stay_in_range(cus, dim):
    lib = B.load_library()
    base_of = lib._ZN4reco13decode_splitsEiii
    call_of = lib._ZN4reco18decode_call_splitsEiiiiii
    caps = [1, 31, 255, 256, 4095, 5120, 9709, 10240, 16640, 32832, 65600, 1 << 20]
    units = sorted({1, 2, 3, 4, 7, 16, 31, 32, 96, 112, 127, 128, 129, 200, 255, 256, 257, 512, 65535, cus, cus + 1})
    for u, cap, group in itertools.product(units, caps, range(1, 17)):
        base = base_of(u, cap, cus)
        s = call_of(base, u, cap, group, dim, cus)
        assert base <= s <= 128, (u, cap, group)
        # group x D outputs and 2 x group statistics a split, in the room of 16 x D + 32 a sized split
        assert s * group * (dim + 2) <= base * (16 * dim + 32), (u, cap, group)
        if base == 1:                # one kernel, whatever the capacity: more splits would add a merge launch
            assert s == 1, (u, cap, group)
        if s > base:
            assert u * s <= 2 * cus and (cap + 32) // 32 >= 64 * s and 2 * u * s >= 3 * cus, (u, cap, group)
