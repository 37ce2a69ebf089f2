"""The argument structs that the binding packs in one call hold the same bytes as the ctypes structures (no GPU)."""
import ctypes

import pytest

from paper_2602_08810_amd import api


@pytest.mark.parametrize("cls,pack", [(api.FwdArgs, api._pack_fwd), (api.BwdArgs, api._pack_bwd), (api.StepArgs, api._pack_step)])
def test_packed_struct_has_the_bytes_of_the_ctypes_one(cls, pack):
    signed = (ctypes.c_int32, ctypes.c_int64)
    values = [-(i + 3) if t in signed and i % 2 else (i + 3) * 0x01010101 % (1 << 31) for i, (_, t) in enumerate(cls._fields_)]
    a = cls()
    for (name, _), v in zip(cls._fields_, values):
        setattr(a, name, v)
    assert pack(*values) == bytes(a)


@pytest.mark.parametrize("v,want", [("zoh", 1), (2, 2), (-1, -1), (1 << 32, 0), ((1 << 31) + 1, -(1 << 31) + 1), (True, 1)])
def test_mode_numbers_become_32_bits(v, want):
    a = api.FwdArgs()
    a.disc = api.DISC[v] if isinstance(v, str) else int(v)
    assert api._code(v, api.DISC) == want == a.disc


def test_unknown_mode_name_is_refused():
    with pytest.raises(KeyError):
        api._code("nearest", api.DISC)
