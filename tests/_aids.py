"""Test aids of a handle (gabp_set_test_aid): conditions that a program cannot bring about at will."""
import ctypes

from paper_0811_2518_amd import binding

SPREAD_TEAMS = 0  # nonzero: a batch's teams take their members from different XCDs
WAIT_LIMIT = 1    # nonzero: limit of the resident solve's waits, in clock ticks plus one
ROLL_LIMIT = 2    # nonzero: limit of the roll calls, in clock ticks plus one (one: they fail at once)
ABORTED = 3       # counts the launches that found no place on the chip
LARGEST_TEAM = 4  # workgroups of the largest team of the last batched solve


def get_aid(solver, which):
    f = binding.lib().gabp_get_test_aid
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int32], ctypes.c_int64
    return f(solver._h, which)


def set_aid(solver, which, value):
    f = binding.lib().gabp_set_test_aid
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64], ctypes.c_int32
    assert f(solver._h, which, value) == binding.OK
